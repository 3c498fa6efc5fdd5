"""The gradient and the image from a copy of the checkpoints at any address:
the same bits as from the buffer fd_run_shot wrote, which is 256-byte aligned
(the step kernels load 16 bytes at a time, so such a copy is restored into the
work buffer before it is read)."""
from __future__ import annotations

import pytest

import fd_inputs as fi

pytestmark = pytest.mark.gpu


def _problem(ndim, nz, ny, nx, nt, seed):
    return fi.Problem(name="addr", ndim=ndim, nz=nz, ny=ny, nx=nx, dh=10.0, dt=1e-3, nt=nt,
                      src=(nz // 3, ny // 2, nx // 2), receivers=fi.Receivers(1, 0, 0, 1, 1, nx, 1, 1, 1),
                      f0=30.0, sponge_width=3, sponge_faces=0x3E, velocity_kind="random", velocity_seed=seed)


def _moved(ck, offset):
    import torch
    big = torch.empty(ck.numel() + 256, dtype=torch.uint8, device="cuda")
    out = big[offset:offset + ck.numel()]
    out.copy_(ck.view(torch.uint8))
    assert out.data_ptr() % 256 == offset
    return out


# every: segments of one launch and of several, of one and two steps, and a
# shorter last one; offsets: less than a float, a float, half a vector
@pytest.mark.parametrize("offset", [1, 4, 8])
@pytest.mark.parametrize("ndim,nz,ny,nx,nt,every", [
    (2, 70, 1, 150, 9, 1), (2, 70, 1, 150, 9, 2), (2, 70, 1, 150, 23, 5), (2, 70, 1, 150, 47, 45),
    (3, 18, 20, 70, 9, 1), (3, 18, 20, 70, 9, 4)])
def test_checkpoints_at_any_address(ndim, nz, ny, nx, nt, every, offset):
    import torch
    from helpers import setup
    p = _problem(ndim, nz, ny, nx, nt, seed=offset)
    model, state, shot = setup(p)
    ck = model.checkpoint_buffer(nt, every)
    tr = model.run_shot(state, shot, ckpt=ck, ckpt_every=every)
    sums = []
    for c in (ck, _moved(ck, offset)):
        grad = torch.zeros(p.ncells, dtype=torch.float64, device="cuda")
        img = torch.zeros_like(grad)
        # two shots of one call, one of them always at the library's address
        model.adjoint_gradient_shots([shot, shot], [tr, tr], [c, ck], every, grad)
        model.rtm_image_shots([shot, shot], [tr, tr], [c, ck], every, img)
        sums.append((grad, img))
    assert torch.equal(sums[0][0], sums[1][0]) and torch.equal(sums[0][1], sums[1][1])
    assert float(sums[0][0].abs().max()) > 0 and float(sums[0][1].abs().max()) > 0
