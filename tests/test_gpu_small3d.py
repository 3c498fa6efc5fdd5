"""The 3D FP32 kernel for small grids (64 x 16 cells of 2 or 4 planes per block,
every load at once) against the routine-per-kernel step and the host back-end's
order of operations, bit for bit, at the edges of its tiles and where the
choice of kernel changes; and the 2D single-step block kernel's tile edges."""
from __future__ import annotations

import numpy as np
import pytest

import fd_inputs as fi

pytestmark = pytest.mark.gpu


def _problem(ndim, nz, ny, nx, nt, seed):
    rng = np.random.default_rng(seed)
    r = fi.Receivers(nz // 2, ny // 3, 0, 1, 1 + (ny - 1 - ny // 3) // 2, 1 + (nx - 1) // 3, 1, 2, 3)
    return fi.Problem(name="small", ndim=ndim, nz=nz, ny=ny, nx=nx, dh=10.0, dt=1e-3, nt=nt,
                      src=(int(rng.integers(nz)), int(rng.integers(ny)), int(rng.integers(nx))),
                      receivers=r, f0=30.0, sponge_width=min(4, nz // 4, nx // 4), sponge_faces=0x3F,
                      velocity_kind="random", velocity_seed=seed)


SHAPES = [(3, 1, 1, 1), (3, 2, 15, 63), (3, 3, 16, 64), (3, 4, 17, 65), (3, 5, 33, 129), (3, 9, 1, 200),
          (3, 41, 40, 3), (3, 7, 31, 191), (3, 64, 48, 64), (3, 33, 250, 1500), (3, 150, 300, 300),
          (3, 90, 700, 300), (3, 30, 900, 1025), (2, 1, 1, 1), (2, 7, 1, 127), (2, 8, 1, 128), (2, 9, 1, 129),
          (2, 33, 1, 1000), (2, 1025, 1, 70)]


@pytest.mark.parametrize("ndim,nz,ny,nx", SHAPES)
def test_step_equals_the_routine_step(ndim, nz, ny, nx):
    """fd_step_routines evaluates every axis in a kernel of its own, with the
    same operations per cell."""
    import torch
    from helpers import setup
    p = _problem(ndim, nz, ny, nx, 4, seed=nz + ny + nx)
    model, a, shot = setup(p)
    b = model.new_state()
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    for st in (a, b):
        st.begin(shot)
    for w in (0, 1):
        v = torch.randn(p.ncells, generator=g, device="cuda")
        for st in (a, b):
            st.set_wavefield(w, v)
    work = torch.empty(model.sizes.routines_work, dtype=torch.uint8, device="cuda")
    rows = torch.full((2, p.nt, shot.nrec), float("nan"), device="cuda")
    for n in range(p.nt):
        a.step(shot, n, rows[0, n])
        b.step_routines(shot, n, work, rows[1, n])
    assert torch.equal(rows[0], rows[1])
    for w in (0, 1):
        assert torch.equal(a.wavefield(w), b.wavefield(w))


@pytest.mark.parametrize("nz,ny,nx", [(5, 17, 65), (18, 33, 70), (12, 16, 128), (40, 20, 193)])
def test_gradient_and_image_against_the_oracle(nz, ny, nx):
    """The recompute and adjoint modes of the kernel (FP32 against FP64 over
    14 steps: the repository's 1e-3 bound on gradients and images)."""
    import torch
    import oracle
    from helpers import rel_l2, setup
    p = _problem(3, nz, ny, nx, 14, seed=nx)
    model, state, shot = setup(p)
    v = p.velocity()
    ck = model.checkpoint_buffer(p.nt, 5)
    model.run_shot(state, shot, ckpt=ck, ckpt_every=5)
    g = torch.Generator(device="cuda")
    g.manual_seed(nz)
    d = torch.randn((p.nt, shot.nrec), generator=g, device="cuda")
    grad = torch.zeros(p.ncells, dtype=torch.float64, device="cuda")
    img = torch.zeros_like(grad)
    model.adjoint_gradient(shot, d, ck, 5, grad)
    model.rtm_image(shot, d, ck, 5, img)
    args = (oracle.grid_of(p), v, p.wavelet(), p.nt, p.src, p.rec_index(), d.cpu().numpy().astype(np.float64))
    gref, _ = oracle.adjoint(*args)
    iref = oracle.image(*args)
    assert rel_l2(grad.cpu().numpy(), np.ravel(gref)) <= 1e-3
    assert rel_l2(img.cpu().numpy(), np.ravel(iref)) <= 1e-3


@pytest.mark.parametrize("storage,c_storage", [(1, 0), (2, 0), (1, 1), (2, 1)])
@pytest.mark.parametrize("nz,nx", [(40, 300), (200, 515), (800, 1100), (1201, 1747), (1500, 3000)])
def test_16bit_2d_tiles_agree(storage, c_storage, nz, nx):
    """The 16-bit 2D step on grids that take 1, 2 and 4 rows per thread and
    the streaming kernel: a grid and the same grid padded with quiet cells far
    from the source give the same codes where the wave has been, whatever
    kernel each takes (9 steps reach 36 cells)."""
    import torch
    from helpers import setup
    p = _problem(2, nz, 1, nx, 9, seed=5).scaled(src=(3, 0, 150), sponge_width=0, velocity_kind="constant",
                                                 receivers=fi.Receivers(2, 0, 100, 1, 1, 100))
    q = p.scaled(nz=2600, nx=4000)
    out = []
    for r in (p, q):
        model, state, shot = setup(r, storage=storage, c_storage=c_storage)
        tr = model.run_shot(state, shot)
        out.append((tr, state.wavefield(0)[:40, 90:211].clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert float(out[0][1].abs().max()) > 0


@pytest.mark.parametrize("storage,c_storage", [(1, 0), (2, 0), (1, 1), (2, 1)])
@pytest.mark.parametrize("nz,ny,nx", [(39, 60, 63), (40, 81, 130), (41, 150, 200)])
def test_16bit_3d_tiles_agree(storage, c_storage, nz, ny, nx):
    """The same in 3D: 2 and 4 planes per block against the streaming kernel
    on the padded grid (8 steps reach 32 cells)."""
    import torch
    from helpers import setup
    p = _problem(3, nz, ny, nx, 8, seed=6).scaled(src=(3, 25, 30), sponge_width=0, velocity_kind="constant",
                                                  receivers=fi.Receivers(2, 10, 5, 1, 30, 50))
    q = p.scaled(nz=120, ny=200, nx=260)
    out = []
    for r in (p, q):
        model, state, shot = setup(r, storage=storage, c_storage=c_storage)
        tr = model.run_shot(state, shot)
        out.append((tr, state.wavefield(0)[:35, :57, :62].clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert float(out[0][1].abs().max()) > 0
