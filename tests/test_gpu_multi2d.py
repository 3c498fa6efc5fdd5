"""Launches of several 2D steps against single steps, bit for bit: whole shots
(fd_run_shot, fd_step_batch) take several steps per launch on tiles with a
halo, fd_step takes one.  Grids at the edges of the tiles (inner tiles of 16
to 112 cells on 64, 96 and 128-cell tiles), one-cell axes and grids that need
several rounds of blocks; step counts that end a run on every remainder."""
from __future__ import annotations

import numpy as np
import pytest

import fd_inputs as fi

pytestmark = pytest.mark.gpu


def _problem(nz, nx, nt, seed, stride=1):
    rng = np.random.default_rng(seed)
    return fi.Problem(name="multi", ndim=2, nz=nz, ny=1, nx=nx, dh=10.0, dt=1e-3, nt=nt,
                      src=(int(rng.integers(nz)), 0, int(rng.integers(nx))),
                      receivers=fi.Receivers(nz // 2, 0, 0, 1 + (nz - 1 - nz // 2) // 3, 1,
                                             1 + (nx - 1) // stride, 3, 1, stride),
                      f0=30.0, sponge_width=min(5, nz // 4, nx // 4), sponge_faces=0x3F,
                      velocity_kind="random", velocity_seed=seed)


def _start(p, seed):
    """Model, shot and a state whose levels hold seeded values everywhere."""
    import torch
    from helpers import setup
    model, state, shot = setup(p)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    levels = [torch.randn((p.nz, p.nx), generator=g, device="cuda") for _ in range(2)]
    state.begin(shot)
    for w, v in enumerate(levels):
        state.set_wavefield(w, v)
    return model, state, shot, levels


def _by_single_steps(model, shot, levels, p):
    import torch
    st = model.new_state()
    st.begin(shot)
    for w, v in enumerate(levels):
        st.set_wavefield(w, v)
    tr = torch.full((shot.nt, shot.nrec), float("nan"), device="cuda")
    for n in range(shot.nt):
        st.step(shot, n, tr[n])
    return tr, st.wavefield(0), st.wavefield(1)


SHAPES = [(1, 1, 9), (1, 300, 12), (300, 1, 13), (16, 16, 12), (17, 65, 11), (31, 64, 7),
          (64, 63, 8), (65, 129, 25), (97, 193, 16), (128, 128, 6), (255, 257, 23),
          (333, 511, 10), (700, 901, 17), (1100, 2113, 11), (2049, 1500, 9), (5, 9001, 14),
          (9001, 5, 14)]


@pytest.mark.parametrize("nz,nx,nt", SHAPES)
def test_several_steps_per_launch_equal_single_steps(nz, nx, nt):
    import torch
    import paper_2311_05038_amd as fd
    p = _problem(nz, nx, nt, seed=nz + 7 * nx, stride=1 + nx % 3)
    model, state, shot, levels = _start(p, 11)
    ref = _by_single_steps(model, shot, levels, p)
    tr = torch.full((nt, shot.nrec), float("nan"), device="cuda")
    # chunks of every length up to the shot's, on one state
    done, k = 0, nt
    while done < nt:
        fd.step_batch([(model, state, shot, tr)], k)
        done += k
        k = min(nt - done, max(1, k // 2))
    assert torch.equal(tr, ref[0])
    assert torch.equal(state.wavefield(0), ref[1]) and torch.equal(state.wavefield(1), ref[2])
    # a whole shot, which starts at rest
    tr2 = model.run_shot(state, shot)
    st = model.new_state()
    st.begin(shot)
    row = torch.empty_like(tr2)
    for n in range(nt):
        st.step(shot, n, row[n])
    assert torch.equal(tr2, row)
    assert torch.equal(state.wavefield(0), st.wavefield(0)) and torch.equal(state.wavefield(1), st.wavefield(1))


def test_a_batch_whose_shots_end_at_different_steps():
    import torch
    import paper_2311_05038_amd as fd
    flights, refs = [], []
    for i, (nz, nx) in enumerate([(40, 70), (130, 90), (64, 256), (1, 33), (200, 201), (513, 97), (77, 1000)]):
        p = _problem(nz, nx, 3 + 4 * i, seed=50 + i)
        model, state, shot, levels = _start(p, 20 + i)
        refs.append(_by_single_steps(model, shot, levels, p))
        flights.append((model, state, shot, torch.full((shot.nt, shot.nrec), float("nan"), device="cuda")))
    while any(f[1].next < f[2].nt for f in flights):
        fd.step_batch(flights, 13)
    for f, ref in zip(flights, refs):
        assert torch.equal(f[3], ref[0])
        assert torch.equal(f[1].wavefield(0), ref[1]) and torch.equal(f[1].wavefield(1), ref[2])


@pytest.mark.parametrize("grids", [
    [(2048, 4095), (2047, 4096)],                                   # one group each
    [(1447, 1449)] * 7,                                             # groups of several
    [(2048, 4095)] * 2 + [(33, 70)] + [(2047, 4096)] * 2,           # together
    [(600, 500), (3001, 3002), (40, 50), (1700, 3100), (2, 2)],     # uneven shares
])
def test_shots_beyond_the_infinity_cache(grids):
    import torch
    import paper_2311_05038_amd as fd
    flights, refs = [], []
    for i, (nz, nx) in enumerate(grids):
        p = _problem(nz, nx, 11 + 2 * (i % 3), seed=80 + i)
        model, state, shot, levels = _start(p, 30 + i)
        refs.append(_by_single_steps(model, shot, levels, p))
        flights.append((model, state, shot, torch.full((shot.nt, shot.nrec), float("nan"), device="cuda")))
    while any(f[1].next < f[2].nt for f in flights):
        fd.step_batch(flights, 9)
    for f, ref in zip(flights, refs):
        assert torch.equal(f[3], ref[0])
        assert torch.equal(f[1].wavefield(0), ref[1]) and torch.equal(f[1].wavefield(1), ref[2])


def test_a_state_buffer_of_two_levels_is_enough():
    """A buffer without the second pair of levels is accepted, as it was, and
    gives the same bits by single steps; one byte less than that is refused."""
    import torch
    import paper_2311_05038_amd as fd
    from paper_2311_05038_amd import _abi
    p = _problem(70, 140, 21, seed=3)
    model, state, shot, levels = _start(p, 5)
    ref = model.run_shot(state, shot)
    field = 70 * 192 * 4
    meta = -(-((16 + 4 * 64) * 4) // 256) * 256
    least = 2 * field + meta
    assert model.sizes.state == least + 2 * field
    buf = torch.empty(least, dtype=torch.uint8, device="cuda")
    h = _abi.fd_create_state(model.handle, buf.data_ptr(), least)
    tr = torch.empty_like(ref)
    _abi.fd_run_shot(model.handle, h, shot._c, tr.data_ptr(), None, 0, 0,
                     torch.cuda.current_stream().cuda_stream)
    out = torch.empty((p.nz, p.nx), device="cuda")
    _abi.fd_get_wavefield(h, 0, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert torch.equal(tr, ref) and torch.equal(out, state.wavefield(0))
    _abi.fd_destroy_state(h)
    with pytest.raises(fd.FDError) as e:
        _abi.fd_create_state(model.handle, buf.data_ptr(), least - 1)
    assert e.value.status == _abi.FD_ERR_INVALID_ARG


@pytest.mark.parametrize("every", [1, 2, 3, 5, 7, 8, 13, 29])
def test_gradient_and_image_do_not_depend_on_the_checkpoint_interval(every):
    """Segments of every length cut the recompute and the adjoint recursion
    into other launches; the sums are the same bits as with one segment, and
    the checkpoints hold the levels of single steps."""
    import torch
    from helpers import setup
    p = _problem(83, 150, 29, seed=9)
    model, state, shot = setup(p)
    out = {}
    for k in (every, 40):
        ck = model.checkpoint_buffer(p.nt, k)
        tr = model.run_shot(state, shot, ckpt=ck, ckpt_every=k)
        grad = torch.zeros(p.ncells, dtype=torch.float64, device="cuda")
        img = torch.zeros_like(grad)
        model.adjoint_gradient(shot, tr, ck, k, grad)
        model.rtm_image(shot, tr, ck, k, img)
        out[k] = (grad, img, ck)
    assert torch.equal(out[every][0], out[40][0]) and torch.equal(out[every][1], out[40][1])
    assert float(out[every][0].abs().max()) > 0
    px, slot = 192, 2 * 83 * 192
    ck = out[every][2].view(torch.float32)
    st = model.new_state()
    st.begin(shot)
    for n in range(p.nt):
        if n % every == 0:
            for w in (0, 1):
                lv = ck[n // every * slot + w * slot // 2:][:83 * px].view(83, px)
                assert torch.equal(lv[:, :p.nx], st.wavefield(w)) and not lv[:, p.nx:].any()
        st.step(shot, n)
