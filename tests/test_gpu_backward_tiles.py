"""The backward pass on grids of every tile shape and kernel, bit for bit.

2D: surveys whose recompute and adjoint launches take each tile shape, several
rounds of tiles, several shots per launch and several groups of shots, against
one shot per call with a checkpoint at every step (launches of one step).
3D: the same shot on a grid and on one that quiet cells lengthen until another
kernel takes its steps; the sums agree wherever the wave has been."""
from __future__ import annotations

import pytest

import fd_inputs as fi

pytestmark = pytest.mark.gpu


# (shots, nz, nx, nt, every): shapes of the launches (rounds of tiles)
SURVEYS = [
    (2, 499, 500, 17, 17),      # 64 x 64 (2) and 96 x 96 (1)
    (3, 401, 531, 17, 9),       # 96 x 96 and 128 x 96 (1)
    (5, 601, 997, 13, 13),      # 64 x 64 (5, 6: one and two steps), 128 x 96 and 128 x 128 (2)
    (2, 999, 2001, 13, 13),     # 96 x 96 (4), 128 x 128 (2)
    (8, 1023, 1023, 17, 17),    # 96 x 96 (6), 128 x 96 (5), 128 x 128 (4)
    (7, 1447, 1449, 9, 9),      # 14.9 M cells: groups of 3 and 4 shots
    (1, 2000, 2000, 11, 5),     # lone adjoint steps split off, launches of several after them
    (2, 700, 1200, 7, 2),       # two steps a segment, a lone one in the first
    (17, 901, 1025, 7, 4),      # more shots than a launch holds, groups of fewer
]


@pytest.mark.parametrize("count,nz,nx,nt,every", SURVEYS)
def test_survey_equals_single_shots_in_single_steps(count, nz, nx, nt, every):
    import torch
    import paper_2311_05038_amd as fd
    from helpers import grid_of
    p = fi.Problem(name="survey", ndim=2, nz=nz, ny=1, nx=nx, dh=10.0, dt=1e-3, nt=nt, src=(1, 0, 1),
                   receivers=fi.Receivers(1, 0, 1, nz // 8, 1, nx // 2, 8, 1, 2), f0=30.0, sponge_width=6,
                   sponge_faces=0x3F, velocity_kind="random", velocity_seed=nz)
    g = torch.Generator(device="cuda")
    g.manual_seed(nx)
    model = fd.Model(grid_of(p), torch.from_numpy(p.velocity().ravel()).cuda())
    rec = fd.Receivers(1, 0, 1, nz // 8, 1, nx // 2, 8, 1, 2)
    w = torch.from_numpy(p.wavelet()).cuda()
    # sources from the first corner to the last
    shots = [fd.Shot(((nz - 1) * i // max(1, count - 1), 0, (nx - 1) * i // max(1, count - 1)), w, rec)
             for i in range(count)]
    # residuals everywhere, so that the adjoint field fills the grid's tiles
    adj = [torch.randn((nt, rec.count), generator=g, device="cuda") for _ in shots]
    # every checkpoint of the reference is set to fields that are not quiet
    # anywhere, and the survey's are the levels of the same recursion
    levels = [torch.randn((2, nz, nx), generator=g, device="cuda") for _ in shots]
    px = (nx + 63) // 64 * 64

    def slot(ck, k):
        return ck.view(torch.float32)[k * 2 * nz * px:(k + 1) * 2 * nz * px].view(2, nz, px)

    out = {}
    for name in ("survey", "single"):
        sums = [torch.zeros(p.ncells, dtype=torch.float64, device="cuda") for _ in range(2)]
        step = every if name == "survey" else 1
        cks = []
        for sh, lv in zip(shots, levels):
            ck = model.checkpoint_buffer(nt, step)
            ck.zero_()
            st = model.new_state()
            st.begin(sh)
            for which in (0, 1):
                st.set_wavefield(which, lv[which])
            for n in range(nt):
                if n % step == 0:
                    for which in (0, 1):
                        slot(ck, n // step)[which, :, :nx] = st.wavefield(which)
                st.step(sh, n)
            cks.append(ck)
            if name == "single":
                model.adjoint_gradient(sh, adj[len(cks) - 1], ck, 1, sums[0])
                model.rtm_image(sh, adj[len(cks) - 1], ck, 1, sums[1])
                cks[-1] = None
        if name == "survey":
            model.adjoint_gradient_shots(shots, adj, cks, every, sums[0])
            model.rtm_image_shots(shots, adj, cks, every, sums[1])
        out[name] = sums
    for a, b in zip(out["survey"], out["single"]):
        assert torch.isfinite(a).all() and float((a != 0).double().mean()) > 0.5
        assert torch.equal(a, b)


# a grid and the planes that lengthen it: the kernels of the adjoint step
PAIRS_3D = [
    (60, 120, 152, 700),     # short, 2 planes a block -> 4 planes (16 M padded cells)
    (60, 120, 152, 1100),    # -> accesses that bypass the caches (25 M)
    (100, 3, 200, 1000),     # 400 blocks of the short kernel -> streaming, 128-wide tiles
    (60, 6, 2048, 6000),     # -> streaming, 256-wide tiles (74 M)
    (60, 37, 300, 1500),     # short -> streaming (37 of 48 rows)
]


@pytest.mark.parametrize("nz,ny,nx,longer", PAIRS_3D)
def test_3d_kernels_agree_on_the_backward_pass(nz, ny, nx, longer):
    import torch
    import paper_2311_05038_amd as fd
    nt, every = 8, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(nx)
    adj = torch.randn((nt, 5 * ny * (nx // 3)), generator=g, device="cuda")
    w = torch.randn(nt, generator=g, device="cuda")
    out = []
    for planes in (nz, longer):
        grid = fd.Grid(ndim=3, nz=planes, ny=ny, nx=nx, dh=10.0, dt=1e-3, sponge_width=0)
        v = torch.full((grid.ncells,), 2500.0, device="cuda")
        model = fd.Model(grid, v)
        shot = fd.Shot((2, ny // 2, nx // 2), w, fd.Receivers(0, 0, 0, 5, ny, nx // 3, 1, 1, 3))
        ck = model.checkpoint_buffer(nt, every)
        tr = model.run_shot(model.new_state(), shot, ckpt=ck, ckpt_every=every)
        sums = [torch.zeros(grid.ncells, dtype=torch.float64, device="cuda") for _ in range(2)]
        model.adjoint_gradient(shot, adj, ck, every, sums[0])
        model.rtm_image(shot, adj, ck, every, sums[1])
        # 8 steps from planes 0 to 4 reach plane 36
        out.append([tr] + [s.view(planes, -1)[:37].clone() for s in sums])
        assert all(float(s.view(planes, -1)[41:].abs().max()) == 0 for s in sums)
        del sums, ck, model, v
    for a, b in zip(*out):
        assert float(a.abs().max()) > 0
        assert torch.equal(a, b)
