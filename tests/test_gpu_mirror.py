"""A grid turned about both axes gives the turned wavefield, bit for bit (the
second differences add the cells at +k and -k in a pair, and a sum of two does
not depend on their order): the last, partial tiles of a grid and its padding
against the first ones.  Levels, velocities and the source are not quiet or
symmetric anywhere."""
from __future__ import annotations

import pytest

import fd_inputs as fi

pytestmark = pytest.mark.gpu

# 1, 2 and 4 rows a thread and the streaming kernel with 16-bit fields (by
# blocks of 128 columns); one-cell axes, half-empty last tiles, odd sizes
SHAPES = [(1, 1), (40, 300), (203, 515), (799, 1101), (1201, 1747), (1501, 3001), (2047, 4033), (2500, 4095),
          (1, 70001), (30001, 33), (17, 20001)]


@pytest.mark.parametrize("storage,c_storage", [(0, 0), (1, 0), (2, 0), (1, 1), (2, 1)])
@pytest.mark.parametrize("nz,nx", SHAPES)
def test_2d_steps_of_the_turned_grid(storage, c_storage, nz, nx):
    import torch
    import paper_2311_05038_amd as fd
    nt = 3
    g = torch.Generator(device="cuda")
    g.manual_seed(nz + nx)
    grid = fd.Grid(ndim=2, nz=nz, ny=1, nx=nx, dh=10.0, dt=1e-3, sponge_width=min(5, nz // 4, nx // 4),
                   sponge_faces=0x3F, storage=storage, c_storage=c_storage)
    v = 1500.0 + 3000.0 * torch.rand((nz, nx), generator=g, device="cuda")
    levels = [torch.randn((nz, nx), generator=g, device="cuda") for _ in range(2)]
    w = torch.randn(nt, generator=g, device="cuda") * 1e6
    src = (nz - 1 - nz // 9, 0, nx - 1 - nx // 9)
    out = []
    for turned in (False, True):
        def turn(f):
            return f.flip(0, 1) if turned else f
        model = fd.Model(grid, turn(v).contiguous().ravel())
        s = (nz - 1 - src[0], 0, nx - 1 - src[2]) if turned else src
        shot = fd.Shot(s, w, fd.Receivers(0, 0, 0, nz, 1, nx, 1, 1, 1))
        st = model.new_state()
        st.begin(shot)
        for which in (0, 1):
            st.set_wavefield(which, turn(levels[which]))
        tr = torch.full((nt, nz, nx), float("nan"), device="cuda")
        for n in range(nt):
            st.step(shot, n, tr[n].view(-1))
        out.append([turn(st.wavefield(which)) for which in (0, 1)] + [turn(t) for t in tr])
    for a, b in zip(*out):
        assert torch.isfinite(a).all() and float(a.abs().max()) > 0
        assert torch.equal(a, b)
