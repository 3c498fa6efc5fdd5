"""Shots that have ended take no part in a batch's plan: the launches are
those of the shots that still run.  (Launches are counted in a recorded
graph; nothing runs.)"""
from __future__ import annotations

import pytest

from test_gpu_state_levels import _flight, _launches

pytestmark = pytest.mark.gpu


def _ended(nz, nx):
    f = _flight(nz, nx, 3)
    f[0].run_shot(f[1], f[2])
    assert f[1].next == f[2].nt
    return f


@pytest.mark.parametrize("ended", [[(2048, 4096)], [(1500, 1500)] * 8, [(64, 64)] * 15])
@pytest.mark.parametrize("nz,nx", [(256, 256), (1024, 1024)])
def test_ended_shots_add_no_launches(ended, nz, nx):
    import paper_2311_05038_amd as fd
    lone = [_flight(nz, nx, 200)]
    alone = _launches(lambda s: fd.step_batch(lone, 50, stream=s))
    batch = [_ended(*e) for e in ended] + [_flight(nz, nx, 200)]
    assert _launches(lambda s: fd.step_batch(batch, 50, stream=s)) == alone


def test_the_rest_of_a_batch_is_planned_for_the_shots_that_run():
    """Large shots with a few steps left beside one with many: once they have
    ended, the small one takes the launches it would take alone."""
    import paper_2311_05038_amd as fd
    batch = [_flight(2048, 4096, 9), _flight(2047, 4095, 9), _flight(256, 256, 400)]
    together = _launches(lambda s: fd.step_batch(batch, 400, stream=s))
    first = [_flight(2048, 4096, 9), _flight(2047, 4095, 9), _flight(256, 256, 400)]
    n = _launches(lambda s: fd.step_batch(first, 9, stream=s))
    lone = [_flight(256, 256, 391)]
    rest = _launches(lambda s: fd.step_batch(lone, 391, stream=s))
    assert together <= n + rest + 4     # a pair of launches may straddle the end


def test_few_steps_beyond_the_cache_are_single_steps():
    """Launches of one or two steps move more bytes there than they save."""
    import torch
    from helpers import setup
    from test_gpu_state_levels import _problem
    model, state, shot = setup(_problem(3000, 5000, 3))
    tr = torch.empty((3, shot.nrec), device="cuda")
    # a clear, the source, three steps
    assert _launches(lambda s: model.run_shot(state, shot, tr, stream=s)) == 5


@pytest.mark.parametrize("nz,nx,count,copied", [(2000, 2000, 1, True), (1000, 1000, 1, True), (100, 100, 8, False)])
def test_an_image_with_a_checkpoint_at_every_step(nz, nx, count, copied):
    """The history is the checkpoints' P: a copy, unless many small shots share
    the launch that stores it."""
    import torch
    from helpers import setup
    from test_gpu_state_levels import _problem
    nt = 4
    model, state, shot = setup(_problem(nz, nx, nt))
    ck = model.checkpoint_buffer(nt, 1)
    tr = model.run_shot(state, shot, ckpt=ck, ckpt_every=1)
    need = model.sizes_for(nt, 1).adjoint_work
    works = [torch.empty(need, dtype=torch.uint8, device="cuda") for _ in range(count)]
    img = torch.zeros(nz * nx, dtype=torch.float64, device="cuda")

    def call(s):
        model.rtm_image_shots([shot] * count, [tr] * count, [ck] * count, 1, img, works=works, stream=s)
    assert _launches(call, copies=True) == (nt * count if copied else 0)
