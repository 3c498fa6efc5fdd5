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
