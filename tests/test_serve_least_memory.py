"""The server's admission with a device that can start a request in less
memory than it would like to (`least_footprint`): a request is admitted where
that smaller size fits, and the budget counts what each shot holds."""
import pytest

from paper_2311_05038_amd.serve import Request, Scheduler
from test_serve_scheduler import FakeDevice


class TwoSizes(FakeDevice):
    """24 bytes a cell if it may, 16 if it must."""

    def __init__(self):
        super().__init__()
        self.least = {}

    def footprint(self, req):
        return 24 * req.nz * req.nx

    def least_footprint(self, req):
        return 16 * req.nz * req.nx

    def start(self, req, least=False):
        h = super().start(req)
        self.least[req.rid] = least
        if least:
            self.alloc -= 8 * req.nz * req.nx
        self.peak_alloc = max(self.peak_alloc, self.alloc)
        return h

    def finish(self, h):
        req = h["req"]
        self.alloc -= (16 if self.least[req.rid] else 24) * req.nz * req.nx
        return None


def test_a_request_between_the_two_sizes_runs():
    dev = TwoSizes()
    reqs = [Request(0, 0.0, 100, 100, 40), Request(1, 0.0, 80, 100, 40), Request(2, 0.0, 130, 100, 40)]
    out = Scheduler(dev, max_slots=4, hbm_budget=200_000).run(reqs)
    assert [out[i].status for i in (0, 1)] == ["ok", "ok"]
    assert out[2].status == "failed: footprint exceeds the HBM budget"
    assert dev.least == {0: True, 1: False} and dev.alloc == 0


@pytest.mark.parametrize("count", [1, 2, 3, 5, 6, 7])
def test_a_budget_holds_as_many_shots_as_at_the_smaller_size(count):
    dev = TwoSizes()
    reqs = [Request(i, 0.0, 100, 100, 40) for i in range(2 * count)]
    sch = Scheduler(dev, max_slots=64, hbm_budget=count * 160_000, chunk=10)
    out = sch.run(reqs)
    assert all(o.status == "ok" for o in out.values())
    # shots that fit whole hold 24 bytes a cell; the rest is filled at 16
    whole = count * 160_000 // 240_000
    assert sch.peak_slots >= whole + (count * 160_000 - whole * 240_000) // 160_000
    assert sch.peak_bytes <= count * 160_000 and dev.alloc == 0
