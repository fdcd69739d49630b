"""The scheduler's march scratch (CPU, fake backend and clock): batches are
admitted by the least scratch that their marches take, and get the larger one,
with room for the grid's faster copy, where it costs no other batch its place."""
import pytest

from paper_2604_03748_amd.serve import Backend, Request, Scheduler
from tests.test_serve_scheduler import FakeBackend, FakeClock, Inst

LEAST, WANTED = 1000, 5000


class ScratchBackend(FakeBackend):
    def __init__(self, clock, n_streams=2):
        super().__init__(clock, n_streams)
        self.granted, self.most = [], 0

    def batch_bytes(self, reqs, instances):
        return LEAST

    def batch_bytes_wanted(self, reqs, instances):
        return WANTED

    def launch(self, slot, reqs, instances, keep_ids=(), march_bytes=None):
        self.granted.append(march_bytes)
        h = super().launch(slot, reqs, instances, keep_ids)
        self.most = max(self.most, len(self.busy))
        return h


def _run(budget, n_streams):
    clock = FakeClock()
    be = ScratchBackend(clock, n_streams)
    sch = Scheduler(be, {0: Inst(10)}, budget, max_batch=1, clock=clock)
    st = sch.run([Request(k, 0, k, 0.0) for k in range(12)])
    assert sch.peak_in_use <= budget and sch.in_use == 0
    return st, be


def test_backend_charges_the_least_scratch():
    class Ctx:
        def march_workspace_bytes(self, *a, bricks=None, least=False):
            return LEAST if least else WANTED

    class One:
        density = bricks = None
        sigma_scale, step_voxels, seed = 8.0, 4.0, 0

        def camera(self, frame):
            return None

    be = Backend.__new__(Backend)
    be.ctx = Ctx()
    reqs = [Request(0, 0, 0, 0.0)]
    assert be.batch_bytes(reqs, {0: One()}) == LEAST
    assert be.batch_bytes_wanted(reqs, {0: One()}) == WANTED


@pytest.mark.parametrize("n_streams", [1, 3])
def test_budget_between_the_sizes_serves_every_request(n_streams):
    # a request is 100 bytes: room for one batch on the least scratch, not on the wanted one
    st, be = _run(LEAST + 150, n_streams)
    assert st["requests"] == 12 and st["rejected"] == 0 and set(be.granted) == {LEAST}


def test_the_larger_scratch_takes_no_batch_its_place():
    st, be = _run(WANTED + 2 * LEAST + 300, 3)
    assert st["requests"] == 12 and be.most == 3
    assert be.granted.count(WANTED) >= 1 and LEAST in be.granted


def test_a_lone_batch_gets_the_larger_scratch():
    # nothing waits, so the free slots keep no room
    clock = FakeClock()
    be = ScratchBackend(clock, 3)
    sch = Scheduler(be, {0: Inst(10)}, WANTED + 200, max_batch=1, clock=clock)
    st = sch.run([Request(k, 0, k, 0.01 * k) for k in range(4)])
    assert st["requests"] == 4 and be.granted == [WANTED] * 4


def test_ample_budget_grants_the_larger_scratch():
    st, be = _run(10**6, 3)
    assert st["requests"] == 12 and set(be.granted) == {WANTED}
