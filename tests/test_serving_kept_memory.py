"""Serving on a simulated device whose library keeps the memory of released
hierarchies: evictions stop as soon as one has made room."""

import threading

from paper_2006_16147_amd.serve import Request, Server


class KeepingBackend:
    """A device of `total` bytes; released hierarchies' bytes stay taken until
    release_freed()."""

    def __init__(self, total, bytes_per_dof=100):
        self.total, self.bpd = total, bytes_per_dof
        self.lock = threading.Lock()
        self.live, self.kept, self.peak = {}, 0, 0

    def make_slot(self, i):
        return {}

    def estimate_bytes(self, req):
        return self.bpd * req.N ** 3

    def solve_bytes(self, req):
        return 0

    def device_free_bytes(self):
        with self.lock:
            return self.total - sum(self.live.values()) - self.kept

    def release_freed(self):
        with self.lock:
            self.kept = 0

    def build(self, req, slot):
        with self.lock:
            self.live[req.op_id] = self.bpd * req.N ** 3
            self.peak = max(self.peak, sum(self.live.values()) + self.kept)
        return req.op_id, self.bpd * req.N ** 3

    def solve(self, handle, req, slot):
        return {"status": 0, "iterations": 1, "converged": True, "rel_res_true": 0.0}

    def release(self, handle):
        with self.lock:
            self.kept += self.live.pop(handle)


def test_one_eviction_for_one_hierarchy():
    one = 100 * 10 ** 3
    be = KeepingBackend(total=4 * one)
    srv = Server(be, slots=1, budget_bytes=10 ** 12, margin_bytes=0)
    # four operators fill the device; the fifth and sixth need the room of one each
    res = srv.run([Request(i, 0.001 * i, i, 10) for i in range(6)])
    assert all(r.status == 0 for r in res)
    assert srv.stats["evictions"] == 2 and sorted(srv.cache) == [2, 3, 4, 5]
    assert be.peak <= be.total
    srv.close()


def test_kept_memory_alone_evicts_nothing():
    one = 100 * 10 ** 3
    be = KeepingBackend(total=4 * one)
    be.kept = 2 * one  # left by hierarchies of another program part
    srv = Server(be, slots=1, budget_bytes=10 ** 12, margin_bytes=0)
    srv.run([Request(i, 0.001 * i, i, 10) for i in range(4)])
    assert srv.stats["evictions"] == 0 and sorted(srv.cache) == [0, 1, 2, 3]
    srv.close()
