"""One-launch solves of several contexts, each on its own stream and thread: the same bits as alone,
also where the blocks of all of them exceed the device (some then take the separate launches), and
side by side rather than one after another."""
import threading
import time

import pytest
import torch

from paper_1811_00893_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


class Worker:
    def __init__(self, L, U, dims, seed, precision=0):
        self.L, self.opts = L, {"precision": precision}
        self.stream = torch.cuda.Stream()
        self.b = inputs.gaussian_source(dims, seed=seed, nrhs=1).to(DEV)
        self.x = torch.zeros_like(self.b)
        torch.cuda.synchronize()
        self.ctx = L.wilson_context_create(self.stream)
        self.g = L.wilson_gauge_load(self.ctx, U, dims, L.WILSON_GAUGE_FP32)

    def solve(self, n=1):
        for _ in range(n):
            st, self.info = self.L.wilson_solve_ex(self.ctx, self.g, self.x, self.b, 1, 0.12, 1e-10, self.opts)
            assert st == 0, self.L.wilson_last_error()
        return self.x.clone()

    def close(self):
        self.L.wilson_gauge_free(self.ctx, self.g)
        self.L.wilson_context_destroy(self.ctx)


def together(workers, n, each=None):
    """Every worker solves n times in a thread of its own; seconds for all."""
    bar, failed = threading.Barrier(len(workers) + 1), []

    def run(k):
        try:
            bar.wait()
            for _ in range(n):
                workers[k].solve()
                if each:
                    each(k)
        except Exception as e:  # noqa: BLE001
            failed.append(e)
    ts = [threading.Thread(target=run, args=(k,)) for k in range(len(workers))]
    for t in ts:
        t.start()
    bar.wait()
    t0 = time.perf_counter()
    for t in ts:
        t.join()
    assert not failed, failed
    return time.perf_counter() - t0


# 6 x 32 blocks fit the device, 6 x 60 (a ragged last tile) and 4 x 128 do not
@pytest.mark.parametrize("dims,nctx,precision", [((8, 8, 8, 8), 6, 0), ((8, 8, 8, 8), 6, 1), ((6, 10, 8, 16), 6, 0),
                                                 ((8, 8, 16, 16), 4, 0)])
def test_contexts_at_once_give_the_bits_of_one(dims, nctx, precision):
    from paper_1811_00893_amd import _lib as L
    U = inputs.gauge_field(dims, eps=0.3, seed=4600).to(DEV)
    workers = [Worker(L, U, dims, 4601 + k, precision) for k in range(nctx)]
    try:
        alone = [w.solve() for w in workers]
        torch.cuda.synchronize()

        def same(k):
            assert torch.equal(workers[k].x, alone[k])
        together(workers, 5, same)
    finally:
        for w in workers:
            w.close()


def test_contexts_run_side_by_side():
    """Four contexts at 8^4 take 0.26 of the time of their solves one after another (0.81 when their
    launches exclude each other); 0.6 leaves room for a busy host."""
    from paper_1811_00893_amd import _lib as L
    dims = (8, 8, 8, 8)
    U = inputs.gauge_field(dims, eps=0.3, seed=4610).to(DEV)
    workers = [Worker(L, U, dims, 4611 + k) for k in range(4)]
    try:
        for w in workers:
            w.solve(3)
        one = min(together(workers[:1], 20) for _ in range(3))
        four = min(together(workers, 20) for _ in range(3))
        print(f"one context {one / 20 * 1e6:.0f} us per solve, four {four / 80 * 1e6:.0f}")
        assert four < 0.6 * 4 * one
    finally:
        for w in workers:
            w.close()
