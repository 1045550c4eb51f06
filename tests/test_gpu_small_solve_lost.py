"""A one-launch solve whose blocks give up waiting for each other (forced with a limit of one poll;
every block still ends by itself) goes on in the separate launches: the same bits, iterations and
hop counts as a solve that took them from the start, and the context stays with them."""
import pytest
import torch

from paper_1811_00893_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dims,nrhs,precision,x0", [
    ((8, 8, 8, 8), 1, 0, False), ((8, 8, 8, 8), 3, 0, True), ((4, 6, 8, 10), 2, 1, False), ((6, 6, 10, 12), 2, 0, False)])
def test_blocks_that_give_up(dims, nrhs, precision, x0, monkeypatch):
    from paper_1811_00893_amd import _lib as L
    U = inputs.gauge_field(dims, eps=0.3, seed=4500).to(DEV)
    b = inputs.gaussian_source(dims, seed=4501, nrhs=nrhs).to(DEV)
    guess = inputs.gaussian_source(dims, seed=4502, nrhs=nrhs).to(DEV)
    if nrhs > 1:
        b[1] = 0
    opts = {"precision": precision, "use_x0": x0}

    def solve(ctx, g):
        x = guess.clone() if x0 else torch.zeros_like(b)
        st, info = L.wilson_solve_ex(ctx, g, x, b, nrhs, 0.12, 1e-10, opts)
        torch.cuda.synchronize()
        assert st == 0, L.wilson_last_error()
        return x, [i["iterations"] for i in info], info[0]["hop_launches"]

    out = {}
    for polls in ("0", "1", "2097152"):
        monkeypatch.setenv("WILSON_ONE_LAUNCH", polls)
        ctx = L.wilson_context_create()
        g = L.wilson_gauge_load(ctx, U, dims, L.WILSON_GAUGE_FP32)
        try:
            out[polls] = [solve(ctx, g)]
            monkeypatch.delenv("WILSON_ONE_LAUNCH")
            out[polls].append(solve(ctx, g))  # the same context without the limit
        finally:
            L.wilson_gauge_free(ctx, g)
            L.wilson_context_destroy(ctx)
    ref = out["0"][0]
    for polls, runs in out.items():
        for x, iters, _ in runs:
            assert torch.equal(x, ref[0]) and iters == ref[1]
    # (the separate launches also enqueue the masked iterations that the one launch leaves out)
    assert out["0"][1][2] < ref[2] and out["2097152"][0][2] < ref[2]
    again = 2 if x0 else 0  # (a start from a guess forms its first residual with two hops)
    assert [r[2] for r in out["1"]] == [ref[2] + again, ref[2]]
