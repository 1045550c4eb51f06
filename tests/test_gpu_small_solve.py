"""BiCGStab in one cooperative launch (small lattices) against the separate launches it
replaces (WILSON_FUSE_FIN=0): the same sums in the same order, so the same bits, iteration
counts and status, at ragged tiles, one to 128 tiles, several right-hand sides (a zero one
among them), two-row and full links, and over more iterations than one launch takes; a solve
with more blocks than the device holds goes through the separate launches."""
import numpy as np
import pytest
import torch

import oracle
from paper_1811_00893_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def L():
    from paper_1811_00893_amd import _lib
    return _lib


def solves(L, monkeypatch, dims, U, b, kappa, tol, opts):
    out = []
    for fuse in ("0", "1"):
        monkeypatch.setenv("WILSON_FUSE_FIN", fuse)
        ctx = L.wilson_context_create()
        g = L.wilson_gauge_load(ctx, U.to(DEV), dims, L.WILSON_GAUGE_FP32)
        try:
            x = torch.zeros_like(b)
            st, info = L.wilson_solve_ex(ctx, g, x, b, b.shape[0], kappa, tol, opts)
            torch.cuda.synchronize()
            out.append((st, x.clone(), [i["iterations"] for i in info], [i["true_residual"] for i in info]))
        finally:
            L.wilson_gauge_free(ctx, g)
            L.wilson_context_destroy(ctx)
    return out


# Vh = 8, 960 (15 tiles), 2160 (the last tile of 48 sites); 12 x 32 tiles exceed the device
@pytest.mark.parametrize("dims,nrhs,precision,scale", [
    ((2, 2, 2, 2), 1, 0, 1.0), ((2, 2, 2, 2), 2, 1, 1.0), ((4, 6, 8, 10), 3, 0, 1.0), ((4, 6, 8, 10), 1, 1, 1.02),
    ((6, 6, 10, 12), 1, 0, 1.02), ((6, 6, 10, 12), 2, 1, 1.0), ((8, 8, 8, 8), 8, 0, 1.0), ((8, 8, 8, 8), 12, 1, 1.0)])
def test_one_launch_is_bitwise_the_launches(L, dims, nrhs, precision, scale, monkeypatch):
    U = scale * inputs.gauge_field(dims, eps=0.3, seed=4300)  # (1.02 U is not SU(3): links kept in full)
    b = inputs.gaussian_source(dims, seed=4301, nrhs=nrhs).to(DEV)
    if nrhs > 1:
        b[1] = 0
    kappa = [0.12 - 0.002 * k for k in range(nrhs)]
    sep, one = solves(L, monkeypatch, dims, U, b, kappa, 1e-10, {"precision": precision})
    assert sep[0] == one[0] == 0 and sep[2:] == one[2:]
    assert torch.equal(sep[1], one[1])
    xn, bn = one[1].cpu().numpy(), b.cpu().numpy()
    for k in range(nrhs):
        n = np.linalg.norm(bn[k])
        r = np.linalg.norm(bn[k] - oracle.apply_D(xn[k], U.numpy(), kappa[k], dims))
        assert r <= 1e-10 * n


def test_iteration_limit_and_long_runs(L, monkeypatch):
    """A solve stopped by maxiter, and one far beyond the critical kappa that runs for more
    iterations than one launch takes before it breaks down."""
    dims = (4, 4, 4, 4)
    U = inputs.gauge_field(dims, eps=1.0, seed=11)
    b = inputs.gaussian_source(dims, seed=5, nrhs=1).to(DEV)
    for kappa, opts in ((0.2, {"maxiter": 7}), (0.4, {"maxiter": 9000, "max_restarts": 0})):
        sep, one = solves(L, monkeypatch, dims, U, b, kappa, 1e-13, opts)
        assert sep[0] == one[0] != 0 and sep[2:] == one[2:]
        assert torch.equal(sep[1], one[1])
    assert one[2][0] > 1024
