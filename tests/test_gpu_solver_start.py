"""A solve starts from r, rhat and p alone: whatever the Krylov fields hold from the solve
before (here one that overflowed to NaN) must not reach it, whether its first iteration goes
on or already converges on s (kappa = 0: x = b), in the one-launch solve, the separate
launches and a batch slot."""
import numpy as np
import pytest
import torch

import oracle
from paper_1811_00893_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def residual(x, b, U, k, dims):
    return float(np.linalg.norm(b - oracle.apply_D(x, U, k, dims)) / np.linalg.norm(b))


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (8, 8, 16, 18)])  # one launch / separate launches
@pytest.mark.parametrize("precision,solver", [(0, 0), (1, 0), (3, 0), (0, 1), (0, 2)])
def test_solve_after_an_overflowed_one(dims, precision, solver):
    from paper_1811_00893_amd import _lib as L
    U = inputs.gauge_field(dims, eps=0.3, seed=4400)
    b = inputs.gaussian_source(dims, seed=4401).to(DEV)
    ctx = L.wilson_context_create()
    g = L.wilson_gauge_load(ctx, U.to(DEV), dims, L.WILSON_GAUGE_FP32)
    opts = {"precision": precision, "solver": solver, "maxiter": 500}
    try:
        for kappa in (0.0, 0.12):
            x = torch.zeros_like(b)
            # H^2 k^2 overflows: every field of that solve ends as NaN or Inf
            assert L.wilson_solve_ex(ctx, g, x, b, 1, 1e200, 1e-10, dict(opts, max_restarts=0))[0] != 0
            st, info = L.wilson_solve_ex(ctx, g, x, b, 1, kappa, 1e-10, opts)
            assert st == 0, (kappa, L.wilson_last_error())
            assert residual(x.cpu().numpy(), b.cpu().numpy(), U.numpy(), kappa, dims) < 1e-10
    finally:
        L.wilson_gauge_free(ctx, g)
        L.wilson_context_destroy(ctx)


@pytest.mark.parametrize("precision", [0, 1])
def test_batch_slot_after_an_overflowed_solve(precision):
    from paper_1811_00893_amd import _lib as L
    dims = (4, 4, 4, 8)
    U = inputs.gauge_field(dims, eps=0.3, seed=4410)
    b = inputs.gaussian_source(dims, seed=4411).to(DEV)
    ctx = L.wilson_context_create()
    g = L.wilson_gauge_load(ctx, U.to(DEV), dims, L.WILSON_GAUGE_FP32)
    bat = L.wilson_batch_create(ctx, g, 2, {"precision": precision, "max_restarts": 0})
    try:
        for kappa in (1e200, 0.0, 1e200, 0.12):
            assert L.wilson_batch_attach(bat, 0, b, kappa, 1e-10, 500) == 0
            for _ in range(600):
                L.wilson_batch_step(bat, 4)
                state, status = L.wilson_batch_poll(bat, 2)
                if state[0] == 2:
                    break
            x = torch.zeros_like(b)
            st, _ = L.wilson_batch_detach(bat, 0, x)
            if kappa < 1:
                assert st == 0
                assert residual(x.cpu().numpy(), b.cpu().numpy(), U.numpy(), kappa, dims) < 1e-10
            else:
                assert st != 0
    finally:
        L.wilson_batch_destroy(bat)
        L.wilson_gauge_free(ctx, g)
        L.wilson_context_destroy(ctx)
