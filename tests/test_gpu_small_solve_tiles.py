"""BiCGStab in one launch at the upper end of its range (65 to 128 tiles of 64 sites per parity: two
partial sums a lane, up to eight rows of a vector kernel), with the direction split pinned so that
the route does not depend on tuning: the bits, iterations and residuals of the separate launches.
That the one launch ran shows in the hop count, which lacks the masked iterations that separate
launches enqueue; a solve with more blocks than the device has CUs counts the same."""
import numpy as np
import pytest
import torch

import oracle
from paper_1811_00893_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


# tiles: 66 (whole), 79 (48 sites in the last), 119 (8 sites), 128 (whole)
@pytest.mark.parametrize("dims,nrhs,precision,scale", [
    ((8, 6, 8, 22), 1, 0, 1.0), ((10, 6, 12, 14), 2, 0, 1.0), ((10, 6, 12, 14), 1, 1, 1.02), ((6, 10, 14, 18), 1, 0, 1.02),
    ((6, 10, 14, 18), 2, 1, 1.0), ((8, 8, 16, 16), 2, 0, 1.0), ((8, 8, 16, 16), 1, 1, 1.0),
    ((6, 10, 14, 18), 3, 0, 1.0), ((8, 8, 16, 16), 3, 1, 1.0)])
def test_many_tiles(dims, nrhs, precision, scale, monkeypatch):
    from paper_1811_00893_amd import _lib as L
    monkeypatch.setenv("WILSON_HOP_CFG", "320,1,1,0,0,0,0,1")
    U = scale * inputs.gauge_field(dims, eps=0.3, seed=4800)  # (1.02 U is not SU(3): links kept in full)
    b = inputs.gaussian_source(dims, seed=4801, nrhs=nrhs).to(DEV)
    kappa = [0.12 - 0.002 * k for k in range(nrhs)]
    out = []
    for polls in ("0", "2097152"):
        monkeypatch.setenv("WILSON_ONE_LAUNCH", polls)
        ctx = L.wilson_context_create()
        g = L.wilson_gauge_load(ctx, U.to(DEV), dims, L.WILSON_GAUGE_FP32)
        try:
            x = torch.zeros_like(b)
            st, info = L.wilson_solve_ex(ctx, g, x, b, nrhs, kappa, 1e-10, {"precision": precision})
            torch.cuda.synchronize()
            assert st == 0, L.wilson_last_error()
            out.append((x, [i["iterations"] for i in info], [i["true_residual"] for i in info], info[0]["hop_launches"]))
        finally:
            L.wilson_gauge_free(ctx, g)
            L.wilson_context_destroy(ctx)
    sep, one = out
    assert torch.equal(sep[0], one[0]) and sep[1:3] == one[1:3]
    tiles = -(-int(np.prod(dims)) // 128)
    assert 64 < tiles <= 128
    if tiles * nrhs <= torch.cuda.get_device_properties(0).multi_processor_count:
        assert one[3] < sep[3]
    else:
        assert one[3] == sep[3]
    xn, bn = one[0].cpu().numpy(), b.cpu().numpy()
    for k in range(nrhs):
        r = np.linalg.norm(bn[k] - oracle.apply_D(xn[k], U.numpy(), kappa[k], dims))
        assert r <= 1e-10 * np.linalg.norm(bn[k])


@pytest.mark.parametrize("dims,nrhs,precision", [((2, 2, 2, 2), 2, 0), ((4, 6, 8, 10), 3, 1), ((8, 8, 8, 8), 8, 0)])
def test_few_tiles_take_one_launch(dims, nrhs, precision, monkeypatch):
    from paper_1811_00893_amd import _lib as L
    U = inputs.gauge_field(dims, eps=0.3, seed=4810).to(DEV)
    b = inputs.gaussian_source(dims, seed=4811, nrhs=nrhs).to(DEV)
    hops = []
    for polls in ("0", "2097152"):
        monkeypatch.setenv("WILSON_ONE_LAUNCH", polls)
        ctx = L.wilson_context_create()
        g = L.wilson_gauge_load(ctx, U, dims, L.WILSON_GAUGE_FP32)
        st, info = L.wilson_solve_ex(ctx, g, torch.zeros_like(b), b, nrhs, 0.12, 1e-10, {"precision": precision})
        assert st == 0
        hops.append(info[0]["hop_launches"])
        L.wilson_gauge_free(ctx, g)
        L.wilson_context_destroy(ctx)
    assert hops[1] < hops[0]
