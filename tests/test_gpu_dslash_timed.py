"""The operator call with per-launch timing (the solvers' hop between conversions) against the call
without (a kernel of its own): the same bits in FP32 and FP16; FP64 to rounding."""
import pytest
import torch

from paper_1811_00893_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


# sites per parity: 8, 960 and 2048 (canonical input, five waves per tile); 4096 and 8000 (planes, unless the
# tuner picks the direction split); 73728 (planes)
@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 2), 1), ((6, 4, 8, 10), 3), ((8, 8, 8, 8), 1), ((8, 8, 8, 16), 1),
                                       ((10, 8, 10, 20), 1), ((32, 16, 16, 18), 1)])
@pytest.mark.parametrize("scale", [1.0, 1.25])  # 1.25 U is not SU(3): links kept in full
def test_timing_keeps_the_results(dims, nrhs, scale):
    from paper_1811_00893_amd import _lib as L
    U = scale * inputs.gauge_field(dims, eps=0.3, seed=4700).to(DEV)
    psi = inputs.gaussian_source(dims, seed=4701, nrhs=nrhs).to(DEV)
    ctx = L.wilson_context_create()
    g = L.wilson_gauge_load(ctx, U, dims, L.WILSON_GAUGE_FP32 | L.WILSON_GAUGE_FP16)
    try:
        for parity in (2, 0, 1):
            for prec in (0, 1, 2, 3) if scale == 1.0 else (0, 1):
                out = []
                for timed in (False, True):
                    o = torch.zeros_like(psi)
                    L.wilson_timing_enable(ctx, timed)
                    L.check(L.wilson_dslash_ex(ctx, g, o, psi, 0.124, parity, prec, nrhs), "dslash")
                    n = L.wilson_timing_read(ctx)[1]
                    L.wilson_timing_enable(ctx, False)
                    torch.cuda.synchronize()
                    out.append(o)
                assert n == (2 if parity == 2 else 1)
                if prec:
                    assert torch.equal(out[0], out[1]), (parity, prec)
                else:  # eight directions added in another order: a few roundings of 2^-53
                    assert torch.linalg.vector_norm(out[0] - out[1]) < 1e-14 * torch.linalg.vector_norm(out[0])
    finally:
        L.wilson_gauge_free(ctx, g)
        L.wilson_context_destroy(ctx)
