"""The operator call's own kernels against the FP64 oracle: D on both parities in one launch
(from parity planes, or from the canonical input on small problems), parity hops through the
canonical conversions, at ragged and tile-sized lattices, with two-row and full links.

Tolerances as for every Dslash: FP64 1e-12, FP32 5e-7, FP16 2e-3, relative (norm-wise)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1811_00893_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
LIMIT = {0: 1e-12, 1: 5e-7, 2: 2e-3, 3: 2e-3}

# sites per parity: 8; 960 (no multiple of 64); 4096 (first size FP32 takes from planes);
# 8000 (ragged in tiles of 128); 73728 (FP64 from planes, plane blocks of two);
# 138600 (the same in memory order, ragged)
CASES = [((2, 2, 2, 2), 2), ((6, 4, 8, 10), 3), ((8, 8, 8, 16), 1), ((10, 8, 10, 20), 1), ((10, 8, 10, 20), 3),
         ((32, 16, 16, 18), 1), ((18, 22, 14, 50), 1)]


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


@pytest.fixture(scope="module")
def L():
    from paper_1811_00893_amd import _lib
    return _lib


@pytest.mark.parametrize("dims,nrhs", CASES)
@pytest.mark.parametrize("scale", [1.0, 1.25])  # 1.25 U is not SU(3): links kept in full
def test_operator_call_matches_oracle(L, dims, nrhs, scale):
    U = scale * inputs.gauge_field(dims, eps=0.3, seed=4100)
    psi = inputs.gaussian_source(dims, seed=4101, nrhs=nrhs)
    Un, pn = U.numpy(), psi.numpy()
    par = oracle.parity_of_sites(dims)
    ctx = L.wilson_context_create()
    g = L.wilson_gauge_load(ctx, U.to(DEV), dims, L.WILSON_GAUGE_FP32 | L.WILSON_GAUGE_FP16)
    try:
        for parity in (2, 0, 1):
            prev = inputs.gaussian_source(dims, seed=77, nrhs=nrhs)
            ref = np.stack([oracle.dslash(pn[k], Un, 0.124, dims, parity, out=prev.numpy()[k]) for k in range(nrhs)])
            on = np.ones(len(par), bool) if parity == 2 else par == parity
            for prec in (0, 1, 2, 3) if scale == 1.0 else (0, 1):
                out = prev.to(DEV).clone()
                L.check(L.wilson_dslash_ex(ctx, g, out, psi.to(DEV), 0.124, parity, prec, nrhs), "dslash")
                torch.cuda.synchronize()
                got = out.cpu().numpy()
                assert rel(got[:, on], ref[:, on]) < LIMIT[prec], (parity, prec)
                assert np.array_equal(got[:, ~on], prev.numpy()[:, ~on]), (parity, prec)
    finally:
        L.wilson_gauge_free(ctx, g)
        L.wilson_context_destroy(ctx)


@pytest.mark.parametrize("dims", [(4, 4, 4, 6), (10, 8, 10, 20)])
def test_overlapping_arrays(L, dims):
    """An output that overlaps the input without being it gives the separate arrays' bits, and
    a parity hop may run in place."""
    V = inputs.volume(dims)
    U = inputs.gauge_field(dims, eps=0.3, seed=4110).to(DEV)
    psi = inputs.gaussian_source(dims, seed=4111).to(DEV)
    ctx = L.wilson_context_create()
    g = L.wilson_gauge_load(ctx, U, dims)
    try:
        apart = torch.zeros_like(psi)
        L.check(L.wilson_dslash_ex(ctx, g, apart, psi, 0.12, 2), "dslash")
        buf = torch.zeros((V + V // 2, 4, 3), dtype=psi.dtype, device=DEV)
        buf[:V] = psi
        out = buf[V // 2:]
        L.check(L.wilson_dslash_ex(ctx, g, out, buf[:V], 0.12, 2), "dslash")
        torch.cuda.synchronize()
        assert rel(out.cpu().numpy(), apart.cpu().numpy()) < 1e-14
        hop = psi.clone()
        L.check(L.wilson_dslash_ex(ctx, g, hop, psi, 0.12, 1), "dslash")
        same = psi.clone()
        L.check(L.wilson_dslash_ex(ctx, g, same, same, 0.12, 1), "dslash")
        torch.cuda.synchronize()
        assert torch.equal(hop, same)
    finally:
        L.wilson_gauge_free(ctx, g)
        L.wilson_context_destroy(ctx)


def test_plain_calls_in_turn(L):
    """The two-call form with links, shapes and storage changing from call to call: the
    buffers it keeps between calls never carry one call's links into the next."""
    shapes = [(4, 4, 4, 6), (6, 4, 10, 6), (4, 4, 4, 6), (10, 8, 10, 20)]
    for n, dims in enumerate(shapes):
        for scale in (1.0, 1.25, 1.0):  # 1.25 U is not SU(3)
            U = scale * inputs.gauge_field(dims, eps=0.3, seed=4200 + n)
            psi = inputs.gaussian_source(dims, seed=4210 + n)
            out = torch.zeros_like(psi, device=DEV)
            assert L.wilson_dslash(out, psi.to(DEV), U.to(DEV), 0.11, dims, 2) == 0
            assert rel(out.cpu().numpy(), oracle.apply_D(psi.numpy(), U.numpy(), 0.11, dims)) < 1e-12
        x = torch.zeros_like(psi, device=DEV)
        assert L.wilson_solve(x, psi.to(DEV), U.to(DEV), 0.11, dims, 1e-10, 1000) == 0
        assert rel(oracle.apply_D(x.cpu().numpy(), U.numpy(), 0.11, dims), psi.numpy()) < 1e-10


# FP64 takes the plane kernels at (18, 10, 14, 22) (27720 sites per parity, ragged in tiles of 64
# and 256) for 5 or 6 right-hand sides, FP32 and FP16 at both sizes for any number; 4, 3 and 6 share
# links in blocks of four and three waves (FP64, FP32), 2 and 5 do not.
@pytest.mark.parametrize("dims,nrhs", [((8, 8, 8, 16), 2), ((8, 8, 8, 16), 4), ((18, 10, 14, 22), 3),
                                       ((18, 10, 14, 22), 5), ((18, 10, 14, 22), 6)])
@pytest.mark.parametrize("scale", [1.0, 1.25])
def test_several_rhs_match_oracle_and_the_timed_path(L, dims, nrhs, scale):
    """Hops that write the canonical layout; with per-launch timing the call goes through the
    solvers' hop, whose FP32 and FP16 results are the same to the bit."""
    U = scale * inputs.gauge_field(dims, eps=0.3, seed=4110)
    psi = inputs.gaussian_source(dims, seed=4111, nrhs=nrhs)
    prev = inputs.gaussian_source(dims, seed=4112, nrhs=nrhs)
    on = {0: oracle.parity_of_sites(dims) == 0, 1: oracle.parity_of_sites(dims) == 1, 2: np.ones(psi.shape[1], bool)}
    ctx = L.wilson_context_create()
    g = L.wilson_gauge_load(ctx, U.to(DEV), dims, L.WILSON_GAUGE_FP32 | L.WILSON_GAUGE_FP16)
    try:
        for parity in (2, 0, 1):
            ref = np.stack([oracle.dslash(psi.numpy()[k], U.numpy(), 0.124, dims, parity, out=prev.numpy()[k])
                            for k in range(nrhs)])
            for prec in (0, 1, 2, 3) if scale == 1.0 else (0, 1):
                got = []
                for timed in (False, True):
                    out = prev.to(DEV).clone()
                    L.wilson_timing_enable(ctx, timed)
                    L.check(L.wilson_dslash_ex(ctx, g, out, psi.to(DEV), 0.124, parity, prec, nrhs), "dslash")
                    L.wilson_timing_enable(ctx, False)
                    torch.cuda.synchronize()
                    got.append(out.cpu().numpy())
                for k in range(nrhs):
                    assert rel(got[0][k][on[parity]], ref[k][on[parity]]) < LIMIT[prec], (parity, prec, k)
                assert np.array_equal(got[0][:, ~on[parity]], prev.numpy()[:, ~on[parity]]), (parity, prec)
                assert prec == 0 or np.array_equal(got[0], got[1]), (parity, prec)
    finally:
        L.wilson_gauge_free(ctx, g)
        L.wilson_context_destroy(ctx)
