// D = 1 - kappa H on both parities in one launch, with the output in the canonical layout
// (the operator call; the solvers stay on parity planes).
//
// Two parity hops in separate launches read every link twice from HBM (each link serves the
// forward hop of one parity and the backward hop of the other) and leave the result in
// planes for another pass to put together.  Here one launch walks both parities of the same
// sites together: the second use of a link, and the identity term, which is the site the
// other parity's stencil is centred on, come from the caches, and a block's result leaves
// as whole canonical rows through LDS.
//
// Three kernels:
//   dslash_full_kernel   from parity planes (large lattices: bound by HBM);
//   dslash_rhs_kernel    one parity of several right-hand sides from parity planes, the
//                        result written to the canonical layout by the wave that has it
//                        instead of to planes that another pass reads back;
//   dslash_small_kernel  from the canonical input itself, five waves per 64 output sites as
//                        in the solvers' direction split (lattices whose fields fit the
//                        caches: the call is bound by launches and latency, and one launch
//                        does what took a conversion of each parity, two hops and two
//                        conversions back).
#include "dslash_kernels.h"

namespace wl {

// What the gather helpers of the hop read of their argument struct.
struct HopSource {
    Spinor in;
    const void *gauge;
};

// o as it reads back from storage precision SP (FP16: scaled by the site's largest component)
template <int SP, typename R>
__device__ __forceinline__ void as_stored(Cx<R> (&o)[12]) {
    if constexpr (SP == P16) {
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < 12; c++) s = fmaxf(s, fmaxf(fabsf(o[c].re), fabsf(o[c].im)));
        const float sd = s > 0.f ? s : 1.f;
#pragma unroll
        for (int c = 0; c < 12; c++) {
            const float re = s > 0.f ? o[c].re / sd : 0.f, im = s > 0.f ? o[c].im / sd : 0.f;
            o[c] = {(float)(_Float16)re * s, (float)(_Float16)im * s};
        }
    }
}

// o + y as the hop's epilogue forms it, so that FP32 and FP16 results do not change in their last
// bits with the kernel: there the product that made o is rounded before a branch that adds y; here
// the compiler would fuse it into the sum (FP64 keeps that).  pinned: FP16's product with the site's
// scale, which made y, is fused, as in the hops that load y where they add it; with plain it is
// not, as in the direction split, which has y loaded before.
template <typename R>
__device__ __forceinline__ Cx<R> add_pinned(Cx<R> o, Cx<R> y) {
    if constexpr (sizeof(R) == 4) asm volatile("" : "+v"(o.re), "+v"(o.im));
    return cadd(o, y);
}
__device__ __forceinline__ Cx<double> add_plain(Cx<double> o, Cx<double> y) { return cadd(o, y); }
#pragma clang fp contract(off)
__device__ __forceinline__ Cx<float> add_plain(Cx<float> o, Cx<float> y) { return {o.re + y.re, o.im + y.im}; }
#pragma clang fp contract(fast)

constexpr int kCanonRow = 13;  // padded LDS row of one site: 12 complex and one unused

// A block holds 128 checkerboard sites of each parity (waves 0, 1 even, 2, 3 odd): the 256
// consecutive canonical sites 2 i0 .. 2 i0 + 255, since checkerboard site i of either parity
// is one of the full sites 2i, 2i + 1.
// Bound by the plane loads, as the hop, and by the canonical rows it writes: 32^3x64 FP64, D takes
// 626 us (142 split + 472 here) against 944 as two conversions each way and two hops of 278;
// what it must move (input, output, links once) is 1.6 GB, 244 us at a copy's 6.6 TB/s.
template <int SP, int GP, int NE, bool SHX>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(HopOcc<SP, 1>::value)))
dslash_full_kernel(const FullArgs p, const VisitOrder vo) {
    using R = real_t<SP>;
    __shared__ __align__(16) Cx<R> buf[256 * kCanonRow];
    const Geom &g = p.g;
    const int tid = threadIdx.x;
    const int par = __builtin_amdgcn_readfirstlane(tid >> 7), l = tid & 127;
    const int b0 = xcd_tile(blockIdx.x, gridDim.x) * 128;
    const int n = min(128, g.Vh - b0);
    const int i0 = visit_order(b0, g, vo);  // (plane blocks are whole tiles: the tile stays contiguous)
    const int i = i0 + (l < n ? l : n - 1);
    const SiteXY c = cb_coords(g, i, par);
    const SiteNbrs nb = site_nbrs(g, i, c);
    const Spinor fp = par ? p.f[1] : p.f[0];
    const HopSource a = {par ? p.f[0] : p.f[1], p.gauge};
    const bool act[1] = {true};
    Cx<R> acc[1][4][3];
    hop_sum<SP, GP, 1, NE, false, false, SHX, false, 0>(acc, a, g, par, i, c, nb, 0, act, g.stride, nullptr);
    // the sums are complete here: the compiler otherwise sinks the arithmetic of all eight
    // directions into the branch that uses it, keeping every load live (1.3 KB of spills)
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int k = 0; k < 3; k++) asm volatile("" : "+v"(acc[0][s][k].re), "+v"(acc[0][s][k].im));
    const R cH = (R)p.cH;
    Cx<R> y[12], o[12];
    load_site<SP, R>(y, fp, g.stride, 0, i);
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int k = 0; k < 3; k++) o[s * 3 + k] = add_pinned(cscale(acc[0][s][k], cH), y[s * 3 + k]);
    as_stored<SP, R>(o);
    if (l < n) {
#pragma unroll
        for (int k = 0; k < 12; k++) buf[(2 * l + c.b) * kCanonRow + k] = o[k];
    }
    __syncthreads();
    dvec2 *dst = reinterpret_cast<dvec2 *>(p.out) + (size_t)i0 * 24;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const int e = k * 256 + tid, site = e / 12;
        if (site < 2 * n) {
            const Cx<R> x = buf[site * kCanonRow + (e - site * 12)];
            dvec2 d;
            d.x = (double)x.re;
            d.y = (double)x.im;
            __builtin_nontemporal_store(d, gptr_w(dst) + e);
        }
    }
}

// One parity of nrhs right-hand sides.  With LL the waves of a block take successive right-hand
// sides of the same 64 sites and share the tile's links through LDS (as the tuned hops of 12
// right-hand sides do); without, a block takes 256 sites of one.  Each wave then turns its 64
// results in LDS (the links' room, one padded row per site) and writes their 192-byte chunks
// five and a third per access.  Bound by the plane loads' requests and the canonical writes: 24^3x48,
// 12 RHS in FP32, one parity 400 us where the hop and the conversion of its result took 497
// (1.15 GB moved at the least).
template <int SP, int GP, int NE, bool SHX, bool LL>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(HopOcc<SP, 1>::value)))
dslash_rhs_kernel(const FullArgs p, int par, int has_y, const VisitOrder vo) {
    using R = real_t<SP>;
    extern __shared__ __align__(16) char rhs_lds[];
    const Geom &g = p.g;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    const int lb = xcd_tile(blockIdx.x, gridDim.x), groups = LL ? p.nrhs / ((int)blockDim.x >> 6) : p.nrhs;
    const int tile = lb / groups, grp = lb - tile * groups;
    const int rhs = LL ? grp * ((int)blockDim.x >> 6) + w : grp;
    const int l = LL ? tile * 64 + lane : tile * 256 + (int)threadIdx.x;
    const bool valid = l < g.Vh;
    const int i = valid ? visit_order(l, g, vo) : g.Vh - 1;
    const SiteXY c = cb_coords(g, i, par);
    const SiteNbrs nb = site_nbrs(g, i, c);
    const Spinor fp = par ? p.f[1] : p.f[0];
    const HopSource a = {par ? p.f[0] : p.f[1], p.gauge};
    const bool act[1] = {true};
    if constexpr (LL) {
        const int lsite[8] = {i, nb.xm, i, nb.ym, i, nb.zm, i, nb.tm};
        stage_links<GP, NE>(rhs_lds, a, par, lsite, g.stride);
    }
    Cx<R> acc[1][4][3];
    hop_sum<SP, GP, 1, NE, false, false, SHX, LL, 0>(acc, a, g, par, i, c, nb, rhs, act, g.stride, rhs_lds);
    // (complete here, as in dslash_full_kernel)
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int k = 0; k < 3; k++) asm volatile("" : "+v"(acc[0][s][k].re), "+v"(acc[0][s][k].im));
    const R cH = (R)p.cH;
    Cx<R> o[12];
#pragma unroll
    for (int k = 0; k < 12; k++) o[k] = cscale(acc[0][k / 3][k % 3], cH);
    if (has_y) {
        Cx<R> y[12];
        load_site<SP, R, true>(y, fp, g.stride, rhs, i);
#pragma unroll
        for (int k = 0; k < 12; k++) o[k] = add_pinned(o[k], y[k]);
    }
    as_stored<SP, R>(o);
    if constexpr (LL) __syncthreads();  // every wave has read the links
    Cx<R> *row = reinterpret_cast<Cx<R> *>(rhs_lds) + w * 64 * kCanonRow;
#pragma unroll
    for (int k = 0; k < 12; k++) row[lane * kCanonRow + k] = o[k];
    __syncthreads();
    const int s = valid ? 2 * i + c.b : -1;
    dvec2 *dst = reinterpret_cast<dvec2 *>(p.out) + (size_t)rhs * g.Vh * 24;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const int e = k * 64 + lane, o_ = e / 12;
        const int so = __shfl(s, o_, 64);
        if (so >= 0) {
            const Cx<R> x = row[o_ * kCanonRow + (e - o_ * 12)];
            dvec2 d;
            d.x = (double)x.re;
            d.y = (double)x.im;
            __builtin_nontemporal_store(d, gptr_w(dst) + ((size_t)so * 12 + (e - o_ * 12)));
        }
    }
}

// Site s of the canonical input as it would read from storage precision SP: components and,
// for FP16, the site's scale.  half: the spin half a t-hop needs (-1: all; FP16 needs the
// whole site for its scale).
template <int SP, typename R>
__device__ __forceinline__ void load_canon(Cx<R> (&v)[12], R &sc, const double2 *in, size_t s, int half) {
    const dvec2 *src = reinterpret_cast<const dvec2 *>(in) + s * 12;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        if (SP == P16 || half < 0 || (k >= 6 * half && k < 6 * half + 6)) {
            const dvec2 d = gptr(src)[k];
            v[k] = {(R)d.x, (R)d.y};
        } else {
            v[k] = {R(0), R(0)};
        }
    }
    sc = R(1);
    if constexpr (SP == P16) {
        float m = 0.f;
#pragma unroll
        for (int k = 0; k < 12; k++) m = fmaxf(m, fmaxf(fabsf(v[k].re), fabsf(v[k].im)));
        const float sd = m > 0.f ? m : 1.f;
#pragma unroll
        for (int k = 0; k < 12; k++)
            v[k] = m > 0.f ? Cx<R>{(float)(_Float16)(v[k].re / sd), (float)(_Float16)(v[k].im / sd)} : Cx<R>{R(0), R(0)};
        sc = m;
    }
}

// Wave 1 + mu of a block: the two hops along MU of the block's 64 output sites.  A neighbour
// of checkerboard index j is the full site 2j + b', where b' is the output site's b for y, z
// and t (the coordinate's parity flips with the site's) and 1 - b along x.
template <int SP, int GP, int NE, int MU>
__device__ __forceinline__ void small_dir(Cx<real_t<SP>> (&acc)[1][4][3], const FullArgs &p, const HopSource &a,
                                          const double2 *in, int par, int i, const SiteXY &c, int jf, int jb) {
    using R = real_t<SP>;
    const Geom &g = p.g;
    const bool act[1] = {true};
    const int bn = MU == 0 ? 1 - c.b : c.b;
    const R one = R(1);
    const R sf = MU == 3 && NE == 6 && c.t == g.L[3] - 1 ? -one : one;
    const R sb = MU == 3 && NE == 6 && c.t == 0 ? -one : one;
    Cx<R> v[12], H[1][2][3];
    R sc;
    load_canon<SP, R>(v, sc, in, 2 * (size_t)jf + bn, MU == 3 ? 1 : -1);
    proj_in<SP, MU, true, false>(v, sc, H[0]);
    hop_dir<SP, GP, 1, NE, false, false, MU, true, 1, false, 0>(acc, a, act, 0, jf, par, i, sf, g.stride, H);
    load_canon<SP, R>(v, sc, in, 2 * (size_t)jb + bn, MU == 3 ? 0 : -1);
    proj_in<SP, MU, false, false>(v, sc, H[0]);
    hop_dir<SP, GP, 1, NE, false, false, MU, false, 1, false, 0>(acc, a, act, 0, jb, 1 - par, jb, sb, g.stride, H);
}

// p.par = 0 or 1: the parity hop alone (out = cH H in on that parity's sites); 2: D on both.
// blockIdx.x = (tile * parities + parity) * nrhs + rhs.  The four directions are added in
// the order of the solvers' direction split.  Bound by latency: D at 8^4 in FP64 6.4 us against
// 24.6 in six launches.
template <int SP, int GP, int NE>
__global__ void __launch_bounds__(320) dslash_small_kernel(const FullArgs p) {
    using R = real_t<SP>;
    const Geom &g = p.g;
    const int lb = blockIdx.x, tp = lb / p.nrhs, rhs = lb - tp * p.nrhs;
    const int par = p.par == 2 ? (tp & 1) : p.par, tile = p.par == 2 ? (tp >> 1) : tp;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    const int l = tile * 64 + lane;
    const bool valid = l < g.Vh;
    const int i = valid ? l : g.Vh - 1;
    const SiteXY c = cb_coords(g, i, par);
    const double2 *in = p.in + (size_t)rhs * g.Vh * 24;
    __shared__ R part[4][24][64];
    Cx<R> y[12];
    R ys = R(1);
    if (wv > 0) {
        Cx<R> acc[1][4][3];
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int k = 0; k < 3; k++) acc[0][s][k] = {R(0), R(0)};
        const HopSource a = {Spinor(), p.gauge};
        const SiteNbrs nb = site_nbrs(g, i, c);
        if (wv == 1) small_dir<SP, GP, NE, 0>(acc, p, a, in, par, i, c, nb.xp, nb.xm);
        else if (wv == 2) small_dir<SP, GP, NE, 1>(acc, p, a, in, par, i, c, nb.yp, nb.ym);
        else if (wv == 3) small_dir<SP, GP, NE, 2>(acc, p, a, in, par, i, c, nb.zp, nb.zm);
        else small_dir<SP, GP, NE, 3>(acc, p, a, in, par, i, c, nb.tp, nb.tm);
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int k = 0; k < 3; k++) {
                part[wv - 1][2 * (s * 3 + k)][lane] = acc[0][s][k].re;
                part[wv - 1][2 * (s * 3 + k) + 1][lane] = acc[0][s][k].im;
            }
    } else if (p.par == 2) {
        load_canon<SP, R>(y, ys, in, 2 * (size_t)i + c.b, -1);
        if constexpr (SP == P16) {
#pragma unroll
            for (int k = 0; k < 12; k++) y[k] = cscale(y[k], ys);
        }
    }
    __syncthreads();
    if (wv != 0) return;
    const R cH = (R)p.cH;
    Cx<R> o[12];
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const Cx<R> t = {((part[0][2 * k][lane] + part[1][2 * k][lane]) + part[2][2 * k][lane]) + part[3][2 * k][lane],
                         ((part[0][2 * k + 1][lane] + part[1][2 * k + 1][lane]) + part[2][2 * k + 1][lane]) +
                             part[3][2 * k + 1][lane]};
        o[k] = cscale(t, cH);
        if (p.par == 2) o[k] = add_plain(o[k], y[k]);
    }
    as_stored<SP, R>(o);
    if (!valid) return;
    dvec2 *dst = reinterpret_cast<dvec2 *>(p.out) + ((size_t)rhs * g.Vh * 2 + 2 * (size_t)i + c.b) * 12;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        dvec2 d;
        d.x = (double)o[k].re;
        d.y = (double)o[k].im;
        gptr_w(dst)[k] = d;
    }
}

template <int SP, int GP>
static hipError_t full_pg(const FullArgs &p, int zblk, hipStream_t s) {
    constexpr bool SHX = SP != P64;  // (FP64 spills with the exchange)
    const dim3 grid((p.g.Vh + 127) / 128), block(256);
    const VisitOrder vo = make_visit_order(p.g, zblk);
    if (p.recon == 12) hipLaunchKernelGGL((dslash_full_kernel<SP, GP, 6, SHX>), grid, block, 0, s, p, vo);
    else hipLaunchKernelGGL((dslash_full_kernel<SP, GP, 9, SHX>), grid, block, 0, s, p, vo);
    return hipGetLastError();
}
template <int SP, int GP>
static hipError_t small_pg(const FullArgs &p, hipStream_t s) {
    const dim3 grid((unsigned)((p.g.Vh + 63) / 64 * (p.par == 2 ? 2 : 1) * p.nrhs)), block(320);
    if (p.recon == 12) hipLaunchKernelGGL((dslash_small_kernel<SP, GP, 6>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((dslash_small_kernel<SP, GP, 9>), grid, block, 0, s, p);
    return hipGetLastError();
}

template <int SP, int GP, int NE>
static hipError_t rhs_pgn(const FullArgs &p, int par, int has_y, hipStream_t s) {
    constexpr bool SHX = SP != P64;
    constexpr size_t turn = 64 * kCanonRow * 2 * sizeof(real_t<SP>);  // one wave's
    // t visited inside eighths of z where a z-plane is whole tiles of 64 sites, memory order
    // elsewhere.  What it is worth depends on size and count, either way by less than a tenth (us, 12 RHS,
    // one parity, eighths / memory order): 32^4 FP64 1435 / 1470, FP32 1011 / 1016; 16^3x32 FP64 145 / 145, FP32
    // 116 / 105.  Ragged planes gain on large lattices only: 24^3x48 FP64 829 / 872, FP32 608 / 630, but
    // 18x10x16x22 FP64 79 / 77, FP32 61 / 57.
    const int zblk = p.g.L[2] % 8 == 0 && (p.g.Lxh * p.g.L[1]) % 64 == 0 ? p.g.L[2] / 8 : 0;
    // Links in LDS for 4 or 3 right-hand sides at a time: at 24^3x48 one parity of 12 takes 631 us
    // against 687 without in FP32 and 881 against 954 in FP64, with the conversion.  Two at a time do
    // not repay the barriers (109 against 103 us in FP32), nor do FP16's short loads (569 against
    // 566); 5, 7 or 11 divide into no such group (5 at 24^3x48: FP32 292 us, 510 through the hop's planes;
    // FP64 412 / 712); whole links (18 reals) take the registers or the LDS (FP32 1141 against 746).
    if constexpr (SP != P16 && NE == 6) {
        const int nw = p.nrhs % 4 == 0 ? 4 : (p.nrhs % 3 == 0 ? 3 : 1);
        if (nw > 1) {
            constexpr size_t links = 8 * LinkElems<GP, NE>::N * 64 * LinkPack<GP>::EB;
            const size_t lds = nw * turn > links ? nw * turn : links;
            const dim3 grid((p.g.Vh + 63) / 64 * (p.nrhs / nw)), block(64 * nw);
            hipLaunchKernelGGL((dslash_rhs_kernel<SP, GP, NE, SHX, true>), grid, block, lds, s, p, par, has_y,
                               make_visit_order(p.g, zblk));
            return hipGetLastError();
        }
    }
    const dim3 grid((p.g.Vh + 255) / 256 * p.nrhs), block(256);
    hipLaunchKernelGGL((dslash_rhs_kernel<SP, GP, NE, SHX, false>), grid, block, 4 * turn, s, p, par, has_y,
                       make_visit_order(p.g, zblk));
    return hipGetLastError();
}
hipError_t launch_dslash_rhs(const FullArgs &p, int par, int has_y, hipStream_t s) {
    const int sp = p.f[1 - par].prec, gp = p.gprec;
    if ((p.recon != 12 && p.recon != 18) || p.nrhs < 1 || p.nrhs > kMaxRhs || par < 0 || par > 1) return hipErrorInvalidValue;
    const bool two = p.recon == 12;
    if (sp == P64 && gp == P64) return two ? rhs_pgn<P64, P64, 6>(p, par, has_y, s) : rhs_pgn<P64, P64, 9>(p, par, has_y, s);
    if (sp == P32 && gp == P32) return two ? rhs_pgn<P32, P32, 6>(p, par, has_y, s) : rhs_pgn<P32, P32, 9>(p, par, has_y, s);
    if (sp == P16 && gp == P16) return two ? rhs_pgn<P16, P16, 6>(p, par, has_y, s) : rhs_pgn<P16, P16, 9>(p, par, has_y, s);
    if (sp == P16 && gp == P32) return two ? rhs_pgn<P16, P32, 6>(p, par, has_y, s) : rhs_pgn<P16, P32, 9>(p, par, has_y, s);
    return hipErrorInvalidValue;
}

hipError_t launch_dslash_full(const FullArgs &p, hipStream_t s) {
    const int sp = p.f[0].prec, gp = p.gprec;
    if ((p.recon != 12 && p.recon != 18) || p.par != 2 || p.nrhs != 1 || p.f[1].prec != sp) return hipErrorInvalidValue;
    const int zblk = full_zblk(p.g);
    if (sp == P64 && gp == P64) return full_pg<P64, P64>(p, zblk, s);
    if (sp == P32 && gp == P32) return full_pg<P32, P32>(p, zblk, s);
    if (sp == P16 && gp == P16) return full_pg<P16, P16>(p, zblk, s);
    if (sp == P16 && gp == P32) return full_pg<P16, P32>(p, zblk, s);
    return hipErrorInvalidValue;
}

hipError_t launch_dslash_small(const FullArgs &p, int sp, hipStream_t s) {
    const int gp = p.gprec;
    if ((p.recon != 12 && p.recon != 18) || p.nrhs < 1 || p.nrhs > kMaxRhs || p.par < 0 || p.par > 2)
        return hipErrorInvalidValue;
    if (sp == P64 && gp == P64) return small_pg<P64, P64>(p, s);
    if (sp == P32 && gp == P32) return small_pg<P32, P32>(p, s);
    if (sp == P16 && gp == P16) return small_pg<P16, P16>(p, s);
    if (sp == P16 && gp == P32) return small_pg<P16, P32>(p, s);
    return hipErrorInvalidValue;
}

}  // namespace wl
