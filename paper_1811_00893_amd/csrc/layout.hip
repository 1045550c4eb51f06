// Layout and precision conversion kernels (boundary of the library, not the hot loop).
//
//   * canonical complex128 spinors [rhs][site][spin][colour]  <->  parity-split planes;
//   * FP64 -> FP32 / FP16-with-per-site-scale encodings (FP16: scale s = max |component|
//     over the 24 reals of the site in FP32, h = fp16_rne(fp32(v / s)));
//   * gauge packing: canonical links -> parity-split planes.  Full (18-real) links carry
//     the antiperiodic sign of the time boundary folded into U_t(x) on the slice
//     t = Lt - 1 (that link serves both the forward hop out of t = Lt-1 and the backward
//     hop out of t = 0).  SU(3) links may instead be stored as their first two rows
//     (12 reals): the third row of a special unitary matrix is the complex conjugate of
//     the cross product of the first two, and the hop kernel rebuilds it and applies the
//     boundary sign itself (a folded sign would flip det U and break that identity);
//   * the defect-correction glue (scaled conversion of the residual, FP64 accumulation
//     of the correction), and a plain streaming copy used as a bandwidth reference.
#include "common.h"
#include "device.h"

namespace wl {

__device__ __forceinline__ int full_site(const Geom &g, int i, int par, int *t_out) {
    const SiteXY c = cb_coords(g, i, par);
    const int x = 2 * c.xh + c.b;
    if (t_out) *t_out = c.t;
    return x + g.L[0] * (c.y + g.L[1] * (c.z + g.L[2] * c.t));
}

// Canonical spinors <-> parity planes.  Both directions move every byte once, so they are
// bound by HBM; a canonical site is 192 contiguous bytes and a plane element 16, so a lane
// that reads its own site from the canonical side touches 64 lines per load and leaves the
// gathering of the sectors to the caches (102 us per parity of 32^3 x 64 in FP64, 4.0 TB/s).
// Here the canonical side is read and written in whole runs and a tile goes through LDS
// (one padded row of 13 elements per site: the 16-byte accesses of 16 lanes fall into
// different banks), where each lane picks up its own site.
//   both parities: checkerboard site i of either parity is one of the full sites 2i, 2i + 1,
//     so a block takes 128 checkerboard sites of each parity = 256 consecutive sites = 48 KB;
//   one parity: a wave takes its 64 sites' 192-byte chunks, five and a third of them per
//     access.
// 32^3 x 64 FP64, both parities in one pass: 142 us (5.7 TB/s) where two passes took 203.  24^3 x 48,
// 12 FP32 right-hand sides, one parity: in 226 us (281 before), out 243 (314); a parity's chunks
// share every third 128-byte line with the other parity, which costs a third more bytes read.
constexpr int kRow = 13;  // padded LDS row: elements of one site

template <int P, bool NORM>
__global__ void __launch_bounds__(256) split_kernel(Spinor fe, Spinor fo, const double2 *canon, Geom g,
                                                    double *partials) {
    using R = real_t<P>;
    __shared__ __align__(16) Cx<R> buf[256 * kRow];
    const int tid = threadIdx.x, rhs = blockIdx.y;
    const int i0 = blockIdx.x * 128;
    const int n = min(128, g.Vh - i0);  // checkerboard sites of each parity in this tile
    const dvec2 *src = reinterpret_cast<const dvec2 *>(canon) + ((size_t)rhs * g.Vh + i0) * 24;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const int e = k * 256 + tid, site = e / 12;
        if (site < 2 * n) {
            const dvec2 d = __builtin_nontemporal_load(gptr(src) + e);
            buf[site * kRow + (e - site * 12)] = {(R)d.x, (R)d.y};
        }
    }
    __syncthreads();
    const int par = __builtin_amdgcn_readfirstlane(tid >> 7), l = tid & 127;
    double red[1] = {0.0};
    if (l < n) {
        const SiteXY c = cb_coords(g, i0 + l, par);
        Cx<R> v[12];
#pragma unroll
        for (int k = 0; k < 12; k++) v[k] = buf[(2 * l + c.b) * kRow + k];
        if constexpr (NORM) {
#pragma unroll
            for (int k = 0; k < 12; k++) red[0] += (double)v[k].re * v[k].re + (double)v[k].im * v[k].im;
        }
        store_site<P, R>(par ? fo : fe, g.stride, rhs, i0 + l, v);
    }
    if constexpr (NORM) block_reduce_to<1>(red, partials + (size_t)rhs * gridDim.x + blockIdx.x, 1);
}

template <int P>
__global__ void __launch_bounds__(256) join_kernel(double2 *canon, Spinor fe, Spinor fo, Geom g) {
    using R = real_t<P>;
    __shared__ __align__(16) Cx<R> buf[256 * kRow];
    const int tid = threadIdx.x, rhs = blockIdx.y;
    const int i0 = blockIdx.x * 128;
    const int n = min(128, g.Vh - i0);
    const int par = __builtin_amdgcn_readfirstlane(tid >> 7), l = tid & 127;
    if (l < n) {
        const SiteXY c = cb_coords(g, i0 + l, par);
        Cx<R> v[12];
        load_site<P, R, true>(v, par ? fo : fe, g.stride, rhs, i0 + l);
#pragma unroll
        for (int k = 0; k < 12; k++) buf[(2 * l + c.b) * kRow + k] = v[k];
    }
    __syncthreads();
    dvec2 *dst = reinterpret_cast<dvec2 *>(canon) + ((size_t)rhs * g.Vh + i0) * 24;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const int e = k * 256 + tid, site = e / 12;
        if (site < 2 * n) {
            const Cx<R> x = buf[site * kRow + (e - site * 12)];
            dvec2 d;
            d.x = (double)x.re;
            d.y = (double)x.im;
            __builtin_nontemporal_store(d, gptr_w(dst) + e);
        }
    }
}

// One parity.  Lane l of a wave owns checkerboard site i0 + l; the wave's chunks are moved
// element by element (element e of the wave: component e % 12 of its site e / 12).
template <int P>
__global__ void __launch_bounds__(256) split_one_kernel(Spinor f, const double2 *canon, Geom g, int par) {
    using R = real_t<P>;
    __shared__ __align__(16) Cx<R> buf[256 * kRow];
    const int i = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63, rhs = blockIdx.y;
    const bool valid = i < g.Vh;
    const int s = full_site(g, valid ? i : g.Vh - 1, par, nullptr);  // (past the end: the last site again)
    const dvec2 *src = reinterpret_cast<const dvec2 *>(canon) + (size_t)rhs * g.Vh * 24;
    Cx<R> *row = buf + (threadIdx.x & ~63) * kRow;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const int e = k * 64 + lane, o = e / 12;
        const int so = __shfl(s, o, 64);
        const dvec2 d = __builtin_nontemporal_load(gptr(src) + ((size_t)so * 12 + (e - o * 12)));
        row[o * kRow + (e - o * 12)] = {(R)d.x, (R)d.y};
    }
    __syncthreads();
    if (!valid) return;
    Cx<R> v[12];
#pragma unroll
    for (int k = 0; k < 12; k++) v[k] = row[lane * kRow + k];
    store_site<P, R>(f, g.stride, rhs, i, v);
}

template <int P>
__global__ void __launch_bounds__(256) join_one_kernel(double2 *canon, Spinor f, Geom g, int par) {
    using R = real_t<P>;
    __shared__ __align__(16) Cx<R> buf[256 * kRow];
    const int i = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63, rhs = blockIdx.y;
    const bool valid = i < g.Vh;
    const int s = valid ? full_site(g, i, par, nullptr) : -1;
    Cx<R> *row = buf + (threadIdx.x & ~63) * kRow;
    if (valid) {
        Cx<R> v[12];
        load_site<P, R, true>(v, f, g.stride, rhs, i);
#pragma unroll
        for (int k = 0; k < 12; k++) row[lane * kRow + k] = v[k];
    }
    __syncthreads();
    dvec2 *dst = reinterpret_cast<dvec2 *>(canon) + (size_t)rhs * g.Vh * 24;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const int e = k * 64 + lane, o = e / 12;
        const int so = __shfl(s, o, 64);
        if (so >= 0) {
            const Cx<R> x = row[o * kRow + (e - o * 12)];
            dvec2 d;
            d.x = (double)x.re;
            d.y = (double)x.im;
            __builtin_nontemporal_store(d, gptr_w(dst) + ((size_t)so * 12 + (e - o * 12)));
        }
    }
}

template <int PD>
__global__ void __launch_bounds__(256) convert_kernel(Spinor dst, Spinor src, Geom g, const RhsState *state,
                                                      int inv_sqrt_aux) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.Vh) return;
    const int rhs = blockIdx.y;
    double c = 1.0;
    if (state && inv_sqrt_aux) {
        const double a = state[rhs].aux;
        c = a > 0.0 ? 1.0 / sqrt(a) : 0.0;
    }
    Cx<double> v[12];
    load_site<P64, double>(v, src, g.stride, rhs, i);
    using R = real_t<PD>;
    Cx<R> o[12];
#pragma unroll
    for (int k = 0; k < 12; k++) o[k] = {(R)(v[k].re * c), (R)(v[k].im * c)};
    store_site<PD, R>(dst, g.stride, rhs, i, o);
}

template <int PE>
__global__ void __launch_bounds__(256) axpy_f64_kernel(Spinor x, Spinor e, Geom g, const RhsState *state,
                                                       int sqrt_aux) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= g.Vh) return;
    const int rhs = blockIdx.y;
    double c = 1.0;
    if (sqrt_aux) {
        const double a = state[rhs].aux;
        c = a > 0.0 ? sqrt(a) : 0.0;
    }
    using R = real_t<PE>;
    Cx<R> ev[12];
    load_site<PE, R>(ev, e, g.stride, rhs, i);
    Cx<double> xv[12];
    load_site<P64, double>(xv, x, g.stride, rhs, i);
#pragma unroll
    for (int k = 0; k < 12; k++) {
        xv[k].re = fma(c, (double)ev[k].re, xv[k].re);
        xv[k].im = fma(c, (double)ev[k].im, xv[k].im);
    }
    store_site<P64, double>(x, g.stride, rhs, i, xv);
}

// Largest deviation of one link from SU(3): max over entries of |U U^dag - 1| and |det U - 1|.
__device__ __forceinline__ double su3_deviation(const Cx<double> (&u)[3][3]) {
    double dev = 0.0;
    for (int a = 0; a < 3; a++)
        for (int b = 0; b < 3; b++) {
            Cx<double> acc = {a == b ? -1.0 : 0.0, 0.0};
            for (int k = 0; k < 3; k++) acc = cfma_conj(acc, u[b][k], u[a][k]);  // (U U^dag)_ab - d_ab
            dev = fmax(dev, fabs(acc.re) + fabs(acc.im));
        }
    // det via the first row and the cofactors of rows 1, 2
    const Cx<double> c0 = csub(cmul(u[1][1], u[2][2]), cmul(u[1][2], u[2][1]));
    const Cx<double> c1 = csub(cmul(u[1][2], u[2][0]), cmul(u[1][0], u[2][2]));
    const Cx<double> c2 = csub(cmul(u[1][0], u[2][1]), cmul(u[1][1], u[2][0]));
    const Cx<double> det = cadd(cadd(cmul(u[0][0], c0), cmul(u[0][1], c1)), cmul(u[0][2], c2));
    return fmax(dev, fabs(det.re - 1.0) + fabs(det.im));
}

// Canonical links -> parity-split planes in up to three precisions: one pass over the links
// (576 B a site, the largest input of the library) where each precision had a pass of its
// own with lanes 1152 B apart on the canonical side.  A block takes 32 checkerboard sites of each
// parity = 64 consecutive sites = 36 KB through LDS (rows padded by one element) and writes
// runs of 32 elements of each plane.  16^3 x 32, FP64, 18 reals a link: 32 us (4.7 TB/s).
constexpr int kPackSites = 32;
constexpr int kPackRow = 37;

template <int P>
__device__ __forceinline__ void pack_planes(void *dst, const double2 *buf, const unsigned char *info, const Geom &g,
                                            int i0, int n, int recon) {
    constexpr int CPL = LinkPack<P>::CPL;
    using R = real_t<P>;
    const int ne = recon == 12 ? 6 : 9, nl = link_elems(P, ne);
    for (int it = threadIdx.x; it < 8 * nl * kPackSites; it += 256) {
        const int c = it % kPackSites, q = it / kPackSites;  // q: plane (par * 4 + mu) * nl + e
        if (c >= n) continue;
        const int pm = q / nl, e = q - pm * nl, par = pm >> 2, mu = pm & 3;
        const double sgn = (recon == 18 && mu == 3 && (info[c] & 2)) ? -1.0 : 1.0;
        const double2 *src = buf + (2 * c + ((info[c] & 1) ^ par)) * kPackRow + mu * 9;
        Cx<R> x[CPL];
#pragma unroll
        for (int k = 0; k < CPL; k++) {
            const int idx = e * CPL + k;  // entries past the last are padding
            const double2 d = idx < ne ? src[idx] : make_double2(0.0, 0.0);
            x[k] = {(R)(sgn * d.x), (R)(sgn * d.y)};
        }
        gchar *base = (gchar *)dst + ((size_t)q * g.stride + i0) * LinkPack<P>::EB;
        st_link_elem<P, R>(base, (unsigned)c * LinkPack<P>::EB, x);
    }
}

__global__ void __launch_bounds__(256) gauge_pack_kernel(void *d64, void *d32, void *d16, const double2 *canon, Geom g,
                                                         int recon) {
    __shared__ __align__(16) double2 buf[2 * kPackSites * kPackRow];
    __shared__ unsigned char info[kPackSites];  // bit 0: x of the even-parity site is odd; bit 1: t = Lt - 1
    const int tid = threadIdx.x, i0 = blockIdx.x * kPackSites;
    const int n = min(kPackSites, g.Vh - i0);
    const dvec2 *src = reinterpret_cast<const dvec2 *>(canon) + (size_t)i0 * 72;
#pragma unroll
    for (int k = 0; k < 9; k++) {
        const int e = k * 256 + tid, site = e / 36;
        if (site < 2 * n) {
            const dvec2 d = __builtin_nontemporal_load(gptr(src) + e);
            buf[site * kPackRow + (e - site * 36)] = make_double2(d.x, d.y);
        }
    }
    if (tid < n) {
        const SiteXY c = cb_coords(g, i0 + tid, 0);
        info[tid] = (unsigned char)(c.b | (c.t == g.L[3] - 1 ? 2 : 0));
    }
    __syncthreads();
    if (d64) pack_planes<P64>(d64, buf, info, g, i0, n, recon);
    if (d32) pack_planes<P32>(d32, buf, info, g, i0, n, recon);
    if (d16) pack_planes<P16>(d16, buf, info, g, i0, n, recon);
}

// Sets *flag if any link is off SU(3) by more than tol.  256 links a block, read in whole runs
// through LDS.  A pass of its own before the packing, not part of it, so that how links are stored
// is known before buffers are made: a load in three precisions, 16^4, links in full, 390 us, and 1340
// when buffers for two rows were made first (two rows at 24^3 x 48: 870, 750 with the check inside
// the packing).
__global__ void __launch_bounds__(256) su3_check_kernel(const double2 *canon, size_t nlinks, double tol, int *flag) {
    __shared__ __align__(16) double2 buf[256 * 9];
    const size_t l0 = (size_t)blockIdx.x * 256;
    const int n = (int)(nlinks - l0 < 256 ? nlinks - l0 : 256), tid = threadIdx.x;
    const double2 *src = canon + l0 * 9;
#pragma unroll
    for (int k = 0; k < 9; k++) {
        const int e = k * 256 + tid;
        if (e < 9 * n) buf[e] = src[e];
    }
    __syncthreads();
    if (tid >= n) return;
    Cx<double> u[3][3];
#pragma unroll
    for (int e = 0; e < 9; e++) u[e / 3][e % 3] = {buf[tid * 9 + e].x, buf[tid * 9 + e].y};
    if (!(su3_deviation(u) <= tol)) *flag = 1;  // (every writer stores the same word)
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Bandwidth probes.  One 16-byte element per thread and no loop: a wave moves one
// contiguous 1 KiB run and ends, which keeps the most requests in flight on gfx950 (a
// thread that loops waits for its own earlier stores before its next loads return).
// Loads and stores are non-temporal, the fastest one-pass pattern measured (a 2 GiB copy
// 6.5-6.6 TB/s against 6.1 with ordinary loads and stores; two or more elements per
// thread were slower still).
__global__ void __launch_bounds__(256) stream_copy_kernel(uint4 *__restrict__ dst, const uint4 *__restrict__ src,
                                                          size_t n16) {
    const size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (k < n16)
        __builtin_nontemporal_store(__builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src) + k),
                                    reinterpret_cast<u32x4 *>(dst) + k);
}

// Read-only stream: each lane folds its 16 bytes into one word and, only when that word
// equals an arbitrary constant, XORs it into one of kStreamSink words.  The branch depends
// on the data, so no load can be elided, and almost no lane ever writes.
constexpr unsigned kStreamSink = 8192;
__global__ void __launch_bounds__(256) stream_read_kernel(const uint4 *__restrict__ src, size_t n16,
                                                          unsigned *sink) {
    const size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (k < n16) {
        const u32x4 a = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src) + k);
        const unsigned w = a.x ^ a.y ^ a.z ^ a.w;
        if (w == 0x9E3779B9u) atomicXor(&sink[k % kStreamSink], w);
    }
}

__global__ void copy_tail_kernel(unsigned char *dst, const unsigned char *src, size_t n) {
    const size_t k = threadIdx.x;
    if (k < n) dst[k] = src[k];
}

__global__ void check_finite_kernel(const double *p, size_t n, int *flag) {
    bool bad = false;
    for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x)
        bad |= !isfinite(p[k]);
    if (bad) atomicOr(flag, 1);
}

// ---------------------------------------------------------------------------------
static inline dim3 site_grid(const Geom &g, int ny) { return dim3((g.Vh + 255) / 256, ny); }

int split_nblocks(const Geom &g) { return (g.Vh + 127) / 128; }

hipError_t launch_split(Spinor fe, Spinor fo, const double *canon, const Geom &g, int nrhs, hipStream_t s,
                        double *partials) {
    if (fe.prec != fo.prec || (partials && fe.prec != P64)) return hipErrorInvalidValue;
    const dim3 grid(split_nblocks(g), nrhs), block(256);
    const double2 *c = reinterpret_cast<const double2 *>(canon);
    switch (fe.prec) {
        case P64:
            if (partials) hipLaunchKernelGGL((split_kernel<P64, true>), grid, block, 0, s, fe, fo, c, g, partials);
            else hipLaunchKernelGGL((split_kernel<P64, false>), grid, block, 0, s, fe, fo, c, g, partials);
            break;
        case P32: hipLaunchKernelGGL((split_kernel<P32, false>), grid, block, 0, s, fe, fo, c, g, partials); break;
        case P16: hipLaunchKernelGGL((split_kernel<P16, false>), grid, block, 0, s, fe, fo, c, g, partials); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_split_one(Spinor f, const double *canon, const Geom &g, int par, int nrhs, hipStream_t s) {
    const dim3 grid = site_grid(g, nrhs), block(256);
    const double2 *c = reinterpret_cast<const double2 *>(canon);
    switch (f.prec) {
        case P64: hipLaunchKernelGGL(split_one_kernel<P64>, grid, block, 0, s, f, c, g, par); break;
        case P32: hipLaunchKernelGGL(split_one_kernel<P32>, grid, block, 0, s, f, c, g, par); break;
        case P16: hipLaunchKernelGGL(split_one_kernel<P16>, grid, block, 0, s, f, c, g, par); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_join(double *canon, Spinor fe, Spinor fo, const Geom &g, int nrhs, hipStream_t s) {
    if (fe.prec != fo.prec) return hipErrorInvalidValue;
    const dim3 grid(split_nblocks(g), nrhs), block(256);
    double2 *c = reinterpret_cast<double2 *>(canon);
    switch (fe.prec) {
        case P64: hipLaunchKernelGGL(join_kernel<P64>, grid, block, 0, s, c, fe, fo, g); break;
        case P32: hipLaunchKernelGGL(join_kernel<P32>, grid, block, 0, s, c, fe, fo, g); break;
        case P16: hipLaunchKernelGGL(join_kernel<P16>, grid, block, 0, s, c, fe, fo, g); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_join_one(double *canon, Spinor f, const Geom &g, int par, int nrhs, hipStream_t s) {
    const dim3 grid = site_grid(g, nrhs), block(256);
    double2 *c = reinterpret_cast<double2 *>(canon);
    switch (f.prec) {
        case P64: hipLaunchKernelGGL(join_one_kernel<P64>, grid, block, 0, s, c, f, g, par); break;
        case P32: hipLaunchKernelGGL(join_one_kernel<P32>, grid, block, 0, s, c, f, g, par); break;
        case P16: hipLaunchKernelGGL(join_one_kernel<P16>, grid, block, 0, s, c, f, g, par); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_convert(Spinor dst, Spinor src, const Geom &g, int nrhs, const RhsState *state, int inv_sqrt_aux,
                          hipStream_t s) {
    if (src.prec != P64) return hipErrorInvalidValue;
    const dim3 grid = site_grid(g, nrhs), block(256);
    switch (dst.prec) {
        case P64: hipLaunchKernelGGL(convert_kernel<P64>, grid, block, 0, s, dst, src, g, state, inv_sqrt_aux); break;
        case P32: hipLaunchKernelGGL(convert_kernel<P32>, grid, block, 0, s, dst, src, g, state, inv_sqrt_aux); break;
        case P16: hipLaunchKernelGGL(convert_kernel<P16>, grid, block, 0, s, dst, src, g, state, inv_sqrt_aux); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_axpy_f64(Spinor x64, Spinor e, const Geom &g, int nrhs, const RhsState *state, int sqrt_aux,
                           hipStream_t s) {
    if (x64.prec != P64 || (sqrt_aux && !state)) return hipErrorInvalidValue;
    const dim3 grid = site_grid(g, nrhs), block(256);
    switch (e.prec) {
        case P64: hipLaunchKernelGGL(axpy_f64_kernel<P64>, grid, block, 0, s, x64, e, g, state, sqrt_aux); break;
        case P32: hipLaunchKernelGGL(axpy_f64_kernel<P32>, grid, block, 0, s, x64, e, g, state, sqrt_aux); break;
        case P16: hipLaunchKernelGGL(axpy_f64_kernel<P16>, grid, block, 0, s, x64, e, g, state, sqrt_aux); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gauge_pack(void *const dst[3], const double *canon, const Geom &g, int recon, hipStream_t s) {
    if ((recon != 12 && recon != 18) || (!dst[P64] && !dst[P32] && !dst[P16])) return hipErrorInvalidValue;
    const dim3 grid((g.Vh + kPackSites - 1) / kPackSites), block(256);
    hipLaunchKernelGGL(gauge_pack_kernel, grid, block, 0, s, dst[P64], dst[P32], dst[P16],
                       reinterpret_cast<const double2 *>(canon), g, recon);
    return hipGetLastError();
}

hipError_t launch_su3_check(const double *canon, size_t nlinks, double tol, int *flag, hipStream_t s) {
    hipLaunchKernelGGL(su3_check_kernel, dim3((unsigned)((nlinks + 255) / 256)), dim3(256), 0, s,
                       reinterpret_cast<const double2 *>(canon), nlinks, tol, flag);
    return hipGetLastError();
}

hipError_t launch_stream_read(const void *src, size_t bytes, unsigned *sink, hipStream_t s) {
    const size_t n16 = bytes / 16;
    if (n16) hipLaunchKernelGGL(stream_read_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, s,
                                (const uint4 *)src, n16, sink);
    return hipGetLastError();
}

hipError_t launch_stream_copy(void *dst, const void *src, size_t bytes, hipStream_t s) {
    const size_t n16 = bytes / 16;
    if (n16)
        hipLaunchKernelGGL(stream_copy_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, s, (uint4 *)dst,
                           (const uint4 *)src, n16);
    const size_t tail = bytes - n16 * 16;
    if (tail)
        hipLaunchKernelGGL(copy_tail_kernel, dim3(1), dim3(64), 0, s, (unsigned char *)dst + n16 * 16,
                           (const unsigned char *)src + n16 * 16, tail);
    return hipGetLastError();
}

hipError_t launch_check_finite(const double *p, size_t n, int *flag, hipStream_t s) {
    hipLaunchKernelGGL(check_finite_kernel, dim3(1024), dim3(256), 0, s, p, n, flag);
    return hipGetLastError();
}

}  // namespace wl
