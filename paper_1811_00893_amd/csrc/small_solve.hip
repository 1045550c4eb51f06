// A whole BiCGStab solve in one launch, for lattices of a few dozen 64-site tiles.
//
// At 8^4 an iteration is nine dependent launches of 2-8 us each with gaps of about the same
// size between them: 58 us for work that takes the memory system under two.  Here one block
// per tile and right-hand side stays for all iterations.  The block's own part of r, rhat, x,
// p, v, s and t lives in its registers; what other tiles read (p, s, the odd intermediate of
// M, partial sums) is exchanged through device memory, with a barrier over the blocks of the
// right-hand side where a launch boundary was: seven per iteration.  What bounds it is the
// latency of those exchanges: of 32 us per iteration at 8^4, 13 are barriers (1.1 us for 32
// blocks that only meet, 1.7-2.0 with a tile's stores to wait for), 10 the four hops (loads
// past the L2, then wave 0's epilogue), 7 the sums and scalar steps.
//
// Exchanged data are read and written with the cache policy of agent-scope atomics (sc1: 16-byte
// buffer accesses for fields, relaxed atomics for sums and counters), so they are coherent
// between the XCDs' L2 caches without writing those back or invalidating them; a block's stores
// have completed (s_waitcnt) before it arrives at a barrier, and it reads only after it has
// seen every arrival.  The block's links are the same in every iteration and stay in registers.
//
// The blocks must run together.  It is an ordinary launch: the host keeps the blocks of all such
// solves in flight on a device within its CUs, and within each XCD's share of them, so there is
// a place for every block (kernels of other kinds end by themselves and make room).  A
// cooperative launch gives the same guarantee by running one such grid at a time: four contexts
// on four streams, 8^4 FP64, 606 us per solve against 194 (368 in separate launches).  Other
// processes are outside both guarantees, so a wait is bounded all the same, and a block that gives
// up marks the right-hand side as lost: the host then runs the separate launches.  The mark has a
// word of its own, which no other store touches: tile 0 may still see the last arrivals and store
// a state that looks finished.
//
// The arithmetic, the order of every sum and the scalar steps are those of the launches it
// replaces (the direction-split hop, the element-wise vector kernels, the one-wave finalize),
// so a solve gives the same bits either way.
#include "dslash_kernels.h"
// the vector kernels and scalar steps are compiled without multiply-add contraction (blas.hip)
#pragma clang fp contract(off)
#include "finalize.h"

namespace wl {

namespace nc {
template <typename R>
__device__ __forceinline__ Cx<R> add(Cx<R> a, Cx<R> b) { return {a.re + b.re, a.im + b.im}; }
template <typename R>
__device__ __forceinline__ Cx<R> sub(Cx<R> a, Cx<R> b) { return {a.re - b.re, a.im - b.im}; }
template <typename R>
__device__ __forceinline__ Cx<R> mul(Cx<R> a, Cx<R> b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
template <typename R>
__device__ __forceinline__ double norm2(Cx<R> v) { return (double)v.re * v.re + (double)v.im * v.im; }
template <typename R>
__device__ __forceinline__ void dot(double (&red)[3], Cx<R> e, Cx<R> r) {  // |r|^2, <e, r>
    red[0] += norm2(r);
    red[1] += (double)e.re * r.re + (double)e.im * r.im;
    red[2] += (double)e.re * r.im - (double)e.im * r.re;
}
}  // namespace nc
#pragma clang fp contract(fast)

namespace {

constexpr int kWaves = 4;  // one per direction (one per SIMD, with all its registers); wave 0 finishes the hop

typedef unsigned long long u64;
__device__ __forceinline__ void st_agent(void *p, u64 v) {
    __hip_atomic_store(reinterpret_cast<u64 *>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 ld_agent(const void *p) {
    return __hip_atomic_load(reinterpret_cast<const u64 *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent_d(double *p, double v) { st_agent(p, __builtin_bit_cast(u64, v)); }
__device__ __forceinline__ double ld_agent_d(const double *p) { return __builtin_bit_cast(double, ld_agent(p)); }

// Exchanged fields, one right-hand side of a field as a buffer resource: plane elements of 16
// bytes moved by one access each, past the L2 like an agent-scope atomic (cache policy sc1).
constexpr int kSc1 = 16;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
using BufRsrc = decltype(__builtin_amdgcn_make_buffer_rsrc((void *)nullptr, (short)0, 0, 0));
template <int P>
__device__ __forceinline__ BufRsrc shared_field(const Spinor &f, int stride, int rhs) {
    const size_t bytes = (size_t)SpinorPack<P>::NEL * stride * 16u;
    char *base = static_cast<char *>(f.data) + rhs * bytes;
    return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, (int)bytes, 0x00027000);  // (raw buffer, checked range)
}
template <int P, typename R>
__device__ __forceinline__ void st_shared_elem(BufRsrc f, int stride, int e, int i, const Cx<R> *x) {
    u32x4 v;
    if constexpr (P == P64) {
        dvec2 d;
        d.x = x[0].re;
        d.y = x[0].im;
        v = __builtin_bit_cast(u32x4, d);
    } else {
        fvec4 d;
        d.x = x[0].re;
        d.y = x[0].im;
        d.z = x[1].re;
        d.w = x[1].im;
        v = __builtin_bit_cast(u32x4, d);
    }
    __builtin_amdgcn_raw_buffer_store_b128(v, f, i * 16, e * stride * 16, kSc1);
}
// site j of an exchanged field; half: the spin half a t-hop needs (-1: all)
template <int P, typename R>
__device__ __forceinline__ void ld_shared_site(Cx<R> (&v)[12], BufRsrc f, int stride, int j, int half) {
    constexpr int CPE = SpinorPack<P>::CPE;
#pragma unroll
    for (int e = 0; e < SpinorPack<P>::NEL; e++) {
        if (half < 0 || (e * CPE >= 6 * half && e * CPE < 6 * half + 6)) {
            const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(f, j * 16, e * stride * 16, kSc1);
            if constexpr (P == P64) {
                const dvec2 d = __builtin_bit_cast(dvec2, w);
                v[e] = {d.x, d.y};
            } else {
                const fvec4 d = __builtin_bit_cast(fvec4, w);
                v[2 * e] = {d.x, d.y};
                v[2 * e + 1] = {d.z, d.w};
            }
        } else {
#pragma unroll
            for (int k = 0; k < CPE; k++) v[e * CPE + k] = {R(0), R(0)};
        }
    }
}

// Barrier over the `tiles` blocks that share *cnt, the n-th: false if the wait gave up.  The
// counter is compared modulo 2^32.
__device__ __forceinline__ bool tiles_barrier(unsigned *cnt, unsigned n, int tiles, unsigned spins, int *ok) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's exchanged stores are done
    __syncthreads();
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned target = n * (unsigned)tiles;
        unsigned polls = 0;
        int good = 1;
        while ((int)(__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) < 0)
            if (++polls > spins) {
                good = 0;
                break;
            }
        *ok = good;
    }
    __syncthreads();
    return *ok != 0;
}

// Sum of n <= kPreFinMax values val(j) by one wave, in the order of wave_sum_fixed.
template <typename F>
__device__ __forceinline__ double wave_sum_of(int n, F &&val) {
    static_assert(kPreFinMax <= 128, "two values per lane");
    const int lane = (int)threadIdx.x & 63;
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < 2; u++) {
        const int j = lane + u * 64;
        if (j < n) acc[u] += val(j);
    }
    double v = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return 0.0 + v;
}

// Sums of N values over a wave (every lane gets them), step by step across the values: the
// exchanges of one value's butterfly depend on each other, those of different values do not.
template <int N>
__device__ __forceinline__ void wave_sums(double (&v)[N]) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        double o[N];
#pragma unroll
        for (int k = 0; k < N; k++) o[k] = __shfl_xor(v[k], off, 64);
#pragma unroll
        for (int k = 0; k < N; k++) v[k] += o[k];
    }
}

// The epilogue's view of one hop (hop_put; what the launched kernel branches on stays a run-time
// value, so that the compiler forms the same multiply-adds).
struct TileHop {
    double cH[1];
    int has_y, red;
    static constexpr int has_z = 0, g5out = 0, nostore = 0, clov_mode = CLV_NONE;
    static constexpr double cz = 0.0;
    static constexpr const void *clov = nullptr;
    Spinor y, z, w;  // (never read: the operands are handed over)
};

struct NoSource {  // (hop_dir loads nothing itself: neighbours and links are handed over)
    Spinor in;
    const void *gauge;
};

// What wave mu of a block needs for one parity's hop along mu: the neighbours' indices, the
// two links with all nine entries (the third row of a two-row link rebuilt as hop_dir does),
// the boundary signs.
template <typename R>
struct DirSite {
    int jf, jb;
    R sf, sb;
    Cx<R> uf[9], ub[9];
};
template <int GP, int NE, typename R>
__device__ __forceinline__ void dir_link(Cx<R> (&u)[9], const Geom &g, const void *gauge, int plane, int site) {
    constexpr int NL = LinkElems<GP, NE>::N, CPL = LinkPack<GP>::CPL;
    Cx<R> ue[NL * CPL], U[3][3];
#pragma unroll
    for (int e = 0; e < NL; e++)
        ld_link_elem<GP, R, false>(&ue[e * CPL], lplane<GP>(gauge, plane * NL + e, g.stride), (unsigned)site * LinkPack<GP>::EB);
#pragma unroll
    for (int e = 0; e < NE; e++) U[e / 3][e % 3] = ue[e];
    if constexpr (NE == 6) {
        const Cx<R> c0 = csub(cmul(U[0][1], U[1][2]), cmul(U[0][2], U[1][1]));
        const Cx<R> c1 = csub(cmul(U[0][2], U[1][0]), cmul(U[0][0], U[1][2]));
        const Cx<R> c2 = csub(cmul(U[0][0], U[1][1]), cmul(U[0][1], U[1][0]));
        U[2][0] = {c0.re, -c0.im};
        U[2][1] = {c1.re, -c1.im};
        U[2][2] = {c2.re, -c2.im};
    }
#pragma unroll
    for (int e = 0; e < 9; e++) u[e] = U[e / 3][e % 3];
}
template <int GP, int NE, typename R>
__device__ __forceinline__ void dir_site(DirSite<R> &d, const Geom &g, const void *gauge, int par, int i, int mu) {
    const SiteXY c = cb_coords(g, i, par);
    const SiteNbrs nb = site_nbrs(g, i, c);
    d.jf = mu == 0 ? nb.xp : (mu == 1 ? nb.yp : (mu == 2 ? nb.zp : nb.tp));
    d.jb = mu == 0 ? nb.xm : (mu == 1 ? nb.ym : (mu == 2 ? nb.zm : nb.tm));
    d.sf = mu == 3 && NE == 6 && c.t == g.L[3] - 1 ? R(-1) : R(1);
    d.sb = mu == 3 && NE == 6 && c.t == 0 ? R(-1) : R(1);
    dir_link<GP, NE, R>(d.uf, g, gauge, par * 4 + mu, i);
    dir_link<GP, NE, R>(d.ub, g, gauge, (1 - par) * 4 + mu, d.jb);
}

// Both hops along MU at the wave's sites, neighbours from an exchanged field.
template <int SP, int GP, int NE, int MU>
__device__ __forceinline__ void tile_dir(Cx<real_t<SP>> (&acc)[1][4][3], BufRsrc in, int stride,
                                         const DirSite<real_t<SP>> &d) {
    using R = real_t<SP>;
    const bool act[1] = {true};
    const NoSource none = {};
    Cx<R> vf[12], vb[12], H[1][2][3];
    ld_shared_site<SP, R>(vf, in, stride, d.jf, MU == 3 ? 1 : -1);
    ld_shared_site<SP, R>(vb, in, stride, d.jb, MU == 3 ? 0 : -1);
    proj_in<SP, MU, true, false>(vf, R(1), H[0]);
    hop_dir<SP, GP, 1, NE, false, false, MU, true, 2, false, 0>(acc, none, act, 0, 0, 0, 0, d.sf, stride, H, nullptr, d.uf);
    proj_in<SP, MU, false, false>(vb, R(1), H[0]);
    hop_dir<SP, GP, 1, NE, false, false, MU, false, 2, false, 0>(acc, none, act, 0, 0, 0, 0, d.sb, stride, H, nullptr, d.ub);
}

// One parity hop of the block's tile: wave mu gathers direction mu into part, wave 0 adds them
// and hands each site's sum to put(acc).  Holds one block barrier.
template <int SP, int GP, int NE, typename PUT>
__device__ __forceinline__ void tile_hop(real_t<SP> (&part)[4][24][64], BufRsrc in, int stride,
                                         const DirSite<real_t<SP>> &d, int wv, int lane, PUT &&put) {
    using R = real_t<SP>;
    {
        Cx<R> acc[1][4][3];
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int k = 0; k < 3; k++) acc[0][s][k] = {R(0), R(0)};
        if (wv == 0) tile_dir<SP, GP, NE, 0>(acc, in, stride, d);
        else if (wv == 1) tile_dir<SP, GP, NE, 1>(acc, in, stride, d);
        else if (wv == 2) tile_dir<SP, GP, NE, 2>(acc, in, stride, d);
        else tile_dir<SP, GP, NE, 3>(acc, in, stride, d);
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int k = 0; k < 3; k++) {
                part[wv][2 * (s * 3 + k)][lane] = acc[0][s][k].re;
                part[wv][2 * (s * 3 + k) + 1][lane] = acc[0][s][k].im;
            }
    }
    __syncthreads();
    if (wv == 0) {
        Cx<R> acc[4][3];
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const int e = 2 * (s * 3 + k);
                acc[s][k] = {((part[0][e][lane] + part[1][e][lane]) + part[2][e][lane]) + part[3][e][lane],
                             ((part[0][e + 1][lane] + part[1][e + 1][lane]) + part[2][e + 1][lane]) + part[3][e + 1][lane]};
            }
        put(acc);
    }
}

template <int SP, int GP, int NE>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(1, 1)))
bicg_small_kernel(const SmallArgs p) {
    using R = real_t<SP>;
    constexpr int CPE = SpinorPack<SP>::CPE, NEL = SpinorPack<SP>::NEL;
    constexpr int EPW = (NEL + kWaves - 1) / kWaves;  // elements of a site per wave: e = wv + kWaves q
    const Geom &g = p.g;
    const int stride = g.stride, tiles = p.tiles;
    const int rhs = blockIdx.x / tiles, tile = blockIdx.x - rhs * tiles;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    const bool valid = tile * 64 + lane < g.Vh;
    const int i = valid ? tile * 64 + lane : g.Vh - 1;

    __shared__ R part[4][24][64];
    __shared__ Cx<R> ysh[12][64];  // the block's own p or s, by component
    __shared__ RhsState loc;       // the state, kept alike by every block of the right-hand side
    __shared__ double sums[3];
    __shared__ int ok;

    // exchanged scalars of this right-hand side: the barrier counter, then partial sums
    char *scr = p.scratch + (size_t)rhs * p.scratch_stride;
    unsigned *cnt = reinterpret_cast<unsigned *>(scr);
    double *hp = reinterpret_cast<double *>(scr + 256);  // hops: [3][tiles]
    double *sp = hp + 3 * tiles;                         // s update: [NEL][tiles]
    double *xp = sp + NEL * tiles;                       // x/r update: [3][NEL][tiles]

    if (threadIdx.x == 0) loc = p.state[rhs];
    __syncthreads();
    if (!(loc.phase & PH_RUN)) return;  // all blocks of the right-hand side alike

    Cx<R> r[EPW][CPE], rh[EPW][CPE], x[EPW][CPE], pp[EPW][CPE], v[EPW][CPE], s[EPW][CPE], t[EPW][CPE];
#pragma unroll
    for (int q = 0; q < EPW; q++) {
        const int e = wv + kWaves * q;
#pragma unroll
        for (int k = 0; k < CPE; k++) pp[q][k] = v[q][k] = s[q][k] = t[q][k] = {R(0), R(0)};
        if (e >= NEL) continue;
        const unsigned off = (unsigned)i * 16u;
        ld_elem<SP, R>(r[q], splane(p.r.data, rhs * NEL + e, stride), off);
        ld_elem<SP, R>(rh[q], splane(p.rh.data, rhs * NEL + e, stride), off);
        ld_elem<SP, R>(x[q], splane(p.x.data, rhs * NEL + e, stride), off);
        if (!p.first) {
            ld_elem<SP, R>(pp[q], splane(p.p.data, rhs * NEL + e, stride), off);
            ld_elem<SP, R>(v[q], splane(p.v.data, rhs * NEL + e, stride), off);
        }
    }
    const BufRsrc fp = shared_field<SP>(p.p, stride, rhs), fs = shared_field<SP>(p.s, stride, rhs),
                  ft = shared_field<SP>(p.tmp, stride, rhs);
    DirSite<R> dir[2];  // the hops onto odd and even sites
    dir_site<GP, NE, R>(dir[0], g, p.gauge, 1, i, wv);
    dir_site<GP, NE, R>(dir[1], g, p.gauge, 0, i, wv);
    unsigned nbar = 0;
    const int nbs = (g.Vh + 1023) / 1024, nblas = NEL * nbs;  // the vector kernels' partial rows

    // partial j of a vector kernel: element j / nbs, 1024 sites = 16 tiles, added in order
    auto blas_row = [&](const double *src) {
        return wave_sum_of(nblas, [&](int j) {
            const int e = j / nbs, t0 = (j - e * nbs) * 16;
            double w[16];
#pragma unroll
            for (int k = 0; k < 16; k++) w[k] = t0 + k < tiles ? ld_agent_d(src + e * tiles + t0 + k) : 0.0;
            double a = 0.0;
#pragma unroll
            for (int k = 0; k < 16; k++) a += w[k];
            return a;
        });
    };
    auto hop_row = [&](int k) { return wave_sum_of(tiles, [&](int j) { return ld_agent_d(hp + k * tiles + j); }); };
    // A scalar step on up to three sums: wave k adds row k, thread 0 steps the state.  Holds two
    // block barriers; the state is the new one after it.
    auto step = [&](int op, int n, auto &&row) {
        if (wv < n) {
            const double a = row(wv);
            if (lane == 0) sums[wv] = a;
        }
        __syncthreads();
        if (threadIdx.x == 0) fin_op_rt(op, &loc, sums[0], n > 1 ? sums[1] : 0.0, n > 2 ? sums[2] : 0.0);
        __syncthreads();
    };
    auto own = [&](Cx<R> (&f)[EPW][CPE]) {
#pragma unroll
        for (int q = 0; q < EPW; q++) {
            const int e = wv + kWaves * q;
            if (e < NEL)
#pragma unroll
                for (int k = 0; k < CPE; k++)
                    f[q][k] = {part[0][2 * (e * CPE + k)][lane], part[0][2 * (e * CPE + k) + 1][lane]};
        }
    };

    bool good = true;
    for (int it = 0; it < p.iters; it++) {
        // Two half steps of the same form: a vector update, M on its result, a scalar.  (Loops, not
        // two copies: the code of the gathers is what fills the instruction cache.)
#pragma unroll 1
        for (int half = 0; half < 2; half++) {
            const bool first = half == 0;
            if (first) {  // p = r + beta (p - omega v)
                const Cx<R> beta = {(R)loc.beta_re, (R)loc.beta_im}, omega = {(R)loc.omega_re, (R)loc.omega_im};
#pragma unroll
                for (int q = 0; q < EPW; q++) {
                    const int e = wv + kWaves * q;
                    if (e >= NEL) continue;
#pragma unroll
                    for (int k = 0; k < CPE; k++) {
                        pp[q][k] = nc::add(r[q][k], nc::mul(beta, nc::sub(pp[q][k], nc::mul(omega, v[q][k]))));
                        ysh[e * CPE + k][lane] = pp[q][k];
                    }
                    if (valid) st_shared_elem<SP, R>(fp, stride, e, i, pp[q]);
                }
            } else {  // s = r - alpha v, |s|^2
                const Cx<R> alpha = {(R)loc.alpha_re, (R)loc.alpha_im};
                double red[EPW];
#pragma unroll
                for (int q = 0; q < EPW; q++) {
                    const int e = wv + kWaves * q;
                    red[q] = 0.0;
                    if (e >= NEL) continue;
#pragma unroll
                    for (int k = 0; k < CPE; k++) {
                        s[q][k] = nc::sub(r[q][k], nc::mul(alpha, v[q][k]));
                        red[q] += nc::norm2(s[q][k]);
                        ysh[e * CPE + k][lane] = s[q][k];
                    }
                    if (valid) st_shared_elem<SP, R>(fs, stride, e, i, s[q]);
                    else red[q] = 0.0;
                }
                wave_sums(red);
#pragma unroll
                for (int q = 0; q < EPW; q++)
                    if (lane == 0 && wv + kWaves * q < NEL) st_agent_d(sp + (wv + kWaves * q) * tiles + tile, red[q]);
            }
            if (!(good = tiles_barrier(cnt, ++nbar, tiles, p.spins, &ok))) break;
            if (!first) {
                step(FIN_BICG_S, 1, [&](int) { return blas_row(sp); });
                if (!(loc.phase & PH_RUN)) break;  // |s| small enough: x += alpha p and stop
            }
            // v = M p with <rhat, v>, or t = M s with <t, s> and |t|^2: the odd hop into tmp, then
            // the even one into part[0] (each lane of wave 0 overwrites the column it has summed)
            TileHop a = {};
            Cx<R> wd[12];
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const BufRsrc in = h == 0 ? (first ? fp : fs) : ft;
                int odd = h;  // (opaque: the epilogue keeps its branches)
                asm volatile("" : "+s"(odd));
                a.cH[0] = odd ? p.cH[rhs] : 1.0;
                a.has_y = odd;
                a.red = odd ? (first ? RED_DOT : RED_TS) : RED_NONE;
                if (wv == 0 && h == 1 && first) load_site<SP, R>(wd, p.rh, stride, rhs, i);
                tile_hop<SP, GP, NE>(part, in, stride, dir[h], wv, lane, [&](const Cx<R> (&acc)[4][3]) {
                    Cx<R> yv[12], zv[12];
#pragma unroll
                    for (int k = 0; k < 12; k++) yv[k] = ysh[k][lane];
                    double rd[3] = {0.0, 0.0, 0.0};
                    hop_put<SP, false, 7, false>(a, i, valid, 0, acc, yv, zv, wd, rd, stride, [&](const Cx<R> (&o)[12]) {
                        if (h == 0) {
#pragma unroll
                            for (int e = 0; e < NEL; e++) st_shared_elem<SP, R>(ft, stride, e, i, &o[e * CPE]);
                        } else {
#pragma unroll
                            for (int k = 0; k < 12; k++) {
                                part[0][2 * k][lane] = o[k].re;
                                part[0][2 * k + 1][lane] = o[k].im;
                            }
                        }
                    });
                    if (h == 1) {
                        wave_sums(rd);
                        if (lane < 3) st_agent_d(hp + lane * tiles + tile, lane == 0 ? rd[0] : (lane == 1 ? rd[1] : rd[2]));
                    }
                });
                if (!(good = tiles_barrier(cnt, ++nbar, tiles, p.spins, &ok))) break;
            }
            if (!good) break;
            if (first) own(v);
            else own(t);
            step(first ? FIN_BICG_ALPHA : FIN_BICG_OMEGA, first ? 2 : 3, hop_row);
            if (!(loc.phase & PH_RUN)) break;
        }
        if (!good) break;
        if (!(loc.phase & (PH_RUN | PH_SCONV))) break;
        {   // x += alpha p + omega s; r = s - omega t; |r|^2, <rhat, r>
            const Cx<R> alpha = {(R)loc.alpha_re, (R)loc.alpha_im}, omega = {(R)loc.omega_re, (R)loc.omega_im};
            double all[3 * EPW];
#pragma unroll
            for (int q = 0; q < EPW; q++) {
                const int e = wv + kWaves * q;
                double red[3] = {0.0, 0.0, 0.0};
                if (e < NEL) {
#pragma unroll
                    for (int k = 0; k < CPE; k++) {
                        x[q][k] = nc::add(x[q][k], nc::add(nc::mul(alpha, pp[q][k]), nc::mul(omega, s[q][k])));
                        r[q][k] = (loc.phase & PH_SCONV) ? s[q][k] : nc::sub(s[q][k], nc::mul(omega, t[q][k]));
                        nc::dot(red, rh[q][k], r[q][k]);
                    }
                }
#pragma unroll
                for (int k = 0; k < 3; k++) all[3 * q + k] = valid ? red[k] : 0.0;
            }
            wave_sums(all);
#pragma unroll
            for (int q = 0; q < EPW; q++)
#pragma unroll
                for (int k = 0; k < 3; k++)
                    if (lane == 0 && wv + kWaves * q < NEL)
                        st_agent_d(xp + (k * NEL + wv + kWaves * q) * tiles + tile, all[3 * q + k]);
        }
        if (!(good = tiles_barrier(cnt, ++nbar, tiles, p.spins, &ok))) break;
        step(FIN_BICG_RHO, 3, [&](int k) { return blas_row(xp + k * NEL * tiles); });
        if (!(loc.phase & PH_RUN)) break;
    }
    const bool more = good && (loc.phase & PH_RUN);  // stopped by the iteration count: another launch goes on
#pragma unroll
    for (int q = 0; q < EPW; q++) {
        const int e = wv + kWaves * q;
        if (e >= NEL || !valid) continue;
        const unsigned off = (unsigned)i * 16u;
        st_elem<SP, R>(const_cast<gchar *>(splane(p.x.data, rhs * NEL + e, stride)), off, x[q]);
        if (more) {
            st_elem<SP, R>(const_cast<gchar *>(splane(p.r.data, rhs * NEL + e, stride)), off, r[q]);
            st_elem<SP, R>(const_cast<gchar *>(splane(p.p.data, rhs * NEL + e, stride)), off, pp[q]);
            st_elem<SP, R>(const_cast<gchar *>(splane(p.v.data, rhs * NEL + e, stride)), off, v[q]);
        }
    }
    if (threadIdx.x == 0) {
        RhsState *st = &p.state[rhs];
        if (!good) {
            __hip_atomic_store(&st->lost, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if (tile == 0) {  // every field but `lost`
            static_assert(offsetof(RhsState, phase) == 14 * sizeof(double) && offsetof(RhsState, lost) == 14 * sizeof(double) + 12);
            for (int k = 0; k < 14; k++) (&st->rho_re)[k] = (&loc.rho_re)[k];
            st->phase = loc.phase;
            st->fail = loc.fail;
            st->iter = loc.iter;
        }
    }
}

template <int P>
const void *small_kernel(int recon) {
    return recon == 12 ? reinterpret_cast<const void *>(bicg_small_kernel<P, P, 6>)
                       : reinterpret_cast<const void *>(bicg_small_kernel<P, P, 9>);
}
const void *small_kernel(int prec, int recon) {
    if (recon != 12 && recon != 18) return nullptr;
    return prec == P64 ? small_kernel<P64>(recon) : (prec == P32 ? small_kernel<P32>(recon) : nullptr);
}

}  // namespace

size_t small_scratch_bytes(const Geom &g, int prec) {
    const size_t tiles = (g.Vh + 63) / 64, nel = prec == P64 ? 12 : 6;
    return 256 + (3 + 4 * nel) * tiles * sizeof(double);
}

int small_max_blocks(int prec, int recon) {
    const void *k = small_kernel(prec, recon);
    int dev = 0, cus = 0, per = 0;
    if (!k || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k, 64 * kWaves, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return per > 0 ? cus : 0;  // (one per CU: blocks of several such kernels can then be placed in any mix)
}

hipError_t launch_bicg_small(const SmallArgs &p, int prec, int recon, hipStream_t s) {
    const void *k = small_kernel(prec, recon);
    const int nb = (prec == P64 ? 12 : 6) * ((p.g.Vh + 1023) / 1024);
    if (!k || p.tiles != (p.g.Vh + 63) / 64 || p.tiles > kPreFinMax || nb > kPreFinMax || p.nrhs < 1 || p.nrhs > kMaxRhs ||
        p.iters < 1 || p.spins < 1 || p.scratch_stride < small_scratch_bytes(p.g, prec))
        return hipErrorInvalidValue;
    SmallArgs a = p;
    void *args[] = {&a};
    const hipError_t e = hipLaunchKernel(k, dim3(p.tiles * p.nrhs), dim3(64 * kWaves), args, 0, s);
    if (e != hipSuccess) (void)hipGetLastError();  // (a refusal must not be reported by a later call)
    return e;
}

}  // namespace wl
