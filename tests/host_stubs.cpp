// Stand-ins for the HIP runtime and the kernel launchers, for running the library's host code
// (dispatch, solve control, failure handling) without a GPU: device memory is host memory,
// launches are recorded and do only what the host reads back (states, norms).  Linked with the
// real runtime.cpp, solver.cpp, capi.cpp and dslash.hip by test_host_dispatch.py, which runs one
// scenario per process.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include "common.h"
#include "layout_lab.h"
#include "runtime.h"
#include "solver.h"
#include "wilson.h"

using namespace wl;

// ---- what the launches leave behind ----------------------------------------------------
static std::map<std::string, int> count;        // launches by name
static std::function<void(const HopArgs &, const LaunchCfg &)> on_hop;
static std::function<hipError_t(const SmallArgs &)> on_small;
static std::function<bool(const LaunchCfg &)> favourite;  // the shape that times best
static LaunchCfg last_cfg;
static bool iterated = false;                   // an iteration or a one-launch solve has run
static bool su3 = true;                         // what the check of links finds
static double residual = 0.0;                   // norms stored once that is so
static size_t allocated = 0, limit = ~size_t(0);
static std::map<void *, size_t> blocks;

// ---- HIP runtime -----------------------------------------------------------------------
extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    if (allocated + n > limit) return hipErrorOutOfMemory;
    count["malloc"]++;
    *p = std::calloc(1, n);
    blocks[*p] = n;
    allocated += n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    allocated -= blocks[p];
    blocks.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned) { return hipErrorNotSupported; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = favourite && favourite(last_cfg) ? 0.1f : 1.f;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorName(hipError_t) { return "error"; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static void *scratch = std::aligned_alloc(256, size_t(256) << 20);  // (touched only where the host reads)
    *p = scratch;
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    for (const auto &b : blocks)
        if (p >= b.first && p < static_cast<char *>(b.first) + b.second) {
            a->type = hipMemoryTypeDevice;
            return hipSuccess;
        }
    return hipErrorInvalidValue;
}
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
}

// ---- kernel launchers ------------------------------------------------------------------
namespace wl {
#define RECORD(name) (count[name]++, hipSuccess)
template <int SP, int GP>
hipError_t launch_hop_r(const HopArgs &a, const LaunchCfg &c, hipStream_t) {
    last_cfg = c;
    if (on_hop) on_hop(a, c);
    return RECORD("hop");
}
template hipError_t launch_hop_r<P64, P64>(const HopArgs &, const LaunchCfg &, hipStream_t);
template hipError_t launch_hop_r<P32, P32>(const HopArgs &, const LaunchCfg &, hipStream_t);
template hipError_t launch_hop_r<P16, P16>(const HopArgs &, const LaunchCfg &, hipStream_t);
template hipError_t launch_hop_r<P16, P32>(const HopArgs &, const LaunchCfg &, hipStream_t);
hipError_t launch_dslash_full(const FullArgs &, hipStream_t) { return RECORD("full"); }
hipError_t launch_dslash_small(const FullArgs &, int, hipStream_t) { return RECORD("small"); }
hipError_t launch_dslash_rhs(const FullArgs &, int, int, hipStream_t) { return RECORD("rhs"); }
hipError_t launch_split(Spinor, Spinor, const double *, const Geom &, int, hipStream_t, double *) { return RECORD("split"); }
hipError_t launch_split_one(Spinor, const double *, const Geom &, int, int, hipStream_t) { return RECORD("split_one"); }
hipError_t launch_join(double *, Spinor, Spinor, const Geom &, int, hipStream_t) { return RECORD("join"); }
hipError_t launch_join_one(double *, Spinor, const Geom &, int, int, hipStream_t) { return RECORD("join_one"); }
int split_nblocks(const Geom &g) { return (g.Vh + 127) / 128; }
hipError_t launch_convert(Spinor, Spinor, const Geom &, int, const RhsState *, int, hipStream_t) { return RECORD("convert"); }
hipError_t launch_axpy_f64(Spinor, Spinor, const Geom &, int, const RhsState *, int, hipStream_t) { return RECORD("axpy"); }
hipError_t launch_zero(const Spinor &, const Geom &, int, hipStream_t) { return RECORD("zero"); }
hipError_t launch_gauge_pack(void *const[3], const double *, const Geom &, int, hipStream_t) { return RECORD("pack"); }
hipError_t launch_su3_check(const double *, size_t, double, int *flag, hipStream_t) {
    if (!su3) *flag = 1;
    return RECORD("check");
}
hipError_t launch_clover_pack(void *, void *, void *, void *, const double *, const Geom &, double, int *, hipStream_t) { return RECORD("clover_pack"); }
hipError_t launch_clover_apply(Spinor, Spinor, const void *, const Geom &, int, hipStream_t) { return RECORD("clover"); }
hipError_t launch_block_gram(BlockArgs, int, hipStream_t) { return RECORD("gram"); }
hipError_t launch_block_solve(int, BlockArgs, hipStream_t) { return RECORD("block_solve"); }
hipError_t launch_block_update(int, BlockArgs, hipStream_t) { return RECORD("block_update"); }
size_t block_partials_doubles(const Geom &) { return 64; }
hipError_t launch_stream_copy(void *, const void *, size_t, hipStream_t) { return hipSuccess; }
hipError_t launch_stream_read(const void *, size_t, unsigned *, hipStream_t) { return hipSuccess; }
int blas_nblocks(const Geom &g, int prec) { return prec == P16 ? (g.Vh + 255) / 256 : (prec == P64 ? 12 : 6) * ((g.Vh + 1023) / 1024); }
hipError_t launch_blas(int op, const BlasArgs &a, hipStream_t) {
    if (a.pre.on)
        for (int k = 0; k < a.nrhs; k++) a.pre.dst[k] = a.pre.src[k];
    return RECORD(op == BL_START ? "start" : "blas");
}
hipError_t launch_init_states(RhsState *st, const StateInit &in, hipStream_t) {
    for (int k = 0; k < in.n; k++) {
        st[k] = RhsState();
        st[k].phase = in.phase[k];
        st[k].stop2 = in.stop2[k];
    }
    return RECORD("states");
}
hipError_t launch_finalize(int op, const double *, int, int, int nrhs, RhsState *st, int mask, hipStream_t, RhsState *mirror) {
    for (int k = 0; k < nrhs; k++) {
        if (st[k].phase & mask) {
            if (op == FIN_STORE_AUX) st[k].aux = iterated ? residual : 1.0;
            if (op == FIN_BICG_RHO || op == FIN_CG_R) {
                st[k].iter++;
                st[k].phase = PH_DONE;
                iterated = true;
            }
        }
        if (mirror) mirror[k] = st[k];
    }
    return RECORD("finalize");
}
int small_max_blocks(int, int) { return 256; }
size_t small_scratch_bytes(const Geom &, int) { return 0; }
hipError_t launch_bicg_small(const SmallArgs &a, int, int, hipStream_t) {
    count["one_launch"]++;
    return on_small ? on_small(a) : hipErrorInvalidValue;
}
// (the layout ablation is not exercised)
bool lab_geom(LabGeom &, const int32_t *, int) { return false; }
size_t lab_spinor_bytes(const LabGeom &, int) { return 0; }
size_t lab_link_bytes(const LabGeom &, int, int) { return 0; }
hipError_t launch_lab_zero(double *, size_t, hipStream_t) { return hipSuccess; }
hipError_t launch_lab_pack_links(void *, const double *, const LabGeom &, int, int, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_lab_pack_spinor(void *, const double *, const LabGeom &, int, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_lab_unpack_spinor(double *, const void *, const LabGeom &, int, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_lab_hop(void *, const void *, const void *, const void *, const LabGeom &, int, int, int, int, double, hipStream_t) { return hipSuccess; }
long long index_check(const int32_t[4], std::string &) { return 0; }
}  // namespace wl

// ---- scenarios -------------------------------------------------------------------------
#define EXPECT(x) \
    do { if (!(x)) { std::printf("line %d: %s is false\n", __LINE__, #x); std::exit(1); } } while (0)

// a device buffer of n doubles
static double *device(size_t n) {
    void *p = nullptr;
    EXPECT(hipMalloc(&p, n * sizeof(double)) == hipSuccess);
    return static_cast<double *>(p);
}
struct Problem {
    int32_t dims[4];
    wilson_ctx *ctx = nullptr;
    wilson_gauge *g = nullptr;
    double *in = nullptr, *out = nullptr;
    size_t V;
    Problem(int x, int y, int z, int t, int nrhs = 1) : dims{x, y, z, t}, V((size_t)x * y * z * t) {
        EXPECT(wilson_context_create(&ctx, nullptr) == WILSON_OK);
        double *U = device(72 * V);
        EXPECT(wilson_gauge_load(ctx, &g, U, dims, WILSON_GAUGE_FP32 | WILSON_GAUGE_FP16) == WILSON_OK);
        hipFree(U);
        in = device(24 * V * nrhs);
        out = device(24 * V * nrhs);
        count.clear();
    }
    int solve(wilson_solve_info *info, int precision = WILSON_FP64, int use_x0 = 0) {
        const double kappa = 0.12, tol = 1e-8;
        wilson_solve_opts o = {};
        o.precision = precision;
        o.maxiter = 100;
        o.use_x0 = use_x0;
        count.clear();
        iterated = false;
        return wilson_solve_ex(ctx, g, out, in, 1, &kappa, &tol, &o, info);
    }
    int dslash(int parity, int precision, int nrhs = 1) {
        count.clear();
        return wilson_dslash_ex(ctx, g, out, in, 0.12, parity, precision, nrhs);
    }
};

// FP32 and FP16 results must not change with the kernel: where the tuned hop adds the directions
// in another order than the kernels that write the canonical layout, one right-hand side keeps
// to the hop as several do.
static void operator_order() {
    for (const bool split : {true, false}) {
        favourite = [&](const LaunchCfg &c) { return split ? c.dsplit == 1 : (!c.dsplit && !c.tm); };
        Problem p(8, 8, 16, split ? 16 : 32);
        for (int precision : {WILSON_FP32, WILSON_FP16, WILSON_FP16_L32})
            for (int nrhs : {1, 2}) {
                double *two = device(24 * p.V * 2), *res = device(24 * p.V * 2);
                EXPECT(wilson_dslash_ex(p.ctx, p.g, res, two, 0.12, 2, precision, nrhs) == WILSON_OK);  // (tunes)
                count.clear();
                EXPECT(wilson_dslash_ex(p.ctx, p.g, res, two, 0.12, 2, precision, nrhs) == WILSON_OK);
                EXPECT(count["hop"] == (split ? 2 : 0));
                EXPECT(count["full"] + count["rhs"] == (split ? 0 : nrhs == 1 ? 1 : 2));
                hipFree(two);
                hipFree(res);
            }
        EXPECT(p.dslash(2, WILSON_FP64) == WILSON_OK);  // FP64 always takes its own kernel
        EXPECT(count["hop"] == 0 && count["full"] + count["small"] == 1);
    }
    favourite = [](const LaunchCfg &c) { return c.ldsl == 2; };  // FP16 links rebuilt and rounded again
    Problem p(8, 8, 16, 32, 12);
    for (int precision : {WILSON_FP32, WILSON_FP16, WILSON_FP16_L32}) {
        EXPECT(p.dslash(1, precision, 12) == WILSON_OK);
        EXPECT(p.dslash(1, precision, 12) == WILSON_OK);
        EXPECT(count["hop"] == (precision == WILSON_FP16) && count["rhs"] == (precision != WILSON_FP16));
    }
}

// A one-launch solve that is refused, or whose blocks lose each other (also where the state looks
// finished), goes on in the separate launches, and the context stays with them.
static void one_launch_lost() {
    wilson_solve_info info;
    for (const int how : {0, 1, 2})
        for (const int precision : {WILSON_FP64, WILSON_FP32}) {
            Problem p(8, 8, 8, 8);
            on_small = [&](const SmallArgs &a) {
                if (how == 1) return hipErrorCooperativeLaunchTooLarge;
                a.state[0].phase = PH_DONE;
                a.state[0].iter = 5;
                a.state[0].lost = how == 2;
                iterated = how == 0;
                return hipSuccess;
            };
            EXPECT(p.solve(&info, precision) == WILSON_OK && info.converged);
            EXPECT(count["one_launch"] == 1);
            EXPECT(info.iterations == (how == 0 ? 5 : 1));
            EXPECT((count["blas"] > 0) == (how != 0));
            EXPECT(p.solve(&info, precision, 1) == WILSON_OK);
            EXPECT(count["one_launch"] == (how == 0 ? 1 : 0));
        }
}

// WILSON_ONE_LAUNCH=0
static void one_launch_off() {
    wilson_solve_info info;
    Problem p(8, 8, 8, 8);
    EXPECT(p.solve(&info) == WILSON_OK && info.converged);
    EXPECT(count["one_launch"] == 0 && count["blas"] > 0);
}

// One-launch solves in flight in several contexts share the device's room: what does not fit takes
// the separate launches, and the room comes back.
static void one_launch_room() {
    favourite = [](const LaunchCfg &c) { return c.dsplit == 1; };
    Problem a(8, 8, 16, 16), b(8, 8, 16, 16), c(4, 4, 4, 4);  // 128, 128 and 1 blocks of 256
    std::vector<Problem *> next;
    int total = 0;
    on_small = [&](const SmallArgs &s) {
        total++;
        if (!next.empty()) {  // (while this one is in flight)
            Problem *p = next.back();
            next.pop_back();
            wilson_solve_info info;
            EXPECT(p->solve(&info) == WILSON_OK);
        }
        s.state[0].phase = PH_DONE;
        iterated = true;
        return hipSuccess;
    };
    for (int round = 0; round < 2; round++) {
        wilson_solve_info info;
        total = 0;
        next = {&c, &b};
        EXPECT(a.solve(&info) == WILSON_OK);
        EXPECT(next.empty() && total == 2);
        total = 0;
        next = {&c};
        EXPECT(b.solve(&info) == WILSON_OK);
        EXPECT(next.empty() && total == 2);
    }
}

// A load makes each buffer once, of the size that its links need, whether they are SU(3) or not.
static void load_allocates_once() {
    for (const bool exact : {true, false}) {
        su3 = exact;
        Problem p(8, 8, 8, 16);
        double *U = device(72 * p.V);
        wilson_gauge *g = nullptr;
        count.clear();
        const size_t before = allocated;
        EXPECT(wilson_gauge_load(p.ctx, &g, U, p.dims, WILSON_GAUGE_FP32 | WILSON_GAUGE_FP16) == WILSON_OK);
        EXPECT(count["malloc"] == 3 && count["pack"] == 1 && count["check"] == 1);
        EXPECT(allocated - before == wilson_gauge_bytes(g));
        EXPECT(wilson_gauge_bytes(g) == wilson_gauge_footprint_bytes(p.dims, 7, exact ? 12 : 18));
    }
}

// Another thread's context tunes the shape of a running solve that may not tune itself, between any
// two of its hops: the solve succeeds.
static void shape_changes() {
    favourite = [](const LaunchCfg &c) { return c.block == 64; };
    wilson_solve_info info;
    Problem p(8, 8, 16, 32);
    TuneTable &T = tune_table();
    EXPECT(p.solve(&info) == WILSON_OK && T.cfg.size() == 1);
    const auto tuned = *T.cfg.begin();
    EXPECT(tuned.second.block == 64);
    const double kappa = 0.12, tol = 1e-8;
    for (int at = 0, hops = 1; at < hops; at++) {
        T.cfg.clear();
        Problem q(8, 8, 16, 32);
        iterated = false;
        hops = 0;
        on_hop = [&](const HopArgs &, const LaunchCfg &) {
            if (hops++ == at) T.cfg.insert(tuned);
        };
        const int st = wilson_solve_noalloc(q.ctx, q.g, q.out, q.in, 1, &kappa, &tol, nullptr, &info);
        if (st != WILSON_OK) std::printf("tuned at hop %d: %s\n", at, wilson_last_error());
        EXPECT(st == WILSON_OK);
        EXPECT(hops > 6 && info.converged);
        on_hop = nullptr;
    }
}

// What the hop class times is the solvers' hop, in every form of the operator call and in solves
// that would otherwise take one launch.
static void timed_calls() {
    for (const int z : {8, 32}) {
        Problem p(8, 8, 8, z, 5);
        for (const bool timed : {false, true}) {
            EXPECT(wilson_timing_enable(p.ctx, timed) == WILSON_OK);
            for (int parity = 0; parity < 3; parity++)
                for (const int precision : {WILSON_FP64, WILSON_FP32, WILSON_FP16, WILSON_FP16_L32})
                    for (const int nrhs : {1, 2, 5}) {
                        EXPECT(p.dslash(parity, precision, nrhs) == WILSON_OK);  // (may tune)
                        double ms, bytes;
                        int64_t n0, n1;
                        EXPECT(wilson_timing_read(p.ctx, WILSON_KERNEL_HOP, &ms, &n0, &bytes) == WILSON_OK);
                        EXPECT(p.dslash(parity, precision, nrhs) == WILSON_OK);
                        EXPECT(wilson_timing_read(p.ctx, WILSON_KERNEL_HOP, &ms, &n1, &bytes) == WILSON_OK);
                        if (!timed) continue;
                        EXPECT(count["hop"] == (parity == 2 ? 2 : 1) && n1 - n0 == count["hop"]);
                        EXPECT(count["small"] + count["full"] + count["rhs"] == 0);
                    }
        }
        wilson_solve_info info;
        EXPECT(p.solve(&info) == WILSON_OK && count["one_launch"] == 0);
    }
}

// What the plain calls keep on the device: links and planes of one shape, nothing of a large one; and
// a later plain call gets the planes' memory if it does not fit otherwise, any other call both.
static void plain_memory() {
    const int32_t small[4] = {16, 16, 16, 16}, large[4] = {32, 32, 32, 64};
    const size_t V = 16 * 16 * 16 * 16, VL = 32 * 32 * 32 * 64, links = 576 * V, planes = 384 * V;
    double *U = device(72 * VL), *in = device(24 * VL), *out = device(24 * VL);
    const size_t base = allocated;
    EXPECT(wilson_dslash(out, in, U, 0.1, large, 2) == WILSON_OK);
    EXPECT(allocated == base);
    EXPECT(wilson_dslash(out, in, U, 0.1, small, 2) == WILSON_OK);
    EXPECT(allocated == base + links + planes);
    limit = base + links + wilson_footprint_bytes(small, 1, nullptr);
    iterated = false;
    EXPECT(wilson_solve(out, in, U, 0.1, small, 1e-8, 100) == WILSON_OK);
    EXPECT(allocated == limit);
    EXPECT(wilson_dslash(out, in, U, 0.1, small, 2) == WILSON_OUT_OF_MEMORY);  // (the solve's workspace stays)
    limit = ~size_t(0);
    EXPECT(wilson_dslash(out, in, U, 0.1, small, 2) == WILSON_OK);
    wilson_ctx *ctx = nullptr;
    wilson_gauge *g = nullptr;
    EXPECT(wilson_context_create(&ctx, nullptr) == WILSON_OK);
    limit = allocated;
    EXPECT(wilson_gauge_load(ctx, &g, U, small, 0) == WILSON_OK);  // takes what the plain calls hold
    limit = ~size_t(0);
    count.clear();
    EXPECT(wilson_dslash(out, in, U, 0.1, small, 2) == WILSON_OK && count["pack"] == 1);
}

int main(int argc, char **argv) {
    const std::map<std::string, void (*)()> all = {{"operator_order", operator_order},
                                                   {"one_launch_lost", one_launch_lost},
                                                   {"one_launch_off", one_launch_off},
                                                   {"one_launch_room", one_launch_room},
                                                   {"load_allocates_once", load_allocates_once},
                                                   {"shape_changes", shape_changes},
                                                   {"timed_calls", timed_calls},
                                                   {"plain_memory", plain_memory}};
    const auto it = all.find(argc > 1 ? argv[1] : "");
    if (it == all.end()) return 2;
    it->second();
    std::printf("ok\n");
    return 0;
}
