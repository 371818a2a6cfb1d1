// Batched energy+gradient and the persistent L-BFGS minimiser (gfx950).
//
// Energy: Eq. (1) of Carmona et al.; minimiser: the paper's L-BFGS-B with no
// active bounds, i.e. L-BFGS (two-loop recursion of Nocedal & Wright,
// Alg. 7.4) with a per-atom step cap and a backtracking Armijo line search
// (Algorithm Overview, step 2).
//
// One workgroup ("team", W wavefronts) owns one cluster at a time and runs
// its whole minimisation on chip: coordinates are staged in LDS for the pair
// loop, all reductions go through wavefront butterflies and (for W > 1) a
// small LDS exchange, and for N <= 256 the m (s, y) history pairs stay in
// registers.  Teams are persistent: they claim clusters from a queue that
// lists the batch by N descending (longest first), one launch per size class
// (the size classes run concurrently on side streams).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lj_lbfgs.hpp"

namespace lj {

constexpr int kHybridRegs = 5;

// ---------------------------------------------------------------------------
// Persistent minimiser kernel: one launch per size class.  A workgroup claims
// the next cluster of its class from the queue (G > 1: the next G clusters,
// one per packed team of 64 / G lanes) and minimises it; it claims again once
// all of its teams are done.
// ---------------------------------------------------------------------------
template <int MIXED, int W, int A, bool HREG, int POT, int L = kWave, int G = 1, int OCC = 1,
          bool TILES = kUseTiles<W, A>>
__global__ __launch_bounds__(kWave* W) __attribute__((amdgpu_waves_per_eu(OCC))) void minimize_kernel(
    MinArgs args) {
    constexpr int T = kWave * W;
    constexpr int LG = kWave / G;  // lanes of a packed team
    __shared__ double4 pos_buf[T * A];
    __shared__ TeamScratch<W, 4 * A> scratch;
    __shared__ int claim;
    __shared__ float tile_rbuf[(MIXED && G == 1 &&
                                ((POT == kPairLJ && TILES) || (W == 1 && A == 1)))
                                   ? 6 * T * A
                                   : 1];

    // one-wavefront, one-cluster Morse kernels at one wavefront per SIMD take
    // the unique-pair FP64 evaluation, with its matrix in dynamic LDS (for
    // Eq. (1) the ordered loop is as fast: its pair terms are too cheap to
    // pay for the matrix's LDS traffic)
    constexpr bool kUp = W == 1 && A == 1 && G == 1 && OCC == 1 && POT == kPairMorse;
    extern __shared__ double2 up_matrix[];
    const int team = G > 1 ? (int)threadIdx.x / LG : 0;
    Team<W, A, POT, L, G, kUp, TILES> tm;
    tm.upm = up_matrix;
    tm.up_n = kUp ? args.up_n : 0;
    tm.uplist = reinterpret_cast<uint2*>(up_matrix + (size_t)tm.up_n * tm.up_n);
    tm.li = G > 1 ? (int)threadIdx.x % LG : (int)threadIdx.x;
    tm.pos64 = pos_buf + team * LG;
    tm.pos32 = reinterpret_cast<float4*>(pos_buf) + team * LG;
    tm.rbuf = tile_rbuf;
    tm.sc = &scratch;
    tm.bank = 0;
    tm.rho = args.rho;
    tm.top = POT == kPairMorse ? (uint32_t)uniform((int)morse_top(args.rho)) : 0u;
    // kernels at two wavefronts per SIMD whose registers do not hold the history
    // keep half of it in LDS
    constexpr bool kHybrid = HREG && A == 1 && G == 1 && OCC == 2 && (MIXED || W > 1);
    typename std::conditional<kHybrid, HistoryHybrid<W, kHybridRegs>, History<W, A, HREG>>::type H;
    __shared__ double hist_uniform[HREG ? 1 : 2 * kMaxM];  // rho and alpha of a history in memory
    __shared__ __align__(16) char hist_ring[kHybrid ? HistoryHybrid<W, kHybridRegs>::kBytes : 16];
    if constexpr (kHybrid) {
        H.init(hist_ring);
    } else {
        constexpr size_t kHistPerWG = (size_t)2 * kMaxM * 3 * A * T;
        H.init(args.hist ? args.hist + kHistPerWG * blockIdx.x : nullptr, hist_uniform, args.p.m);
    }

    const int start = args.plan.cls[args.cls];
    const int count = args.plan.cls[kNumClasses + args.cls];
    for (;;) {
        if (threadIdx.x == 0) claim = atomicAdd(&args.plan.queue[args.cls], G);
        __syncthreads();
        const int idx0 = claim;
        __syncthreads();
        if (idx0 >= count) break;
        const int idx = idx0 + team;
        const bool has = idx < count;  // a packed team past the end idles
        const int b = has ? args.plan.list[start + idx] : 0;
        const int o = has ? args.offset[b] : 0;
        const int n = has ? args.offset[b + 1] - o : 0;
        tm.n = n;  // the plan guarantees 0 <= n <= T*A (G > 1: <= 64 / G)
        tm.prepare();

        minimize_cluster<MIXED, A>(args, tm, H, b, o, n, has);
    }
}

// ---------------------------------------------------------------------------
// Plan: list the (active) clusters by N descending and split the list into
// size classes.  One workgroup; rejects clusters whose N is outside
// [0, max_n] with a per-cluster status instead of running them.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void plan_kernel(const int32_t* offset, int num, int max_n,
                                                    const int32_t* active, Plan plan,
                                                    int32_t* status) {
    __shared__ int cnt[LJ_MAX_ATOMS_MIN + 1];
    const int t = threadIdx.x;
    for (int k = t; k <= LJ_MAX_ATOMS_MIN; k += blockDim.x) cnt[k] = 0;
    __syncthreads();
    for (int b = t; b < num; b += blockDim.x) {
        if (active && !active[b]) continue;
        const int n = offset[b + 1] - offset[b];
        if (n < 0 || n > max_n) {
            if (status) status[b] = kStatusBadSize;
            continue;
        }
        atomicAdd(&cnt[n], 1);
    }
    __syncthreads();
    if (t == 0) {
        // descending exclusive scan of the size counts; sizes above max_n were
        // rejected, so their counts (and scan values) are zero: start at max_n
        const int top = max_n < LJ_MAX_ATOMS_MIN ? max_n : LJ_MAX_ATOMS_MIN;
        int run = 0;
        for (int k = top; k >= 0; --k) {
            const int c = cnt[k];
            cnt[k] = run;
            run += c;
        }
        // classes: (256, 1024], (128, 256], (64, 128], [0, 64]
        const int s3 = 0, s2 = cnt[256], s1 = cnt[128], s0 = cnt[64];
        plan.cls[3] = s3;
        plan.cls[2] = s2;
        plan.cls[1] = s1;
        plan.cls[0] = s0;
        plan.cls[kNumClasses + 3] = s2 - s3;
        plan.cls[kNumClasses + 2] = s1 - s2;
        plan.cls[kNumClasses + 1] = s0 - s1;
        plan.cls[kNumClasses + 0] = run - s0;
        for (int c = 0; c < kNumClasses; ++c) plan.queue[c] = 0;
    }
    __syncthreads();
    for (int b = t; b < num; b += blockDim.x) {
        if (active && !active[b]) continue;
        const int n = offset[b + 1] - offset[b];
        if (n < 0 || n > max_n) continue;
        const int pos = atomicAdd(&cnt[n], 1);
        plan.list[pos] = b;
    }
}

// ---------------------------------------------------------------------------
// Batched energy + gradient: one workgroup per cluster.
// ---------------------------------------------------------------------------
template <int MIXED, int W, int A, int POT>
__global__ __launch_bounds__(kWave* W) void energy_grad_kernel(const int32_t* offset, int64_t total,
                                                               const double* xyz, double* energy,
                                                               double* grad, double rho, Units u) {
    constexpr int T = kWave * W;
    __shared__ double4 pos_buf[T * A];
    __shared__ TeamScratch<W, 4 * A> scratch;
    __shared__ float tile_rbuf[(MIXED && ((POT == kPairLJ && kUseTiles<W, A>) || (W == 1 && A == 1)))
                                   ? 6 * T * A
                                   : 1];
    const int b = blockIdx.x;
    const int o = offset[b];
    const int n = offset[b + 1] - o;
    if (n < 0 || n > T * A) {  // offsets disagree with the host max_n
        if (threadIdx.x == 0) energy[b] = __builtin_nan("");
        return;
    }
    Team<W, A, POT> tm;
    tm.upm = nullptr;
    tm.uplist = nullptr;
    tm.up_n = 0;
    tm.pos64 = pos_buf;
    tm.pos32 = reinterpret_cast<float4*>(pos_buf);
    tm.rbuf = tile_rbuf;
    tm.sc = &scratch;
    tm.bank = 0;
    tm.n = n;
    tm.li = threadIdx.x;
    tm.rho = rho;
    tm.top = POT == kPairMorse ? (uint32_t)uniform((int)morse_top(rho)) : 0u;
    double x[3][A], g[3][A];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const int i = a * T + threadIdx.x;
            x[c][a] = i < n ? xyz[c * total + o + i] : 0.0;
            if (u.scaled) x[c][a] = x[c][a] / u.sigma;
        }
    const double E = tm.template eval<MIXED != 0>(x, g);
    if (threadIdx.x == 0) energy[b] = E * u.escale;
    if (grad) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int a = 0; a < A; ++a) {
                const int i = a * T + threadIdx.x;
                if (i < n) grad[c * total + o + i] = g[c][a] * u.gscale;
            }
    }
}

// ---------------------------------------------------------------------------
// Host-side launchers (internal C++ interface used by the C ABI layer).
// ---------------------------------------------------------------------------
EvalShape eval_shape(int max_n) {
    const int n = max_n < 1 ? 1 : max_n;
    if (n <= 64) return {1, 1};
    if (n <= 128) return {2, 1};
    if (n <= 256) return {4, 1};
    if (n <= 512) return {8, 1};
    if (n <= 1024) return {16, 1};
    if (n <= 2048) return {16, 2};
    return {16, 4};
}

bool eval_shape_supported(EvalShape s) {
    const bool w = s.W == 1 || s.W == 2 || s.W == 4 || s.W == 8 || s.W == 16;
    const bool a = s.A == 1 || s.A == 2 || s.A == 4;
    return w && a;
}

template <int MIXED, int POT>
static hipError_t launch_eval_t(EvalShape s, int num, const int32_t* off, int64_t total,
                                const double* xyz, double* e, double* g, double rho, Units u,
                                hipStream_t st) {
    dim3 grid(num), block(kWave * s.W);
#define LJ_EVAL_CASE(WW, AA)                                                                  \
    if (s.W == WW && s.A == AA) {                                                             \
        hipLaunchKernelGGL((energy_grad_kernel<MIXED, WW, AA, POT>), grid, block, 0, st, off, \
                           total, xyz, e, g, rho, u);                                         \
        return hipGetLastError();                                                             \
    }
    LJ_EVAL_CASE(1, 1)
    LJ_EVAL_CASE(2, 1)
    LJ_EVAL_CASE(4, 1)
    LJ_EVAL_CASE(8, 1)
    LJ_EVAL_CASE(16, 1)
    LJ_EVAL_CASE(1, 2)
    LJ_EVAL_CASE(2, 2)
    LJ_EVAL_CASE(4, 2)
    LJ_EVAL_CASE(8, 2)
    LJ_EVAL_CASE(16, 2)
    LJ_EVAL_CASE(1, 4)
    LJ_EVAL_CASE(2, 4)
    LJ_EVAL_CASE(4, 4)
    LJ_EVAL_CASE(8, 4)
    LJ_EVAL_CASE(16, 4)
#undef LJ_EVAL_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_energy_grad(int mixed, int pot, EvalShape s, int num, const int32_t* off,
                              int64_t total, const double* xyz, double* e, double* g, double rho,
                              Units u, hipStream_t st) {
    if (pot == kPairMorse)
        return mixed ? launch_eval_t<1, kPairMorse>(s, num, off, total, xyz, e, g, rho, u, st)
                     : launch_eval_t<0, kPairMorse>(s, num, off, total, xyz, e, g, rho, u, st);
    return mixed ? launch_eval_t<1, kPairLJ>(s, num, off, total, xyz, e, g, rho, u, st)
                 : launch_eval_t<0, kPairLJ>(s, num, off, total, xyz, e, g, rho, u, st);
}

// Minimiser shapes.  Classes 0-2 keep the history in registers; class 3
// (N in 257..1024) keeps it in a global ring.  Each class has interchangeable
// shapes (the schedule table or the built-in rule picks one per call):
//   class 0 (N <= 64):   0  one wavefront per cluster
//                        1  one wavefront, reductions over one 16-lane row
//                           (N <= 16)
//                        2  two clusters per wavefront, 32 lanes each (N <= 32)
//                        3  four clusters per wavefront, 16 lanes each (N <= 16)
//                        4-7  shapes 0-3 compiled for two wavefronts per SIMD (at
//                           most 256 registers; mixed 4 and 5 keep half of the
//                           history in LDS, mixed 6 and 7 spill 39 registers,
//                           Morse 63): for batches of more wavefronts than SIMDs
//   class 1 (N <= 128):  0  two wavefronts;  1  the same with FP32 pairs summed
//                           in the ordered loop
//   class 2 (N <= 256):  0  four wavefronts;  1  three wavefronts (N <= 192)
//                        (classes 1 and 2: compiled for one and for two
//                        wavefronts per SIMD, kDenseShape added to the number)
//   class 3 (N <= 1024): 0  16 wavefronts x 1 atom, 1  8 x 2, 2  4 x 4
struct ClassShape {
    int W, A;
    bool hreg;
    int G;     // clusters per workgroup
    int max_n; // largest cluster the shape holds
};
constexpr int kMaxShapes = 8;
constexpr int kShapes[kNumClasses] = {8, 2, 2, 3};
constexpr ClassShape kShape[kNumClasses][kMaxShapes] = {
    {{1, 1, true, 1, 64}, {1, 1, true, 1, 16}, {1, 1, true, 2, 32}, {1, 1, true, 4, 16},
     {1, 1, true, 1, 64}, {1, 1, true, 1, 16}, {1, 1, true, 2, 32}, {1, 1, true, 4, 16}},
    {{2, 1, true, 1, 128}, {2, 1, true, 1, 128}},
    {{4, 1, true, 1, 256}, {3, 1, true, 1, 192}},
    {{16, 1, false, 1, 1024}, {8, 2, false, 1, 1024}, {4, 4, false, 1, 1024}}};

int class_shapes(int c) { return c >= 0 && c < kNumClasses ? kShapes[c] : 0; }
static const ClassShape& shape_of(int c, int shape) { return kShape[c][shape & ~kDenseShape]; }
int shape_max_n(int c, int shape) {
    return is_relay(shape) ? kClassMaxN[c] : shape_of(c, shape).max_n;
}
int shape_clusters_per_wg(int c, int shape) {
    return is_relay(shape) ? 1 : shape_of(c, shape).G;
}

int class_of(int n) {
    for (int c = 0; c < kNumClasses; ++c)
        if (n <= kClassMaxN[c]) return c;
    return -1;
}

size_t class_hist_bytes_per_wg(int c, int shape) {
    if (is_relay(shape)) return 0;
    const ClassShape s = shape_of(c, shape);
    return s.hreg ? 0 : (size_t)2 * kMaxM * 3 * s.A * kWave * s.W * sizeof(double);
}

template <int MIXED, int W, int A, bool HREG, int POT, int L = kWave, int G = 1, int OCC = 1,
          bool TILES = kUseTiles<W, A>>
static const void* min_kernel_ptr() {
    return reinterpret_cast<const void*>(
        &minimize_kernel<MIXED, W, A, HREG, POT, L, G, OCC, TILES>);
}

template <int MIXED, int POT>
static const void* minimize_kernel_pm(int c, int shape) {
    if (shape & kDenseShape) {
        switch (c * kMaxShapes + (shape & ~kDenseShape)) {
            case kMaxShapes + 0: return min_kernel_ptr<MIXED, 2, 1, true, POT, kWave, 1, 2>();
            case kMaxShapes + 1:
                return min_kernel_ptr<MIXED, 2, 1, true, POT, kWave, 1, 2, MIXED == 0>();
            case 2 * kMaxShapes + 0: return min_kernel_ptr<MIXED, 4, 1, true, POT, kWave, 1, 2>();
            case 2 * kMaxShapes + 1: return min_kernel_ptr<MIXED, 3, 1, true, POT, kWave, 1, 2>();
        }
        return nullptr;
    }
    switch (c * kMaxShapes + shape) {
        case 0: return min_kernel_ptr<MIXED, 1, 1, true, POT>();
        case 1: return min_kernel_ptr<MIXED, 1, 1, true, POT, 16>();
        case 2: return min_kernel_ptr<MIXED, 1, 1, true, POT, kWave, 2>();
        case 3: return min_kernel_ptr<MIXED, 1, 1, true, POT, kWave, 4>();
        case 4: return min_kernel_ptr<MIXED, 1, 1, true, POT, kWave, 1, 2>();
        case 5: return min_kernel_ptr<MIXED, 1, 1, true, POT, 16, 1, 2>();
        case 6: return min_kernel_ptr<MIXED, 1, 1, true, POT, kWave, 2, 2>();
        case 7: return min_kernel_ptr<MIXED, 1, 1, true, POT, kWave, 4, 2>();
        case kMaxShapes + 0: return min_kernel_ptr<MIXED, 2, 1, true, POT>();
        case kMaxShapes + 1:
            return min_kernel_ptr<MIXED, 2, 1, true, POT, kWave, 1, 1, MIXED == 0>();
        case 2 * kMaxShapes + 0: return min_kernel_ptr<MIXED, 4, 1, true, POT>();
        case 2 * kMaxShapes + 1: return min_kernel_ptr<MIXED, 3, 1, true, POT>();
        case 3 * kMaxShapes + 0: return min_kernel_ptr<MIXED, 16, 1, false, POT>();
        case 3 * kMaxShapes + 1: return min_kernel_ptr<MIXED, 8, 2, false, POT>();
        case 3 * kMaxShapes + 2: return min_kernel_ptr<MIXED, 4, 4, false, POT>();
    }
    return nullptr;
}

const void* minimize_kernel_for(int mixed, int pot, int c, int shape) {
    if (is_relay(shape)) return relay_kernel_for(mixed, pot, c, shape);
    if (c < 0 || c >= kNumClasses || shape < 0 || (shape & ~kDenseShape) >= kShapes[c])
        return nullptr;
    if (pot == kPairMorse)
        return mixed ? minimize_kernel_pm<1, kPairMorse>(c, shape)
                     : minimize_kernel_pm<0, kPairMorse>(c, shape);
    return mixed ? minimize_kernel_pm<1, kPairLJ>(c, shape) : minimize_kernel_pm<0, kPairLJ>(c, shape);
}

int class_block(int c, int shape) {
    return is_relay(shape) ? relay_block(shape) : kWave * shape_of(c, shape).W;
}

int class_up_n(int c, int shape, int max_n, int pot) {
    if (pot != kPairMorse || c < 0 || c >= kNumClasses || shape < 0 || shape >= kShapes[c])
        return 0;
    const ClassShape s = kShape[c][shape];
    // the one-wavefront, one-cluster shapes at one wavefront per SIMD
    if (!(s.W == 1 && s.A == 1 && s.G == 1 && !(c == 0 && shape >= 4))) return 0;
    int n = max_n < s.max_n ? max_n : s.max_n;
    if (n > kUpMaxN) n = kUpMaxN;
    return n >= 2 ? n : 0;
}

size_t class_dyn_lds(int c, int shape, int max_n, int pot) {
    const size_t n = (size_t)class_up_n(c, shape, max_n, pot);
    return n * n * sizeof(double2) + n * (n > 0 ? n - 1 : 0) / 2 * sizeof(uint2);
}

hipError_t launch_plan(const int32_t* offset, int num, int max_n, const int32_t* active, Plan plan,
                       int32_t* status, hipStream_t st) {
    hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(1024), 0, st, offset, num, max_n, active, plan,
                       status);
    return hipGetLastError();
}

hipError_t launch_minimize_class(int mixed, int c, int shape, int grid, const MinArgs& a,
                                 hipStream_t st) {
    const void* k = minimize_kernel_for(mixed, a.pot, c, shape);
    if (!k) return hipErrorInvalidValue;
    MinArgs b = a;
    b.up_n = class_up_n(c, shape, a.max_n, a.pot);
    void* args[] = {&b};
    return hipLaunchKernel(k, dim3(grid), dim3(class_block(c, shape)), args,
                           class_dyn_lds(c, shape, a.max_n, a.pot), st);
}

}  // namespace lj
