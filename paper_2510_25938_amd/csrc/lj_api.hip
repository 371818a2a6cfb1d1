// C ABI of liblj_bh.so: argument validation, workspace layout, launch
// scheduling and the HIP-graph cache of the basin-hopping step.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "lj_kernels.hpp"

namespace {

thread_local std::string g_err;

lj_status fail(lj_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return s;
}

#define LJ_HIP_TRY(expr)                                                                   \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess)                                                              \
            return fail(LJ_E_HIP, "%s failed: %s", #expr, hipGetErrorString(e_));         \
    } while (0)

struct DeviceInfo {
    bool valid = false;
    bool gfx950 = false;
    int cus = 0;
};

std::mutex g_dev_mu;
std::vector<DeviceInfo> g_dev;

lj_status device_info(DeviceInfo& out) {
    int dev = 0;
    LJ_HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_dev_mu);
    if ((int)g_dev.size() <= dev) g_dev.resize(dev + 1);
    if (!g_dev[dev].valid) {
        hipDeviceProp_t prop;
        LJ_HIP_TRY(hipGetDeviceProperties(&prop, dev));
        g_dev[dev].cus = prop.multiProcessorCount;
        g_dev[dev].gfx950 = std::strncmp(prop.gcnArchName, "gfx950", 6) == 0;
        g_dev[dev].valid = true;
    }
    out = g_dev[dev];
    if (!out.gfx950) return fail(LJ_E_UNSUPPORTED, "device %d is not gfx950", dev);
    return LJ_OK;
}

lj_status check_batch(const lj_batch* b, int limit, const char* what) {
    if (!b) return fail(LJ_E_ARG, "%s: batch is NULL", what);
    if (b->num < 0) return fail(LJ_E_ARG, "%s: num = %d < 0", what, b->num);
    if (b->num > 0 && !b->offset) return fail(LJ_E_ARG, "%s: offset is NULL", what);
    if (b->max_n < 0) return fail(LJ_E_ARG, "%s: max_n = %d < 0", what, b->max_n);
    if (b->max_n > limit)
        return fail(LJ_E_UNSUPPORTED, "%s: max_n = %d exceeds the limit %d", what, b->max_n, limit);
    if (b->total_atoms < 0 || b->total_atoms > INT32_MAX)
        return fail(LJ_E_ARG, "%s: total_atoms = %lld out of range", what,
                    (long long)b->total_atoms);
    if ((int64_t)b->num * b->max_n < b->total_atoms)
        return fail(LJ_E_ARG, "%s: total_atoms exceeds num * max_n", what);
    if (b->pair != LJ_PAIR_LJ && b->pair != LJ_PAIR_MORSE)
        return fail(LJ_E_ARG, "%s: pair = %d is neither LJ_PAIR_LJ nor LJ_PAIR_MORSE", what,
                    b->pair);
    if (b->pair == LJ_PAIR_MORSE && !(b->pair_rho > 0.0 && b->pair_rho <= 1.0e6))
        return fail(LJ_E_ARG, "%s: Morse pair_rho = %g is not in (0, 1e6]", what, b->pair_rho);
    if (!(b->sigma == 0.0 || (b->sigma > 0.0 && std::isfinite(b->sigma))) ||
        !(b->epsilon == 0.0 || (b->epsilon > 0.0 && std::isfinite(b->epsilon))))
        return fail(LJ_E_ARG, "%s: sigma = %g and epsilon = %g must be finite and > 0 (or 0 for 1)",
                    what, b->sigma, b->epsilon);
    return LJ_OK;
}

// The batch's units; a zero sigma or epsilon means 1.
lj::Units units_of(const lj_batch* b) {
    const double sg = b->sigma == 0.0 ? 1.0 : b->sigma;
    const double ep = b->epsilon == 0.0 ? 1.0 : b->epsilon;
    return lj::Units{sg, ep, ep / sg, sg != 1.0};
}

bool reduced_units(const lj_batch* b) {
    const lj::Units u = units_of(b);
    return u.sigma == 1.0 && u.escale == 1.0;
}

lj_status check_params(const lj_lbfgs_params* p) {
    if (!p) return fail(LJ_E_ARG, "params is NULL");
    if (p->m < 0 || p->m > LJ_MAX_M) return fail(LJ_E_ARG, "m = %d outside [0, %d]", p->m, LJ_MAX_M);
    if (!(p->gtol > 0.0)) return fail(LJ_E_ARG, "gtol must be > 0");
    if (p->max_iter < 0) return fail(LJ_E_ARG, "max_iter < 0");
    if (!(p->max_step > 0.0)) return fail(LJ_E_ARG, "max_step must be > 0");
    if (!(p->c1 > 0.0 && p->c1 < 1.0)) return fail(LJ_E_ARG, "c1 must be in (0, 1)");
    if (p->max_ls < 1) return fail(LJ_E_ARG, "max_ls must be >= 1");
    if (!(p->curv_eps >= 0.0)) return fail(LJ_E_ARG, "curv_eps must be >= 0");
    if (!(p->gtol_mixed_per_atom >= 0.0)) return fail(LJ_E_ARG, "gtol_mixed_per_atom < 0");
    if (!(p->ls_noise >= 0.0)) return fail(LJ_E_ARG, "ls_noise < 0");
    return LJ_OK;
}

lj::LbfgsDev to_dev(const lj_lbfgs_params* p) {
    lj::LbfgsDev d;
    d.m = p->m;
    d.gtol = p->gtol;
    d.max_iter = p->max_iter;
    d.max_step = p->max_step;
    d.c1 = p->c1;
    d.max_ls = p->max_ls;
    d.curv_eps = p->curv_eps;
    d.gtol_mixed_per_atom = p->gtol_mixed_per_atom;
    d.polish = p->polish;
    d.ls_noise = p->ls_noise;
    return d;
}

constexpr size_t kAlign = 256;
size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// Launch-schedule table, filled by lj_autotune / lj_set_schedule.  Keys:
// eval: (precision, next_pow2(max_n)); large minimiser: (precision).
std::mutex g_sched_mu;
std::map<std::pair<int, int>, lj::EvalShape> g_eval_sched;
int g_large_sched[2] = {1, 0};  // FP64: 8 x 2 (no spills); mixed: 16 x 1 (tiled FP32 loop)

int pow2_at_least(int n) {
    int p = 1;
    while (p < n) p *= 2;
    return p;
}

lj::EvalShape eval_schedule(int precision, int max_n) {
    std::lock_guard<std::mutex> lk(g_sched_mu);
    auto it = g_eval_sched.find({precision, pow2_at_least(max_n < 1 ? 1 : max_n)});
    if (it != g_eval_sched.end() && it->second.W * 64 * it->second.A >= max_n) return it->second;
    return lj::eval_shape(max_n);
}

// Scratch bytes of the evaluation spread over many workgroups, 0 where one
// workgroup per cluster is the faster.  nt: 64-atom tiles of the largest cluster.
//   FP64   one workgroup per tile, a round of the chip for every `cus` tiles,
//          1.7 us per 64 partners and round (Morse pair 2.7), against 4.6, 6.4, 12
//          and 23 us per 64 partners at nt = 4, 8, 16 and 32 with one workgroup
//          (Morse 12, 13, 25, 49).  Up to a third as many rounds as nt the
//          spread is the faster at every size: at the limit 102 x LJ300 26
//          instead of 34 us, 96 x LJ500 53 and 55, 93 x LJ700 93 and 105, 80 x
//          LJ1000 156 and 191, 85 x LJ1500 355 and 415, 84 x LJ4096 2426 and
//          2998; Morse 41 and 66, 87 and 107, 151 and 215, 259 and 400, 579 and
//          884, 4020 and 6783; one cluster of 1000 beside 1050 of 13 atoms 160
//          and 189.  Up to 256 atoms the second launch costs what the split saves
//          (8 x LJ256: 19.0 instead of 18.9 us).
//   FP32   one wavefront per unit (a pair of tiles), 2.6 ns each and three
//          launches (18 us), against 0.32 nt^2 us: 64 x LJ500 23.0 instead of
//          27.8 us, 128 28.1 instead of 28.7; 128 x LJ1000 64.9 instead of
//          90.3 us.  At most 40000 units; the scratch holds those of a power
//          of two of tiles per cluster, since a cluster above max_n is evaluated
//          if it fits the launch shape: at most 169 MB (173 x 1344 atoms).
size_t split_rule_ws(const lj_batch* b, int precision, int cus) {
    const int mixed = precision == LJ_MIXED;
    if (b->max_n <= 256) return 0;
    const long nt = (b->max_n + 63) / 64;
    if (!mixed) {
        const long tiles = std::min((long)b->num * nt, (long)(b->total_atoms / 64) + b->num);
        const long rounds = (tiles + cus - 1) / cus;
        if (3 * rounds > nt + 1) return 0;
    } else {
        const long units = (long)b->num * lj::split_units(b->pair, (int)nt);
        if (units > std::min(100 * nt * nt - 4000, 40000L)) return 0;
    }
    return lj::split_eval_bytes(mixed, b->pair, b->num, b->max_n);
}

// Whether two shapes of clusters above 256 atoms give the same bits: FP64 has one
// summation order, and the FP32 Morse pair too, while Eq. (1) in FP32 has two
// (64-atom tiles or the ordered loop).
bool same_eval_bits(int mixed, int pot, lj::EvalShape s, lj::EvalShape d) {
    return !mixed || pot == LJ_PAIR_MORSE || lj::use_tiles(s.W, s.A) == lj::use_tiles(d.W, d.A);
}

// The same for a call.  The schedule table's shape is that of one workgroup per
// cluster, and its key has no cluster count: an entry tuned on many clusters says
// nothing of a few, and only one whose sums have another order keeps a call from
// being spread (one LJ1000: 36 us spread, 189 us by one workgroup).
size_t split_eval_ws(const lj_batch* b, int precision, int cus) {
    if (b->max_n <= 256 ||
        !same_eval_bits(precision == LJ_MIXED, b->pair, eval_schedule(precision, b->max_n),
                        lj::eval_shape(b->max_n)))
        return 0;
    return split_rule_ws(b, precision, cus);
}

int large_schedule(int precision) {
    std::lock_guard<std::mutex> lk(g_sched_mu);
    return g_large_sched[precision == LJ_MIXED ? 1 : 0];
}

// Minimiser shapes of classes 0-2, filled by lj_autotune / lj_set_schedule:
// (precision, class, largest class of the batch, power of two >= the class's
// largest N) -> shape.
std::map<std::array<int, 4>, int> g_class_sched;

// The largest N that class c can hold in a batch whose largest N is max_n.
int class_cap(int c, int max_n) {
    const int cap = lj::kClassMaxN[c];
    return max_n < cap ? (max_n < 0 ? 0 : max_n) : cap;
}

std::array<int, 4> class_key(int precision, int c, int max_n) {
    return {precision == LJ_MIXED ? 1 : 0, c, lj::class_of(max_n < 0 ? 0 : max_n),
            pow2_at_least(class_cap(c, max_n) < 1 ? 1 : class_cap(c, max_n))};
}

// The calls that the built-in rule expects beside one another on the device: the
// caller streams that made two or more of the last eight larger minimisations (or
// four, the device's hardware queues, where four or more streams made them).  One
// call on another stream does not count.  Basin-hopping steps run on a stream
// because the null stream cannot be captured, often one per chain set and in turn,
// and chains are batched into one call: they are taken to be alone.  Helper
// wavefronts take SIMDs that a call by itself leaves idle but that calls on other
// streams would fill, so their limits are divided by
// that number; calls of up to a quarter of the CUs fit beside three like them and
// are not counted.  Only a choice among forms with the same results depends on it.
// Measured, ms for 1, 2 and 4 calls at once, without / with helper wavefronts: 1024 x
// LJ38 2.9, 3.8, 5.9 / 2.7, 4.1, 7.1; 512 x LJ38 2.9, 3.6, 4.6 / 2.5, 3.5, 6.4; 256 x
// LJ98 12.9, 28.9, 18.5 / 10.4, 23.1, 27.1; 512 x Morse38 4.4, 4.4, 5.9 / 3.5, 4.7,
// 8.6; but at a quarter of the limits 128 x LJ38 2.9 (2), 5.7 (4) / 2.2, 4.2; 128 x
// LJ20 1.28, 1.36 / 1.22, 1.26; 64 x LJ98 11.5, 11.6 / 9.2, 9.4; 128 x Morse32 2.35,
// 2.74 / 2.31, 2.61; 64 of 20..120 atoms 12.3, 25.2 / 9.9, 18.4.  Asking events whether
// other calls are still in flight instead let the first calls of every burst
// take the chip (4 x 256 x LJ98 22.0 ms).
constexpr int kRecentCalls = 8;
struct RecentCalls {
    hipStream_t stream[kRecentCalls];
    int count = 0, at = 0;
};
std::mutex g_recent_mu;
std::vector<RecentCalls> g_recent;  // per device

// note: the call of num clusters is about to be enqueued on st.  A call under
// capture says nothing of when it will run: it is taken to be alone.
int calls_at_once(hipStream_t st, int num, int cus, bool note) {
    if (num <= cus / 4) return 1;  // within a quarter of every limit
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 1;
    if (st && (hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone))
        return 1;
    std::lock_guard<std::mutex> lk(g_recent_mu);
    if ((int)g_recent.size() <= dev) g_recent.resize(dev + 1);
    RecentCalls& r = g_recent[dev];
    if (note) {
        r.stream[r.at] = st;
        r.at = (r.at + 1) % kRecentCalls;
        r.count = std::min(r.count + 1, kRecentCalls);
    }
    std::map<hipStream_t, int> made;
    made[st] += 2;
    for (int k = 0; k < r.count; ++k) ++made[r.stream[k]];
    if (made.size() >= 4) return 4;
    int calls = 0;
    for (const auto& m : made) calls += m.second >= 2;
    return calls;
}

// Built-in rule for the shape of class c (0-2); mean: the batch's mean size,
// calls: calls_at_once.
int default_class_shape(int c, int max_n, int top_class, int mixed, int pot, int num, double mean,
                        int cus, int calls) {
    const int cmax = class_cap(c, max_n);
    // Helper wavefronts (FP64) while every cluster's workgroup is resident at
    // once, so that they run on SIMDs which would idle.  Four wavefronts per
    // cluster: two workgroups per CU for class 0 by itself, one for class 1 or
    // beside other classes.  8 x LJ38: 1.71 instead of 2.14 ms, 512 x LJ38 2.45
    // instead of 2.82 ms, 640 x LJ38 3.22 instead of 2.80 ms (hence the limit);
    // 8 x LJ98 7.3 instead of 8.9 ms, 384 x LJ98 17.3 instead of 15.4 ms.  For the
    // Morse pair, whose other kernel evaluates unique pairs up to 40 atoms, from 32
    // atoms on (400 x Morse24 1.67 instead of 1.48 ms, 8 x Morse28 1.31 instead
    // of 1.27, 8 x Morse38 2.33 instead of 2.77, 512 x Morse38 3.32 instead of 3.42,
    // 256 x Morse98 15.3 instead of 20.5).
    // Two wavefronts per cluster (Eq. (1), class 0 by itself) up to one cluster
    // per SIMD: 1024, 700 and 512 x LJ38 2.63, 2.52 and 2.51 instead of 2.85, 2.80
    // and 2.79 ms, 1024 x LJ64 5.2 instead of 5.7.
    // Their one hand-over costs less than three, so below 28 atoms they are the
    // better for any count, and where most clusters are much smaller below 32
    // (one / two / four wavefronts: 100 x LJ20 1.24 / 1.11 / 1.21, 512 x LJ24
    // 1.41 / 1.30 / 1.30, 512 x LJ28 2.26 / 2.15 / 1.97 ms; 511 x LJ13 beside one
    // LJ20 0.737 / 0.727 / 0.796, one LJ24 0.767 / 0.759 / 0.800, one LJ28 0.864 /
    // 0.815 / 0.881, one LJ38 1.61 / 1.35 / 1.30 ms; 512 of 8..24 atoms 1.24 / 1.12 /
    // 1.18).
    const bool eq1 = pot == LJ_PAIR_LJ, class0_alone = c == 0 && top_class == 0;
    const int four_from = !eq1 ? 32 : !class0_alone ? 20 : mean >= 20.0 ? 28 : 32;
    if (!mixed && c <= 1 && cmax >= four_from && num * calls <= (class0_alone ? 2 : 1) * cus)
        return lj::kRelayShape;
    if (!mixed && eq1 && class0_alone && cmax >= 20 && num * calls <= 4 * cus)
        return lj::kRelayPairShape;
    if (c == 0) {
        // Several clusters per wavefront once the batch has more than one
        // cluster per SIMD: each wavefront then does the work of two or four
        // (2048 x LJ13 FP64 0.76 instead of 0.88 ms, mixed 0.74 instead of
        // 0.97; 2048 x LJ30 2.28 instead of 2.90; 16384 x LJ13 1.76 instead of
        // 4.2).  Up to two clusters per SIMD only where the sizes are much
        // alike, since a packed wavefront waits for the slowest of its clusters
        // (2048 of 4..16 atoms: 0.98 instead of 0.91 ms).  Above 16 atoms in
        // FP64 and beyond two clusters per SIMD alone: the mixed path's packed
        // teams sum 20 atoms and more in another order.  The Morse pair's
        // one-cluster FP64 kernel evaluates unique pairs, the packed ones do not,
        // so there the sizes must be closer still (2048 x Morse13 1.13 packed,
        // 1.38 not, 2048 x Morse30 3.4 and 4.1, but 2048 of 17..32 atoms 3.2
        // and 2.7).
        const bool many = num > 2 * 4 * cus;
        const bool alike = num > 4 * cus && mean > (pot == LJ_PAIR_LJ || mixed ? 0.7 : 0.9) * cmax;
        int shape = 0;
        if (cmax <= 16)
            shape = many || alike ? 3 : 1;
        else if (cmax <= 32 && (many || (alike && !mixed)))
            shape = 2;
        // Two wavefronts per SIMD (at most 256 registers) once the call has more
        // wavefronts than SIMDs: the second wavefront fills the first one's
        // issue gaps (2048 x LJ38 mixed 3.47 instead of 4.33 ms; 16384 x LJ13
        // FP64 1.76 instead of 2.27).  The mixed kernel keeps half of its
        // history in LDS then, and wins beside class 1 too (512 chains x 8 of
        // 38..75 atoms: 8.3 instead of 9.0 ms per step; 256 chains level).
        // Morse pair, FP64: not where that ends the unique-pair evaluation (up to
        // 40 atoms, one cluster per wavefront: 2048 x Morse38 6.3 instead of 6.5
        // to 7.0 ms, 3000 of 20..64 atoms 9.4 instead of 11.1, but 1500 x Morse48
        // 9.1 instead of 9.7 and 4096 x Morse48 15.6 instead of 17.3).
        const long per_wg = lj::shape_clusters_per_wg(0, shape);
        const long waves = ((long)num + per_wg - 1) / per_wg;
        bool two = waves > 4L * cus && (top_class == 0 || (mixed && top_class == 1 && num > 8 * cus));
        if (pot == LJ_PAIR_MORSE) two = two && (mixed || per_wg > 1 || mean > 45.0);
        return two ? shape + 4 : shape;
    }
    if (c == 2) return cmax <= 192 ? 1 : 0; // three wavefronts
    // Class 1 beside larger classes sums its FP32 pairs in the ordered loop
    // (a choice of summation order, kept so that results stay what they were).
    return top_class >= 2 ? 1 : 0;
}

// Whether the teams of classes 1 and 2 run two wavefronts per SIMD (half of the
// history in LDS, 256 registers) or one (512 registers).  Two wavefronts fill
// each other's issue gaps (a lone one issues FP64 every 6 and FP32 every 6
// cycles, two together every 4.6 and 3), but a call that does not fill the chip
// is better spread out.  The sizes are taken as uniform between
// 2 mean - max and max.  Measured (ms, one / two wavefronts per SIMD, mixed):
// 600, 800, 1024, 1500 and 4096 clusters of 13..150 atoms 16.1 / 18.1,
// 16.9 / 17.1, 19.2 / 16.6, 22.7 / 17.0 and 49.6 / 31.7; 512, 640 and 2048 x LJ98
// 11.8 / 12.3, 15.9 / 12.8 and 29.7 / 21.7; 300 and 600 of 65..250 atoms
// 19.4 / 22.4 and 28.3 / 26.2; 256, 300 and 512 x LJ160 (one team per CU
// otherwise) 18.3 / 17.6, 20.9 / 17.8 and 26.3 / 20.5.
bool dense_classes(int num, int max_n, double mean, int cus) {
    const double lo = std::max(0.0, 2.0 * mean - max_n), span = max_n - lo + 1.0;
    const double w2 = max_n <= 192 ? 3.0 : 4.0;
    auto share = [&](double a, double b) {  // of the sizes in (a, b]
        return std::max(0.0, std::min(b, (double)max_n) - std::max(a, lo - 1.0)) / span;
    };
    const double waves =
        num * (share(-1, 64) + 2.0 * share(64, 128) + w2 * share(128, 256) + 16.0 * share(256, 1024));
    return waves > 1.25 * 4 * cus || (mean > 128.0 && max_n <= 256 && num > cus);
}

int class_schedule(int precision, int c, int max_n, int pot, int num, double mean, int cus,
                   int calls) {
    const int top = lj::class_of(max_n < 0 ? 0 : max_n);
    if (c == 3) return large_schedule(precision);
    {
        std::lock_guard<std::mutex> lk(g_sched_mu);
        auto it = g_class_sched.find(class_key(precision, c, max_n));
        if (it != g_class_sched.end() && lj::shape_max_n(c, it->second) >= class_cap(c, max_n))
            return it->second;
    }
    return default_class_shape(c, max_n, top, precision == LJ_MIXED, pot, num, mean, cus, calls);
}

// Workspace carve-up of one minimisation call, and the shape of each class.
struct MinLayout {
    size_t list = 0, cls = 0, queue = 0, hist = 0, total = 0;
    int top_class = -1;
    int shape[lj::kNumClasses] = {0, 0, 0, 0};
    int grid[lj::kNumClasses] = {0, 0, 0, 0};
};

// calls: calls_at_once (the sizes do not depend on it).  force (nullable): a shape
// per class, -1 for the schedule table's choice.
lj_status min_layout(int num, int max_n, int64_t total, int mixed, int pot, int calls,
                     MinLayout& L, const int* force = nullptr) {
    DeviceInfo di;
    lj_status s = device_info(di);
    if (s != LJ_OK) return s;
    const int prec = mixed ? LJ_MIXED : LJ_FP64;
    size_t off = 0;
    L.list = off;
    off = align_up(off + sizeof(int32_t) * (size_t)(num > 0 ? num : 1));
    L.cls = off;
    off = align_up(off + sizeof(int32_t) * 2 * lj::kNumClasses);
    L.queue = off;
    off = align_up(off + sizeof(int32_t) * lj::kNumClasses);
    // the plan rejects clusters above max_n, so max_n bounds every class
    L.top_class = lj::class_of(max_n < 0 ? 0 : max_n);
    const double mean = (double)total / (num > 0 ? num : 1);
    for (int c = 0; c <= L.top_class; ++c) {
        L.shape[c] = (force && force[c] >= 0)
                         ? force[c]
                         : class_schedule(prec, c, max_n, pot, num, mean, di.cus, calls);
        if ((c == 1 || c == 2) && L.shape[c] < lj::class_shapes(c) &&
            dense_classes(num, max_n, mean, di.cus))
            L.shape[c] |= lj::kDenseShape;
        if (L.shape[c] < 0 ||
            ((L.shape[c] & ~lj::kDenseShape) >= lj::class_shapes(c) &&
             !lj::is_relay(L.shape[c])) ||
            lj::shape_max_n(c, L.shape[c]) < class_cap(c, max_n))
            return fail(LJ_E_ARG, "minimiser shape %d of class %d does not hold %d atoms",
                        L.shape[c], c, class_cap(c, max_n));
    }
    auto grid_for = [&](int c, int shape, int& g_out) -> lj_status {
        int per_cu = 0;
        LJ_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu, lj::minimize_kernel_for(mixed, pot, c, shape), lj::class_block(c, shape),
            lj::class_dyn_lds(c, shape, max_n, pot)));
        if (per_cu < 1) per_cu = 1;
        const int per_wg = lj::shape_clusters_per_wg(c, shape);
        long g = (long)per_cu * di.cus;
        const long need = ((long)num + per_wg - 1) / per_wg;
        if (g > need) g = need;
        if (g < 1) g = 1;
        g_out = (int)g;
        return LJ_OK;
    };
    for (int c = 0; c <= L.top_class; ++c)
        if ((s = grid_for(c, L.shape[c], L.grid[c])) != LJ_OK) return s;
    L.hist = off;
    if (L.top_class >= 3) {
        // sized for the largest grid of any large-cluster shape, so a workspace
        // stays valid whichever shape the schedule table selects
        size_t hist = 0;
        for (int k = 0; k < lj::class_shapes(3); ++k) {
            int g = 0;
            if ((s = grid_for(3, k, g)) != LJ_OK) return s;
            const size_t b = lj::class_hist_bytes_per_wg(3, k) * (size_t)g;
            if (b > hist) hist = b;
        }
        off = align_up(off + hist);
    }
    L.total = off;
    return LJ_OK;
}

// Side streams (default priority) and events used to run the minimiser's size
// classes concurrently: fork from the caller's stream after the plan kernel,
// the largest class on the caller's stream and each other class on a side
// stream, join back before returning.  The pattern is also
// valid under stream capture (parallel graph branches).  Each (device, caller
// stream) pair has its own set: a side stream pulled into a capture stays in
// capture mode until the capture ends, so a set shared with callers on other
// streams would let their eager launches land in that graph.
struct SideStreams {
    bool ready = false;
    hipStream_t s[lj::kNumClasses];
    hipEvent_t fork;
    hipEvent_t join[lj::kNumClasses];
    std::mutex mu;
};
std::mutex g_side_mu;
std::map<std::pair<int, hipStream_t>, SideStreams*> g_side;
constexpr size_t kMaxSideSets = 16;  // beyond this, classes run in turn on the caller's stream

// out = nullptr (and LJ_OK) once kMaxSideSets caller streams have a set.
lj_status side_streams(hipStream_t caller, SideStreams*& out) {
    out = nullptr;
    int dev = 0;
    LJ_HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_side_mu);
    auto it = g_side.find({dev, caller});
    if (it == g_side.end()) {
        if (g_side.size() >= kMaxSideSets) return LJ_OK;
        it = g_side.emplace(std::make_pair(dev, caller), new SideStreams()).first;  // kept until exit
    }
    SideStreams* ss = it->second;
    if (!ss->ready) {
        for (int c = 0; c < lj::kNumClasses; ++c) {
            LJ_HIP_TRY(hipStreamCreateWithFlags(&ss->s[c], hipStreamNonBlocking));
            LJ_HIP_TRY(hipEventCreateWithFlags(&ss->join[c], hipEventDisableTiming));
        }
        LJ_HIP_TRY(hipEventCreateWithFlags(&ss->fork, hipEventDisableTiming));
        ss->ready = true;
    }
    out = ss;
    return LJ_OK;
}

lj_status enqueue_minimize(const lj_batch* b, const int32_t* active, double* xyz, double* energy,
                           double* gnorm, int32_t* iters, int32_t* evals, int32_t* status,
                           double* xyz_switch, const lj::LbfgsDev& p, int mixed,
                           const MinLayout& L, char* ws, hipStream_t st,
                           bool concurrent = true) {
    if (b->num == 0) return LJ_OK;
    lj::Plan plan;
    plan.list = reinterpret_cast<int32_t*>(ws + L.list);
    plan.cls = reinterpret_cast<int32_t*>(ws + L.cls);
    plan.queue = reinterpret_cast<int32_t*>(ws + L.queue);
    LJ_HIP_TRY(lj::launch_plan(b->offset, b->num, b->max_n, active, plan, status, st));
    lj::MinArgs a;
    a.offset = b->offset;
    a.total = b->total_atoms;
    a.xyz = xyz;
    a.energy = energy;
    a.gnorm = gnorm;
    a.iters = iters;
    a.evals = evals;
    a.status = status;
    a.xyz_switch = mixed ? xyz_switch : nullptr;
    a.plan = plan;
    a.p = p;
    a.pot = b->pair;
    a.rho = b->pair_rho;
    a.u = units_of(b);
    a.max_n = b->max_n;
    a.up_n = 0;
    if (L.top_class == 0) {
        a.cls = 0;
        a.hist = nullptr;
        LJ_HIP_TRY(lj::launch_minimize_class(mixed, 0, L.shape[0], L.grid[0], a, st));
        return LJ_OK;
    }
    // several size classes: run them concurrently on side streams
    SideStreams* ss = nullptr;
    if (concurrent) {
        lj_status r = side_streams(st, ss);
        if (r != LJ_OK) return r;
    }
    if (!ss) {  // no side streams (for this caller stream): the classes run in turn
        for (int c = L.top_class; c >= 0; --c) {
            a.cls = c;
            a.hist = (c == 3) ? reinterpret_cast<double*>(ws + L.hist) : nullptr;
            LJ_HIP_TRY(lj::launch_minimize_class(mixed, c, L.shape[c], L.grid[c], a, st));
        }
        return LJ_OK;
    }
    std::lock_guard<std::mutex> lk(ss->mu);
    LJ_HIP_TRY(hipEventRecord(ss->fork, st));
    // The largest class goes first, on the caller's stream, and the others on
    // the first side streams.  Streams share the device's few hardware queues,
    // which run in order: with a side stream per class, two classes could land
    // on one queue and run one after the other (the uneven 4096-cluster batch
    // took 60 instead of 47 ms that way).
    a.cls = L.top_class;
    a.hist = (L.top_class == 3) ? reinterpret_cast<double*>(ws + L.hist) : nullptr;
    LJ_HIP_TRY(lj::launch_minimize_class(mixed, L.top_class, L.shape[L.top_class],
                                         L.grid[L.top_class], a, st));
    a.hist = nullptr;
    for (int c = L.top_class - 1; c >= 0; --c) {
        const int k = L.top_class - 1 - c;
        a.cls = c;
        LJ_HIP_TRY(hipStreamWaitEvent(ss->s[k], ss->fork, 0));
        LJ_HIP_TRY(lj::launch_minimize_class(mixed, c, L.shape[c], L.grid[c], a, ss->s[k]));
        LJ_HIP_TRY(hipEventRecord(ss->join[k], ss->s[k]));
    }
    for (int k = 0; k < L.top_class; ++k) LJ_HIP_TRY(hipStreamWaitEvent(st, ss->join[k], 0));
    return LJ_OK;
}

// Basin-hopping workspace carve-up.
struct BhLayout {
    size_t xc = 0, cand_off = 0, ce = 0, cg = 0, ci = 0, cv = 0, cs = 0, dec = 0, pe = 0, pg = 0,
           pi = 0, pv = 0, ps = 0, min = 0, total = 0;
    MinLayout cand_min, polish_min;
    int64_t cand_total = 0;
    int cand_num = 0;
};

lj_status bh_layout(const lj_batch* ch, const lj_bh_params* bh, int mixed, BhLayout& L) {
    const int n = bh->cands;
    L.cand_num = ch->num * n;
    L.cand_total = ch->total_atoms * n;
    if (L.cand_total > INT32_MAX) return fail(LJ_E_ARG, "candidate atom count exceeds int32");
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off = align_up(off + (bytes > 0 ? bytes : 1));
        return at;
    };
    L.xc = take(sizeof(double) * 3 * (size_t)L.cand_total);
    L.cand_off = take(sizeof(int32_t) * ((size_t)L.cand_num + 1));
    L.ce = take(sizeof(double) * (size_t)L.cand_num);
    L.cg = take(sizeof(double) * (size_t)L.cand_num);
    L.ci = take(sizeof(int32_t) * (size_t)L.cand_num);
    L.cv = take(sizeof(int32_t) * (size_t)L.cand_num);
    L.cs = take(sizeof(int32_t) * (size_t)L.cand_num);
    L.dec = take(sizeof(int32_t) * 2 * (size_t)ch->num);
    L.pe = take(sizeof(double) * (size_t)ch->num);
    L.pg = take(sizeof(double) * (size_t)ch->num);
    L.pi = take(sizeof(int32_t) * (size_t)ch->num);
    L.pv = take(sizeof(int32_t) * (size_t)ch->num);
    L.ps = take(sizeof(int32_t) * (size_t)ch->num);
    lj_status s = min_layout(L.cand_num, ch->max_n, L.cand_total, mixed, ch->pair, 1, L.cand_min);
    if (s != LJ_OK) return s;
    s = min_layout(ch->num, ch->max_n, ch->total_atoms, 0, ch->pair, 1, L.polish_min);
    if (s != LJ_OK) return s;
    L.min = off;
    const size_t m = L.cand_min.total > L.polish_min.total ? L.cand_min.total : L.polish_min.total;
    off = align_up(off + m);
    L.total = off;
    return LJ_OK;
}

lj_status check_bh(const lj_batch* ch, const lj_bh_params* bh) {
    if (!bh) return fail(LJ_E_ARG, "bh params is NULL");
    if (!reduced_units(ch))
        return fail(LJ_E_UNSUPPORTED, "basin hopping runs in reduced units: sigma and epsilon "
                    "of the chains' batch must be 1 (or 0)");
    if (bh->cands < 1 || bh->cands > LJ_MAX_CANDS)
        return fail(LJ_E_ARG, "cands = %d outside [1, %d]", bh->cands, LJ_MAX_CANDS);
    if (!(bh->kT > 0.0)) return fail(LJ_E_ARG, "kT must be > 0");
    if (bh->adapt_interval < 1) return fail(LJ_E_ARG, "adapt_interval must be >= 1");
    if (!(bh->factor > 0.0)) return fail(LJ_E_ARG, "factor must be > 0");
    if (!std::isfinite(bh->target_rate)) return fail(LJ_E_ARG, "target_rate not finite");
    if ((int64_t)ch->num * bh->cands > INT32_MAX) return fail(LJ_E_ARG, "too many candidates");
    return LJ_OK;
}

// One basin-hopping step enqueued on st.
lj_status enqueue_bh_step(const lj_batch* ch, const lj::BhStateDev& s, const lj::BhDev& p,
                          const lj_lbfgs_params* lp, int mixed, const lj::BhTraceDev& tr,
                          const BhLayout& L, char* ws, hipStream_t st) {
    double* xc = reinterpret_cast<double*>(ws + L.xc);
    int32_t* cand_off = reinterpret_cast<int32_t*>(ws + L.cand_off);
    double* ce = reinterpret_cast<double*>(ws + L.ce);
    int32_t* dec = reinterpret_cast<int32_t*>(ws + L.dec);
    LJ_HIP_TRY(lj::launch_perturb(ch->offset, ch->num, ch->max_n, ch->total_atoms, s, p, xc,
                                  cand_off, st));
    lj_batch cb;
    cb.num = L.cand_num;
    cb.offset = cand_off;
    cb.max_n = ch->max_n;
    cb.total_atoms = L.cand_total;
    cb.pair = ch->pair;
    cb.pair_rho = ch->pair_rho;
    cb.sigma = 1.0;
    cb.epsilon = 1.0;
    lj::LbfgsDev d = to_dev(lp);
    if (mixed) d.polish = 0;  // only the accepted candidate is polished
    lj_status r = enqueue_minimize(&cb, nullptr, xc, ce, reinterpret_cast<double*>(ws + L.cg),
                                   reinterpret_cast<int32_t*>(ws + L.ci),
                                   reinterpret_cast<int32_t*>(ws + L.cv),
                                   reinterpret_cast<int32_t*>(ws + L.cs), nullptr, d, mixed,
                                   L.cand_min, ws + L.min, st);
    if (r != LJ_OK) return r;
    // without a polish, decide also finalizes the step (one launch fewer)
    LJ_HIP_TRY(lj::launch_decide(ch->offset, ch->num, ch->max_n, ch->total_atoms, s, p, xc, ce, dec,
                                 mixed ? nullptr : &tr, st));
    if (!mixed) return LJ_OK;
    // FP64 polish of the accepted candidates (the active mask is the accepted flags)
    double* pe = reinterpret_cast<double*>(ws + L.pe);
    r = enqueue_minimize(ch, dec + ch->num, s.xyz_cur, pe, reinterpret_cast<double*>(ws + L.pg),
                         reinterpret_cast<int32_t*>(ws + L.pi),
                         reinterpret_cast<int32_t*>(ws + L.pv),
                         reinterpret_cast<int32_t*>(ws + L.ps), nullptr, to_dev(lp), 0,
                         L.polish_min, ws + L.min, st);
    if (r != LJ_OK) return r;
    LJ_HIP_TRY(lj::launch_finalize(ch->offset, ch->num, ch->max_n, ch->total_atoms, s, p, ce, dec, pe,
                                   reinterpret_cast<const int32_t*>(ws + L.ps), tr, st));
    return LJ_OK;
}

// HIP-graph cache of one basin-hopping step, keyed by every argument byte.
// `done` is recorded after each launch, so an evicted graph is destroyed only
// once its last launch has finished.
struct GraphEntry {
    std::vector<unsigned char> key;
    int device;
    hipGraphExec_t exec;
    hipEvent_t done;
};
std::mutex g_graph_mu;
std::vector<GraphEntry> g_graphs;
constexpr size_t kMaxGraphs = 16;

std::atomic<int64_t> g_graph_captures{0};

// Appends the bytes of one scalar or pointer.  Structs are keyed field by
// field: their padding bytes are indeterminate and would make equal
// arguments compare unequal.
template <typename T>
void key_add(std::vector<unsigned char>& k, const T& v) {
    static_assert(std::is_arithmetic<T>::value || std::is_pointer<T>::value,
                  "key structs field by field");
    const unsigned char* p = reinterpret_cast<const unsigned char*>(&v);
    k.insert(k.end(), p, p + sizeof(T));
}

std::vector<unsigned char> step_key(const lj_batch* ch, const lj::BhStateDev& sd,
                                    const lj::BhDev& pd, const lj_lbfgs_params* lp,
                                    int32_t precision, const lj::BhTraceDev& td, const void* ws,
                                    size_t ws_bytes, hipStream_t st, const BhLayout& L) {
    std::vector<unsigned char> k;
    k.reserve(320);
    key_add(k, ch->num);
    key_add(k, ch->offset);
    key_add(k, ch->max_n);
    key_add(k, ch->total_atoms);
    key_add(k, ch->pair);
    key_add(k, ch->pair_rho);
    key_add(k, ch->sigma);
    key_add(k, ch->epsilon);
    for (const void* ptr : {(const void*)sd.xyz_cur, (const void*)sd.e_cur, (const void*)sd.step,
                            (const void*)sd.win_accepts, (const void*)sd.step_index,
                            (const void*)sd.e_best_seen, (const void*)sd.e_best_acc,
                            (const void*)sd.xyz_best})
        key_add(k, ptr);
    key_add(k, pd.cands);
    key_add(k, pd.kT);
    key_add(k, pd.adapt_interval);
    key_add(k, pd.target_rate);
    key_add(k, pd.factor);
    key_add(k, pd.seed);
    key_add(k, lp->m);
    key_add(k, lp->gtol);
    key_add(k, lp->max_iter);
    key_add(k, lp->max_step);
    key_add(k, lp->c1);
    key_add(k, lp->max_ls);
    key_add(k, lp->curv_eps);
    key_add(k, lp->gtol_mixed_per_atom);
    key_add(k, lp->polish);
    key_add(k, lp->ls_noise);
    key_add(k, precision);
    for (const void* ptr : {(const void*)td.e_trial, (const void*)td.accepted,
                            (const void*)td.e_best, (const void*)td.e_best_acc,
                            (const void*)td.e_cur, (const void*)td.step, (const void*)td.e_cand,
                            (const void*)td.polish_status})
        key_add(k, ptr);
    key_add(k, td.cap);
    key_add(k, ws);
    key_add(k, ws_bytes);
    key_add(k, st);
    // a graph keeps the launch shapes it captured: the candidates' minimiser
    // shapes and, on the mixed path, those of the accepted candidates' polish
    for (int c = 0; c < lj::kNumClasses; ++c) {
        key_add(k, L.cand_min.shape[c]);
        key_add(k, L.polish_min.shape[c]);
    }
    return k;
}


}  // namespace

// Scratch of lj_bh_minimize_batch_noalloc: the work list, size-class table and
// claim counters of one call, in a fixed array that every device holding the
// library keeps until the process ends.  Host code never uses this name as an
// address: the device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[LJ_NOALLOC_SCRATCH_BYTES];

namespace {

std::mutex g_scratch_mu;
std::vector<char*> g_scratch_ptr;  // per device

lj_status noalloc_scratch(char*& out) {
    int dev = 0;
    LJ_HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if ((int)g_scratch_ptr.size() <= dev) g_scratch_ptr.resize(dev + 1, nullptr);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        LJ_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(LJ_E_HIP, "hipGetSymbolAddress returned NULL for the scratch array");
        g_scratch_ptr[dev] = static_cast<char*>(p);
    }
    out = g_scratch_ptr[dev];
    return LJ_OK;
}

}  // namespace

extern "C" {

const char* lj_status_string(lj_status s) {
    switch (s) {
        case LJ_OK: return "LJ_OK";
        case LJ_E_ARG: return "LJ_E_ARG: invalid argument";
        case LJ_E_HIP: return "LJ_E_HIP: HIP runtime error";
        case LJ_E_WORKSPACE: return "LJ_E_WORKSPACE: workspace missing or too small";
        case LJ_E_UNSUPPORTED: return "LJ_E_UNSUPPORTED: size above the compiled limit or not gfx950";
    }
    return "unknown lj_status";
}

const char* lj_last_error(void) { return g_err.c_str(); }

int32_t lj_abi_version(void) { return LJ_ABI_VERSION; }

int64_t lj_bh_graph_captures(void) { return g_graph_captures.load(); }

void lj_lbfgs_defaults(lj_lbfgs_params* p) {
    if (!p) return;
    p->m = 10;
    p->gtol = 1e-6;
    p->max_iter = 10000;
    p->max_step = 0.2;
    p->c1 = 1e-4;
    p->max_ls = 30;
    p->curv_eps = 1e-10;
    p->gtol_mixed_per_atom = 1e-5;
    p->polish = 1;
    p->ls_noise = 5e-7;
}

size_t lj_energy_grad_workspace_bytes(const lj_batch* batch, int32_t precision) {
    if (check_batch(batch, LJ_MAX_ATOMS_EVAL, "lj_energy_grad_workspace_bytes") != LJ_OK) return 0;
    DeviceInfo di;
    if (batch->num == 0 || device_info(di) != LJ_OK) return 0;
    return split_eval_ws(batch, precision, di.cus);
}

lj_status lj_energy_grad_batch(const lj_batch* batch, const double* xyz, double* energy,
                               double* grad, int32_t precision, void* stream) {
    return lj_energy_grad_batch_ws(batch, xyz, energy, grad, precision, nullptr, 0, stream);
}

lj_status lj_energy_grad_batch_ws(const lj_batch* batch, const double* xyz, double* energy,
                                  double* grad, int32_t precision, void* ws, size_t ws_bytes,
                                  void* stream) {
    g_err.clear();
    lj_status s = check_batch(batch, LJ_MAX_ATOMS_EVAL, "lj_energy_grad_batch");
    if (s != LJ_OK) return s;
    if (precision != LJ_FP64 && precision != LJ_MIXED)
        return fail(LJ_E_ARG, "precision = %d is neither LJ_FP64 nor LJ_MIXED", precision);
    if (batch->num == 0) return LJ_OK;
    if (!energy) return fail(LJ_E_ARG, "energy is NULL");
    if (batch->total_atoms > 0 && !xyz) return fail(LJ_E_ARG, "xyz is NULL");
    DeviceInfo di;
    s = device_info(di);
    if (s != LJ_OK) return s;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const size_t need = ws ? split_eval_ws(batch, precision, di.cus) : 0;
    if (need > 0 && ws_bytes >= need) {
        LJ_HIP_TRY(lj::launch_split_eval(precision == LJ_MIXED, batch->pair, batch->num,
                                         batch->max_n, batch->offset, batch->total_atoms, xyz,
                                         energy, grad, batch->pair_rho, units_of(batch),
                                         static_cast<char*>(ws), st));
        return LJ_OK;
    }
    LJ_HIP_TRY(lj::launch_energy_grad(precision == LJ_MIXED, batch->pair,
                                      eval_schedule(precision, batch->max_n), batch->num,
                                      batch->offset, batch->total_atoms, xyz, energy, grad,
                                      batch->pair_rho, units_of(batch), st));
    return LJ_OK;
}

size_t lj_minimize_workspace_bytes(const lj_batch* batch, const lj_lbfgs_params* params,
                                   int32_t precision) {
    (void)params;
    if (check_batch(batch, LJ_MAX_ATOMS_MIN, "lj_minimize_workspace_bytes") != LJ_OK) return 0;
    MinLayout L;
    if (min_layout(batch->num, batch->max_n, batch->total_atoms, precision == LJ_MIXED, batch->pair,
                   1, L) != LJ_OK)
        return 0;
    return L.total;
}

lj_status lj_minimize_forms(const lj_batch* batch, int32_t precision, void* stream,
                            int32_t* forms) {
    g_err.clear();
    lj_status s = check_batch(batch, LJ_MAX_ATOMS_MIN, "lj_minimize_forms");
    if (s != LJ_OK) return s;
    if (precision != LJ_FP64 && precision != LJ_MIXED)
        return fail(LJ_E_ARG, "precision = %d is neither LJ_FP64 nor LJ_MIXED", precision);
    if (!forms) return fail(LJ_E_ARG, "forms is NULL");
    DeviceInfo di;
    if ((s = device_info(di)) != LJ_OK) return s;
    const int calls = calls_at_once(static_cast<hipStream_t>(stream), batch->num, di.cus, false);
    MinLayout L;
    if ((s = min_layout(batch->num, batch->max_n, batch->total_atoms, precision == LJ_MIXED,
                        batch->pair, calls, L)) != LJ_OK)
        return s;
    for (int c = 0; c < lj::kNumClasses; ++c) forms[c] = c <= L.top_class ? L.shape[c] : -1;
    return LJ_OK;
}

lj_status lj_bh_minimize_batch(const lj_batch* batch, double* xyz, double* energy, double* gnorm,
                               int32_t* iters, int32_t* evals, int32_t* status,
                               double* xyz_switch, const lj_lbfgs_params* params,
                               int32_t precision, void* ws, size_t ws_bytes, void* stream) {
    g_err.clear();
    lj_status s = check_batch(batch, LJ_MAX_ATOMS_MIN, "lj_bh_minimize_batch");
    if (s != LJ_OK) return s;
    if ((s = check_params(params)) != LJ_OK) return s;
    if (precision != LJ_FP64 && precision != LJ_MIXED)
        return fail(LJ_E_ARG, "precision = %d is neither LJ_FP64 nor LJ_MIXED", precision);
    if (batch->num == 0) return LJ_OK;
    if (!energy || !gnorm || !iters || !evals || !status)
        return fail(LJ_E_ARG, "an output array is NULL");
    if (batch->total_atoms > 0 && !xyz) return fail(LJ_E_ARG, "xyz is NULL");
    DeviceInfo di;
    if ((s = device_info(di)) != LJ_OK) return s;
    const int calls = calls_at_once(static_cast<hipStream_t>(stream), batch->num, di.cus, true);
    MinLayout L;
    if ((s = min_layout(batch->num, batch->max_n, batch->total_atoms, precision == LJ_MIXED,
                        batch->pair, calls, L)) != LJ_OK)
        return s;
    if (!ws || ws_bytes < L.total)
        return fail(LJ_E_WORKSPACE, "workspace of %zu bytes given, %zu needed", ws_bytes, L.total);
    return enqueue_minimize(batch, nullptr, xyz, energy, gnorm, iters, evals, status, xyz_switch,
                            to_dev(params), precision == LJ_MIXED, L, static_cast<char*>(ws),
                            static_cast<hipStream_t>(stream));
}

lj_status lj_bh_minimize_batch_noalloc(const lj_batch* batch, double* xyz, double* energy,
                                       double* gnorm, int32_t* iters, int32_t* evals,
                                       int32_t* status, double* xyz_switch,
                                       const lj_lbfgs_params* params, int32_t precision,
                                       void* stream) {
    g_err.clear();
    lj_status s = check_batch(batch, LJ_MAX_ATOMS_MIN, "lj_bh_minimize_batch_noalloc");
    if (s != LJ_OK) return s;
    if ((s = check_params(params)) != LJ_OK) return s;
    if (precision != LJ_FP64 && precision != LJ_MIXED)
        return fail(LJ_E_ARG, "precision = %d is neither LJ_FP64 nor LJ_MIXED", precision);
    if (batch->num == 0) return LJ_OK;
    if (!energy || !gnorm || !iters || !evals || !status)
        return fail(LJ_E_ARG, "an output array is NULL");
    if (batch->total_atoms > 0 && !xyz) return fail(LJ_E_ARG, "xyz is NULL");
    if (batch->max_n > LJ_NOALLOC_MAX_ATOMS)
        return fail(LJ_E_UNSUPPORTED,
                    "lj_bh_minimize_batch_noalloc: max_n = %d exceeds %d (larger clusters keep "
                    "their L-BFGS history in a workspace; use lj_bh_minimize_batch)",
                    batch->max_n, LJ_NOALLOC_MAX_ATOMS);
    if (batch->num > LJ_NOALLOC_MAX_CLUSTERS)
        return fail(LJ_E_WORKSPACE,
                    "lj_bh_minimize_batch_noalloc: %d clusters exceed the %d that its %d-byte "
                    "static scratch holds; use lj_bh_minimize_batch",
                    batch->num, LJ_NOALLOC_MAX_CLUSTERS, LJ_NOALLOC_SCRATCH_BYTES);
    MinLayout L;
    // calls that overlap would race, so this one has the device
    if ((s = min_layout(batch->num, batch->max_n, batch->total_atoms, precision == LJ_MIXED,
                        batch->pair, 1, L)) != LJ_OK)
        return s;
    if (L.total > (size_t)LJ_NOALLOC_SCRATCH_BYTES)
        return fail(LJ_E_WORKSPACE, "lj_bh_minimize_batch_noalloc: %zu bytes of scratch needed, "
                    "%d available", L.total, LJ_NOALLOC_SCRATCH_BYTES);
    char* ws = nullptr;
    if ((s = noalloc_scratch(ws)) != LJ_OK) return s;
    // the size classes run in turn on the caller's stream (no side streams are
    // created); the plan kernel rewrites the whole scratch it uses, counters
    // included, before the minimiser reads it
    return enqueue_minimize(batch, nullptr, xyz, energy, gnorm, iters, evals, status, xyz_switch,
                            to_dev(params), precision == LJ_MIXED, L, ws,
                            static_cast<hipStream_t>(stream), false);
}

size_t lj_bh_workspace_bytes(const lj_batch* chains, const lj_bh_params* bh,
                             const lj_lbfgs_params* params, int32_t precision) {
    (void)params;
    if (check_batch(chains, LJ_MAX_ATOMS_MIN, "lj_bh_workspace_bytes") != LJ_OK) return 0;
    if (check_bh(chains, bh) != LJ_OK) return 0;
    BhLayout L;
    if (bh_layout(chains, bh, precision == LJ_MIXED, L) != LJ_OK) return 0;
    return L.total;
}

lj_status lj_bh_step(const lj_batch* chains, const lj_bh_state* state, const lj_bh_params* bh,
                     const lj_lbfgs_params* params, int32_t precision, int32_t num_steps,
                     const lj_bh_trace* trace, void* ws, size_t ws_bytes, void* stream) {
    g_err.clear();
    lj_status s = check_batch(chains, LJ_MAX_ATOMS_MIN, "lj_bh_step");
    if (s != LJ_OK) return s;
    if ((s = check_params(params)) != LJ_OK) return s;
    if ((s = check_bh(chains, bh)) != LJ_OK) return s;
    if (precision != LJ_FP64 && precision != LJ_MIXED)
        return fail(LJ_E_ARG, "precision = %d is neither LJ_FP64 nor LJ_MIXED", precision);
    if (num_steps < 0) return fail(LJ_E_ARG, "num_steps < 0");
    if (!state) return fail(LJ_E_ARG, "state is NULL");
    if (chains->num == 0 || num_steps == 0) return LJ_OK;
    if (!state->xyz_cur || !state->e_cur || !state->step || !state->win_accepts ||
        !state->step_index || !state->e_best_seen || !state->e_best_acc || !state->xyz_best)
        return fail(LJ_E_ARG, "a state array is NULL");
    if (trace && trace->capacity_steps < 0) return fail(LJ_E_ARG, "trace capacity < 0");
    const int mixed = precision == LJ_MIXED;
    BhLayout L;
    if ((s = bh_layout(chains, bh, mixed, L)) != LJ_OK) return s;
    if (!ws || ws_bytes < L.total)
        return fail(LJ_E_WORKSPACE, "workspace of %zu bytes given, %zu needed", ws_bytes, L.total);

    lj::BhStateDev sd{state->xyz_cur, state->e_cur,       state->step,       state->win_accepts,
                      state->step_index, state->e_best_seen, state->e_best_acc, state->xyz_best};
    lj::BhDev pd{bh->cands, bh->kT, bh->adapt_interval, bh->target_rate, bh->factor, bh->seed};
    lj::BhTraceDev td{};
    if (trace)
        td = lj::BhTraceDev{trace->e_trial, trace->accepted, trace->e_best, trace->e_best_acc,
                            trace->e_cur,   trace->step,     trace->e_cand, trace->polish_status,
                            trace->capacity_steps};
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* w = static_cast<char*>(ws);

    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (st) LJ_HIP_TRY(hipStreamIsCapturing(st, &cap));
    if (!st || cap != hipStreamCaptureStatusNone) {
        for (int k = 0; k < num_steps; ++k)
            if ((s = enqueue_bh_step(chains, sd, pd, params, mixed, td, L, w, st)) != LJ_OK) return s;
        return LJ_OK;
    }

    int dev = 0;
    LJ_HIP_TRY(hipGetDevice(&dev));
    const std::vector<unsigned char> key =
        step_key(chains, sd, pd, params, precision, td, ws, ws_bytes, st, L);
    // Graphs are launched with the cache locked, so another thread's insertion
    // cannot evict and destroy a graph between its lookup and its launch.
    {
        std::lock_guard<std::mutex> lk(g_graph_mu);
        for (auto& e : g_graphs)
            if (e.device == dev && e.key == key) {
                for (int k = 0; k < num_steps; ++k) LJ_HIP_TRY(hipGraphLaunch(e.exec, st));
                LJ_HIP_TRY(hipEventRecord(e.done, st));
                return LJ_OK;
            }
    }
    LJ_HIP_TRY(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
    s = enqueue_bh_step(chains, sd, pd, params, mixed, td, L, w, st);
    hipGraph_t graph = nullptr;
    hipError_t ec = hipStreamEndCapture(st, &graph);
    if (s != LJ_OK) {
        if (graph) (void)hipGraphDestroy(graph);
        return s;
    }
    if (ec != hipSuccess) return fail(LJ_E_HIP, "hipStreamEndCapture: %s", hipGetErrorString(ec));
    hipGraphExec_t exec = nullptr;
    ec = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (ec != hipSuccess) return fail(LJ_E_HIP, "hipGraphInstantiate: %s", hipGetErrorString(ec));
    hipEvent_t done = nullptr;
    ec = hipEventCreateWithFlags(&done, hipEventDisableTiming);
    if (ec != hipSuccess) {
        (void)hipGraphExecDestroy(exec);
        return fail(LJ_E_HIP, "hipEventCreateWithFlags: %s", hipGetErrorString(ec));
    }
    std::lock_guard<std::mutex> lk(g_graph_mu);
    if (g_graphs.size() >= kMaxGraphs) {
        GraphEntry& old = g_graphs.front();
        (void)hipEventSynchronize(old.done);  // its last launch has finished
        (void)hipGraphExecDestroy(old.exec);
        (void)hipEventDestroy(old.done);
        g_graphs.erase(g_graphs.begin());
    }
    g_graphs.push_back(GraphEntry{key, dev, exec, done});
    g_graph_captures.fetch_add(1);
    for (int k = 0; k < num_steps; ++k) LJ_HIP_TRY(hipGraphLaunch(exec, st));
    LJ_HIP_TRY(hipEventRecord(done, st));
    return LJ_OK;
}

lj_status lj_set_schedule(int32_t kind, int32_t precision, int32_t max_n, int32_t w, int32_t a) {
    g_err.clear();
    if (precision != LJ_FP64 && precision != LJ_MIXED) return fail(LJ_E_ARG, "bad precision");
    if (kind == LJ_SCHED_EVAL) {
        lj::EvalShape sh{w, a};
        if (!lj::eval_shape_supported(sh)) return fail(LJ_E_ARG, "unsupported shape %dx%d", w, a);
        if (max_n < 0 || max_n > LJ_MAX_ATOMS_EVAL) return fail(LJ_E_ARG, "max_n out of range");
        if (64 * w * a < max_n) return fail(LJ_E_ARG, "shape %dx%d holds fewer than %d atoms", w, a, max_n);
        std::lock_guard<std::mutex> lk(g_sched_mu);
        g_eval_sched[{precision, pow2_at_least(max_n < 1 ? 1 : max_n)}] = sh;
        return LJ_OK;
    }
    if (kind == LJ_SCHED_MIN_LARGE) {
        if (w < 0 || w >= lj::kNumLargeShapes) return fail(LJ_E_ARG, "large-cluster shape %d", w);
        std::lock_guard<std::mutex> lk(g_sched_mu);
        g_large_sched[precision == LJ_MIXED ? 1 : 0] = w;
        return LJ_OK;
    }
    if (kind >= LJ_SCHED_MIN_CLASS0 && kind <= LJ_SCHED_MIN_CLASS2) {
        const int c = kind - LJ_SCHED_MIN_CLASS0;
        if (max_n < 0 || max_n > LJ_MAX_ATOMS_MIN) return fail(LJ_E_ARG, "max_n out of range");
        if (lj::class_of(max_n) < c)
            return fail(LJ_E_ARG, "a batch of at most %d atoms has no class-%d clusters", max_n, c);
        if (w == -1) {  // back to the built-in rule
            std::lock_guard<std::mutex> lk(g_sched_mu);
            g_class_sched.erase(class_key(precision, c, max_n));
            return LJ_OK;
        }
        if (w < 0 || w >= lj::class_shapes(c)) return fail(LJ_E_ARG, "class-%d shape %d", c, w);
        if (lj::shape_max_n(c, w) < class_cap(c, max_n))
            return fail(LJ_E_ARG, "class-%d shape %d holds at most %d atoms, not %d", c, w,
                        lj::shape_max_n(c, w), class_cap(c, max_n));
        std::lock_guard<std::mutex> lk(g_sched_mu);
        g_class_sched[class_key(precision, c, max_n)] = w;
        return LJ_OK;
    }
    return fail(LJ_E_ARG, "unknown schedule kind %d", kind);
}

lj_status lj_get_schedule(int32_t kind, int32_t precision, int32_t max_n, int32_t* w, int32_t* a) {
    g_err.clear();
    if (!w || !a) return fail(LJ_E_ARG, "NULL output");
    if (precision != LJ_FP64 && precision != LJ_MIXED) return fail(LJ_E_ARG, "bad precision");
    if (kind == LJ_SCHED_EVAL) {
        const lj::EvalShape sh = eval_schedule(precision, max_n);
        *w = sh.W;
        *a = sh.A;
        return LJ_OK;
    }
    if (kind == LJ_SCHED_MIN_LARGE) {
        *w = large_schedule(precision);
        *a = 0;
        return LJ_OK;
    }
    if (kind >= LJ_SCHED_MIN_CLASS0 && kind <= LJ_SCHED_MIN_CLASS2) {
        const int c = kind - LJ_SCHED_MIN_CLASS0;
        if (max_n < 0 || max_n > LJ_MAX_ATOMS_MIN) return fail(LJ_E_ARG, "max_n out of range");
        std::lock_guard<std::mutex> lk(g_sched_mu);
        auto it = g_class_sched.find(class_key(precision, c, max_n));
        *w = it == g_class_sched.end() ? -1 : it->second;
        *a = *w < 0 ? 0 : lj::shape_clusters_per_wg(c, *w);
        return LJ_OK;
    }
    return fail(LJ_E_ARG, "unknown schedule kind %d", kind);
}

size_t lj_autotune_workspace_bytes(const lj_batch* batch, int32_t precision) {
    if (check_batch(batch, LJ_MAX_ATOMS_EVAL, "lj_autotune_workspace_bytes") != LJ_OK) return 0;
    size_t off = align_up(sizeof(double) * (size_t)(batch->num > 0 ? batch->num : 1));  // energy
    off = align_up(off + sizeof(double) * 3 * (size_t)batch->total_atoms);              // grad
    // then the scratch of the spread evaluation, or (later) the minimiser's
    DeviceInfo di;
    const size_t spread =
        batch->num > 0 && device_info(di) == LJ_OK ? split_rule_ws(batch, precision, di.cus) : 0;
    const size_t eval_end = align_up(off + spread);
    if (batch->max_n <= LJ_MAX_ATOMS_MIN) {
        off = align_up(off + sizeof(double) * 3 * (size_t)batch->total_atoms);  // xyz copy
        off = align_up(off + 5 * sizeof(double) * (size_t)batch->num);          // outputs
        MinLayout L;
        if (min_layout(batch->num, batch->max_n, batch->total_atoms, precision == LJ_MIXED,
                       batch->pair, 1, L) != LJ_OK)
            return 0;
        off = align_up(off + L.total);
    }
    return std::max(off, eval_end);
}

lj_status lj_autotune(const lj_batch* batch, const double* xyz, int32_t precision, void* ws,
                      size_t ws_bytes, void* stream, float* best_eval_ms, float* best_min_ms) {
    g_err.clear();
    lj_status s = check_batch(batch, LJ_MAX_ATOMS_EVAL, "lj_autotune");
    if (s != LJ_OK) return s;
    if (precision != LJ_FP64 && precision != LJ_MIXED) return fail(LJ_E_ARG, "bad precision");
    if (batch->num == 0) return LJ_OK;
    if (batch->total_atoms > 0 && !xyz) return fail(LJ_E_ARG, "xyz is NULL");
    DeviceInfo di;
    if ((s = device_info(di)) != LJ_OK) return s;
    const size_t need = lj_autotune_workspace_bytes(batch, precision);
    if (!ws || ws_bytes < need)
        return fail(LJ_E_WORKSPACE, "workspace of %zu bytes given, %zu needed", ws_bytes, need);
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* w = static_cast<char*>(ws);
    double* e = reinterpret_cast<double*>(w);
    size_t off = align_up(sizeof(double) * (size_t)batch->num);
    double* g = reinterpret_cast<double*>(w + off);
    off = align_up(off + sizeof(double) * 3 * (size_t)batch->total_atoms);
    const int mixed = precision == LJ_MIXED;
    struct Events {  // destroyed on every return path
        hipEvent_t e[2] = {nullptr, nullptr};
        ~Events() {
            for (hipEvent_t x : e)
                if (x) (void)hipEventDestroy(x);
        }
    } evs;
    LJ_HIP_TRY(hipEventCreate(&evs.e[0]));
    LJ_HIP_TRY(hipEventCreate(&evs.e[1]));
    hipEvent_t e0 = evs.e[0], e1 = evs.e[1];
    // median of five timed launches after a warm-up (a minimum would follow
    // the luckiest launch of a shape whose launches vary)
    auto time_it = [&](auto&& launch, float& ms) -> lj_status {
        lj_status r = launch();  // warm-up
        if (r != LJ_OK) return r;
        constexpr int kReps = 5;
        float t[kReps];
        for (int rep = 0; rep < kReps; ++rep) {
            LJ_HIP_TRY(hipEventRecord(e0, st));
            if ((r = launch()) != LJ_OK) return r;
            LJ_HIP_TRY(hipEventRecord(e1, st));
            LJ_HIP_TRY(hipEventSynchronize(e1));
            LJ_HIP_TRY(hipEventElapsedTime(&t[rep], e0, e1));
        }
        std::sort(t, t + kReps);
        ms = t[kReps / 2];
        return LJ_OK;
    };
    // pair kernel: every shape holding max_n atoms without more than doubling the padding
    const int need_slots = batch->max_n < 1 ? 1 : batch->max_n;
    const int cap = 2 * (pow2_at_least(need_slots) < 64 ? 64 : pow2_at_least(need_slots));
    lj::EvalShape best_shape = lj::eval_shape(batch->max_n);
    float best_ms = 1e30f;
    // a batch that is spread over many workgroups is timed that way too; the table
    // gets the best shape of one workgroup per cluster all the same, for callers
    // without scratch memory, unless that shape would end the spread
    const size_t spread = split_eval_ws(batch, precision, di.cus);
    const int Ws[] = {1, 2, 4, 8, 16}, As[] = {1, 2, 4};
    for (int wi : Ws)
        for (int ai : As) {
            const int slots = 64 * wi * ai;
            if (slots < need_slots || slots > cap) continue;
            lj::EvalShape sh{wi, ai};
            if (spread > 0 && !same_eval_bits(mixed, batch->pair, sh, lj::eval_shape(batch->max_n)))
                continue;
            float ms = 0.f;
            s = time_it([&]() -> lj_status {
                LJ_HIP_TRY(lj::launch_energy_grad(mixed, batch->pair, sh, batch->num,
                                                  batch->offset, batch->total_atoms, xyz, e, g,
                                                  batch->pair_rho, units_of(batch), st));
                return LJ_OK;
            }, ms);
            if (s != LJ_OK) break;
            if (ms < best_ms) {
                best_ms = ms;
                best_shape = sh;
            }
        }
    if (s == LJ_OK) {
        std::lock_guard<std::mutex> lk(g_sched_mu);
        g_eval_sched[{precision, pow2_at_least(need_slots)}] = best_shape;
    }
    if (s == LJ_OK && spread > 0) {
        float ms = 0.f;
        s = time_it([&]() -> lj_status {
            LJ_HIP_TRY(lj::launch_split_eval(mixed, batch->pair, batch->num, batch->max_n,
                                             batch->offset, batch->total_atoms, xyz, e, g,
                                             batch->pair_rho, units_of(batch), w + off, st));
            return LJ_OK;
        }, ms);
        if (s == LJ_OK && ms < best_ms) best_ms = ms;
    }
    if (best_eval_ms) *best_eval_ms = best_ms;
    // Minimiser shapes (batches of at most LJ_MAX_ATOMS_MIN atoms): the
    // large-cluster class on a 3-iteration minimisation of a copy per shape;
    // then classes 2, 1, 0 in turn, each shape on a whole minimisation of a
    // copy (at most 1000 iterations per phase) with the other classes at their
    // current choice.  A shape replaces the current one when it is at least
    // 2 % faster; the choices go into the schedule table.
    float best_min = -1.f;
    if (s == LJ_OK && batch->max_n <= LJ_MAX_ATOMS_MIN) {
        double* xc = reinterpret_cast<double*>(w + off);
        off = align_up(off + sizeof(double) * 3 * (size_t)batch->total_atoms);
        double* outs = reinterpret_cast<double*>(w + off);
        off = align_up(off + 5 * sizeof(double) * (size_t)batch->num);
        int32_t* it = reinterpret_cast<int32_t*>(outs + 2 * (size_t)batch->num);
        int32_t* ev = it + batch->num;
        int32_t* stt = ev + batch->num;
        MinLayout base;
        const int calls = calls_at_once(st, batch->num, di.cus, false);
        if ((s = min_layout(batch->num, batch->max_n, batch->total_atoms, mixed, batch->pair, calls,
                            base)) != LJ_OK)
            return s;
        int chosen[lj::kNumClasses] = {-1, -1, -1, -1};
        for (int c = 0; c <= base.top_class; ++c) chosen[c] = base.shape[c] & ~lj::kDenseShape;
        lj_lbfgs_params lp;
        lj_lbfgs_defaults(&lp);
        auto time_shapes = [&](const int* force, const lj_lbfgs_params& prm, float& ms) -> lj_status {
            MinLayout L;
            lj_status r = min_layout(batch->num, batch->max_n, batch->total_atoms, mixed, batch->pair, calls,
                                     L, force);
            if (r != LJ_OK) return r;
            return time_it([&]() -> lj_status {
                LJ_HIP_TRY(hipMemcpyAsync(xc, xyz, sizeof(double) * 3 * (size_t)batch->total_atoms,
                                          hipMemcpyDeviceToDevice, st));
                return enqueue_minimize(batch, nullptr, xc, outs, outs + batch->num, it, ev, stt,
                                        nullptr, to_dev(&prm), mixed, L, w + off, st);
            }, ms);
        };
        if (base.top_class >= 3) {
            lj_lbfgs_params lp3 = lp;
            lp3.max_iter = 3;
            lp3.polish = 0;
            float best3 = 1e30f;
            for (int k = 0; k < lj::class_shapes(3) && s == LJ_OK; ++k) {
                int force[lj::kNumClasses];
                for (int c = 0; c < lj::kNumClasses; ++c) force[c] = chosen[c];
                force[3] = k;
                float ms = 0.f;
                s = time_shapes(force, lp3, ms);
                if (s == LJ_OK && ms < best3) {
                    best3 = ms;
                    chosen[3] = k;
                }
            }
            if (s == LJ_OK) {
                std::lock_guard<std::mutex> lk(g_sched_mu);
                g_large_sched[mixed] = chosen[3];
            }
        }
        lp.max_iter = 1000;
        float cur = 0.f;
        if (s == LJ_OK) s = time_shapes(chosen, lp, cur);
        // the class sizes of this batch, from the plan of the last timed call
        int32_t counts[2 * lj::kNumClasses] = {0};
        if (s == LJ_OK) {
            MinLayout L;
            if ((s = min_layout(batch->num, batch->max_n, batch->total_atoms, mixed, batch->pair,
                                calls, L, chosen)) != LJ_OK)
                return s;
            LJ_HIP_TRY(hipMemcpyAsync(counts, w + off + L.cls, sizeof(counts),
                                      hipMemcpyDeviceToHost, st));
            LJ_HIP_TRY(hipStreamSynchronize(st));
        }
        for (int c = base.top_class < 2 ? base.top_class : 2; c >= 0 && s == LJ_OK; --c) {
            if (counts[lj::kNumClasses + c] == 0) continue;  // no cluster of this class
            const int cap = class_cap(c, batch->max_n);
            // the numbered shapes, and the built-in rule's form where that has no
            // number (helper wavefronts): an entry found in the table may have been
            // tuned on many clusters
            const int rule = default_class_shape(c, batch->max_n, base.top_class, mixed,
                                                 batch->pair, batch->num,
                                                 (double)batch->total_atoms / batch->num, di.cus,
                                                 calls);
            for (int q = 0; q <= lj::class_shapes(c) && s == LJ_OK; ++q) {
                const int k = q < lj::class_shapes(c) ? q : rule;
                if (k == chosen[c] || lj::shape_max_n(c, k) < cap) continue;
                if (q == lj::class_shapes(c) && !lj::is_relay(rule)) continue;
                // class 1, FP64: both shapes are one kernel
                if (lj::minimize_kernel_for(mixed, batch->pair, c, k) ==
                    lj::minimize_kernel_for(mixed, batch->pair, c, chosen[c]))
                    continue;
                int force[lj::kNumClasses];
                for (int i = 0; i < lj::kNumClasses; ++i) force[i] = chosen[i];
                force[c] = k;
                float ms = 0.f;
                s = time_shapes(force, lp, ms);
                if (s == LJ_OK && ms < 0.98f * cur) {
                    cur = ms;
                    chosen[c] = k;
                }
            }
            if (s == LJ_OK) {
                // where a form with helper wavefronts is fastest, no entry: the
                // built-in rule takes it
                std::lock_guard<std::mutex> lk(g_sched_mu);
                if (lj::is_relay(chosen[c]))
                    g_class_sched.erase(class_key(precision, c, batch->max_n));
                else
                    g_class_sched[class_key(precision, c, batch->max_n)] = chosen[c];
            }
        }
        if (s == LJ_OK) best_min = cur;
    }
    if (best_min_ms) *best_min_ms = best_min;
    return s;
}

}  // extern "C"
