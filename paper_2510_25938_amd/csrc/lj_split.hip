// Energy and gradient of a few large clusters (gfx950), the work of one cluster
// spread over many workgroups.
//
// energy_grad_kernel gives a cluster one workgroup, which leaves most of the
// chip idle when a call holds fewer large clusters than the chip has CUs.
// Here the parts of a cluster's sums that do not depend on one another run on
// workgroups of their own, and the parts whose order is fixed are added in
// that order, so results are those of energy_grad_kernel bit for bit:
//   FP64   one workgroup per 64-atom tile (split64_kernel), then a reduction
//          of the tiles' energies (split_energy_kernel);
//   FP32   one wavefront per pair of 64-atom tiles (split32_kernel), whose FP32
//          partial sums are independent, then per tile their FP64 sums in
//          order (split32_sum_kernel), then the energies as above.
// One workgroup per cluster -> spread, us: 3 x LJ3000 FP64 2157 -> 94, FP32
// 1284 -> 39; 8 x LJ1000 188 -> 35 and 84 -> 17; 8 x Morse1000 396 -> 56 and 177 -> 19.
#include <hip/hip_runtime.h>

#include "lj_lbfgs.hpp"

namespace lj {

// ---------------------------------------------------------------------------
// FP64: the partners of one tile's 64 atoms in chunks of 64.  The producer
// wavefronts form a chunk's pair terms (kShare partners each) into LDS while
// wavefronts 0-3 add the previous chunk's, one of the sums e, gx, gy, gz each,
// partners ascending.  A lone wavefront would issue about 28 instructions per
// partner at 6 cycles each; here three wavefronts per SIMD share 23 + 4 x 3.5
// over four SIMDs.
// ---------------------------------------------------------------------------
constexpr int kChunk = kWave;
constexpr int kProducers = 8;
constexpr int kShare = kChunk / kProducers;
constexpr int kSplitBlock = (4 + kProducers) * kWave;

struct SplitLds {
    double pos[2][3][kChunk];      // partner coordinates, per component
    double f[2][kChunk][kWave];    // gradient coefficients [partner][lane]
    double e[2][kChunk][kWave];    // energy terms
};

template <int POT, bool IEEE, bool SELF>
__device__ __forceinline__ void split_terms(SplitLds& lds, int buf, int k0, int cnt,
                                            const double (&x)[3], double rho, double c,
                                            double k24, double km48, int lane) {
    constexpr int G = 4;
    // the Morse pair by its general forms: the short ones (about 45 instead of 70
    // instructions) would need the repeat that Eq. (1) has; not tried here
    constexpr bool GEN = IEEE || POT == kPairMorse;
    MorseRange range;
    if constexpr (POT == kPairMorse) range.coefs.hold();
    for (int k = k0; k < k0 + cnt; k += G) {
        double p[3][G];
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int u = 0; u < G; ++u) p[d][u] = lds.pos[buf][d][k + u];
        uint64_t self = SELF ? 1ull << k : 0;
#pragma unroll
        for (int u = 0; u < G; ++u, self <<= 1) {
            double f, e;
            pair_term64<POT, GEN>(x[0] - p[0][u], x[1] - p[1][u], x[2] - p[2][u],
                                   SELF && in_mask(self), rho, c, k24, km48, f, e, range);
            lds.f[buf][k + u][lane] = f;
            lds.e[buf][k + u][lane] = e;
        }
    }
}

// One pass over all partners.  Returns the sum of this wavefront's chain
// (wavefronts 0-3: e, gx, gy, gz of the lane's atom).
template <int POT, bool IEEE>
__device__ __forceinline__ double split_pass(SplitLds& lds, int n, int tile, int wave, int lane,
                                             const double* __restrict__ px, int64_t total,
                                             const Units& u, const double (&x)[3], double rho) {
    const int chunks = (n + kChunk - 1) / kChunk;
    const double c = -2.0 * rho;
    double k24, km48;
    hold_constants(k24, km48);
    double sum = 0.0;
    const int q = wave - 4;  // producer: partners kShare q .. of a chunk
    // the coordinates of a producer's next partners, one lane per partner
    // and component; partners past the end are given the last one's (their
    // terms are not added)
    auto fetch = [&](int ch) {
        const int d = lane / kShare, j = min(ch * kChunk + kShare * q + lane % kShare, n - 1);
        double v = d < 3 ? px[d * total + j] : 0.0;
        return u.scaled ? v / u.sigma : v;
    };
    double next = 0.0;
    if (q >= 0) next = fetch(0);
    for (int it = 0; it <= chunks; ++it) {
        if (q >= 0) {
            if (it < chunks) {
                const int buf = it & 1;
                if (lane < 3 * kShare)
                    lds.pos[buf][lane / kShare][kShare * q + lane % kShare] = next;
                if (it + 1 < chunks) next = fetch(it + 1);
                wave_sync();
                const int k0 = kShare * q, cnt = min(kShare, n - it * kChunk - k0);
                if (it == tile)
                    split_terms<POT, IEEE, true>(lds, buf, k0, cnt, x, rho, c, k24, km48, lane);
                else
                    split_terms<POT, IEEE, false>(lds, buf, k0, cnt, x, rho, c, k24, km48, lane);
            }
        } else if (it > 0) {
            const int buf = (it - 1) & 1;
            const int cnt = min(kChunk, n - (it - 1) * kChunk);
            constexpr int G = 8;
            int k = 0;
            if (wave == 0) {
                for (; k + G <= cnt; k += G) {
                    double t[G];
#pragma unroll
                    for (int g = 0; g < G; ++g) t[g] = lds.e[buf][k + g][lane];
#pragma unroll
                    for (int g = 0; g < G; ++g) sum = sum + t[g];
                }
                for (; k < cnt; ++k) sum = sum + lds.e[buf][k][lane];
            } else {
                const double* pd = lds.pos[buf][wave - 1];
                const double xd = wave == 1 ? x[0] : wave == 2 ? x[1] : x[2];
                for (; k + G <= cnt; k += G) {
                    double t[G], p[G];
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        t[g] = lds.f[buf][k + g][lane];
                        p[g] = pd[k + g];
                    }
#pragma unroll
                    for (int g = 0; g < G; ++g) sum = fma(t[g], xd - p[g], sum);
                }
                for (; k < cnt; ++k) sum = fma(lds.f[buf][k][lane], xd - pd[k], sum);
            }
        }
        __syncthreads();
    }
    return sum;
}

// Workgroup (x, b, z) takes tile x + z nt of cluster b: first the tiles that clusters
// up to max_n have (nt of them, z = 0), then those that only a cluster above
// max_n has (z = 1).  Workgroups go to the eight XCDs in turn, so with nt_max (a power
// of two) of them per cluster in order the empty ones of every cluster fell to
// the same XCDs: 102 x LJ300, 5 of 8 tiles, 26 us now and 46 so, 93 x LJ700 93 and
// 132.  The FP32 path's workgroups, many per cluster or short, gain nothing by it.
template <int POT>
__global__ __launch_bounds__(kSplitBlock) void split64_kernel(const int32_t* offset, int64_t total,
                                                              const double* xyz, double* grad,
                                                              double* partial, int nt_max,
                                                              double rho, Units u) {
    __shared__ SplitLds lds;
    __shared__ int again;
    const int b = blockIdx.y, tile = blockIdx.x + blockIdx.z * gridDim.x;
    const int o = offset[b], n = offset[b + 1] - o;
    if (n <= tile * kWave || n > nt_max * kWave) return;  // (the second: reported as NaN)
    const int lane = threadIdx.x % kWave, wave = uniform((int)threadIdx.x / kWave);
    const int i = tile * kWave + lane;
    const double* px = xyz + o;
    double x[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        x[c] = i < n ? px[c * total + i] : 0.0;
        if (u.scaled) x[c] = x[c] / u.sigma;
    }
    double s = split_pass<POT, false>(lds, n, tile, wave, lane, px, total, u, x, rho);
    double es = 0.0;
    if (wave == 0) es = wave_sum(i < n ? s : 0.0);
    if constexpr (POT == kPairLJ) {
        // a pair distance outside the range of recip_in_range makes the sums of
        // both its atoms' tiles not finite: those tiles repeat with the IEEE
        // division (in the others the two forms give the same bits)
        if (threadIdx.x == 0) again = !isfinite(es);
        __syncthreads();
        if (again) {
            s = split_pass<POT, true>(lds, n, tile, wave, lane, px, total, u, x, rho);
            if (wave == 0) es = wave_sum(i < n ? s : 0.0);
        }
    }
    if (threadIdx.x == 0) partial[b * nt_max + tile] = es;
    if (grad && wave >= 1 && wave <= 3 && i < n) grad[(wave - 1) * total + o + i] = s * u.gscale;
}

// The energy of each cluster: the pairwise sum of its tiles' sums.
template <int POT>
__global__ __launch_bounds__(kWave) void split_energy_kernel(const int32_t* offset,
                                                             const double* partial, int nt_max,
                                                             double* energy, Units u) {
    const int b = blockIdx.x, t = threadIdx.x;
    const int n = offset[b + 1] - offset[b];
    if (n < 0 || n > nt_max * kWave) {  // offsets disagree with the host max_n
        if (t == 0) energy[b] = __builtin_nan("");
        return;
    }
    const double s = wave_sum(t * kWave < n ? partial[b * nt_max + t] : 0.0);
    if (t == 0) energy[b] = (POT == kPairMorse ? 0.5 : 2.0) * s * u.escale;
}

// ---------------------------------------------------------------------------
// FP32.  A unit is one pair of 64-atom tiles; its wavefront stores, per lane,
// its FP32 sums (own[unit][lane] = e, gx, gy, gz) and, on the unique-pair
// tiles, the reaction on the partner tile's atoms (react[unit][component]).
// Unique-pair tiles (as pairs_tiles; Eq. (1), 32 < n <= 2048): unit
// t nt + tau is round t of tile tau, round 0 its own pairs.  Otherwise (as
// pairs_mixed): unit J nt + tau holds tile tau's sums over tile J.
// ---------------------------------------------------------------------------
constexpr int kUnitWaves = 4;

__device__ __forceinline__ bool unit_tiles(int pot, int n, int nt_max) {
    return pot == kPairLJ && nt_max * kWave <= 2048 && tiles_for(n);
}
__device__ __forceinline__ int unit_count(bool tiles, int nt) {
    return tiles ? nt * (nt / 2 + 1) : nt * nt;
}

template <int POT>
__global__ __launch_bounds__(kUnitWaves* kWave) void split32_kernel(
    const int32_t* offset, int64_t total, const double* xyz, float4* own, float* react, int nt_max,
    int units_max, double rho, Units u) {
    __shared__ float4 stage[kUnitWaves][2 * kWave];
    const int wg_per = (units_max + kUnitWaves - 1) / kUnitWaves;
    const int b = blockIdx.x / wg_per;
    const int wave = uniform((int)threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int unit = (blockIdx.x % wg_per) * kUnitWaves + wave;
    const int o = offset[b], n = offset[b + 1] - o;
    if (n <= 0 || n > nt_max * kWave) return;
    const int nt = (n + kWave - 1) / kWave;
    const bool tiles = unit_tiles(POT, n, nt_max);
    if (unit >= unit_count(tiles, nt)) return;
    const int tau = unit % nt, round = unit / nt;
    auto load = [&](int i) {
        if (i >= n) return tile_pad(i);
        float v[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            double t = xyz[c * total + o + i];
            if (u.scaled) t = t / u.sigma;
            v[c] = (float)t;
        }
        return make_float4(v[0], v[1], v[2], 0.0f);
    };
    float4* pos = stage[wave];
    const float4 pi = load(tau * kWave + lane);
    const size_t at = (size_t)b * units_max + unit;
    if (!tiles) {
        const int j0 = round * kWave, j1 = min(n, j0 + kWave);
        pos[lane] = load(j0 + lane);
        wave_sync();
        const float rf = (float)rho, cf = -2.0f * rf;
        const int self = round == tau ? lane : -1;
        float te = 0.0f, tx = 0.0f, ty = 0.0f, tz = 0.0f;
        auto pair = [&](const float4 p, bool is_self) {
            if constexpr (POT == kPairMorse)
                pair_morse32(p, is_self, pi.x, pi.y, pi.z, rf, cf, te, tx, ty, tz);
            else
                pair_fp32(p, is_self, pi.x, pi.y, pi.z, te, tx, ty, tz);
        };
        const int cnt = j1 - j0;
        int k = 0;
        for (; k + kGroup32 <= cnt; k += kGroup32) {
            float4 p[kGroup32];
#pragma unroll
            for (int v = 0; v < kGroup32; ++v) p[v] = pos[k + v];
#pragma unroll
            for (int v = 0; v < kGroup32; ++v) pair(p[v], k + v == self);
        }
        for (; k < cnt; ++k) pair(pos[k], k == self);
        own[at * kWave + lane] = make_float4(te, tx, ty, tz);
        return;
    }
    if constexpr (POT == kPairLJ) {
        int J = tau + round;
        if (J >= nt) J -= nt;
        const float4 pj = round == 0 ? pi : load(J * kWave + lane);
        pos[lane] = pj;
        pos[kWave + lane] = pj;
        wave_sync();
        float te = 0.0f, tx = 0.0f, ty = 0.0f, tz = 0.0f;
        float3 r;
        int d = lane;  // the partner atom whose reaction this lane ends with
        if (round == 0) {
            r = tile_diagonal(pi, pos, lane, te, tx, ty, tz);
        } else if (nt % 2 == 0 && round == nt / 2) {
            const int k_begin = tau < nt / 2 ? 0 : 1;
            r = tile_pair<kWave / 2>(pi, pos, lane, k_begin, te, tx, ty, tz);
            d = (lane + k_begin + kWave / 2 - 1) & (kWave - 1);
        } else {
            r = tile_pair<kWave>(pi, pos, lane, 0, te, tx, ty, tz);
            d = (lane + kWave - 1) & (kWave - 1);
        }
        own[at * kWave + lane] = make_float4(te, tx, ty, tz);
        float* rr = react + at * 3 * kWave + d;
        rr[0] = r.x;
        rr[kWave] = r.y;
        rr[2 * kWave] = r.z;
    }
}

// One wavefront per tile: the units' FP32 sums added in FP64 in the order of
// pairs_tiles / pairs_mixed.
template <int POT>
__global__ __launch_bounds__(kWave) void split32_sum_kernel(const int32_t* offset, int64_t total,
                                                            const float4* own, const float* react,
                                                            double* grad, double* partial,
                                                            int nt_max, int units_max, Units u) {
    const int b = blockIdx.x / nt_max, tau = blockIdx.x % nt_max;
    const int o = offset[b], n = offset[b + 1] - o;
    if (n <= tau * kWave || n > nt_max * kWave) return;
    const int nt = (n + kWave - 1) / kWave, lane = threadIdx.x;
    const bool tiles = unit_tiles(POT, n, nt_max);
    const float4* ow = own + (size_t)b * units_max * kWave + lane;
    const float* re = react + (size_t)b * units_max * 3 * kWave + lane;
    double e = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
    if (tiles) {
        for (int t = 0; t <= nt / 2; ++t) {
            const float4 s = ow[(size_t)(t * nt + tau) * kWave];
            int from = tau - t;  // the tile whose partner in round t is this one
            if (from < 0) from += nt;
            const float* r = re + (size_t)(t * nt + from) * 3 * kWave;
            const float rx = r[0], ry = r[kWave], rz = r[2 * kWave];
            e += 2.0 * (double)s.x;
            gx += (double)s.y;
            gy += (double)s.z;
            gz += (double)s.w;
            gx += (double)rx;
            gy += (double)ry;
            gz += (double)rz;
        }
    } else {
        for (int J = 0; J < nt; ++J) {
            const float4 s = ow[(size_t)(J * nt + tau) * kWave];
            e += (double)s.x;
            gx += (double)s.y;
            gy += (double)s.z;
            gz += (double)s.w;
        }
    }
    const int i = tau * kWave + lane;
    const double es = wave_sum(i < n ? e : 0.0);
    if (lane == 0) partial[blockIdx.x] = es;
    if (grad && i < n) {
        grad[o + i] = gx * u.gscale;
        grad[total + o + i] = gy * u.gscale;
        grad[2 * total + o + i] = gz * u.gscale;
    }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
int split_units(int pot, int nt) {
    return pot == kPairLJ && nt * kWave <= 2048 ? nt * (nt / 2 + 1) : nt * nt;
}

static size_t align256(size_t v) { return (v + 255) / 256 * 256; }

size_t split_eval_bytes(int mixed, int pot, int num, int max_n) {
    const EvalShape s = eval_shape(max_n);
    const int nt = s.W * s.A;  // the tiles that the one-workgroup kernel would hold
    size_t bytes = align256((size_t)num * nt * sizeof(double));
    if (mixed) {
        const size_t units = (size_t)num * split_units(pot, nt);
        bytes += align256(units * kWave * sizeof(float4));
        if (pot == kPairLJ && nt * kWave <= 2048)
            bytes += align256(units * 3 * kWave * sizeof(float));
    }
    return bytes;
}

template <int POT>
static hipError_t launch_split_t(int mixed, int num, int max_n, const int32_t* off, int64_t total,
                                 const double* xyz, double* energy, double* grad, double rho,
                                 Units u, char* ws, hipStream_t st) {
    const EvalShape s = eval_shape(max_n);
    const int nt_max = s.W * s.A, nt = (max_n + kWave - 1) / kWave;  // max_n > 256
    double* partial = reinterpret_cast<double*>(ws);
    if (!mixed) {
        // nt <= nt_max < 2 nt, and the rule keeps num below 65536
        hipLaunchKernelGGL((split64_kernel<POT>), dim3(nt, num, nt < nt_max ? 2 : 1),
                           dim3(kSplitBlock), 0, st, off, total, xyz, grad, partial, nt_max, rho,
                           u);
    } else {
        const int units = split_units(POT, nt_max);
        char* p = ws + align256((size_t)num * nt_max * sizeof(double));
        float4* own = reinterpret_cast<float4*>(p);
        float* react =
            reinterpret_cast<float*>(p + align256((size_t)num * units * kWave * sizeof(float4)));
        const int wgs = num * ((units + kUnitWaves - 1) / kUnitWaves);
        hipLaunchKernelGGL((split32_kernel<POT>), dim3(wgs), dim3(kUnitWaves * kWave), 0, st, off,
                           total, xyz, own, react, nt_max, units, rho, u);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((split32_sum_kernel<POT>), dim3(num * nt_max), dim3(kWave), 0, st, off,
                           total, own, react, grad, partial, nt_max, units, u);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((split_energy_kernel<POT>), dim3(num), dim3(kWave), 0, st, off, partial,
                       nt_max, energy, u);
    return hipGetLastError();
}

hipError_t launch_split_eval(int mixed, int pot, int num, int max_n, const int32_t* off,
                             int64_t total, const double* xyz, double* energy, double* grad,
                             double rho, Units u, char* ws, hipStream_t st) {
    return pot == kPairMorse ? launch_split_t<kPairMorse>(mixed, num, max_n, off, total, xyz,
                                                          energy, grad, rho, u, ws, st)
                             : launch_split_t<kPairLJ>(mixed, num, max_n, off, total, xyz, energy,
                                                       grad, rho, u, ws, st);
}

}  // namespace lj
