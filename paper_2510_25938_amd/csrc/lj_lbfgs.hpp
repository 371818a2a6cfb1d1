// The team of one cluster (LDS buffers, reductions, evaluation), the L-BFGS
// history and the L-BFGS loop itself, shared by the minimiser kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "lj_kernels.hpp"

namespace lj {

// ---------------------------------------------------------------------------
// Team: LDS buffers and the collective operations of one workgroup, or (G > 1)
// of one of the G clusters packed in a one-wavefront workgroup, each on its
// own 64 / G lanes.  A packed team's values are uniform over its lanes only,
// so its reductions stay within those lanes and nothing is read out as a
// wavefront-uniform scalar; LDS order within one wavefront needs no barrier
// (a wavefront's LDS instructions execute in issue order).
// ---------------------------------------------------------------------------
// UP (Morse pair): the FP64 evaluation takes the unique-pair form
// (pairs_morse64_up) for clusters of at most up_n atoms, with an up_n x up_n
// pair matrix at upm.
// TILES: FP32 evaluations above 32 atoms take the unique-pair tiles (their own
// summation order; without, the ordered loop).
template <int W, int A, int POT, int L = kWave, int G = 1, bool UP = false,
          bool TILES = kUseTiles<W, A>>
struct Team {
    static_assert(G == 1 || (W == 1 && A == 1 && L == kWave), "packing: one wavefront, one slot");
    static_assert(!UP || (W == 1 && A == 1 && G == 1 && POT == kPairMorse),
                  "unique pairs: Morse pair, one wavefront, one cluster");
    static constexpr int T = kWave * W;
    static constexpr int NVMAX = 4 * A;
    static constexpr int kG = G;
    double4* pos64;  // this team's atoms (a packed team: its own part of the buffer)
    float4* pos32;
    float* rbuf;  // reaction buffers of the FP32 tiles and the one-wavefront ring
    TeamScratch<W, NVMAX>* sc;
    int bank;
    int n;
    int li;      // atom index of this thread's slot 0 within the cluster
    double rho;  // Morse range (POT == kPairMorse)
    uint32_t top;  // morse_top(rho)
    double2* upm;    // up_n x up_n pair matrix
    uint2* uplist;   // up_n (up_n - 1) / 2 pair-list entries
    int up_n;

    // Before the first evaluation of a cluster (n set): its pair list.
    __device__ __forceinline__ void prepare() {
        if constexpr (UP) {
            if (n <= up_n) {
                up_pair_list(n, uplist, li);
                __syncthreads();
            }
        }
    }

    __device__ __forceinline__ bool active(int a) const { return a * T + li < n; }

    // a value uniform over the team, as the team's scalar
    __device__ __forceinline__ int uni(int v) const {
        if constexpr (G > 1)
            return v;
        else
            return uniform(v);
    }

    __device__ __forceinline__ void sync() const {
        if constexpr (G > 1) {
            wave_sync();
        } else {
            __syncthreads();
        }
    }

    __device__ __forceinline__ double dot(const double (&u)[3][A], const double (&v)[3][A]) {
        double p[1][A], o[1];
#pragma unroll
        for (int a = 0; a < A; ++a) p[0][a] = fma(u[2][a], v[2][a], fma(u[1][a], v[1][a], u[0][a] * v[0][a]));
        if constexpr (G > 1) return group_sum<G>(p[0][0]);
        team_sum<W, A, 1, NVMAX, L>(p, o, *sc, bank);
        return o[0];
    }

    // (s.y, y.y, s.s, w.w) in one reduction.
    __device__ __forceinline__ void dot4(const double (&s)[3][A], const double (&y)[3][A],
                                         const double (&w)[3][A], double& sy, double& yy,
                                         double& ss, double& ww) {
        double p[4][A], o[4];
#pragma unroll
        for (int a = 0; a < A; ++a) {
            p[0][a] = fma(s[2][a], y[2][a], fma(s[1][a], y[1][a], s[0][a] * y[0][a]));
            p[1][a] = fma(y[2][a], y[2][a], fma(y[1][a], y[1][a], y[0][a] * y[0][a]));
            p[2][a] = fma(s[2][a], s[2][a], fma(s[1][a], s[1][a], s[0][a] * s[0][a]));
            p[3][a] = fma(w[2][a], w[2][a], fma(w[1][a], w[1][a], w[0][a] * w[0][a]));
        }
        if constexpr (G > 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = group_sum<G>(p[k][0]);
        } else {
            team_sum<W, A, 4, NVMAX, L>(p, o, *sc, bank);
        }
        sy = o[0];
        yy = o[1];
        ss = o[2];
        ww = o[3];
    }

    // Largest per-atom squared norm of v.
    __device__ __forceinline__ double max_atom_norm2(const double (&v)[3][A]) {
        double m[A];
#pragma unroll
        for (int a = 0; a < A; ++a) m[a] = fma(v[2][a], v[2][a], fma(v[1][a], v[1][a], v[0][a] * v[0][a]));
        if constexpr (G > 1) return group_max<G>(m[0]);
        return team_max<W, A, NVMAX, L>(m, *sc, bank);
    }

    // u.v and the largest per-atom squared norm of v, with the same values as
    // dot() and max_atom_norm2() but one exchange between the wavefronts.
    // vmax2 is exact whenever it exceeds cap2; otherwise it is some value
    // <= cap2 (one wavefront: a ballot over the lanes skips the max when no
    // atom exceeds cap2).
    __device__ __forceinline__ void dot_max(const double (&u)[3][A], const double (&v)[3][A],
                                            double& uv, double& vmax2, double cap2) {
        double p[A], m = 0.0;
        double ws[A];
#pragma unroll
        for (int a = 0; a < A; ++a) {
            p[a] = fma(u[2][a], v[2][a], fma(u[1][a], v[1][a], u[0][a] * v[0][a]));
            const double n2 = fma(v[2][a], v[2][a], fma(v[1][a], v[1][a], v[0][a] * v[0][a]));
            m = a == 0 ? n2 : fmax(m, n2);
        }
        if constexpr (G > 1) {
            // a packed team: any value <= cap2 serves when no atom of the
            // wavefront exceeds cap2
            uv = group_sum<G>(p[0]);
            vmax2 = __builtin_amdgcn_ballot_w64(m > cap2) != 0 ? group_max<G>(m) : 0.0;
            return;
        }
        if constexpr (W == 1 && A == 2) {
            uv = wave_sum_slots(p[0], p[1]);
            vmax2 = __builtin_amdgcn_ballot_w64(m > cap2) != 0 ? wave_max<L>(m) : 0.0;
            return;
        }
#pragma unroll
        for (int a = 0; a < A; ++a) ws[a] = wave_sum<L>(p[a]);
        if constexpr (W == 1) {
            uv = tree<A>(ws);
            vmax2 = __builtin_amdgcn_ballot_w64(m > cap2) != 0 ? wave_max<L>(m) : 0.0;
        } else {
            m = wave_max<L>(m);
            const int w = threadIdx.x / kWave;
            if (threadIdx.x % kWave == 0) {
#pragma unroll
                for (int a = 0; a < A; ++a) sc->v[bank][a][w] = ws[a];
                sc->v[bank][A][w] = m;
            }
            __syncthreads();
            double r[A];
#pragma unroll
            for (int a = 0; a < A; ++a) {
                if constexpr (W >= 8) {
                    r[a] = lane_tree<W>(sc->v[bank][a]);
                } else {
                    double rw[W];
#pragma unroll
                    for (int q = 0; q < W; ++q) rw[q] = sc->v[bank][a][q];
                    r[a] = tree_w<W>(rw);
                }
            }
            double mx = sc->v[bank][A][0];
            if constexpr (W >= 8) {
                mx = lane_max<W>(sc->v[bank][A]);
            } else {
#pragma unroll
                for (int q = 1; q < W; ++q) mx = fmax(mx, sc->v[bank][A][q]);
            }
            bank ^= 1;
            uv = uniform(tree<A>(r));
            vmax2 = uniform(mx);
        }
    }

    // E and g at x.  FP64: the ordered-pair loop in the oracle's order.
    // F32: FP32 pair arithmetic and per-atom FP32 partial sums, FP64 totals;
    // the unique-pair ring for one-wavefront clusters of 20 to 43 atoms, the
    // unique-pair 64-atom tiles above 32 atoms otherwise (Eq. (1)), else the
    // ordered loop.  Every loop reports e_i in the ordered-pair convention,
    // which counts each pair twice: E = 2 sum_i e_i for Eq. (1) (e_i holds
    // r^-12 - r^-6, a quarter of the pair energy) and E = 0.5 sum_i e_i for
    // the Morse pair (e_i holds V).
    template <bool F32>
    __device__ __forceinline__ double eval(const double (&x)[3][A], double (&g)[3][A]) {
        constexpr bool kTiles = F32 && POT == kPairLJ && TILES && G == 1;
        constexpr bool kRing = F32 && W == 1 && A == 1 && G == 1;
        bool ring = false, tiles = false;
        if constexpr (kRing) ring = ring_for(n);
        if constexpr (kTiles) tiles = !ring && tiles_for(n);
        sync();  // previous readers of the position and reaction buffers are done
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const int i = a * T + li;
            if (ring) {  // ring layout: pos[j] = atom j mod n for j < 64 + steps
                if (i < n) {
                    const float4 p = make_float4((float)x[0][a], (float)x[1][a], (float)x[2][a],
                                                 0.0f);
                    const int end = kWave + ring_steps(n);
                    for (int j = i; j < end; j += n) pos32[j] = p;
                }
            } else if (tiles) {  // tile layout: each 64-atom tile twice, padded
                if (i < ((n + kWave - 1) / kWave) * kWave) {
                    const float4 p = i < n ? make_float4((float)x[0][a], (float)x[1][a],
                                                         (float)x[2][a], 0.0f)
                                           : tile_pad(i);
                    pos32[2 * i - (i & 63)] = p;
                    pos32[2 * i - (i & 63) + 64] = p;
                }
            } else if (i < n) {
                if constexpr (F32)
                    pos32[i] = make_float4((float)x[0][a], (float)x[1][a], (float)x[2][a], 0.0f);
                else
                    pos64[i] = make_double4(x[0][a], x[1][a], x[2][a], 0.0);
            }
        }
        sync();
        double e[1][A], o[1];
        if (ring) {
            if constexpr (kRing) pairs_ring<POT>(n, pos32, rbuf, e[0][0], g, rho);
        } else if (tiles) {
            if constexpr (kTiles) pairs_tiles<W, A>(n, pos32, rbuf, e[0], g);
        } else if constexpr (F32) {
            pairs_mixed<A, T, POT>(n, pos32, x, e[0], g, rho,
                                   W == 1 ? 0 : uniform((int)threadIdx.x / kWave), li);
        } else {
            MorseRange range;
            bool general = POT == kPairMorse && top == 0;
            if (!general) {
                if constexpr (POT == kPairMorse) range.coefs.hold();
                fp64_pairs<false>(x, e[0], g, range);
                // a pair outside the range of the short forms: this wavefront
                // repeats its sums with the general square root and division
                // (unique pairs: every lane takes some; else the lanes of atoms)
                if constexpr (POT == kPairMorse) {
                    const bool takes = (UP && n <= up_n) || active(0);
                    general = __builtin_amdgcn_ballot_w64(takes && !range.holds(top)) != 0;
                }
            }
            if (POT == kPairMorse && general) {
                MorseRange any;
                any.coefs.hold();
                fp64_pairs<true>(x, e[0], g, any);
            }
        }
#pragma unroll
        for (int a = 0; a < A; ++a)
            if (!active(a)) e[0][a] = g[0][a] = g[1][a] = g[2][a] = 0.0;
        sum_energy(e, o);
        if constexpr (!F32 && POT == kPairLJ) {
            // only a pair distance outside the range of recip_in_range can make
            // 1/r2 differ from the IEEE quotient, and it makes E not finite:
            // then the evaluation is repeated with the IEEE division
            if (!isfinite(o[0])) {
                MorseRange range;
                fp64_pairs<true>(x, e[0], g, range);
#pragma unroll
                for (int a = 0; a < A; ++a)
                    if (!active(a)) e[0][a] = g[0][a] = g[1][a] = g[2][a] = 0.0;
                sum_energy(e, o);
            }
        }
        return (POT == kPairMorse ? 0.5 : 2.0) * o[0];
    }

    template <bool IEEE>
    __device__ __forceinline__ void fp64_pairs(const double (&x)[3][A], double (&e)[A],
                                               double (&g)[3][A], MorseRange& range) {
        if constexpr (UP) {
            if (n <= up_n) {
                pairs_morse64_up<IEEE>(n, pos64, upm, uplist, x, e, g, rho, li, range);
                return;
            }
        }
        pairs_fp64<A, T, POT, IEEE, (G > 1)>(
            n, pos64, x, e, g, rho, W == 1 ? 0 : uniform((int)threadIdx.x / kWave), li, range);
    }

    __device__ __forceinline__ void sum_energy(double (&e)[1][A], double (&o)[1]) {
        if constexpr (G > 1)
            o[0] = group_sum<G>(e[0][0]);
        else
            team_sum<W, A, 1, NVMAX, L>(e, o, *sc, bank);
    }
};

// ---------------------------------------------------------------------------
// L-BFGS history.  rho is kept by age (slot 0 = newest) in registers; the
// vectors either by age in registers (HREG, shifted on every push) or in a
// global ring owned by the persistent workgroup.
// ---------------------------------------------------------------------------
template <int W, int A, bool HREG>
struct History;

template <int W, int A>
struct History<W, A, true> {
    double S[kMaxM][3][A];
    double Y[kMaxM][3][A];
    double rho[kMaxM];
    int hist = 0;
    double gamma = 1.0;

    __device__ __forceinline__ void init(double*, double*, int) { hist = 0; gamma = 1.0; }
    __device__ __forceinline__ void clear() { hist = 0; }

    __device__ __forceinline__ void push(const double (&s)[3][A], const double (&y)[3][A], double r,
                                         double gam, int m) {
#pragma unroll
        for (int k = kMaxM - 1; k > 0; --k) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int a = 0; a < A; ++a) {
                    S[k][c][a] = S[k - 1][c][a];
                    Y[k][c][a] = Y[k - 1][c][a];
                }
            rho[k] = rho[k - 1];
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int a = 0; a < A; ++a) {
                S[0][c][a] = s[c][a];
                Y[0][c][a] = y[c][a];
            }
        rho[0] = r;
        gamma = gam;
        hist = hist < m ? hist + 1 : m;
    }

    // r <- H r with all kMaxM pairs present: the same operations as apply(),
    // with no per-pair guards (no branches or register copies between pairs).
    template <class TM>
    __device__ __forceinline__ void apply_full(TM& tm, double (&r)[3][A]) {
        double al[kMaxM];
#pragma unroll
        for (int k = 0; k < kMaxM; ++k) {
            const double a = rho[k] * tm.dot(S[k], r);
            al[k] = a;
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int q = 0; q < A; ++q) r[c][q] = fma(-a, Y[k][c][q], r[c][q]);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int q = 0; q < A; ++q) r[c][q] = gamma * r[c][q];
#pragma unroll
        for (int k = kMaxM - 1; k >= 0; --k) {
            const double b = rho[k] * tm.dot(Y[k], r);
            const double w = al[k] - b;
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int q = 0; q < A; ++q) r[c][q] = fma(w, S[k][c][q], r[c][q]);
        }
    }

    // r <- H r (r holds g on entry).
    template <class TM>
    __device__ __forceinline__ void apply(TM& tm, double (&r)[3][A]) {
        const int h = tm.uni(hist);
        if (h == kMaxM) {
            apply_full(tm, r);
            return;
        }
        double al[kMaxM];
#pragma unroll
        for (int k = 0; k < kMaxM; ++k) {
            if (k < h) {
                const double a = rho[k] * tm.dot(S[k], r);
                al[k] = a;
#pragma unroll
                for (int c = 0; c < 3; ++c)
#pragma unroll
                    for (int q = 0; q < A; ++q) r[c][q] = fma(-a, Y[k][c][q], r[c][q]);
            }
        }
        if (h > 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int q = 0; q < A; ++q) r[c][q] = gamma * r[c][q];
        }
#pragma unroll
        for (int k = kMaxM - 1; k >= 0; --k) {
            if (k < h) {
                const double b = rho[k] * tm.dot(Y[k], r);
                const double w = al[k] - b;
#pragma unroll
                for (int c = 0; c < 3; ++c)
#pragma unroll
                    for (int q = 0; q < A; ++q) r[c][q] = fma(w, S[k][c][q], r[c][q]);
            }
        }
    }
};

// One atom per lane, two wavefronts per SIMD (256 registers): the kMaxM pairs
// take 120 registers, which the mixed kernel does not have beside its two
// evaluations.  The KR newest pairs stay in registers by age; a push
// hands the oldest of them to a ring in LDS, where an atom's pair is a 48-byte
// record (three 16-byte reads per lane, which touch every bank once per eight
// lanes), read ahead of the reductions.  With it the mixed kernels of 1, 2 and 3
// wavefronts fit 256 registers with at most 28 bytes of scratch for Eq. (1) and 48
// for the Morse pair (304, 410 and 410 registers, Morse 322 and 396, with the
// whole history in registers; four wavefronts: 56 and 88 bytes of scratch).
template <int W, int KR>
struct HistoryHybrid {
    static constexpr int T = kWave * W;
    static constexpr int R = kMaxM - KR;  // pairs in LDS
    static constexpr int kRecord = 3;     // double2
    static constexpr int kBytes =
        R * T * kRecord * (int)sizeof(double2) + kMaxM * (int)sizeof(double);
    double S[KR][3], Y[KR][3];
    double rho[kMaxM];
    double2* ring;  // this lane's record in slot 0
    double* alpha;  // the recursion's alphas, equal in every lane
    int at = 0;     // slot of age KR
    int hist = 0;
    double gamma = 1.0;

    struct Pair {
        double s[3][1], y[3][1];
    };

    __device__ __forceinline__ void init(char* lds) {
        ring = reinterpret_cast<double2*>(lds) + threadIdx.x * kRecord;
        alpha = reinterpret_cast<double*>(lds + R * T * kRecord * sizeof(double2));
        at = 0;
        hist = 0;
        gamma = 1.0;
    }
    __device__ __forceinline__ void clear() { hist = 0; }

    __device__ __forceinline__ Pair pair(int age) const {
        Pair p;
        if (age < KR) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                p.s[c][0] = S[age][c];
                p.y[c][0] = Y[age][c];
            }
        } else {
            int k = at - (age - KR);
            if (k < 0) k += R;
            const double2* q = ring + k * T * kRecord;
            const double2 u = q[0], v = q[1], w = q[2];
            p.s[0][0] = u.x;
            p.s[1][0] = u.y;
            p.s[2][0] = v.x;
            p.y[0][0] = v.y;
            p.y[1][0] = w.x;
            p.y[2][0] = w.y;
        }
        return p;
    }

    __device__ __forceinline__ void push(const double (&s)[3][1], const double (&y)[3][1], double r,
                                         double gam, int m) {
        at = at + 1 == R ? 0 : at + 1;
        double2* q = ring + at * T * kRecord;
        q[0] = make_double2(S[KR - 1][0], S[KR - 1][1]);
        q[1] = make_double2(S[KR - 1][2], Y[KR - 1][0]);
        q[2] = make_double2(Y[KR - 1][1], Y[KR - 1][2]);
#pragma unroll
        for (int k = KR - 1; k > 0; --k)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                S[k][c] = S[k - 1][c];
                Y[k][c] = Y[k - 1][c];
            }
#pragma unroll
        for (int k = kMaxM - 1; k > 0; --k) rho[k] = rho[k - 1];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            S[0][c] = s[c][0];
            Y[0][c] = y[c][0];
        }
        rho[0] = r;
        gamma = gam;
        hist = hist < m ? hist + 1 : m;
    }

    template <bool FULL, class TM>
    __device__ __forceinline__ void apply_n(TM& tm, double (&r)[3][1], int h) {
        Pair ahead = pair(KR);  // the pair of age KR, ahead of its turn
#pragma unroll
        for (int k = 0; k < kMaxM; ++k) {
            if (FULL || k < h) {
                const Pair p = k < KR ? pair(k) : ahead;
                if (k >= KR && k + 1 < kMaxM) ahead = pair(k + 1);
                const double a = rho[k] * tm.dot(p.s, r);
                alpha[k] = a;
#pragma unroll
                for (int c = 0; c < 3; ++c) r[c][0] = fma(-a, p.y[c][0], r[c][0]);
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) r[c][0] = gamma * r[c][0];
        if (FULL || h > KR) ahead = pair(FULL ? kMaxM - 1 : h - 1);
#pragma unroll
        for (int k = kMaxM - 1; k >= 0; --k) {
            if (FULL || k < h) {
                const Pair p = k < KR ? pair(k) : ahead;
                if (k > KR) ahead = pair(k - 1);
                const double b = rho[k] * tm.dot(p.y, r);
                const double w = alpha[k] - b;
#pragma unroll
                for (int c = 0; c < 3; ++c) r[c][0] = fma(w, p.s[c][0], r[c][0]);
            }
        }
    }

    template <class TM>
    __device__ __forceinline__ void apply(TM& tm, double (&r)[3][1]) {
        const int h = tm.uni(hist);
        if (h == kMaxM)
            apply_n<true>(tm, r, h);
        else if (h > 0)
            apply_n<false>(tm, r, h);
    }
};

// In global memory: a ring of kMaxM slots per workgroup; a slot holds, per atom
// slot and thread, the pair (s, y) as three 16-byte words, so a wavefront reads
// 1 KB at a time.  At N = 1000 the 256 rings (123 MB) are read from the last-level
// cache twice per iteration.  Both recursions read ahead of the reductions
// (their barriers wait for LDS only, so reads stay in flight across them), and
// the oldest kKeep pairs, the last of the first recursion and the first of the
// second, are kept in registers in between.  rho and the alphas, uniform over
// the workgroup, live in LDS (written by thread 0, read after a reduction's
// barrier) instead of 40 registers.  256 x LJ1000, per iteration: FP32 phase
// 127 -> 99 us, FP64 253 -> 220 us; 256 x LJ300 FP32 phase 63 -> 33 us (with 3 or
// 4 pairs kept at A = 1: 102 and 103 us, spills).
template <int W, int A>
struct History<W, A, false> {
    static constexpr int T = kWave * W;
    static constexpr int kSlot = 3 * A * T;  // double2 per slot
    static constexpr int kKeep = A == 1 ? 2 : A == 2 ? 3 : 1;
    double2* base;
    double* rho;    // LDS [slot]
    double* alpha;  // LDS [age]
    int hist = 0;
    int newest = -1;
    int m = 1;
    double gamma = 1.0;

    struct Pair {
        double2 v[A][3];  // (sx, sy), (sz, yx), (yy, yz)
        __device__ __forceinline__ void s(double (&o)[3][A]) const {
#pragma unroll
            for (int q = 0; q < A; ++q) {
                o[0][q] = v[q][0].x;
                o[1][q] = v[q][0].y;
                o[2][q] = v[q][1].x;
            }
        }
        __device__ __forceinline__ void y(double (&o)[3][A]) const {
#pragma unroll
            for (int q = 0; q < A; ++q) {
                o[0][q] = v[q][1].y;
                o[1][q] = v[q][2].x;
                o[2][q] = v[q][2].y;
            }
        }
    };

    __device__ __forceinline__ void init(double* b, double* lds, int mm) {
        base = reinterpret_cast<double2*>(b) + threadIdx.x;
        rho = lds;
        alpha = lds + kMaxM;
        m = mm > 0 ? mm : 1;
        hist = 0;
        newest = -1;
        gamma = 1.0;
    }
    __device__ __forceinline__ void clear() { hist = 0; }

    __device__ __forceinline__ int slot(int age) const {
        const int k = newest - age;
        return k < 0 ? k + m : k;
    }
    __device__ __forceinline__ Pair load(int age) const {
        const double2* p = base + (size_t)slot(age) * kSlot;
        Pair r;
#pragma unroll
        for (int q = 0; q < A; ++q)
#pragma unroll
            for (int w = 0; w < 3; ++w) r.v[q][w] = p[(q * 3 + w) * T];
        return r;
    }

    __device__ __forceinline__ void push(const double (&s)[3][A], const double (&y)[3][A], double r,
                                         double gam, int mm) {
        newest = newest + 1 == m ? 0 : newest + 1;
        double2* p = base + (size_t)newest * kSlot;
#pragma unroll
        for (int q = 0; q < A; ++q) {
            p[(q * 3 + 0) * T] = make_double2(s[0][q], s[1][q]);
            p[(q * 3 + 1) * T] = make_double2(s[2][q], y[0][q]);
            p[(q * 3 + 2) * T] = make_double2(y[1][q], y[2][q]);
        }
        if (threadIdx.x == 0) rho[newest] = r;
        gamma = gam;
        hist = hist < mm ? hist + 1 : mm;
    }

    // r <- r - a y, a = rho s.r
    template <class TM>
    __device__ __forceinline__ void first(TM& tm, const Pair& p, int age, double (&r)[3][A]) {
        double v[3][A];
        p.s(v);
        const double sr = tm.dot(v, r);
        const double a = rho[slot(age)] * sr;
        if (threadIdx.x == 0) alpha[age] = a;
        p.y(v);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int q = 0; q < A; ++q) r[c][q] = fma(-a, v[c][q], r[c][q]);
    }
    // r <- r + (alpha - rho y.r) s
    template <class TM>
    __device__ __forceinline__ void second(TM& tm, const Pair& p, int age, double (&r)[3][A]) {
        double v[3][A];
        p.y(v);
        const double yr = tm.dot(v, r);
        const double b = rho[slot(age)] * yr;
        const double w = alpha[age] - b;
        p.s(v);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int q = 0; q < A; ++q) r[c][q] = fma(w, v[c][q], r[c][q]);
    }

    template <class TM>
    __device__ __forceinline__ void apply(TM& tm, double (&r)[3][A]) {
        const int h = tm.uni(hist);
        if (h == 0) return;
        const int keep = h < kKeep ? h : kKeep;
        const int cut = h - keep;  // ages cut .. h - 1 are kept between the recursions
        Pair kept[kKeep];
        if (cut > 0) {
            Pair cur = load(0), next = load(1);
#pragma unroll 1
            for (int k = 0; k < cut; ++k) {
                const Pair ahead = load(k + 2 < h ? k + 2 : h - 1);
                first(tm, cur, k, r);
                cur = next;
                next = ahead;
            }
            kept[0] = cur;
            if constexpr (kKeep > 1) kept[1] = next;
        } else {
            kept[0] = load(0);
            if constexpr (kKeep > 1) kept[1] = load(h > 1 ? 1 : 0);
        }
#pragma unroll
        for (int c = 2; c < kKeep; ++c) kept[c] = load(cut + c < h ? cut + c : h - 1);
#pragma unroll
        for (int c = 0; c < kKeep; ++c)
            if (c < keep) first(tm, kept[c], cut + c, r);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int q = 0; q < A; ++q) r[c][q] = gamma * r[c][q];
        Pair cur = load(cut > 0 ? cut - 1 : 0), next = load(cut > 1 ? cut - 2 : 0);
#pragma unroll
        for (int c = kKeep - 1; c >= 0; --c)
            if (c < keep) second(tm, kept[c], cut + c, r);
#pragma unroll 1
        for (int k = cut - 1; k >= 0; --k) {
            const Pair ahead = load(k > 2 ? k - 2 : 0);
            second(tm, cur, k, r);
            cur = next;
            next = ahead;
        }
    }
};

// Phase outcomes (LJ_* statuses, plus the FP32 phase's stall exit).
constexpr int kStall = 100;
// Relative energy change that the FP64 line search treats as rounding noise.
constexpr double kLsResolution = 0x1.0p-50;
// The FP32 phase treats energy changes as noise-limited only once
// ||g|| < kNoiseZone * its tolerance: there the Armijo allowance and the exit
// after five accepted steps without a decrease apply.
constexpr double kNoiseZone = 100.0;
// Inside the noise zone the FP32 phase also ends after kZonePatience accepted
// steps without lowering the best gradient norm of the zone by 10 %.
constexpr int kZonePatience = 30;

// E and g at x with FP32 pair arithmetic when f32 (only compiled when CAN32).
template <bool CAN32, int A, class TM>
__device__ __forceinline__ double eval_phase(TM& tm, const double (&x)[3][A], double (&g)[3][A],
                                             bool f32) {
    if constexpr (CAN32) {
        if (f32) return tm.template eval<true>(x, g);
    }
    return tm.template eval<false>(x, g);
}

// One L-BFGS run from x (history cleared).  On return x, g, E hold the last
// accepted iterate.  f32 (a uniform runtime flag, so the mixed kernel holds a
// single copy of this loop for both phases) selects the FP32 pair arithmetic,
// the Armijo noise allowance and the stall exit of the mixed path's first
// phase.
template <bool CAN32, int A, class TM, class HS>
__device__ int lbfgs_run(TM& tm, HS& H, double (&x)[3][A], double (&g)[3][A], double& E,
                         double& gnorm, int& iters, int& evals, const LbfgsDev& p, double gtol,
                         int max_iter, bool f32_flag) {
    const bool F32 = CAN32 && f32_flag;
    double d[3][A], xt[3][A], gt[3][A];
    H.clear();
    E = eval_phase<CAN32>(tm, x, g, F32);
    ++evals;
    double gg = tm.dot(g, g);  // later iterations get it from the curvature reduction
    gnorm = sqrt(gg);
    int it = 0;
    int stall = 0;
    int zone_wait = 0;
    double zone_best = 1.0e300;
    const double ms2 = p.max_step * p.max_step;
    for (;;) {
        if (!isfinite(E) || !isfinite(gg)) {
            iters += it;
            return LJ_NONFINITE;
        }
        if (gnorm < gtol) {
            iters += it;
            return LJ_CONVERGED;
        }
        if (it >= max_iter) {
            iters += it;
            return LJ_MAXITER;
        }
        // d = -H g
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int a = 0; a < A; ++a) d[c][a] = g[c][a];
        H.apply(tm, d);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int a = 0; a < A; ++a) d[c][a] = -d[c][a];
        double gd, dmax2;
        tm.dot_max(g, d, gd, dmax2, ms2);
        if (tm.uni(H.hist) > 0 && !(gd < 0.0)) {
            H.clear();
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int a = 0; a < A; ++a) d[c][a] = -g[c][a];
            tm.dot_max(g, d, gd, dmax2, ms2);
        }
        if (dmax2 > ms2) {
            const double sc = p.max_step / sqrt(dmax2);
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int a = 0; a < A; ++a) d[c][a] = d[c][a] * sc;
            gd = tm.dot(g, d);
        }
        // backtracking Armijo line search
        const bool noise_zone = F32 && gnorm < kNoiseZone * gtol;
        double alpha = 1.0, Et = 0.0;
        bool ok = false;
        // relative energy change below which the energy comparison is decided
        // by rounding: 4 ulps of E in FP64, the FP32 noise allowance in the
        // FP32 phase
        const double resolution = F32 ? p.ls_noise : kLsResolution;
        for (int ls = 0; ls < p.max_ls; ++ls) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int a = 0; a < A; ++a) xt[c][a] = fma(alpha, d[c][a], x[c][a]);
            Et = eval_phase<CAN32>(tm, xt, gt, F32);
            ++evals;
            double rhs = fma(p.c1 * alpha, gd, E);
            // FP32 phase near its tolerance: the full quasi-Newton step may be
            // accepted within the FP32 energy noise; a backtracked step, or any
            // step farther from convergence, must show a real decrease
            if (noise_zone && alpha == 1.0) rhs = rhs + p.ls_noise * fabs(E);
            if (Et <= rhs) {
                ok = true;
                break;
            }
            // An energy change within the resolution of E cannot decide the
            // test; the gradients can (approximate Armijo condition:
            // g_t.d <= (2 c1 - 1) g.d).  In the FP32 phase this carries the
            // descent on below the gradient norm at which energy changes
            // vanish in the FP32 noise (about 0.04 at LJ38), down to the
            // phase's tolerance, so the FP64 polish starts close to the minimum
            if (fabs(Et - E) <= resolution * fabs(E) &&
                tm.dot(gt, d) <= (2.0 * p.c1 - 1.0) * gd) {
                ok = true;
                break;
            }
            alpha = alpha * 0.5;
        }
        // FP32 phase while atoms still overlap (E > 0): a step that lowers E
        // by less than the FP32 resolution of E made no measurable progress
        // (its direction was scaled down by the curvature of one extremely
        // stiff pair) and counts as a failed line search, so the history is
        // dropped for a steepest-descent restart
        if (ok && F32 && E > 0.0 && !(E - Et > p.ls_noise * E)) ok = false;
        if (!ok) {
            if (tm.uni(H.hist) > 0) {
                H.clear();
                continue;
            }
            iters += it;
            return LJ_LSFAIL;
        }
        // s = xt - x (into d), y = gt - g (into g)
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int a = 0; a < A; ++a) {
                d[c][a] = xt[c][a] - x[c][a];
                g[c][a] = gt[c][a] - g[c][a];
            }
        double sy, yy, ss, ggt;
        tm.dot4(d, g, gt, sy, yy, ss, ggt);
        if (ss == 0.0) {
            // Null step: the accepted trial point equals x, so no progress is
            // possible along d; treated as a failed line search.  g holds y
            // here; x_t == x implies g_t == g, so restore g from g_t.
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int a = 0; a < A; ++a) g[c][a] = gt[c][a];
            if (tm.uni(H.hist) > 0) {
                H.clear();
                continue;
            }
            iters += it;
            return LJ_LSFAIL;
        }
        // the square roots and quotients of this step are independent of one
        // another: formed together so their latencies overlap
        const double gn_t = sqrt(ggt);
        const double syy = sqrt(ss * yy);
        const double rho_t = 1.0 / sy;
        const double gam_t = sy / yy;
        if (p.m > 0 && sy > p.curv_eps * syy) H.push(d, g, rho_t, gam_t, p.m);
        stall = (Et < E || !noise_zone) ? 0 : stall + 1;
        if (noise_zone) {
            if (gnorm < 0.9 * zone_best) {
                zone_best = gnorm;
                zone_wait = 0;
            } else {
                ++zone_wait;
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int a = 0; a < A; ++a) {
                x[c][a] = xt[c][a];
                g[c][a] = gt[c][a];
            }
        E = Et;
        gg = ggt;
        gnorm = gn_t;
        ++it;
        if (stall >= 5 || zone_wait >= kZonePatience) {  // FP32 phase's noise zone only
            iters += it;
            return kStall;
        }
    }
}

// One cluster from its load to its results: atoms o .. o + n - 1 of the batch,
// results in row b (has: the team holds a cluster).
template <int MIXED, int A, class TM, class HS>
__device__ __forceinline__ void minimize_cluster(const MinArgs& args, TM& tm, HS& H, int b, int o,
                                                 int n, bool has) {
    constexpr int T = TM::T;
    const int64_t total = args.total;
    double x[3][A], g[3][A];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const int i = a * T + tm.li;
            x[c][a] = i < n ? args.xyz[c * total + o + i] : 0.0;
            if (args.u.scaled) x[c][a] = x[c][a] / args.u.sigma;
        }
    double E = 0.0, gn = 0.0;
    int iters = 0, evals = 0, st = LJ_CONVERGED;
    // Mixed: phase 0 is the FP32 phase, phase 1 the FP64 polish from its
    // end point (one call site, so one copy of the L-BFGS loop).
    for (int phase = MIXED ? 0 : 1; phase < 2; ++phase) {
        const bool f32 = phase == 0;
        const double gt = f32 ? fmax(args.p.gtol, args.p.gtol_mixed_per_atom * (double)n)
                              : args.p.gtol;
        const int r = lbfgs_run<MIXED != 0>(tm, H, x, g, E, gn, iters, evals, args.p, gt,
                                            args.p.max_iter, f32);
        if (!f32) {
            st = r;
            break;
        }
        if (args.xyz_switch) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int a = 0; a < A; ++a) {
                    const int i = a * T + tm.li;
                    if (i < n)
                        args.xyz_switch[c * total + o + i] =
                            args.u.scaled ? x[c][a] * args.u.sigma : x[c][a];
                }
        }
        if (!args.p.polish) {
            // report the FP32 end point re-evaluated in FP64
            E = tm.template eval<false>(x, g);
            ++evals;
            const double gg = tm.dot(g, g);
            gn = sqrt(gg);
            if (!isfinite(E) || !isfinite(gg))
                st = LJ_NONFINITE;
            else if (gn < args.p.gtol)
                st = LJ_CONVERGED;
            else if (r == LJ_CONVERGED || r == kStall || r == LJ_LSFAIL)
                st = LJ_SWITCHED;  // the FP32 phase reached its tolerance or resolution
            else
                st = r == LJ_NONFINITE ? LJ_LSFAIL : r;
            break;
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const int i = a * T + tm.li;
            if (i < n)
                args.xyz[c * total + o + i] = args.u.scaled ? x[c][a] * args.u.sigma : x[c][a];
        }
    if (has && tm.li == 0) {
        args.energy[b] = E * args.u.escale;
        args.gnorm[b] = gn * args.u.gscale;
        args.iters[b] = iters;
        args.evals[b] = evals;
        args.status[b] = st;
    }
}

}  // namespace lj
