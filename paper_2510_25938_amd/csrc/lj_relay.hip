// The minimiser with helper wavefronts (gfx950): one cluster of at most 128 atoms
// per workgroup, for calls that leave most of the chip idle.
//
// A lone wavefront issues one FP64 instruction every 6 cycles whatever the
// dependences, so a call of few clusters is bound by the instruction count of
// one wavefront: about half of it the ordered pair loop, the rest the L-BFGS
// recursion, which is serial.  Here wavefront 0 (the leader) runs the L-BFGS
// loop with its history in registers, and one or three more wavefronts, on the
// CU's other SIMDs, share the pair loop.  Its sums have a fixed order (partners
// ascending), so the partners are cut into consecutive segments: every
// wavefront forms the terms of its segment at once, in registers, and the
// per-atom sums are then handed from segment to segment through LDS, each
// wavefront adding its terms in turn.  Every addition is the one of the
// single-wavefront loop in the same order, so results are bitwise equal.
//
// Measured, us per L-BFGS iteration: LJ38 5.1 -> 4.1, LJ64 6.7 -> 4.7, LJ98
// 12.0 -> 9.9, Morse38 6.0 -> 4.8, Morse98 16.7 -> 12.2 (four wavefronts); 1024 x
// LJ38 3.2 -> 2.9 ms, 1024 x LJ64 5.7 -> 5.2 ms (two, with one workgroup's
// wavefronts filling the issue gaps of another's).  The history in LDS
// instead of the leader's registers cost 0.3-0.6 us per iteration.
#include <hip/hip_runtime.h>

#include "lj_lbfgs.hpp"

namespace lj {

// What the leader asks of the other wavefronts at an evaluation's first barrier.
enum RelayCmd { kRelayEval = 0, kRelayEvalIeee, kRelayNew, kRelayExit };

template <int A>
struct RelayLds {
    double4 pos[kWave * A];    // coordinates
    double2 acc[A][2][kWave];  // sums on their way: (e, gx), (gy, gz) per tile and lane
    int cmd, n;
    int outside[4];  // per tile and segment: a Morse pair outside the short forms' range
};

// First partner of segment s of S (s = S: n).  Segments grow, so that a
// wavefront's terms are ready when its predecessor hands over: with t
// instructions per term (21 for Eq. (1), about 50 for the Morse pair), 4 per
// term for the sums and about 35 for an exchange,
// n_1 t = n_0 (t + 4) + 35 and n_{s+1} t = n_s (t + 4) + 35.  Two segments of one
// tile: the second is at most the 20 terms that a helper's registers hold (64
// atoms, 30 in the second: 1024 x LJ64 5.8 instead of 5.2 ms).
template <int S, int POT, int A = 1>
__device__ __forceinline__ int relay_cut(int s, int n) {
    static_assert(S == 2 || S == 4, "2 or 4 segments");
    if (s <= 0) return 0;
    if (s >= S) return n;
    int v;
    if constexpr (S == 2)
        v = POT == kPairMorse ? 31 * n - 22
            : A == 1          ? max(29 * n - 48, 64 * (n - 20))
                              : 29 * n - 48;
    else if (POT == kPairMorse)
        v = s == 1 ? 14 * n - 57 : s == 2 ? 29 * n - 72 : 46 * n - 60;
    else
        v = s == 1 ? 12 * n - 130 : s == 2 ? 26 * n - 190 : 43 * n - 160;
    v >>= 6;
    return v < 0 ? 0 : v;
}

// One wavefront's way through the barriers of an evaluation after the first:
// its segment is taken after barrier seg (barrier 0 published the
// coordinates), and the last barrier publishes the last segments' sums.
template <int S>
__device__ __forceinline__ void relay_wait_turn(int seg) {
    for (int s = 0; s < seg; ++s) __syncthreads();
}
template <int S>
__device__ __forceinline__ void relay_wait_rest(int seg) {
    for (int s = seg; s < S; ++s) __syncthreads();
}

// Written by each wavefront in each Morse evaluation, before its last barrier.
__device__ __forceinline__ void relay_outside(int& out, bool atom, const MorseRange& range,
                                              uint32_t top) {
    out = __builtin_amdgcn_ballot_w64(atom && !range.holds(top)) != 0;
}

// Segment 0 of a tile (the leader's own, and with A = 2 a helper's): partners
// 0 .. j1 - 1, added directly, and handed on.
template <int A, int POT, bool IEEE>
__device__ __forceinline__ void relay_first(RelayLds<A>& lds, int j1, int tile, int lane,
                                            int n, const double (&x)[3][1], double rho,
                                            uint32_t top, double c, double k24, double km48) {
    MorseRange range;
    if constexpr (POT == kPairMorse) range.coefs.hold();
    double e[1] = {0.0}, g[3][1] = {{0.0}, {0.0}, {0.0}};
    // j1 <= 64: only tile 0 meets its own atoms
    if (tile == 0)
        pairs_fp64_range<1, POT, IEEE, true, false>(0, j1, 0, lane, lds.pos, x, e, g, rho, c, k24,
                                                   km48, range);
    else
        pairs_fp64_range<1, POT, IEEE, false, false>(0, j1, 0, lane, lds.pos, x, e, g, rho, c, k24,
                                                    km48, range);
    lds.acc[tile][0][lane] = make_double2(e[0], g[0][0]);
    lds.acc[tile][1][lane] = make_double2(g[1][0], g[2][0]);
    if constexpr (POT == kPairMorse && !IEEE)
        relay_outside(lds.outside[tile], tile * kWave + lane < n, range, top);
}

// Helper of a one-tile cluster (segment seg >= 1): NG groups of 4 terms and
// their coordinate differences in registers (a longer segment forms the rest
// while it adds them).  Entered with an evaluation's first barrier passed;
// serves evaluations until the leader asks for something else, and returns
// that.
template <int W, int POT, bool IEEE, int NG>
__device__ __forceinline__ int relay_helper(RelayLds<1>& lds, int n, int seg, int lane,
                                            double rho, uint32_t top) {
    constexpr int S = W;
    constexpr int CAP = kGroup64 * NG;
    const int j0 = relay_cut<S, POT>(seg, n), cnt = relay_cut<S, POT>(seg + 1, n) - j0;
    const int last = cnt > 0 ? cnt - 1 : 0;
    const int own = lane - j0;  // this lane's atom within the segment
    const double c = -2.0 * rho;
    double k24, km48;
    hold_constants(k24, km48);
    const double4* src = lds.pos + j0;
    for (;;) {
        // every read of this part is issued before the first wait
        const int cmd_v = lds.cmd;
        const double4 pi = lds.pos[lane];
        double dx[CAP], dy[CAP], dz[CAP], f[CAP], et[CAP];
#pragma unroll
        for (int u = 0; u < CAP; ++u) {
            const double4 p = src[min(u, last)];
            dx[u] = p.x;
            dy[u] = p.y;
            dz[u] = p.z;
        }
        const int cmd = uniform(cmd_v);
        if (cmd != (IEEE ? kRelayEvalIeee : kRelayEval)) return cmd;
        const double xi = pi.x, yi = pi.y, zi = pi.z;
        MorseRange range;
        if constexpr (POT == kPairMorse) range.coefs.hold();
        // past the segment's end the last partner is taken again with a zero
        // term, which leaves every sum as it is
#pragma unroll
        for (int u = 0; u < CAP; ++u) {
            dx[u] = xi - dx[u];
            dy[u] = yi - dy[u];
            dz[u] = zi - dz[u];
            pair_term64<POT, IEEE>(dx[u], dy[u], dz[u], u == own || u >= cnt, rho, c, k24, km48,
                                   f[u], et[u], range);
            // formed here, before the turn comes (the compiler would sink it)
            asm volatile("" : "+v"(f[u]), "+v"(et[u]));
        }
        relay_wait_turn<S>(seg);
        const double2 u01 = lds.acc[0][0][lane], u23 = lds.acc[0][1][lane];
        double es = u01.x, gx = u01.y, gy = u23.x, gz = u23.y;
#pragma unroll
        for (int u = 0; u < CAP; ++u) {
            es = es + et[u];
            gx = fma(f[u], dx[u], gx);
            gy = fma(f[u], dy[u], gy);
            gz = fma(f[u], dz[u], gz);
        }
        for (int k = CAP; k < cnt; ++k) {
            const double4 p = src[k];
            const double ex = xi - p.x, ey = yi - p.y, ez = zi - p.z;
            double ff, ee;
            pair_term64<POT, IEEE>(ex, ey, ez, k == own, rho, c, k24, km48, ff, ee, range);
            es = es + ee;
            gx = fma(ff, ex, gx);
            gy = fma(ff, ey, gy);
            gz = fma(ff, ez, gz);
        }
        lds.acc[0][0][lane] = make_double2(es, gx);
        lds.acc[0][1][lane] = make_double2(gy, gz);
        if constexpr (POT == kPairMorse && !IEEE)
            relay_outside(lds.outside[seg], lane < n, range, top);
        relay_wait_rest<S>(seg);
        __syncthreads();  // the next evaluation's first barrier
    }
}

// Helper of a two-tile cluster: segment 0 (the second tile's) adds directly;
// segment 1, of up to 71 partners, holds its terms in a buffer of its own in
// LDS ([term][lane], read back by the lane that wrote it).
constexpr int kRelayTerms = 72;

template <int POT, bool IEEE>
__device__ __forceinline__ int relay_helper2(RelayLds<2>& lds, double2* __restrict__ terms, int n,
                                             int tile, int seg, int lane, double rho,
                                             uint32_t top) {
    constexpr int S = 2;  // four wavefronts, two tiles
    const int j0 = relay_cut<S, POT, 2>(seg, n), j1 = relay_cut<S, POT, 2>(seg + 1, n);
    const int own = tile * kWave + lane;
    const double c = -2.0 * rho;
    double k24, km48;
    hold_constants(k24, km48);
    for (;;) {
        const int cmd_v = lds.cmd;
        const double4 pi = lds.pos[tile * kWave + lane];
        const int cmd = uniform(cmd_v);
        if (cmd != (IEEE ? kRelayEvalIeee : kRelayEval)) return cmd;
        const double xi = pi.x, yi = pi.y, zi = pi.z;
        if (seg == 0) {
            const double x[3][1] = {{xi}, {yi}, {zi}};
            relay_first<2, POT, IEEE>(lds, j1, tile, lane, n, x, rho, top, c, k24, km48);
            relay_wait_rest<S>(0);
            __syncthreads();
            continue;
        }
        double2* t = terms + lane;
        MorseRange range;
        if constexpr (POT == kPairMorse) range.coefs.hold();
        int j = j0;
        for (; j + kGroup64 <= j1; j += kGroup64, t += kGroup64 * kWave) {
            double4 p[kGroup64];
#pragma unroll
            for (int u = 0; u < kGroup64; ++u) p[u] = lds.pos[j + u];
#pragma unroll
            for (int u = 0; u < kGroup64; ++u) {
                double ff, ee;
                pair_term64<POT, IEEE>(xi - p[u].x, yi - p[u].y, zi - p[u].z, j + u == own, rho, c,
                                       k24, km48, ff, ee, range);
                t[u * kWave] = make_double2(ff, ee);
            }
        }
        for (; j < j1; ++j, t += kWave) {
            const double4 p = lds.pos[j];
            double ff, ee;
            pair_term64<POT, IEEE>(xi - p.x, yi - p.y, zi - p.z, j == own, rho, c, k24, km48, ff,
                                   ee, range);
            *t = make_double2(ff, ee);
        }
        relay_wait_turn<S>(seg);
        const double2 u01 = lds.acc[tile][0][lane], u23 = lds.acc[tile][1][lane];
        double es = u01.x, gx = u01.y, gy = u23.x, gz = u23.y;
        auto add = [&](const double4 p, const double2 v) {
            es = es + v.y;
            gx = fma(v.x, xi - p.x, gx);
            gy = fma(v.x, yi - p.y, gy);
            gz = fma(v.x, zi - p.z, gz);
        };
        constexpr int GA = 6;
        t = terms + lane;
        j = j0;
        for (; j + GA <= j1; j += GA, t += GA * kWave) {
            double4 p[GA];
            double2 v[GA];
#pragma unroll
            for (int u = 0; u < GA; ++u) {
                p[u] = lds.pos[j + u];
                v[u] = t[u * kWave];
            }
#pragma unroll
            for (int u = 0; u < GA; ++u) add(p[u], v[u]);
        }
        for (; j < j1; ++j, t += kWave) add(lds.pos[j], *t);
        lds.acc[tile][0][lane] = make_double2(es, gx);
        lds.acc[tile][1][lane] = make_double2(gy, gz);
        if constexpr (POT == kPairMorse && !IEEE)
            relay_outside(lds.outside[2 + tile], own < n, range, top);
        relay_wait_rest<S>(seg);
        __syncthreads();
    }
}

// Every wavefront but the leader, until the leader is done.  role: tile role mod A, segment
// role / A.
template <int A, int W, int POT>
__device__ __forceinline__ void relay_helpers(RelayLds<A>& lds, double2* terms, int role, int lane,
                                              double rho, uint32_t top) {
    constexpr int S = W / A;
    const int seg = role / A;
    int n = 0;
    __syncthreads();
    int cmd = uniform(lds.cmd);
    while (cmd != kRelayExit) {
        if (cmd == kRelayNew) {
            n = uniform(lds.n);
            __syncthreads();  // read: the leader may ask for the first evaluation
            __syncthreads();
            cmd = uniform(lds.cmd);
        } else if constexpr (A == 2) {
            double2* own = terms + (role - 2) * kRelayTerms * kWave;  // segment 1: roles 2 and 3
            cmd = cmd == kRelayEval
                      ? relay_helper2<POT, false>(lds, own, n, role % A, seg, lane, rho, top)
                      : relay_helper2<POT, true>(lds, own, n, role % A, seg, lane, rho, top);
        } else if (cmd == kRelayEvalIeee) {
            cmd = relay_helper<W, POT, true, 1>(lds, n, seg, lane, rho, top);
        } else {
            // the fewest groups that hold the segment
            const int cnt = relay_cut<S, POT>(seg + 1, n) - relay_cut<S, POT>(seg, n);
            if (cnt <= 4)
                cmd = relay_helper<W, POT, false, 1>(lds, n, seg, lane, rho, top);
            else if (cnt <= 8)
                cmd = relay_helper<W, POT, false, 2>(lds, n, seg, lane, rho, top);
            else if (cnt <= 12)
                cmd = relay_helper<W, POT, false, 3>(lds, n, seg, lane, rho, top);
            else if (cnt <= 16)
                cmd = relay_helper<W, POT, false, 4>(lds, n, seg, lane, rho, top);
            else
                cmd = relay_helper<W, POT, false, 5>(lds, n, seg, lane, rho, top);
        }
    }
}

// The leader's team: one wavefront with A atoms per lane, its evaluation
// shared with the workgroup's other wavefronts.
template <int A, int W, int POT>
struct RelayTeam : Team<1, A, POT> {
    RelayLds<A>* lds;

    // Before the first evaluation of a cluster (n set).
    __device__ __forceinline__ void announce() {
        if (this->li == 0) {
            lds->cmd = kRelayNew;
            lds->n = this->n;
        }
        __syncthreads();
        __syncthreads();
    }
    __device__ __forceinline__ void finish() {
        if (this->li == 0) lds->cmd = kRelayExit;
        __syncthreads();
    }

    template <bool F32>
    __device__ __forceinline__ double eval(const double (&x)[3][A], double (&g)[3][A]) {
        static_assert(!F32, "FP64 only");
        const int lane = this->li, n = this->n;
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const int i = a * kWave + lane;
            if (i < n) lds->pos[i] = make_double4(x[0][a], x[1][a], x[2][a], 0.0);
        }
        double e[1][A], o[1];
        bool general = POT == kPairMorse && this->top == 0;
        if (!general) {
            share<false>(x, e[0], g);
            general = POT == kPairMorse && uniform(lds->outside[0] | lds->outside[1] |
                                                   lds->outside[2] | lds->outside[3]);
        }
        // as in Team::eval: repeated by the general forms
        if (POT == kPairMorse && general) share<true>(x, e[0], g);
        this->sum_energy(e, o);
        if constexpr (POT == kPairLJ) {
            // as in Team::eval: repeated with the IEEE division if not finite
            if (!isfinite(uniform(o[0]))) {
                share<true>(x, e[0], g);
                this->sum_energy(e, o);
            }
        }
        return (POT == kPairMorse ? 0.5 : 2.0) * o[0];
    }

    template <bool IEEE>
    __device__ __forceinline__ void share(const double (&x)[3][A], double (&e)[A],
                                          double (&g)[3][A]) {
        constexpr int S = W / A;
        const int lane = this->li;
        if (lane == 0) lds->cmd = IEEE ? kRelayEvalIeee : kRelayEval;
        __syncthreads();
        double k24, km48;
        hold_constants(k24, km48);
        const double x0[3][1] = {{x[0][0]}, {x[1][0]}, {x[2][0]}};
        relay_first<A, POT, IEEE>(*lds, relay_cut<S, POT, A>(1, this->n), 0, lane, this->n, x0,
                                  this->rho, this->top, -2.0 * this->rho, k24, km48);
        relay_wait_rest<S>(0);
#pragma unroll
        for (int a = 0; a < A; ++a) {
            const double2 u = lds->acc[a][0][lane], v = lds->acc[a][1][lane];
            const bool on = this->active(a);
            e[a] = on ? u.x : 0.0;
            g[0][a] = on ? u.y : 0.0;
            g[1][a] = on ? v.x : 0.0;
            g[2][a] = on ? v.y : 0.0;
        }
    }
};

// Two wavefronts per SIMD for one-tile clusters (256 registers), one for two-tile
// clusters (the leader's history alone takes 240).
template <int A, int W, int POT>
__global__ __launch_bounds__(kWave* W) __attribute__((amdgpu_waves_per_eu(A == 1 ? 2 : 1))) void
relay_kernel(MinArgs args) {
    __shared__ RelayLds<A> lds;
    __shared__ double2 terms[A == 2 ? 2 * kRelayTerms * kWave : 1];
    const int lane = threadIdx.x % kWave;
    int role = uniform((int)threadIdx.x / kWave);
    const uint32_t top =
        POT == kPairMorse ? (uint32_t)uniform((int)morse_top(args.rho)) : 0u;
    // two wavefronts: four workgroups share a CU, and in every other workgroup of
    // an XCD (consecutive workgroups go to the eight XCDs in turn) the second
    // wavefront leads, so that leaders are spread over the SIMDs (1024 x LJ38:
    // 2.88 instead of 2.95 ms)
    if (W == 2) role ^= (int)(blockIdx.x >> 3) & 1;
    if (role != 0) {
        relay_helpers<A, W, POT>(lds, terms, role, lane, args.rho, top);
        return;
    }
    RelayTeam<A, W, POT> tm;
    tm.lds = &lds;
    tm.li = lane;
    tm.bank = 0;
    tm.rho = args.rho;
    tm.top = top;
    tm.up_n = 0;
    History<1, A, true> H;
    H.init(nullptr, nullptr, args.p.m);
    const int start = args.plan.cls[args.cls];
    const int count = args.plan.cls[kNumClasses + args.cls];
    for (;;) {
        int idx = 0;
        if (lane == 0) idx = atomicAdd(&args.plan.queue[args.cls], 1);
        idx = uniform(idx);
        if (idx >= count) break;
        const int b = uniform(args.plan.list[start + idx]);
        const int o = uniform(args.offset[b]);
        tm.n = uniform(args.offset[b + 1]) - o;  // the plan guarantees 0 <= n <= 64 A
        tm.announce();
        minimize_cluster<0, A>(args, tm, H, b, o, tm.n, true);
    }
    tm.finish();
}

int relay_block(int shape) { return kWave * (shape == kRelayShape ? 4 : 2); }

const void* relay_kernel_for(int mixed, int pot, int c, int shape) {
    if (mixed || c < 0 || c > 1) return nullptr;
    if (shape == kRelayPairShape)
        return c == 0 && pot == kPairLJ ? reinterpret_cast<const void*>(&relay_kernel<1, 2, kPairLJ>)
                                        : nullptr;
#define LJ_RELAY(A)                                                                 \
    (pot == kPairMorse ? reinterpret_cast<const void*>(&relay_kernel<A, 4, kPairMorse>) \
                       : reinterpret_cast<const void*>(&relay_kernel<A, 4, kPairLJ>))
    return c == 0 ? LJ_RELAY(1) : LJ_RELAY(2);
#undef LJ_RELAY
}

}  // namespace lj
