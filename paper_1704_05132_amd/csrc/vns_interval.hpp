// Interval pricing: the exact cost of every move of a pattern from one parallel decode of the pattern itself.
//
// The forward decode needs no period-by-period walk.  Between two setups the limit, the last remanufacturing
// and the last manufacturing setup are fixed, so a setup interval with demand d remanufactures
// min(XR + d, lim) - XR units as a whole; and an interval's only effect on what follows is XR (and, until the
// next manufacturing setup, which period makes the shortfalls).  So a move at period t changes the pattern's
// cost in three places:
//   * its own one or two intervals, recomputed from the state before t;
//   * later remanufacturing intervals, while the total remanufactured differs from the unchanged pattern's by
//     d != 0: an interval that had shortage c (units of its demand not remanufactured) and headroom E (returns
//     left over), at most one of them positive, turns d into min(d + c, E), and the difference is made at its
//     own periods instead, weight w per unit.  |d| never grows and most moves are done after one or two;
//   * the shortfalls up to the next manufacturing setup M1, when the move changes which period makes them.
// One lane holds one period (two for T > 64): the pattern's own states come from five wavefront scans, and every
// move of the lane's period is then priced from registers, one 8-byte record of the next setup and of M1, and
// the remanufacturing intervals' records {c, E, w, period} in LDS.
//
// What bounds it: VALU issue.  The sweep of 1024 instances (K 100..1000, T 52 or 104) x 16 chains issues 6.9e9 VALU
// instructions in 10.7 ms, 1.05 per SIMD and four cycles (a part of them at the double rate) with 58% of their lanes
// enabled.  A full decode costs every move 14 T operations (728 at T = 52); here the scans and records are about 130
// instructions per pattern, a move takes 20 to 35, and four records of a walk 22 to 30, of which the slowest of 64 lanes
// needs 2 to 3 rounds (1.3 records on average; local optima, T = 52): 600 VALU instructions for a pattern's 156 slots in
// place of 2000.  Best move of every pattern of 256 instances (K 100..1000, T 52 or 104) x 16 chains: 15.9 -> 2.78 ms; of
// 1024 instances (K 10..200, T 12, 24 or 52) x 8: 1.18 -> 0.43 ms.  Short horizons share a wavefront (16 or 32 lanes per
// pattern), which halves the instructions per pattern at T = 24 and quarters them at T = 12.
//
// Integers: for a "compact" product (compact_product below: sums of demand and returns, weights and unit terms
// below 2^23, worst-case cost below 2^31) every product here has two signed 24-bit factors and every sum is
// taken modulo 2^32 with a result below 2^31, so 32-bit arithmetic is exact; contexts with other products and
// the disposal reading keep the period-by-period decode.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vns_device.hpp"

namespace vns {

constexpr int32_t kBad32 = INT32_MAX;   // price of an infeasible move or of a slot that is no move

namespace iv {

// Inclusive scans over groups of G lanes with identity 0 (the group's lanes are in order): row shifts, then the
// last lane of each row of 16 into the next rows.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp0(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, ROWS == 0xf);
}
template <int G, class Op>
__device__ __forceinline__ uint32_t scan(uint32_t x, Op op) {
    x = op(x, dpp0<0x111, 0xf>(x));
    x = op(x, dpp0<0x112, 0xf>(x));
    x = op(x, dpp0<0x114, 0xf>(x));
    x = op(x, dpp0<0x118, 0xf>(x));
    if constexpr (G >= 32) x = op(x, dpp0<0x142, 0xa>(x));   // lane 15 of rows 0, 2 into rows 1, 3
    if constexpr (G >= 64) x = op(x, dpp0<0x143, 0xc>(x));   // lane 31 into rows 2, 3
    return x;
}
template <int G>
__device__ __forceinline__ uint32_t scan_add(uint32_t x) {
    return scan<G>(x, [](uint32_t a, uint32_t b) { return a + b; });
}
template <int G>
__device__ __forceinline__ uint32_t scan_max(uint32_t x) {
    return scan<G>(x, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
}
// The previous lane's value (0 before the wavefront's first lane) and the next lane's (last after the last).
__device__ __forceinline__ uint32_t prev_lane(uint32_t x, uint32_t first = 0) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)x, 0x138, 0xf, 0xf, false);
}
__device__ __forceinline__ int32_t next_lane(int32_t x, int32_t last = 0) {
    return __builtin_amdgcn_update_dpp(last, x, 0x130, 0xf, 0xf, false);
}
__device__ __forceinline__ int32_t last_lane(uint32_t x) { return __builtin_amdgcn_readlane((int)x, 63); }

// a * b and acc + a * b, a and b signed 24-bit.  Written as instructions: where the compiler does not see both ranges
// in the block of the product, it takes the quarter-rate 32-bit multiply.
__device__ __forceinline__ int32_t mul24(int32_t a, int32_t b) {
    int32_t r;
    asm("v_mul_i32_i24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ int32_t mad24(int32_t a, int32_t b, int32_t acc) {
    int32_t r;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(acc));
    return r;
}

// A product's parameters in 32 bits (exact for a compact product).
struct Cost {
    int32_t kM, kR, hM, wd;   // wd = hR - hM: a remanufactured unit's weight per period of its lot
    int32_t cXR;
};
__device__ __forceinline__ Cost cost_of(const ProdParams &pp) {
    return Cost{pp.kM, pp.kR, pp.hM, pp.hR - pp.hM, (int32_t)pp.cXR};
}

// A group of G lanes prices one pattern: one period per lane for T <= G, G = 16, 32 or 64, or two periods per lane
// for T <= 128 (G = 64, NV = 2).
template <int G>
using Word = typename std::conditional<(G < 64), uint32_t, uint64_t>::type;

// Setup bits, word v: periods 64 v ...  G = 64: the same words in every lane (scalar registers); fewer: per lane.
template <int G, int NV>
struct Masks {
    Word<G> m[NV], r[NV];
};

template <int G, int NV>
__device__ __forceinline__ Masks<G, NV> masks_of(const Bits &b) {
    Masks<G, NV> k;
    if constexpr (G < 64) {
        k.m[0] = b.m[0];
        k.r[0] = b.r[0];
    } else {
        auto word = [](uint32_t lo, uint32_t hi) {
            return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)lo) |
                   (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)hi) << 32;
        };
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            k.m[v] = word(b.m[2 * v], b.m[2 * v + 1]);
            k.r[v] = word(b.r[2 * v], b.r[2 * v + 1]);
        }
    }
    return k;
}

// This lane's bit of a word.
template <int G>
__device__ __forceinline__ bool lane_bit(Word<G> w) {
    if constexpr (G < 64) return (w >> (threadIdx.x & (G - 1))) & 1u;
    else return __builtin_amdgcn_inverse_ballot_w64(w);
}
// The word of the next periods' bits: bit t = bit t + 1 of z.
template <int G, int NV>
__device__ __forceinline__ Word<G> next_bits(const Word<G> (&z)[NV], int v) {
    if constexpr (NV == 1) return z[0] >> 1;
    else return v == 0 ? (z[0] >> 1) | (z[1] << 63) : z[1] >> 1;
}
// Periods t with t + 1 < T whose bits t and t + 1 of z differ: the swaps that are moves.
template <int G, int NV>
__device__ __forceinline__ Word<G> swap_bits(const Word<G> (&z)[NV], int v, int T) {
    const int lim = T - 1 - 64 * v;   // periods of this word
    const Word<G> all = (Word<G>)~(Word<G>)0;
    const Word<G> keep = lim <= 0 ? (Word<G>)0 : lim >= 8 * (int)sizeof(Word<G>) ? all : (Word<G>)~(all << lim);
    return (z[v] ^ next_bits<G, NV>(z, v)) & keep;
}

// The n lowest bits (n <= 64, none below 1).
__device__ __forceinline__ uint64_t first_bits(int n) { return n <= 0 ? 0ull : n >= 64 ? ~0ull : ~(~0ull << n); }

// LDS of one wavefront: per group, pos[k] = (XR, H) before period k, H the units manufactured (the demand before k
// less XR), and the remanufacturing setups' records with kWalk that end every walk.
constexpr int kWalk = 4;   // records a walk takes per round: their reads are in flight together
template <int G, int NV>
struct Lds {
    static constexpr int kPos = G * NV + 1;
    static constexpr int kRec = G * NV + kWalk;
    int4 rec[(64 / G) * kRec];
    int2 pos[(64 / G) * kPos];
};

// One period of the unchanged pattern.
struct Period {
    int32_t t, D, PR;
    int32_t xb, xa, Hb;           // XR before and after t, H before t
    int32_t lmz, lsz, cap0;       // last M and R setup before t (0 if none), returns at the latter
    int32_t lm;                   // last M setup up to t
    int32_t ls;                   // last R setup up to t
    int32_t XRn, Hn, Hm;          // XR and H before the next setup after t, H before the next M setup after t
    int32_t M1;                   // the latter's period, or T
    int32_t j;                    // R setups up to t: the ordinal of the first one after t
    int32_t w;                    // cost of a unit remanufactured for a period of t's interval
    bool m, r;
    bool reg0, hm0, hm;           // remanufacturing open before t; an M setup before t, up to t
    bool blk0;                    // strict reading: no manufacturing allowed before t
};

__device__ __forceinline__ void lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A row past the horizon: no demand, and returns that never bind.
__device__ __forceinline__ int2 no_row() { return make_int2(0, 1 << 23); }

// A pattern's periods in this lane, and the cost change of its moves.
template <int G, int NV, bool STRICT>
struct Pattern {
    Period p[NV];
    const int4 *rec;   // this group's records

    // row: this lane's periods' rows (no_row() past T).
    __device__ __forceinline__ void build(const Masks<G, NV> &k, const int2 (&row)[NV], int T, const Cost &c,
                                          Lds<G, NV> &sh) {
        const int lane = threadIdx.x & 63, t0 = lane & (G - 1), grp = lane / G;
        int4 *grec = sh.rec + grp * Lds<G, NV>::kRec;
        int2 *pos = sh.pos + grp * Lds<G, NV>::kPos;
        rec = grec;
        uint32_t lm1[NV], key[NV], pda[NV];   // last setups as period + 1; key = returns at the last R setup << 8 | it
        // 1. last setups, open capacity, demand and remanufactured units up to each period
        int32_t cm = 0, ckey = 0, cpd = 0, cA = 0, cS = 0;   // carries into the second word
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            Period &q = p[v];
            q.t = t0 + 64 * v;
            q.D = row[v].x;
            q.PR = row[v].y;
            q.m = lane_bit<G>(k.m[v]);
            q.r = lane_bit<G>(k.r[v]);
            lm1[v] = scan_max<G>(q.m ? (uint32_t)(q.t + 1) : 0u);
            key[v] = scan_max<G>(q.r ? ((uint32_t)q.PR << 8) + (uint32_t)(q.t + 1) : 0u);   // returns never drop
            pda[v] = scan_add<G>((uint32_t)q.D);
            if (v > 0) {
                lm1[v] = max(lm1[v], (uint32_t)cm);
                key[v] = max(key[v], (uint32_t)ckey);
                pda[v] += (uint32_t)cpd;
            }
            const uint32_t ls1 = key[v] & 255u;
            const bool open = ls1 >= max(lm1[v], 1u);
            // while open, XR follows the demand A of the open periods and lags by the largest excess of A over the
            // open capacity so far (XR <- min(XR + d, cap) composed over the periods)
            const uint32_t A = scan_add<G>(open ? (uint32_t)q.D : 0u) + (v > 0 ? (uint32_t)cA : 0u);
            uint32_t S = scan_max<G>((uint32_t)(open ? max((int32_t)A - (int32_t)(key[v] >> 8), 0) : 0));
            if (v > 0) S = max(S, (uint32_t)cS);
            q.xa = (int32_t)(A - S);
            pos[q.t + 1] = make_int2(q.xa, (int)pda[v] - q.xa);
            if (NV > 1 && v == 0) {
                cm = last_lane(lm1[0]);
                ckey = last_lane(key[0]);
                cpd = last_lane(pda[0]);
                cA = last_lane(A);
                cS = last_lane(S);
            }
        }
        lds_fence();
        // 2. the state before each period, the next setup and the next M setup
        int nR = 0;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            Period &q = p[v];
            uint32_t l0, k0, x0;
            if (v > 0) {
                l0 = prev_lane(lm1[v], last_lane(lm1[v - 1]));
                k0 = prev_lane(key[v], last_lane(key[v - 1]));
                x0 = prev_lane((uint32_t)q.xa, last_lane((uint32_t)p[v - 1].xa));
            } else {
                l0 = prev_lane(lm1[v]);
                k0 = prev_lane(key[v]);
                x0 = prev_lane((uint32_t)q.xa);
                if (G < 64 && t0 == 0) l0 = k0 = x0 = 0u;
            }
            const uint32_t s0 = k0 & 255u, s1 = key[v] & 255u;
            q.xb = (int32_t)x0;
            q.Hb = (int32_t)pda[v] - q.D - q.xb;
            q.hm0 = l0 != 0u;
            q.hm = lm1[v] != 0u;
            q.lmz = (int32_t)max(l0, 1u) - 1;
            q.lm = (int32_t)max(lm1[v], 1u) - 1;
            q.lsz = (int32_t)max(s0, 1u) - 1;
            q.ls = (int32_t)max(s1, 1u) - 1;
            q.cap0 = (int32_t)(k0 >> 8);
            q.reg0 = s0 >= max(l0, 1u);
            q.blk0 = s0 > l0 || l0 == 0u;
            const int n = next_setup(k.m, k.r, v, t0, T);
            q.M1 = next_setup(k.m, k.m, v, t0, T);
            if constexpr (G < 64) {
                q.j = __popc(k.r[0] & ~(~0u << 1 << t0));
                nR = __popc(k.r[0]);
            } else {
                q.j = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(k.r[v] >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)k.r[v], (uint32_t)nR)) +
                      (q.r ? 1 : 0);
                nR += __popcll(k.r[v]);
            }
            const int2 an = pos[n];
            q.XRn = an.x;
            q.Hn = an.y;
            q.Hm = pos[q.M1].y;
            q.w = mad24(c.hM, q.lm, mul24(c.wd, q.ls));
            // 3. the record of a remanufacturing setup (its ls is t itself)
            if (q.r) grec[q.j - 1] = make_int4(q.Hn - q.Hb, q.PR - q.XRn, q.w, STRICT && !q.m ? q.t + 256 : q.t);
        }
        // the horizon's end takes every difference: its units are worth -cXR each
        if (t0 < kWalk) grec[nR + t0] = t0 == 0 ? make_int4(1 << 28, 0, -c.cXR, 255) : make_int4(0, 0, 0, 255);
        lds_fence();
    }

    // The first setup after period t0 + 64 v of the words a | b (lane-varying), or T; T in the lanes past the horizon.
    static __device__ __forceinline__ int next_setup(const Word<G> (&a)[NV], const Word<G> (&b)[NV], int v, int t0, int T) {
        if constexpr (G < 64) {
            return min(__builtin_ctzg((a[0] | b[0]) & (~0u << 1 << t0), 32), T);
        } else if constexpr (NV == 1) {
            return min(__builtin_ctzg((a[0] | b[0]) & (~0ull << 1 << t0), 64), T);
        } else {
            const uint64_t hi = a[1] | b[1], x = (v ? hi : a[0] | b[0]) & (~0ull << 1 << t0);
            const int past = v == 0 && hi ? 64 + __builtin_ctzll(hi) : T;
            return x ? 64 * v + __builtin_ctzll(x) : past;
        }
    }

    // The pattern's own cost without the setups' and the constant: sum of u w - hM D lm over the periods, plus cXR XR
    // (modulo 2^32), in every lane of a wavefront (G = 64).
    __device__ __forceinline__ int32_t own_cost(const Cost &c) const {
        static_assert(G == 64, "one pattern per wavefront");
        uint32_t s = 0;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const Period &q = p[v];
            s += (uint32_t)(mul24(q.xa - q.xb, q.w) - mul24(q.D, mul24(c.hM, q.lm)));
        }
        s = scan_add<64>(s);
        const int32_t xr = last_lane((uint32_t)p[NV - 1].xa);
        return last_lane(s) + mul24(c.cXR, xr);
    }

    // The difference d of the remanufactured units passed on to R setup j and those after it; returns its cost.
    // dM: what is left of it at M1.  kWalk records per round: those after the horizon's change nothing.
    template <bool TRACK>
    __device__ __forceinline__ int32_t walk(int j, int32_t d, int32_t M1, int32_t &dM, bool &bad, int &steps) const {
        int32_t acc = 0;
        const int4 *at = rec + j;
        dM = d;
        while (d != 0) {
            int4 r[kWalk];
#pragma unroll
            for (int h = 0; h < kWalk; ++h) r[h] = at[h];
#pragma unroll
            for (int h = 0; h < kWalk; ++h) {
                const int4 q = r[h];
                const int32_t dn = min(d + q.x, q.y), du = dn - d;
                acc = mad24(du, q.z, acc);
                if constexpr (TRACK) dM = (STRICT ? q.w & 255 : q.w) < M1 ? dn : dM;
                if constexpr (STRICT) bad |= q.w > 255 && du < 0;   // a remanufacture-only interval runs short
                d = dn;
            }
            at += kWalk;
            steps += kWalk;
        }
        return acc;
    }

    // Cost change of flipping zM(t).  The interval of t: nothing changes if t remanufactures; else a new M setup closes
    // what was open before t (v0 units), and a removed one leaves it open.
    __device__ __forceinline__ int32_t flip_m(const Period &q, const Cost &c, int &steps) const {
        const int32_t dseg = (q.XRn + q.Hn) - (q.xb + q.Hb);
        const int32_t v0 = q.reg0 ? min(dseg, q.cap0 - q.xb) : 0;
        const int32_t d = q.r ? 0 : q.m ? v0 : -v0;
        const int32_t wL = mad24(c.hM, q.lm, mul24(c.wd, q.lsz));
        bool bad = false;
        int32_t dM;
        const int32_t x = mad24(d, wL, walk<true>(q.j, d, q.M1, dM, bad, steps));
        const int32_t S = q.Hm - q.Hb - dM;   // shortfalls up to M1, made at t or at the M setup before it
        const int32_t y = c.kM - mul24(mul24(c.hM, q.t - q.lmz), S);
        bad |= q.m && !q.hm0 && S > 0;
        if constexpr (STRICT) bad |= q.m && (q.r || q.blk0) && dseg - (q.XRn - q.xb + d) > 0;
        return bad ? kBad32 : x + (q.m ? -y : y);
    }

    // Cost change of flipping zR(t): the interval remanufactures a units with it, b without.
    __device__ __forceinline__ int32_t flip_r(const Period &q, const Cost &c, int &steps) const {
        const int32_t dseg = (q.XRn + q.Hn) - (q.xb + q.Hb), hl = mul24(c.hM, q.lm);
        const int32_t a = min(dseg, q.PR - q.xb), b = q.reg0 && !q.m ? min(dseg, q.cap0 - q.xb) : 0;
        const int32_t y = mul24(a, mad24(c.wd, q.t, hl)) - mul24(b, mad24(c.wd, q.lsz, hl)) + c.kR;
        const int32_t d = q.r ? b - a : a - b;
        bool bad = false;
        int32_t dM, x;
        if (__any(!q.hm)) {   // before the first M setup a shortfall cannot be made
            x = walk<true>(q.j, d, q.M1, dM, bad, steps);
            bad |= !q.hm && q.Hm - q.Hb - dM > 0;
        } else {
            x = walk<false>(q.j, d, q.M1, dM, bad, steps);
        }
        if constexpr (STRICT) bad |= !q.m && dseg - (q.r ? b : a) > 0 && (!q.r || q.blk0);
        return bad ? kBad32 : x + (q.r ? -y : y);
    }

    // What a swap of periods t, t + 1 needs of period t + 1.
    struct Next {
        int32_t PR, M1, XRn, Hn, Hm, j, w;
        bool m, r;
    };
    __device__ __forceinline__ Next next_of(const Masks<G, NV> &k, int v) const {
        const Period &q = p[v], &o = p[NV - 1];   // the second word's lane 0 follows lane 63
        auto nx = [&](int32_t a, int32_t b) {
            return next_lane(a, NV > 1 && v == 0 ? __builtin_amdgcn_readlane(b, 0) : 0);
        };
        Next x;
        x.PR = nx(q.PR, o.PR);
        x.M1 = nx(q.M1, o.M1);
        x.XRn = nx(q.XRn, o.XRn);
        x.Hn = nx(q.Hn, o.Hn);
        x.Hm = nx(q.Hm, o.Hm);
        x.w = nx(q.w, o.w);
        x.m = lane_bit<G>(next_bits<G, NV>(k.m, v));
        x.r = lane_bit<G>(next_bits<G, NV>(k.r, v));
        x.j = q.j + (x.r ? 1 : 0);
        return x;
    }

    // Cost change of swapping zM(t), zM(t + 1), which differ.  e0, e1: more units remanufactured for period t and for
    // t + 1 up to the next setup; their lots are the pattern's own.  What is manufactured for t and, up to the next
    // M setup, after it moves by one period or back to the M setup before t.
    __device__ __forceinline__ int32_t swap_m(const Period &q, const Next &x, const Cost &c, bool valid, int &steps) const {
        const int32_t Ha = q.Hb + q.D - (q.xa - q.xb), d1 = (x.XRn + x.Hn) - (q.xa + Ha);
        const int32_t c0 = q.reg0 ? min(q.D, q.cap0 - q.xb) : 0;
        const int32_t e0 = q.r ? 0 : q.m ? c0 : -c0;
        const int32_t x1 = q.xa + e0;
        const int32_t u1 = x.r ? min(d1, x.PR - x1) : q.r && !q.m ? min(d1, q.PR - q.xa) : 0;
        const int32_t e1 = u1 - (x.XRn - q.xa);
        const int32_t d = valid ? e0 + e1 : 0;
        bool bad = false;
        int32_t dM;
        const int32_t y = mad24(e1, x.w, mad24(e0, q.w, walk<true>(x.j, d, x.M1, dM, bad, steps)));
        const int32_t S = x.Hm - dM - (Ha - e0), made0 = q.D - (x1 - q.xb);
        const int32_t z = mul24(c.hM, S) - mul24(mul24(c.hM, q.t - q.lmz), made0);
        bad |= q.m && !q.hm0 && made0 > 0;
        if constexpr (STRICT) {
            const bool blk = q.m && (q.r || q.blk0);   // m: the M setup leaves t
            bad |= blk && made0 > 0;
            bad |= !q.m && x.r && d1 - u1 > 0;         // !m: it leaves t + 1
        }
        return bad ? kBad32 : y + (q.m ? -z : z);
    }

    // Cost change of swapping zR(t), zR(t + 1), which differ.
    __device__ __forceinline__ int32_t swap_r(const Period &q, const Next &x, const Cost &c, bool valid, int &steps) const {
        const int32_t hl = mul24(c.hM, q.lm), Ha = q.Hb + q.D - (q.xa - q.xb), d1 = (x.XRn + x.Hn) - (q.xa + Ha);
        const int32_t a0 = min(q.D, q.PR - q.xb), b0 = q.reg0 && !q.m ? min(q.D, q.cap0 - q.xb) : 0;
        const int32_t y0 = mul24(a0, mad24(c.wd, q.t, hl)) - mul24(b0, mad24(c.wd, q.lsz, hl));
        const int32_t u0 = q.r ? b0 : a0, x1 = q.xb + u0;
        const int32_t u1 = q.r ? min(d1, x.PR - x1) : x.m ? 0 : min(d1, q.PR - x1);
        const int32_t w1 = mad24(c.wd, q.t + (q.r ? 1 : 0), x.m ? mul24(c.hM, q.t + 1) : hl);
        const int32_t d = valid ? x1 + u1 - x.XRn : 0;
        int32_t y = mad24(u1, w1, q.r ? -y0 : y0) - mul24(x.XRn - q.xa, x.w);
        bool bad = false;
        int32_t dM;
        if (__any(valid && !q.hm)) {
            y += walk<true>(x.j, d, x.M1, dM, bad, steps);
            bad |= !q.hm && q.D - u0 > 0;
            bad |= !(q.hm || x.m) && x.Hm - dM - (q.Hb + q.D - u0) > 0;
        } else {
            y += walk<false>(x.j, d, x.M1, dM, bad, steps);
        }
        if constexpr (STRICT) {
            const bool blk = !q.m && (!q.r || q.blk0);   // after t: an R-only setup came to it, or it lost one
            bad |= blk && q.D - u0 > 0;
            bad |= !x.m && (q.r || blk) && d1 - u1 > 0;
        }
        return bad ? kBad32 : y;
    }
};

// The VND (Algorithm 1) of one product by one wavefront.  A neighbourhood is priced once per pattern: the pattern's
// decode is built when a move has been applied, and a neighbourhood met again on the same pattern finds nothing again
// (it still counts its evaluations, as Algorithm 1 prices it in every pass).  now() is read before a pricing and
// compared with `round` after it: false means the caller's round moved on and the product was given up.
// ident: the pattern's own cost is not known yet; the local optimum's is computed instead (x's is known) and the
// pattern's follows from the moves applied.  x, x_cost: with has_x, a pattern of the product known to be a local optimum
// of this list, and its cost: most shaken products return to it (86 to 91% of single flips at T = 12..104), and no
// neighbourhood of it improves.
// Choose: NoChoice takes a neighbourhood's best move; the learned VND's choice (kRanks) gives the moves' scores, and takes
// the best of the best-ranked if it improves and the best of all otherwise.
struct NoChoice {
    static constexpr bool kRanks = false;
    __device__ __forceinline__ int count(int) const { return 0; }   // moves ranked of a neighbourhood's
};
struct Vnd {
    int64_t cost;    // in: the pattern's cost (without ident); out: the local optimum's
    int64_t start;   // out: the pattern's own cost
    int64_t evals;   // move-evaluations, added to
    int32_t err;     // out: 1 if the pass guard was hit
    int64_t ranked = 0, fallbacks = 0;   // learned: neighbourhood evaluations, and those priced whole
};

template <int NV, bool STRICT, class Row, class Choose, class Now>
__device__ __forceinline__ bool vnd(Bits &b, Vnd &s, bool ident, Row row_at, int T, const ProdParams &pp,
                                    bool has_x, const Bits &x, int64_t x_cost, uint32_t nb_list, int n_nb, bool memo,
                                    Lds<64, NV> &sh, Choose &choose, int32_t round, Now now) {
    const int lane = threadIdx.x & 63;
    const Cost c = cost_of(pp);
    int2 row[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        row[v] = no_row();
        if (lane + 64 * v < T) row[v] = row_at(lane + 64 * v);
    }
    Masks<64, NV> k = masks_of<64, NV>(b);
    const Masks<64, NV> kx = masks_of<64, NV>(x);
    auto at_x = [&]() {
        bool same = has_x;
#pragma unroll
        for (int v = 0; v < NV; ++v) same = same && k.m[v] == kx.m[v] && k.r[v] == kx.r[v];
        return same;
    };
    auto pack = [](const Masks<64, NV> &z) {
        Bits o;
#pragma unroll
        for (int v = 0; v < kWords / 2; ++v) {
            const uint64_t m = v < NV ? z.m[v] : 0, r = v < NV ? z.r[v] : 0;
            o.m[2 * v] = (uint32_t)m;
            o.m[2 * v + 1] = (uint32_t)(m >> 32);
            o.r[2 * v] = (uint32_t)r;
            o.r[2 * v + 1] = (uint32_t)(r >> 32);
        }
        return o;
    };
    auto shifts = [&]() {
        int n = 0;
#pragma unroll
        for (int v = 0; v < NV; ++v) n += __popcll(swap_bits<64, NV>(k.m, v, T)) + __popcll(swap_bits<64, NV>(k.r, v, T));
        return n;
    };
    // counts the neighbourhoods in `list` (one id per nibble: 1, 2 or 4) as priced without an improving move
    auto count = [&](uint32_t list, int n_shift) {
        const int flips = __popc(list & 0x3333u), shift = __popc(list & 0x4444u);
        s.evals += flips * (T + choose.count(T)) + shift * (n_shift + choose.count(n_shift));
        if constexpr (Choose::kRanks) {
            s.ranked += flips + shift;
            s.fallbacks += flips + (n_shift > 0 ? shift : 0);
        }
    };
    s.err = 0;
    s.start = s.cost;
    if (at_x()) {   // the shake undid itself: one pass finds nothing
        count(nb_list, shifts());
        s.start = s.cost = x_cost;
        return true;
    }
    Pattern<64, NV, STRICT> pat;
    int32_t gain = 0;                  // cost change of the moves applied
    int q = 0, passes = 1;             // place in the list, pass
    bool improved = false, alive = true, back = false;
    for (;;) {   // one pattern
        pat.build(k, row, T, c, sh);
        uint32_t priced = 0, clean = 0;   // ids priced on this pattern, and list places passed on it, without improving
        int n_shift = 0;                  // the pattern's shifts, once priced
        int32_t best = 0;
        uint32_t nb = 0;
        int32_t dx[2][NV];   // changes of the flips or zM swaps, and of the zR swaps
        // the lowest slot whose change in x is x0: zR swap, period
        auto place = [&](const int32_t (&x)[2][NV], int32_t x0, int &z, int &t) {
            z = 0;
            t = -1;
#pragma unroll
            for (int v = NV - 1; v >= 0; --v) {
                const uint64_t w = __ballot(x[0][v] == x0);
                t = w ? 64 * v + (int)__builtin_ctzll(w) : t;
            }
            if (nb == 4u && t < 0) {
                z = 1;
#pragma unroll
                for (int v = NV - 1; v >= 0; --v) {
                    const uint64_t w = __ballot(x[1][v] == x0);
                    t = w ? 64 * v + (int)__builtin_ctzll(w) : t;
                }
            }
        };
        for (;;) {
            if (q == n_nb) {   // the pass is over
                if (!improved) break;
                if (++passes > kMaxPasses) {
                    s.err = 1;
                    break;
                }
                improved = false;
                q = 0;
            }
            if (memo && ((clean >> q) & 1u)) {   // same pattern: nothing to find
                ++q;
                continue;
            }
            nb = (nb_list >> (4 * q)) & 0xFu;
            if (priced & nb) {
                count(nb, n_shift);
                clean |= 1u << q++;
                continue;
            }
            const int32_t seen = now();
            int steps = 0, n = T;
            if (nb == 1u) {
#pragma unroll
                for (int v = 0; v < NV; ++v) dx[0][v] = lane + 64 * v < T ? pat.flip_m(pat.p[v], c, steps) : kBad32;
            } else if (nb == 2u) {
#pragma unroll
                for (int v = 0; v < NV; ++v) dx[0][v] = lane + 64 * v < T ? pat.flip_r(pat.p[v], c, steps) : kBad32;
            } else {
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const typename Pattern<64, NV, STRICT>::Next nx = pat.next_of(k, v);
                    const bool sm = lane_bit<64>(swap_bits<64, NV>(k.m, v, T)), sr = lane_bit<64>(swap_bits<64, NV>(k.r, v, T));
                    const int32_t y = pat.swap_m(pat.p[v], nx, c, sm, steps);
                    const int32_t z = pat.swap_r(pat.p[v], nx, c, sr, steps);
                    dx[0][v] = sm ? y : kBad32;
                    dx[1][v] = sr ? z : kBad32;
                }
                n = n_shift = shifts();
            }
            if (__builtin_amdgcn_readfirstlane(seen) != round) {
                alive = false;
                break;
            }
            // the lowest change, as the sweep finds it
            auto lowest = [&](const int32_t (&x)[2][NV]) {
                uint32_t low = 0;
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    low = max(low, ~((uint32_t)x[0][v] ^ 0x80000000u));
                    if (nb == 4u) low = max(low, ~((uint32_t)x[1][v] ^ 0x80000000u));
                }
                return (int32_t)(~(uint32_t)last_lane(scan_max<64>(low)) ^ 0x80000000u);
            };
            best = lowest(dx);
            if constexpr (Choose::kRanks) {
                const int n_sel = choose.count(n);
                ++s.ranked;
                bool whole = n > 0;   // the neighbourhood was priced whole
                if (best < 0) {
                    // The choice is the best improving move among the n_sel best-ranked, or the best of all if none of them
                    // improves.  So scores are needed only when a move improves, and then the improving moves are tried
                    // in the order of their prices: the first with fewer than n_sel moves ranked before it is the choice.
                    uint32_t sc[2][NV];
                    uint64_t is[2][NV];   // the moves by period: flips or zM swaps, and zR swaps
                    int32_t left[2][NV];  // the changes of those not tried yet
                    const Bits pb = pack(k);
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        is[0][v] = nb == 4u ? swap_bits<64, NV>(k.m, v, T) : first_bits(T - 64 * v);
                        is[1][v] = nb == 4u ? swap_bits<64, NV>(k.r, v, T) : 0ull;
                        sc[0][v] = choose.score(pb, nb == 4u ? 2 : nb == 2u ? 1 : 0, lane + 64 * v, lane_bit<64>(is[0][v]));
                        sc[1][v] = nb == 4u ? choose.score(pb, 3, lane + 64 * v, lane_bit<64>(is[1][v])) : 0u;
                        left[0][v] = dx[0][v];
                        left[1][v] = nb == 4u ? dx[1][v] : kBad32;
                    }
                    for (int32_t x0 = best; x0 < 0; x0 = lowest(left)) {
                        int z, t;
                        place(left, x0, z, t);
                        uint32_t mine = 0;   // its score
#pragma unroll
                        for (int v = 0; v < NV; ++v)
                            if (t >> 6 == v) mine = (uint32_t)__builtin_amdgcn_readlane((int)(z ? sc[1][v] : sc[0][v]), t & 63);
                        int before = 0;
#pragma unroll
                        for (int v = 0; v < NV; ++v)
#pragma unroll
                            for (int y = 0; y < 2; ++y) {
                                // of equal scores the lower slots
                                const uint64_t lower = y < z || (y == z && v < t >> 6) ? ~0ull : y == z && v == t >> 6 ? (1ull << (t & 63)) - 1 : 0ull;
                                before += __popcll((__ballot(sc[y][v] < mine) | (__ballot(sc[y][v] == mine) & lower)) & is[y][v]);
                            }
                        if (before < n_sel) {
                            // the choice: what improves more was not among the best-ranked
                            best = x0;
#pragma unroll
                            for (int v = 0; v < NV; ++v) {
                                dx[0][v] = left[0][v];
                                dx[1][v] = left[1][v];
                            }
                            whole = false;
                            break;
                        }
#pragma unroll
                        for (int v = 0; v < NV; ++v) {
                            const bool here = lane + 64 * v == t;
                            left[0][v] = here && !z ? kBad32 : left[0][v];
                            left[1][v] = here && z ? kBad32 : left[1][v];
                        }
                    }
                }
                s.fallbacks += whole ? 1 : 0;
                n = n_sel + (whole ? n : 0);
            }
            s.evals += n;
            if (best < 0) break;
            priced |= nb;
            clean |= 1u << q++;
        }
        if (best >= 0 || !alive) break;   // a local optimum (or given up)
        int at_z, t;
        place(dx, best, at_z, t);
        const bool on_r = nb == 2u || at_z;
        const uint64_t w = nb == 4u ? 3ull : 1ull;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const uint64_t y = t >> 6 == v ? w << (t & 63) : v == 1 && t == 63 ? w >> 1 : 0ull;   // 63 reaches the next word
            k.m[v] ^= on_r ? 0ull : y;
            k.r[v] ^= on_r ? y : 0ull;
        }
        gain += best;
        improved = true;
        ++q;
        if (at_x()) {
            // nothing improves on x: the rest of this pass, and the pass that finds nothing (with the memo, which skips what
            // this pass has passed on x, only its places up to the move's)
            const int m = shifts();
            count(nb_list, m);
            if (!memo && q < n_nb) count(nb_list >> (4 * q), m);
            back = true;
            break;
        }
    }
    if (back) {
        s.cost = x_cost;
    } else if (ident) {
        int nM = 0, nR = 0;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            nM += __popcll(k.m[v]);
            nR += __popcll(k.r[v]);
        }
        s.cost = (int32_t)((uint32_t)pp.C + (uint32_t)pat.own_cost(c) + (uint32_t)c.kM * (uint32_t)nM + (uint32_t)c.kR * (uint32_t)nR);
    } else {
        s.cost += gain;
    }
    if (ident) s.start = s.cost - gain;
    b = pack(k);
    return alive;
}

}  // namespace iv
}  // namespace vns
