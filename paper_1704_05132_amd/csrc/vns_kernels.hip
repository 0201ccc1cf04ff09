// Kernels of the lot-sizing VNS for gfx950.
//
//   k_init_costs    exact cost of every (chain, product) of the current solutions; F per chain
//   k_eval          one workgroup per (product, group of chains of its instance): exact price of every move
//                   of the selected neighbourhoods, one lane per move (Section 3: the new objective value of
//                   each product is computed independently of the others).  Moves are compacted (pads and
//                   swaps of equal bits never take a lane) and the chains of the group share one LDS copy of
//                   the product's row, so a wavefront is full whatever T is
//   k_eval_iv       the same prices from one parallel decode of each pattern (vns_interval.hpp), where every product is
//                   compact and the reading has no disposal
//   k_chain_best    per chain: lexicographic (price, slot) minimum over its products
//   k_run           one workgroup per chain running whole GVNS iterations (Algorithm 2): Philox shake,
//                   VND (Algorithm 1) with one wavefront per product that needs it, acceptance
//   k_run_spec      the same with the neighbourhoods of a product's VND priced side by side
//   k_run_learned   the same with the learned scorer choosing which moves are priced exactly
//   k_run_iv, k_run_coop_iv, k_run_learned_iv   these searches with the VND by interval pricing; the forms above are
//                   left for the disposal reading, products past the compact bounds and runs that keep a move log
#include <hip/hip_runtime.h>

#include <algorithm>

#include "vns_device.hpp"
#include "vns_interval.hpp"
#include "vns_launch.hpp"
#include "vns_search.hpp"

namespace vns {


// ---------------------------------------------------------------------------------------------------
// k_init_costs: one workgroup per chain.  Costs of the current solution, copy to the working solution,
// F, best, shake size 1.
// ---------------------------------------------------------------------------------------------------
template <int MODEL>
__global__ __launch_bounds__(256) void k_init_costs(InitArgs a) {
    const int g = a.chain0 + blockIdx.x;
    const ChainInfo ci = a.chains[g];
    int64_t sum = 0;
    int inf = 0;
    for (int p = threadIdx.x; p < ci.K; p += blockDim.x) {
        const ProdParams pp = a.prod[ci.prod0 + p];
        const int64_t cp = ci.cp0 + p;
        const Bits b = a.cur[cp];
        const int64_t c = decode_cost<kWords, MODEL>(b, a.rows + pp.row, ci.T, pp);
        a.cur_cost[cp] = c;
        a.work[cp] = b;
        a.work_cost[cp] = c;
        a.best[cp] = b;
        if (c == kInf) inf = 1; else sum += c;
    }
    __shared__ int64_t s_sum[4];
    __shared__ int s_inf[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    sum = wave_sum_i64(sum);
    const int any_inf = __any(inf);
    if (lane == 0) { s_sum[wave] = sum; s_inf[wave] = any_inf; }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t F = 0;
        int bad = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) { F += s_sum[w]; bad |= s_inf[w]; }
        ChainState cs;
        cs.F = bad ? kInf : F;
        cs.F_best = cs.F;
        cs.evals = 0;
        cs.k = 1;
        cs.lopt = 0;
        cs.err = 0;
        cs.bsync = 1;
        cs.nb_evals = 0;
        cs.fallbacks = 0;
        cs.discarded = 0;
        a.cstate[g] = cs;
    }
}

// ---------------------------------------------------------------------------------------------------
// k_eval
// ---------------------------------------------------------------------------------------------------
namespace {

struct EvalShared {
    int2 row[kTMax];              // the rows of the workgroup's products, one after the other (np T <= kTMax)
    ProdParams pp[kEvalProds];    // their parameters (more than one product)
    Bits bits[kEvalPairs];        // per (chain, product) pair j = product index * chains + chain index
    unsigned long long key[kEvalPairs];
    int64_t F[kEvalPairs];
    int64_t cost[kEvalPairs];
    int64_t out_off[kEvalPairs];
    int32_t off[kEvalPairs + 1];
    uint8_t pidx[kEvalPairs];     // product index of each pair within the workgroup's products
    // the workgroup's moves, pair by pair (flips, then zM swaps, then zR swaps): pair << 9 | block << 7 | t
    uint16_t item[kEvalItems];
    int32_t tcount[kTMax];        // incremental pricing: moves per period, then their offsets
    int32_t decoded;              //   and the period-steps its batches ran, per lane
};
static_assert(kEvalPairs <= 128 && kTMax <= 128, "item packing");
static_assert(kEvalPairs <= 64, "one wavefront scans the pairs' move counts");
static_assert(kEvalGroup * 4 * kTMax <= kEvalItems, "one product of a full group of chains fits the item table");

__device__ __forceinline__ uint16_t pack_item(int j, int blk, int t) { return (uint16_t)((j << 9) | (blk << 7) | t); }

// One lane per item: apply the move to the pair's pattern, decode, fold (cost, slot) into the pair's key.
// One product (np = 1): its row and parameters are the same for every lane; several (short horizons): each
// lane reads those of its pair's product.
template <int NW, int MODEL>
__device__ __forceinline__ void eval_items(const EvalArgs &a, EvalShared &sh, int N, int T, const ProdParams &pp,
                                           int np) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int basei = wave * 64; basei < N; basei += blockDim.x) {
        const int idx = basei + lane;
        const bool in = idx < N;
        const int e = sh.item[in ? idx : basei];
        const int j = e >> 9, blk = (e >> 7) & 3, t = e & 127;
        const int slot = blk * T + t;
        Bits mb = sh.bits[j];
        xor_move<NW>(mb, blk, t);
        int64_t c;
        if (np == 1) {
            c = decode_cost<NW, MODEL>(mb, sh.row, T, pp);
        } else {
            const int pi = sh.pidx[j];
            c = decode_cost<NW, MODEL>(mb, sh.row + pi * T, T, sh.pp[pi]);
        }
        if (in) {
            if (c != kInf) atomicMin(&sh.key[j], ((unsigned long long)c << kSlotBits) | (unsigned long long)slot);
            if (a.slot_price) a.slot_price[sh.out_off[j] + slot] = c == kInf ? kInf : sh.F[j] - sh.cost[j] + c;
        }
    }
}

// Incremental exact pricing.  A move changes the pattern only from its first changed period t on, so its
// decode starts from the base pattern's state before t (snapshot, per chain and period: A = (lim, XR, lsR,
// last manufacturing setup or -1 before the first one), B = (A1, A2)).  Once every changed period is
// decoded and the moved pattern's state A equals the base's before some period, every later step adds the
// same amounts to both, so the cost is the base cost plus the setup-count change, -hM (dA1 + dA2) and hR dA1
// (the forward decode's cost is linear in A1, A2 and the final XR).  A decode that turns infeasible stops
// there (kInf).
__device__ __forceinline__ int32_t enc_last(const DecodeState &s) { return s.nolast ? -1 : s.lastM; }

// The base pattern b of one chain, decoded by one lane: its state before every period 0..T.
template <int NW>
__device__ __forceinline__ void base_snapshot(const Bits &b, const int2 *row, int T, int4 *sa, int2 *sb) {
    DecodeState s;
    for (int tau = 0; tau < T; ++tau) {
        sa[tau] = make_int4(s.lim, s.XR, s.lsR, enc_last(s));
        sb[tau] = make_int2(s.A1, s.A2);
        const int w = tau >> 5;
        uint32_t m = b.m[0], r = b.r[0];
#pragma unroll
        for (int q = 1; q < NW; ++q) {
            m = w == q ? b.m[q] : m;
            r = w == q ? b.r[q] : r;
        }
        decode_step(s, __builtin_amdgcn_sbfe((int32_t)m, tau & 31, 1), __builtin_amdgcn_sbfe((int32_t)r, tau & 31, 1),
                    tau, row[tau]);
    }
    sa[T] = make_int4(s.lim, s.XR, s.lsR, enc_last(s));
    sb[T] = make_int2(s.A1, s.A2);
}

// Moves sorted by first changed period, 64 at a time: every lane of a batch starts from the base's state
// before the batch's first period t0 (a move changes nothing before its own first period, so its decode
// there equals the base's) and the lanes step through the same periods, reading rows and setup bits at a
// uniform position as the full decode does: single periods up to a multiple of 8, then blocks of 8 in the
// full decode's form (two chunks of four, the setup words chosen once per block), then single periods to the
// horizon.  Before each block every lane checks whether it has rejoined the base (or turned infeasible); the
// batch ends when all have, or at the horizon.
template <int NW>
__device__ __forceinline__ void eval_items_inc(const EvalArgs &a, EvalShared &sh, const int4 *snapA, const int2 *snapB,
                                               int N, int T, const ProdParams &pp) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int decoded = 0;
    for (int basei = wave * 64; basei < N; basei += blockDim.x) {
        const int idx = basei + lane;
        const bool in = idx < N;
        const int e = sh.item[in ? idx : basei];
        const int j = e >> 9, blk = (e >> 7) & 3, t = e & 127;
        const int slot = blk * T + t;
        const int t0 = __builtin_amdgcn_readfirstlane(sh.item[basei] & 127);   // sorted: the batch's first period
        Bits mb = sh.bits[j];
        const int dnM = blk == 0 ? (test_bit(mb.m, t) ? -1 : 1) : 0;   // a swap keeps the number of setups
        const int dnR = blk == 1 ? (test_bit(mb.r, t) ? -1 : 1) : 0;
        xor_move<NW>(mb, blk, t);
        const int t1 = blk >= 2 ? t + 1 : t;                             // last changed period
        DecodeState s;
        {
            const int4 sa = snapA[j * (T + 1) + t0];
            const int2 sb = snapB[j * (T + 1) + t0];
            s.lim = sa.x;
            s.XR = sa.y;
            s.lsR = sa.z;
            s.lastM = sa.w < 0 ? 0 : sa.w;
            s.nolast = sa.w < 0 ? -1 : 0;
            s.A1 = sb.x;
            s.A2 = sb.y;
        }
        bool done = !in;
        int64_t c = kInf;
        // the lane's setup word w (w wave-uniform)
        auto word = [&](const uint32_t (&v)[kWords], int w) {
            uint32_t x = v[0];
#pragma unroll
            for (int q = 1; q < NW; ++q) x = w == q ? v[q] : x;
            return (int32_t)x;
        };
        // before period tau: has this lane rejoined the base (its cost is then known) or turned infeasible?
        // True when every lane of the batch is done.
        auto check = [&](int tau) -> bool {
            if (!done) {
                if (s.bad) {   // infeasible: kInf
                    done = true;
                } else if (tau > t1) {
                    const int4 sa = snapA[j * (T + 1) + tau];
                    if (sa.x == s.lim && sa.y == s.XR && sa.z == s.lsR && sa.w == enc_last(s)) {   // rejoined
                        const int2 sb = snapB[j * (T + 1) + tau];
                        const int64_t dA1 = (int64_t)s.A1 - sb.x, dA2 = (int64_t)s.A2 - sb.y;
                        c = sh.cost[j] + (int64_t)pp.kM * dnM + (int64_t)pp.kR * dnR - (int64_t)pp.hM * (dA1 + dA2) +
                            (int64_t)pp.hR * dA1;
                        done = true;
                    }
                }
            }
            return !__any(!done);
        };
        auto single = [&](int tau) {
            const int w = tau >> 5;
            decode_step(s, __builtin_amdgcn_sbfe(word(mb.m, w), tau & 31, 1),
                        __builtin_amdgcn_sbfe(word(mb.r, w), tau & 31, 1), tau, sh.row[tau]);
        };
        int tau = t0;
        bool all = false;
        for (; tau < T && (tau & 7) != 0; ++tau) single(tau);
        int2 ca[4], cb[4];
        for (; tau + 8 <= T; tau += 8) {
            if (tau > t0 && check(tau)) {
                all = true;
                break;
            }
            load_chunk(sh.row, tau, ca);
            load_chunk(sh.row, tau + 4, cb);
            const int w = tau >> 5;   // a block of 8 never crosses a setup word
            const int32_t m = word(mb.m, w), r = word(mb.r, w);
            decode_chunk(s, m, r, tau, ca);
            decode_chunk(s, m, r, tau + 4, cb);
        }
        if (!all && tau < T && tau > t0 && (tau & 7) == 0) all = check(tau);
        for (; !all && tau < T; ++tau) single(tau);
        if (!done) c = decode_finish<NW>(s, mb, T, pp);   // decoded to the horizon (kInf when infeasible)
        if (in) {
            decoded += tau - t0;                           // period-steps this lane's batch ran
            if (c != kInf) atomicMin(&sh.key[j], ((unsigned long long)c << kSlotBits) | (unsigned long long)slot);
            if (a.slot_price) a.slot_price[sh.out_off[j] + slot] = c == kInf ? kInf : sh.F[j] - sh.cost[j] + c;
        }
    }
    atomicAdd(&sh.decoded, decoded);
}

// Pair j of a pricing workgroup: its product index pi within the workgroup's products and its chain index ci
// (from g0), in the rectangular form (j = pi * nc + ci) or the range form.
__device__ __forceinline__ void eval_pair(const EvalWg &d, int j, int &pi, int &ci) {
    if (d.G > 0) {
        const int q = d.q0 + j;
        pi = q / d.G - d.p;
        ci = q - (q / d.G) * d.G;
    } else {
        pi = j / d.n;
        ci = j - pi * d.n;
    }
}

template <bool INC, int MODEL = 0>
__device__ __forceinline__ void eval_body(const EvalArgs &a, const EvalWg *__restrict__ wg, EvalShared &sh,
                                          int4 *s_snap) {
    const EvalWg d = wg[blockIdx.x];
    if (d.n == 0) return;   // an empty entry (uniform for the workgroup)
    const int g0 = d.g0, K = d.K, T = d.T, p = d.p;
    const int np = INC ? 1 : max(d.np, 1);
    const int n = d.G > 0 ? d.n : d.n * np;   // pairs
    const ProdParams pp = a.prod[d.prod];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int t = threadIdx.x; t < np * T; t += blockDim.x) sh.row[t] = a.rows[d.row + t];
    if (np > 1)
        for (int q = threadIdx.x; q < np; q += blockDim.x) sh.pp[q] = a.prod[d.prod + q];
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        int pi, ci;
        eval_pair(d, j, pi, ci);
        const int64_t cp = d.cp + (int64_t)ci * K + pi;
        sh.pidx[j] = (uint8_t)pi;
        sh.bits[j] = a.cur[cp];
        sh.cost[j] = a.cur_cost[cp];
        sh.F[j] = a.cstate[g0 + ci].F;
        sh.key[j] = kInfKey;
        sh.out_off[j] = a.slot_price ? a.price_off[g0 + ci] + (int64_t)(p + pi) * 4 * T : 0;
    }
    __syncthreads();

    const bool fm = a.nb_mask & 1u, fr = a.nb_mask & 2u, shift = a.nb_mask & 4u;
    const int nflip = (fm ? T : 0) + (fr ? T : 0);
    // the pairs' move counts (one lane per pair, n <= 64) and their exclusive prefix, by wavefront 0
    if (wave == 0) {
        int cnt = 0;
        if (lane < n) {
            cnt = nflip;
            if (shift) {
                uint32_t vm[kWords], vr[kWords];
                swap_valid(sh.bits[lane].m, T, vm);
                swap_valid(sh.bits[lane].r, T, vr);
                cnt += popc_words(vm) + popc_words(vr);
            }
        }
        int inc = cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int up = __shfl_up(inc, d, 64);
            inc += lane >= d ? up : 0;
        }
        if (lane < n) sh.off[lane] = inc - cnt;
        if (lane == 63) sh.off[n] = inc;
    }
    if (a.slot_price) {  // every slot of the group starts as "not a priced move"
        for (int j = 0; j < n; ++j)
            for (int l = threadIdx.x; l < 4 * T; l += blockDim.x) a.slot_price[sh.out_off[j] + l] = kInf;
    }
    __syncthreads();
    // the item table: flips (zM then zR), then each chain's valid swaps in period order; for incremental
    // pricing sorted by period instead (period t: every chain's flips and valid swaps at t)
    const int fblk0 = fm ? 0 : 1;
    if constexpr (INC) {
        for (int t = threadIdx.x; t < T; t += blockDim.x) {
            int cnt = 0;
            for (int j = 0; j < n; ++j) {
                const Bits &b = sh.bits[j];
                cnt += (fm ? 1 : 0) + (fr ? 1 : 0);
                if (shift && t + 1 < T) {
                    cnt += test_bit(b.m, t) != test_bit(b.m, t + 1);
                    cnt += test_bit(b.r, t) != test_bit(b.r, t + 1);
                }
            }
            sh.tcount[t] = cnt;
        }
        __syncthreads();
        if (wave == 0) {   // exclusive prefix over the periods (T <= 128: two per lane)
            const int c0 = 2 * lane < T ? sh.tcount[2 * lane] : 0;
            const int c1 = 2 * lane + 1 < T ? sh.tcount[2 * lane + 1] : 0;
            int inc = c0 + c1;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int up = __shfl_up(inc, d, 64);
                inc += lane >= d ? up : 0;
            }
            const int ex = inc - c0 - c1;
            if (2 * lane < T) sh.tcount[2 * lane] = ex;
            if (2 * lane + 1 < T) sh.tcount[2 * lane + 1] = ex + c0;
        }
        __syncthreads();
        for (int t = threadIdx.x; t < T; t += blockDim.x) {
            int o = sh.tcount[t];
            for (int j = 0; j < n; ++j) {
                const Bits &b = sh.bits[j];
                if (fm) sh.item[o++] = pack_item(j, 0, t);
                if (fr) sh.item[o++] = pack_item(j, 1, t);
                if (shift && t + 1 < T) {
                    if (test_bit(b.m, t) != test_bit(b.m, t + 1)) sh.item[o++] = pack_item(j, 2, t);
                    if (test_bit(b.r, t) != test_bit(b.r, t + 1)) sh.item[o++] = pack_item(j, 3, t);
                }
            }
        }
    }
    for (int j = wave; j < n && !INC; j += nw) {
        uint16_t *it = sh.item + sh.off[j];
        for (int i = lane; i < nflip; i += 64) {
            const int blk = fblk0 + (i >= T ? 1 : 0);
            it[i] = pack_item(j, blk, i - (i >= T ? T : 0));
        }
        if (shift)   // each chain's valid swaps in period order, the zM swaps first
            compact_swaps(sh.bits[j], T, it + nflip, [j](int z, int t) { return pack_item(j, 2 + z, t); });
    }
    __syncthreads();

    const int N = sh.off[n];
    if constexpr (INC) {
        int4 *snapA = s_snap;                                              // [n][T+1]
        int2 *snapB = reinterpret_cast<int2 *>(s_snap + (size_t)n * (T + 1));   // [n][T+1]
        if (threadIdx.x < n) {
            const int j = threadIdx.x;
            if (T <= 64)
                base_snapshot<2>(sh.bits[j], sh.row, T, snapA + j * (T + 1), snapB + j * (T + 1));
            else
                base_snapshot<4>(sh.bits[j], sh.row, T, snapA + j * (T + 1), snapB + j * (T + 1));
        }
        if (threadIdx.x == 0) sh.decoded = 0;
        __syncthreads();
        if (T <= 64)
            eval_items_inc<2>(a, sh, snapA, snapB, N, T, pp);
        else
            eval_items_inc<4>(a, sh, snapA, snapB, N, T, pp);
    } else {
        if (T <= 64)
            eval_items<2, MODEL>(a, sh, N, T, pp, np);
        else
            eval_items<4, MODEL>(a, sh, N, T, pp, np);
    }
    __syncthreads();
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        int pi, ci;
        eval_pair(d, j, pi, ci);
        a.prod_key[d.cp + (int64_t)ci * K + pi] = sh.key[j];
    }
    if (threadIdx.x == 0) {
        unsigned long long *ctr = a.evals + (size_t)(blockIdx.x & (kCounterSlots - 1)) * kCounterStride;
        atomicAdd(ctr, (unsigned long long)N);
        atomicAdd(ctr + 1, (unsigned long long)N * (unsigned long long)T);
        // period-steps decoded: the base snapshots and the moves' incremental decodes, or every move in full
        atomicAdd(ctr + 2, INC ? (unsigned long long)sh.decoded + (unsigned long long)n * T
                               : (unsigned long long)N * (unsigned long long)T);
    }
}

}  // namespace

template <int MODEL>
__global__ __launch_bounds__(256) void k_eval(EvalArgs a, const EvalWg *__restrict__ wg) {
    __shared__ EvalShared sh;
    eval_body<false, MODEL>(a, wg, sh, nullptr);
}

// The same with 512-1024-thread workgroups (the range form spread over the compute units).
template <int MODEL>
__global__ __launch_bounds__(1024) void k_eval_wide(EvalArgs a, const EvalWg *__restrict__ wg) {
    __shared__ EvalShared sh;
    eval_body<false, MODEL>(a, wg, sh, nullptr);
}

// The same sweep priced incrementally; dynamic LDS holds the base snapshots (24 bytes per chain and period).
__global__ __launch_bounds__(256) void k_eval_inc(EvalArgs a, const EvalWg *__restrict__ wg) {
    __shared__ EvalShared sh;
    extern __shared__ __attribute__((aligned(16))) int4 s_snap[];
    eval_body<true>(a, wg, sh, s_snap);
}

// ---------------------------------------------------------------------------------------------------
// k_eval_iv: the sweep by interval pricing.  A wavefront takes per_wave consecutive (chain, product) pairs, one at
// a time for T > 32, two at a time (32 lanes each) for T > 16, four at a time up to 16, and prices the four slot
// blocks of each with one period per lane.  No workgroup synchronisation and no move list: a slot is (block,
// lane).
//
// Bound by VALU issue, as k_eval: at 256 instances (K 100..1000, T 52 or 104) x 16 chains 2.78 ms in place of 15.9, at 1024 instances (K 10..200, T 12, 24 or 52) x 8 chains 0.43 in place of 1.18, at one of
// 100 x 52 with 64 chains 14 us in place of 32.
// ---------------------------------------------------------------------------------------------------
namespace {

// A value every lane of the wavefront reads alike, through the scalar cache (written before the launch only).
template <class T>
__device__ __forceinline__ T load_uniform(const T *p) {
    static_assert(sizeof(T) % 4 == 0, "whole words");
    typedef const __attribute__((address_space(4))) uint32_t *Words;
    const Words w = (Words)(uintptr_t)p;
    uint32_t r[sizeof(T) / 4];
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 4; ++i) r[i] = w[i];
    T out;
    __builtin_memcpy(&out, r, sizeof(T));
    return out;
}

template <int G, int NV, bool STRICT, bool STEPS>
__device__ __forceinline__ void eval_unit(const EvalArgs &a, const ChainInfo &ci, int g, int64_t F, int64_t cp, int cnt,
                                          iv::Lds<G, NV> &sh, uint32_t &moves, uint32_t &decoded) {
    const int lane = threadIdx.x & 63, t0 = lane & (G - 1), grp = lane / G;
    const int T = ci.T, p0 = (int)(cp - ci.cp0);
    const int my = G == 64 ? 0 : min(grp, cnt - 1);   // a group without a pair repeats the last one's
    const bool live = G == 64 || grp < cnt;
    int2 row[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int t = t0 + 64 * v;
        row[v] = t < T ? a.rows[ci.row0 + (p0 + my) * T + t] : iv::no_row();
    }
    const ProdParams pp = G == 64 ? load_uniform(a.prod + ci.prod0 + p0) : a.prod[ci.prod0 + p0 + my];
    const Bits b = G == 64 ? load_uniform(a.cur + cp) : a.cur[cp + my];
    const int64_t base = G == 64 ? load_uniform(a.cur_cost + cp) : a.cur_cost[cp + my];
    const iv::Cost c = iv::cost_of(pp);
    const iv::Masks<G, NV> k = iv::masks_of<G, NV>(b);
    iv::Pattern<G, NV, STRICT> pat;
    pat.build(k, row, T, c, sh);

    const bool fm = a.nb_mask & 1u, fr = a.nb_mask & 2u, shift = a.nb_mask & 4u;
    int32_t x[4][NV];   // cost changes by slot block
    iv::Word<G> vm[NV], vr[NV];
    int steps = 0;
    uint32_t n = (fm ? T : 0) + (fr ? T : 0);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const iv::Period &q = pat.p[v];
        const bool in = q.t < T;
        x[0][v] = x[1][v] = x[2][v] = x[3][v] = kBad32;
        if (fm) {
            const int32_t y = pat.flip_m(q, c, steps);
            x[0][v] = in ? y : kBad32;
        }
        if (fr) {
            const int32_t y = pat.flip_r(q, c, steps);
            x[1][v] = in ? y : kBad32;
        }
        if (shift) {
            vm[v] = iv::swap_bits<G, NV>(k.m, v, T);
            vr[v] = iv::swap_bits<G, NV>(k.r, v, T);
            const bool sm = iv::lane_bit<G>(vm[v]), sr = iv::lane_bit<G>(vr[v]);
            const typename iv::Pattern<G, NV, STRICT>::Next nx = pat.next_of(k, v);
            const int32_t y = pat.swap_m(q, nx, c, sm, steps), z = pat.swap_r(q, nx, c, sr, steps);
            x[2][v] = sm ? y : kBad32;
            x[3][v] = sr ? z : kBad32;
            n += G < 64 ? __popc((uint32_t)vm[v]) + __popc((uint32_t)vr[v]) : __popcll(vm[v]) + __popcll(vr[v]);
        }
    }
    if (a.slot_price) {
        int64_t *out = a.slot_price + (a.price_off[g] + (int64_t)(p0 + my) * 4 * T);
#pragma unroll
        for (int blk = 0; blk < 4; ++blk)
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int t = t0 + 64 * v;
                if (live && t < T) out[blk * T + t] = x[blk][v] == kBad32 ? kInf : F + x[blk][v];
            }
    }
    // the lowest (cost, slot): the cost first, then the lowest slot that has it.  (x as unsigned from the lowest int32:
    // kBad32 is the largest.)
    uint32_t low = 0;
#pragma unroll
    for (int blk = 0; blk < 4; ++blk)
#pragma unroll
        for (int v = 0; v < NV; ++v) low = max(low, ~((uint32_t)x[blk][v] ^ 0x80000000u));
    low = iv::scan_max<G>(low);
    const int last = lane | (G - 1);
    int slot = 0;
    if constexpr (G == 64) {
        const int32_t best = (int32_t)(~(uint32_t)iv::last_lane(low) ^ 0x80000000u);
#pragma unroll
        for (int blk = 3; blk >= 0; --blk)
#pragma unroll
            for (int v = NV - 1; v >= 0; --v) {
                const uint64_t at = __ballot(x[blk][v] == best);
                slot = at ? blk * T + 64 * v + __builtin_ctzll(at) : slot;
            }
        if (lane == 0)
            a.prod_key[cp] = best == kBad32 ? kInfKey : ((uint64_t)(base + best) << kSlotBits) | (uint64_t)slot;
    } else {
        const int32_t best = (int32_t)(~(uint32_t)__shfl((int)low, last, 64) ^ 0x80000000u);
        uint32_t at = 0;
#pragma unroll
        for (int blk = 3; blk >= 0; --blk) at = x[blk][0] == best ? 0x10000u - (uint32_t)(blk * T + t0) : at;
        at = iv::scan_max<G>(at);
        if (lane == last && live)
            a.prod_key[cp + my] =
                best == kBad32 ? kInfKey : ((uint64_t)(base + best) << kSlotBits) | (uint64_t)(0x10000u - at);
    }
    if (t0 == 0 && live) moves += n;
    if constexpr (STEPS) decoded += live ? (uint32_t)steps + (t0 == 0 ? n + (uint32_t)T : 0u) : 0u;
}

}  // namespace

template <bool LONG, bool STRICT, bool STEPS>
__global__ __launch_bounds__(256) void k_eval_iv(EvalArgs a, int64_t cp_begin, int64_t n_cp, int32_t per_wave) {
    constexpr size_t kBytes = std::max({sizeof(iv::Lds<16, 1>), sizeof(iv::Lds<32, 1>), sizeof(iv::Lds<64, 1>),
                                        LONG ? sizeof(iv::Lds<64, 2>) : (size_t)0});
    __shared__ __attribute__((aligned(16))) unsigned char lds[4][kBytes];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t first = ((int64_t)blockIdx.x * 4 + wave) * per_wave;
    const int64_t end = cp_begin + min(first + per_wave, n_cp);
    uint32_t moves = 0, psteps = 0, decoded = 0;   // per lane (at most 16 pairs of 4 T <= 512 moves)
    for (int64_t cp = cp_begin + first; cp < end;) {
        const int g = load_uniform(a.cp_chain + cp);
        const ChainInfo ci = load_uniform(a.chains + g);
        const int64_t F = a.slot_price ? load_uniform(&a.cstate[g].F) : 0;
        const int64_t left = min(end, ci.cp0 + ci.K) - cp;
        const int T = ci.T;
        uint32_t m = 0;
        int cnt = 1;
        if (T <= 16) {
            cnt = (int)min(left, (int64_t)4);
            eval_unit<16, 1, STRICT, STEPS>(a, ci, g, F, cp, cnt, *reinterpret_cast<iv::Lds<16, 1> *>(lds[wave]), m, decoded);
        } else if (T <= 32) {
            cnt = (int)min(left, (int64_t)2);
            eval_unit<32, 1, STRICT, STEPS>(a, ci, g, F, cp, cnt, *reinterpret_cast<iv::Lds<32, 1> *>(lds[wave]), m, decoded);
        } else if (!LONG || T <= 64) {
            eval_unit<64, 1, STRICT, STEPS>(a, ci, g, F, cp, cnt, *reinterpret_cast<iv::Lds<64, 1> *>(lds[wave]), m, decoded);
        } else if constexpr (LONG) {
            eval_unit<64, 2, STRICT, STEPS>(a, ci, g, F, cp, cnt, *reinterpret_cast<iv::Lds<64, 2> *>(lds[wave]), m, decoded);
        }
        moves += m;
        psteps += m * (uint32_t)T;
        cp += cnt;
    }
    const int32_t n = iv::last_lane(iv::scan_add<64>(moves)), ps = iv::last_lane(iv::scan_add<64>(psteps));
    const int32_t dec = STEPS ? iv::last_lane(iv::scan_add<64>(decoded)) : ps;
    if (lane == 0 && first < n_cp) {
        unsigned long long *ctr = a.evals + (size_t)((blockIdx.x * 4 + wave) & (kCounterSlots - 1)) * kCounterStride;
        atomicAdd(ctr, (unsigned long long)n);
        atomicAdd(ctr + 1, (unsigned long long)ps);
        atomicAdd(ctr + 2, (unsigned long long)dec);
    }
}

// The pricing table for chains g0 .. g0+ng-1 and zeroed counters, on the device (see EvalPrepArgs).
__global__ __launch_bounds__(256) void k_eval_prep(EvalPrepArgs a) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = tid; i < a.n_cp; i += stride) {
        const int64_t cp = a.cp_begin + i;
        const int g = a.cp_chain[cp];
        const ChainInfo ci = a.chains[g];
        const int first = max(a.g0, ci.inst * a.chains_per_inst);            // the instance's first chain in range
        const int end = min(a.g0 + a.ng, (ci.inst + 1) * a.chains_per_inst);  // and one past its last
        EvalWg w{};
        if ((g - first) % a.group == 0) {
            const int p = (int)(cp - ci.cp0);
            w.cp = cp;
            w.g0 = g;
            w.n = min(a.group, end - g);
            w.K = ci.K;
            w.T = ci.T;
            w.p = p;
            w.prod = ci.prod0 + p;
            w.row = a.prod[ci.prod0 + p].row;
            w.np = 1;
        }
        a.table[i] = w;
    }
    for (int64_t j = tid; j < counter_words(); j += stride) a.counters[j] = 0ull;
}

// ---------------------------------------------------------------------------------------------------
// k_chain_best<CHAINS>: per-product (price, slot) and each chain's lexicographic minimum, CHAINS chains to a workgroup.
// One more workgroup sums the pricing launch's counters and clears them.  Results go where the host reads them (mapped
// host memory when they are small), so that a call ends with the launch and one wait: six copies and a memset of up to
// 16 KB each waited for the one before and were 120 of a small call's 131 us.
//
// CHAINS = 1: the workgroup's four wavefronts share one chain, the shortest way through few chains.  CHAINS = 16: a
// wavefront for each chain, and the sixteen results leave in two stores of 128 and 64 bytes; one at a time, 8192 chains'
// results are 16384 stores across the host link (28 -> 10 us; at 4096 chains of up to
// 1000 products 18.2 -> 17.8 us, at 64 chains CHAINS = 1 is the faster, 4.0 against 5.0 us).
// ---------------------------------------------------------------------------------------------------
template <int CHAINS>
__global__ __launch_bounds__(CHAINS == 1 ? 256 : 64 * CHAINS) void k_chain_best(ChainBestArgs a) {
    constexpr int kWavesPer = CHAINS == 1 ? 4 : 1;   // wavefronts to a chain
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (blockIdx.x == gridDim.x - 1) {
        static_assert(kCounterSlots == 256, "one slot per thread of the first four wavefronts");
        __shared__ unsigned long long s_sum[3][4];
        if (threadIdx.x < kCounterSlots) {
            unsigned long long *c = a.counters + (size_t)threadIdx.x * kCounterStride;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int64_t n = wave_sum_i64((int64_t)c[i]);
                if (lane == 0) s_sum[i][wave] = (unsigned long long)n;
                c[i] = 0ull;
            }
        }
        __syncthreads();
        if (threadIdx.x < 3) a.totals[threadIdx.x] = s_sum[threadIdx.x][0] + s_sum[threadIdx.x][1] + s_sum[threadIdx.x][2] + s_sum[threadIdx.x][3];
        return;
    }
    const int b0 = blockIdx.x * CHAINS, b = b0 + (CHAINS == 1 ? 0 : wave);   // b: this wavefront's chain of the launch
    int64_t bp = kInf;
    int64_t bs = -1;
    if (b < a.n_chains) {
        const int g = a.chain0 + b;
        const ChainInfo ci = a.chains[g];
        const int64_t F = a.cstate[g].F;
#pragma unroll CHAINS == 1 ? 1 : 4
        for (int p = CHAINS == 1 ? (int)threadIdx.x : lane; p < ci.K; p += 64 * kWavesPer) {
            const int64_t cp = ci.cp0 + p;
            const uint64_t key = a.prod_key[cp];
            int64_t price = kInf;
            int32_t slot = -1;
            if (key != kInfKey) {
                price = F - a.cur_cost[cp] + (int64_t)(key >> kSlotBits);
                slot = (int32_t)(key & ((1u << kSlotBits) - 1));
            }
            if (a.prod_price) a.prod_price[cp] = price;
            if (a.prod_slot) a.prod_slot[cp] = slot;
            const int64_t gs = slot < 0 ? -1 : (int64_t)p * 4 * ci.T + slot;
            if (slot >= 0 && (price < bp || (price == bp && gs < bs))) { bp = price; bs = gs; }
        }
    }
    // lexicographic (price, slot) minimum over the wavefront
    for (int off = 32; off >= 1; off >>= 1) {
        const int64_t op = __shfl_xor(bp, off, 64);
        const int64_t os = __shfl_xor(bs, off, 64);
        if (os >= 0 && (bs < 0 || op < bp || (op == bp && os < bs))) { bp = op; bs = os; }
    }
    __shared__ int64_t s_p[CHAINS * kWavesPer], s_s[CHAINS * kWavesPer];
    if (lane == 0) { s_p[wave] = bp; s_s[wave] = bs; }
    __syncthreads();
    if ((int)threadIdx.x < CHAINS && b0 + (int)threadIdx.x < a.n_chains) {
        bp = s_p[threadIdx.x];
        bs = s_s[threadIdx.x];
        for (int w = 1; w < kWavesPer; ++w) {
            if (s_s[w] >= 0 && (bs < 0 || s_p[w] < bp || (s_p[w] == bp && s_s[w] < bs))) { bp = s_p[w]; bs = s_s[w]; }
        }
        a.best[b0 + threadIdx.x] = bs < 0 ? kInf : bp;
        a.best_slot[b0 + threadIdx.x] = (int32_t)bs;
    }
}

// ---------------------------------------------------------------------------------------------------
// k_run: persistent GVNS.  One workgroup per chain, W wavefronts.  Invariant at every iteration start:
// work == cur for every product of the chain.  The instance's rows sit in LDS when they fit
// (K*T <= a.lds_rows), otherwise each wavefront stages the row of the product it works on.  The first
// iteration index comes from device memory so that a captured launch can be replayed unchanged.
// ---------------------------------------------------------------------------------------------------
namespace {

typedef uint16_t SwapList[2 * kTMax];   // compacted swap moves of a wavefront's product

struct RunShared {
    Bits db[kShakeMax];                    // shaken products (dirty list): bits after the shake
    int32_t dp[kShakeMax];                 //   and product index
    int64_t part[kMaxWaves];
    int64_t shk[kMaxWaves];
    int64_t ev[kMaxWaves];
    int64_t fb[kMaxWaves];
    int32_t verr[kMaxWaves];
    int32_t nd;
    int64_t draw_it;                       // the iteration whose draws are in draw (-1: none)
    uint32_t draw[64];
    // speculative iterations: the chain's state at a round start (read by one thread, so that the whole
    // workgroup decides alike), the round's accepted slot (-1: none) and abort flag
    ChainState coop_cs;
    int64_t coop_done_it;
    int32_t coop_round;   // the round this workgroup computes
    int32_t next_prod;    // VND: the next product index to hand to a wavefront that has finished its own
    int32_t coop_stop;
    int32_t coop_acc;
    int32_t coop_abort;
    int32_t coop_bmode;   // the round's update of the best solution: 0 none, 1 the accepted products, 2 all of x
    int64_t nbr[kMaxWaves];   // a round's learned counters per wavefront
    int64_t fbr[kMaxWaves];
};

// The next VND product index of a wavefront: one LDS add by lane 0, the value in lane 0.
__device__ __forceinline__ int next_index(int32_t &counter, int lane) {
    int v = 0;
    if (lane == 0) v = atomicAdd(&counter, 1);
    return __shfl(v, 0, 64);
}


// Speculative VND (plain search): each product in work is handled by a group of n_nb wavefronts, one per
// neighbourhood of the list.  In every round the neighbourhoods not yet settled in the current pass are
// priced in parallel on the group's current pattern; the group's leader then walks them in list order and
// applies the first strictly improving best move; results priced after an applied move are stale and are
// priced again in the next round on the new pattern.  The moves applied, and so the result, are those of
// the sequential pass of Algorithm 1; only the consumed evaluations are counted.
struct SpecGroup {
    Bits b;               // current pattern of the group's product
    int64_t cost;         // its exact cost (kInf until the unchanged pattern of a shaken product is priced)
    int64_t c_cur;        // cost of the product in x (before the shake)
    uint64_t res[4];      // best-move key of each neighbourhood priced this round
    uint64_t ck[4];       // contrast keys for the move log
    int64_t idc;          // cost of the unchanged pattern (first round of a shaken product)
    int32_t cnt[4];       // moves priced per neighbourhood this round
    int32_t p, q, improved, active, need_ident, passes;
};

struct SpecShared {
    SpecGroup grp[kMaxWaves];
    int32_t next;         // next product index to hand out
};

// A value in LDS, through pointers that say so.  (Two accesses of one branch each, to LDS and to device memory through
// generic pointers, are merged into one flat access before their address spaces are known.)
template <class T>
__device__ __forceinline__ T lds_load(const T *p) {
    static_assert(sizeof(T) % 8 == 0, "8-byte words");
    typedef const __attribute__((address_space(3))) uint64_t *Words;
    const Words w = (Words)p;
    uint64_t r[sizeof(T) / 8];
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 8; ++i) r[i] = w[i];
    T out;
    __builtin_memcpy(&out, r, sizeof(T));
    return out;
}
template <class T>
__device__ __forceinline__ void lds_store(T *p, const T &v) {
    static_assert(sizeof(T) % 8 == 0, "8-byte words");
    typedef __attribute__((address_space(3))) uint64_t *Words;
    const Words w = (Words)p;
    uint64_t r[sizeof(T) / 8];
    __builtin_memcpy(r, &v, sizeof(T));
#pragma unroll
    for (size_t i = 0; i < sizeof(T) / 8; ++i) w[i] = r[i];
}

// The flip of draw j (< kdraw) of iteration it, as product << 8 | its flip slot (K <= 2^20, 2T <= 256).
__device__ __forceinline__ uint32_t shake_flip(const RunArgs &a, int g, int64_t it, uint64_t stream, int j, uint64_t n, int T) {
    if (j >= a.kdraw) return 0u;
    const uint32_t f = shake_draw(a.seed, (uint64_t)g, (uint64_t)it, (uint64_t)j, n, stream), p = f / (uint32_t)(2 * T);
    return p << 8 | (f - p * (uint32_t)(2 * T));
}

// IV: the plain search's VND by interval pricing, with one (1) or up to two (2) periods per lane; 0: by full decodes.
template <bool SPEC, bool LEARNED, bool COOP = false, int MODEL = 0, bool PACK = false, bool MULTI = false, int IV = 0>
__device__ __forceinline__ void run_chain(const RunArgs &a, RunShared &sh, SwapList *lists, SpecShared &sp, int2 *s_rows) {
    static_assert(!PACK || LEARNED, "the packed form is the learned VND's");
    static_assert(!(SPEC && LEARNED), "the speculative VND prices whole neighbourhoods");
    static_assert(!(COOP && SPEC), "speculative iterations run the sequential VND");
    static_assert(!IV || !(SPEC || PACK || MULTI || (MODEL & kModelDispose)), "interval pricing: one product per wavefront");
    int g = blockIdx.x, slot = 0;   // chain, and (speculative iterations) the iteration of a round it computes
    if constexpr (COOP) {
        const int m = a.coop_m;
        if (a.coop_xcd) {   // consecutive workgroups go to consecutive XCDs: keep a chain's m on one
            const int xcd = blockIdx.x & 7, w = blockIdx.x >> 3;
            g = (w / m) * 8 + xcd;
            slot = w % m;
        } else {
            g = blockIdx.x / m;
            slot = blockIdx.x % m;
        }
    }
    if constexpr (COOP) {
        // Issue priority by slot: a round always needs slot 0 and needs slot j only if iterations 0..j-1 are
        // all rejected, so on a shared SIMD the earlier slots go first and the later ones take what is left.
        // (The best-of-G form needs every slot; its streams are alike.)
        if (!a.best_of) {
            if (slot == 0)
                __builtin_amdgcn_s_setprio(3);
            else if (slot < 4)
                __builtin_amdgcn_s_setprio(2);
            else if (slot < 8)
                __builtin_amdgcn_s_setprio(1);
        }
    }
    const ChainInfo ci = a.chains[g];
    const int K = ci.K, T = ci.T;
    const int64_t cp0 = ci.cp0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int W = blockDim.x >> 6;
    const int2 *inst_rows = a.rows + a.prod[ci.prod0].row;   // an instance's rows are contiguous
    const bool rows_in_lds = K * T <= a.lds_rows;
    const int64_t it_first = *a.it0;

    if (rows_in_lds) {
        for (int i = threadIdx.x; i < K * T; i += blockDim.x) s_rows[i] = inst_rows[i];
        __syncthreads();
    }
    // the chain's solution state, indexed by product: in LDS for the whole launch when it fits (copied in
    // here and back at the end), else in device memory
    // (accessors that branch on the place: a pointer that may be either is a flat access, which waits for both
    // kinds of memory)
    const bool st_lds = !COOP && a.state_off >= 0;
    Bits *l_cur = reinterpret_cast<Bits *>(reinterpret_cast<char *>(s_rows) + (st_lds ? a.state_off : 0)), *l_work = l_cur + K;
    int64_t *l_cur_cost = reinterpret_cast<int64_t *>(l_work + K), *l_work_cost = l_cur_cost + K;
    Bits *g_cur = a.cur + cp0, *g_work = a.work + cp0;
    int64_t *g_cur_cost = a.cur_cost + cp0, *g_work_cost = a.work_cost + cp0;
    if (COOP) {   // x in device memory, shared by the chain's workgroups; each iteration's VND into its slot
        const int64_t sb = ((int64_t)g * a.coop_m + slot) * a.coop_kmax;
        g_work = a.coop_res + sb;   // (a split round uses slot 0's region)
        g_work_cost = a.coop_res_cost + sb;
    } else if (st_lds) {
        for (int i = threadIdx.x; i < K; i += blockDim.x) {
            l_cur[i] = g_cur[i];
            l_work[i] = g_work[i];
            l_cur_cost[i] = g_cur_cost[i];
            l_work_cost[i] = g_work_cost[i];
        }
        __syncthreads();
    }
    auto cur_bits = [&](int p) -> Bits {
        if (st_lds) return lds_load(l_cur + p);
        return g_cur[p];
    };
    auto cur_cost = [&](int p) -> int64_t {
        if (st_lds) return lds_load(l_cur_cost + p);
        return g_cur_cost[p];
    };
    auto set_work = [&](int p, const Bits &b, int64_t cost) {
        if (st_lds) {
            lds_store(l_work + p, b);
            lds_store(l_work_cost + p, cost);
        } else {
            g_work[p] = b;
            g_work_cost[p] = cost;
        }
    };

    ChainState cs = a.cstate[g];
    int64_t evals = 0;   // per wavefront (uniform)
    int vnd_err = 0;     // per wavefront (uniform)
    int64_t nb_evals = 0, fallbacks = 0;   // learned mode, per wavefront
    // learned search: this wavefront's tiles after the rows region (kept 16-byte aligned), and the scorer's
    // weight fragments
    const int rows_entries = run_rows_entries(a.lds_rows, IV && !LEARNED ? 0 : W);
    // (the packed form: one region for the workgroup), and interval pricing's states and records after them
    constexpr int kTiles = LEARNED ? kLearnedWaveBytes : 0;
    constexpr int kIvBytes = IV == 2 ? (int)sizeof(iv::Lds<64, 2>) : IV == 1 ? (int)sizeof(iv::Lds<64, 1>) : 0;
    char *lbase = reinterpret_cast<char *>(s_rows + rows_entries) + (PACK ? 0 : wave * (kTiles + kIvBytes));
    char *ivbase = lbase + kTiles;
    LearnedLds L{reinterpret_cast<__bf16 *>(lbase), reinterpret_cast<uint16_t *>(lbase + 64 * 16 * 2)};
    mlp::Frags fr;
    if constexpr (LEARNED) mlp::load_frags(a.mlp, fr);
    const uint64_t nflip_all = 2ull * (uint64_t)K * (uint64_t)T;
    const uint64_t stream = COOP && a.best_of ? (uint64_t)slot : 0u;   // best-of-G: each workgroup its own
    if (threadIdx.x == 0) sh.draw_it = -1;
    __syncthreads();

    int32_t coop_round = 0;   // speculative iterations: the round this workgroup computes
    int32_t coop_known = -1;  //   thread 0: the round counter as last acquired (-1: not yet)
    int64_t done_it = 0;      //   and the iterations resolved before it
    int64_t executed = 0;     //   move-evaluations this workgroup computed (thread 0)
    for (int i = 0; COOP || i < a.iters; ++i) {
        int64_t it = it_first + i;
        int kshake = cs.k;
        bool go = true;           // this workgroup has an iteration to compute in this round
        int active = 1;           // iterations computed in this round
        bool split = false;       // one iteration whose products are shared out over the chain's workgroups
        int vfirst = wave, vstep = W;   // this wavefront's products in the VND loop
        bool may_abandon = false;       // the iteration is dropped once the leader resolves the round without it
        const int64_t ev_round = evals, nb_round = nb_evals, fb_round = fallbacks;
        if constexpr (COOP) {
            // the chain's state as the leader left it.  The round counter comes first: a workgroup that
            // computed an abandoned iteration may join a round the leader has already moved past, and
            // then reads a newer state than that round's; its summary carries the older round and is
            // never used.
            if (threadIdx.x == 0) {
                sh.coop_round = coop_known >= 0 ? coop_known
                                                : __hip_atomic_load(&a.coop_ctl[g].round, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
                sh.coop_cs = a.cstate[g];
                sh.coop_done_it = a.coop_ctl[g].iters_done;
                sh.coop_stop = sh.coop_done_it >= a.iters ||
                               __hip_atomic_load(&a.coop_ctl[g].abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            cs = sh.coop_cs;
            done_it = sh.coop_done_it;
            coop_round = sh.coop_round;
            if (sh.coop_stop) break;
            // Until x is known to be a local optimum an iteration runs the VND of every product (the first
            // iteration from the initial solution is most of a short run's time): then the m workgroups
            // share that one iteration's products, which are independent (Section 3), each shaking alike
            // and writing its products' results into slot 0's region.  Otherwise each workgroup computes
            // its own iteration of the round.
            // Best-of-G: every workgroup runs the same iteration from x, shaking with its own stream (slot).
            split = !cs.lopt && !a.best_of;
            active = (split || a.best_of) ? 1 : (int)min<int64_t>(a.coop_m, a.iters - done_it);
            go = split || a.best_of || slot < active;
            it = it_first + done_it + ((split || a.best_of) ? 0 : slot);
            may_abandon = !split && !a.best_of && slot > 0;
            kshake = cs.k;   // the shake size after this workgroup's slot rejections
            for (int q = 0; q < slot && !split && !a.best_of; ++q) kshake = kshake >= a.kmax ? 1 : kshake + 1;
            const int64_t sb = ((int64_t)g * a.coop_m + (split ? 0 : slot)) * a.coop_kmax;
            g_work = a.coop_res + sb;
            g_work_cost = a.coop_res_cost + sb;
            if (split) {
                vfirst = slot * W + wave;
                vstep = a.coop_m * W;
            }
        }
        int nd = 0;
        int64_t part = 0, shk = 0;
        if (go) {

        // ---- Shake(x, k): wavefront 0 draws k flips and keeps the feasible ones in the dirty list ----
        if (wave == 0) {
            const bool draw = lane < kshake;
            // lane j: product and flip slot of draw j, drawn ahead during the last iteration's VND if it guessed this one
            uint32_t f = sh.draw[lane];
            if (sh.draw_it != it) {
                f = shake_flip(a, g, it, stream, lane, nflip_all, T);
                sh.draw[lane] = f;
                wave_sync_lds();
            }
            const int pd = (int)(f >> 8), ld = (int)(f & 255u);
            bool dup = false;                                        // an earlier draw hit the same product
            for (int j = 0; j < kshake; ++j) {
                const int pj = __builtin_amdgcn_readlane(pd, j);
                dup |= draw && j < lane && pj == pd;
            }
            int nd = 0;
            // (k_run under the strict reading takes the second form for every shake: its full decode inlined at both places
            // costs the fourth wavefront per SIMD, 1.6x the time at eight wavefronts a workgroup.  The other searches keep
            // their wavefronts with both, and distinct draws are 2 to 4% of a short horizon's iteration faster so.)
            constexpr bool kOneForm = (MODEL & kModelStrict) != 0 && !(IV || COOP || MULTI);
            if (!kOneForm && !__any(dup)) {
                // distinct products: the draws are independent, so each lane resolves its own and the
                // feasible ones are compacted in draw order
                bool ok = false;
                Bits b = cur_bits(draw ? pd : 0);
                if (draw) {
                    apply_move(b, ld, T);
                    const ProdParams pp = a.prod[ci.prod0 + pd];
                    ok = rows_in_lds ? shake_feasible<MODEL>(b, s_rows + pd * T, T, pp)
                                     : shake_feasible<MODEL>(b, inst_rows + pd * T, T, pp);
                }
                const unsigned long long okm = __ballot(ok);
                if (ok) {
                    const int e = __popcll(okm & ((1ull << lane) - 1ull));
                    sh.dp[e] = pd;
                    sh.db[e] = b;
                }
                nd = __popcll(okm);
            } else {
                // products still are independent of each other: the first lane that drew a product resolves its draws
                // in order, each kept if it leaves the product feasible.  (In place of one draw after the other by the
                // whole wavefront: the search of a 10-product instance, where most shakes of three and more meet a
                // product twice, 2.63 -> 2.52 ms for 500 iterations.)
                uint64_t own = 0;   // the draws of this lane's product
                for (int j = 0; j < kshake; ++j) own |= (uint64_t)(__builtin_amdgcn_readlane(pd, j) == pd ? 1u : 0u) << j;
                int first = -1;     // the first draw that stays
                Bits b = cur_bits(draw ? pd : 0);
                if (draw && !dup) {
                    const ProdParams pp = a.prod[ci.prod0 + pd];
                    do {
                        const int j = (int)__builtin_ctzll(own);
                        own &= own - 1;
                        Bits bj = b;
                        apply_move(bj, (int)(sh.draw[j] & 255u), T);
                        const bool ok = rows_in_lds ? shake_feasible<MODEL>(bj, s_rows + pd * T, T, pp)
                                                    : shake_feasible<MODEL>(bj, inst_rows + pd * T, T, pp);
                        if (ok) b = bj;
                        first = ok && first < 0 ? j : first;
                    } while (own != 0);
                }
                // the dirty list, in the order of the products' first draws that stay
                uint64_t firsts = 0;
                for (int j = 0; j < kshake; ++j) {
                    const int fj = __builtin_amdgcn_readlane(first, j);
                    firsts |= fj >= 0 ? 1ull << fj : 0ull;
                }
                if (first >= 0) {
                    const int e = __popcll(firsts & ((1ull << first) - 1ull));
                    sh.dp[e] = pd;
                    sh.db[e] = b;
                }
                nd = __popcll(firsts);
            }
            if (lane == 0) {
                sh.nd = nd;
                sh.next_prod = W;   // wavefront w starts with product index w
            }
        }
        __syncthreads();
        nd = sh.nd;
        // the next iteration's draws (ten rounds of 64-bit products, half as long as a short VND), by the last wavefront
        // beside the others' VND: the iteration is the next one, or with speculative iterations this workgroup's
        // next one if the round is rejected as a whole; a wrong guess is drawn again
        if (wave == W - 1) {
            const int64_t ahead = it + (COOP && !split && !a.best_of ? a.coop_m : 1);
            sh.draw[lane] = shake_flip(a, g, ahead, stream, lane, nflip_all, T);
            if (lane == 0) sh.draw_it = ahead;
        }

        // ---- speculative VND: groups of n_nb wavefronts, one neighbourhood each ----
        if constexpr (SPEC) {
            const int nprod = cs.lopt ? nd : K;
            const int gsz = a.n_nb, G = W / gsz;
            const int gid = wave / gsz, role = wave - gid * gsz;
            int staged = -1;   // product whose row this wavefront holds in its LDS slice (uniform)
            // hands the group its next product (one lane)
            auto take = [&](SpecGroup &gr) {
                const int idx = atomicAdd(&sp.next, 1);
                if (idx >= nprod) {
                    gr.active = 0;
                    return;
                }
                int p, e = -1;
                if (cs.lopt) {
                    p = sh.dp[idx];
                    e = idx;
                } else {
                    p = idx;
                    for (int q = 0; q < nd; ++q) e = (e < 0 && sh.dp[q] == p) ? q : e;
                }
                gr.p = p;
                if (e >= 0) gr.b = sh.db[e];
                else gr.b = cur_bits(p);
                gr.c_cur = cur_cost(p);
                gr.cost = e >= 0 ? kInf : gr.c_cur;
                gr.need_ident = e >= 0;
                gr.q = 0;
                gr.improved = 0;
                gr.passes = 0;
                gr.active = 1;
            };
            if (threadIdx.x == 0) sp.next = 0;
            __syncthreads();
            if (gid < G && role == 0 && lane == 0) take(sp.grp[gid]);
            __syncthreads();
            for (;;) {
                bool any = false;
                for (int gg = 0; gg < G; ++gg) any |= sp.grp[gg].active != 0;
                if (!any) break;
                // pricing: every neighbourhood not settled in this pass, on the group's current pattern
                if (gid < G && sp.grp[gid].active && role >= sp.grp[gid].q) {
                    SpecGroup &gr = sp.grp[gid];
                    const int p = gr.p;
                    const ProdParams pp = a.prod[ci.prod0 + p];
                    const int2 *row;
                    if (rows_in_lds) {
                        row = s_rows + p * T;
                    } else {
                        int2 *slice = s_rows + wave * kTMax;
                        if (staged != p) {
                            for (int t = lane; t < T; t += 64) slice[t] = inst_rows[p * T + t];
                            wave_sync_lds();
                            staged = p;
                        }
                        row = slice;
                    }
                    const uint32_t nb = (a.nb_list >> (4 * role)) & 0xFu;
                    const bool id = gr.need_ident && role == gr.q;
                    const int chash = a.log_x ? (int)(((uint32_t)it * 2654435761u + (uint32_t)p * 40503u +
                                                       (uint32_t)(role + 4 * gr.passes) * 97u) & 0x7FFFFFFFu) : -1;
                    int64_t idc = 0, dummy = 0;
                    uint64_t ckey = kInfKey;
                    int nitems = 0;
                    const Bits b = gr.b;
                    const uint64_t key = wave_best_move(b, row, T, pp, nb, lists[wave], id, &idc, dummy, chash, &ckey,
                                                        &nitems);
                    if (lane == 0) {
                        gr.res[role] = key;
                        gr.ck[role] = ckey;
                        gr.cnt[role] = nitems;
                        if (id) gr.idc = idc;
                    }
                }
                __syncthreads();
                // resolution in list order by the group's leader lane
                if (gid < G && role == 0 && lane == 0 && sp.grp[gid].active) {
                    SpecGroup &gr = sp.grp[gid];
                    if (gr.need_ident) {
                        gr.cost = gr.idc;
                        shk += gr.idc - gr.c_cur;
                        gr.need_ident = 0;
                    }
                    bool applied = false;
                    for (int j = gr.q; j < gsz; ++j) {
                        evals += gr.cnt[j];
                        const uint64_t key = gr.res[j];
                        if (key != kInfKey && (int64_t)(key >> kSlotBits) < gr.cost) {
                            const int slot = (int)(key & ((1u << kSlotBits) - 1));
                            const int64_t c = (int64_t)(key >> kSlotBits);
                            if (a.log_x) {
                                const ProdParams pp = a.prod[ci.prod0 + gr.p];
                                const uint64_t ck = gr.ck[j];
                                const bool has_c = ck != kInfKey && ck != key;
                                const int2 *row = rows_in_lds ? s_rows + gr.p * T : inst_rows + gr.p * T;
                                log_moves(gr.b, row, T, pp, slot, c - gr.cost, has_c ? (int)(ck & 0xFFFFu) : -1,
                                          has_c ? (int64_t)(ck >> kSlotBits) - gr.cost : 0, a.log_x, a.log_y, a.log_n,
                                          a.log_cap);
                            }
                            apply_move(gr.b, slot, T);
                            gr.cost = c;
                            gr.improved = 1;
                            gr.q = j + 1;
                            applied = true;
                            break;
                        }
                    }
                    if (!applied || gr.q == gsz) {   // the pass is over
                        if (gr.improved && ++gr.passes <= kMaxPasses) {
                            gr.q = 0;
                            gr.improved = 0;
                        } else {
                            if (gr.improved) vnd_err = 1;
                            set_work(gr.p, gr.b, gr.cost);
                            part += gr.cost - gr.c_cur;
                            take(gr);
                        }
                    }
                }
                __syncthreads();
            }
        } else {
            // ---- VND (Algorithm 1) per product: the shaken products, or every product until x is known to
            //      be a local optimum ----
            const int nprod = cs.lopt ? nd : K;
            bool stale = false;   // the round moved on without this iteration (uniform)
            // Products go to wavefronts as they finish (a product's VND length varies, and a shake of more
            // products than wavefronts would otherwise put two on one wavefront however short the others
            // are); the products of a split round are shared out over the chain's workgroups in fixed order.
            const bool dyn = vstep == W;
            if constexpr (PACK) {
                // the packed learned VND: batches of up to P products, each searched by the whole workgroup
                // (a split round's batches shared out over the chain's workgroups in fixed order)
                const int P = a.learned_pack;
                const PackLds PL = pack_lds(lbase, W, P);
                auto round_now = [&]() -> int32_t {
                    if constexpr (COOP) {
                        if (may_abandon)
                            return __hip_atomic_load(&a.coop_ctl[g].round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                    return coop_round;
                };
                const int bfirst = dyn ? 0 : vfirst / W, bstep = dyn ? 1 : vstep / W;   // in batches
                for (int base = bfirst * P; base < nprod && !stale; base += bstep * P) {
                    const int cnt = min(P, nprod - base);
                    if (threadIdx.x == 0) {
                        for (int i = 0; i < cnt; ++i) {
                            const int idx = base + i;
                            int p, e = -1;
                            if (cs.lopt) {
                                p = sh.dp[idx];
                                e = idx;
                            } else {
                                p = idx;
                                for (int q = 0; q < nd; ++q) e = (e < 0 && sh.dp[q] == p) ? q : e;
                            }
                            PackProd &pr = PL.pk[i];
                            pr.p = p;
                            if (e >= 0) pr.b = sh.db[e];
                            else pr.b = cur_bits(p);
                            pr.c_cur = cur_cost(p);
                            pr.cost = e >= 0 ? kInf : pr.c_cur;   // a shaken product is priced with its first list
                            pr.need_ident = e >= 0 ? 1 : 0;
                        }
                    }
                    __syncthreads();
                    if (!learned_vnd_packed(PL, cnt, rows_in_lds ? s_rows : nullptr, inst_rows, a.prod + ci.prod0, T,
                                            a.nb_list, a.n_nb, a.memo, fr, a.permille, evals, nb_evals, fallbacks,
                                            coop_round, round_now)) {
                        stale = true;
                        break;
                    }
                    for (int i = 0; i < cnt; ++i) {
                        const PackProd &pr = PL.pk[i];
                        if (threadIdx.x == 0) set_work(pr.p, pr.b, pr.cost);
                        if (wave == 0) {   // the per-wavefront sums, once
                            part += pr.cost - pr.c_cur;
                            shk += pr.shk;
                            vnd_err |= pr.err;
                        }
                    }
                    __syncthreads();
                }
            } else {
            for (int idx = vfirst; idx < nprod && !stale;
                 idx = !dyn ? idx + vstep : nprod <= W ? nprod : __builtin_amdgcn_readfirstlane(next_index(sh.next_prod, lane))) {
                int p, e = -1;
                if (cs.lopt) {
                    p = sh.dp[idx];
                    e = idx;
                } else {
                    p = idx;
                    for (int q = 0; q < nd; ++q) e = (e < 0 && sh.dp[q] == p) ? q : e;
                }
                if constexpr (IV != 0) {
                    p = __builtin_amdgcn_readfirstlane(p);
                    const ProdParams pp = load_uniform(a.prod + ci.prod0 + p);
                    const Bits xb = cur_bits(p);
                    const int64_t c_cur = cur_cost(p);
                    Bits b = xb;
                    if (e >= 0) b = sh.db[e];
                    const bool has_x = cs.lopt && a.x_opt;
                    iv::Vnd vs{c_cur, 0, evals, 0};
                    auto round_now = [&]() -> int32_t {
                        if constexpr (COOP) {
                            if (may_abandon)
                                return __hip_atomic_load(&a.coop_ctl[g].round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                        return coop_round;
                    };
                    constexpr bool kStrict = (MODEL & kModelStrict) != 0;
                    auto row_at = [&](int t) -> int2 {
                        if (rows_in_lds) return lds_load(s_rows + p * T + t);
                        return inst_rows[p * T + t];
                    };
                    bool done;
                    auto vnd = [&](auto &choose) {
                        if (IV == 1 || T <= 64)
                            done = iv::vnd<1, kStrict>(b, vs, e >= 0, row_at, T, pp, has_x, xb, c_cur, a.nb_list, a.n_nb, a.memo != 0,
                                                       *reinterpret_cast<iv::Lds<64, 1> *>(ivbase), choose, coop_round, round_now);
                        else if constexpr (IV == 2)
                            done = iv::vnd<2, kStrict>(b, vs, e >= 0, row_at, T, pp, has_x, xb, c_cur, a.nb_list, a.n_nb, a.memo != 0,
                                                       *reinterpret_cast<iv::Lds<64, 2> *>(ivbase), choose, coop_round, round_now);
                    };
                    if constexpr (LEARNED) {
                        const int2 *row = s_rows + p * T;   // the scorer reads any period: a row in LDS
                        if (!rows_in_lds) {
                            int2 *slice = s_rows + wave * kTMax;
                            for (int t = lane; t < T; t += 64) slice[t] = inst_rows[p * T + t];
                            wave_sync_lds();
                            row = slice;
                        }
                        LearnedChoice choose{row, T, pp, L.sx, fr, a.permille};
                        vnd(choose);
                        nb_evals += vs.ranked;
                        fallbacks += vs.fallbacks;
                    } else {
                        iv::NoChoice choose;
                        vnd(choose);
                    }
                    evals = vs.evals;
                    vnd_err |= vs.err;
                    if (e >= 0) shk += vs.start - c_cur;
                    if (!done) {
                        stale = true;
                        break;
                    }
                    if (lane == 0) set_work(p, b, vs.cost);
                    part += vs.cost - c_cur;
                    continue;
                }
                const ProdParams pp = a.prod[ci.prod0 + p];
                const int2 *row;
                if (rows_in_lds) {
                    row = s_rows + p * T;
                } else {
                    int2 *slice = s_rows + wave * kTMax;
                    for (int t = lane; t < T; t += 64) slice[t] = inst_rows[p * T + t];
                    wave_sync_lds();
                    row = slice;
                }
                Bits b;
                if (e >= 0) b = sh.db[e];
                else b = cur_bits(p);
                const int64_t c_cur = cur_cost(p);
                int64_t cost = e >= 0 ? kInf : c_cur;   // a shaken product is priced with its first move list
                bool need_ident = e >= 0;
                bool improved = true;
                int passes = 0;
                uint32_t clean = 0;   // neighbourhoods priced without improvement since the last applied move
                // short horizons: consecutive neighbourhoods priced side by side in one pass when they fit 64 lanes
                // (a kernel of its own, so that the others keep their registers)
                const bool multi = MULTI && !a.log_x && !a.memo && T <= kMultiMaxT;
                while (improved && !stale) {
                    if (++passes > kMaxPasses) {
                        vnd_err = 1;
                        break;
                    }
                    improved = false;
                    for (int q = 0; q < a.n_nb;) {
                        if (multi) {
                            int32_t rnow = coop_round;
                            if constexpr (COOP) {
                                if (may_abandon)
                                    rnow = __hip_atomic_load(&a.coop_ctl[g].round, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT);
                            }
                            int used = 1;
                            const bool id = need_ident;
                            const uint64_t key = wave_best_move_multi<2, MODEL>(b, row, T, pp, a.nb_list, q, a.n_nb,
                                                                                lists[wave], id, cost, evals, used);
                            if (id) {
                                shk += cost - c_cur;
                                need_ident = false;
                            }
                            if (key != kInfKey) {   // improving by construction
                                apply_move(b, (int)(key & ((1u << kSlotBits) - 1)), T);
                                cost = (int64_t)(key >> kSlotBits);
                                improved = true;
                            }
                            q += used;
                            wave_sync_lds();
                            if (__builtin_amdgcn_readfirstlane(rnow) != coop_round) {
                                stale = true;
                                break;
                            }
                            continue;
                        }
                        if (a.memo && ((clean >> q) & 1u)) {   // same pattern: nothing to find
                            ++q;
                            continue;
                        }
                        // the round counter, read before the evaluation and looked at after it, so that the
                        // load's latency is hidden behind the pricing
                        int32_t rnow = coop_round;
                        if constexpr (COOP) {
                            if (may_abandon)
                                rnow = __hip_atomic_load(&a.coop_ctl[g].round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                        bool applied = false;
                        const uint32_t nb = (a.nb_list >> (4 * q)) & 0xFu;
                        uint64_t key, ckey = kInfKey;
                        int nitems = 0;
                        // contrast move for the log: a fixed pseudo-random item of this evaluation
                        const int chash = a.log_x ? (int)(((uint32_t)it * 2654435761u + (uint32_t)p * 40503u +
                                                           (uint32_t)(q + 4 * passes) * 97u) & 0x7FFFFFFFu) : -1;
                        if constexpr (LEARNED) {
                            int fb = 0;
                            const bool id = need_ident;
                            key = learned_best_move(b, row, T, pp, nb, lists[wave], L, fr, a.permille, id, cost,
                                                    evals, fb);
                            ++nb_evals;
                            fallbacks += fb;
                            if (id) {
                                shk += cost - c_cur;
                                need_ident = false;
                            }
                        } else {
                            int64_t idc = 0;
                            key = wave_best_move<MODEL>(b, row, T, pp, nb, lists[wave], need_ident, &idc, evals, chash,
                                                        &ckey,
                                                 &nitems);
                            if (need_ident) {
                                cost = idc;
                                shk += idc - c_cur;
                                need_ident = false;
                            }
                        }
                        if (key != kInfKey) {
                            const int64_t c = (int64_t)(key >> kSlotBits);
                            if (c < cost) {
                                const int slot = (int)(key & ((1u << kSlotBits) - 1));
                                if (!LEARNED && a.log_x) {
                                    const bool has_c = ckey != kInfKey && ckey != key;
                                    log_moves(b, row, T, pp, slot, c - cost, has_c ? (int)(ckey & 0xFFFFu) : -1,
                                              has_c ? (int64_t)(ckey >> kSlotBits) - cost : 0, a.log_x, a.log_y, a.log_n,
                                              a.log_cap);
                                }
                                apply_move(b, slot, T);
                                cost = c;
                                improved = true;
                                applied = true;
                            }
                        }
                        // a move changes the pattern: every earlier pricing is stale
                        clean = applied ? 0u : (clean | (1u << q));
                        ++q;
                        wave_sync_lds();
                        if (__builtin_amdgcn_readfirstlane(rnow) != coop_round) {
                            stale = true;
                            break;
                        }
                    }
                }
                if (stale) break;
                if (lane == 0) set_work(p, b, cost);
                part += cost - c_cur;
            }
            }
        }
        }   // go
        if (lane == 0) {
            sh.part[wave] = part;
            sh.shk[wave] = shk;
            if constexpr (COOP) {
                sh.ev[wave] = evals - ev_round;
                sh.verr[wave] = vnd_err;
                sh.nbr[wave] = nb_evals - nb_round;
                sh.fbr[wave] = fallbacks - fb_round;
            }
        }
        __syncthreads();

        if constexpr (COOP) {
            CoopCtl *ctl = a.coop_ctl + g;
            CoopSlot *mine = a.coop_slot + (int64_t)g * a.coop_m + slot;
            if (go && threadIdx.x == 0) {   // this iteration's summary
                int64_t delta = 0, dshake = 0, ev = 0, nbe = 0, fbe = 0;
                int err = 0;
                for (int w = 0; w < W; ++w) {
                    delta += sh.part[w];
                    dshake += sh.shk[w];
                    ev += sh.ev[w];
                    err |= sh.verr[w];
                    nbe += sh.nbr[w];
                    fbe += sh.fbr[w];
                }
                executed += ev;
                mine->F_local = cs.F + delta;
                mine->F_shaken = cs.F + dshake;
                mine->evals = ev;
                mine->nb_evals = nbe;
                mine->fallbacks = fbe;
                mine->err = err;
                mine->n_touch = cs.lopt ? nd : -1;   // -1: every product
                for (int q = 0; q < nd; ++q) mine->dp[q] = sh.dp[q];
            }
            // the VND results (written by every wavefront) and the summary, before the stamp: each wavefront's
            // stores completed, then one agent-scope release (it writes back the XCD's L2, whoever stored)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __syncthreads();
            if (go && threadIdx.x == 0)
                __hip_atomic_store(&mine->stamp, coop_round + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            if (slot == 0) {
                // the leader resolves the round in iteration order: the first accepted iteration ends it, so
                // it waits only for the slots up to that one (a split or best-of round needs all of them).
                // Wavefront 0 polls the m stamps side by side (lane j: slot j), loads each summary once its
                // slot and every earlier one have reported, and resolves them with wave-uniform arithmetic;
                // lane 0 writes.
                if (wave == 0) {
                    const int need = (split || a.best_of) ? a.coop_m : active;   // slots holding this round
                    const CoopSlot *sj = a.coop_slot + (int64_t)g * a.coop_m + min(lane, a.coop_m - 1);
                    int64_t dl = 0, ds = 0, le = 0;   // lane j: slot j's F_local - F, F_shaken - F, evaluations
                    int64_t lnb = 0, lfb = 0;          //   and its learned counters
                    int lerr = 0;
                    int have = 0;                      // leading slots whose summaries are loaded (uniform)
                    bool ok = true;
                    const int64_t t0 = wall_clock64();
                    for (uint32_t n = 0;; ++n) {
                        const int32_t st =
                            lane < need ? __hip_atomic_load(&sj->stamp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
                        const unsigned long long rdy = __ballot(lane < need && st == coop_round + 1);
                        const int r = (int)__builtin_ctzll(~rdy);   // need <= 16, so ~rdy has a zero bit
                        if (r > have) {
                            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // the summaries behind the stamps
                            if (lane >= have && lane < r) {
                                dl = sj->F_local - cs.F;
                                ds = sj->F_shaken - cs.F;
                                le = sj->evals;
                                lerr = sj->err;
                                lnb = sj->nb_evals;
                                lfb = sj->fallbacks;
                            }
                            have = r;
                        }
                        if (have >= need) break;
                        // no earlier iteration of the round is accepted, so iteration j is accepted when its
                        // local cost is below F
                        if (!(split || a.best_of) && __ballot(lane < have && dl < 0)) break;
                        if (n >= kCoopSpinLimit || wall_clock64() - t0 > a.coop_wait_ticks) {
                            ok = false;
                            break;
                        }
                        __builtin_amdgcn_s_sleep(2);
                    }
                    if (split) {   // the one iteration is the sum of every slot's share
                        dl = wave_sum_i64(dl);
                        ds = wave_sum_i64(ds);
                        le = wave_sum_i64(le);
                        lnb = wave_sum_i64(lnb);
                        lfb = wave_sum_i64(lfb);
                        lerr = __any(lerr != 0) ? 1 : 0;
                    }
                    int sel = 0;   // best-of-G: the stream whose result is kept
                    if (a.best_of) {
                        // the minimum local cost over the G streams, the lowest stream among equal values; every
                        // stream's evaluations count
                        const bool mine = ok && lane < a.coop_m;
                        const uint64_t myF = mine ? (uint64_t)(cs.F + dl) : ~0ull;
                        const uint64_t minF = wave_min_u64(myF);
                        const unsigned long long at = __ballot(mine && myF == minF);
                        sel = at ? (int)__builtin_ctzll(at) : 0;
                        dl = __shfl(dl, sel, 64);
                        ds = __shfl(ds, sel, 64);
                        le = wave_sum_i64(le);
                        lnb = wave_sum_i64(lnb);
                        lfb = wave_sum_i64(lfb);
                        lerr = __any(lerr != 0) ? 1 : 0;
                    }
                    const bool literal = a.best_of && a.best_literal;   // k fixed, the minimum always kept
                    int acc = -1, consumed = active, k = cs.k, err = ok ? 0 : 2;
                    int64_t F = cs.F, Fb = cs.F_best, ev = 0, nbe = 0, fbe = 0;
                    for (int j = 0; j < active && ok; ++j) {
                        const int64_t Fl = cs.F + __shfl(dl, j, 64), Fs = cs.F + __shfl(ds, j, 64);
                        ev += __shfl(le, j, 64);
                        nbe += __shfl(lnb, j, 64);
                        fbe += __shfl(lfb, j, 64);
                        err |= __shfl(lerr, j, 64);
                        const int accepted = literal ? 1 : Fl < F;
                        if (a.trace && lane == 0) {
                            Record r;
                            r.iter = (int32_t)(it_first + done_it + j);
                            r.k = k;
                            r.accepted = accepted;
                            r.winner = sel;
                            r.F_shaken = Fs;
                            r.F_local = Fl;
                            r.F_best = (accepted && Fl < Fb) ? Fl : Fb;
                            a.trace[(int64_t)g * a.iters + done_it + j] = r;
                        }
                        if (accepted) {
                            acc = a.best_of ? sel : j;   // the slot whose VND results x takes
                            consumed = j + 1;
                            F = Fl;
                            Fb = Fl < Fb ? Fl : Fb;
                            k = literal ? k : 1;
                            break;
                        }
                        k = k >= a.kmax ? 1 : k + 1;
                    }
                    // the best solution follows x when x becomes the cheapest so far: the accepted products
                    // when it held x before, all of x otherwise (x had moved to a worse solution)
                    const int bmode = (ok && acc >= 0 && F < cs.F_best) ? (cs.bsync ? 1 : 2) : 0;
                    if (lane == 0) {
                        sh.coop_acc = ok ? acc : -1;
                        sh.coop_abort = !ok;
                        sh.coop_bmode = bmode;
                        if (ok) {
                            cs.F = F;
                            cs.F_best = Fb;
                            cs.k = k;
                            cs.bsync = bmode ? 1 : (acc >= 0 ? 0 : cs.bsync);
                            if (acc >= 0) cs.lopt = 1;
                            ctl->iters_done = done_it + consumed;
                            ctl->evals += ev;
                            ctl->nb_evals += nbe;
                            ctl->fallbacks += fbe;
                        }
                        if (err) atomicOr(&ctl->err, err);
                    }
                }
                // (wavefront 0's acquires after the stamps invalidated the caches the compute unit reads
                // through; the barrier orders every thread's reads of the results after them)
                __syncthreads();
                const int acc = sh.coop_acc, bmode = sh.coop_bmode;
                if (acc >= 0) {   // x takes the accepted iteration's VND results
                    const CoopSlot *sj = a.coop_slot + (int64_t)g * a.coop_m + acc;
                    const int64_t sb = ((int64_t)g * a.coop_m + acc) * a.coop_kmax;
                    const int n = sj->n_touch < 0 ? K : sj->n_touch;
                    for (int q = threadIdx.x; q < n; q += blockDim.x) {
                        const int p = sj->n_touch < 0 ? q : sj->dp[q];
                        const Bits b = a.coop_res[sb + p];
                        a.cur[cp0 + p] = b;
                        a.cur_cost[cp0 + p] = a.coop_res_cost[sb + p];
                        if (bmode == 1) a.best[cp0 + p] = b;
                    }
                }
                if (bmode == 2) {
                    __syncthreads();
                    for (int q = threadIdx.x; q < K; q += blockDim.x) a.best[cp0 + q] = a.cur[cp0 + q];
                }
                // every wavefront's stores to x completed, then one agent-scope release with the round count
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __syncthreads();
                if (threadIdx.x == 0) {
                    a.cstate[g] = cs;
                    if (sh.coop_abort) ctl->abort = 1;
                    __hip_atomic_fetch_add(&ctl->round, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                    coop_known = coop_round + 1;
                }
            } else if (threadIdx.x == 0) {
                // (the wait's acquire invalidates the caches the whole compute unit reads through; the barrier
                // then orders the workgroup's later reads of x after it)
                if (!coop_wait_ge(&ctl->round, coop_round + 1, a.coop_wait_ticks, &coop_known)) {
                    __hip_atomic_store(&ctl->abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    atomicOr(&ctl->err, 2);
                    coop_known = -1;
                }
            }
            __syncthreads();
            continue;
        }

        // ---- acceptance ----
        int64_t delta = 0, dshake = 0;
        for (int w = 0; w < W; ++w) {
            delta += sh.part[w];
            dshake += sh.shk[w];
        }
        const int64_t F_local = cs.F + delta;
        const int accepted = F_local < cs.F;
        // the best solution follows x when x becomes the cheapest so far: the touched products when it held
        // x before, all of x otherwise
        const int bmode = (accepted && F_local < cs.F_best) ? (cs.bsync ? 1 : 2) : 0;
        // once x is a local optimum only the shaken products were touched: wavefront 0, which shakes next, takes them
        // alone, and the others go on to wait for its shake
        const bool few = cs.lopt != 0;
        const int ntouch = few ? nd : K;
        for (int idx = few ? (wave == 0 ? lane : ntouch) : (int)threadIdx.x; idx < ntouch; idx += few ? 64 : (int)blockDim.x) {
            const int p = few ? sh.dp[idx] : idx;
            if (st_lds) {
                if (accepted) {
                    const Bits b = lds_load(l_work + p);
                    lds_store(l_cur + p, b);
                    lds_store(l_cur_cost + p, lds_load(l_work_cost + p));
                    if (bmode == 1) a.best[cp0 + p] = b;
                } else {
                    lds_store(l_work + p, lds_load(l_cur + p));
                    lds_store(l_work_cost + p, lds_load(l_cur_cost + p));
                }
            } else if (accepted) {
                g_cur[p] = g_work[p];
                g_cur_cost[p] = g_work_cost[p];
                if (bmode == 1) a.best[cp0 + p] = g_work[p];
            } else {
                g_work[p] = g_cur[p];
                g_work_cost[p] = g_cur_cost[p];
            }
        }
        if (a.trace && threadIdx.x == 0) {
            Record r;
            r.iter = (int32_t)it;
            r.k = kshake;
            r.accepted = accepted;
            r.winner = 0;
            r.F_shaken = cs.F + dshake;
            r.F_local = F_local;
            r.F_best = (accepted && F_local < cs.F_best) ? F_local : cs.F_best;
            a.trace[(int64_t)g * a.iters + i] = r;
        }
        if (bmode == 2) {
            __syncthreads();
            for (int q = threadIdx.x; q < K; q += blockDim.x) a.best[cp0 + q] = cur_bits(q);
        }
        if (accepted) {
            cs.F = F_local;
            cs.k = 1;
            cs.lopt = 1;
            cs.bsync = bmode ? 1 : 0;
        } else {
            cs.k = cs.k >= a.kmax ? 1 : cs.k + 1;
        }
        cs.F_best = cs.F < cs.F_best ? cs.F : cs.F_best;
        // (what the next iteration writes first, its shake, is read after the shake's barrier; its sums are written
        // after that one)
        if (few && bmode != 2) wave_sync_lds();
        else __syncthreads();
    }

    if constexpr (COOP) {
        CoopCtl *ctl = a.coop_ctl + g;
        if (slot == 0) {   // the leader: this launch's counters, and work == cur for the other search kernels
            __syncthreads();
            for (int q = threadIdx.x; q < K; q += blockDim.x) {
                a.work[cp0 + q] = a.cur[cp0 + q];
                a.work_cost[cp0 + q] = a.cur_cost[cp0 + q];
            }
            if (threadIdx.x == 0) {
                cs.evals = ctl->evals;
                cs.discarded = 0;
                cs.err |= ctl->err;
                cs.nb_evals = ctl->nb_evals;
                cs.fallbacks = ctl->fallbacks;
                a.cstate[g] = cs;
            }
        }
        // the last workgroup of the chain to leave records the move-evaluations computed and not consumed
        // (the iterations after an accepted one, finished or abandoned), and any error a slot raised
        if (threadIdx.x == 0) {
            __hip_atomic_fetch_add(&ctl->executed, executed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const int32_t n = __hip_atomic_fetch_add(&ctl->exited, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            if (n == a.coop_m - 1) {
                const int64_t ex = __hip_atomic_load(&ctl->executed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                a.cstate[g].discarded = ex - ctl->evals;
                a.cstate[g].err |= __hip_atomic_load(&ctl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        return;
    }
    __syncthreads();
    if (st_lds) {
        for (int i = threadIdx.x; i < K; i += blockDim.x) {
            g_cur[i] = l_cur[i];
            g_work[i] = l_work[i];
            g_cur_cost[i] = l_cur_cost[i];
            g_work_cost[i] = l_work_cost[i];
        }
    }
    if (lane == 0) {
        sh.ev[wave] = evals;
        sh.part[wave] = vnd_err;
        sh.shk[wave] = nb_evals;
        sh.fb[wave] = fallbacks;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t e = 0, ne = 0, nf = 0;
        int32_t err = 0;
        for (int w = 0; w < W; ++w) {
            e += sh.ev[w];
            err |= (int32_t)sh.part[w];
            ne += sh.shk[w];
            nf += sh.fb[w];
        }
        cs.evals = e;
        cs.err |= err;
        cs.nb_evals = ne;
        cs.fallbacks = nf;
        cs.discarded = 0;
        a.cstate[g] = cs;
    }
}

}  // namespace

template <int MODEL>
__global__ __launch_bounds__(512) void k_run(RunArgs a) {
    __shared__ RunShared sh;
    __shared__ SwapList lists[kRunWaves];
    __shared__ SpecShared sp;
    extern __shared__ __attribute__((aligned(16))) int2 s_rows[];
    run_chain<false, false, false, MODEL>(a, sh, lists, sp, s_rows);
}

// The same for batches with short horizons (up to kMultiMaxT): consecutive neighbourhoods priced side by side.
// Bounded to 128 registers: four wavefronts per SIMD for every decode reading.
template <int MODEL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void k_run_short(RunArgs a) {
    __shared__ RunShared sh;
    __shared__ SwapList lists[kRunWaves];
    __shared__ SpecShared sp;
    extern __shared__ __attribute__((aligned(16))) int2 s_rows[];
    run_chain<false, false, false, MODEL, false, true>(a, sh, lists, sp, s_rows);
}

// The plain search with interval pricing (contexts of compact products, no move log), one workgroup per chain and
// with speculative iterations or best-of-G.  IV: 1 when every horizon is at most 64, else 2.
//
// Bound by a lone wavefront's instruction issue and LDS waits along the chain of shake, one product's VND and acceptance
// (100 x 52, 64 chains side by side: 16% of the chip's VALU issue).  Full decodes -> interval pricing: 500 iterations of 10 x 12 4.66 -> 2.4 ms; 512 instances
// (K 10..200, T 12, 24 or 52) x 8 chains x 50 5.4 -> 1.17 ms; 64 instances (T 52 or 104) x 16 7.2 -> 0.83 ms; with
// speculative iterations 100 x 52, 64 chains x 200 1.46 -> 0.65 ms under the profiler; best of 4, 300 x 52 2.2 -> 0.87 ms.
// Four wavefronts per SIMD for one period a lane, three for two (2 registers spill, 14 under the strict reading; at four
// many more).
template <int IV, int MODEL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(IV == 2 ? 3 : 4))) void k_run_iv(RunArgs a) {
    __shared__ RunShared sh;
    __shared__ SwapList lists[kRunWaves];
    __shared__ SpecShared sp;
    extern __shared__ __attribute__((aligned(16))) int2 s_rows[];
    run_chain<false, false, false, MODEL, false, false, IV>(a, sh, lists, sp, s_rows);
}

template <int IV, int MODEL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(3))) void k_run_coop_iv(RunArgs a) {
    __shared__ RunShared sh;
    __shared__ SwapList lists[kRunWaves];
    __shared__ SpecShared sp;
    extern __shared__ __attribute__((aligned(16))) int2 s_rows[];
    run_chain<false, false, true, MODEL, false, false, IV>(a, sh, lists, sp, s_rows);
}

// The learned search with interval pricing: 50 iterations of 100 x 52, 64 chains, 8 side by side, 1.56 -> 0.53 ms.  Scores
// are computed only where a move improves (0.98 -> 0.53 ms of it); the weights' fragments hold it at two wavefronts per SIMD.
template <int IV, bool COOP>
__global__ __launch_bounds__(512) void k_run_learned_iv(RunArgs a) {
    __shared__ RunShared sh;
    __shared__ SwapList lists[kRunWaves];
    __shared__ SpecShared sp;
    extern __shared__ __attribute__((aligned(16))) int2 s_rows[];
    run_chain<false, true, COOP, 0, false, false, IV>(a, sh, lists, sp, s_rows);
}

__global__ __launch_bounds__(1024) void k_run_spec(RunArgs a) {
    __shared__ RunShared sh;
    __shared__ SwapList lists[kMaxWaves];
    __shared__ SpecShared sp;
    extern __shared__ __attribute__((aligned(16))) int2 s_rows[];
    run_chain<true, false>(a, sh, lists, sp, s_rows);
}

// speculative iterations: m workgroups per chain compute the next m iterations side by side (cooperative
// launch: every workgroup of a chain is resident while it waits for the others)
template <int MODEL>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(3))) void k_run_coop(RunArgs a) {
    __shared__ RunShared sh;
    __shared__ SwapList lists[kRunWaves];
    __shared__ SpecShared sp;
    extern __shared__ __attribute__((aligned(16))) int2 s_rows[];
    run_chain<false, false, true, MODEL>(a, sh, lists, sp, s_rows);
}

// learned VND: the scorer's weight fragments stay in registers for the whole launch
// speculative iterations of the learned search
__global__ __launch_bounds__(512) void k_run_learned_coop(RunArgs a) {
    __shared__ RunShared sh;
    __shared__ SwapList lists[kRunWaves];
    __shared__ SpecShared sp;
    extern __shared__ __attribute__((aligned(16))) int2 s_rows[];
    run_chain<false, true, true>(a, sh, lists, sp, s_rows);
}

__global__ __launch_bounds__(512) void k_run_learned(RunArgs a) {
    __shared__ RunShared sh;
    __shared__ SwapList lists[kRunWaves];
    __shared__ SpecShared sp;
    extern __shared__ __attribute__((aligned(16))) int2 s_rows[];
    run_chain<false, true>(a, sh, lists, sp, s_rows);
}

// the packed learned VND (batches of products per wavefront), alone and with speculative iterations
__global__ __launch_bounds__(512) void k_run_learned_packed(RunArgs a) {
    __shared__ RunShared sh;
    __shared__ SwapList lists[kRunWaves];
    __shared__ SpecShared sp;
    extern __shared__ __attribute__((aligned(16))) int2 s_rows[];
    run_chain<false, true, false, 0, true>(a, sh, lists, sp, s_rows);
}

__global__ __launch_bounds__(512) void k_run_learned_coop_packed(RunArgs a) {
    __shared__ RunShared sh;
    __shared__ SwapList lists[kRunWaves];
    __shared__ SpecShared sp;
    extern __shared__ __attribute__((aligned(16))) int2 s_rows[];
    run_chain<false, true, true, 0, true>(a, sh, lists, sp, s_rows);
}

// ---------------------------------------------------------------------------------------------------
// k_eval_learned: one wavefront per (chain, product) of a chain range: the learned choice of one
// neighbourhood's move for the current solution, with the scores and the selection of every move.
// ---------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_eval_learned(EvalLearnedArgs a, int64_t cp_begin) {
    __shared__ int2 s_row[kTMax];
    __shared__ uint16_t s_list[2 * kTMax];
    __shared__ uint16_t s_sel[2 * kTMax];
    __shared__ __attribute__((aligned(16))) __bf16 s_x[64 * 16];   // read as 16-byte vectors
    const int64_t cp = cp_begin + blockIdx.x;
    const int g = a.cp_chain[cp];
    const ChainInfo ci = a.chains[g];
    const int T = ci.T;
    const int p = (int)(cp - ci.cp0);
    const ProdParams pp = a.prod[ci.prod0 + p];
    for (int t = threadIdx.x; t < T; t += 64) s_row[t] = a.rows[pp.row + t];
    wave_sync_lds();
    mlp::Frags fr;
    mlp::load_frags(a.mlp, fr);
    const Bits b = a.cur[cp];
    int64_t cost = a.cur_cost[cp], evals = 0;
    int fb = 0;
    const int64_t off = a.slot_off[g] + (int64_t)p * 4 * T;
    LearnedLds L{s_x, s_sel};
    const uint64_t key = learned_best_move(b, s_row, T, pp, a.nb, s_list, L, fr, a.permille, false, cost, evals,
                                           fb, a.scores ? a.scores + off : nullptr, a.selected ? a.selected + off : nullptr);
    if (threadIdx.x == 0) {
        const int64_t F = a.cstate[g].F;
        a.prod_price[cp] = key == kInfKey ? kInf : F - cost + (int64_t)(key >> kSlotBits);
        a.prod_slot[cp] = key == kInfKey ? -1 : (int32_t)(key & 0xFFFFu);
        a.fallback[cp] = (uint8_t)fb;
        atomicAdd(a.evals + (size_t)(blockIdx.x & (kCounterSlots - 1)) * kCounterStride, (unsigned long long)evals);
    }
}

// k_run_done: the iteration counter moves on once every chain of the launch has read it, and the chains' counts are
// summed for the host (one workgroup: 16384 chains are 16 rounds of it).
__global__ __launch_bounds__(1024) void k_run_done(RunDoneArgs a) {
    int64_t v[5] = {0, 0, 0, 0, 0};
    int err = 0;
    for (int64_t g = threadIdx.x; g < a.n_chains; g += blockDim.x) {
        const ChainState cs = a.cstate[g];
        v[0] += cs.evals;
        v[1] += cs.evals * a.chains[g].T;
        v[2] += cs.discarded;
        v[3] += cs.nb_evals;
        v[4] += cs.fallbacks;
        err |= cs.err;
    }
    __shared__ int64_t s_v[5][16];
    __shared__ int s_err[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int e = (__any(err & 1) ? 1 : 0) | (__any(err & 2) ? 2 : 0);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int64_t n = wave_sum_i64(v[i]);
        if (lane == 0) s_v[i][wave] = n;
    }
    if (lane == 0) s_err[wave] = e;
    __syncthreads();
    if (threadIdx.x == 0) {
        RunTotals t{};
        for (int w = 0; w < 16; ++w) {
            t.evals += s_v[0][w];
            t.steps += s_v[1][w];
            t.discarded += s_v[2][w];
            t.nb_evals += s_v[3][w];
            t.fallbacks += s_v[4][w];
            t.err |= s_err[w];
        }
        *a.out = t;
        *a.it_counter += a.iters;
    }
}

__global__ __launch_bounds__(256) void k_rows_out(RowsOutArgs a) {
    const int64_t n = (int64_t)a.K * a.T;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int k = (int)(i / a.T), t = (int)(i - (int64_t)k * a.T);
        const Bits &b = a.x[k];
        a.zM[i] = (uint8_t)((b.m[t >> 5] >> (t & 31)) & 1u);
        a.zR[i] = (uint8_t)((b.r[t >> 5] >> (t & 31)) & 1u);
    }
}

__global__ __launch_bounds__(256) void k_costs_out(CostsOutArgs a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n) return;
    const ChainState &cs = a.cstate[i];
    a.F[i] = cs.F;
    a.F_best[i] = cs.F_best;
}

// ---------------------------------------------------------------------------------------------------
// Host-side launchers (called by the runtime).
// ---------------------------------------------------------------------------------------------------
// One instantiation per decode reading (kModelStrict | kModelDispose).
template <template <int> class Pick>
static const void *by_model(int model) {
    switch (model) {
        case 1: return Pick<1>::fn();
        case 2: return Pick<2>::fn();
        case 3: return Pick<3>::fn();
        default: return Pick<0>::fn();
    }
}
template <int M> struct PickInit { static const void *fn() { return reinterpret_cast<const void *>(&k_init_costs<M>); } };
template <int M> struct PickEval { static const void *fn() { return reinterpret_cast<const void *>(&k_eval<M>); } };
template <int M> struct PickEvalWide {
    static const void *fn() { return reinterpret_cast<const void *>(&k_eval_wide<M>); }
};
template <int M> struct PickRun { static const void *fn() { return reinterpret_cast<const void *>(&k_run<M>); } };
template <int M> struct PickRunShort {
    static const void *fn() { return reinterpret_cast<const void *>(&k_run_short<M>); }
};
template <int M> struct PickCoop { static const void *fn() { return reinterpret_cast<const void *>(&k_run_coop<M>); } };

hipError_t launch_init(const InitArgs &a, int n_chains, hipStream_t s, int model) {
    if (n_chains <= 0) return hipSuccess;
    InitArgs args = a;
    void *params[] = {&args};
    return hipLaunchKernel(by_model<PickInit>(model), dim3(n_chains), dim3(256), params, 0, s);
}

hipError_t launch_eval(const EvalArgs &a, const EvalWg *wg, int64_t n_wg, hipStream_t s, int model, int waves) {
    if (n_wg <= 0) return hipSuccess;
    if (waves != 4 && waves != 8 && waves != 12 && waves != 16) return hipErrorInvalidValue;
    EvalArgs args = a;
    const EvalWg *w = wg;
    void *params[] = {&args, &w};
    const void *fn = waves == 4 ? by_model<PickEval>(model) : by_model<PickEvalWide>(model);
    return hipLaunchKernel(fn, dim3((unsigned)n_wg), dim3(64 * waves), params, 0, s);
}

hipError_t launch_eval_iv(const EvalArgs &a, int64_t cp_begin, int64_t n_cp, int n_cu, bool long_T, bool count_steps,
                          hipStream_t s, int model) {
    if (n_cp <= 0) return hipSuccess;
    // about 16 wavefronts per SIMD's worth of ranges, at most 16 pairs each (a multiple of 4: short horizons are priced
    // four pairs at a time)
    int64_t per = n_cp / ((int64_t)n_cu * 64);
    per = per < 1 ? 1 : per > 16 ? 16 : per > 3 ? per & ~(int64_t)3 : per;
    const int32_t per_wave = (int32_t)per;
    const int64_t waves = (n_cp + per - 1) / per;
    const dim3 grid((unsigned)((waves + 3) / 4)), block(256);
    const bool strict = (model & kModelStrict) != 0;
#define VNS_IV(L, S, C) hipLaunchKernelGGL((k_eval_iv<L, S, C>), grid, block, 0, s, a, cp_begin, n_cp, per_wave)
    if (count_steps) {
        if (long_T) VNS_IV(true, false, true);
        else VNS_IV(false, false, true);
    } else if (strict) {
        if (long_T) VNS_IV(true, true, false);
        else VNS_IV(false, true, false);
    } else {
        if (long_T) VNS_IV(true, false, false);
        else VNS_IV(false, false, false);
    }
#undef VNS_IV
    return hipGetLastError();
}

hipError_t launch_eval_prep(const EvalPrepArgs &a, hipStream_t s) {
    const int64_t n = std::max<int64_t>(a.n_cp, counter_words());
    const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_eval_prep, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_eval_inc(const EvalArgs &a, const EvalWg *wg, int64_t n_wg, size_t lds_bytes, hipStream_t s) {
    if (n_wg <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_eval_inc, dim3((unsigned)n_wg), dim3(256), lds_bytes, s, a, wg);
    return hipGetLastError();
}

hipError_t launch_chain_best(const ChainBestArgs &a, hipStream_t s) {
    // more chains than the chip holds workgroups of four wavefronts at once: a wavefront per chain
    constexpr int kMany = 16;
    if (a.n_chains > 2048)
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_chain_best<kMany>), dim3((a.n_chains + kMany - 1) / kMany + 1), dim3(64 * kMany), 0, s, a);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_chain_best<1>), dim3(a.n_chains + 1), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_run_done(const RunDoneArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(k_run_done, dim3(1), dim3(1024), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_rows_out(const RowsOutArgs &a, hipStream_t s) {
    const int64_t n = (int64_t)a.K * a.T;
    hipLaunchKernelGGL(k_rows_out, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1024)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_costs_out(const CostsOutArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(k_costs_out, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_eval_learned(const EvalLearnedArgs &a, int64_t cp_begin, int64_t n_cp, hipStream_t s) {
    if (n_cp <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_eval_learned, dim3((unsigned)n_cp), dim3(64), 0, s, a, cp_begin);
    return hipGetLastError();
}

static const void *interval_kernel(bool coop, bool long_T, int model) {
#define VNS_IV(K)                                                                                                     \
    (long_T ? ((model & kModelStrict) ? reinterpret_cast<const void *>(&K<2, 1>) : reinterpret_cast<const void *>(&K<2, 0>)) \
            : ((model & kModelStrict) ? reinterpret_cast<const void *>(&K<1, 1>) : reinterpret_cast<const void *>(&K<1, 0>)))
    return coop ? VNS_IV(k_run_coop_iv) : VNS_IV(k_run_iv);
#undef VNS_IV
}

int64_t interval_wave_bytes(bool long_T) {
    return long_T ? (int64_t)sizeof(iv::Lds<64, 2>) : (int64_t)sizeof(iv::Lds<64, 1>);
}

static const void *run_kernel(RunKind kind, int model) {
    switch (kind) {
        case RunKind::kInterval: return interval_kernel(false, false, model);
        case RunKind::kIntervalLong: return interval_kernel(false, true, model);
        case RunKind::kLearnedInterval: return reinterpret_cast<const void *>(&k_run_learned_iv<1, false>);
        case RunKind::kLearnedIntervalLong: return reinterpret_cast<const void *>(&k_run_learned_iv<2, false>);
        case RunKind::kSpec: return reinterpret_cast<const void *>(&k_run_spec);
        case RunKind::kLearned: return reinterpret_cast<const void *>(&k_run_learned);
        case RunKind::kLearnedPacked: return reinterpret_cast<const void *>(&k_run_learned_packed);
        case RunKind::kPlainShort: return by_model<PickRunShort>(model);
        default: return by_model<PickRun>(model);
    }
}

hipError_t run_kernel_lds(RunKind kind, size_t *static_bytes, size_t dynamic_bytes, int model) {
    const void *fn = run_kernel(kind, model);
    hipFuncAttributes fa;
    hipError_t e = hipFuncGetAttributes(&fa, fn);
    if (e != hipSuccess) return e;
    *static_bytes = fa.sharedSizeBytes;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dynamic_bytes);
}

static const void *coop_kernel(RunKind kind, int model) {
    if (kind == RunKind::kLearned) return reinterpret_cast<const void *>(&k_run_learned_coop);
    if (kind == RunKind::kLearnedPacked) return reinterpret_cast<const void *>(&k_run_learned_coop_packed);
    if (kind == RunKind::kLearnedInterval) return reinterpret_cast<const void *>(&k_run_learned_iv<1, true>);
    if (kind == RunKind::kLearnedIntervalLong) return reinterpret_cast<const void *>(&k_run_learned_iv<2, true>);
    if (kind == RunKind::kInterval || kind == RunKind::kIntervalLong)
        return interval_kernel(true, kind == RunKind::kIntervalLong, model);
    return by_model<PickCoop>(model);
}

hipError_t coop_fits(int waves, size_t lds_bytes, int64_t blocks, bool *fits, RunKind kind, int model) {
    *fits = false;
    const void *fn = coop_kernel(kind, model);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return e;
    int per_cu = 0, dev = 0, cus = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 64 * waves, lds_bytes);
    if (e != hipSuccess) return e;
    e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    *fits = (int64_t)per_cu * cus >= blocks;
    return hipSuccess;
}

hipError_t launch_run_coop(const RunArgs &a, int n_chains, int waves, size_t lds_bytes, hipStream_t s, RunKind kind,
                           int model) {
    if (n_chains <= 0 || a.iters <= 0) return hipSuccess;
    RunArgs args = a;
    void *params[] = {&args};
    return hipLaunchCooperativeKernel(coop_kernel(kind, model), dim3((unsigned)(n_chains * a.coop_m)), dim3(64 * waves),
                                      params, (unsigned)lds_bytes, s);
}

hipError_t launch_run(const RunArgs &a, RunKind kind, int n_chains, int waves, size_t lds_bytes, hipStream_t s, int model) {
    if (n_chains <= 0 || a.iters <= 0) return hipSuccess;
    RunArgs args = a;
    void *params[] = {&args};
    return hipLaunchKernel(run_kernel(kind, model), dim3(n_chains), dim3(64 * waves), params, lds_bytes, s);
}

}  // namespace vns
