// Routing, cost-aware pruning, compensation and token permutation for one
// MoE layer call: token-parallel kernels, and for batches of up to 16 tokens
// one 1024-thread workgroup that runs every phase.
//
//   phase A (one wavefront per token): sigmoid scores, group-limited top-k
//            K_t and normalised gate weights G(t)_e (Sec. II-A);
//   phase B (whole workgroup): importance, mandatory/candidate split,
//            per-bin baseline cost F_base and cost-invariant expansion
//            (Sec. IV-A, IV-B steps 1-4);
//   phase C (one wavefront per token): masking of pruned experts and
//            top-k refill from A_trans (Sec. IV-C), weight renormalisation;
//   permute: stable counting sort of the (token, expert) pairs by expert,
//            the shared experts' rows first, and the FFN work lists (small
//            and big expert chunks).
//
// Every decision is taken in float64 with ties to the lower index, so the
// result does not depend on the order in which lanes or waves finish.
#include <math.h>

#include "caee_internal.h"
#include "fp8_codec.h"

namespace caee {
namespace {

#include "ffn_tile.h"

constexpr int kTokWaves = 4;                       // tokens (wavefronts) per workgroup
constexpr int kTokThreads = kTokWaves * kWave;
// Batches up to this many tokens are routed by one fused single-workgroup kernel.
#ifndef CAEE_FUSED_T
#define CAEE_FUSED_T 16
#endif
constexpr int kFusedT = CAEE_FUSED_T;
constexpr int kNoIdx = 0x7fffffff;

// Cross-lane moves within a 16-lane row through DPP (no LDS round trip).
template <int C>
__device__ inline int dpp_i(int v) {
    return __builtin_amdgcn_mov_dpp(v, C, 0xF, 0xF, false);
}
template <int C>
__device__ inline double dpp_d(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = dpp_i<C>((int)b);
    const int hi = dpp_i<C>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ inline double readlane_d(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// DPP controls that pair every lane of a row with another one:
// quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror, row_mirror.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;


// Row broadcasts of gfx9 DPP: lane 15 of each row to the next row, lane 31
// to rows 2 and 3.  Rows outside `RM` keep their own value (update_dpp's
// old operand), so a max or min with it changes nothing there.
constexpr int kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143;
template <int C, int RM>
__device__ inline int dpp_upd_i(int v) {
    return __builtin_amdgcn_update_dpp(v, v, C, RM, 0xF, false);
}
template <int C, int RM>
__device__ inline double dpp_upd_d(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = dpp_upd_i<C, RM>((int)b);
    const int hi = dpp_upd_i<C, RM>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Wave-wide max, all in VALU: butterfly inside each 16-lane row,
// then row 1 takes row 0's result and row 3 row 2's, then row 3 takes row
// 1's; lane 63 ends with the wave's result, which every lane reads.
__device__ inline double wave_max_d(double v) {
    v = fmax(v, dpp_d<kDppXor1>(v));
    v = fmax(v, dpp_d<kDppXor2>(v));
    v = fmax(v, dpp_d<kDppHalfMirror>(v));
    v = fmax(v, dpp_d<kDppMirror>(v));
    v = fmax(v, dpp_upd_d<kDppRowBcast15, 0xA>(v));
    v = fmax(v, dpp_upd_d<kDppRowBcast31, 0xC>(v));
    return readlane_d(v, 63);
}
// Inclusive prefix sum over the 64 lanes, in VALU: shifts by 1, 2, 4, 8
// within each row (lanes shifted in from outside the row read 0), then
// rows 1 and 3 add the last lane of rows 0 and 2, rows 2 and 3 that of row 1.
__device__ inline int wave_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowBcast15, 0xA, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, kDppRowBcast31, 0xC, 0xF, false);
    return v;
}

// The bits of a double as an unsigned integer in the same order (no NaN);
// 0 stands for "none" below every value.
__device__ inline unsigned long long sortable(double v) {
    const long long b = __double_as_longlong(v);
    return (unsigned long long)b ^ ((unsigned long long)(b >> 63) | 0x8000000000000000ull);
}

// Wave-wide max of unsigned words: the same moves as wave_max_d, each one
// instruction with its max.
template <int C, int RM>
__device__ inline unsigned dpp_max_u(unsigned v) {
    return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, C, RM, 0xF, false));
}
__device__ inline unsigned wave_max_u(unsigned v) {
    v = dpp_max_u<kDppXor1, 0xF>(v);
    v = dpp_max_u<kDppXor2, 0xF>(v);
    v = dpp_max_u<kDppHalfMirror, 0xF>(v);
    v = dpp_max_u<kDppMirror, 0xF>(v);
    v = dpp_max_u<kDppRowBcast15, 0xA>(v);
    v = dpp_max_u<kDppRowBcast31, 0xC>(v);
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// Lane holding the largest v, the lowest such lane on ties; -1 when every
// lane holds 0.  The high words decide unless they tie.  (Experts are spread
// over the lanes in index order, so the lowest lane holds the lowest index.
// With float64 max and an index min, 12 double-word moves a pick, a top-8
// selection took 2.2 us of a one-token call.)
__device__ inline int wave_argmax_lane(unsigned long long v) {
    const unsigned hi = (unsigned)(v >> 32), lo = (unsigned)v;
    const unsigned mh = wave_max_u(hi);
    if (mh == 0u) return -1;   // (0 in the high word is below every value's)
    unsigned long long m = __ballot(hi == mh);
    if (m & (m - 1ull)) {
        const unsigned ml = wave_max_u(hi == mh ? lo : 0u);
        m = __ballot(hi == mh && lo == ml);
    }
    return __ffsll((long long)m) - 1;
}

// Largest of the lane's open keys (0 if none) and which one it is.
template <int EPL>
__device__ inline unsigned long long lane_best(const unsigned long long (&key)[EPL], const bool (&open)[EPL],
                                               int& which) {
    unsigned long long v = 0ull;
    which = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        if (open[i] && key[i] > v) {
            v = key[i];
            which = i;
        }
    }
    return v;
}

// Argmax of (v, i) over the first 16 lanes: the largest v, and among the
// lanes holding it the lowest i.  Values are never NaN; lanes 0 to 15 get the
// result.
__device__ inline void row_argmax(double& v, int& i) {
    double m = v;
    m = fmax(m, dpp_d<kDppXor1>(m));
    m = fmax(m, dpp_d<kDppXor2>(m));
    m = fmax(m, dpp_d<kDppHalfMirror>(m));
    m = fmax(m, dpp_d<kDppMirror>(m));
    i = v == m ? i : kNoIdx;
    i = min(i, dpp_i<kDppXor1>(i));
    i = min(i, dpp_i<kDppXor2>(i));
    i = min(i, dpp_i<kDppHalfMirror>(i));
    i = min(i, dpp_i<kDppMirror>(i));
    v = m;
}

// Merge two (largest, second largest) pairs.
__device__ inline void top2_merge(double& t1, double& t2, double o1, double o2) {
    const double n1 = fmax(t1, o1);
    const double n2 = fmax(fmin(t1, o1), fmax(t2, o2));
    t1 = n1;
    t2 = n2;
}
template <int C>
__device__ inline void top2_step(double& t1, double& t2) {
    top2_merge(t1, t2, dpp_d<C>(t1), dpp_d<C>(t2));
}

// Lane `lane` holds experts lane*EPL .. lane*EPL+EPL-1.
template <int EPL>
__device__ inline void load_scores(const RouteParams& p, int t, int lane, double (&s)[EPL],
                                   double (&key)[EPL]) {
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const int e = lane * EPL + i;
        if (e < p.E) {
            const double z = (double)p.logits[(size_t)t * p.E + e];
            const double sv = 1.0 / (1.0 + exp(-z));
            s[i] = sv;
            key[i] = sv + (p.bias ? (double)p.bias[e] : 0.0);
        } else {
            s[i] = 0.0;
            key[i] = -INFINITY;
        }
    }
}

// Each lane's score s of expert `e` (its own, or 0 when `valid` is false),
// fetched from the lane that holds it: one shuffle per element slot, for all
// lanes at once.
template <int EPL>
__device__ inline double fetch_score(const double (&s)[EPL], int e, bool valid, int E) {
    const bool ok = valid && e >= 0 && e < E;
    const int src = ok ? e / EPL : 0;
    const int which = ok ? e % EPL : 0;
    double got = 0.0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const double c = __shfl(s[i], src);
        if (which == i) got = c;
    }
    return ok ? got : 0.0;
}

// Groups ranked in one pass (each lane reads every group's score) when
// there are at most this many; more groups take one wave argmax per pick.
constexpr int kRankGroups = 16;

// Phase A for token t: writes K_t (rank order), G(t) and the token's top expert.
template <int EPL>
__device__ void route_token(const RouteParams& p, int t, int lane, int* ids, double* gout,
                            int* top1, uint8_t* mflag) {
    double s[EPL], key[EPL];
    load_scores<EPL>(p, t, lane, s, key);
    const bool lane_valid = lane * EPL < p.E;

    // Group score: sum of the two largest keys of the group.
    double t1 = -INFINITY, t2 = -INFINITY;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        if (key[i] > t1) {
            t2 = t1;
            t1 = key[i];
        } else if (key[i] > t2) {
            t2 = key[i];
        }
    }
    // Reduce over the lpg lanes holding one group (aligned blocks of lpg lanes).
    if (p.lpg >= 2) top2_step<kDppXor1>(t1, t2);
    if (p.lpg >= 4) top2_step<kDppXor2>(t1, t2);
    if (p.lpg >= 8) top2_step<kDppHalfMirror>(t1, t2);
    if (p.lpg >= 16) top2_step<kDppMirror>(t1, t2);
    for (int off = 16; off < p.lpg; off <<= 1) top2_merge(t1, t2, __shfl_xor(t1, off), __shfl_xor(t2, off));
    const double gscore = p.gsize >= 2 ? t1 + t2 : t1;
    const int my_group = lane_valid ? (lane * EPL) / p.gsize : kNoIdx;

    bool gsel = false;
    if (p.n_group <= kRankGroups) {
        // The group's rank: groups with a larger score, or the same score and
        // a lower index, come first; the first topk_group are selected.
        int rank = 0;
        for (int g2 = 0; g2 < p.n_group; ++g2) {
            const double o = readlane_d(gscore, g2 * p.lpg);   // the group's first lane
            rank += (o > gscore) | ((o == gscore) & (g2 < my_group));
        }
        gsel = lane_valid && rank < p.topk_group;
    } else {
        const unsigned long long gk = lane_valid ? sortable(gscore) : 0ull;
        for (int r = 0; r < p.topk_group; ++r) {
            const int l = max(wave_argmax_lane(gsel ? 0ull : gk), 0);
            if (lane_valid && my_group == __builtin_amdgcn_readlane(my_group, l)) gsel = true;
        }
    }

    // Top-k keys of the selected groups; lane r keeps the r-th pick.
    bool open[EPL];
    unsigned long long ukey[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        open[i] = gsel;
        ukey[i] = sortable(key[i]);
    }
    int my_id = kNoIdx;
    double my_s = 0.0;
    for (int r = 0; r < p.k; ++r) {
        int which;
        // (k keys are always open; the max only guards against NaN inputs)
        const int l = max(wave_argmax_lane(lane_best<EPL>(ukey, open, which)), 0);
#pragma unroll
        for (int i = 0; i < EPL; ++i)
            if (lane == l && i == which) open[i] = false;
        const int ei = l * EPL + __builtin_amdgcn_readlane(which, l);
        if (lane == r) my_id = ei;
    }
    my_s = fetch_score<EPL>(s, my_id, lane < p.k, p.E);
    // G(t): each score over the token's k scores summed in rank order (the
    // same additions on every lane), one slot per lane.
    double total = 0.0;
    for (int r = 0; r < p.k; ++r) total += readlane_d(my_s, r);
    const bool mine = lane < p.k;
    const double g = my_s / total;
    double bg = mine ? g : -INFINITY;
    int best = mine ? my_id : kNoIdx;
    row_argmax(bg, best);   // the token's top expert by G, ties to the lower index (lanes < k hold the slots)
    // Pairs that are mandatory on their own: the threshold (MAX) or the
    // cumulative-ratio prefix (CIR), and with keep_top1 the token's top expert.
    uint32_t flags = (uint32_t)__ballot(
        mine && ((p.keep_top1 && my_id == best) || (p.rule == CAEE_IMPORTANCE_MAX && g >= p.tau)));
    if (mine) {
        ids[lane] = my_id;
        gout[lane] = g;
        if (p.sslot) p.sslot[(size_t)t * p.k + lane] = my_s;
    }
    if (lane == 0) *top1 = best;
    if (p.rule == CAEE_IMPORTANCE_CIR) {
        // Slots in gate order (score descending, lower expert first on ties):
        // each slot's lane counts the slots ahead of it; the prefix then
        // walks the positions in order, the same additions on every lane.
        int ahead = 0;
        for (int j = 0; j < p.k; ++j) {
            const double sj = readlane_d(my_s, j);
            const int ij = __builtin_amdgcn_readlane(my_id, j);
            ahead += (sj > my_s || (sj == my_s && ij < my_id)) ? 1 : 0;
        }
        auto lane_at = [&](int q) { return __ffsll((long long)__ballot(mine && ahead == q)) - 1; };
        double sum = 0.0;
        for (int q = 0; q < p.k; ++q) sum += readlane_d(my_s, lane_at(q));
        double cum = 0.0;
        for (int q = 0; q < p.k; ++q) {
            const int l = lane_at(q);
            cum += readlane_d(my_s, l);
            flags |= 1u << l;
            if (cum / sum >= p.tau) break;
        }
    }
    if (mine) mflag[lane] = (uint8_t)((flags >> lane) & 1u);
}

// SplitMix64 output for `state` (Steele, Lea and Flood 2014): golden-gamma
// increment, two xor-shift-multiply rounds, a final xor-shift.
__device__ inline uint64_t splitmix64(uint64_t state) {
    uint64_t z = state + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Phase C for token t: K_final = (K_t ∩ A_trans) refilled from A_trans \ K_t.
template <int EPL>
__device__ void compensate_token(const RouteParams& p, int t, int lane, const int* orig,
                                 const uint8_t* trans, int* n_refill, int* n_pad) {
    bool in_k[EPL], tr[EPL], out_f[EPL];
    // K_t: lane r < k holds its r-th expert; the list is broadcast lane by lane.
    const int my_orig = lane < p.k ? orig[lane] : -1;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        in_k[i] = false;
        tr[i] = lane * EPL + i < p.E && trans[lane * EPL + i];
        out_f[i] = false;
    }
    for (int r = 0; r < p.k; ++r) {
        const int o = __builtin_amdgcn_readlane(my_orig, r);
#pragma unroll
        for (int i = 0; i < EPL; ++i) in_k[i] |= (o == lane * EPL + i);
    }
    const bool kept = my_orig >= 0 && trans[my_orig];
    const uint64_t kept_mask = __ballot(kept);
    const int n_keep = __popcll(kept_mask);
    int avail = 0;   // experts of A_trans outside K_t
#pragma unroll
    for (int i = 0; i < EPL; ++i) avail += __popcll(__ballot(tr[i] && !in_k[i]));
    if (p.refill != CAEE_REFILL_LITERAL && (p.refill == CAEE_REFILL_NONE || n_keep == p.k || avail == 0)) {
        // Nothing to refill: K_final = K_t ∩ A_trans in K_t's own (rank)
        // order.  Each kept slot's score is recomputed by its lane with the
        // same expression as the full pass, and summed in the same order.
        double my_s = 0.0;
        if (kept)
            my_s = p.sslot ? p.sslot[(size_t)t * p.k + lane]
                           : 1.0 / (1.0 + exp(-(double)p.logits[(size_t)t * p.E + my_orig]));
        double total = 0.0;
        for (int r = 0; r < p.k; ++r)
            if ((kept_mask >> r) & 1ull) total += readlane_d(my_s, r);
        const int pos = __popcll(kept_mask & ((1ull << lane) - 1ull));
        if (kept) {
            const size_t o = (size_t)t * p.k + pos;
            p.topk_ids[o] = my_orig;
            p.topk_w[o] = (float)(p.rs * (my_s / total));
        }
        if (lane >= n_keep && lane < p.k) {
            const size_t o = (size_t)t * p.k + lane;
            p.topk_ids[o] = -1;
            p.topk_w[o] = 0.0f;
        }
        if (lane == 0 && n_keep < p.k) atomicAdd(n_pad, p.k - n_keep);
        return;
    }
    double s[EPL], key[EPL];
    load_scores<EPL>(p, t, lane, s, key);

    // Refill order: router key (the paper's compensation) or, for the
    // ablation, a 53-bit random key (exact in a double) per (token, expert).
    // LITERAL: K_final is the top-k of all of A_trans by key, whether in K_t
    // or not.
    const bool literal = p.refill == CAEE_REFILL_LITERAL;
    unsigned long long rv[EPL];
    bool open[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const uint64_t ctr = ((uint64_t)p.seed << 32) | (uint64_t)(t * p.E + lane * EPL + i);
        rv[i] = sortable(p.refill == CAEE_REFILL_RANDOM ? (double)(splitmix64(ctr) >> 11) : key[i]);
        open[i] = tr[i] && (literal || !in_k[i]);
    }
    // The kept experts of K_t in lanes 0 .. n_keep - 1 (rank order), then the
    // picks, one lane each.
    int my_id = -1, got = 0;
    if (!literal) {
        const int from = __popcll(kept_mask & ((1ull << lane) - 1ull));   // this lane's place if kept
        for (int r = 0; r < n_keep; ++r) {
            const int src = __ffsll((long long)__ballot(kept && from == r)) - 1;
            const int o = __builtin_amdgcn_readlane(my_orig, src);
            if (lane == r) my_id = o;
        }
    }
    const int first = literal ? 0 : n_keep;
    const int to_fill = p.refill == CAEE_REFILL_NONE ? 0 : p.k - first;
    for (int r = 0; r < to_fill; ++r) {
        int which;
        const int l = wave_argmax_lane(lane_best<EPL>(rv, open, which));
        if (l < 0) break;
#pragma unroll
        for (int i = 0; i < EPL; ++i)
            if (lane == l && i == which) {
                open[i] = false;
                out_f[i] = true;
            }
        const int ei = l * EPL + __builtin_amdgcn_readlane(which, l);
        if (lane == first + r) my_id = ei;
        ++got;
    }
    const int m = first + got;
    // Rank order of K_final (key descending, lower index first): each slot's
    // lane counts the slots ahead of it.  (LITERAL picked in that order.)
    if (!literal && got > 0) {
        const double my_key = fetch_score<EPL>(key, my_id, lane < m, p.E);
        int ahead = 0;
        for (int j = 0; j < m; ++j) {
            const double kj = readlane_d(my_key, j);
            const int ij = __builtin_amdgcn_readlane(my_id, j);
            ahead += (kj > my_key || (kj == my_key && ij < my_id)) ? 1 : 0;
        }
        int id = -1;
        for (int j = 0; j < m; ++j) {
            const int src = __ffsll((long long)__ballot(lane < m && ahead == j)) - 1;
            const int o = __builtin_amdgcn_readlane(my_id, src);
            if (lane == j) id = o;
        }
        my_id = id;
    }
    double my_s = 0.0;
    my_s = fetch_score<EPL>(s, my_id, lane < m, p.E);
    if (literal) {   // slots that hold an expert from outside K_t
        got = 0;
#pragma unroll
        for (int i = 0; i < EPL; ++i) got += __popcll(__ballot(out_f[i] && !in_k[i]));
    }
    // Weights: scores over their sum in rank order (the same additions on
    // every lane), one slot per lane; slots past m are padding.
    double total = 0.0;
    for (int r = 0; r < m; ++r) total += readlane_d(my_s, r);
    if (lane < p.k) {
        const size_t o = (size_t)t * p.k + lane;
        const bool have = lane < m;
        p.topk_ids[o] = have ? my_id : -1;
        p.topk_w[o] = have ? (float)(p.rs * (my_s / total)) : 0.0f;
    }
    if (lane == 0) {
        atomicAdd(n_refill, got);
        atomicAdd(n_pad, p.k - m);
    }
}

// Routing kernel: one wavefront per token (phase A).
template <int EPL>
__global__ __launch_bounds__(kTokThreads) void k_route_tokens(RouteParams p) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int t = blockIdx.x * kTokWaves + wave;
    if (t < p.T)
        route_token<EPL>(p, t, lane, p.orig_ids + (size_t)t * p.k, p.gbuf + (size_t)t * p.k, p.top1 + t,
                         p.mflag + (size_t)t * p.k);
}

// What pruning needs to know of each routed expert, one workgroup per expert
// over all tokens: whether any token chose it, whether one of its pairs is
// mandatory on its own, and its importance -- the largest gate weight (MAX,
// CIR), or the gate weights added in ascending token order (SUM).
//
// Bound by latency: each wave reads its quarter of a tile of tokens, kStatBlk
// 64-token blocks of K_t at a time (all their loads in flight together), and
// leaves the gate weights of its hits in LDS in token order; then the SUM
// rule's one chain of additions runs over LDS (about 9 cycles an addition).
// A popular expert of a 4096-token batch has thousands of hits, so that chain
// is what is left: 4096 skewed tokens, SUM: 30 us (one wave per
// expert reading block after block, readlane per hit: 258 us).
constexpr int kStatWaves = 4, kStatBlk = 4;
constexpr int kStatTile = 4096;                       // tokens per tile
constexpr int kStatWaveTok = kStatTile / kStatWaves;  // a wave's part of it
constexpr int kStatAct = 1, kStatMust = 2;            // flags left in p.trans

// Whether a batch above kFusedT tokens takes its statistics from this kernel.
// SUM: always (nothing else computes the sums).  MAX and CIR: k_prune gathers
// them itself from the pairs, in time by the pairs; this kernel takes time by
// the tokens, in whole tiles, whatever k is.  So it pays for long lists from
// 33000 pairs on, for k = 8 where the tokens fill their tiles or are many, and
// never for k <= 4 or rows that are not 16-byte aligned.  caee_route_prune, MAX, N(0,1)
// logits, pairs / this kernel:
//   k = 16, E = 256: T = 1500 29.9 / 32.3 us, 2000 equal, 2500 38.2 / 35.9,
//                    4096 50.7 / 40.8, 65536 593 / 392;
//   k = 12, E = 256: T = 2000 27.8 / 29.7, 2800 33.7 / 32.4, 8192 70.7 / 57.1;
//   k = 8, E = 256:  T = 2048 23.2 / 27.3, 4096 33.4 / 31.8, 6000 43.5 / 44.8,
//                    8192 53.9 / 50.1, 9001 58.6 / 59.5, 22000 124 / 116;
//         E = 64:    T = 9001 46.4 / 52.1, 12288 59.2 / 56.7, 32768 141 / 135;
//   k = 6, E = 64:   T = 6000 29.3 / 52.3, 65536 215 / 364;
//   k = 4, E = 256:  T = 8192 36.7 / 41.9;  k = 2, E = 64: T = 65536 110 / 250.
inline bool takes_pair_stats(const RouteParams& p) {
    if (p.rule == CAEE_IMPORTANCE_SUM) return true;
    if (p.k % 4 != 0 || p.k < 8) return false;
    if (p.k > 8) return (long long)p.T * p.k >= 33000;
    const int last = p.T % kStatTile;   // k = 8: four tiles, or the last one at least 15/16 full
    return p.T >= 4 * kStatTile || (p.T >= kStatTile && (last == 0 || last >= kStatTile / 16 * 15));
}

__global__ __launch_bounds__(kStatWaves * kWave) void k_expert_stats(RouteParams p) {
    __shared__ __align__(16) double s_g[kStatWaves][kStatWaveTok + 16];   // read up to 16 past the end
    __shared__ int s_n[kStatWaves];
    __shared__ double s_max[kStatWaves];
    __shared__ int s_must[kStatWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int e = blockIdx.x, k = p.k;
    const bool sum_rule = p.rule == CAEE_IMPORTANCE_SUM;
    double gmax = 0.0, sum = 0.0;
    bool any = false, must = false;
    for (int base = 0; base < p.T; base += kStatTile) {
        const int t0 = base + wave * kStatWaveTok;
        const int t1 = min(p.T, t0 + kStatWaveTok);
        int n = 0;
        for (int tb = t0; tb < t1; tb += kStatBlk * kWave) {
            int slot[kStatBlk];
#pragma unroll
            for (int u = 0; u < kStatBlk; ++u) slot[u] = -1;
            if (k % 4 == 0) {   // rows of K_t are 16-byte aligned
                int4 v[kStatBlk][kMaxK / 4];
#pragma unroll
                for (int u = 0; u < kStatBlk; ++u) {
                    const int t = tb + u * kWave + lane;
#pragma unroll
                    for (int q = 0; q < kMaxK / 4; ++q)
                        v[u][q] = 4 * q < k && t < t1 ? *(const int4*)(p.orig_ids + (size_t)t * k + 4 * q)
                                                      : make_int4(-1, -1, -1, -1);
                }
#pragma unroll
                for (int u = 0; u < kStatBlk; ++u)
#pragma unroll
                    for (int q = 0; q < kMaxK / 4; ++q) {
                        if (v[u][q].x == e) slot[u] = 4 * q;
                        if (v[u][q].y == e) slot[u] = 4 * q + 1;
                        if (v[u][q].z == e) slot[u] = 4 * q + 2;
                        if (v[u][q].w == e) slot[u] = 4 * q + 3;
                    }
            } else {
                for (int r = 0; r < k; ++r) {
#pragma unroll
                    for (int u = 0; u < kStatBlk; ++u) {
                        const int t = tb + u * kWave + lane;
                        if (t < t1 && p.orig_ids[(size_t)t * k + r] == e) slot[u] = r;
                    }
                }
            }
            double g[kStatBlk];
            bool mf[kStatBlk];
#pragma unroll
            for (int u = 0; u < kStatBlk; ++u) {
                const size_t i = (size_t)(tb + u * kWave + lane) * k + (slot[u] < 0 ? 0 : slot[u]);
                g[u] = slot[u] >= 0 ? p.gbuf[i] : 0.0;
                mf[u] = slot[u] >= 0 && p.mflag[i];
            }
#pragma unroll
            for (int u = 0; u < kStatBlk; ++u) {
                const unsigned long long m = __ballot(slot[u] >= 0);
                gmax = fmax(gmax, g[u]);
                must |= mf[u];
                any |= m != 0ull;
                if (sum_rule && slot[u] >= 0) s_g[wave][n + __popcll(m & ((1ull << lane) - 1ull))] = g[u];
                n += __popcll(m);
            }
        }
        if (sum_rule) {
            if (lane == 0) s_n[wave] = n;
            __syncthreads();
            if (wave == 0) {   // the same additions on every lane
                for (int w = 0; w < kStatWaves; ++w) {
                    const double* sg = s_g[w];
                    const int m = s_n[w];
                    // Sixteen values ahead of the additions, read without
                    // conditions (what lies past the last is not added).
                    constexpr int kU = 16;
                    double cur[kU], nxt[kU];
#pragma unroll
                    for (int i = 0; i < kU; ++i) cur[i] = sg[i];
                    int j = 0;
                    for (; j + kU <= m; j += kU) {
#pragma unroll
                        for (int i = 0; i < kU; ++i) nxt[i] = sg[j + kU + i];
#pragma unroll
                        for (int i = 0; i < kU; ++i) sum += cur[i];
#pragma unroll
                        for (int i = 0; i < kU; ++i) cur[i] = nxt[i];
                    }
#pragma unroll
                    for (int i = 0; i < kU; ++i)
                        if (j + i < m) sum += cur[i];
                }
            }
            __syncthreads();
        }
    }
    gmax = wave_max_d(gmax);
    const bool wave_must = __ballot(must) != 0ull;
    if (lane == 0) {
        s_max[wave] = gmax;
        s_must[wave] = (any ? kStatAct : 0) | (wave_must ? kStatMust : 0);
    }
    __syncthreads();
    if (tid == 0) {
        double m = 0.0;
        int f = 0;
        for (int w = 0; w < kStatWaves; ++w) {
            m = fmax(m, s_max[w]);
            f |= s_must[w];
        }
        p.imp_sum[e] = sum_rule ? sum : m;
        p.trans[e] = (uint8_t)f;
    }
}

// The SUM rule's sums for small batches, one thread per expert walking the
// (token, slot) pairs in order (reads of one LDS word by every thread).
__device__ void importance_sum_small(const RouteParams& p, int tid, int nthr) {
    const int n = p.T * p.k;
    for (int e = tid; e < p.E; e += nthr) {
        // Pairs of other experts add zero, which changes no sum: the reads need
        // not wait for a comparison (with a branch per pair 4 us at 64 pairs).
        double sum = 0.0;
        int i = 0;
        constexpr int kU = 8;
        for (; i + kU <= n; i += kU) {
            double g[kU];
            int id[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                id[u] = p.orig_ids[i + u];
                g[u] = p.gbuf[i + u];
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) sum += id[u] == e ? g[u] : 0.0;
        }
        for (; i < n; ++i) sum += p.orig_ids[i] == e ? p.gbuf[i] : 0.0;
        p.imp_sum[e] = sum;
    }
}

// Pruning kernel (one workgroup): Sec. IV-B steps 1-4 over the whole batch.
// Bin loads are float64 sums of fp32 costs; while a bin's nonzero costs span
// less than 2^20 every such sum is exact, so the order of the additions (LDS
// atomics here) does not change any value or decision.
struct PruneShared {
    unsigned long long imp[kMaxE];
    uint8_t act[kMaxE], must[kMaxE], prom[kMaxE];
    float cost[kMaxE];
    int bin[kMaxE];
    int cand[kMaxE];        // candidates as gathered
    unsigned long long cimp[kMaxE];   // their importance bits
    int sorted[kMaxE];      // candidates in visiting order
    int cbin[kMaxE];        // their bins
    float ccost[kMaxE];     // their costs
    double aload[kMaxBins], mload[kMaxBins];
    double fbase;
    int ncand;
    int stat[5];            // step-4 counts: active, mandatory, promoted, pruned, kept
    int fallback;           // A_trans came out empty: steps 2-3 rerun with each token's top expert mandatory
};

// Steps 2-3 of Sec. IV-B from the membership in sh.act / sh.must: per-bin
// loads of A_act and A_must, F_base, the candidates (active, not mandatory)
// in visiting order (importance descending, index ascending), and the
// cost-invariant expansion into sh.prom, one bin per wave.  Expects sh.prom,
// the loads and the candidate count zeroed; ends with a barrier unless there
// are no candidates.
__device__ void prune_expand(const RouteParams& p, int tid, int nthr, PruneShared& sh) {
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int E = p.E, nb = p.n_bins;
    for (int e0 = wave * kWave; e0 < E; e0 += nthr) {
        const int e = e0 + lane;
        const bool act = e < E && sh.act[e], must = e < E && sh.must[e];
        if (act || must) {
            const double c = (double)sh.cost[e];
            const int b = sh.bin[e];
            if (act && b >= 0) atomicAdd(&sh.aload[b], c);
            if (must && b >= 0) atomicAdd(&sh.mload[b], c);
        }
        // One count per wave; the candidates' order here does not matter.
        const unsigned long long m = __ballot(act && !must);
        int at = 0;
        if (lane == 0 && m) at = atomicAdd(&sh.ncand, __popcll(m));
        at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1ull));
        if (act && !must) {
            sh.cand[at] = e;
            sh.cimp[at] = sh.imp[e];
        }
    }
    __syncthreads();
    const int n_cand = sh.ncand;
    if (n_cand == 0) {   // nothing to expand (uniform): A_trans = A_must
        for (int b = tid; b < nb && p.bin_loads; b += nthr) {
            p.bin_loads[b] = sh.aload[b];
            p.bin_loads[nb + b] = p.bin_loads[2 * nb + b] = sh.mload[b];
        }
        return;
    }
    // Each candidate's rank, counted by kRankLanes neighbouring lanes (one
    // thread per candidate over 124 of them: 5 us).
    constexpr int kRankLanes = 8;
    for (int i0 = tid / kRankLanes; i0 - lane / kRankLanes < n_cand; i0 += nthr / kRankLanes) {
        const int i = min(i0, n_cand - 1);   // whole waves take part in the moves below
        const int e = sh.cand[i];
        const unsigned long long ie = sh.cimp[i];
        int rank = 0;
        for (int j = lane % kRankLanes; j < n_cand; j += kRankLanes) {
            const unsigned long long io = sh.cimp[j];
            const int o = sh.cand[j];
            rank += (io > ie || (io == ie && o < e)) ? 1 : 0;
        }
        rank += dpp_i<kDppXor1>(rank);
        rank += dpp_i<kDppXor2>(rank);
        rank += dpp_i<kDppHalfMirror>(rank);
        if (lane % kRankLanes == 0 && i0 < n_cand) {
            sh.sorted[rank] = e;
            sh.cbin[rank] = sh.bin[e];
            sh.ccost[rank] = sh.cost[e];
        }
    }
    __syncthreads();
    if (wave == 0) {
        double fb = 0.0;
        for (int b = lane; b < nb; b += kWave) fb = fmax(fb, sh.mload[b]);
        fb = wave_max_d(fb);
        if (lane == 0) sh.fbase = fb;
    }
    for (int b = tid; b < nb && p.bin_loads; b += nthr) {
        p.bin_loads[b] = sh.aload[b];
        p.bin_loads[nb + b] = sh.mload[b];
    }
    __syncthreads();

    // Step 3: expansion, walking the candidates in visiting order: one wave
    // per bin (bins are independent), a 64-candidate block at a time, its
    // lanes holding them (one thread per bin walking every candidate through
    // LDS took 5 us for 124 candidates).
    const double fbase = sh.fbase;
    for (int b = wave; b < nb; b += nthr / kWave) {
        double load = sh.mload[b];
        for (int r0 = 0; r0 < n_cand; r0 += kWave) {
            const int r = r0 + lane;
            const bool in = r < n_cand && sh.cbin[r] == b;
            const double c = in ? (double)sh.ccost[r] : 0.0;
            unsigned long long todo = __ballot(in), taken = 0ull;
            while (todo) {
                const int l = __ffsll((long long)todo) - 1;
                const double cl = readlane_d(c, l);
                if (load + cl <= fbase) {
                    taken |= 1ull << l;
                    load += cl;
                }
                todo &= todo - 1ull;
            }
            if ((taken >> lane) & 1ull) sh.prom[sh.sorted[r]] = 1;
        }
        if (p.bin_loads && lane == 0) p.bin_loads[2 * nb + b] = load;
    }
    __syncthreads();
}

// Run by one workgroup of `nthr` threads (a multiple of the wave size).
__device__ void prune_all(const RouteParams& p, int tid, int nthr, PruneShared& sh) {
    unsigned long long* s_imp = sh.imp;
    uint8_t *s_act = sh.act, *s_must = sh.must, *s_prom = sh.prom;
    float* s_cost = sh.cost;
    int* s_bin = sh.bin;
    double *s_aload = sh.aload, *s_mload = sh.mload;
    int& s_ncand = sh.ncand;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int T = p.T, E = p.E, k = p.k, nb = p.n_bins;

    for (int e = tid; e < E; e += nthr) {
        const int f = p.pair_stats ? p.trans[e] : 0;
        s_imp[e] = p.pair_stats ? (unsigned long long)__double_as_longlong(p.imp_sum[e]) : 0ull;
        s_act[e] = (f & kStatAct) != 0;
        s_must[e] = (f & kStatMust) != 0;
        s_prom[e] = 0;
        s_cost[e] = p.cost[e];
        const int b = p.bin ? p.bin[e] : 0;
        s_bin[e] = (b >= 0 && b < nb) ? b : -1;   // out-of-range bins (a precondition violation) count nowhere
    }
    for (int b = tid; b < nb; b += nthr) s_aload[b] = s_mload[b] = 0.0;
    if (tid == 0) {
        s_ncand = 0;
        sh.fallback = 0;
    }
    if (tid < 5) sh.stat[tid] = 0;
    __syncthreads();

    // Step 1: A_act, importance, A_must (pairs mandatory on their own, and
    // for the SUM rule every expert whose summed weight reaches tau): from
    // k_expert_stats, or from the pairs here, in batches of 8 per thread,
    // whose loads are issued together.
    constexpr int kB = 8;
    const int pairs = p.pair_stats ? 0 : T * k;
    for (int i0 = tid; i0 < pairs; i0 += kB * nthr) {
        int ev[kB];
        double gv[kB];
        uint8_t mv[kB];
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            const int i = i0 + b * nthr;
            const bool in = i < T * k;
            ev[b] = in ? p.orig_ids[i] : -1;
            gv[b] = in ? p.gbuf[i] : 0.0;
            mv[b] = in ? p.mflag[i] : 0;
        }
#pragma unroll
        for (int b = 0; b < kB; ++b) {
            if (ev[b] < 0) continue;
            atomicMax(&s_imp[ev[b]], (unsigned long long)__double_as_longlong(gv[b]));
            s_act[ev[b]] = 1;
            if (mv[b]) s_must[ev[b]] = 1;
        }
    }
    __syncthreads();
    if (p.rule == CAEE_IMPORTANCE_SUM) {
        for (int e = tid; e < E; e += nthr) {
            if (!s_act[e]) continue;
            const double I = p.imp_sum[e];
            s_imp[e] = (unsigned long long)__double_as_longlong(I);
            if (I >= p.tau) s_must[e] = 1;
        }
        __syncthreads();
    }

    prune_expand(p, tid, nthr, sh);
    // A_trans = A_must + promoted is empty only when no thread sees a member.
    // Then Sec. IV-C's final top-k would have nothing to choose from: steps
    // 2-3 run again with every token's own top expert mandatory (the only
    // departure from step 1 as written).
    // (Without candidates A_must is A_act, which no batch leaves empty.)
    bool member = s_ncand == 0;
    for (int e = tid; e < E; e += nthr) member |= (s_must[e] | s_prom[e]) != 0;
    if (s_ncand > 0 && !__syncthreads_or(member)) {   // (nothing was promoted either: s_prom stays zero)
        for (int t = tid; t < T; t += nthr) s_must[p.top1[t]] = 1;
        for (int b = tid; b < nb; b += nthr) s_aload[b] = s_mload[b] = 0.0;
        if (tid == 0) {
            s_ncand = 0;
            sh.fallback = 1;
        }
        __syncthreads();
        prune_expand(p, tid, nthr, sh);
    }
    const int n_cand = s_ncand;

    // Step 4: A_trans = A_must + promoted; masks and counters by ballot,
    // one 64-expert block per wave, counts added in LDS.
    for (int e = tid; e < E; e += nthr) {
        p.trans[e] = s_must[e] | s_prom[e];
        if (p.trans_host) p.trans_host[e] = s_must[e] | s_prom[e];
    }
    const int words = (E + 31) / 32;
    for (int base = wave * kWave; base < E; base += nthr) {
        const int e = base + lane;
        const bool v = e < E;
        const bool act = v && s_act[e], must = v && s_must[e], prom = v && s_prom[e];
        const bool trans = must || prom;
        const unsigned long long ba = __ballot(act), bm = __ballot(must), bt = __ballot(trans),
                                 bp = __ballot(act && !trans), bpr = __ballot(prom);
        if (lane == 0) {
            atomicAdd(&sh.stat[0], __popcll(ba));
            atomicAdd(&sh.stat[1], __popcll(bm));
            atomicAdd(&sh.stat[2], __popcll(bpr));
            atomicAdd(&sh.stat[3], __popcll(bp));
            atomicAdd(&sh.stat[4], __popcll(bt));
        }
        if (p.masks && lane < 2) {
            const int w = base / 32 + lane;
            if (w < words) {
                const int sh_ = 32 * lane;
                p.masks[w] = (uint32_t)(ba >> sh_);
                p.masks[words + w] = (uint32_t)(bm >> sh_);
                p.masks[2 * words + w] = (uint32_t)(bt >> sh_);
                p.masks[3 * words + w] = (uint32_t)(bp >> sh_);
            }
        }
    }
    __syncthreads();
    if (tid < 2) p.counts[tid] = 0;   // compensation adds to these
    if (p.stats && tid == 0) {
        p.stats[0] = sh.stat[0];   // |A_act|
        p.stats[1] = sh.stat[1];   // |A_must|
        p.stats[2] = n_cand;
        p.stats[3] = sh.stat[2];   // promoted
        p.stats[4] = sh.stat[3];   // pruned
        p.stats[5] = sh.stat[4];   // |A_trans|
        p.stats[8] = sh.fallback;
    }
}

__global__ __launch_bounds__(kRouteThreads) void k_prune(RouteParams p) {
    __shared__ PruneShared sh;
    prune_all(p, threadIdx.x, kRouteThreads, sh);
}

// Row offsets of every expert slot and the FFN work lists, from the slot
// row counts in s_cnt (run by one wavefront).  Slot x (x < E routed, E+s
// shared) owns rows [off[x], off[x] + count); the shared slots come first
// (shared expert s owns rows s*T .. s*T + T - 1, known before routing), then
// the routed ones in expert order.  Then one small chunk per slot with at
// most chunk_small rows, and ceil(rows / chunk_big) near-equal big chunks per
// larger slot, the small chunks listed first.  s_work collects the big
// chunks' work (16-token tiles, and two for what an item costs at any width)
// by list position modulo 8; publish_balance, after a barrier, tells the FFN
// whether those shares are within 5 % of even.
__device__ void build_lists(const RouteParams& p, const int* s_cnt, int* s_off, int* s_work, int tid) {
    // Run by the first four waves of the workgroup (every thread calls it:
    // it holds a barrier).  Lane gl of the 256 takes slots [gl*per, gl*per+per)
    // in row order, so the scans below follow the slots' row order.
    constexpr int kW = 4;
    __shared__ int s_tot[kW][3];
    const int nx = p.E + p.n_shared, ns = p.n_shared, E = p.E;
    const int cs = p.chunk_small, cb = p.chunk_big;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const bool active = wave < kW;   // uniform per wave
    if (tid < kXcds) s_work[tid] = 0;
    const int per = (nx + kW * kWave - 1) / (kW * kWave);
    const int gl = wave * kWave + lane;
    const int lo = gl * per;
    const int hi = min(lo + per, nx);
    auto slot_at = [&](int j) { return j < ns ? E + j : j - ns; };   // j-th slot in row order
    int sum = 0, ssum = 0, bsum = 0, inc = 0, sinc = 0, binc = 0;
    if (active) {
        for (int j = lo; j < hi; ++j) {
            const int n = s_cnt[slot_at(j)];
            sum += n;
            ssum += (n > 0 && n <= cs) ? 1 : 0;
            bsum += n > cs ? (n + cb - 1) / cb : 0;
        }
        inc = wave_incl_scan(sum);
        sinc = wave_incl_scan(ssum);
        binc = wave_incl_scan(bsum);
        if (lane == kWave - 1) {
            s_tot[wave][0] = inc;
            s_tot[wave][1] = sinc;
            s_tot[wave][2] = binc;
        }
    }
    __syncthreads();
    if (!active) return;
    int base = 0, sbase = 0, bbase = 0, total = 0, stotal = 0, btotal = 0;
    for (int w = 0; w < kW; ++w) {
        if (w < wave) {
            base += s_tot[w][0];
            sbase += s_tot[w][1];
            bbase += s_tot[w][2];
        }
        total += s_tot[w][0];
        stotal += s_tot[w][1];
        btotal += s_tot[w][2];
    }
    int run = base + inc - sum, srun = sbase + sinc - ssum, brun = stotal + bbase + binc - bsum;
    for (int j = lo; j < hi; ++j) {
        const int x = slot_at(j);
        const int cnt = s_cnt[x];
        s_off[x] = run;
        p.perm_off[x] = run;
        if (cnt > 0 && cnt <= cs) {
            int* chk = p.chunks + 4 * srun++;
            chk[0] = x;
            chk[1] = run;
            chk[2] = cnt;
            chk[3] = 0;
        } else if (cnt > cs) {
            const int pieces = (cnt + cb - 1) / cb;
            const int size = (cnt + pieces - 1) / pieces;
            for (int c = 0; c < pieces; ++c) {
                int* chk = p.chunks + 4 * (brun + c);
                chk[0] = x;
                chk[1] = run + c * size;
                chk[2] = min(size, cnt - c * size);
                chk[3] = pieces > 1;
                atomicAdd(&s_work[(brun + c - stotal) % kXcds], (chk[2] + 15) / 16 + 2);
            }
            brun += pieces;
        }
        run += cnt;
    }
    if (gl == 0) {
        s_off[nx] = total;
        p.perm_off[nx] = total;
        p.n_chunks[0] = stotal;
        p.n_chunks[1] = btotal;
    }
}

__device__ inline void publish_balance(const RouteParams& p, const int* s_work, int tid) {
    if (tid != 0 || p.T <= 32) return;   // no big chunks up to 32 tokens
    int most = 0, total = 0;
    for (int i = 0; i < kXcds; ++i) {
        most = max(most, s_work[i]);
        total += s_work[i];
    }
    p.n_chunks[kEvenShares] = (long long)most * kXcds * 20 <= (long long)total * 21;
}

// Token-block bitmasks: bit (t - t0) of word (x, (t - t0) / 64) is set when
// token t of [t0, t0 + tn) chose routed expert x.  W words per expert.  An
// expert named twice in one token's list sets one bit: it gets one row, which
// both slots read.
__device__ void token_masks(const RouteParams& p, int t0, int tn, int W, int tid, int nthr,
                            unsigned long long* s_mask) {
    const int E = p.E, k = p.k;
    for (int i = tid; i < E * W; i += nthr) s_mask[i] = 0ull;
    __syncthreads();
    for (int i = tid; i < tn * k; i += nthr) {
        const int e = p.topk_ids[(size_t)t0 * k + i];
        if (e >= 0 && e < E) {
            const int tl = i / k;
            atomicOr(&s_mask[e * W + (tl >> 6)], 1ull << (tl & 63));
        }
    }
    __syncthreads();
}

// The bitmasks, and per word the number of set bits in the words before it.
__device__ void fill_masks(const RouteParams& p, int t0, int tn, int W, int tid, int nthr,
                           unsigned long long* s_mask, int* s_pre) {
    const int E = p.E;
    token_masks(p, t0, tn, W, tid, nthr, s_mask);
    // s_pre[e*W + w]: tokens of words 0..w-1 that chose expert e.
    for (int i = tid; i < E * W; i += nthr) {
        const int w = i % W;
        int c = 0;
        for (int v = i - w; v < i; ++v) c += __popcll(s_mask[v]);
        s_pre[i] = c;
    }
    __syncthreads();
}

// Rows of the (token, slot) entries of tokens [t0, t0 + tn): routed entry
// of expert e goes to row base[e] + (number of earlier tokens of the block
// that chose e); caller-supplied ids outside [0, E) are empty slots.
__device__ void place_entries(const RouteParams& p, int t0, int tn, int W, const int* base, int tid, int nthr,
                              const unsigned long long* s_mask, const int* s_pre) {
    const int E = p.E, k = p.k, slots = k + p.n_shared;
    for (int i = tid; i < tn * k; i += nthr) {
        const int tl = i / k, j = i - tl * k;
        const int t = t0 + tl;
        const int e = p.topk_ids[(size_t)t * k + j];
        if (e < 0 || e >= E) {
            p.perm_pos[(size_t)t * slots + j] = -1;
            continue;
        }
        const int w = e * W + (tl >> 6);
        const int rank = s_pre[w] + __popcll(s_mask[w] & ((1ull << (tl & 63)) - 1ull));
        const int pos = base[e] + rank;
        p.perm_tok[pos] = t;
        p.perm_pos[(size_t)t * slots + j] = pos;
    }
}

// Shared experts: every token, in order.
__device__ void place_shared(const RouteParams& p, const int* s_off, int tid, int nthr) {
    const int T = p.T, E = p.E, k = p.k, slots = k + p.n_shared;
    for (int i = tid; i < T * p.n_shared; i += nthr) {
        const int t = i / p.n_shared, sh = i - t * p.n_shared;
        const int pos = s_off[E + sh] + t;
        p.perm_tok[pos] = t;
        p.perm_pos[(size_t)t * slots + k + sh] = pos;
    }
}

// Permutation of K_final (read from global memory) by expert slot, tokens
// ascending within a slot, plus the FFN work lists, for batches of at most
// kMaskT tokens: one workgroup; each expert's tokens are a bitmask in LDS and
// every (token, slot) entry finds its row independently by counting set bits.
struct PermShared {
    int cnt[kMaxE + kMaxShared];
    int off[kMaxE + kMaxShared + 1];
    int work[kXcds];
    unsigned long long mask[kMaxE * (kMaskT / 64)];
    int pre[kMaxE * (kMaskT / 64)];
};

__device__ void permute_small(const RouteParams& p, int tid, int nthr, PermShared& sh) {
    int* s_cnt = sh.cnt;
    int* s_off = sh.off;
    unsigned long long* s_mask = sh.mask;
    const int T = p.T, E = p.E;
    const int W = (T + 63) / 64;
    fill_masks(p, 0, T, W, tid, nthr, s_mask, sh.pre);
    for (int x = tid; x < E + p.n_shared; x += nthr) {
        int c = T;
        if (x < E) {
            c = 0;
            for (int w = 0; w < W; ++w) c += __popcll(s_mask[x * W + w]);
        }
        s_cnt[x] = c;
    }
    __syncthreads();
    build_lists(p, s_cnt, s_off, sh.work, tid);
    __syncthreads();
    publish_balance(p, sh.work, tid);
    place_shared(p, s_off, tid, nthr);
    place_entries(p, 0, T, W, s_off, tid, nthr, s_mask, sh.pre);
}

__global__ __launch_bounds__(kRouteThreads) void k_permute(RouteParams p) {
    __shared__ PermShared sh;
    permute_small(p, threadIdx.x, kRouteThreads, sh);
}

// Larger batches: the tokens are cut into blocks of kMaskT.
// (1) per block, each routed expert's token count;
// counted from the same bitmasks (k_permute_place) as the rows are placed,
// so a repeated expert in one token's list counts once;
__global__ __launch_bounds__(kRouteThreads) void k_permute_count(RouteParams p) {
    __shared__ unsigned long long s_mask[kMaxE * (kMaskT / 64)];
    const int tid = threadIdx.x, b = blockIdx.x;
    const int t0 = b * kMaskT, tn = min(kMaskT, p.T - t0);
    const int W = (tn + 63) / 64;
    token_masks(p, t0, tn, W, tid, kRouteThreads, s_mask);
    for (int e = tid; e < p.E; e += kRouteThreads) {
        int c = 0;
        for (int w = 0; w < W; ++w) c += __popcll(s_mask[e * W + w]);
        p.perm_blk[(size_t)b * p.E + e] = c;
    }
}

// (2) one workgroup: slot totals, offsets and work lists, each block's first
// row per expert (replacing its count), the shared experts' rows;
__global__ __launch_bounds__(kRouteThreads) void k_permute_scan(RouteParams p) {
    __shared__ int s_cnt[kMaxE + kMaxShared];
    __shared__ int s_off[kMaxE + kMaxShared + 1];
    __shared__ int s_work[kXcds];
    const int tid = threadIdx.x, E = p.E;
    const int nblk = (p.T + kMaskT - 1) / kMaskT;
    for (int x = tid; x < E + p.n_shared; x += kRouteThreads) {
        int c = p.T;
        if (x < E) {
            c = 0;
            for (int b = 0; b < nblk; ++b) c += p.perm_blk[(size_t)b * E + x];
        }
        s_cnt[x] = c;
    }
    __syncthreads();
    build_lists(p, s_cnt, s_off, s_work, tid);
    __syncthreads();
    publish_balance(p, s_work, tid);
    for (int x = tid; x < E; x += kRouteThreads) {
        int run = s_off[x];
        for (int b = 0; b < nblk; ++b) {
            const int c = p.perm_blk[(size_t)b * E + x];
            p.perm_blk[(size_t)b * E + x] = run;
            run += c;
        }
    }
    place_shared(p, s_off, tid, kRouteThreads);
}

// (3) per block, the rows of its (token, slot) entries.
__global__ __launch_bounds__(kRouteThreads) void k_permute_place(RouteParams p) {
    __shared__ unsigned long long s_mask[kMaxE * (kMaskT / 64)];
    __shared__ int s_pre[kMaxE * (kMaskT / 64)];
    const int tid = threadIdx.x, b = blockIdx.x;
    const int t0 = b * kMaskT, tn = min(kMaskT, p.T - t0);
    const int W = (tn + 63) / 64;
    fill_masks(p, t0, tn, W, tid, kRouteThreads, s_mask, s_pre);
    place_entries(p, t0, tn, W, p.perm_blk + (size_t)b * p.E, tid, kRouteThreads, s_mask, s_pre);
}

hipError_t launch_permutation(const RouteParams& p, hipStream_t s) {
    if (p.T <= kMaskT) {
        hipLaunchKernelGGL(k_permute, dim3(1), dim3(kRouteThreads), 0, s, p);
        return hipGetLastError();
    }
    const dim3 blocks((p.T + kMaskT - 1) / kMaskT);
    hipLaunchKernelGGL(k_permute_count, blocks, dim3(kRouteThreads), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_permute_scan, dim3(1), dim3(kRouteThreads), 0, s, p);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_permute_place, blocks, dim3(kRouteThreads), 0, s, p);
    return hipGetLastError();
}

// Compensation kernel: one wavefront per token (phase C).
template <int EPL>
__global__ __launch_bounds__(kTokThreads) void k_compensate(RouteParams p) {
    __shared__ uint8_t s_trans[kMaxE];
    __shared__ int s_cnt[2];   // refilled and empty slots of the workgroup's tokens
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    for (int e = tid; e < p.E; e += kTokThreads) s_trans[e] = p.trans[e];
    if (tid < 2) s_cnt[tid] = 0;
    __syncthreads();
    for (int t = blockIdx.x * kTokWaves + wave; t < p.T; t += gridDim.x * kTokWaves)
        compensate_token<EPL>(p, t, lane, p.orig_ids + (size_t)t * p.k, s_trans, &s_cnt[0], &s_cnt[1]);
    // One global update per workgroup (per-token updates of the same two
    // words serialise in the L2).
    __syncthreads();
    if (tid == 0) {
        if (s_cnt[0]) atomicAdd(&p.counts[0], s_cnt[0]);
        if (s_cnt[1]) atomicAdd(&p.counts[1], s_cnt[1]);
    }
}

// Small batches: the whole routing step (phases A-C and the permutation)
// in one workgroup of 16 wavefronts, one launch instead of four or five.
// Phases are separated by workgroup barriers.  Everything one phase hands to
// the next (K_t, G, the mandatory flags, the cost and bin tables, A_trans,
// K_final and its weights, the counters) stays in LDS: the phases run on a
// copy of the parameters whose arrays point there, and the results the
// caller and the FFN read are copied out at the end.
constexpr int kFusedWaves = kRouteThreads / kWave;

template <int EPL>
__device__ void route_fused_body(const RouteParams& p) {
    __shared__ PruneShared sp;
    __shared__ PermShared sq;
    __shared__ int32_t l_orig[kFusedT * kMaxK], l_top1[kFusedT], l_fin[kFusedT * kMaxK];
    __shared__ double l_g[kFusedT * kMaxK], l_isum[kMaxE];
    __shared__ float l_w[kFusedT * kMaxK], l_cost[kMaxE];
    __shared__ int32_t l_bin[kMaxE];
    __shared__ uint8_t l_mflag[kFusedT * kMaxK], l_trans[kMaxE];
    __shared__ uint32_t l_masks[4 * (kMaxE / 32)];
    __shared__ int32_t l_stats[kStats];
    int32_t* const l_counts = l_stats + 6;
    __shared__ double l_bl[3 * kMaxE];
    __shared__ double l_s[kFusedT * kMaxK];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int k = p.k, E = p.E;
    RouteParams q = p;
    q.orig_ids = l_orig;
    q.gbuf = l_g;
    q.top1 = l_top1;
    q.mflag = l_mflag;
    q.cost = l_cost;
    q.bin = p.bin ? l_bin : nullptr;
    q.trans = l_trans;
    q.topk_ids = l_fin;
    q.topk_w = l_w;
    q.counts = l_counts;
    q.imp_sum = l_isum;
    q.masks = p.masks ? l_masks : nullptr;
    q.stats = p.stats ? l_stats : nullptr;
    q.bin_loads = p.bin_loads && p.n_bins <= kMaxE ? l_bl : p.bin_loads;
    q.sslot = l_s;
    // The tables, read by the waves that route no token while the others do.
    for (int e = tid; e < E; e += kRouteThreads) {
        l_cost[e] = p.cost[e];
        if (p.bin) l_bin[e] = p.bin[e];
    }
    for (int t = wave; t < p.T; t += kFusedWaves)
        route_token<EPL>(q, t, lane, q.orig_ids + (size_t)t * k, q.gbuf + (size_t)t * k, q.top1 + t,
                         q.mflag + (size_t)t * k);
    __syncthreads();
    if (p.rule == CAEE_IMPORTANCE_SUM) {
        importance_sum_small(q, tid, kRouteThreads);
        __syncthreads();
    }
    prune_all(q, tid, kRouteThreads, sp);
    __syncthreads();
    __shared__ int s_cnt[2];
    if (tid < 2) s_cnt[tid] = 0;
    __syncthreads();
    if (sp.stat[3] == 0 && p.refill != CAEE_REFILL_LITERAL) {
        // Nothing was pruned: every token keeps its list, one thread per slot
        // with compensate_token's arithmetic.
        for (int i = tid; i < p.T * k; i += kRouteThreads) {
            const int t0 = i / k * k;
            double total = 0.0;
            for (int r = 0; r < k; ++r) total += l_s[t0 + r];
            l_fin[i] = l_orig[i];
            l_w[i] = (float)(p.rs * (l_s[i] / total));
        }
    } else {
        for (int t = wave; t < p.T; t += kFusedWaves)
            compensate_token<EPL>(q, t, lane, q.orig_ids + (size_t)t * k, l_trans, &s_cnt[0], &s_cnt[1]);
    }
    __syncthreads();
    if (tid < 2) l_counts[tid] = s_cnt[tid];   // the only workgroup: the call's totals
    __syncthreads();
    if (p.do_permute) permute_small(q, tid, kRouteThreads, sq);
    // Results read after this kernel: K_t, K_final and its weights, A_trans.
    for (int i = tid; i < p.T * k; i += kRouteThreads) {
        p.orig_ids[i] = l_orig[i];
        p.topk_ids[i] = l_fin[i];
        p.topk_w[i] = l_w[i];
    }
    for (int e = tid; e < E; e += kRouteThreads) p.trans[e] = l_trans[e];
    const int words = (E + 31) / 32;
    if (p.masks)
        for (int i = tid; i < 4 * words; i += kRouteThreads) p.masks[i] = l_masks[i];
    if (p.stats && tid < kStats) p.stats[tid] = l_stats[tid];
    if (q.bin_loads == l_bl)
        for (int i = tid; i < 3 * p.n_bins; i += kRouteThreads) p.bin_loads[i] = l_bl[i];
}

template <int EPL>
__global__ __launch_bounds__(kRouteThreads) void k_route_fused(RouteParams p) {
    route_fused_body<EPL>(p);
}

// The shared experts' gate/up for a batch of at most 16 tokens, run by the
// workgroups after the first in the routing launch.  Item = one 16-column
// tile (gate and up rows) of one shared expert; the 16 waves of the
// workgroup take consecutive ranges of the contraction, and wave 0 adds the
// 16 partial sums in wave order (deterministic) and stores the SwiGLU rows.
// Shared expert s owns rows s*T .. s*T + T - 1 (row s*T + t for token t).
template <class M>
__device__ void shared_gate_up(const FfnParams& p, int wg, int n_wg) {
    constexpr int kWaves = kRouteThreads / kWave;
    __shared__ f32x4_t s_part[kWaves][2][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int r = lane & 15, g = lane >> 4;
    const int tiles = p.f / 16;
    const size_t row_units = (size_t)p.d * M::kElemBytes / 16;
    const int ksteps = (int)(row_units / 4);
    const int kper = (ksteps + kWaves - 1) / kWaves;
    const int k0 = min(ksteps, wave * kper), k1 = min(ksteps, k0 + kper);
    const size_t expert_bytes = (size_t)2 * p.f * p.d * M::kElemBytes;
    const int astep = p.tiled ? 64 : 4;
    for (int item = wg; item < p.n_shared * tiles; item += n_wg) {
        const int sh = item / tiles, jt = item - sh * tiles;
        const u32x4_t* wb = (const u32x4_t*)((const char*)p.sh_w13 + (size_t)sh * expert_bytes);
        const u32x4_t* const a[2] = {
            p.tiled ? wb + ((size_t)jt * ksteps + k0) * 64 + lane
                    : wb + (size_t)(jt * 16 + r) * row_units + g + 4 * (size_t)k0,
            p.tiled ? wb + ((size_t)(tiles + jt) * ksteps + k0) * 64 + lane
                    : wb + (size_t)(p.f + jt * 16 + r) * row_units + g + 4 * (size_t)k0};
        const int t = r < p.T ? r : 0;   // padded token columns read a valid row; results dropped
        const u32x4_t* const xb[1] = {(const u32x4_t*)p.x + (size_t)t * row_units + g + 4 * (size_t)k0};
        f32x4_t acc[2][1] = {{f32x4_t{0.f, 0.f, 0.f, 0.f}}, {f32x4_t{0.f, 0.f, 0.f, 0.f}}};
        if (k1 > k0) tile_contract<M, kRouteSharedU, 2, 1>(a, astep, xb, 1, k1 - k0, acc);   // short rows leave waves idle
        s_part[wave][0][lane] = acc[0][0];
        s_part[wave][1][lane] = acc[1][0];
        __syncthreads();
        if (wave == 0 && r < p.T) {
            f32x4_t gs = s_part[0][0][lane], us = s_part[0][1][lane];
            for (int w = 1; w < kWaves; ++w) {
                gs += s_part[w][0][lane];
                us += s_part[w][1][lane];
            }
            float h[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) h[v] = silu_mul(gs[v], us[v]);
            store_h<M>(p, (size_t)(sh * p.T + r) * p.f + jt * 16 + 4 * g, h);
        }
        __syncthreads();
    }
}

template <int EPL, class M>
__global__ __launch_bounds__(kRouteThreads) void k_route_fused_shared(RouteParams p, FfnParams fp) {
    if (blockIdx.x == 0) route_fused_body<EPL>(p);
    else shared_gate_up<M>(fp, blockIdx.x - 1, gridDim.x - 1);
}

// 8-bit batches of at most 16 tokens: the workgroups after the first quantise
// x (what the gate/up launch reads next), 64 blocks of 128 values each, so
// that no launch of its own does.  Batches of at most kSharedFp8T tokens also
// run the shared experts' gate/up here, in the workgroups behind those; a wave
// quantises the piece of x that its contraction range reads for itself (more
// tokens would make that longer than the routing chain).  R1-shaped layer, one
// box: T = 1 91.1 -> 86.3 us, T = 2 133.5 -> 126.7, T = 8 (x only) 195 -> 193.
typedef int i32x8_t __attribute__((ext_vector_type(8)));
constexpr int kSharedFp8T = 4;
constexpr int kSharedFp8K = 4;    // 128-wide blocks a wave contracts at a time
constexpr int kRouteQuantBlocks = kRouteThreads / kQuantLanes;

__device__ inline i32x8_t join8(const u32x4_t& lo, const u32x4_t& hi) {
    return i32x8_t{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
}

__device__ void route_quant_x(const FfnParams& p, int wg) {
    const int b = wg * kRouteQuantBlocks + threadIdx.x / kQuantLanes, l = threadIdx.x % kQuantLanes;
    if (b >= p.T * (p.d / 128)) return;   // uniform over the block's lanes
    float v[8];
    load8((const uint16_t*)p.x + (size_t)b * 128 + 8 * l, v);
    const float sc = quant_block(v, p.xq + (size_t)b * 128, l);
    if (l == 0) p.xs[b] = sc;
}

// What the lanes of a wave have written to LDS is read by its other lanes
// after this, and what they have read may be overwritten.
__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Item: one 16-column tile (gate and up rows) of one shared expert, the 16
// waves on consecutive ranges of the contraction, their partial sums added in
// wave order; fp32 SwiGLU rows, as the gate/up launch stores them.
__device__ void shared_gate_up_fp8(const FfnParams& p, int wg, int n_wg) {
    constexpr int kWaves = kRouteThreads / kWave;
    __shared__ __align__(16) uint8_t s_q[kWaves][kSharedFp8T][kSharedFp8K * 128];
    __shared__ float s_xs[kWaves][kSharedFp8T][kSharedFp8K];
    __shared__ f32x4_t s_part[kWaves][2][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int r = lane & 15, g = lane >> 4;
    const int tiles = p.f / 16, kblocks = p.d / 128;
    const size_t ksteps = (size_t)p.d / 64, row_units = (size_t)p.d / 16;
    const int kper = (kblocks + kWaves - 1) / kWaves;
    const int k0 = min(kblocks, wave * kper), k1 = min(kblocks, k0 + kper);
    const size_t expert_bytes = (size_t)2 * p.f * p.d;
    const size_t scales = (size_t)(2 * p.f / 128) * kblocks;
    const int n = r < p.T ? r : 0;   // padded token columns read a valid row; results dropped
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    for (int item = wg; item < p.n_shared * tiles; item += n_wg) {
        const int sh = item / tiles, jt = item - sh * tiles;
        const u32x4_t* wb = (const u32x4_t*)((const char*)p.sh_w13 + (size_t)sh * expert_bytes);
        const float* ws = p.sh_w13_scale + (size_t)sh * scales;
        f32x4_t acc[2] = {zero, zero};
        for (int kb = k0; kb < k1; kb += kSharedFp8K) {
            // The range's weights, all in flight (blocks past it re-read the last).
            u32x4_t w[kSharedFp8K][2][2];
            float sc[kSharedFp8K][2];
#pragma unroll
            for (int u = 0; u < kSharedFp8K; ++u) {
                const int b = min(kb + u, k1 - 1);
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const int row = m * p.f + jt * 16;
                    const u32x4_t* a = p.tiled ? wb + ((size_t)(row / 16) * ksteps + 2 * b) * 64 + lane
                                               : wb + (size_t)(row + r) * row_units + g + 8 * (size_t)b;
                    w[u][m][0] = load_stream(a);
                    w[u][m][1] = load_stream(a + (p.tiled ? 64 : 4));
                    sc[u][m] = ws[(size_t)(row / 128) * kblocks + b];
                }
            }
            // x of the range: 16 lanes per block, one block of each token at a
            // time.  The codes and scales go to other lanes of the wave
            // through LDS: ordered by the fences below (the wave's LDS
            // operations run in order; the fences keep the compiler to it).
            const int qb = lane / kQuantLanes, ql = lane % kQuantLanes;
            for (int t = 0; t < p.T; ++t) {
                float v[8];
                load8((const uint16_t*)p.x + (size_t)t * p.d + (size_t)min(kb + qb, k1 - 1) * 128 + 8 * ql, v);
                const float s = quant_block(v, &s_q[wave][t][qb * 128], ql);
                if (ql == 0) s_xs[wave][t][qb] = s;
            }
            wave_lds_sync();
#pragma unroll
            for (int u = 0; u < kSharedFp8K; ++u) {
                if (kb + u >= k1) break;
                const u32x4_t* q = (const u32x4_t*)&s_q[wave][n][u * 128];
                const i32x8_t x = join8(q[g], q[4 + g]);
                const float xs = s_xs[wave][n][u];
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const f32x4_t part = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(
                        join8(w[u][m][0], w[u][m][1]), x, zero, 0, 0, 0, 127, 0, 127);   // E8M0 127: 1.0
                    acc[m] += part * (sc[u][m] * xs);
                }
            }
            wave_lds_sync();   // before the next range's codes replace these
        }
        s_part[wave][0][lane] = acc[0];
        s_part[wave][1][lane] = acc[1];
        __syncthreads();
        if (wave == 0 && r < p.T) {
            f32x4_t gs = s_part[0][0][lane], us = s_part[0][1][lane];
            for (int q = 1; q < kWaves; ++q) {
                gs += s_part[q][0][lane];
                us += s_part[q][1][lane];
            }
            float h[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) h[v] = silu_mul(gs[v], us[v]);
            *(float4*)((float*)p.h + (size_t)(sh * p.T + r) * p.f + jt * 16 + 4 * g) =
                make_float4(h[0], h[1], h[2], h[3]);
        }
        __syncthreads();
    }
}

template <int EPL>
__global__ __launch_bounds__(kRouteThreads) void k_route_fused_fp8(RouteParams p, FfnParams fp, int quant_wgs) {
    const int b = blockIdx.x;
    if (b == 0) route_fused_body<EPL>(p);
    else if (b <= quant_wgs) route_quant_x(fp, b - 1);
    else shared_gate_up_fp8(fp, b - 1 - quant_wgs, gridDim.x - 1 - quant_wgs);
}

}  // namespace

bool route_runs_shared(const caee_layer_desc_t& d) {
    // one 16-token block: the workgroups' tiles hold every token of the batch
    if (d.w_dtype == CAEE_FP8_E4M3) return kRouteShared && d.T <= kSharedFp8T && d.n_shared > 0;
    return kRouteShared && d.T <= 16 && d.T <= kFusedT && d.n_shared > 0;
}

bool route_quantises_x(const caee_layer_desc_t& d) { return d.w_dtype == CAEE_FP8_E4M3 && d.T <= kFusedT; }

hipError_t launch_route_shared(const RouteParams& p, const FfnParams& fp, int w_dtype, bool shared, hipStream_t s) {
    const int items = shared ? fp.n_shared * (fp.f / 16) : 0;
    const int quant_wgs =
        w_dtype == CAEE_FP8_E4M3 ? (p.T * (fp.d / 128) + kRouteQuantBlocks - 1) / kRouteQuantBlocks : 0;
    const int cap = device_cu_count() - 1 - quant_wgs > 1 ? device_cu_count() - 1 - quant_wgs : 1;
    const dim3 grid(1 + quant_wgs + (items < cap ? items : cap));
    if (w_dtype == CAEE_FP8_E4M3) {
        switch (p.epl) {
            case 1: hipLaunchKernelGGL(k_route_fused_fp8<1>, grid, dim3(kRouteThreads), 0, s, p, fp, quant_wgs); break;
            case 2: hipLaunchKernelGGL(k_route_fused_fp8<2>, grid, dim3(kRouteThreads), 0, s, p, fp, quant_wgs); break;
            case 4: hipLaunchKernelGGL(k_route_fused_fp8<4>, grid, dim3(kRouteThreads), 0, s, p, fp, quant_wgs); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    auto go = [&](auto k) -> hipError_t {
        hipLaunchKernelGGL(k, grid, dim3(kRouteThreads), 0, s, p, fp);
        return hipGetLastError();
    };
    const bool bf16 = w_dtype == CAEE_BF16;
    if (w_dtype != CAEE_BF16 && w_dtype != CAEE_F32) return hipErrorInvalidValue;
    switch (p.epl) {
        case 1: return bf16 ? go(k_route_fused_shared<1, Bf16Math>) : go(k_route_fused_shared<1, F32Math>);
        case 2: return bf16 ? go(k_route_fused_shared<2, Bf16Math>) : go(k_route_fused_shared<2, F32Math>);
        case 4: return bf16 ? go(k_route_fused_shared<4, Bf16Math>) : go(k_route_fused_shared<4, F32Math>);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_route(const RouteParams& p, hipStream_t s) {
    const dim3 tok_grid((p.T + kTokWaves - 1) / kTokWaves);
    auto token_kernels = [&](auto route_k, auto comp_k, auto fused_k) -> hipError_t {
        if (p.T <= kFusedT) {
            hipLaunchKernelGGL(fused_k, dim3(1), dim3(kRouteThreads), 0, s, p);
            return hipGetLastError();
        }
        hipLaunchKernelGGL(route_k, tok_grid, dim3(kTokThreads), 0, s, p);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        RouteParams q = p;
        q.pair_stats = takes_pair_stats(p);
        if (q.pair_stats) {
            hipLaunchKernelGGL(k_expert_stats, dim3(p.E), dim3(kStatWaves * kWave), 0, s, p);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(k_prune, dim3(1), dim3(kRouteThreads), 0, s, q);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(comp_k, tok_grid, dim3(kTokThreads), 0, s, p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        return p.do_permute ? launch_permutation(p, s) : hipSuccess;
    };
    switch (p.epl) {
        case 1: return token_kernels(k_route_tokens<1>, k_compensate<1>, k_route_fused<1>);
        case 2: return token_kernels(k_route_tokens<2>, k_compensate<2>, k_route_fused<2>);
        case 4: return token_kernels(k_route_tokens<4>, k_compensate<4>, k_route_fused<4>);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_permute(const RouteParams& p, hipStream_t s) {
    return launch_permutation(p, s);
}

}  // namespace caee
