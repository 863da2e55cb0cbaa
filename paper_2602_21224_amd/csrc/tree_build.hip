// Draft-tree builder for gfx950: token-info sampling (Alg. 1) followed by the
// verification-budget pruning (§5.2). It produces the parent / token arrays
// (and per-sequence node counts) that the verification calls consume.
//
// At step i a frontier node's children are the k most probable tokens of
// softmax(l_i + r), r being the node token's row of the hot-token table (§5.1
// collapses the token-info embedding into an additive logit table; §6.1 keeps
// it for the hot tokens only). What depends on the node are the H hot columns;
// the non-hot entries of l_i are reduced once per (sequence, step). The steps
// depend on each other, so the number of launches and the chain inside each
// decide the time: one launch per step (tb_step_kernel) in which
//   * every workgroup of a sequence first combines the previous step's partial
//     results into children, joint probabilities and the frontier, each for
//     itself (in less time than another launch takes), then expands the
//     frontier on its share of the hot columns;
//   * further workgroups, on the same CUs, reduce the non-hot entries of this
//     step, which the next launch needs.
// tb_finish_kernel selects the last step's children and keeps the `budget`
// nodes of largest joint probability, in creation order. Without hot tokens
// only the rows (tb_rows_kernel) and tb_finish_kernel run. More than 8 branches,
// and first trees of large batches, take tree_build_many.hip's separate launches
// (one_launch_per_step).
//
// Decisions: candidates are ranked by the fp32 sum l + r (the precision of the
// logits; ties to the lower vocabulary id) through a packed 64-bit key; -inf and
// NaN are no candidates, so a node with fewer than k others has children without
// a token (-1, probability 0).
// Probabilities and joint probabilities are fp64 (exp and sums in double), so
// frontier and pruning decisions agree with an fp64 evaluation unless two
// joint probabilities are equal to within about 1e-13.
//
// Top-k of a set held in registers: the maxima of k or more disjoint groups of
// it are k candidates, so none of the k largest lies below the smallest of
// those maxima. The entries at or above that floor (about 22) are listed in LDS
// and ranked by counting; a long list (many equal entries, or groups without any) is
// made again from whole keys, value and vocabulary id, above the k-th largest of all
// lanes' maxima, which no more than k lanes reach. Long is more than 128: of random
// entries fewer than one set in a million is (more than 64, one in 650). Measured
// (us per call): 16 sequences, 7 steps, 128256 tokens of which 32768 hot, k 8, all but
// 64 logits masked to -1e4: 485 with k rounds of a plain maximum in place of the
// second list, 213 with it; 4 sequences, 7 steps, 2343 tokens of which 201 hot, k 4:
// 124 with lists of 201 ranked as they are, 71 so.
//
// Measured (16 sequences, 7 steps, vocabulary 128256, 32768 hot tokens, k 8):
// 199 us per call with a launch for all rows and two launches per step, 157 us
// now; 3 sequences, 5 steps, 32000 tokens, all hot, k 4: 74 -> 42 us. A step is
// 22 us, 19 without its rows, which took 43 us of their own for the seven steps.
#include "tree_build_common.h"

#include <algorithm>
#include <climits>

namespace tv {
namespace {

constexpr int kTbThreads = 512;            // 8 waves: one per frontier node (k <= 8)
constexpr int kTbWaves = kTbThreads / kWave;
constexpr int kTbList = 4 * kWave;         // listed candidates of one wave: room,
constexpr int kTbLong = 2 * kWave;         // and from where on a narrower floor pays
constexpr int kRowsList = 2 * kWave;       // listed candidates of a rows workgroup
constexpr int kMaxParts = 32;              // most segments of a row, most chunks of the hot columns
constexpr int kMaxBranches = 8;            // most branches of these kernels
constexpr int kPruneSlots = 1024;          // nodes of an unpruned tree
static_assert(1 + kMaxBranches + (kTbMaxSteps - 1) * kMaxBranches * kMaxBranches <= kPruneSlots, "pruning slots");
static_assert(kMaxBranches <= kTbWaves, "one wave per frontier node");
constexpr int kBuckets = 1024;             // of joint probabilities, for the pruning

// Partial reductions over sets of candidates, contiguous per reader: of each
// part its maximum and the sum of exp(x - max) in fp64, its top-k keys in
// descending order (0 = none) and, of column parts, their hot columns; kk keys
// per part, the power of two at or above k. Part p of a row: (b S + step) segs +
// segment; of the columns: (b k + slot) chunks + chunk.
struct TbSum {
    double s;
    float m;
    int pad;
};
struct TbParts {
    TbSum *sum;
    unsigned long long *key;
    int *col;
};

// The frontier of one sequence: its node count and, per slot (frontier order),
// the node, the hot row of its token (-1: none) and its joint probability.
struct TbSlot {
    int node, h;
    double joint;
};
struct TbFrontier {
    int count, pad;
    TbSlot slot[kTbMaxK];
};

__device__ __forceinline__ unsigned long long umin64(unsigned long long a, unsigned long long b) {
    return a < b ? a : b;
}

// LDS traffic of one wave between its own lanes: the writes before are done,
// and the compiler keeps the reads behind them.
__device__ __forceinline__ void wave_lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }


template <int C>
__device__ __forceinline__ unsigned long long dpp64u(unsigned long long v) {
    return ((unsigned long long)dpp32<C>((unsigned int)(v >> 32)) << 32) | dpp32<C>((unsigned int)v);
}

// Smallest of the maxima of `groups` (8, 4, 2 or 1, wave-uniform; >= k) groups of
// lanes: at least as many of the lanes' values are at or above it. Fewer groups give
// a higher floor and a shorter list (16 sequences of 32000 tokens, all hot, k 4: 74 us
// with 8 groups, 68 with 4; selects in place of the branches cost 0.5 % at 8).
__device__ __forceinline__ float wave_floor(float v, int groups) {
    const auto mx = [](float a, unsigned b) { return fmaxf(a, __uint_as_float(b)); };
    const auto mn = [](float a, unsigned b) { return fminf(a, __uint_as_float(b)); };
    const auto rest = [&](float x, auto first, auto second, auto third) {
        x = first(x, dpp32<kDppMirror>(__float_as_uint(x)));
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        x = second(__uint_as_float(r[0]), r[1]);
        const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return third(__uint_as_float(h[0]), h[1]);
    };
    v = mx(v, dpp32<kDppXor1>(__float_as_uint(v)));
    v = mx(v, dpp32<kDppXor2>(__float_as_uint(v)));
    v = mx(v, dpp32<kDppHalfMirror>(__float_as_uint(v)));
    if (groups == 8) return rest(v, mn, mn, mn);
    if (groups == 4) return rest(v, mx, mn, mn);
    if (groups == 2) return rest(v, mx, mx, mn);
    return rest(v, mx, mx, mx);
}
__device__ __forceinline__ unsigned long long wave_floor64(unsigned long long v) {
    v = umax64(v, dpp64u<kDppXor1>(v));
    v = umax64(v, dpp64u<kDppXor2>(v));
    v = umax64(v, dpp64u<kDppHalfMirror>(v));
    v = umin64(v, dpp64u<kDppMirror>(v));
    #pragma unroll
    for (int half = 0; half < 2; ++half) {
        const unsigned int lo = (unsigned int)v, hi = (unsigned int)(v >> 32);
        const auto l = half == 0 ? __builtin_amdgcn_permlane16_swap(lo, lo, false, false)
                                 : __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = half == 0 ? __builtin_amdgcn_permlane16_swap(hi, hi, false, false)
                                 : __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        v = umin64(((unsigned long long)h[0] << 32) | l[0], ((unsigned long long)h[1] << 32) | l[1]);
    }
    return v;
}

// A floor for lists of whole keys: the k-th largest of the lanes' largest keys (1
// when fewer lanes have any). Keys have no equals, so only k lanes hold keys at
// or above it.
__device__ __forceinline__ unsigned long long wave_kth64(unsigned long long v, int k) {
    unsigned long long f = 0ull;
    for (int q = 0; q < k; ++q) {
        f = wave_max64(v);
        if (v == f) v = 0ull;
    }
    return umax64(f, 1ull);
}

// Lanes of `mask` below this one.
__device__ __forceinline__ int below(unsigned long long mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

template <typename T>
__device__ __forceinline__ void tie(T &x) {
    asm volatile("" : "+v"(x));
}

// How many of list[0 .. n) exceed `a` and `b`. The list is readable and zero (no
// key) up to the next multiple of 8; eight reads are in flight together.
__device__ __forceinline__ void count_above(const unsigned long long *list, int n, unsigned long long a,
                                            unsigned long long b, int &ra, int &rb) {
    for (int i = 0; i < n; i += 8) {
        unsigned long long o[8];
        #pragma unroll
        for (int u = 0; u < 8; ++u) o[u] = list[i + u];
        #pragma unroll
        for (int u = 0; u < 8; ++u) {
            ra += o[u] > a;
            rb += o[u] > b;
        }
    }
}

// The k largest of a wave's list[0 .. n) (room for 8 more entries) and, with
// `more`, of the k keys in old, in descending order into win (0 = none), with
// their columns. By one wave, which has synchronised its LDS writes; it is
// synchronised again on return.
__device__ __forceinline__ void list_winners(unsigned long long *list, const int *lcol, int n, int k, int lane,
                                             bool more, const unsigned long long *old, const int *ocol,
                                             unsigned long long *win, int *wcol) {
    if (lane < 8) list[n + lane] = 0ull;
    if (lane < kTbMaxK) win[lane] = 0ull;
    wave_lds_sync();
    unsigned long long prev = more && lane < k ? old[lane] : 0ull;
    int prank = 0;
    for (int b0 = 0; b0 < n; b0 += kWave) {          // one round unless the list is long
        const unsigned long long mine = b0 + lane < n ? list[b0 + lane] : 0ull;
        const int col = lcol[min(b0 + lane, n - 1)];
        int rank = 0, unused = 0;
        count_above(list, n, mine, ~0ull, rank, unused);
        if (more) count_above(old, k, mine, ~0ull, rank, unused);
        if (mine != 0ull && rank < k) {
            win[rank] = mine;
            wcol[rank] = col;
        }
    }
    if (more) {
        int unused = 0;
        count_above(list, n, prev, ~0ull, prank, unused);
        count_above(old, k, prev, ~0ull, prank, unused);
        if (prev != 0ull && prank < k) {
            win[prank] = prev;
            wcol[prank] = ocol[lane];
        }
    }
    wave_lds_sync();
}

// (m, s) += (m2, s2), s being a sum of exp(x - m).
__device__ __forceinline__ void merge_sum(float &m, double &s, float m2, double s2, const double *tab) {
    if (m2 == kNegInf) return;
    if (m == kNegInf) { m = m2; s = s2; return; }
    const float mn = fmaxf(m, m2);
    s = s * exp_nonpos((double)m - (double)mn, tab) + s2 * exp_nonpos((double)m2 - (double)mn, tab);
    m = mn;
}

// LDS of a rows reduction.
struct RowsShared {
    double exp2[kExpTab];
    float gm[kTbWaves];                              // the waves' maxima: 8 groups
    double sum[kTbWaves];
    unsigned long long list[kRowsList], win[kTbMaxK];
    int n;
};

// Node-independent part of one (sequence, step): the non-hot tokens of the
// step's logits, one segment of the vocabulary per workgroup, in passes of U
// tokens per thread held in registers (one pass unless the vocabulary is larger
// than 32 segments of them). Bound by its instructions (about 35 per token, two
// thirds of them the fp64 exponential), not by the logits' bytes.
template <int U>
__device__ __forceinline__ void reduce_row(RowsShared &sh, const float *__restrict__ l,
                                           const int32_t *__restrict__ hot_index, int V, int H, int k, int kk,
                                           int v0, int v1, TbSum *sum_out, unsigned long long *key_out) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    double *const s_exp2 = sh.exp2, *const s_sum = sh.sum;
    float *const s_gm = sh.gm;
    unsigned long long *const s_list = sh.list, *const s_win = sh.win;
    int &s_n = sh.n;
    fill_exp2_table(s_exp2);
    if (tid < kTbMaxK) s_win[tid] = 0ull;
    float M = kNegInf;                               // thread 0: the segment so far
    double sum = 0.0;
    for (int vb = v0; vb < v1; vb += U * kTbThreads) {
        float xv[U];
        {
            int hv[U];
            #pragma unroll
            for (int u = 0; u < U; ++u) {            // every load before any use (indices clamped)
                const int v = min(vb + u * kTbThreads + tid, v1 - 1);
                hv[u] = H > 0 ? hot_index[v] : -1;
                xv[u] = l[v];
            }
            #pragma unroll
            for (int u = 0; u < U; ++u) {            // outside, or hot (handled per node): unused
                xv[u] = (unsigned)hv[u] >= (unsigned)H ? xv[u] : kNegInf;
                xv[u] = tid < v1 - vb - u * kTbThreads ? xv[u] : kNegInf;
                tie(xv[u]);                          // one mask at a time
            }
        }
        float m = kNegInf;
        #pragma unroll
        for (int u = 0; u < U; ++u) m = fmaxf(m, xv[u]);
        __syncthreads();                             // the previous pass's lists are done with
        if (tid == 0) s_n = 0;
        m = wave_allmax(m);
        if (lane == 0) s_gm[wave] = m;
        __syncthreads();
        float pm = kNegInf, fl = -kNegInf;
        #pragma unroll
        for (int g = 0; g < kTbWaves; ++g) {
            pm = fmaxf(pm, s_gm[g]);
            fl = fminf(fl, s_gm[g]);
        }
        if (pm == kNegInf) continue;                 // uniform: no candidate in this pass
        fl = fmaxf(k == 1 ? pm : fl, -__FLT_MAX__);  // -inf is no candidate
        double ps = 0.0;
        #pragma unroll
        for (int u = 0; u < U; ++u) ps += exp_nonpos((double)xv[u] - (double)pm, s_exp2);
        ps = wave_allsum(ps);
        if (lane == 0) s_sum[wave] = ps;
        bool full = false;                           // too long already
        #pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned long long mask = __ballot(xv[u] >= fl);
            if (mask == 0ull || full) continue;      // wave-uniform
            int at = 0;
            if (lane == 0) at = atomicAdd(&s_n, __popcll(mask));
            at = __builtin_amdgcn_readfirstlane(at);
            full = at >= kRowsList;
            at += below(mask);
            if (((mask >> lane) & 1ull) && at < kRowsList)
                s_list[at] = pack_key(order_key(xv[u]), (unsigned)(vb + u * kTbThreads + tid));
        }
        __syncthreads();
        int nl = s_n;
        if (nl > kRowsList) {
            // Many equal values at the floor (a masked vocabulary): again by whole
            // keys, above the k-th largest of the threads' largest keys, which the
            // waves' k largest of them give (k U keys at most).
            auto key = [&](int u) {
                return xv[u] > kNegInf ? pack_key(order_key(xv[u]), (unsigned)(vb + u * kTbThreads + tid)) : 0ull;
            };
            unsigned long long c = 0ull;
            #pragma unroll
            for (int u = 0; u < U; ++u) c = umax64(c, key(u));
            for (int q = 0; q < 8; ++q) {
                const unsigned long long best = q < k ? wave_max64(c) : 0ull;
                if (c == best) c = 0ull;
                if (lane == 0) s_list[wave * 8 + q] = best;
            }
            __syncthreads();
            if (tid == 0) s_n = 0;
            const unsigned long long kfl = wave_kth64(s_list[lane], k);
            __syncthreads();
            #pragma unroll
            for (int u = 0; u < U; ++u) {
                tie(xv[u]);                          // the first pass's tests are not kept
                const unsigned long long mask = __ballot(key(u) >= kfl);
                if (mask == 0ull) continue;          // wave-uniform
                int at = 0;
                if (lane == 0) at = atomicAdd(&s_n, __popcll(mask));
                at = __builtin_amdgcn_readfirstlane(at) + below(mask);
                if ((mask >> lane) & 1ull) s_list[at] = key(u);
            }
            __syncthreads();
            nl = s_n;
        }
        // rank the listed keys and the earlier passes' winners by counting
        if (tid < 8 && nl + tid < kRowsList) s_list[nl + tid] = 0ull;
        __syncthreads();
        const bool more = vb > v0;                   // earlier passes exist
        unsigned long long mine = tid < nl ? s_list[tid] : 0ull;
        unsigned long long old = (more && tid < k) ? s_win[tid] : 0ull;
        int rank = 0, orank = 0;
        if (wave * kWave < nl || more) {
            count_above(s_list, nl, mine, old, rank, orank);
            if (more) count_above(s_win, k, mine, old, rank, orank);
        }
        __syncthreads();
        if (tid < kTbMaxK) s_win[tid] = 0ull;
        __syncthreads();
        if (mine != 0ull && rank < k) s_win[rank] = mine;
        if (old != 0ull && orank < k) s_win[orank] = old;
        if (tid == 0) {
            double t = 0.0;
            for (int w = 0; w < kTbWaves; ++w) t += s_sum[w];
            merge_sum(M, sum, pm, t, s_exp2);
        }
    }
    __syncthreads();
    if (tid < kk) key_out[tid] = s_win[tid];
    if (tid == 0) {
        sum_out->s = sum;
        sum_out->m = M;
    }
}

// LDS of a selection.
struct SelShared {
    double joint[kMaxBranches * kMaxBranches];       // the step's children
    int col[kMaxBranches * kMaxBranches];
    unsigned long long list[kTbWaves][kTbList + 8];  // candidates of a wave; also the expansion's
    int lcol[kTbWaves][kTbList];
    unsigned long long win[2][kTbWaves][kTbMaxK];    // its k largest
    int wcol[2][kTbWaves][kTbMaxK];
    TbSlot slot[kTbMaxK];                            // the next frontier
    int nf;
};

// Selection of step `step` of sequence b by a whole workgroup: per frontier
// node (one wave each) the step's row partials and the node's column partials
// become its k children (token, probability, joint probability), then the k
// children of largest joint probability become the next frontier (sh.slot,
// sh.nf). `writer`: this workgroup stores the children and the next frontier.
// `between` runs once, after the first loads are issued, and the workgroup
// synchronises behind it (it may fill tab) and before the return.
template <int CPL, typename F>      // candidate keys per lane
__device__ __forceinline__ void select_step(SelShared &sh, TbParts rows, int segs, TbParts parts, int chunks,
                                            TbWindow win, int b, int S, int k, int step,
                                            int max_nodes, const TbFrontier *fr, TbFrontier *next,
                                            bool writer, const double *tab, int32_t *node_tok,
                                            int32_t *node_par, double *node_joint, F between) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int nparts = segs + chunks;
    // nodes before this step: the root, then k children per frontier node of
    // every earlier step (1 at step 0, k afterwards)
    const int base = step == 0 ? 1 : 1 + k + (step - 1) * k * k;
    // Key i of part q (the rows', then the columns') belongs to lane
    // (q kk + i) mod 64.
    const int ksh = k <= 1 ? 0 : 32 - __builtin_clz(k - 1);
    const size_t rp = ((size_t)b * S + win.first + step) * segs;
    const int nkeys = nparts << ksh, rkeys = segs << ksh;
    int nf = 0;
    {
        const int j = wave, jr = min(j, k - 1);      // slots past nf load stale data, unused
        const size_t cp = ((size_t)b * k + jr) * chunks;
        // unconditional loads, clamped (without hot tokens parts are never read)
        const TbSum *ps1 = lane < segs || chunks == 0 ? rows.sum + rp + min(lane, segs - 1)
                                                      : parts.sum + cp + (min(lane, nparts - 1) - segs);
        float pm = ps1->m;
        double ps = ps1->s;
        unsigned long long cand[CPL];
        int col[CPL];
        #pragma unroll
        for (int u = 0; u < CPL; ++u) {
            const int x = min(lane + u * kWave, nkeys - 1);
            const unsigned long long *kp = x < rkeys ? rows.key + (rp << ksh) + x : parts.key + (cp << ksh) + (x - rkeys);
            cand[u] = *kp;
            col[u] = chunks > 0 ? parts.col[(cp << ksh) + max(x - rkeys, 0)] : -1;
        }
        const TbSlot sl = fr->slot[jr];
        const int count = fr->count;
        between();
        __syncthreads();
        nf = count;
        if (j < nf) {
            pm = lane < nparts ? pm : kNegInf;
            #pragma unroll
            for (int u = 0; u < CPL; ++u) {
                if (lane + u * kWave >= nkeys) cand[u] = 0ull;
                if (lane + u * kWave < rkeys) col[u] = -1;
            }
            const float m = wave_allmax(pm);
            const double s = wave_allsum(pm == kNegInf ? 0.0 : ps * exp_nonpos((double)pm - (double)m, tab));
            unsigned long long lm = 0ull;
            #pragma unroll
            for (int u = 0; u < CPL; ++u) lm = umax64(lm, cand[u]);
            const unsigned long long fl = umax64(wave_floor64(lm), 1ull);    // 0 is no key
            int n = 0;
            #pragma unroll
            for (int u = 0; u < CPL; ++u) {
                const bool pass = cand[u] >= fl;
                const unsigned long long mask = __ballot(pass);
                if (mask == 0ull) continue;              // wave-uniform
                const int at = n + below(mask);
                if (pass && at < kTbList) {
                    sh.list[wave][at] = cand[u];
                    sh.lcol[wave][at] = col[u];
                }
                n += __popcll(mask);
            }
            if constexpr (CPL * kWave > kTbList) {
                if (n > kTbList) {                       // by the narrower floor (k CPL keys at most)
                    const unsigned long long kfl = wave_kth64(lm, k);
                    n = 0;
                    #pragma unroll
                    for (int u = 0; u < CPL; ++u) {
                        const unsigned long long mask = __ballot(cand[u] >= kfl);
                        const int at = n + below(mask);
                        if (cand[u] >= kfl && at < kTbList) {
                            sh.list[wave][at] = cand[u];
                            sh.lcol[wave][at] = col[u];
                        }
                        n = min(n + __popcll(mask), kTbList);
                    }
                }
            }
            wave_lds_sync();
            list_winners(sh.list[wave], sh.lcol[wave], n, k, lane, false, nullptr, nullptr, sh.win[0][wave],
                         sh.wcol[0][wave]);
            if (lane < k) {                              // lane i: child i; a rank without a key has no token
                const unsigned long long key = sh.win[0][wave][lane];
                // exp, not exp_nonpos: a masked token's probability is 0 (or a
                // subnormal), and its rank among its equals is its place
                const double joint = key == 0ull ? 0.0 : sl.joint * (exp((double)key_value(key) - (double)m) / s);
                sh.joint[j * k + lane] = joint;
                sh.col[j * k + lane] = key == 0ull ? -1 : sh.wcol[0][wave][lane];
                if (writer) {
                    const size_t at = (size_t)b * max_nodes + base + j * k + lane;
                    node_tok[at] = key == 0ull ? -1 : key_index(key);
                    node_par[at] = sl.node;
                    node_joint[at] = joint;
                }
            }
        }
    }
    __syncthreads();
    // next frontier: the k children of this step with the largest joint
    // probabilities, largest first, ties to the earlier child. Child i's rank
    // is the number of children before it in that order.
    // tpc threads share child i's count (consecutive lanes, nc * tpc <= the
    // workgroup's threads), then add their parts.
    const int nc = nf * k;
    int tpc = 16;
    while (tpc > 1 && nc * tpc > kTbThreads) tpc >>= 1;
    {
        const int i = tid / tpc, part = tid % tpc;
        int rank = 0;
        double ji = 0.0;
        if (i < nc) {
            ji = sh.joint[i];
            const long long ki = joint_key(ji);
            for (int q = part; q < nc; q += tpc) {
                const long long kq = joint_key(sh.joint[q]);
                rank += (kq > ki || (kq == ki && q < i)) ? 1 : 0;
            }
        }
        rank = group_sum(rank, tpc);
        if (i < nc && part == 0 && rank < k) {
            const TbSlot sl = {base + i, sh.col[i], ji};
            sh.slot[rank] = sl;
            if (writer) next->slot[rank] = sl;
        }
    }
    if (tid == 0) {
        sh.nf = min(k, nc);
        if (writer) next->count = min(k, nc);
    }
    __syncthreads();
}

// LDS of a step workgroup: one of its roles.
template <int U>
struct StepShared {
    static constexpr int kCols = U * kWave;          // columns of one pass
    SelShared sel;
    double exp2[kExpTab];
    float x[kCols];                                  // the chunk's logits and vocabulary ids
    int id[kCols];
    u16x8 t[kTbWaves][kCols / 8];                    // a wave's table row, by its lanes' columns
};

struct StepArgs {
    const float *logits;
    const uint16_t *table;
    const int32_t *hot_vocab, *hot_index, *root_token, *accept_len;
    TbParts rows, parts_in, parts_out;
    const TbFrontier *fr_in;
    TbFrontier *fr_out;
    int32_t *node_tok, *node_par;
    double *node_joint;
    int r, S, V, H, k, kk, step, chunks, chunk_len, segs, seg_len, max_nodes;
};

// Step `step`, workgroups 0 .. B chunks - 1: the selection of the step before
// (at step 0 the frontier is the root), then the expansion of the frontier on
// one chunk of the hot columns, x = l_step[hot[c]] + table[row of the node's
// token][c], one wave per frontier node, in passes of 64 U columns (one pass
// unless there are more than 32 chunks of them). The chunk's logits are gathered
// once for all nodes, while the selection runs. Workgroup (b, chunk 0) stores
// what the selection found. parts and frontier are double buffered by the step's
// parity: this launch reads the step before's while it writes its own.
// The other B segs workgroups reduce this step's non-hot tokens (RU per thread).
// Bound by the chain partials -> children -> table row -> columns; two workgroups
// share a CU, so the second kind costs little beside the first.
template <int CPL, int U, int RU>
__global__ __launch_bounds__(kTbThreads, 4) void tb_step_kernel(StepArgs p) {
    constexpr int kCols = StepShared<U>::kCols;
    constexpr int kG = kCols / kTbThreads;           // columns gathered per thread
    __shared__ union Sh {
        __device__ Sh() {}
        StepShared<U> step;
        RowsShared rows;
    } shared;
    const int S = p.S, V = p.V, H = p.H, k = p.k, step = p.step, chunks = p.chunks;
    const int nexp = (int)gridDim.x / (chunks + p.segs) * chunks;
    if ((int)blockIdx.x >= nexp) {
        const int x = blockIdx.x - nexp, rb = x / p.segs, seg = x % p.segs;
        const TbWindow rw = tb_window(p.accept_len, rb, S, p.r);
        if (step >= rw.count) return;
        const size_t row = (size_t)rb * S + rw.first + step, at = row * p.segs + seg;
        const int v0 = seg * p.seg_len;
        reduce_row<RU>(shared.rows, p.logits + row * V, p.hot_index, V, H, k, p.kk, v0, min(V, v0 + p.seg_len),
                       p.rows.sum + at, p.rows.key + at * p.kk);
        return;
    }
    SelShared &sh = shared.step.sel;
    double *const s_exp2 = shared.step.exp2;
    float *const s_x = shared.step.x;
    int *const s_id = shared.step.id;
    const uint16_t *const table = p.table;
    const int32_t *const hot_vocab = p.hot_vocab;
    const int b = blockIdx.x / chunks, c = blockIdx.x % chunks, chunk_len = p.chunk_len;
    const TbWindow win = tb_window(p.accept_len, b, S, p.r);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    if (step == 0 && c == 0 && tid == 0) {           // the root
        const int t = p.root_token[b];
        const size_t at = (size_t)b * p.max_nodes;
        p.node_tok[at] = t;
        p.node_par[at] = -1;
        p.node_joint[at] = 1.0;
        p.fr_out[b].count = win.count > 0 ? 1 : 0;
        p.fr_out[b].slot[0] = TbSlot{0, hot_row(p.hot_index, t, V, H), 1.0};
    }
    const bool expand = step < win.count;
    const bool select = step > 0 && step - 1 < win.count;
    if (!expand && !(select && c == 0)) return;      // this sequence's tree is complete
    const int c0 = c * chunk_len, c1 = min(H, c0 + chunk_len);
    // (the last row stands in where there is nothing to expand)
    const float *l = p.logits + ((size_t)b * S + min(win.first + step, S - 1)) * V;
    int id[kG];
    float gx[kG];
    // Loads only: indices are clamped and what lies outside becomes -inf when
    // the columns are staged, so nothing waits here.
    auto load_ids = [&](int p0) {
        #pragma unroll
        for (int g = 0; g < kG; ++g) id[g] = hot_vocab[min(p0 + tid + g * kTbThreads, c1 - 1)];
    };
    auto gather = [&]() {
        #pragma unroll
        for (int g = 0; g < kG; ++g) gx[g] = l[(unsigned)id[g] < (unsigned)V ? id[g] : 0];
    };
    load_ids(c0);
    if (select) {
        select_step<CPL>(sh, p.rows, p.segs, p.parts_in, chunks, win, b, S, k, step - 1, p.max_nodes,
                         p.fr_in + b, p.fr_out + b, c == 0, s_exp2, p.node_tok, p.node_par, p.node_joint,
                         [&] {
                             gather();
                             fill_exp2_table(s_exp2);
                         });
        if (!expand) return;
    } else {
        const int h = tid == 0 ? hot_row(p.hot_index, p.root_token[b], V, H) : -1;
        gather();
        fill_exp2_table(s_exp2);
        if (tid == 0) {
            sh.nf = 1;
            sh.slot[0] = TbSlot{0, h, 1.0};
        }
        __syncthreads();
    }
    const int nf = sh.nf;
    const bool aligned = (H & 7) == 0 && (c0 & 7) == 0 && (reinterpret_cast<uintptr_t>(table) & 15) == 0;
    {
        const int j = wave;                          // k <= 8 here
        const int h = j < nf ? sh.slot[j].h : -1;
        const uint16_t *trow = table + (size_t)max(h, 0) * H;
        float M = kNegInf;
        double sum = 0.0;
        int cur = 0;                                 // which of sel.win holds the passes so far
        if (lane < kTbMaxK) sh.win[0][wave][lane] = 0ull;
        for (int p0 = c0; p0 < c1; p0 += kCols) {
            // lane's columns: p0 + 512 q + 8 lane + e
            u16x8 tv[U / 8];
            if (j < nf && h >= 0) {
                if (aligned) {                       // what lies past the chunk is not used
                    #pragma unroll
                    for (int q = 0; q < U / 8; ++q)
                        tv[q] = *reinterpret_cast<const u16x8 *>(trow + min(p0 + q * 512 + lane * 8, H - 8));
                } else {
                    #pragma unroll
                    for (int q = 0; q < U / 8; ++q)
                        #pragma unroll
                        for (int e = 0; e < 8; ++e) tv[q][e] = trow[min(p0 + q * 512 + lane * 8 + e, c1 - 1)];
                }
            } else {
                #pragma unroll
                for (int q = 0; q < U / 8; ++q) tv[q] = u16x8{0, 0, 0, 0, 0, 0, 0, 0};
            }
            if (p0 > c0) {                           // the first pass was gathered before
                load_ids(p0);
                gather();
                __syncthreads();                     // every wave is done with the previous pass
            }
            #pragma unroll
            for (int g = 0; g < kG; ++g) {
                const bool use = (unsigned)id[g] < (unsigned)V && p0 + tid + g * kTbThreads < c1;
                s_x[tid + g * kTbThreads] = use ? gx[g] : kNegInf;
                s_id[tid + g * kTbThreads] = id[g];
            }
            __syncthreads();
            if (j >= nf) continue;
            float xv[U];
            #pragma unroll
            for (int q = 0; q < U / 8; ++q) {
                const f32x4 a = *reinterpret_cast<const f32x4 *>(s_x + q * 512 + lane * 8);
                const f32x4 d = *reinterpret_cast<const f32x4 *>(s_x + q * 512 + lane * 8 + 4);
                #pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float x = e < 4 ? a[e] : d[e - 4];
                    xv[q * 8 + e] = h >= 0 ? x + __uint_as_float((unsigned)tv[q][e] << 16) : x;
                }
            }
            float lm = kNegInf;
            #pragma unroll
            for (int u = 0; u < U; ++u) lm = fmaxf(lm, xv[u]);
            const float pm = wave_allmax(lm);
            const bool more = p0 > c0;
            if (pm == kNegInf) continue;             // wave-uniform: no candidate
            const float fl = fmaxf(wave_floor(lm, p.kk), -__FLT_MAX__);     // -inf is no candidate
            unsigned bits = 0u;
            #pragma unroll
            for (int u = 0; u < U; ++u) bits |= xv[u] >= fl ? 1u << u : 0u;
            #pragma unroll
            for (int q = 0; q < U / 8; ++q) shared.step.t[wave][q * kWave + lane] = tv[q];
            // value of the pass's column cl, from LDS
            auto value_at = [&](int cl) {
                const unsigned t = reinterpret_cast<const uint16_t *>(shared.step.t[wave])[cl];
                return h >= 0 ? s_x[cl] + __uint_as_float(t << 16) : s_x[cl];
            };
            int n = 0;
            for (unsigned long long mask; (mask = __ballot(bits != 0u)) != 0ull && n <= kTbLong;) {
                const int at = n + below(mask);
                if (bits != 0u && at < kTbList) sh.lcol[wave][at] = (__builtin_ctz(bits) << 6) | lane;
                bits &= bits - 1u;
                n += __popcll(mask);
            }
            if (n > kTbLong) {
                // Many equal values at the floor (a node without a table row in a
                // masked vocabulary), or lanes without a column (fewer than 512): by
                // whole keys (k U at most).
                auto at_col = [&](int u) { return (u >> 3) * 512 + lane * 8 + (u & 7); };
                auto key = [&](int u) {
                    return xv[u] > kNegInf ? pack_key(order_key(xv[u]), (unsigned)s_id[at_col(u)]) : 0ull;
                };
                unsigned long long c = 0ull;
                #pragma unroll
                for (int u = 0; u < U; ++u) c = umax64(c, key(u));
                const unsigned long long kfl = wave_kth64(c, k);
                n = 0;
                #pragma unroll
                for (int u = 0; u < U; ++u) {
                    tie(xv[u]);                      // the first pass's tests are not kept
                    const unsigned long long x = key(u), mask = __ballot(x >= kfl);
                    const int at = n + below(mask);
                    if (x >= kfl && at < kTbList) {
                        sh.list[wave][at] = x;
                        sh.lcol[wave][at] = p0 + at_col(u);
                    }
                    n = min(n + __popcll(mask), kTbList);
                }
                wave_lds_sync();
            } else {
                wave_lds_sync();                     // the listed entries become keys
                for (int i = lane; i < n; i += kWave) {
                    const int e = sh.lcol[wave][i], u = e >> 6;
                    const int cl = (u >> 3) * 512 + (e & (kWave - 1)) * 8 + (u & 7);
                    sh.list[wave][i] = pack_key(order_key(value_at(cl)), (unsigned)s_id[cl]);
                    sh.lcol[wave][i] = p0 + cl;
                }
            }
            double ps = 0.0;
            #pragma unroll
            for (int u = 0; u < U; ++u) ps += exp_nonpos((double)xv[u] - (double)pm, s_exp2);
            ps = wave_allsum(ps);
            wave_lds_sync();
            list_winners(sh.list[wave], sh.lcol[wave], n, k, lane, more, sh.win[cur][wave], sh.wcol[cur][wave],
                         sh.win[cur ^ 1][wave], sh.wcol[cur ^ 1][wave]);
            cur ^= 1;
            merge_sum(M, sum, pm, ps, s_exp2);
        }
        if (j < nf) {
            const size_t at = ((size_t)b * k + j) * chunks + c;
            if (lane < p.kk) {
                p.parts_out.key[at * p.kk + lane] = sh.win[cur][wave][lane];
                p.parts_out.col[at * p.kk + lane] = sh.wcol[cur][wave][lane];
            }
            if (lane == 0) {
                p.parts_out.sum[at].s = sum;
                p.parts_out.sum[at].m = M;
            }
        }
    }
}

// The rows alone (no hot tokens): every (sequence, step), and the roots.
template <int RU>
__global__ __launch_bounds__(kTbThreads, 4) void tb_rows_kernel(StepArgs p) {
    __shared__ RowsShared sh;
    const int row = blockIdx.x, seg = blockIdx.y, b = row / p.S, step = row % p.S;
    const TbWindow win = tb_window(p.accept_len, b, p.S, p.r);
    if (seg == 0 && step == 0 && threadIdx.x == 0) {
        const size_t at = (size_t)b * p.max_nodes;
        p.node_tok[at] = p.root_token[b];
        p.node_par[at] = -1;
        p.node_joint[at] = 1.0;
        p.fr_out[b].count = win.count > 0 ? 1 : 0;
        p.fr_out[b].slot[0] = TbSlot{0, -1, 1.0};
    }
    if (step < win.first || step - win.first >= win.count) return;   // a row that no step uses
    const size_t at = (size_t)row * p.segs + seg;
    const int v0 = seg * p.seg_len;
    reduce_row<RU>(sh, p.logits + (size_t)row * p.V, nullptr, p.V, 0, p.k, p.kk, v0, min(p.V, v0 + p.seg_len),
                   p.rows.sum + at, p.rows.key + at * p.kk);
}

// One workgroup per sequence: the selections of steps from .. S - 1 (the last
// one, or all of them without hot tokens, where a step's children come from the
// row partials alone), then the `budget` nodes of largest joint probability
// (ties to the earlier node), in creation order, parents renumbered. The
// budget-th largest is found by a histogram over 1024 buckets of joint
// probability (32 per octave): better buckets are kept whole, the nodes of the
// bucket it falls in are ranked by counting.
template <int CPL>
__global__ __launch_bounds__(kTbThreads) void tb_finish_kernel(
    TbParts rows, int segs, TbParts parts0, TbParts parts1, int chunks, const int32_t *__restrict__ accept_len, int r,
    int S, int k, int from, int budget, int max_nodes, TbFrontier *fr0, TbFrontier *fr1,
    int32_t *node_tok, int32_t *node_par, double *node_joint, int32_t *__restrict__ parent,
    int32_t *__restrict__ token, float *__restrict__ joint, int32_t *__restrict__ num_nodes) {
    __shared__ SelShared sh;
    __shared__ double s_exp2[kExpTab];
    __shared__ int s_hist[kBuckets];
    __shared__ int s_warp[kTbWaves];
    __shared__ short s_new[kPruneSlots];
    __shared__ short s_mem[kPruneSlots];             // nodes of the threshold bucket,
    __shared__ long long s_mj[kPruneSlots];          // their joint probabilities' keys
    __shared__ int s_bucket, s_before, s_nmem;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const TbWindow win = tb_window(accept_len, b, S, r);
    for (int i = tid; i < kBuckets; i += kTbThreads) s_hist[i] = 0;
    if (tid == 0) s_nmem = 0;
    for (int step = from; step < S && step < win.count; ++step)
        select_step<CPL>(sh, rows, segs, (step & 1) ? parts1 : parts0, chunks, win, b, S, k, step, max_nodes,
                         ((step & 1) ? fr1 : fr0) + b, ((step & 1) ? fr0 : fr1) + b, true, s_exp2, node_tok,
                         node_par, node_joint, [&] { if (step == from) fill_exp2_table(s_exp2); });
    const size_t nb = (size_t)b * max_nodes;
    const int n = win.count < 0 ? 0 : win.count == 0 ? 1 : 1 + k + (win.count - 1) * k * k;
    const int kept = min(budget, n);
    constexpr int kPer = kPruneSlots / kTbThreads;   // consecutive nodes per thread
    // bucket 0 holds 1.0; 32 buckets per halving, everything below 2^-32 in the last
    auto bucket_of = [](double j) {
        const unsigned hi = (unsigned)((unsigned long long)__double_as_longlong(j) >> 32);
        return (int)min((0x3FF00000u - min(hi, 0x3FF00000u)) >> 15, (unsigned)(kBuckets - 1));
    };
    double jn[kPer];
    const int i0 = tid * kPer;
    __syncthreads();
    #pragma unroll
    for (int u = 0; u < kPer; ++u) jn[u] = i0 + u < n ? node_joint[nb + i0 + u] : 0.0;
    #pragma unroll
    for (int u = 0; u < kPer; ++u)
        if (i0 + u < n) atomicAdd(&s_hist[bucket_of(jn[u])], 1);
    __syncthreads();
    // inclusive prefix over the buckets, two per thread: the one holding the
    // kept-th node
    constexpr int kBpt = kBuckets / kTbThreads;
    int f[kBpt], run = 0;
    #pragma unroll
    for (int u = 0; u < kBpt; ++u) { f[u] = s_hist[tid * kBpt + u]; run += f[u]; }
    auto block_exclusive = [&](int total) {          // exclusive prefix of `total` over the threads
        int incl = total;
        #pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int o = __shfl_up(incl, off);
            if (lane >= off) incl += o;
        }
        if (lane == kWave - 1) s_warp[wave] = incl;
        __syncthreads();
        int before = incl - total;
        for (int q = 0; q < wave; ++q) before += s_warp[q];
        __syncthreads();
        return before;
    };
    int before = block_exclusive(run);
    #pragma unroll
    for (int u = 0; u < kBpt; ++u) {
        if (before < kept && before + f[u] >= kept) { s_bucket = tid * kBpt + u; s_before = before; }
        before += f[u];
    }
    __syncthreads();
    const int tb = kept > 0 ? s_bucket : -1, left = kept > 0 ? kept - s_before : 0;
    #pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int i = i0 + u;
        if (i >= n) continue;
        const int bk = bucket_of(jn[u]);
        s_new[i] = bk < tb ? 1 : 0;
        if (bk == tb) {
            const int at = atomicAdd(&s_nmem, 1);
            s_mem[at] = (short)i;
            s_mj[at] = joint_key(jn[u]);
        }
    }
    __syncthreads();
    const int nm = s_nmem;
    if (tid < 8 && nm + tid < kPruneSlots) s_mj[nm + tid] = LLONG_MIN;   // below every node's
    __syncthreads();
    for (int x = tid; x < nm; x += kTbThreads) {
        const int i = s_mem[x];
        const long long ki = s_mj[x];
        int rank = 0;
        for (int q = 0; q < nm && rank < left; q += 8) {     // eight reads in flight together
            long long kq[8];
            int iq[8];
            #pragma unroll
            for (int u = 0; u < 8; ++u) {
                kq[u] = s_mj[q + u];
                iq[u] = s_mem[q + u];
            }
            #pragma unroll
            for (int u = 0; u < 8; ++u) rank += (kq[u] > ki) | ((kq[u] == ki) & (iq[u] < i));
        }
        if (rank < left) s_new[i] = 1;
    }
    __syncthreads();
    // ranks in creation order
    int g[kPer];
    run = 0;
    #pragma unroll
    for (int u = 0; u < kPer; ++u) { g[u] = i0 + u < n ? s_new[i0 + u] : 0; run += g[u]; }
    before = block_exclusive(run);
    #pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (i0 + u < n) s_new[i0 + u] = g[u] ? (short)before : (short)-1;
        before += g[u];
    }
    __syncthreads();
    #pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int i = i0 + u;
        if (!g[u]) continue;
        const int ni = s_new[i], pp = node_par[nb + i];
        parent[(size_t)b * budget + ni] = pp < 0 ? -1 : s_new[pp];
        token[(size_t)b * budget + ni] = node_tok[nb + i];
        joint[(size_t)b * budget + ni] = (float)jn[u];
    }
    for (int i = kept + tid; i < budget; i += kTbThreads) {
        parent[(size_t)b * budget + i] = -1;
        token[(size_t)b * budget + i] = -1;
        joint[(size_t)b * budget + i] = 0.f;
    }
    if (tid == 0) num_nodes[b] = kept;
}

// Workgroups that fill the chip.
constexpr int kFill = 256;

// Parts of n entries, `per` in each.
long parts_of(long n, long per) {
    const long x = (n + per - 1) / per;
    return n <= 0 ? 0l : x > kMaxParts ? (long)kMaxParts : x;
}

// Whether a step is one launch, or its launches are separate (tree_build_many.hip).
// Without hot tokens there are no steps to launch, and these kernels win up to 8
// branches (256 sequences of 32000 tokens, 5 steps, k 4: 70 against 95 us). With
// more branches, nodes and selection would take two rounds per wave (k 10, 16
// sequences 297 against 231 us). Otherwise one launch saves about 10 us per step
// while its workgroups run at once, two per CU; past that every further round
// repeats the selection in each of its workgroups and fills few of its waves, as
// many as there are branches, and the segments' reductions, which weigh more than
// the chunks, no longer run beside something that waits. Measured (us, one launch
// per step / separate launches; 7 steps; segments + chunks per sequence):
//   16 + 16 (128256 tokens, 32768 hot), k 8: 16 sequences 154 / 186, 32 275 / 295;
//     k 4: 32 sequences 237 / 229; k 2: 8 sequences 97 / 106, 16 136 / 129, 32 234 / 203;
//   19 + 16 (151936, 32768), k 4: 8 sequences 120 / 123, 16 181 / 153;
//   16 + 4 (128256, 8192), k 4: 16 sequences 108 / 119, 24 156 / 131; k 8: 16
//     117 / 146, 64 286 / 236.
// Where the chunks are most of it (all of 32000 tokens hot: 4 + 16), or with 7 and 8
// branches as many, separate launches pass over them too often: k 4, 32 sequences
// 147 / 158, 64 232 / 272; 16 + 16, k 8, 64 sequences 475 / 503. (The first step has
// one node to expand, which costs separate launches little: with one or two steps
// only up to two rounds of workgroups; 16 + 16, k 8, 64 sequences, 2 steps 1.10 times.) And
// re-sampled trees use one launch per step: separate launches reduce the rows of
// the accepted positions too and cannot tell how many steps remain (32 sequences of
// 128256 tokens, 32768 hot, k 4, 1 to 4 positions accepted: 187 / 226).
bool one_launch_per_step(bool resample, int B, int S, int V, int H, int k) {
    if (k > kMaxBranches) return false;
    const long segs = parts_of(V, 16 * kTbThreads), chunks = parts_of(H, 32 * kWave);
    const long wgs = B * (segs + chunks), weight = B * (4 * segs + chunks);
    if (resample || chunks == 0) return true;
    if (((chunks >= segs && k >= 7) || (chunks >= 2 * segs && k >= 3)) && (S >= 3 || wgs <= 4 * kFill)) return true;
    if (k >= 7) return weight <= 214 * (k + 4);
    return 2 * chunks < segs ? wgs <= 440 : wgs <= 2 * kFill && weight <= 200 * (k + 4);
}

}  // namespace

TreeBuildPlan tree_build_plan(int B, int S, int V, int H, int k) {
    TreeBuildPlan pl;
    const long rows = (long)B * S;
    // Tokens of a rows workgroup: 16 per thread, or 4 while that leaves CUs idle
    // (and needs no more than 32 segments). Columns of a step workgroup: 32 per
    // lane, or 16 likewise. Measured (us, 5 steps, small against large): tokens, 32000
    // and none hot, k 8, 3 sequences 29.8 against 31.9, but k 4, 12 sequences 30.8
    // against 28.8 (with hot tokens a step does not wait for its rows: no
    // difference); columns, 32000 tokens all hot, k 4, 3 sequences 54 against 60, 6
    // 60 against 67; 128256 tokens, 8192 hot, k 8, 6 sequences 71 against 80, but
    // 32768 hot, k 4, 6 sequences 79 against 75.
    // Small ones only while a selection's keys stay 4 per lane, so that one instance
    // has 8. (With small parts and 8 keys: 128256 tokens, 32768 hot, k 8, 1 sequence
    // 74 -> 65, 3 84 -> 73, 6 84 -> 87.)
    pl.kk = k <= 1 ? 1 : k <= 2 ? 2 : k <= 4 ? 4 : 8;
    const bool small_r = (long)B * parts_of(V, 16 * kTbThreads) < kFill / 2 && (long)V <= 4l * kTbThreads * kMaxParts;
    const bool small_c = (long)B * parts_of(H, 32 * kWave) < kFill / 2 && (long)H <= 16l * kWave * kMaxParts;
    auto keys = [&](bool sr, bool sc) {
        return (parts_of(V, (sr ? 4 : 16) * kTbThreads) + parts_of(H, (sc ? 16 : 32) * kWave)) * pl.kk;
    };
    const bool sr = small_r && keys(true, false) <= 4 * kWave;
    const bool sc = small_c && keys(sr, true) <= 4 * kWave;
    pl.row_u = sr ? 4 : 16;
    pl.col_u = sc ? 16 : 32;
    const long segs = parts_of(V, (long)pl.row_u * kTbThreads);
    pl.segs = (int)segs;
    pl.seg_len = (int)(((long)V + segs - 1) / segs);
    const long chunks = parts_of(H, (long)pl.col_u * kWave);
    pl.chunks = (int)chunks;
    // a multiple of 8 columns, for the wide table loads
    pl.chunk_len = chunks > 0 ? (int)((((long)H + chunks - 1) / chunks + 7) / 8 * 8) : 0;
    pl.max_nodes = 1 + k + (S - 1) * k * k;
    // workspace: as many parts as any split of these sizes has, and enough for
    // either builder, so that it does not grow for a smaller call
    pl.row_parts = (size_t)rows * parts_of(V, 4 * kTbThreads);
    pl.col_parts = (size_t)B * k * parts_of(H, 16 * kWave);
    pl.frontier_bytes = (size_t)B * sizeof(TbFrontier);
    pl.bytes = 256;
    auto add = [&](size_t bytes) { pl.bytes += (bytes + 255) & ~(size_t)255; };
    add(pl.row_parts * sizeof(TbSum));
    add(pl.row_parts * pl.kk * sizeof(unsigned long long));
    for (int i = 0; i < 2; ++i) {
        add(pl.col_parts * sizeof(TbSum));
        add(pl.col_parts * pl.kk * sizeof(unsigned long long));
        add(pl.col_parts * pl.kk * sizeof(int32_t));
        add(pl.frontier_bytes);
    }
    const size_t nn = (size_t)B * pl.max_nodes;
    add(nn * sizeof(int32_t));
    add(nn * sizeof(int32_t));
    add(nn * sizeof(double));
    pl.bytes = std::max(pl.bytes, tree_build_many_bytes(B, S, V, H, k));
    return pl;
}

hipError_t launch_tree_build(const float *logits, const int32_t *root_token,
                             const uint16_t *table, const int32_t *hot_vocab,
                             const int32_t *hot_index, const int32_t *accept_len, int r, int B,
                             int S, int V, int H, int k, int budget, int32_t *parent,
                             int32_t *token, float *joint, int32_t *num_nodes, void *workspace,
                             hipStream_t s) {
    if (B == 0) return hipSuccess;
    if (!one_launch_per_step(accept_len != nullptr, B, S, V, H, k))
        return launch_tree_build_many(logits, root_token, table, hot_vocab, hot_index, accept_len, r, B, S, V, H, k,
                                      budget, parent, token, joint, num_nodes, workspace, s);
    const TreeBuildPlan pl = tree_build_plan(B, S, V, H, k);
    char *base = static_cast<char *>(workspace);
    auto carve = [&](size_t bytes) {
        char *p = base;
        base += (bytes + 255) & ~(size_t)255;
        return p;
    };
    auto carve_parts = [&](size_t parts, bool cols) {
        TbParts t;
        t.sum = reinterpret_cast<TbSum *>(carve(parts * sizeof(TbSum)));
        t.key = reinterpret_cast<unsigned long long *>(carve(parts * pl.kk * sizeof(unsigned long long)));
        t.col = cols ? reinterpret_cast<int *>(carve(parts * pl.kk * sizeof(int32_t))) : nullptr;
        return t;
    };
    const TbParts rows = carve_parts(pl.row_parts, false);
    TbParts parts[2];
    TbFrontier *frontier[2];
    for (auto &t : parts) t = carve_parts(pl.col_parts, true);
    const size_t nn = (size_t)B * pl.max_nodes;
    int32_t *node_tok = reinterpret_cast<int32_t *>(carve(nn * sizeof(int32_t)));
    int32_t *node_par = reinterpret_cast<int32_t *>(carve(nn * sizeof(int32_t)));
    double *node_joint = reinterpret_cast<double *>(carve(nn * sizeof(double)));
    for (auto &f : frontier) f = reinterpret_cast<TbFrontier *>(carve(pl.frontier_bytes));

    // candidate keys per lane of a selection: (segs + chunks) parts of kk keys
    const int per_lane = ((pl.segs + pl.chunks) * pl.kk + kWave - 1) / kWave;
    StepArgs a{logits, table, hot_vocab, hot_index, root_token, accept_len, rows, parts[1], parts[0],
               frontier[1], frontier[0], node_tok, node_par, node_joint, r, S, V, H, k, pl.kk, 0,
               pl.chunks, pl.chunk_len, pl.segs, pl.seg_len, pl.max_nodes};
    hipError_t e = hipSuccess;
    if (pl.chunks == 0) {
        e = launch_kernel(pl.row_u == 16 ? tb_rows_kernel<16> : tb_rows_kernel<4>, dim3(B * S, pl.segs),
                          dim3(kTbThreads), s, a);
    }
    if (pl.chunks > 0) {
        auto sk = per_lane > 4     ? tb_step_kernel<8, 32, 16>       // the plan has no small parts then
                  : pl.col_u == 32 ? (pl.row_u == 16 ? tb_step_kernel<4, 32, 16> : tb_step_kernel<4, 32, 4>)
                                   : (pl.row_u == 16 ? tb_step_kernel<4, 16, 16> : tb_step_kernel<4, 16, 4>);
        for (int i = 0; i < S && e == hipSuccess; ++i) {
            a.step = i;
            a.parts_in = parts[(i + 1) & 1];
            a.parts_out = parts[i & 1];
            a.fr_in = frontier[(i + 1) & 1];
            a.fr_out = frontier[i & 1];
            e = launch_kernel(sk, dim3(B * (pl.chunks + pl.segs)), dim3(kTbThreads), s, a);
        }
    }
    if (e == hipSuccess)
        e = launch_kernel(per_lane <= 4 ? tb_finish_kernel<4> : tb_finish_kernel<8>, dim3(B), dim3(kTbThreads), s,
                          rows, pl.segs, parts[0], parts[1], pl.chunks, accept_len, r, S, k,
                          pl.chunks > 0 ? S - 1 : 0, budget, pl.max_nodes, frontier[0], frontier[1],
                          node_tok, node_par, node_joint, parent, token, joint, num_nodes);
    return e;
}

}  // namespace tv
