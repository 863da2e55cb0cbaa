// What the tree builder's kernels share (tree_build.hip, tree_build_many.hip):
// keys, cross-lane reductions, the double-precision exponential of the sums and
// the steps of a sequence.
#pragma once

#include "tv_internal.h"

namespace tv {
namespace {

constexpr int kExpTab = 64;                // entries of exp_nonpos's table
constexpr float kNegInf = -__builtin_huge_valf();

// Joint probabilities in the order the builder ranks them by. They are not
// negative, so their bits order as they do, and a NaN (only logits that are not
// finite give one) has a place in the order too: ranks by counting are always a
// permutation, so no slot or node that a later step indexes by stays unwritten.
__device__ __forceinline__ long long joint_key(double j) { return __double_as_longlong(j); }

// Hot row of token t (-1 when it has none).
__device__ __forceinline__ int hot_row(const int32_t *hot_index, int t, int V, int H) {
    int h = (H > 0 && t >= 0 && t < V) ? hot_index[t] : -1;
    return h >= H ? -1 : h;
}

__device__ __forceinline__ unsigned long long umax64(unsigned long long a, unsigned long long b) {
    return a > b ? a : b;
}

__device__ __forceinline__ float key_value(unsigned long long key) {
    const unsigned int k = (unsigned int)(key >> 32);
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

__device__ __forceinline__ int key_index(unsigned long long key) {
    return (int)(0xFFFFFFFFu - (unsigned int)key);
}

// Cross-lane helpers without LDS.
__device__ __forceinline__ unsigned long long readlane64(unsigned long long v, int src) {
    const unsigned int lo = __builtin_amdgcn_readlane((int)(unsigned int)v, src);
    const unsigned int hi = __builtin_amdgcn_readlane((int)(unsigned int)(v >> 32), src);
    return ((unsigned long long)hi << 32) | lo;
}

template <int C>
__device__ __forceinline__ unsigned int dpp32(unsigned int v) {
    return (unsigned int)__builtin_amdgcn_update_dpp((int)v, (int)v, C, 0xF, 0xF, false);
}

// Largest 64-bit key over the wave, by a scan of per-row maxima (no LDS).
__device__ __forceinline__ unsigned long long wave_max64(unsigned long long v) {
    #pragma unroll
    for (int sh = 1; sh < 16; sh <<= 1) {        // row_shr:sh; lanes below sh keep their value
        const int lo = (int)(unsigned int)v, hi = (int)(unsigned int)(v >> 32);
        const unsigned int nlo = sh == 1 ? __builtin_amdgcn_update_dpp(lo, lo, 0x111, 0xF, 0xF, false)
                               : sh == 2 ? __builtin_amdgcn_update_dpp(lo, lo, 0x112, 0xF, 0xF, false)
                               : sh == 4 ? __builtin_amdgcn_update_dpp(lo, lo, 0x114, 0xF, 0xF, false)
                                         : __builtin_amdgcn_update_dpp(lo, lo, 0x118, 0xF, 0xF, false);
        const unsigned int nhi = sh == 1 ? __builtin_amdgcn_update_dpp(hi, hi, 0x111, 0xF, 0xF, false)
                               : sh == 2 ? __builtin_amdgcn_update_dpp(hi, hi, 0x112, 0xF, 0xF, false)
                               : sh == 4 ? __builtin_amdgcn_update_dpp(hi, hi, 0x114, 0xF, 0xF, false)
                                         : __builtin_amdgcn_update_dpp(hi, hi, 0x118, 0xF, 0xF, false);
        v = umax64(v, ((unsigned long long)nhi << 32) | nlo);
    }
    // lane 15 of every row now holds its row's maximum
    return umax64(umax64(readlane64(v, 15), readlane64(v, 31)),
                  umax64(readlane64(v, 47), readlane64(v, 63)));
}

// Whole-wave reductions without LDS: butterflies inside each row of 16 lanes
// by DPP (swap neighbours, swap pairs, mirror each half row, mirror the row:
// after each step every lane of the group holds the group's result), then
// across rows by the row-pair and half-wave swaps. Every lane ends with the
// result.
template <int C>
__device__ __forceinline__ double dpp64(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned int lo = dpp32<C>((unsigned int)b), hi = dpp32<C>((unsigned int)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

__device__ __forceinline__ float wave_allmax(float v) {
    v = fmaxf(v, __uint_as_float(dpp32<kDppXor1>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(dpp32<kDppXor2>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(dpp32<kDppHalfMirror>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(dpp32<kDppMirror>(__float_as_uint(v))));
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
}

__device__ __forceinline__ double wave_allsum(double v) {
    v += dpp64<kDppXor1>(v);
    v += dpp64<kDppXor2>(v);
    v += dpp64<kDppHalfMirror>(v);
    v += dpp64<kDppMirror>(v);
    #pragma unroll
    for (int half = 0; half < 2; ++half) {         // row pairs, then the wave's halves
        const unsigned long long b = (unsigned long long)__double_as_longlong(v);
        const unsigned int lo = (unsigned int)b, hi = (unsigned int)(b >> 32);
        const auto l = half == 0 ? __builtin_amdgcn_permlane16_swap(lo, lo, false, false)
                                 : __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = half == 0 ? __builtin_amdgcn_permlane16_swap(hi, hi, false, false)
                                 : __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        v = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
            __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
    }
    return v;
}

// Sum over aligned groups of n consecutive lanes (n = 1, 2, 4, 8 or 16,
// wave-uniform); every lane of a group ends with the group's sum.
__device__ __forceinline__ int group_sum(int v, int n) {
    if (n >= 2) v += (int)dpp32<kDppXor1>((unsigned int)v);
    if (n >= 4) v += (int)dpp32<kDppXor2>((unsigned int)v);
    if (n >= 8) v += (int)dpp32<kDppHalfMirror>((unsigned int)v);
    if (n >= 16) v += (int)dpp32<kDppMirror>((unsigned int)v);
    return v;
}

// 2^(j/64), j = 0..63, rounded to nearest.
__device__ const double kExp2Table[kExpTab] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0,
    0x1.0874518759bc8p+0, 0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0,
    0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0, 0x1.172b83c7d517bp+0,
    0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0,
    0x1.2d285a6e4030bp+0, 0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0,
    0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0, 0x1.3dea64c123422p+0,
    0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0,
    0x1.56f4736b527dap+0, 0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0,
    0x1.6247eb03a5585p+0, 0x1.6623882552225p+0, 0x1.6a09e667f3bcdp+0,
    0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0,
    0x1.868d99b4492edp+0, 0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0,
    0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0, 0x1.9c49182a3f090p+0,
    0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0,
    0x1.bcc1e904bc1d2p+0, 0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0,
    0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0, 0x1.d5818dcfba487p+0,
    0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0,
    0x1.fa7c1819e90d8p+0,
};

// exp(x) for x <= 0 in double precision, by Tang's table-driven method (ACM
// TOMS 15(2), 1989): x = (64 n + j) ln2/64 + r with |r| <= ln2/128, so
// e^x = 2^n 2^(j/64) e^r; e^r - 1 from its degree-5 Taylor polynomial
// (truncation below 4e-17 on that interval); 2^(j/64) from a table (tab, a copy
// of kExp2Table in LDS). ln2/64 is split into kL1 (its 37 leading significant
// bits, so N kL1 is exact for |N| < 2^16) and kL2 = ln2/64 - kL1 rounded to
// double. N is rounded by adding 1.5 2^52, whose low word then holds it.
// For sums only: arguments below -700 (and -inf, NaN) count as -700: 1e-304, below any
// rounding of a sum whose largest term is 1. About 1 ulp.
__device__ __forceinline__ double exp_nonpos(double x, const double *tab) {
    const double kInvL = 92.33248261689366;          // 64 / ln2
    const double kL1 = 0.010830424696223417;
    const double kL2 = 2.572804622327669e-14;
    const double kRound = 6755399441055744.0;
    x = __builtin_fmax(x, -700.0);
    const double z = __builtin_fma(x, kInvL, kRound);
    const double N = z - kRound;
    double r = __builtin_fma(-N, kL1, x);
    r = __builtin_fma(-N, kL2, r);
    double q = __builtin_fma(r, 1.0 / 120.0, 1.0 / 24.0);
    q = __builtin_fma(q, r, 1.0 / 6.0);
    q = __builtin_fma(q, r, 0.5);
    q = __builtin_fma(q, r, 1.0);
    q *= r;                                          // e^r - 1
    const unsigned int n = (unsigned int)__double_as_longlong(z);
    const unsigned long long t0 = (unsigned long long)__double_as_longlong(tab[n & (kExpTab - 1)]);
    const unsigned int hi = (unsigned int)(t0 >> 32) + ((n << 14) & 0xFFF00000u);
    const double t = __longlong_as_double((long long)(((unsigned long long)hi << 32) | (unsigned int)t0));
    return __builtin_fma(t, q, t);
}

// The table into LDS for exp_nonpos; the caller synchronises.
__device__ __forceinline__ void fill_exp2_table(double *tab) {
    if (threadIdx.x < kExpTab) tab[threadIdx.x] = kExp2Table[threadIdx.x];
}

// Steps of sequence b: logits rows [first, first + count). A first tree uses all
// S rows. A re-sampled tree (Alg. 2; accept_len given) starts after the first
// rejected position -- the accepted path counts the root, so that position is
// accept_len and the remaining rows are accept_len .. S-1 -- and is the single
// ground-truth node unless more than r rows remain. A sequence that verified
// nothing has no tree (count -1).
struct TbWindow {
    int first, count;
};

__device__ __forceinline__ TbWindow tb_window(const int32_t *accept_len, int b, int S, int r) {
    if (!accept_len) return {0, S};
    const int a = accept_len[b];
    if (a <= 0) return {0, -1};
    const int remain = S - a;
    return {min(a, S), remain > r ? remain : 0};
}

}  // namespace
}  // namespace tv
