// LM head fused with the vocabulary argmax for gfx950: greedy verification
// without materialised logits.
//
// The target model's logit of tree node row r and vocabulary entry v is the
// dot product of the row's final hidden state with row v of the LM-head
// weight (the logits of many nodes are one matrix product, as the paper does
// on the draft side, §4.2), and greedy verification (§7.1: temperature 0;
// accepted path and bonus token, §5.3) needs only each row's argmax. This
// kernel computes hidden x W^T tile by tile on the matrix cores and reduces
// every tile straight to one 64-bit key per row, with the ordering of the
// stand-alone argmax (larger value first, NaN above everything, -0 == +0,
// lower id on ties), so the [rows, V] fp32 logits never exist in memory.
//
// Two kernels: up to 128 rows the call is a stream of the weight
// (lm_head_stream_kernel, described there); more rows take a tiled matrix
// product (lm_head_argmax_kernel):
//
//   * Tile: 256 vocabulary entries (MFMA M) x 256 hidden rows (MFMA N), the
//     largest whose fp32 accumulators fit a CU's registers. Four waves, one per
//     SIMD, in a 2 x 2 arrangement, each accumulating a 128 x 128 block in 16
//     v_mfma_f32_32x32x16_bf16 accumulators (256 registers): a wave's LDS reads
//     per MFMA are a third less than with eight waves of 128 x 64, whose reads
//     and incoming lines together need the LDS for as long as the products need
//     the matrix cores.
//   * Both operands are K-contiguous (W is [V, d], hidden is [R, d]) and both
//     stream into LDS through global_load_lds_dwordx4 in 64-deep units (each
//     row's 128 bytes = whole cache lines; a 1 KB load covers 8 rows): the
//     weight, whose load latency bounds the stream, through a 3-stage ring, the
//     hidden rows, re-read from L2, through a 2-stage ring. Together 160 KB: the
//     whole LDS. The 16-byte chunks of each row are XOR-swizzled by the row
//     index so the operand reads are free of bank conflicts.
//   * One barrier per unit. Each 16-deep K step's 16 MFMAs carry the next step's
//     8 fragment reads and a quarter of the unit's loads.
//   * One workgroup per CU walks its tiles without draining the rings between
//     them; its best keys stay in registers while its row block stays the same.
//   * The four row blocks of one vocabulary tile run together on one XCD and
//     share its L2 copy of the weight tile; each takes the units of every
//     aligned group of four in an order rotated by its row block, so the four
//     ask HBM for different lines at any time (more distinct bytes in flight)
//     and find the others' lines in L2 a few units later.
//   * A tile's values become keys by a maximum and then a search for its lowest
//     entry (fold below); lanes l and l ^ 32 combine, and a 64-bit atomic
//     maximum per row merges waves and workgroups into the row's key, which the
//     greedy acceptance kernel then decodes.
// Measured at 1024 rows x 128256 x 4096: 835 us (1290 TFLOP/s, matrix pipe busy
// 75 % of the cycles) against 898-915 us (66 %) for eight waves, one tile per
// workgroup and a 64-bit compare per value. Of the rest, about 130 us is the
// issue of the loads: without them the same loop takes 707 us.
#include "tv_internal.h"

namespace tv {
namespace {

#define LDS_AS __attribute__((address_space(3)))
#define GLOBAL_AS __attribute__((address_space(1)))

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;                              // one per SIMD
constexpr int kLmThreads = kWaves * kWave;
constexpr int kTileM = 256;                            // vocabulary entries per workgroup
constexpr int kTileN = 256;                            // hidden rows per workgroup
constexpr int kUnitK = 64;                             // K depth of one weight unit
constexpr int kWRow = kUnitK * 2;                      // bytes of one weight row's unit (128)
constexpr int kWUnitBytes = kTileM * kWRow;            // 32 KB
constexpr int kWStages = 3;
constexpr int kHStages = 2;
constexpr int kLoads = kWUnitBytes / (kLmThreads * 16);     // 1 KB loads per wave and unit, each operand
constexpr int kWaveM = 128, kWaveN = 128;              // per-wave block: 2 x 2 waves
constexpr int kFragM = kWaveM / 32, kFragN = kWaveN / 32;
constexpr int kReads = kFragM + kFragN;                // fragment reads per K step
constexpr int kSteps = kFragM * kFragN;                // MFMAs per K step
constexpr int kPre = 2;                                // MFMAs before the hand-off
constexpr int kStreamRows = 128;                       // most rows of lm_head_stream_kernel
static_assert(kLoads * kWaves * 8 == kTileM && kTileM == kTileN && kFragM == kFragN, "load blocks");
static_assert((kWStages + kHStages) * kWUnitBytes <= 160 * 1024, "LDS");

__shared__ __attribute__((aligned(1024))) unsigned char g_lm_w[kWStages * kWUnitBytes];
__shared__ __attribute__((aligned(1024))) unsigned char g_lm_h[kHStages * kWUnitBytes];

__device__ __forceinline__ unsigned lds_addr(const void *p) {
    return (unsigned)(size_t)(const LDS_AS void *)p;
}

template <typename T>
__device__ __forceinline__ void tie(T &x) {
    asm volatile("" : "+v"(x));
}

__device__ __forceinline__ void lds_wait_all() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// s_waitcnt vmcnt(N) (gfx9 encoding: vmcnt in [3:0] and [15:14]).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

__device__ __forceinline__ unsigned long long umax64(unsigned long long a, unsigned long long b) {
    return a > b ? a : b;
}

// Maximum of three values, NaN if any is NaN.
__device__ __forceinline__ float maximum3(float a, float b, float c) {
    float r;
    asm("v_maximum3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Maximum of a 64-bit key held by lanes l and l ^ 32.
__device__ __forceinline__ unsigned long long halves_max64(unsigned long long x) {
    const unsigned lo = (unsigned)x, hi = (unsigned)(x >> 32);
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    const unsigned long long a = ((unsigned long long)h[0] << 32) | l[0];
    const unsigned long long b = ((unsigned long long)h[1] << 32) | l[1];
    return umax64(a, b);
}

// Maximum of a 64-bit key held by lanes l and l ^ 16.
__device__ __forceinline__ unsigned long long rows_max64(unsigned long long x) {
    const unsigned lo = (unsigned)x, hi = (unsigned)(x >> 32);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    const unsigned long long a = ((unsigned long long)h[0] << 32) | l[0];
    const unsigned long long b = ((unsigned long long)h[1] << 32) | l[1];
    return umax64(a, b);
}

__global__ void lm_keys_clear_kernel(unsigned long long *__restrict__ keys, int R) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < R) keys[i] = 0ull;                  // below every real key
}

// Workgroups: any number; `groups` = kNumXcd * ceil(vtiles / kNumXcd) * rblocks
// tiles. d is a multiple of kUnitK.
__global__ __launch_bounds__(kLmThreads, 1) void lm_head_argmax_kernel(
    const uint16_t *__restrict__ hidden, const uint16_t *__restrict__ w, int R, int V, int d,
    int vtiles, int rblocks, int groups, unsigned long long *__restrict__ keys) {
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid & (kWave - 1);
    const int U = d / kUnitK;
    const int step_id = gridDim.x;
    // Tile `id`: vocabulary tile and row block. Ids past the last vocabulary
    // tile (the last group of eight) are empty and skipped.
    auto vt_of = [&](int id) { return (id / kNumXcd / rblocks) * kNumXcd + id % kNumXcd; };
    auto rb_of = [&](int id) { return (id / kNumXcd) % rblocks; };
    auto next_id = [&](int id) {
        do id += step_id; while (id < groups && vt_of(id) >= vtiles);
        return id;
    };
    const int first = next_id((int)blockIdx.x - step_id);
    if (first >= groups) return;                 // whole workgroup, before any barrier
    int total = 0;                               // units of this workgroup
    for (int id = first; id < groups; id = next_id(id)) total += U;

    // Loads: instruction i of wave w fills 1 KB block (8w + i) of a weight or
    // hidden unit = rows 8 (8w + i) .. +7; lane p writes row p / 8, position
    // p % 8, which holds chunk (p % 8) ^ ((row >> 1) & 7). Rows past the end of
    // W or hidden read the last row (finite data; the results are discarded).
    // A cursor is an operand's unit to load next: wave-uniform state only (the
    // lane's offset is computed behind each MFMA that a load follows; d < 2^23,
    // so it fits 32 bits and the factors 24).
    int lrow = wave * kLoads * 8 + (lane >> 3);
    unsigned lchunk0 = (unsigned)(((lane & 7) ^ ((lane >> 4) & 3)) << 4);   // rows 8 (8w + i) + .., i even
    const unsigned rowb = (unsigned)d * 2;
    // Unit order: inside every complete aligned group of four, rotated by the
    // row block (a permutation of 0 .. U - 1).
    const int U4 = U & ~3;
    struct Cursor {
        const char *base, *at;                           // the tile's first row; the unit in it
        int last;                                        // the tile's last existing row
        int id, u, rb;
        unsigned stage;                                  // LDS byte offset
    } cw, ch;
    auto set_unit = [&](Cursor &c) {
        c.at = c.base + (size_t)(c.u < U4 ? (c.u & ~3) | ((c.u + c.rb) & 3) : c.u) * kWRow;
    };
    auto set_tile = [&](Cursor &c, const uint16_t *p, int r0, int rows) {
        c.rb = rb_of(c.id);
        c.base = reinterpret_cast<const char *>(p) + (size_t)r0 * rowb;
        c.last = rows - 1 - r0;
    };
    auto set_w = [&]() { set_tile(cw, w, vt_of(cw.id) * kTileM, V); };
    auto set_h = [&]() { set_tile(ch, hidden, rb_of(ch.id) * kTileN, R); };
    auto issue = [&](const Cursor &c, unsigned char *ring, int i) {
        const unsigned row = (unsigned)min(lrow + 8 * i, c.last);
        const unsigned off = __umul24(row, rowb) + (lchunk0 ^ (unsigned)((i & 1) << 6));
        __builtin_amdgcn_global_load_lds((const GLOBAL_AS void *)(c.at + off),
                                         (LDS_AS void *)(ring + c.stage + (wave * kLoads + i) * 1024), 16, 0, 0);
    };
    auto issue_w = [&](int i) { issue(cw, g_lm_w, i); };
    auto issue_h = [&](int i) { issue(ch, g_lm_h, i); };
    auto advance_w = [&]() {
        cw.stage = cw.stage == (kWStages - 1) * kWUnitBytes ? 0 : cw.stage + kWUnitBytes;
        if (++cw.u == U) {
            cw.u = 0;
            cw.id = next_id(cw.id);
            if (cw.id < groups) set_w();
        }
        set_unit(cw);
    };
    auto advance_h = [&]() {
        ch.stage ^= kWUnitBytes;
        if (++ch.u == U) {
            ch.u = 0;
            ch.id = next_id(ch.id);
            if (ch.id < groups) set_h();
        }
        set_unit(ch);
    };
    cw.id = ch.id = first;
    cw.u = ch.u = 0;
    cw.stage = ch.stage = 0;
    set_w();
    set_h();
    set_unit(cw);
    set_unit(ch);

    // Operand fragments of v_mfma_f32_32x32x16_bf16: lane l reads row l % 32
    // of a 32-row block, K elements 8 (l / 32) .. +7 of the 16-deep step.
    // Step s (0..3) of a unit is chunk 2 s + l / 32, at position
    // (l / 32) ^ ((row >> 1) & 7) ^ 2 s.
    const int wm = wave & 1, wn = wave >> 1;
    const unsigned swz = (unsigned)((((lane >> 5) ^ (lane >> 1)) & 7) << 4);
    const unsigned a_lane = lds_addr(g_lm_w) + (unsigned)((wm * kWaveM + (lane & 31)) * kWRow) + swz;
    const unsigned b_lane = lds_addr(g_lm_h) + (unsigned)((wn * kWaveN + (lane & 31)) * kWRow) + swz;

    f32x16 acc[kFragM][kFragN];
    u32x4 fa[2][kFragM], fb[2][kFragN];
    auto clear = [&]() {
        #pragma unroll
        for (int m = 0; m < kFragM; ++m)
            #pragma unroll
            for (int n = 0; n < kFragN; ++n)
                #pragma unroll
                for (int e = 0; e < 16; ++e) acc[m][n][e] = 0.f;
    };
    clear();
    // Read q (0..7) of a fragment set, in the order the products use them.
    auto read_q = [&](int set, unsigned aa, unsigned ba, int q) {
        if (q & 1)
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fb[set][q >> 1]) : "v"(ba), "i"((q >> 1) * 32 * kWRow));
        else
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fa[set][q >> 1]) : "v"(aa), "i"((q >> 1) * 32 * kWRow));
    };
    auto ready = [&](int set) {             // after lds_wait_all: the set is in registers
        #pragma unroll
        for (int m = 0; m < kFragM; ++m) tie(fa[set][m]);
        #pragma unroll
        for (int n = 0; n < kFragN; ++n) tie(fb[set][n]);
    };
    auto mfma_q = [&](int set, int q) {
        const int m = q / kFragN, n = q % kFragN;
        acc[m][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8, fa[set][m]), __builtin_bit_cast(bf16x8, fb[set][n]),
            acc[m][n], 0, 0, 0);
    };

    // Best key of hidden row 32 n + l % 32 of the wave's block so far.
    unsigned long long best[kFragN];
    #pragma unroll
    for (int n = 0; n < kFragN; ++n) best[n] = 0ull;
    // acc[m][n][e] of lane l: hidden row 32 n + l % 32 of the wave's block,
    // vocabulary entry 32 m + 8 (e / 4) + 4 (l / 32) + e % 4. The largest value
    // first (NaN propagating), then the lowest entry that has it: for a finite
    // nonzero maximum t, x - t has the sign bit unless x == t, so the minimum of
    // bits(x - t) | entry over the lane's values is that entry. Rows past the
    // end of W were loaded as its last row, and stand for it.
    auto fold = [&](int vt) {
        const int vbase = vt * kTileM + wm * kWaveM + 4 * (lane >> 5);
        #pragma unroll
        for (int n = 0; n < kFragN; ++n) {
            float t = acc[0][n][0];
            #pragma unroll
            for (int q = 1; q + 1 < kFragM * 16; q += 2)
                t = maximum3(t, acc[q >> 4][n][q & 15], acc[(q + 1) >> 4][n][(q + 1) & 15]);
            t = maximum3(t, acc[kFragM - 1][n][15], acc[kFragM - 1][n][15]);
            unsigned at = 0xFFu;
            if (__any(!(fabsf(t) < __builtin_huge_valf()) || t == 0.f)) {   // -0 == +0
                const bool tn = t != t;
                #pragma unroll
                for (int q = kFragM * 16 - 1; q >= 0; --q) {
                    const float x = acc[q >> 4][n][q & 15];
                    if (x == t || (tn && x != x)) at = (unsigned)q;
                    tie(at);
                }
            } else {
                #pragma unroll
                for (int q = 0; q < kFragM * 16; q += 2)
                    at = min(at, min(__float_as_uint(acc[q >> 4][n][q & 15] - t) | (unsigned)q,
                                     __float_as_uint(acc[q >> 4][n][(q & 15) + 1] - t) | (unsigned)(q + 1)));
            }
            const int v = min(vbase + (int)(32 * (at >> 4) + 8 * ((at >> 2) & 3) + (at & 3)), V - 1);
            best[n] = umax64(best[n], pack_key(order_key(t), (unsigned)v));
        }
        clear();
    };
    // One atomic maximum per row and M-wave once the row block is done.
    auto flush = [&](int rb) {
        #pragma unroll
        for (int n = 0; n < kFragN; ++n) {
            const unsigned long long b = halves_max64(best[n]);
            const int row = rb * kTileN + wn * kWaveN + 32 * n + lane;
            if (lane < 32 && row < R) atomicMax(keys + row, b);
            best[n] = 0ull;
        }
    };

    // W0, H0, W1 and half of H1 up front; unit 0 needs the first 2 kLoads.
    constexpr int kHalf = kLoads / 2;
    #pragma unroll
    for (int i = 0; i < kLoads; ++i) issue_w(i);
    #pragma unroll
    for (int i = 0; i < kLoads; ++i) issue_h(i);
    advance_w();
    advance_h();
    if (total > 1) {
        #pragma unroll
        for (int i = 0; i < kLoads; ++i) issue_w(i);
        #pragma unroll
        for (int i = 0; i < kHalf; ++i) issue_h(i);
        advance_w();
        wait_vmcnt<kLoads + kHalf>();
    } else {
        wait_vmcnt<0>();
    }
    __builtin_amdgcn_s_barrier();
    #pragma unroll
    for (int q = 0; q < kReads; ++q) read_q(0, a_lane, b_lane, q);
    lds_wait_all();
    ready(0);

    // One unit x: 4 steps of 16 MFMAs, step s's fragments in set s & 1, the
    // next step's reads behind the first MFMAs, one load behind every fourth
    // MFMA. In step 3 every fragment of unit x is in registers: the hand-off
    // (unit x + 1 has landed everywhere; every wave is done with unit x) is
    // followed by the reads of unit x + 1 and the first half of the hidden unit
    // x + 2 (into the stage of unit x), whose second half follows in the next
    // unit's step 0; steps 1 and 2 load the weight of unit x + 2 (into the stage
    // of unit x - 1). sched_barrier pins the interleaving. kSteady: x + 2 < total, so every load exists and the waits are constant.
    int wst = 0;
    unsigned hst = 0;
    auto unit = [&](int x, auto steady_c) {
        constexpr bool kSteady = decltype(steady_c)::value;
        const int wnx = wst == kWStages - 1 ? 0 : wst + 1;
        const unsigned a0 = a_lane + (unsigned)wst * kWUnitBytes, a1 = a_lane + (unsigned)wnx * kWUnitBytes;
        const unsigned b0 = b_lane + hst, b1 = b_lane + (hst ^ kWUnitBytes);
        const bool next = kSteady || x + 1 < total;
        tie(lrow);                                       // keep the lane offsets out of registers
        tie(lchunk0);
        auto step = [&](auto sc) {
            constexpr int s = decltype(sc)::value;
            constexpr int set = s & 1;
            const unsigned aa = s == 3 ? a1 : a0 ^ ((unsigned)(s + 1) << 5);
            const unsigned ba = s == 3 ? b1 : b0 ^ ((unsigned)(s + 1) << 5);
            lds_wait_all();
            ready(set);
            #pragma unroll
            for (int q = 0; q < kSteps; ++q) {
                mfma_q(set, q);
                if (s == 3) {
                    if (q == kPre - 1 && next) {
                        if (kSteady) wait_vmcnt<kLoads>();        // W(x + 2) may be in flight
                        else wait_vmcnt<0>();
                        __builtin_amdgcn_s_barrier();
                    }
                    if (q >= kPre && q < kPre + kReads && next) read_q(set ^ 1, aa, ba, q - kPre);
                } else {
                    if (q < kReads) read_q(set ^ 1, aa, ba, q);
                }
                // step 3: behind the hand-off's reads, else every second MFMA
                constexpr int kLoad0 = s == 3 ? kPre + kReads + 1 : kReads, kEvery = s == 3 ? 1 : 2;
                if (q >= kLoad0 && (q - kLoad0) % kEvery == 0 && (q - kLoad0) / kEvery < kHalf) {
                    const int i = (q - kLoad0) / kEvery;
                    if (s == 0) { if (next) issue_h(kHalf + i); }
                    else if (s == 3) { if (kSteady) issue_h(i); }
                    else if (kSteady) issue_w((s - 1) * kHalf + i);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (s == 0 && next) advance_h();
            if (s == 2 && kSteady) advance_w();
        };
        step(std::integral_constant<int, 0>());
        step(std::integral_constant<int, 1>());
        step(std::integral_constant<int, 2>());
        step(std::integral_constant<int, 3>());
        wst = wnx;
        hst ^= kWUnitBytes;
    };
    int id = first, x = 0;
    while (x < total) {
        const int end = x + U;
        for (; x < end && x + 2 < total; ++x) unit(x, std::true_type());
        for (; x < end; ++x) unit(x, std::false_type());
        lds_wait_all();                                  // the next unit's first fragments
        ready(0);
        fold(vt_of(id));
        const int nid = next_id(id);
        if (nid >= groups || rb_of(nid) != rb_of(id)) flush(rb_of(id));
        id = nid;
    }
}

// ---------------------------------------------------------------------------
// Few rows (R <= kStreamRows): the weight stream is the whole cost.
//
// The 256-row tile multiplies mostly padding here (24 rows: ten times the
// matrix work they need) and leaves CUs without a tile at small vocabularies
// (32000 entries: 125 of 256). Instead the vocabulary is cut into one equal
// range of rows per workgroup; a workgroup walks its range in tiles of WV
// waves x 16 MB rows, every wave with all hidden rows (NB blocks of 16) on
// v_mfma_f32_16x16x32_bf16.
//   * Weight and hidden units of 64 elements (whole 128-byte lines) stream into
//     one S-stage LDS ring, S - 1 units in flight, one barrier per unit: a
//     unit's matrix work is a fraction of the time its lines take to arrive.
//     The ring does not drain between tiles. The weight is read once, so its
//     loads are non-temporal and leave the L2 to the hidden rows, which every
//     workgroup re-reads (64 rows over 128256 x 4096: 196 -> 180 us).
//   * A wave whose rows of the range's last tile are all past the range's end
//     neither loads nor multiplies.
//   * The best key per hidden row stays in registers over the tiles: one atomic
//     maximum per row and workgroup.
// Every vocabulary row is summed in the same K order, so equal weight rows give
// equal sums. The time depends on the memory that a weight was given: between
// buffers of one size and process it differs by up to a fifth. Measured per call
// (three buffers each; us, d = 4096), this kernel against the 256-row tile: 24 rows
// x 32000 entries 51 against 80 (the kernel alone 45-54, 4.9-5.8 TB/s of weight), 64 x
// 128256 177-213 against 247-252 (alone 152-219, 4.8-6.9 TB/s), 64 x 50257 79-84
// against 99-120, 100 x 128256 191-220 against 248-260.
template <int NB, int MB, int S, int WV>
__global__ __launch_bounds__(WV * kWave, 1) void lm_head_stream_kernel(
    const uint16_t *__restrict__ hidden, const uint16_t *__restrict__ w, int R, int V, int d,
    unsigned long long *__restrict__ keys) {
    constexpr int kTM = WV * MB * 16;                    // vocabulary rows of a tile
    constexpr int kHR = NB * 16 < WV * 8 ? WV * 8 : NB * 16;       // hidden rows staged
    constexpr int kStage = (kTM + kHR) * kWRow;
    constexpr int kWL = MB * 2;                          // 1 KB loads per wave and unit: weight,
    constexpr int kHL = kHR / (WV * 8);                  // hidden
    constexpr int kStreamed = 2;                         // cache policy: non-temporal
    __shared__ __attribute__((aligned(1024))) unsigned char ring[S * kStage];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid & (kWave - 1);
    const int U = d / kUnitK;
    const int vbeg = (int)((long long)V * blockIdx.x / gridDim.x);
    const int vend = (int)((long long)V * (blockIdx.x + 1) / gridDim.x);
    const int total = (vend - vbeg + kTM - 1) / kTM * U; // units of this workgroup

    // Load block i of a wave: 8 rows, lane p fills row p / 8, position p % 8,
    // which holds chunk (p % 8) ^ ((row >> 1) & 7). Rows past the end of W or
    // hidden read the last row (finite data; the results are discarded).
    const char *hsrc[kHL];
    #pragma unroll
    for (int i = 0; i < kHL; ++i) {
        const int row = (wave * kHL + i) * 8 + (lane >> 3);
        hsrc[i] = reinterpret_cast<const char *>(hidden + (size_t)min(row, R - 1) * d) +
                  (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    }
    const char *wsrc[kWL];
    bool iw;                                             // this wave has rows in the tile being loaded
    auto set_tile = [&](int v0) {
        iw = wave * MB * 16 < vend - v0;
        #pragma unroll
        for (int i = 0; i < kWL; ++i) {
            const int row = (wave * kWL + i) * 8 + (lane >> 3);
            wsrc[i] = reinterpret_cast<const char *>(w + (size_t)(v0 + min(row, vend - 1 - v0)) * d) +
                      (((lane & 7) ^ ((row >> 1) & 7)) << 4);
        }
    };
    int ik = 0, iv = vbeg, istage = 0;                   // next unit to load
    set_tile(iv);
    auto issue = [&]() {
        unsigned char *st = ring + istage * kStage;
        const size_t ko = (size_t)ik * kWRow;
        if (iw) {
            #pragma unroll
            for (int i = 0; i < kWL; ++i)
                __builtin_amdgcn_global_load_lds((const GLOBAL_AS void *)(wsrc[i] + ko),
                                                 (LDS_AS void *)(st + (wave * kWL + i) * 1024),
                                                 16, 0, kStreamed);
        }
        #pragma unroll
        for (int i = 0; i < kHL; ++i)
            __builtin_amdgcn_global_load_lds((const GLOBAL_AS void *)(hsrc[i] + ko),
                                             (LDS_AS void *)(st + kTM * kWRow + (wave * kHL + i) * 1024),
                                             16, 0, 0);
        istage = istage == S - 1 ? 0 : istage + 1;
        if (++ik == U) {
            ik = 0;
            iv += kTM;
            set_tile(iv);
        }
    };
    #pragma unroll
    for (int x = 0; x < S - 1; ++x)
        if (x < total) issue();

    // Fragments of v_mfma_f32_16x16x32_bf16: lane l reads row l % 16 of a
    // 16-row block, chunk 4 s + l / 16 of step s.
    const unsigned base = lds_addr(ring);
    const unsigned swz = (unsigned)((lane >> 4) ^ ((lane >> 1) & 7));
    const unsigned a_lane = base + (unsigned)((wave * MB * 16 + (lane & 15)) * kWRow);
    const unsigned b_lane = base + (unsigned)((kTM + (lane & 15)) * kWRow);
    f32x4 acc[MB][NB];
    unsigned long long best[NB];
    #pragma unroll
    for (int n = 0; n < NB; ++n) {
        best[n] = 0ull;
        #pragma unroll
        for (int m = 0; m < MB; ++m) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    int k = 0, stage = 0, v0 = vbeg;
    for (int x = 0; x < total; ++x) {
        // unit x has landed: S - 2 units of loads may be in flight (fewer at the
        // end; hidden loads alone once this wave has no weight rows to load)
        if (x + S - 2 >= total) wait_vmcnt<0>();
        else if (iw) wait_vmcnt<(S - 2) * (kWL + kHL)>();
        else wait_vmcnt<(S - 2) * kHL>();
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (x + S - 1 < total) issue();                  // into the stage that held unit x - 1
        if (wave * MB * 16 < vend - v0) {
            u32x4 fa[2][MB], fb[2][NB];
            auto reads = [&](int s) {
                const unsigned off = (unsigned)stage * kStage + ((swz ^ (unsigned)(4 * s)) << 4);
                #pragma unroll
                for (int m = 0; m < MB; ++m)
                    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fa[s][m]) : "v"(a_lane + off), "i"(m * 16 * kWRow));
                #pragma unroll
                for (int n = 0; n < NB; ++n)
                    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(fb[s][n]) : "v"(b_lane + off), "i"(n * 16 * kWRow));
            };
            reads(0);
            #pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (s == 0) {
                    reads(1);
                    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(MB + NB) : "memory");
                } else {
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                }
                #pragma unroll
                for (int m = 0; m < MB; ++m) tie(fa[s][m]);
                #pragma unroll
                for (int n = 0; n < NB; ++n) tie(fb[s][n]);
                #pragma unroll
                for (int n = 0; n < NB; ++n)
                    #pragma unroll
                    for (int m = 0; m < MB; ++m)
                        acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, fa[s][m]), __builtin_bit_cast(bf16x8, fb[s][n]),
                            acc[m][n], 0, 0, 0);
            }
        }
        stage = stage == S - 1 ? 0 : stage + 1;
        if (++k == U) {
            // acc[m][n][e] of lane l: hidden row 16 n + l % 16, vocabulary
            // entry 16 m + 4 (l / 16) + e of the wave's rows
            const int vb = v0 + wave * MB * 16 + 4 * (lane >> 4);
            #pragma unroll
            for (int n = 0; n < NB; ++n)
                #pragma unroll
                for (int m = 0; m < MB; ++m) {
                    #pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int v = vb + 16 * m + e;
                        const unsigned long long key = pack_key(order_key(acc[m][n][e]), (unsigned)v);
                        best[n] = v < vend ? umax64(best[n], key) : best[n];
                    }
                    acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            k = 0;
            v0 += kTM;
        }
    }
    // lanes l, l ^ 16, l ^ 32, l ^ 48 hold the same hidden row; then the waves
    // meet in LDS (free once every wave is past its last fragment read)
    unsigned long long *kx = reinterpret_cast<unsigned long long *>(ring);
    __syncthreads();
    #pragma unroll
    for (int n = 0; n < NB; ++n) {
        const unsigned long long b = halves_max64(rows_max64(best[n]));
        if (lane < 16) kx[wave * NB * 16 + n * 16 + lane] = b;
    }
    __syncthreads();
    if (tid < NB * 16 && tid < R) {
        unsigned long long b = kx[tid];
        #pragma unroll
        for (int u = 1; u < WV; ++u) b = umax64(b, kx[u * NB * 16 + tid]);
        atomicMax(keys + tid, b);
    }
}

}  // namespace

namespace {

template <int NB, int MB, int S, int WV>
hipError_t launch_stream(int groups, const uint16_t *hidden, const uint16_t *w, int R, int V, int d,
                         unsigned long long *keys, hipStream_t s) {
    const int most = (V + 15) / 16;                  // no range shorter than one wave's 16 rows
    return launch_kernel(lm_head_stream_kernel<NB, MB, S, WV>, dim3(groups < most ? groups : most),
                         dim3(WV * kWave), s, hidden, w, R, V, d, keys);
}

// Which split of the vocabulary the weight stream takes, by the rows a CU gets
// (V / 256). us per call at d = 4096 unless stated, both sides on the same weights,
// three buffers each:
//   * V >= 98304 (384 rows per CU, at least 1.5 tiles of 256): one workgroup of
//     8 waves x 32 rows per CU; the taller tile re-reads the hidden rows half as
//     often (V = 128256, 64 rows: 177-213 against 198-218 with 16 rows per wave and
//     202-207 with two workgroups per CU, 24 rows 173-202 against 193-210 and
//     194-199; V = 98304 143-170 against 144-158 with the next one; V = 75000, d =
//     2048: 74-83 against 72-78).
//   * 40960 <= V: two workgroups of 8 waves x 16 rows per CU (V = 50257, 64 rows:
//     79-84 against 86-97 with one workgroup per CU, 80-96 with 32 rows per wave).
//   * 24576 <= V and d >= 2048: two workgroups of 4 waves x 16 rows per CU, a
//     range of at most 80 rows each (V = 32000, 24 rows: 51 against 57-60, 64 rows 60
//     against 62-63).
//   * below, or with a short K loop, starting 512 workgroups costs more than
//     their overlap gains: one workgroup of 8 waves x 16 rows per CU (24 rows, d =
//     1024: V = 12000 17 against 20, V = 32000 20 against 23).
// More than 64 rows: the hidden units fill the ring, one workgroup per CU; 32
// rows per wave halve its LDS reads of them (100 rows: V = 128256 191-220 against
// 214-227, V = 50257 87-102 against 99-108).
hipError_t launch_stream_rows(const uint16_t *hidden, const uint16_t *w, int R, int V, int d,
                              unsigned long long *keys, hipStream_t s) {
    if (R > 64) return launch_stream<8, 2, 3, 8>(256, hidden, w, R, V, d, keys, s);
    if (V >= 98304)
        return R > 32 ? launch_stream<4, 2, 4, 8>(256, hidden, w, R, V, d, keys, s)
                      : launch_stream<2, 2, 4, 8>(256, hidden, w, R, V, d, keys, s);
    if (V >= 24576 && V < 40960 && d >= 2048)
        return R > 32 ? launch_stream<4, 1, 4, 4>(512, hidden, w, R, V, d, keys, s)
                      : launch_stream<2, 1, 6, 4>(512, hidden, w, R, V, d, keys, s);
    const int groups = V >= 40960 ? 512 : 256;
    return R > 32 ? launch_stream<4, 1, 3, 8>(groups, hidden, w, R, V, d, keys, s)
                  : launch_stream<2, 1, 3, 8>(groups, hidden, w, R, V, d, keys, s);
}

}  // namespace

int lm_head_vocab_tiles(int V) { return (int)(((long long)V + kTileM - 1) / kTileM); }

hipError_t launch_lm_head_argmax_accept(const uint16_t *hidden, const uint16_t *w,
                                        const int32_t *draft, const int32_t *parent,
                                        const int32_t *num_nodes, int B, int N, int V, int d,
                                        int32_t *argmax_out, int32_t *accept_len,
                                        int32_t *accept_idx, int32_t *bonus,
                                        unsigned long long *keys, hipStream_t s) {
    if (B == 0) return hipSuccess;
    const int R = B * N;
    hipError_t e = launch_kernel(lm_keys_clear_kernel, dim3((R + 255) / 256), dim3(256), s, keys, R);
    if (e != hipSuccess) return e;
    // the tiled product's offsets inside a tile fit 32 bits only below this d
    if (R <= kStreamRows || d >= 1 << 23) {
        for (int r0 = 0; r0 < R; r0 += kStreamRows) {
            e = launch_stream_rows(hidden + (size_t)r0 * d, w, R - r0 < kStreamRows ? R - r0 : kStreamRows,
                                   V, d, keys + r0, s);
            if (e != hipSuccess) return e;
        }
        return launch_accept(keys, 1, draft, parent, num_nodes, B, N, argmax_out, accept_len,
                             accept_idx, bonus, s);
    }
    const int vtiles = lm_head_vocab_tiles(V);
    const int rblocks = (R + kTileN - 1) / kTileN;
    const int groups = (vtiles + kNumXcd - 1) / kNumXcd * kNumXcd * rblocks;
    const int wgs = groups < 256 ? groups : 256;     // one workgroup per CU (its LDS)
    e = launch_kernel(lm_head_argmax_kernel, dim3(wgs), dim3(kLmThreads), s, hidden, w, R, V, d,
                      vtiles, rblocks, groups, keys);
    if (e != hipSuccess) return e;
    return launch_accept(keys, 1, draft, parent, num_nodes, B, N, argmax_out, accept_len,
                         accept_idx, bonus, s);
}

}  // namespace tv
