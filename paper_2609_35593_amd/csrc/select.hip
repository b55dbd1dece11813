// Drift-based block selection (Secs. 4.2-4.3), one launch for every row of a
// layer: pooled map, drift scores, exact top-c, R budget-neutral restoration
// rounds with track-best, and compaction of the kept-block lists.
//
// Work layout. A workgroup of NW waves owns NW x R query blocks ("rows") of one
// head; each wave owns R of them.
//  - Per-candidate quantities live "lane <-> key block": lane l, slot c holds key
//    block j = l + 64 c (CPL slots). P_ij and s_ij^2 stay in registers for all rounds;
//    product results, order keys and swap lists take turns in one LDS staging row per
//    row. The vectors that a product needs from every row (Qbar, vbar, S vbar with S
//    the symmetric part of M, g, M g) pass through two LDS vector slots per row; the
//    owner keeps vbar and g lane <-> channel in registers.
//  - The contractions are float64 matrix products of the workgroup's rows
//    (padded to a multiple of 16) with the head's row-major pooled tensors, on
//    the matrix cores (16x16x4 float64 steps): over channels, the pooled logits
//    against Kbar and the drift scores (expanded as in Eq. 9; a row's block with
//    P > 1/2 gets e^T M e directly) and every round's gains against Vbar;
//    over key blocks, the dense pooled output vbar and the net drift g against
//    Vbar. Each output element is one chain of matrix steps in a fixed order: reruns
//    are bit-identical.
//  - Every top-k is exact: a search for a threshold of order-preserving 64-bit keys
//    that exactly k reach, using wave ballots and popcounts, ties broken by the lower
//    block index. No atomics and no data-dependent reduction order.
//
// What bounds it. Row work (gains, searches, swap lists) is a chain of short vector
// and scalar steps, so it wants waves: up to 16 per workgroup, one workgroup per CU,
// which is why a row's results wait in LDS and not in registers (128 to 256 per lane).
// The products want 16 rows per tile and their B tiles in few cache-line requests
// (load_tile). Measured (select_kernel alone, 16 heads, us; before: 8 waves of one to
// three rows with the products' results in registers): 8 views 46 -> 42, 16 views
// 88 -> 63, 32 views 192 -> 160, 100 views 2,010 -> 1,160; with 64-token key blocks 16
// views 130 -> 92, 32 views 475 -> 282 and (4 heads) 100 views 4,520 -> 1,140. Of the
// 100-view time the products take about 45%, the searches 15%, gains 10-15%.
// All arithmetic is float64 (the discrete decisions stay stable).
#include <math.h>

#include "ress_internal.h"

namespace ress {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

// Word 3 of a raw buffer descriptor on gfx9-family chips (32-bit data format,
// no swizzle, no index stride): loads past num_records bytes return zero.
constexpr int kBufWord3 = 0x00020000;

// Buffer descriptor over one head's row-major pooled tensor (nkb x 64 doubles).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pooled_rsrc(const double *base, int nkb)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(base), 0, kD * nkb * (int)sizeof(double),
                                             kBufWord3);
}

// Channel `lane` of row j (wave-uniform) of a row-major pooled tensor.
__device__ __forceinline__ double pooled_row(__amdgpu_buffer_rsrc_t rs, int j, int lane)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                          rs, (unsigned)lane * (unsigned)sizeof(double),
                                          __builtin_amdgcn_readfirstlane(j) * kD * (int)sizeof(double), 0));
}

// 16 bytes at byte offset `off` of a pooled tensor (zero past its end).
__device__ __forceinline__ double2 pooled_16(__amdgpu_buffer_rsrc_t rs, int off)
{
    return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
}

// Wave reductions on registers only (no LDS permutes): DPP exchanges within 16
// lanes (lane i with i^1, i^2, then with 7-i within 8 and 15-i within 16, each
// step adding a symmetric pair, so every lane holds the same partial), then the
// gfx950 row swaps, whose two results added give x[l] + x[l^16] and
// x[l] + x[l^32] in every lane. Commutative adds in a fixed pattern: the result
// is identical in every lane and on every run.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)u, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Lane l's value and that of lane l^16 (ROW32: l^32), in an order that is the
// same for both lanes of the pair.
template <bool ROW32>
__device__ __forceinline__ void swap_pair(double x, double &d0, double &d1)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = (unsigned)u, hi = (unsigned)(u >> 32);
    const auto a = ROW32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                         : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = ROW32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                         : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    d0 = __longlong_as_double((long long)(((unsigned long long)b[0] << 32) | a[0]));
    d1 = __longlong_as_double((long long)(((unsigned long long)b[1] << 32) | a[1]));
}

template <bool ROW32>
__device__ __forceinline__ double swap_sum(double x)
{
    double d0, d1;
    swap_pair<ROW32>(x, d0, d1);
    return d0 + d1;
}

__device__ __forceinline__ double wave_sum(double x)
{
    x += dpp_f64<0xB1>(x);   // quad_perm [1,0,3,2]: lane i^1
    x += dpp_f64<0x4E>(x);   // quad_perm [2,3,0,1]: lane i^2
    x += dpp_f64<0x141>(x);  // row_half_mirror: lane 7-i within 8
    x += dpp_f64<0x140>(x);  // row_mirror: lane 15-i within 16
    x = swap_sum<false>(x);  // + the partner 16-lane row
    return swap_sum<true>(x);  // + the other 32 lanes
}

// Two wave sums with their exchanges interleaved.
__device__ __forceinline__ void wave_sum2(double a, double b, double &sa, double &sb)
{
    a += dpp_f64<0xB1>(a);
    b += dpp_f64<0xB1>(b);
    a += dpp_f64<0x4E>(a);
    b += dpp_f64<0x4E>(b);
    a += dpp_f64<0x141>(a);
    b += dpp_f64<0x141>(b);
    a += dpp_f64<0x140>(a);
    b += dpp_f64<0x140>(b);
    a = swap_sum<false>(a);
    b = swap_sum<false>(b);
    sa = swap_sum<true>(a);
    sb = swap_sum<true>(b);
}

__device__ __forceinline__ double wave_max(double x)
{
    x = fmax(x, dpp_f64<0xB1>(x));
    x = fmax(x, dpp_f64<0x4E>(x));
    x = fmax(x, dpp_f64<0x141>(x));
    x = fmax(x, dpp_f64<0x140>(x));
    double d0, d1;
    swap_pair<false>(x, d0, d1);
    x = fmax(d0, d1);
    swap_pair<true>(x, d0, d1);
    return fmax(d0, d1);
}

__device__ __forceinline__ v4d mfma_f64(double a, double b, v4d c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Order-preserving map of a double to uint64 (larger value -> larger key);
// -0 is folded onto +0 so that equal values get equal keys.
__device__ __forceinline__ unsigned long long order_key(double x)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(x + 0.0);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// One bit per slot of a lane.
template <bool WIDE>
struct slot_bits {
    using type = unsigned int;
};
template <>
struct slot_bits<true> {
    using type = unsigned long long;
};

// x / d for normal d far from the ends of the range and finite x: the reciprocal
// by two Newton steps and one corrected quotient, without the compiler's scaling
// and special cases (a third fewer instructions; the same value but for a last bit
// now and then).
__device__ __forceinline__ double quot(double x, double d)
{
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    const double q = x * r;
    return fma(fma(-d, q, x), r, q);
}

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ double uniform(double x)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

template <int CTRL>
__device__ __forceinline__ unsigned int dpp_max_u32(unsigned int x)
{
    const unsigned int y = (unsigned int)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, false);
    return y > x ? y : x;
}

// Largest 32-bit unsigned value over the wave, as a scalar.
__device__ __forceinline__ unsigned int wave_max_u32(unsigned int x)
{
    x = dpp_max_u32<0xB1>(x);
    x = dpp_max_u32<0x4E>(x);
    x = dpp_max_u32<0x141>(x);
    x = dpp_max_u32<0x140>(x);
    auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = a[0] > a[1] ? a[0] : a[1];
    a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return __builtin_amdgcn_readfirstlane(a[0] > a[1] ? a[0] : a[1]);
}

// Threshold search over member high words h[0..NS) (zero for non-members): a t that
// exactly k of them reach (found), or else the k-th largest word, which more than k
// reach. From the largest word down in steps of 1/4 octave (of the float64 value
// behind the word), 1, 4, 16, ... octaves, then by halving: the k-th largest of a few
// hundred gains mostly lies within two octaves of the largest, and 4-6 counts find a
// separating threshold (measured over the 8- and 32-view layers; bit by bit from the
// top: 14-18). lo is reached by at least k members, hi by fewer (0 < hi - lo in
// modular arithmetic, it shrinks with every count). All of it wave-uniform, on scalar
// registers and branches.
template <int NS>
__device__ __forceinline__ unsigned int search_high(const unsigned int (&h)[NS], int k, int &found)
{
    unsigned int m = h[0];
#pragma unroll
    for (int c = 1; c < NS; ++c) m = h[c] > m ? h[c] : m;
    unsigned int t = wave_max_u32(m), at, lo = 0, hi = t + 1, step = 1u << 18;
    do {
        int cnt = 0;
#pragma unroll
        for (int c = 0; c < NS; ++c) cnt += __popcll(__ballot(h[c] >= t));
        found = cnt == k;
        at = t;
        lo = cnt > k ? t : lo;
        hi = cnt > k ? hi : t;
        const unsigned int down = hi > step ? hi - step : 1u, mid = lo + ((hi - lo) >> 1);
        t = __builtin_amdgcn_readfirstlane(lo == 0u ? down : mid);
        step = step >= 1u << 30 ? ~0u : step << 2;
    } while (!found && hi - lo != 1u);
    return found ? at : lo;
}

// Exact top-k of the member slots by (key desc, block index asc). The slots' order
// keys are the 8-byte words keys[64 c] (this lane's pointer into its wave's LDS row;
// they are read from there for each search, which needs one register a slot). Bit c
// of mbits marks this lane's slot c as a member. Non-member high words are replaced
// by 0, below every member's (an order key of a finite value has a nonzero high
// word), so one ballot per slot counts members only. search_high first; where no
// high word separates the top k, a key reaches a candidate (t, x) (x >= 1), t the
// k-th largest high word, exactly when the 32-bit value "all ones if its high word
// is above t, its low word if equal, zero if below" reaches x, and the low word is
// found bit by bit. Returns this lane's chosen slots as a bit mask. Requires 0 <= k
// <= number of members.
template <int CPL>
__device__ __forceinline__ typename slot_bits<(CPL > 32)>::type topk_slots(const double *keys,
                                                                           typename slot_bits<(CPL > 32)>::type mbits,
                                                                           int k, unsigned long long lane_lt)
{
    k = __builtin_amdgcn_readfirstlane(k);
    if (k <= 0) return 0;
    unsigned int hm[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c)
        hm[c] = ((mbits >> c) & 1) ? (unsigned int)((unsigned long long)__double_as_longlong(keys[64 * c]) >> 32) : 0u;
    int found = 0;
    const unsigned int thi = search_high<CPL>(hm, k, found);
    typename slot_bits<(CPL > 32)>::type chosen = 0;
    const auto one = (typename slot_bits<(CPL > 32)>::type)1;
    if (found) {  // exactly k keys reach (thi, 0): they are the top k
#pragma unroll
        for (int c = 0; c < CPL; ++c)
            if (hm[c] >= thi) chosen |= one << c;
        return chosen & mbits;
    }
    // Low word, against the high word thi of the k-th largest key.
    unsigned int l2[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c)
        l2[c] = hm[c] > thi ? 0xffffffffu
                            : (hm[c] == thi ? (unsigned int)__double_as_longlong(keys[64 * c]) : 0u);
    unsigned int tlo = 0, bit = 0x80000000u;
    do {
        const unsigned int cand = __builtin_amdgcn_readfirstlane(tlo | bit);
        int cnt = 0;
#pragma unroll
        for (int c = 0; c < CPL; ++c) cnt += __popcll(__ballot(l2[c] >= cand));
        tlo = cnt >= k ? cand : tlo;
        found = cnt == k;
        bit >>= 1;
    } while (!found && bit != 0u);
    if (found) {
#pragma unroll
        for (int c = 0; c < CPL; ++c)
            if (l2[c] >= tlo) chosen |= one << c;
        return chosen & mbits;
    }
    // (thi, tlo) is the k-th largest key and is tied: take all larger keys and the
    // lowest-index ties.
    int gt = 0;
#pragma unroll
    for (int c = 0; c < CPL; ++c) gt += __popcll(__ballot(hm[c] > thi || (hm[c] == thi && l2[c] > tlo)));
    const int need = k - gt;
    int before = 0;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const bool above = hm[c] > thi || (hm[c] == thi && l2[c] > tlo);
        const bool tie = hm[c] == thi && l2[c] == tlo;
        const unsigned long long tb = __ballot(tie);
        const int rank = before + __popcll(tb & lane_lt);
        if (above || (tie && rank < need)) chosen |= one << c;
        before += __popcll(tb);
    }
    return chosen & mbits;
}

// Sizes of a workgroup configuration: NW waves of R rows each, RW = NW R rows in MT
// 16-row tiles; WPC workgroups share a CU. LDS holds, per row, one staging row of SW
// slots (64 key blocks each, padded by 16 bytes so that rows start on different banks)
// and two vectors of 64 channels (padded likewise), and M_h where it fits beside them.
template <int CPL, int R, int NW, int WPC>
struct SelCfg {
    static constexpr int RW = NW * R;
    static constexpr int MT = (RW + 15) / 16;
    // Key-block splits of the weighted sums: 2 MT KS items, one per wave; the KS
    // partial tiles of a row sit side by side in its staging row.
    static constexpr int KS = NW / (2 * MT) < 8 ? NW / (2 * MT) : 8;
    static constexpr int SW = CPL > KS ? (CPL > 3 ? CPL : 3) : (KS > 3 ? KS : 3);  // at least 3: the swap list
    static constexpr int SROW = SW * 64 + 2;  // doubles per staging row
    static constexpr int VROW = kD + 2;       // doubles per vector
    static constexpr int BYTES = RW * (SROW + 2 * VROW) * 8;
    static constexpr bool M_LDS = WPC * (BYTES + kD * (kD + 1) * 4 + 64) <= 163840;
    static constexpr int TPW = (4 * CPL + NW - 1) / NW;  // key-block tiles per wave, at most
    // Tiles of Vbar a wave keeps in registers for all its passes (32 registers
    // each), as far as they fit beside the rows' state.
    static constexpr int REGS = 2048 / (NW * WPC);  // registers per lane
    static constexpr int STATE = 4 * R * CPL + CPL + 60 + 25 * R;
    static constexpr int VT = STATE + 32 * TPW <= REGS ? TPW : (STATE + 32 <= REGS ? 1 : 0);
    static constexpr int FENCE = REGS - 4 * R * CPL - 32 * VT >= 128 ? 0 : (REGS - 4 * R * CPL - 32 * VT >= 90 ? 2 : 1);
    using bits = typename slot_bits<(CPL > 32)>::type;
    static_assert(WPC * BYTES <= 163840, "LDS of one CU");
    static_assert(KS >= 1, "one weighted-sum item per wave at most");
    static_assert(4 * MT <= NW, "one mat-vec item per wave at most");
};

template <int CPL, int R, int NW, int WPC>
__global__ void __launch_bounds__(NW * 64, NW * WPC / 4) select_kernel(const SelectParams p)
{
    using Cfg = SelCfg<CPL, R, NW, WPC>;
    constexpr int RW = Cfg::RW, MT = Cfg::MT, SROW = Cfg::SROW, VROW = Cfg::VROW, KS = Cfg::KS, VT = Cfg::VT;
    constexpr int TPW = Cfg::TPW;
    constexpr bool M_LDS = Cfg::M_LDS;
    __shared__ __align__(16) double stage[RW * SROW];
    __shared__ __align__(16) double vecs[2 * RW * VROW];  // vector slots 0 and 1 of every row
    __shared__ int flags[NW];
    __shared__ float Ms[M_LDS ? kD * (kD + 1) : 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned long long lane_lt = (1ull << lane) - 1ull;
    // Workgroups are numbered so that each of the 8 XCDs gets a contiguous range
    // of (head, row group) items: the rows of a head share one XCD's L2.
    const int groups = (p.n_qb + RW - 1) / RW;
    const int item = (blockIdx.x & 7) * p.items_per_xcd + (blockIdx.x >> 3);
    if (item >= p.H * groups) return;  // the whole workgroup
    const int h = item / groups;
    const int row0 = (item % groups) * RW + wave * R;
    const int nkb = p.n_kb, nqb = p.n_qb;
    const int ntiles = (nkb + 15) >> 4;
    const __amdgpu_buffer_rsrc_t rsK = pooled_rsrc(p.pooled.kbar + (size_t)h * nkb * kD, nkb);
    const __amdgpu_buffer_rsrc_t rsV = pooled_rsrc(p.pooled.vbar + (size_t)h * nkb * kD, nkb);
    const float *Mh = p.gram + (size_t)h * kD * kD;
    auto m_at = [&](int r, int c) __attribute__((always_inline)) -> double {
        return (double)(M_LDS ? Ms[r * (kD + 1) + c] : Mh[r * kD + c]);
    };
    auto row_vec = [&](int slot, int m) __attribute__((always_inline)) -> double * {
        return vecs + (slot * RW + m) * VROW;
    };
    // Keeps the compiler from interleaving the work of more than FENCE slots, whose
    // temporaries would not fit the registers.
    auto slot_fence = [&](int c) __attribute__((always_inline)) {
        if (Cfg::FENCE > 0 && c % (Cfg::FENCE > 0 ? Cfg::FENCE : 1) == Cfg::FENCE - 1)
            __builtin_amdgcn_sched_barrier(0);
    };
    // n_kb anew for each use, so that the compiler compares a slot's block index with it
    // there instead of keeping one mask per slot.
    auto nkb_here = [&]() __attribute__((always_inline)) -> int {
        int n = nkb;
        asm("" : "+s"(n));
        return n;
    };
    auto own = [&](int r) __attribute__((always_inline)) -> double * { return stage + (wave * R + r) * SROW; };
    const int grp = lane >> 4, col = lane & 15;  // matrix-step lane coordinates

    // Tile t of a pooled tensor (16 key blocks; zero past its end): lane l holds, of key
    // block 16 t + l % 16, channels 8 u + 2 (l / 16) + e (u < 8, e = 0, 1) as b[2 u + e].
    // Loaded as they lie, a lane's neighbours would hold other key blocks and each load
    // take the L1 one cycle a lane (measured at 1,074 key blocks: a pass took 35 K cycles,
    // all of it these loads, with half as much matrix work). So four lanes read 64
    // contiguous bytes of a key block (lane l: block l / 4, 16 bytes l % 4) and the wave
    // exchanges them in 512 bytes of LDS of its own, `buf` (a wave's LDS accesses are in
    // order); the odd half of the blocks swaps its 16-byte pairs, so that the reads are
    // free of conflicts.
    auto load_tile = [&](__amdgpu_buffer_rsrc_t rs, int t, double *buf, double (&b)[16])
                         __attribute__((always_inline)) {
        const int off = (16 * t + (lane >> 2)) * kD * (int)sizeof(double) + (lane & 3) * 16;
        double *put = buf + ((lane & ~3) | ((lane & 3) ^ ((lane >> 5) << 1)));
        const double *get = buf + 4 * col + (grp ^ ((col >> 3) << 1));
        double2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = pooled_16(rs, off + 64 * u);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            *put = v[u].x;
            __builtin_amdgcn_wave_barrier();
            b[2 * u] = *get;
            __builtin_amdgcn_wave_barrier();
            *put = v[u].y;
            __builtin_amdgcn_wave_barrier();
            b[2 * u + 1] = *get;
            __builtin_amdgcn_wave_barrier();
        }
    };
    auto buf_of = [&](int slot) __attribute__((always_inline)) -> double * { return row_vec(slot, 0) + 64 * wave; };
    // Products of every row's vector `xs` with the 16 key blocks of tile t, into the
    // staging rows (in step 2 u + e the k index l / 16 stands for channel
    // 8 u + 2 (l / 16) + e, in A as in B; rows past RW repeat the last one and are not
    // stored).
    auto tile_product = [&](int xs, int t, const double (&b)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const double *arow = row_vec(xs, min(16 * mt + col, RW - 1)) + 2 * grp;
            v4d c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const double2 a = *reinterpret_cast<const double2 *>(arow + 8 * u);
                c = mfma_f64(a.x, b[2 * u], c);
                c = mfma_f64(a.y, b[2 * u + 1], c);
                if (Cfg::FENCE > 0 && u % 2 == 1) __builtin_amdgcn_sched_barrier(0);
            }
            // c[v] = C[16 mt + 4 v + l / 16][16 t + l % 16]
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = 16 * mt + 4 * v + grp;
                if (RW % 16 == 0 || m < RW) stage[m * SROW + 16 * t + col] = c[v];
            }
        }
    };
    // stage[m][j] = X_m . T_j for the workgroup's rows m and key blocks j, X_m vector
    // `xs` of row m, T the head's pooled tensor behind rs. Tile t belongs to wave
    // t mod NW; its first VT tiles come from the registers `res`. The caller has
    // every row's vector in place and nobody reading the staging rows; ends with a
    // barrier, after which the owners read their rows.
    auto dot_pass = [&](int xs, __amdgpu_buffer_rsrc_t rs, const double (&res)[VT > 0 ? VT : 1][16])
                        __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < VT; ++i)
            if (wave + NW * i < ntiles) tile_product(xs, wave + NW * i, res[i]);
        if constexpr (TPW > VT) {
#pragma unroll 1
            for (int t = wave + NW * VT; t < ntiles; t += NW) {
                double b[16];
                load_tile(rs, t, buf_of(xs ^ 1), b);  // in the vector slot not in use
                tile_product(xs, t, b);
            }
        }
        __syncthreads();
    };
    // out_m[d] = sum_j w_m(j) Vbar_j[d] for every row m of the workgroup, with w_m(j) =
    // w(r, c) of the owning wave (zero for key blocks past n_kb): vector slot 0 of row m,
    // and out[r] = channel `lane` of the wave's rows. The owners stage their weights.
    // Item (mt, np, ks) of wave mt 2 KS + np KS + ks accumulates the 16 rows of tile mt
    // against channels 32 np + 2 n + e (n < 16, e = 0, 1) over the key-block octets
    // o = ks (mod KS): in each step the k index l / 16 stands for key block
    // 8 o + 2 (l / 16) + (0 or 1), so one 16-byte read gives the A values of two steps
    // and one 16-byte read of a key block's channel pair the B values of two products.
    // The KS partial tiles are then added in split order by the owners. Ends with a
    // barrier.
    auto wsum_pass = [&](auto w, double (&out)[R]) __attribute__((always_inline)) {
        const bool mine = wave < 2 * MT * KS;
        const int it = mine ? wave : 0;
        const int ks = it % KS, np = (it / KS) & 1, mt = it / (2 * KS);
        v4d c0 = {0.0, 0.0, 0.0, 0.0}, c1 = c0;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < CPL; ++c) own(r)[c * 64 + lane] = w(r, c);
        __syncthreads();
        if (mine) {
            const double *arow = stage + min(16 * mt + col, RW - 1) * SROW + 2 * grp;
            const int boff = (32 * np + 2 * col) * (int)sizeof(double) + 2 * grp * kD * (int)sizeof(double);
            const int noct = (nkb + 7) >> 3;
            // Four octets at a time (weights and pooled rows past the last block are zero
            // or read as zero, the staged row reaches 64 CPL blocks).
            for (int o = ks; o < noct; o += 4 * KS) {
                double2 a[4], b0[4], b1[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int ou = o + u * KS, off = 8 * ou * kD * (int)sizeof(double) + boff;
                    b0[u] = pooled_16(rsV, off);
                    b1[u] = pooled_16(rsV, off + kD * (int)sizeof(double));
                    a[u] = *reinterpret_cast<const double2 *>(arow + 8 * min(ou, noct - 1));
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool in = o + u * KS < noct;  // wave-uniform
                    if (!in) break;
                    c0 = mfma_f64(a[u].x, b0[u].x, c0);
                    c1 = mfma_f64(a[u].x, b0[u].y, c1);
                    c0 = mfma_f64(a[u].y, b1[u].x, c0);
                    c1 = mfma_f64(a[u].y, b1[u].y, c1);
                }
            }
        }
        __syncthreads();
        // c_e[v] = partial of row 16 mt + 4 v + l / 16, channel 32 np + 2 (l % 16) + e
        if (mine) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = 16 * mt + 4 * v + grp;
                if (RW % 16 == 0 || m < RW)
                    *reinterpret_cast<double2 *>(stage + m * SROW + ks * kD + 32 * np + 2 * col) =
                        double2{c0[v], c1[v]};
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double *src = own(r) + lane;
            double tot = src[0];
#pragma unroll
            for (int k2 = 1; k2 < KS; ++k2) tot += src[k2 * kD];
            out[r] = tot;
        }
    };

    // x_m = A y_m for every row m of the workgroup (y: vector slot 0, x: vector slot 1)
    // with A = M_h, or with SYM its symmetric part (M + M^T) / 2 (the same quadratic
    // form; exact in float64 from float32 entries). Item (mt, nt) of 4 MT, on
    // wave mt 4 + nt: the 16 rows of tile mt against output channels 16 nt .. +15,
    // k <-> channel 16 u + 4 (l / 16) + e in step 4 u + e. Begins and ends with
    // a barrier (the owners write y before and read x after).
    auto mv_pass = [&](auto sym) __attribute__((always_inline)) {
        constexpr bool SYM = decltype(sym)::value;
        __syncthreads();
        if (wave < 4 * MT) {
            const int mt = wave >> 2, nt = wave & 3;
            const double *arow = row_vec(0, min(16 * mt + col, RW - 1)) + 4 * grp;
            const int n = 16 * nt + col;
            v4d c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = 16 * u + 4 * grp;
                const double2 a0 = *reinterpret_cast<const double2 *>(arow + 16 * u);
                const double2 a1 = *reinterpret_cast<const double2 *>(arow + 16 * u + 2);
                const double a[4] = {a0.x, a0.y, a1.x, a1.y};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    double b = m_at(n, k + e);
                    if (SYM) b = 0.5 * (b + m_at(k + e, n));
                    c = mfma_f64(a[e], b, c);
                }
            }
            // c[v] = x[row 16 mt + 4 v + l / 16][channel n]
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = 16 * mt + 4 * v + grp;
                if (RW % 16 == 0 || m < RW) row_vec(1, m)[n] = c[v];
            }
        }
        __syncthreads();
    };
    using plain_mv = std::integral_constant<bool, false>;
    using sym_mv = std::integral_constant<bool, true>;

    const double eps = p.eps;
    const double *cT = p.pooled.cT + (size_t)h * nkb;
    const int c_h = p.budgets[h];
    const int n_p = p.first_forced;  // candidates are the key blocks j < first_forced

    int irow[R];
    bool live[R], dense[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        live[r] = row0 + r < nqb;
        irow[r] = live[r] ? row0 + r : nqb - 1;
        dense[r] = !live[r] || irow[r] >= p.first_dense_qb || c_h >= n_p;
    }
    using bits = typename Cfg::bits;  // one bit per slot of this lane
    bits cand_bits = 0;               // bit c: slot c is a candidate
#pragma unroll
    for (int c = 0; c < CPL; ++c)
        if (lane + 64 * c < n_p) cand_bits |= (bits)1 << c;

    double res[VT > 0 ? VT : 1][16];  // this wave's resident tiles: Kbar, then Vbar
    {
        constexpr int T = NW * 64, M4 = M_LDS ? (kD * kD / 4 + T - 1) / T : 1;
        float4 mreg[M4];
        double qreg[R];
#pragma unroll
        for (int r = 0; r < R; ++r) qreg[r] = p.pooled.qbar[((size_t)h * nqb + irow[r]) * kD + lane];
        if (M_LDS)
#pragma unroll
            for (int u = 0; u < M4; ++u)
                mreg[u] = reinterpret_cast<const float4 *>(Mh)[min(u * T + tid, kD * kD / 4 - 1)];
#pragma unroll
        for (int i = 0; i < VT; ++i) load_tile(rsK, wave + NW * i, buf_of(1), res[i]);
#pragma unroll
        for (int r = 0; r < R; ++r) row_vec(0, wave * R + r)[lane] = qreg[r];
        if (M_LDS)
#pragma unroll
            for (int u = 0; u < M4; ++u) {
                const int e = 4 * (u * T + tid);
                if (e < kD * kD) {
                    float *dst = Ms + (e >> 6) * (kD + 1) + (e & 63);
                    dst[0] = mreg[u].x;
                    dst[1] = mreg[u].y;
                    dst[2] = mreg[u].z;
                    dst[3] = mreg[u].w;
                }
            }
    }
    __syncthreads();  // M_h and every row's Qbar in place

    // Pooled logits Qbar_i . Kbar_j / sqrt(D) (Eq. 1), softmax over all key blocks.
    dot_pass(0, rsK, res);
#pragma unroll
    for (int i = 0; i < VT; ++i) load_tile(rsV, wave + NW * i, buf_of(1), res[i]);
    double P[R][CPL], S2[R][CPL];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int nkb = nkb_here();
        double mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            P[r][c] = own(r)[c * 64 + lane] * 0.125;  // 1/sqrt(64)
            if (lane + 64 * c < nkb) mx = fmax(mx, P[r][c]);
        }
        mx = wave_max(mx);
        double z = 0.0;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            P[r][c] = lane + 64 * c < nkb ? exp(P[r][c] - mx) : 0.0;
            z += P[r][c];
            slot_fence(c);
        }
        z = wave_sum(z);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            P[r][c] = P[r][c] / z;
            slot_fence(c);
        }
        if (p.prob_out && live[r]) {
            const int nkb = nkb_here();
            double *po = p.prob_out + ((size_t)h * nqb + irow[r]) * nkb;
#pragma unroll
            for (int c = 0; c < CPL; ++c)
                if (lane + 64 * c < nkb) po[lane + 64 * c] = P[r][c];
        }
    }

    // Dense pooled output vbar_i = sum_j P_ij Vbar_j, w_i = S vbar_i with S the symmetric
    // part of M (lane <-> channel), and vbar_i^T S vbar_i.
    double vb[R], vsv[R];
    wsum_pass([&](int r, int c) { return P[r][c]; }, vb);
#pragma unroll
    for (int r = 0; r < R; ++r) row_vec(0, wave * R + r)[lane] = vb[r];
    mv_pass(sym_mv{});
#pragma unroll
    for (int r = 0; r < R; ++r) vsv[r] = wave_sum(vb[r] * row_vec(1, wave * R + r)[lane]);

    // q_ij = e^T M e with e = vbar_i - Vbar_j (Eq. 9), expanded through the symmetric
    // part S of M (same quadratic form): q = vbar_i^T S vbar_i - 2 Vbar_j . w_i +
    // Vbar_j^T M Vbar_j, the last term per block from the pooling pass.
    // s_ij = P_ij sqrt(q_ij), key_ij = s_ij / max(1 - P_ij, eps) (Eqs. 6-7).
    dot_pass(1, rsV, res);

    // Initial selection (Eq. 7), then the state of each drop set (Eqs. 10-12):
    // g = sum_{j in D} P_j (vbar - Vbar_j), K = 1 - sum_{j in D} P_j, G = g^T M g.
    // The criterion picks the ranking: the key (drift), P (probability) or the
    // negated key (drift maximisation from the start). A CDF cap (probability
    // only) shrinks the row's kept count to the shortest descending-P prefix
    // whose mass, forced blocks included, reaches cdf_tau.
    const int crit = p.criterion;
    const bool maximise = crit == RESS_CRITERION_DRIFT_MAX_SWAP || crit == RESS_CRITERION_DRIFT_MAX_FULL;
    const bool capped = crit == RESS_CRITERION_PROBABILITY && p.cdf_tau > 0.0;
    bits inD[R], best[R];
    double K[R], G[R], J[R], Jb[R], msum[R];  // wave-uniform
    int crow[R];  // kept candidates of the row
    // Order keys go into the row's staging row (this lane's slots only).
    auto put_key = [&](int r, int c, double x) __attribute__((always_inline)) {
        own(r)[c * 64 + lane] = __longlong_as_double((long long)order_key(x));
    };
#pragma unroll
    for (int r = 0; r < R; ++r) {
        double acc[CPL];
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c] = own(r)[c * 64 + lane];
        // The block with P > 1/2, if a row has one (at most one does): there e = vbar_i -
        // Vbar_j shrinks with 1 - P while the expansion's terms do not, so the expansion
        // would leave mostly rounding error (a single-block row: e = 0 exactly). Its q is
        // taken directly as e^T M e (e through the row's staging row, read out above):
        // lane t forms e_t (M e)_t.
        const int nkb = nkb_here();
        int dom_c = -1, dom_l = 0;
        double q_dom = 0.0;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const unsigned long long b = __ballot(lane + 64 * c < nkb && P[r][c] > 0.5);
            if (b != 0ull) {
                dom_c = c;
                dom_l = __builtin_ctzll(b);
            }
        }
        if (dom_c >= 0) {
            double *ebuf = own(r);
            const double e = vb[r] - pooled_row(rsV, dom_l + 64 * dom_c, lane);
            __builtin_amdgcn_wave_barrier();
            ebuf[lane] = e;
            __builtin_amdgcn_wave_barrier();
            double u = 0.0;
            for (int c = 0; c < kD; ++c) u = fma(m_at(lane, c), ebuf[c], u);
            __builtin_amdgcn_wave_barrier();
            q_dom = wave_sum(e * u);
        }
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const double cj = cT[min(lane + 64 * c, nkb - 1)];
            const double q = (c == dom_c && lane == dom_l) ? q_dom : fma(-2.0, acc[c], vsv[r] + cj);
            const double s = P[r][c] * sqrt(q > 0.0 ? q : 0.0);
            const double den = 1.0 - P[r][c];
            S2[r][c] = s * s;
            acc[c] = s / (den > eps ? den : eps);  // ranking key
            slot_fence(c);
        }
        if (p.key_out && live[r]) {
            const int nkb = nkb_here();
            double *ko = p.key_out + ((size_t)h * nqb + irow[r]) * nkb;
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const int j = lane + 64 * c;
                if (j < nkb) ko[j] = j < n_p ? acc[c] : -1.0;
            }
        }
        inD[r] = 0;
        crow[r] = c_h;
        if (!dense[r]) {
#pragma unroll
            for (int c = 0; c < CPL; ++c)
                put_key(r, c, crit == RESS_CRITERION_PROBABILITY ? P[r][c]
                              : crit == RESS_CRITERION_DRIFT_MAX_FULL ? -acc[c] : acc[c]);
            const double *keys = own(r) + lane;
            if (capped) {
                // mass(n) = forced mass + the n largest candidate P: smallest n <= c_h
                // with mass(n) >= tau by bisection (mass is non-decreasing in n).
                const int nkb = nkb_here();
                double fm = 0.0;
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    const int j = lane + 64 * c;
                    if (j < nkb && j >= n_p) fm += P[r][c];
                }
                fm = wave_sum(fm);
                auto mass = [&](int n) {
                    const bits sel = topk_slots<CPL>(keys, cand_bits, n, lane_lt);
                    double m = 0.0;
#pragma unroll
                    for (int c = 0; c < CPL; ++c)
                        if ((sel >> c) & 1) m += P[r][c];
                    return fm + wave_sum(m);
                };
                int lo = 0, hi_n = c_h;
                if (mass(hi_n) >= p.cdf_tau) {
                    while (lo < hi_n) {
                        const int mid = (lo + hi_n) >> 1;
                        if (mass(mid) >= p.cdf_tau)
                            hi_n = mid;
                        else
                            lo = mid + 1;
                    }
                    const int floor2 = max(0, 2 - (nkb - n_p));
                    crow[r] = max(lo, min(floor2, n_p));
                }
            }
            const bits keep = topk_slots<CPL>(keys, cand_bits, crow[r], lane_lt);
            inD[r] = cand_bits & ~keep;
        }
        double mass = 0.0;
#pragma unroll
        for (int c = 0; c < CPL; ++c) mass += ((inD[r] >> c) & 1) ? P[r][c] : 0.0;
        msum[r] = wave_sum(mass);
        K[r] = uniform(1.0 - msum[r]);
    }
    // g = sum_{j in D} P_j (vbar - Vbar_j) = (sum_{j in D} P_j) vbar - sum_{j in D} P_j Vbar_j
    double gr[R];
    wsum_pass([&](int r, int c) { return ((inD[r] >> c) & 1) ? P[r][c] : 0.0; }, gr);
#pragma unroll
    for (int r = 0; r < R; ++r) gr[r] = fma(msum[r], vb[r], -gr[r]);
    // h = M g, G = g . h, J = G / max(K, eps)^2, and vbar . h for the next round's gains.
    double vmg[R];
    auto objective = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < R; ++r) row_vec(0, wave * R + r)[lane] = gr[r];
        mv_pass(plain_mv{});
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double hh = row_vec(1, wave * R + r)[lane];
            wave_sum2(gr[r] * hh, vb[r] * hh, G[r], vmg[r]);
            const double Kh = K[r] > eps ? K[r] : eps;
            J[r] = uniform(G[r] / (Kh * Kh));
            G[r] = uniform(G[r]);
            vmg[r] = uniform(vmg[r]);
        }
    };
    objective();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        Jb[r] = J[r];
        if (p.drift && live[r] && lane == 0) p.drift[2 * ((size_t)h * nqb + irow[r])] = J[r];
        best[r] = inD[r];
    }

    // Budget-neutral restoration rounds (Eqs. 13-17) with track-best. The swap
    // count follows each row's kept count; the workgroup stops once no row of it
    // swaps anything (the rows that are not dense keep c_h candidates each, unless a
    // CDF cap makes the counts differ).
    auto swaps = [&](int kept, double share) {  // share = rho 2^-(r+1) of round r (Eq. 17)
        return min(max((int)floor(share * (double)kept), p.swap_floor), min(n_p - kept, kept));
    };
    const bool any_row = (item % groups) * RW < p.first_dense_qb && c_h < n_p;
    double share = p.rho;
    for (int rr = 0; rr < p.rounds; ++rr) {
        share *= 0.5;
        const int m_all = __builtin_amdgcn_readfirstlane(swaps(c_h, share));
        if (capped) {
            int mmax = 0;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (!dense[r]) mmax = max(mmax, swaps(crow[r], share));
            if (lane == 0) flags[wave] = mmax;
            __syncthreads();
            mmax = 0;
            for (int w = 0; w < NW; ++w) mmax = max(mmax, flags[w]);
            __syncthreads();
            if (mmax <= 0) break;
        } else if (!any_row || m_all <= 0) {
            break;
        }
        // (Negated copies of P are formed where they are used, not kept over the rounds.)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < CPL; ++c) asm("" : "+v"(P[r][c]));
        // e_k . (M g) = vbar . (M g) - Vbar_k . (M g) for every candidate k of every row.
        dot_pass(1, rsV, res);
        // Gains of every single restore / drop at the round-start state; the m best
        // of each kind are applied together, g and K following Eq. 13.
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int m = dense[r] ? 0 : (capped ? swaps(crow[r], share) : m_all);
            if (m <= 0) continue;
            // Eqs. 14-16 with P_k negated for the blocks outside the drop set:
            // dG = -2 P_k e_k . (M g) + s_k^2, K' = K + P_k, dJ = J - (G + dG) / max(K', eps)^2.
            auto gains = [&](auto quotient) __attribute__((always_inline)) {
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    const double sp = ((inD[r] >> c) & 1) ? P[r][c] : -P[r][c];
                    const double ek = vmg[r] - own(r)[c * 64 + lane];
                    const double num = fma(-2.0 * sp, ek, G[r] + S2[r][c]);
                    const double Kn = K[r] + sp;
                    const double Knh = Kn > eps ? Kn : eps;
                    const double dJ = J[r] - quotient(num, Knh * Knh);
                    put_key(r, c, maximise ? -dJ : dJ);
                    slot_fence(c);
                }
            };
            if (eps >= 1e-100 && eps <= 1e100)  // the divisor, at least eps^2, is far from the range's ends
                gains([](double x, double d) { return quot(x, d); });
            else
                gains([](double x, double d) { return x / d; });
            const double *keys = own(r) + lane;
            const bits rest = topk_slots<CPL>(keys, inD[r], m, lane_lt);
            const bits drop = topk_slots<CPL>(keys, cand_bits & ~inD[r], m, lane_lt);
            inD[r] = (inD[r] & ~rest) | drop;
            double mr = 0.0, md = 0.0;
            // The swapped blocks, in slot order, are gathered into a list of (block, weight)
            // pairs in the row's staging row (its keys are no longer needed; where the row
            // might not hold them all, half of the slots at a time) and applied 8 rows of Vbar
            // at a time: restores subtract d_k, drops add it. The list is padded to a multiple
            // of 8 with zero-weight entries of block 0, which leave g unchanged.
            int lane_here = lane;  // block indices formed here, not kept per slot
            asm("" : "+v"(lane_here));
            constexpr int HALF = (CPL + 1) / 2;
            static_assert((64 * HALF + 8) * 12 <= SROW * 8, "swap list");
            double *swap_w = own(r);
            int *swap_j = reinterpret_cast<int *>(own(r) + 64 * HALF + 8);
            int nbuf = 0;
            auto apply = [&]() __attribute__((always_inline)) {
                const int nr = (nbuf + 7) & ~7;
                if (lane < nr - nbuf) {
                    swap_j[nbuf + lane] = 0;
                    swap_w[nbuf + lane] = 0.0;
                }
                asm volatile("" ::: "memory");
                for (int t0 = 0; t0 < nr; t0 += 8) {
                    double vj[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) vj[u] = pooled_row(rsV, swap_j[t0 + u], lane);
#pragma unroll
                    for (int u = 0; u < 8; ++u) gr[r] = fma(swap_w[t0 + u], vb[r] - vj[u], gr[r]);
                }
                nbuf = 0;
                asm volatile("" ::: "memory");
            };
            asm volatile("" ::: "memory");  // the row changes its type
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                if (c == HALF && 2 * m > 64 * HALF) apply();  // the rest may not fit beside these
                const bool is_rest = (rest >> c) & 1ull, is_drop = (drop >> c) & 1ull;
                const unsigned long long sm = __ballot(is_rest || is_drop);
                if (sm == 0ull) continue;
                if (is_rest || is_drop) {
                    const int pos = nbuf + __popcll(sm & lane_lt);
                    swap_j[pos] = lane_here + 64 * c;
                    swap_w[pos] = is_drop ? P[r][c] : -P[r][c];
                }
                if (is_rest) mr += P[r][c];
                if (is_drop) md += P[r][c];
                nbuf += __popcll(sm);
            }
            if (nbuf > 0) apply();
            K[r] = uniform(K[r] + wave_sum(mr - md));
        }
        objective();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (!dense[r] && (maximise ? J[r] > Jb[r] : J[r] < Jb[r])) {
                Jb[r] = J[r];
                best[r] = inD[r];
            }
    }

    // Kept lists: (P \ D_best) u F in ascending block order, padded with -1.
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!live[r]) continue;
        const int nkb = nkb_here();
        const size_t row = (size_t)h * nqb + irow[r];
        int32_t *out = p.kept_idx + row * nkb;
        int before = 0;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const bool kept = lane + 64 * c < nkb && !((best[r] >> c) & 1);
            const unsigned long long km = __ballot(kept);
            if (kept) out[before + __popcll(km & lane_lt)] = lane + 64 * c;
            before += __popcll(km);
        }
        for (int t = before + lane; t < nkb; t += 64) out[t] = -1;
        if (lane == 0) {
            p.kept_count[row] = before;
            if (p.drift) p.drift[2 * row + 1] = Jb[r];
        }
    }
}

template <int CPL, int R, int NW, int WPC = 1>
hipError_t launch_cfg(const SelectParams &p, hipStream_t s)
{
    SelectParams q = p;
    const int groups = (p.n_qb + NW * R - 1) / (NW * R);
    q.items_per_xcd = (p.H * groups + 7) / 8;
    hipLaunchKernelGGL((select_kernel<CPL, R, NW, WPC>), dim3((unsigned)(8 * q.items_per_xcd)), dim3(NW * 64), 0, s, q);
    return hipGetLastError();
}

// Rows per workgroup: 4, 8, 12 or 16 waves of one row, or (up to 6 slots per lane) 12
// waves of two, by the smallest number of rounds of workgroups over the chip's 256
// compute units times the time of one workgroup. The latter were measured per round
// over 8, 16, 32 and 100 views (us with 4 / 8 / 12 / 16 / 24 rows): 67 / 73 / 85 / 90 /
// 158 at 344 key blocks, - / 129 / 140 / 158 at 687, - / 176 / 193 / 231 at 1,074; more
// waves hide each other's latencies until they share the vector unit, more rows per
// wave only add up. In hundredths of 8 rows: 90, 100, 112, 127, 210. (Every shape tried
// at 21 key-block counts from 3 to 1,074 and 4 to 256 heads: the rule takes the fastest
// or one within 2% of it.)
// Up to 2 slots there is also 8 waves of two, two workgroups a CU, 215 for two at once
// and 135 for a CU's odd last one: layers of many heads and few key blocks fill the chip
// several times over, where full 16-row tiles and two workgroups in turn count for more
// than a row's latency. At 100 key blocks, 64 / 128 / 256 heads: 154 / 295 / 549 us
// without it, 139 / 264 / 486 with it; 128 key blocks 175 / 339 / 677 and 160 / 307 / 604.
constexpr long long kCUs = 256;
template <int CPL>
hipError_t launch_rows(const SelectParams &p, hipStream_t s)
{
    auto rounds = [&](int rows) {
        const long long wg = (long long)p.H * ((p.n_qb + rows - 1) / rows);
        return (wg + kCUs - 1) / kCUs;
    };
    int best = 8;
    long long bc = rounds(8) * 100;
    auto consider = [&](int rows, int weight) {
        if (rounds(rows) * weight < bc) best = rows, bc = rounds(rows) * weight;
    };
    consider(4, 90);
    consider(12, 112);
    consider(16, 127);
    if constexpr (CPL <= 6) consider(24, 210);
    if constexpr (CPL <= 2) {
        const long long each = rounds(16);
        if (each / 2 * 215 + each % 2 * 135 < bc) return launch_cfg<CPL, 2, 8, 2>(p, s);
    }
    if constexpr (CPL <= 6)
        if (best == 24) return launch_cfg<CPL, 2, 12>(p, s);
    if (best == 16) return launch_cfg<CPL, 1, 16>(p, s);
    if (best == 12) return launch_cfg<CPL, 1, 12>(p, s);
    if (best == 8) return launch_cfg<CPL, 1, 8>(p, s);
    return launch_cfg<CPL, 1, 4>(p, s);
}

}  // namespace

hipError_t launch_select(const SelectParams &p, hipStream_t s)
{
    if (p.H == 0 || p.n_qb == 0) return hipSuccess;
    const int n = p.n_kb;
    if (n <= 128) return launch_rows<2>(p, s);
    if (n <= 256) return launch_rows<4>(p, s);
    if (n <= 384) return launch_rows<6>(p, s);
    if (n <= 512) return launch_rows<8>(p, s);
    if (n <= 768) return launch_rows<12>(p, s);
    if (n <= 1088) return launch_rows<17>(p, s);
    if (n <= 1536) return launch_cfg<24, 1, 8>(p, s);
    if (n <= 2304) return launch_cfg<36, 1, 8>(p, s);
    return launch_cfg<64, 1, 4>(p, s);
}

}  // namespace ress
