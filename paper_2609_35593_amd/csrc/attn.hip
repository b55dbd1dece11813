// Exact attention over kept key blocks (block-sparse, Sec. 3 step (3)) or over
// all key blocks (dense), bf16 inputs, bf16 MFMA products with float32
// accumulation, float32 online softmax.
//
// One workgroup per (head, query block), G groups of BQ/32 waves (G = 1 but for small
// layers, see launch_bk), each wave owning 32 query rows. The score tile is computed
// transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16: its accumulator puts one
// query per lane (lane l and l+32 share query l%32, each holding 16 of every 32 keys),
// so row sums stay in the lane except for one exchange with lane l^32, and the
// probabilities already sit in the B-operand layout of O^T = V^T P^T.
//
// Keys are consumed in 64-key chunks (one 64-key block of the kept list, or half of a
// 128-key block). A chunk is two 32-key sub-tiles; a wave issues the 4 score MFMAs of
// each, forms the probabilities and issues the 8 PV MFMAs. Latency is hidden by
// occupancy rather than by a software pipeline across chunks: K and V chunks sit in
// two-slot rings of 8 KB per tensor and slot (32 KB per group), and the kernel fits
// 128 registers, so four single-group 128-query workgroups, or two of two groups or
// one of four, share a CU (four waves per SIMD), and the matrix and vector pipes of a
// SIMD serve whichever of its waves is ready. (Measured: at D = 64 the softmax needs
// about as many issue slots as the MFMAs; two waves per SIMD with a software pipeline
// reached the same rate as three without one, four waves run 4-8% faster.)
//
// Chunks move from global memory straight into LDS (buffer_load ... lds, 16
// bytes per lane, 1 KB per wave instruction, 32-bit offsets against a per-head
// buffer resource): chunk c+1 is loaded while chunk c is computed, and one
// barrier per chunk both publishes chunk c+1 and frees chunk c's slots. Rows stay
// row-major (64 channels = 128 bytes per key) with their 16-byte chunks
// XOR-swizzled per key; the swizzle is applied by choosing each lane's source
// chunk, since a DMA instruction fills LDS contiguously. The V^T operand comes
// from ds_read_b64_tr_b16: within 16 lanes, lane s points at 4 channels of key
// k0 + s/4 and lane i receives channel d0 + i of keys k0..k0+3, which is the
// transpose the PV product needs. The kept list is read through the scalar
// cache (wave-uniform addresses).
//
// Softmax: base-2 exponentials; row sums over the bf16-rounded probabilities
// (the values the PV product consumes) with packed bf16 dot products. There is
// no per-tile maximum: every row starts with reference 0. While every row of a wave
// has reference 0, the wave runs a loop of its own whose probabilities are exp2 of the
// score accumulators with nothing else: Q is multiplied by scale*log2(e) when its
// fragments are loaded (one extra bf16 rounding of Q), so the accumulators are base-2
// logits. It looks at a chunk's sum once, before the PV products: when it exceeds 2^50,
// or the row's running sum is still below 2^-100, the wave goes over to the general
// loop with that chunk. There every row forms its probabilities against its own
// reference, and a chunk that leaves the same range is formed again after the row's
// reference has moved to 32 above its largest base-2 logit (O rescaled), which leaves
// room on both sides. A wave whose first 64 scores reach beyond +-24 in some row
// reloads Q unscaled and starts in the general loop, its references taken from those
// scores, so large logits are formed exactly; either way every score of a row has one
// form (all key groups of a row take their choice from the list's first 64 keys).
// Softmax is invariant to the reference, so this changes rounding only.
// (Measured, one loop over both forms with a look at every sub-tile -> two loops, one
// look a chunk: the compiler kept two copies of O and moved all of it every other
// chunk; 32 views, 75% sparsity 2,020 -> 1,885 us, dense 7,680 -> 7,165, 1,105 TFLOP/s.
// In the general loop, with Q 12 times as large, the one loop took 2,375 and 8,629 us at
// 32 views and 652 and 2,212 at 16; a general loop that looked at each sub-tile and
// rounded references within +-40 to 0 2,500 and 9,070, 779 and 2,488; this one 2,159 and
// 8,172, 588 and 2,097. References 32 above the largest logit rather than at it save
// 5-12% with Q 30 times as large.)
//
// Workgroups are numbered so that neighbouring query blocks of a head share an
// XCD and its L2, where their K/V chunks are re-read, and heads of different cost
// (ragged budgets) still split evenly over the XCDs (see row_of).
#include <type_traits>

#include "ress_internal.h"

namespace ress {
namespace {

typedef __bf16 bf16x8 __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef __bf16 bf16x2 __attribute__((__vector_size__(2 * sizeof(__bf16))));
typedef short s16x4 __attribute__((__vector_size__(4 * sizeof(short))));
typedef float f32x16 __attribute__((__vector_size__(16 * sizeof(float))));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr float kSumLimit = 0x1p50f;  // largest probability sum a chunk may reach
constexpr float kTiny = 0x1p-100f;    // a row whose running sum is below this has no usable reference
constexpr float kHeadroom = 32.f;     // a new reference's distance above the row's largest logit so far
constexpr float kStartBand = 24.f;    // first-chunk maxima a wave may have to start with reference 0

__device__ __forceinline__ unsigned int bf16_bits(float x)
{
    return (unsigned int)__builtin_bit_cast(unsigned short, (__bf16)x);
}

// XOR applied to the 16-byte chunk index of LDS row `row` (K and V tiles, 128-byte
// rows, two rows per 256-byte bank row). With s = swz(row):
//  - 16 consecutive rows read at one logical chunk (score operand, 16 lanes x 16 B)
//    land on 16 distinct (bank half, chunk) pairs, since (row>>1)&7 -> s is a bijection;
//  - the transpose reads (32 lanes x 8 B: keys 8n..8n+3 or 8n+4..8n+7, each at the 4
//    chunks of one 32-channel half) are split by bit 2 of s between rows 8n and 8n+2.
__device__ __forceinline__ int swz(int row) { return (((row >> 1) & 1) << 2) | ((row >> 2) & 3); }

__device__ __forceinline__ void wait_vm_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)

// Work order, two forms; within a head, last blocks first (the dense special
// blocks early). Returns false for a workgroup with no row.
//  - Segments (the K and V of all heads fit the infinity cache): the (head, query
//    block) rows, head-major, are cut into 8 contiguous segments of about equal
//    work, one per XCD, so that each XCD fills its L2 with few heads' K and V
//    (neighbouring query blocks of a head share it) while ragged per-head budgets
//    stay balanced. A row's work is its head's kept count of query block 0 (the
//    rows of a head keep the same number of blocks, the dense special rows aside;
//    dense attention: equal). Boundaries follow the work split, clamped so that no
//    segment exceeds seg_cap rows (the grid is 8 x seg_cap workgroups; every row
//    lands in exactly one segment).
//  - Rotation (larger layers): XCD x runs, head after head, a chunk of seg_cap
//    consecutive query blocks of every head, chunk (x - h) mod 8 of head h, so
//    that each head's chunks are spread over all XCDs and the XCDs move through the
//    heads together (the grid is 8 x H x seg_cap workgroups).
__device__ __forceinline__ bool row_of(const AttnParams &p, bool sparse, int xcd, int local, int &h, int &i)
{
    const int H = p.H, n = p.n_qb;
    if (p.rotate) {
        const int chunk = p.seg_cap;
        const int slot = local / chunk, r = local - slot * chunk;
        if (slot >= H) return false;
        h = (xcd + slot) % H;
        const int i_fwd = ((xcd - h % 8 + 8) & 7) * chunk + r;
        if (i_fwd >= n) return false;
        i = n - 1 - i_fwd;
        return true;
    }
    const long long T = (long long)H * n, cap = p.seg_cap;
    // Lane l holds the weights of heads l, l + 64, ... and their running sums (one load
    // and one scan for all of them: head after head, each a dependent load, this took up
    // to 10 us of every workgroup on the last XCDs).
    constexpr int HC = RESS_MAX_HEADS / 64;
    const int lane = threadIdx.x & 63;
    int w[HC], sum[HC], total = 0;
    if (sparse) {
#pragma unroll
        for (int c = 0; c < HC; ++c) {
            w[c] = sum[c] = 0;
            if (64 * c < H) {
                const int hh = 64 * c + lane;
                if (hh < H) w[c] = min(max(p.kept_count[(size_t)hh * n], 1), p.n_kb);  // sums fit 31 bits
                int x = w[c];
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int y = __shfl_up(x, o);
                    x += lane >= o ? y : 0;
                }
                sum[c] = total + x;
                total = __builtin_amdgcn_readlane(sum[c], 63);
            }
        }
    } else {
        total = H;
    }
    const long long W = (long long)total * n;
    // First row whose work prefix reaches x W / 8.
    auto split = [&](int x) -> long long {
        const long long target = (W / 8) * x + ((W % 8) * x + 7) / 8;
        if (!sparse) return target;
#pragma unroll
        for (int c = 0; c < HC; ++c)
            if (64 * c < H) {
                const unsigned long long at =
                    __builtin_amdgcn_ballot_w64(64 * c + lane < H && (long long)sum[c] * n >= target);
                if (at != 0ull) {
                    const int l = __builtin_ctzll(at);
                    const int wl = __builtin_amdgcn_readlane(w[c], l);
                    const long long acc = (long long)(__builtin_amdgcn_readlane(sum[c], l) - wl) * n;
                    // target - acc <= wl n < 2^31
                    return (long long)(64 * c + l) * n + ((int)(target - acc) + wl - 1) / wl;
                }
            }
        return T;
    };
    long long b = 0, e = 0;
    for (int x = 1; x <= xcd + 1; ++x) {
        const long long lo = max(e, T - (8 - x) * cap), hi = min(e + cap, T);
        b = e;
        e = min(max(split(x), lo), hi);
    }
    const int g = (int)b + local;  // rows < 2^31 (checked on the host)
    if (g >= (int)e) return false;
    h = g / n;
    i = n - 1 - (g - h * n);
    return true;
}

// Four waves per SIMD for 128-query blocks (four 32 KB workgroups per CU); 64-query
// blocks are held to two by the LDS (five 2-wave workgroups per CU).
//
// G > 1: G groups of BQ/32 waves share a query block, group g with its own slots taking
// chunks g, g + G, ... of its list; the groups' O and sums are merged through the
// slots at the end.
template <int BQ, int BK, bool SPARSE, int G>
__global__ void __launch_bounds__(BQ * 2 * G, BQ == 128 ? 4 : 2) attn_kernel(const AttnParams p)
{
    constexpr int T = BQ * 2;                 // threads of a group
    constexpr int NW = BQ / 32;               // waves of a group
    constexpr int CPE = BK / 64;              // 64-key chunks per kept-list entry
    constexpr int LPC = 64 * 8 / T;           // 16-byte DMA loads per thread, tensor and chunk
    constexpr int SLOT = 64 * 128;            // bytes of one chunk of K (or V)
    static_assert(64 * 8 % T == 0 && LPC >= 1, "a chunk must split evenly over the threads");
    __shared__ __attribute__((aligned(1024))) unsigned char k_a0[G * SLOT];
    __shared__ __attribute__((aligned(1024))) unsigned char k_a1[G * SLOT];
    __shared__ __attribute__((aligned(1024))) unsigned char v_a0[G * SLOT];
    __shared__ __attribute__((aligned(1024))) unsigned char v_a1[G * SLOT];

    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    int h, i;
    if (!row_of(p, SPARSE, xcd, local, h, i)) return;
    const int N = p.N, n_kb = p.n_kb;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = G > 1 ? wave_wg / NW : 0, wave = wave_wg - grp * NW;  // key group, wave within it
    unsigned char *const k_s0 = k_a0 + grp * SLOT, *const k_s1 = k_a1 + grp * SLOT;
    unsigned char *const v_s0 = v_a0 + grp * SLOT, *const v_s1 = v_a1 + grp * SLOT;
    const int hh = lane >> 5, ql = lane & 31;
    const int g16 = (lane >> 4) & 1, s16 = lane & 15;
    const int q0 = i * BQ + wave * 32 + ql;
    const size_t head = (size_t)h * N;

    // Q fragments, pre-multiplied by scale*log2(e) so that scores are base-2 logits,
    // unless the wave's first scores show logits beyond kStartBand (then unscaled).
    const float c = p.scale_log2;
    bf16x8 qf[4];
    auto load_q = [&](bool scaled) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            if (q0 < N) {
                const bf16x8 x = *reinterpret_cast<const bf16x8 *>(p.q + (head + q0) * kD + kk * 16 + hh * 8);
                if (scaled) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) qf[kk][e] = (__bf16)((float)x[e] * c);
                } else {
                    qf[kk] = x;
                }
            } else {
                qf[kk] = bf16x8{};
            }
        }
    };
    load_q(true);

    int n_ent;  // key blocks to visit
    const int32_t *list = nullptr;
    if constexpr (SPARSE) {
        const size_t row = (size_t)h * p.n_qb + i;
        n_ent = min(max(p.kept_count[row], 0), n_kb);
        list = p.kept_idx + row * n_kb;
    } else {
        n_ent = n_kb;
    }
    int C_all = n_ent * CPE;  // 64-key chunks of the list
    if (CPE == 2 && n_ent > 0 && N - (n_kb - 1) * BK <= 64) {
        // The last block holds at most 64 tokens: its second chunk is empty.
        int jl;
        if constexpr (SPARSE) jl = list[n_ent - 1];
        else jl = n_ent - 1;
        if (__builtin_amdgcn_readfirstlane(jl) == n_kb - 1) C_all -= 1;
    }
    // This group's chunks: chunk ch of the group is chunk grp + G ch of the list.
    const int C = (C_all - grp + G - 1) / G;

    // Kept block indices through the scalar cache (wave-uniform addresses; the list
    // is read-only here).
    typedef const __attribute__((address_space(4))) int32_t cint32;
    const cint32 *klist = (const cint32 *)list;
    auto block_of = [&](int ch) __attribute__((always_inline)) -> int {
        const int e = (grp + G * ch) / CPE;
        if constexpr (SPARSE) return e < n_ent ? klist[e] : -1;
        else return e < n_ent ? e : -1;
    };
    // First token of chunk ch of block j, and how many of its 64 keys are real (none for
    // an entry outside the layer).
    auto chunk_row0 = [&](int j, int ch) __attribute__((always_inline)) -> int {
        return j >= 0 && j < n_kb ? j * BK + 64 * ((grp + G * ch) & (CPE - 1)) : N;
    };
    auto chunk_keys = [&](int row0) __attribute__((always_inline)) -> int { return N - row0 < 64 ? N - row0 : 64; };

    // This head's K and V as buffer resources: N * 128 bytes (at most 2^31 for
    // N <= 2^24, as a 32-bit unsigned record count; row offsets stay below 2^31).
    const int head_bytes = (int)((unsigned int)N * 128u);
    const __amdgpu_buffer_rsrc_t krs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.k + head * kD), 0, head_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t vrs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.v + head * kD), 0, head_bytes, 0x00020000);
    // DMA lane constants: load u of a thread fills row r0 + 8 NW u of the slot, at
    // physical chunk lane & 7, from source chunk (lane & 7) ^ swz(row) (the same for
    // every u: the swizzle depends on row bits 1-3 only).
    const int r0 = wave * 8 + (lane >> 3);
    const unsigned int coff = (unsigned int)(((lane & 7) ^ swz(r0)) << 4);
    unsigned int doff[LPC];  // byte offsets of a full chunk's loads, against the chunk's first row
#pragma unroll
    for (int u = 0; u < LPC; ++u) doff[u] = (unsigned int)((r0 + 8 * NW * u) * 128) + coff;
    // Rows row0..row0+63 of one tensor into a slot; rows past N repeat row N-1 (the chunks
    // that have any, and entries outside the layer, take the second form).
    auto dma_chunk = [&](__amdgpu_buffer_rsrc_t rs, int row0, unsigned char *dst) __attribute__((always_inline)) {
        if (row0 + 64 <= N) {
#pragma unroll
            for (int u = 0; u < LPC; ++u) {
                const unsigned int off = doff[u];
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(dst + (u * NW + wave) * 1024), 16, off,
                                                         row0 * 128, 0, 0);
            }
        } else {
#pragma unroll
            for (int u = 0; u < LPC; ++u) {
                const unsigned int off = (unsigned int)(min(row0 + r0 + 8 * NW * u, N - 1) * 128) + coff;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(dst + (u * NW + wave) * 1024), 16, off, 0, 0,
                                                         0);
            }
        }
    };

    // Per-lane LDS byte offsets of the operand reads (chunk-relative; the key offset
    // of a sub-tile is added as an immediate).
    int koff[4];  // score operand: key ql, logical chunk 2kk+hh
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) koff[kk] = ql * 128 + (((2 * kk + hh) ^ swz(ql)) << 4);
    int voff[2][2];  // transpose reads: key 8r + 4hh + s16/4, channels 32dh + 16g16 + 4(s16&3)
#pragma unroll
    for (int dh = 0; dh < 2; ++dh)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int key = 8 * r + 4 * hh + (s16 >> 2);
            const int d = 32 * dh + 16 * g16 + 4 * (s16 & 3);
            voff[dh][r] = key * 128 + (((d >> 3) ^ swz(key)) << 4) + (d & 7) * 2;
        }

    float mref = 0.f;   // reference of this lane's query row (shared with lane^32), base-2 logits
    float cw = 1.f;     // wave-uniform: base-2 logit per unit score (1 for pre-scaled Q, else c)
    float lrow = 0.f;
    float lpart = 0.f;  // lane^32's part of the row's sum, as of the last change of reference
    f32x16 acc_o[2];
#pragma unroll
    for (int dh = 0; dh < 2; ++dh)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_o[dh][v] = 0.f;
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

    // S^T of sub-tile t (32 keys) of a chunk: 4 MFMAs.
    auto qk = [&](const unsigned char *kt, int t, f32x16 &s) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const bf16x8 a = *reinterpret_cast<const bf16x8 *>(kt + t * 32 * 128 + koff[kk]);
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], s, 0, 0, 0);
        }
    };
    // O^T += V^T P^T for sub-tile t, 16 keys per MFMA.
    auto pv = [&](const unsigned char *vt, int t, const bf16x8 (&pb)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int dh = 0; dh < 2; ++dh) {
                const unsigned char *base = vt + (t * 32 + u * 16) * 128;
                const s16x4 r0v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(base + voff[dh][0]));
                const s16x4 r1v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(base + voff[dh][1]));
                const bf16x8 a = __builtin_bit_cast(
                    bf16x8, (short __attribute__((__vector_size__(8 * sizeof(short))))){
                                r0v[0], r0v[1], r0v[2], r0v[3], r1v[0], r1v[1], r1v[2], r1v[3]});
                acc_o[dh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[u], acc_o[dh], 0, 0, 0);
            }
    };
    // Key of element v of sub-tile t: t 32 + (v / 4) 8 + (v % 4) + 4 hh; compared as
    // 4 hh >= nv - (the lane-independent part), a scalar per element.
    const int hh4 = hh * 4;
    auto mask = [&](f32x16 &s, int nv, int t) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int lim = __builtin_amdgcn_readfirstlane(nv - (t * 32 + (v >> 2) * 8 + (v & 3)));
            if (hh4 >= lim) s[v] = -INFINITY;
        }
    };
    // Probabilities of a sub-tile, exp2(s) when every row has reference 0 (z), else
    // exp2(s * cw - mref); l0 and l1 gather the lane's sum of the bf16-rounded values.
    auto probs = [&](auto z, const f32x16 &s, bf16x8 (&pb)[2], float &l0, float &l1) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float e[8];
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) {
                const float x = s[u * 8 + jj];
                e[jj] = __builtin_amdgcn_exp2f(decltype(z)::value ? x : fmaf(x, cw, -mref));
            }
            pb[u] = bf16x8{(__bf16)e[0], (__bf16)e[1], (__bf16)e[2], (__bf16)e[3],
                           (__bf16)e[4], (__bf16)e[5], (__bf16)e[6], (__bf16)e[7]};
#pragma unroll
            for (int jj = 0; jj < 8; jj += 4) {
                l0 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pb[u][jj], pb[u][jj + 1]}, ones, l0, false);
                l1 = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pb[u][jj + 2], pb[u][jj + 3]}, ones, l1, false);
            }
        }
    };
    using general = std::integral_constant<bool, false>;
    using zero = std::integral_constant<bool, true>;
    // New references for a chunk that leaves the range (its probabilities are then formed
    // again): each row's true maximum over the chunk; O and the running sum rescaled.
    auto rescale = [&](const unsigned char *ks, int nv) __attribute__((always_inline)) {
        float tmax = -INFINITY;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x16 s;
            qk(ks, t, s);
            mask(s, nv, t);
#pragma unroll
            for (int v = 0; v < 16; ++v) tmax = fmaxf(tmax, s[v]);
        }
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32)) * cw + kHeadroom;
        // Decisions about the row's mass use the row's running sum: lanes l and
        // l^32 each sum half of the row's keys (one of them may have no mass yet
        // while the row has), and both must take the same reference.
        lpart = __shfl_xor(lrow, 32);
        const float lsum = lrow + lpart;
        // The reference only rises, except while the row has no usable mass yet:
        // then it may fall to this chunk's maximum, but not below
        // mref + log2(lsum), an upper bound of every earlier logit of the row, so
        // that the rescaled running sums stay at most 1 (finite).
        float mnew = fmaxf(mref, tmax);
        // (log2 of a denormal sum may come back as -inf: -149 bounds it.)
        if (lsum < kTiny) mnew = lsum > 0.f ? fmaxf(tmax, mref + fmaxf(__log2f(lsum), -149.f)) : tmax;
        if (tmax == -INFINITY) mnew = mref;  // a fully masked chunk says nothing
        // A row without mass has nothing to rescale (and 0 * exp2(large) must not
        // happen); otherwise the factor is applied as two halves, each finite
        // for shifts up to 2^8 (a running sum as small as the smallest denormal).
        const float alpha = lsum > 0.f ? __builtin_amdgcn_exp2f(0.5f * (mref - mnew)) : 0.f;
        lrow = (lrow * alpha) * alpha;
        lpart = (lpart * alpha) * alpha;
#pragma unroll
        for (int dh = 0; dh < 2; ++dh)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc_o[dh][v] = (acc_o[dh][v] * alpha) * alpha;
        mref = mnew;
    };
    // A chunk against the rows' present references (all 0 in the zero form): the
    // probabilities of both sub-tiles are formed first and their sums looked at once.
    // False (rare): the chunk leaves the range.
    // Partial chunks pay for the mask on a real branch (the empty asm keeps the
    // compiler from if-converting it into every sub-tile).
    auto chunk_probs = [&](auto z, const unsigned char *ks, int nv, bf16x8 (&p0)[2], bf16x8 (&p1)[2], float have,
                           float &lh) __attribute__((always_inline)) -> bool {
        // (The compiler's MFMA/LDS interleaving: 2% with key groups, -1% without.)
        if constexpr (G > 1) __builtin_amdgcn_iglp_opt(0);
        float l0 = 0.f, l1 = 0.f;
        {
            f32x16 s;
            qk(ks, 0, s);
            if (nv < 64) {
                asm volatile("" ::: "memory");
                mask(s, nv, 0);
            }
            probs(z, s, p0, l0, l1);
        }
        {
            f32x16 s;
            qk(ks, 1, s);
            if (nv < 64) {
                asm volatile("" ::: "memory");
                mask(s, nv, 1);
            }
            probs(z, s, p1, l0, l1);
        }
        lh = l0 + l1;
        return __builtin_amdgcn_ballot_w64(!(lh <= kSumLimit) || have + lh < kTiny) == 0ull;
    };

    int nv0 = 0, nv1 = 0;  // real keys of chunks ch and ch+1
    int jnext = -1;        // block of chunk ch+1, read one chunk ahead
    // The DMA of chunk ch+1 into (kd, vd), the slots of chunk ch-1 (free since the
    // barrier that ended it).
    auto fetch = [&](int ch, unsigned char *kd, unsigned char *vd) __attribute__((always_inline)) {
        if (ch + 1 < C) {
            const int row1 = chunk_row0(jnext, ch + 1);
            jnext = ch + 2 < C ? block_of(ch + 2) : -1;
            nv1 = chunk_keys(row1);
            dma_chunk(krs, row1, kd);
            dma_chunk(vrs, row1, vd);
        }
    };
    auto finish = [&]() __attribute__((always_inline)) {
        wait_vm_all();    // this wave's loads of the next chunk have landed
        __syncthreads();  // ... and every wave's; this chunk's slots are no longer read
        nv0 = nv1;
    };

    if (G > 1 && C <= 0 && C_all > 0) __syncthreads();  // the others' first chunk
    if (C > 0) {
        {
            const int row0 = chunk_row0(block_of(0), 0);
            nv0 = chunk_keys(row0);
            dma_chunk(krs, row0, k_s0);
            dma_chunk(vrs, row0, v_s0);
            jnext = C > 1 ? block_of(1) : -1;
        }
        wait_vm_all();
        __syncthreads();
        bool zref;  // wave-uniform: every row has reference 0 (Q then is pre-scaled)
        {
            // Start with reference 0 only if every row's first 64 logits lie within
            // kStartBand; otherwise use unscaled Q (exact scores) from the start. Every
            // key group looks at the list's first chunk (group 0's slot, not refilled
            // before the barrier that ends chunk 0): with a choice of their own, the groups
            // could weigh one row's keys by pre-scaled and by exact scores, which differ by
            // up to 2^-8 of the logit.
            float m0 = -INFINITY;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                f32x16 s0;
                qk(k_a0, t, s0);
#pragma unroll
                for (int v = 0; v < 16; ++v) m0 = fmaxf(m0, s0[v]);
            }
            m0 = fmaxf(m0, __shfl_xor(m0, 32));
            zref = __all(fabsf(m0) <= kStartBand);
            if (!zref) {
                load_q(false);
                cw = c;
                // (A whole number: the probabilities round as they do against reference 0.)
                if (fabsf(m0) < INFINITY) mref = rintf(m0) + kHeadroom;
                wait_vm_all();  // Q lands here, not at the first MFMA of every chunk
            }
        }
        int ch = 0;
        // Two loops, so that O keeps its registers in each (one loop over both forms
        // copied all 32 of them every other chunk). A wave leaves the zero form for good
        // with the first chunk that does not fit it (that chunk's successor is on its way by
        // then); its Q stays pre-scaled (cw = 1), so every score of a row has one form.
        bool fetched = false;
        if (zref) {
            auto zero_chunk = [&](const unsigned char *ks, const unsigned char *vs, unsigned char *kd,
                                  unsigned char *vd) __attribute__((always_inline)) -> bool {
                bf16x8 p0[2], p1[2];
                float lh;
                fetch(ch, kd, vd);
                if (!chunk_probs(zero{}, ks, nv0, p0, p1, lrow, lh)) {
                    fetched = true;
                    return false;
                }
                if constexpr (G > 1) __builtin_amdgcn_iglp_opt(0);
                lrow += lh;
                pv(vs, 0, p0);
                pv(vs, 1, p1);
                finish();
                return ++ch < C;
            };
            while (zero_chunk(k_s0, v_s0, k_s1, v_s1) && zero_chunk(k_s1, v_s1, k_s0, v_s0)) {
            }
        }
        auto general_chunk = [&](const unsigned char *ks, const unsigned char *vs, unsigned char *kd,
                                 unsigned char *vd) __attribute__((always_inline)) -> bool {
            bf16x8 p0[2], p1[2];
            float lh;
            if (!fetched) fetch(ch, kd, vd);
            fetched = false;
            if (!chunk_probs(general{}, ks, nv0, p0, p1, lrow + lpart, lh)) {
                rescale(ks, nv0);
                chunk_probs(general{}, ks, nv0, p0, p1, lrow + lpart, lh);
            }
            if constexpr (G > 1) __builtin_amdgcn_iglp_opt(0);
            lrow += lh;
            pv(vs, 0, p0);
            pv(vs, 1, p1);
            finish();
            return ++ch < C;
        };
        // (A copy of the chunk for each slot: slot addresses formed at run time cost 2-8%.
        // Of the ways to enter at either slot, this one leaves O in its registers.)
        bool odd = ch & 1;
        while (ch < C) {
            if (odd || general_chunk(k_s0, v_s0, k_s1, v_s1)) general_chunk(k_s1, v_s1, k_s0, v_s0);
            odd = false;
        }
    }

    if constexpr (G > 1) {
        // Groups with a chunk less wait at its barrier too.
        for (int ch = max(C, 0); ch < (C_all + G - 1) / G; ++ch) __syncthreads();
        // Every group but the first leaves its references, sums and O in LDS (the slots are
        // free): 34 floats a lane, each a row of 64 lanes. The first rescales all of them
        // to the largest reference among the groups that hold mass and adds them up in
        // group order.
        constexpr int PER = 34 * 64;  // floats per wave
        constexpr int FIT = G * SLOT / (PER * 4);  // waves per slot array
        static_assert((G - 1) * NW <= 4 * FIT, "merge area: the four slot arrays");
        auto area = [&](int w) __attribute__((always_inline)) -> float * {
            unsigned char *const a = w < FIT ? k_a0 : w < 2 * FIT ? v_a0 : w < 3 * FIT ? k_a1 : v_a1;
            return reinterpret_cast<float *>(a) + w % FIT * PER;
        };
        lrow += __shfl_xor(lrow, 32);  // lanes l and l^32 share the row
        if (grp > 0) {
            float *m = area((grp - 1) * NW + wave) + lane;
            m[0] = mref;
            m[64] = lrow;
#pragma unroll
            for (int dh = 0; dh < 2; ++dh)
#pragma unroll
                for (int v = 0; v < 16; ++v) m[(2 + dh * 16 + v) * 64] = acc_o[dh][v];
        }
        __syncthreads();
        if (grp > 0) return;
        float mtop = lrow > 0.f ? mref : -INFINITY;
#pragma unroll
        for (int g = 1; g < G; ++g) {
            const float *m = area((g - 1) * NW + wave) + lane;
            if (m[64] > 0.f) mtop = fmaxf(mtop, m[0]);
        }
        const float a0 = lrow > 0.f ? __builtin_amdgcn_exp2f(mref - mtop) : 0.f;
        lrow *= a0;
#pragma unroll
        for (int dh = 0; dh < 2; ++dh)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc_o[dh][v] *= a0;
#pragma unroll
        for (int g = 1; g < G; ++g) {
            const float *m = area((g - 1) * NW + wave) + lane;
            const float a = m[64] > 0.f ? __builtin_amdgcn_exp2f(m[0] - mtop) : 0.f;
            lrow = fmaf(m[64], a, lrow);
#pragma unroll
            for (int dh = 0; dh < 2; ++dh)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc_o[dh][v] = fmaf(m[(2 + dh * 16 + v) * 64], a, acc_o[dh][v]);
        }
    }
    // Each lane summed half of its row's keys; lanes l and l^32 share the row.
    const float ltot = G > 1 ? lrow : lrow + __shfl_xor(lrow, 32);
    const float inv = ltot > 0.f ? 1.f / ltot : 0.f;
    if (q0 < N && p.o32) {
        float *orow = p.o32 + (head + q0) * kD;
#pragma unroll
        for (int dh = 0; dh < 2; ++dh)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int d0 = dh * 32 + g * 8 + hh * 4;
                *reinterpret_cast<float4 *>(orow + d0) =
                    make_float4(acc_o[dh][g * 4 + 0] * inv, acc_o[dh][g * 4 + 1] * inv,
                                acc_o[dh][g * 4 + 2] * inv, acc_o[dh][g * 4 + 3] * inv);
            }
    } else if (q0 < N) {
        uint16_t *orow = p.o + (head + q0) * kD;
#pragma unroll
        for (int dh = 0; dh < 2; ++dh)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int d0 = dh * 32 + g * 8 + hh * 4;
                const unsigned int lo = bf16_bits(acc_o[dh][g * 4 + 0] * inv) |
                                        (bf16_bits(acc_o[dh][g * 4 + 1] * inv) << 16);
                const unsigned int hi = bf16_bits(acc_o[dh][g * 4 + 2] * inv) |
                                        (bf16_bits(acc_o[dh][g * 4 + 3] * inv) << 16);
                *reinterpret_cast<uint2 *>(orow + d0) = make_uint2(lo, hi);
            }
    }
}

template <int BQ, int BK, int G>
hipError_t launch_groups(const AttnParams &p, bool sparse, hipStream_t s)
{
    const dim3 grid((unsigned)(p.rotate ? 8 * p.H * p.seg_cap : 8 * p.seg_cap)), block(BQ * 2 * G);
    if (sparse)
        hipLaunchKernelGGL((attn_kernel<BQ, BK, true, G>), grid, block, 0, s, p);
    else
        hipLaunchKernelGGL((attn_kernel<BQ, BK, false, G>), grid, block, 0, s, p);
    return hipGetLastError();
}

// Key groups per query block, by the layer's rows and its chunks per head (the most a
// list can hold: the lists' own lengths are on the device). One rule for sparse and dense
// attention, so that a list of every block gives the dense result bit for bit. Measured
// with one against two groups, 128 queries unless 64 is said, us:
//  - Two groups take 64 KB, two workgroups of them fill a CU: up to 512 rows, one round,
//    they halve the time of a row (dense, 16 heads of 1,374 tokens 22 / 19.5; 64: 4 heads
//    of 5,496 90 / 58), but for lists of a few chunks, where the merge costs more.
//  - Up to 3,072 rows, three fillings of the 1,024 places of single groups, they shorten
//    the last round and the rows that keep every block: 8 views 161 / 129 at 90% and
//    294 / 279 at 50% sparsity, 16 views 380 / 313 at 90% and 564 / 548 at 75%; dense 8
//    views 532 / 530, 16 views 1,948 / 1,973. That takes lists long enough: below 64 chunks
//    (64 queries: 32) one group is faster (256 heads of 1,400 tokens, dense 148 / 173; 128
//    heads of 2,000, 50% sparsity 109 / 128).
//  - Above, their shared barriers only cost: 32 views 1,937 / 2,071.
// Four where even two leave most of the chip idle (at most a workgroup per CU) and rows
// can be long enough to pay for the merge: 4 heads of 4 views 69 / 54 / 47 with one / two
// / four.
template <int BQ, int BK>
hipError_t launch_bk(const AttnParams &p, bool sparse, hipStream_t s)
{
    const long long rows = (long long)p.H * p.n_qb;
    const int chunks = p.n_kb * (BK / 64);
    if (rows <= 256 && chunks >= 64) return launch_groups<BQ, BK, 4>(p, sparse, s);
    const int least = rows <= 512 ? 7 : BQ == 128 ? 64 : 32;
    if (rows <= 3072 && chunks >= least) return launch_groups<BQ, BK, 2>(p, sparse, s);
    return launch_groups<BQ, BK, 1>(p, sparse, s);
}

}  // namespace

hipError_t launch_attn(const AttnParams &p, int bq, int bk, bool sparse, hipStream_t s)
{
    if (p.H == 0 || p.n_qb == 0) return hipSuccess;
    if (bq == 128 && bk == 128) return launch_bk<128, 128>(p, sparse, s);
    if (bq == 128 && bk == 64) return launch_bk<128, 64>(p, sparse, s);
    if (bq == 64 && bk == 128) return launch_bk<64, 128>(p, sparse, s);
    return launch_bk<64, 64>(p, sparse, s);
}

}  // namespace ress
