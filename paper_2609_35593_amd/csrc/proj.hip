// The two steps on either side of the path, as bf16 MFMA GEMMs with fused
// epilogues (token-major activations, nn.Linear-style [out][in] weights):
//  - QKV projection, [Q K V] = X W_qkv^T, written head-major [H][N][64], with the
//    block mean pooling of Sec. 3 step (1) taken from the bf16-rounded outputs in
//    the epilogue (plus c_j = Vbar_j^T M_h Vbar_j for Eq. 9), so the selection never reads
//    Q, K, V again;
//  - output projection and residual add, R' = R + concat_h(O_h) W_O^T, reading
//    the head-major attention output directly (the k-slice of one 64-wide k-tile
//    is one head), into a bf16 or a float32 residual stream.
//
// Tiling: 256 x 256 output tile per workgroup, k-tiles of 64, 8 waves, each wave
// a 64 x 128 sub-tile of 2 x 4 v_mfma_f32_32x32x16_bf16 accumulators (lane l
// holds output column l%32 of each 32 x 32 block, 16 of its rows); half tiles of 128
// rows (32 x 128 per wave) finish a layer whose full tiles would leave the last round
// of workgroups nearly empty (tile_rows). A and B k-tiles (256 rows x 128 bytes each)
// move global -> LDS with global_load_lds in two slots; rows keep their 16-byte chunks
// XOR-swizzled per row, applied by choosing each lane's source chunk. Rows of A past
// the last token repeat the last token and are excluded from every output.
//
// What bounds it. A tile's 16 k-tiles (H = 16) take 22-25 us and its epilogue used to
// take 9 (QKV) to 16 us (residual, one dependent load after another): one workgroup
// fits a CU, so nothing hides it. Residual pieces are now loaded a phase ahead, and
// stores go out in batches of eight. Measured (us, before -> now, back to back): QKV
// projection 98 -> 87 at 8 views, 170 -> 156 at 16, 316 -> 290 at 32 (277 GFLOP, 950
// TFLOP/s; with the caches flushed before each call 348 -> 315, between other kernels and
// with cold operands, as bench.py times it, 370 -> 339); output projection, bf16 stream
// 117 -> 104 at 32 views, 69 -> 56 at 16, 32 -> 18 at 2. (Two workgroups of 128 x 256
// tiles per CU, each hiding the other's epilogue, reached 169 and 125 us at 16 and 32
// views: they fetch 1.5 times the operand bytes past L2, which the k-loop then waits for.)
#include "ress_internal.h"

namespace ress {
namespace {

typedef __bf16 bf16x8 __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef float f32x16 __attribute__((__vector_size__(16 * sizeof(float))));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kThreads = 512;
constexpr int BM = 256, BN = 256;   // output tile
constexpr int kTileBytes = 256 * 128;  // one operand k-tile: 256 rows x 64 bf16
constexpr int kStageRow = BN * 2 + 16;  // bf16 staging row of the output tile (padded)
constexpr int kOperandBytes = 2 * 2 * kTileBytes;                        // two slots of A and B
constexpr int kEpilogue0 = BM * kStageRow + 2 * 4 * BN * (int)sizeof(double);  // tile + sums + means
constexpr int kEpilogue1 = 2 * 64 * (BN + 4) * (int)sizeof(float);      // two quarters of a float32 tile
constexpr int kSmem = kEpilogue0 > kOperandBytes ? (kEpilogue0 > kEpilogue1 ? kEpilogue0 : kEpilogue1)
                                                 : (kOperandBytes > kEpilogue1 ? kOperandBytes : kEpilogue1);
static_assert(kSmem <= 160 * 1024, "LDS per workgroup");

__device__ __forceinline__ int swz(int row) { return (((row >> 1) & 1) << 2) | ((row >> 2) & 3); }
__device__ __forceinline__ void wait_vm_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)

__device__ __forceinline__ float bf16_round(float x) { return (float)(__bf16)x; }
__device__ __forceinline__ unsigned int bf16_bits(float x)
{
    return (unsigned int)__builtin_bit_cast(unsigned short, (__bf16)x);
}

// A thread's 16-byte pieces of the residual in one 64-row epilogue phase.
template <int MODE>
struct Residual {
    static constexpr int kPer = MODE == 2 ? 4 : 8;                  // elements per piece
    static constexpr int kPieces = 64 * (BN / kPer) / kThreads;     // per thread
    uint4 r[kPieces];

    __device__ __forceinline__ static int row(int u, int tid) { return (u * kThreads + tid) / (BN / kPer); }
    __device__ __forceinline__ static int col(int tid) { return tid % (BN / kPer) * kPer; }
    __device__ __forceinline__ void load(const ProjParams &p, int m0, int n0, int ph, int tid)
    {
        const char *base = MODE == 2 ? reinterpret_cast<const char *>(p.resid_in_f32)
                                     : reinterpret_cast<const char *>(p.resid_in);
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {  // rows past the last token repeat it and are not stored
            const int t = min(m0 + 64 * ph + row(u, tid), p.T - 1);
            r[u] = *reinterpret_cast<const uint4 *>(base + ((size_t)t * 64 * p.H + n0 + col(tid)) * (16 / kPer));
        }
    }
    __device__ __forceinline__ void store(const ProjParams &p, int m0, int n0, int ph, int tid, const float *stage,
                                          int sr) const
    {
        char *base = MODE == 2 ? reinterpret_cast<char *>(p.resid_out_f32) : reinterpret_cast<char *>(p.resid_out);
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
            const int t = m0 + 64 * ph + row(u, tid);
            const float *st = stage + row(u, tid) * sr + col(tid);
            const unsigned int w[4] = {r[u].x, r[u].y, r[u].z, r[u].w};
            unsigned int o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (MODE == 2) {  // one float32 addition per element
                    o[e] = __float_as_uint(__uint_as_float(w[e]) + st[e]);
                } else {  // added in float32, rounded to bf16 once
                    const float lo = __uint_as_float(w[e] << 16) + st[2 * e];
                    const float hi = __uint_as_float(w[e] & 0xffff0000u) + st[2 * e + 1];
                    o[e] = bf16_bits(lo) | (bf16_bits(hi) << 16);
                }
            }
            if (t < p.T)
                *reinterpret_cast<uint4 *>(base + ((size_t)t * 64 * p.H + n0 + col(tid)) * (16 / kPer)) =
                    make_uint4(o[0], o[1], o[2], o[3]);
        }
    }
};

// 0: QKV projection + pooling, 1: output projection + bf16 residual, 2: output
// projection + float32 residual.
// MI: 32-row blocks per wave; the tile has 128 MI rows (256, or 128 for the half tiles
// that finish a layer), at row m0 and output column n0.
template <int MODE, int MI>
__device__ __forceinline__ void proj_tile(const ProjParams &p, unsigned char *smem, int m0, int n0)
{
    using Resid = Residual<MODE>;
    constexpr int TM = 128 * MI;
    auto slot_ptr = [&](int slot, int b_operand) __attribute__((always_inline)) {
        return smem + (2 * slot + b_operand) * kTileBytes;
    };
    const int T = p.T, dm = 64 * p.H, KT = p.H;              // k-tiles of 64: one head each
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 3, wn = wave >> 2;  // rows 32 MI wm, columns 128 wn of the tile
    const int hh = lane >> 5, ql = lane & 31;

    // DMA: each thread moves 2 MI chunks of A and 4 of B per k-tile; instruction u of
    // wave w fills rows 8 (8u + w) .. +7 (lane / 8), physical chunk lane & 7.
    int arow[4], brow[4];
    unsigned int chunk_off[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int r = (u * 8 + wave) * 8 + (lane >> 3);
        arow[u] = min(m0 + r, T - 1);
        brow[u] = n0 + r;
        chunk_off[u] = (unsigned int)(((lane & 7) ^ swz(r)) << 4);
    }
    auto dma = [&](int kt, int slot) __attribute__((always_inline)) {
        unsigned char *a_dst = slot_ptr(slot, 0), *b_dst = slot_ptr(slot, 1);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint16_t *asrc = MODE == 0 ? p.a + (size_t)arow[u] * dm + kt * 64
                                             : p.a + ((size_t)kt * T + arow[u]) * 64;
            const uint16_t *bsrc = p.w + (size_t)brow[u] * dm + kt * 64;
            if (u < 2 * MI)
                __builtin_amdgcn_global_load_lds((const void *)((const unsigned char *)asrc + chunk_off[u]),
                                                 (lds_void *)(a_dst + (u * 8 + wave) * 1024), 16, 0, 0);
            __builtin_amdgcn_global_load_lds((const void *)((const unsigned char *)bsrc + chunk_off[u]),
                                             (lds_void *)(b_dst + (u * 8 + wave) * 1024), 16, 0, 0);
        }
    };
    // Operand read offsets: row, logical chunk 2 kk + hh.
    int aoff[MI][4], boff[4][4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            const int r = 32 * MI * wm + 32 * mi + ql;
            aoff[mi][kk] = r * 128 + (((2 * kk + hh) ^ swz(r)) << 4);
        }
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) {
            const int r = 128 * wn + 32 * ni + ql;
            boff[ni][kk] = r * 128 + (((2 * kk + hh) ^ swz(r)) << 4);
        }
    }

    f32x16 acc[MI][4];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;

    // Operand fragments are read one k-step (16) ahead into two register sets, so
    // the LDS latency of step kk+1 hides behind the 8 MFMAs of step kk; the first
    // step of the next k-tile is read right after the barrier, beside the MFMAs of
    // the last step of this one.
    bf16x8 fa[2][MI], fb[2][4];
    auto read_frags = [&](int slot, int kk, int buf) __attribute__((always_inline)) {
        const unsigned char *A = slot_ptr(slot, 0), *B = slot_ptr(slot, 1);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) fa[buf][mi] = *reinterpret_cast<const bf16x8 *>(A + aoff[mi][kk]);
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) fb[buf][ni] = *reinterpret_cast<const bf16x8 *>(B + boff[ni][kk]);
    };
    auto mfmas = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < 4; ++ni)
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[buf][mi], fb[buf][ni], acc[mi][ni], 0, 0, 0);
    };

    // One k-step: the LDS reads of the next step's fragments go between the first
    // MFMAs (left alone, the compiler puts each step's reads after the previous step's
    // MFMAs and waits for them before its own).
    auto step_schedule = [&]() __attribute__((always_inline)) {
        if (MI == 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // five reads, four MFMAs
#pragma unroll
        for (int u = 0; u < 4 * MI; ++u) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
            if (u < 4 + MI) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one LDS read
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // k-steps 0..2 of the k-tile in `slot`.
    auto steps = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 3; ++kk) {
            read_frags(slot, kk + 1, (kk + 1) & 1);
            mfmas(kk & 1);
            step_schedule();
        }
    };

    dma(0, 0);
    wait_vm_all();
    __syncthreads();
    read_frags(0, 0, 0);
    for (int kt = 0; kt + 1 < KT; ++kt) {
        const int slot = kt & 1;
        dma(kt + 1, slot ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        steps(slot);
        wait_vm_all();    // k-tile kt + 1 has landed (this wave's part) ...
        __syncthreads();  // ... every wave's, and slot kt & 1 is no longer read
        __builtin_amdgcn_sched_barrier(0);
        read_frags(slot ^ 1, 0, 0);
        mfmas(1);  // step 3 of this k-tile
        step_schedule();
    }
    // The residual pieces that the first epilogue phase needs are on their way during
    // the last k-tile.
    Resid resid;
    if constexpr (MODE != 0) resid.load(p, m0, n0, 0, tid);
    __builtin_amdgcn_sched_barrier(0);
    steps((KT - 1) & 1);
    mfmas(1);
    __syncthreads();  // the operand slots are free for the epilogue

    // Accumulator element (mi, ni, v) of this lane: tile row and column.
    auto row_of = [&](int mi, int v) __attribute__((always_inline)) {
        return 32 * MI * wm + 32 * mi + (v >> 2) * 8 + hh * 4 + (v & 3);
    };
    auto col_of = [&](int ni) __attribute__((always_inline)) { return 128 * wn + 32 * ni + ql; };

    if constexpr (MODE == 0) {
        // Round to the bf16 outputs; everything below uses the rounded values.
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < 4; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mi][ni][v] = bf16_round(acc[mi][ni][v]);

        // Pooling: column sums over this wave's 32 MI rows (valid tokens only), in
        // float64 (exact for bf16 values of moderate span).
        double csum[4];
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) {
            double s = 0.0;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    s += (m0 + row_of(mi, v) < T) ? (double)acc[mi][ni][v] : 0.0;
            csum[ni] = s + __shfl_xor(s, 32);
        }
        // Output tile as bf16, staged row-major in LDS (the operand slots are free).
        unsigned char *stage = smem;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < 4; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    *reinterpret_cast<unsigned short *>(stage + row_of(mi, v) * kStageRow + col_of(ni) * 2) =
                        (unsigned short)bf16_bits(acc[mi][ni][v]);
        // Per-wave column sums next to it: psum[wm][column].
        double *psum = reinterpret_cast<double *>(stage + BM * kStageRow);
        if (hh == 0) {
#pragma unroll
            for (int ni = 0; ni < 4; ++ni) psum[wm * BN + col_of(ni)] = csum[ni];
        }
        __syncthreads();

        // Head-major bf16 stores: 16 bytes (8 channels of one token) per thread and step.
        const int which = n0 / dm;  // 0: Q, 1: K, 2: V (a tile never straddles two)
        uint16_t *dst = which == 0 ? p.q : which == 1 ? p.k : p.v;
        {
            const int c8 = (tid & 31) * 8, f = n0 - which * dm + c8, h = f >> 6, d = f & 63;
            uint16_t *col = dst + (size_t)h * T * 64 + d;
            constexpr int RS = kThreads / 32;  // rows per step
#pragma unroll 8
            for (int r = tid >> 5; r < TM; r += RS) {
                const uint4 x = *reinterpret_cast<const uint4 *>(stage + r * kStageRow + c8 * 2);
                if (m0 + r < T) *reinterpret_cast<uint4 *>(col + (size_t)(m0 + r) * 64) = x;
            }
        }

        // Block means: a block of b rows is b / (32 MI) wave row groups.
        const int b = which == 0 ? p.bq : p.bk;
        const int groups = b / (32 * MI);
        double *vmean = psum + 4 * BN;  // Vbar of each (block, column) of the tile, for U
        for (int e = tid; e < (TM / b) * BN; e += kThreads) {
            const int blk = e / BN, c = e % BN;
            const int t0 = m0 + blk * b;
            if (t0 >= T) continue;
            double s = 0.0;
            for (int g = 0; g < groups; ++g) s += psum[(blk * groups + g) * BN + c];
            const double mean = s / (double)min(b, T - t0);
            const int blk_g = t0 / b;
            const int f = n0 - which * dm + c, h = f >> 6, d = f & 63;
            if (which == 0) {
                p.pooled.qbar[((size_t)h * p.n_qb + blk_g) * 64 + d] = mean;
            } else if (which == 1) {
                p.pooled.kbar[((size_t)h * p.n_kb + blk_g) * 64 + d] = mean;
            } else {
                p.pooled.vbar[((size_t)h * p.n_kb + blk_g) * 64 + d] = mean;
                vmean[blk * BN + c] = mean;
            }
        }
        if (which == 2) {
            // c_j = Vbar_j . (M_h Vbar_j): one wave per (block, head) of the tile, lane <->
            // channel, in the same order as the pooling pass of the selection.
            __syncthreads();
            const int nblk = TM / b, pairs = nblk * (BN / 64);
            for (int pr = wave; pr < pairs; pr += kThreads / 64) {
                const int blk = pr / (BN / 64), hl = pr % (BN / 64);
                const int t0 = m0 + blk * b;
                if (t0 >= T) continue;
                const int h = (n0 - 2 * dm) / 64 + hl;
                const float *Mrow = p.gram + ((size_t)h * 64 + lane) * 64;
                const double *vb = vmean + blk * BN + hl * 64;
                double u = 0.0;
#pragma unroll 8
                for (int c = 0; c < 64; ++c) u = fma((double)Mrow[c], vb[c], u);
                double cj = u * vb[lane];
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) cj += __shfl_xor(cj, o);
                if (lane == 0) p.pooled.cT[(size_t)h * p.n_kb + t0 / b] = cj;
            }
        }
    } else {
        // R' = R + acc (bf16 stream: rounded once), in 2 MI phases of 64 rows: the waves
        // that hold the rows stage them as float32, then all threads combine them with R in
        // 16-byte pieces. A phase's pieces of R are loaded while the phase before is at
        // work (a thread reads and writes the same elements, so R' may be R); the two
        // halves of the staging area take turns.
        constexpr int SR = BN + 4;  // padded float row
#pragma unroll
        for (int ph = 0; ph < 2 * MI; ++ph) {
            float *stage = reinterpret_cast<float *>(smem) + (ph & 1) * 64 * SR;
            if (wm * MI / 2 == ph) {
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < 4; ++ni)
#pragma unroll
                        for (int v = 0; v < 16; ++v)
                            stage[(row_of(mi, v) - 64 * ph) * SR + col_of(ni)] = acc[mi][ni][v];
            }
            __syncthreads();
            const Resid cur = resid;
            if (ph < 2 * MI - 1) resid.load(p, m0, n0, ph + 1, tid);
            cur.store(p, m0, n0, ph, tid, stage, SR);
        }
    }
}

template <int MODE>
__global__ void __launch_bounds__(kThreads, 1) proj_kernel(const ProjParams p)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kSmem];  // operand slots, then epilogue staging
    // Each XCD runs its range of the full tiles, then its range of the half tiles. Tile
    // order within a range: groups of 8 M tiles, N-major inside a group, so the ~32
    // tiles an XCD runs at once share 8 A and ~4 B k-slices in its L2 (measured: 4-6%
    // faster than sweeping all N tiles of one M tile at a time).
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    constexpr int GM = 8;
    auto place = [&](int item, int m_tiles, int &mt, int &nt) {
        const int grp = item / (GM * p.n_tiles), rem = item % (GM * p.n_tiles);
        const int gmc = min(GM, m_tiles - grp * GM);  // M tiles in this group (fewer in the last)
        mt = grp * GM + rem % gmc;
        nt = rem / gmc;
    };
    int mt, nt;
    if (local < p.full_per_xcd) {
        const int item = xcd * p.full_per_xcd + local;
        if (item >= p.m_full * p.n_tiles) return;
        place(item, p.m_full, mt, nt);
        proj_tile<MODE, 2>(p, smem, mt * BM, nt * BN);
    } else {
        const int item = xcd * p.half_per_xcd + local - p.full_per_xcd;
        if (item >= p.m_half * p.n_tiles) return;
        place(item, p.m_half, mt, nt);
        proj_tile<MODE, 1>(p, smem, p.m_full * BM + mt * (BM / 2), nt * BN);
    }
}

}  // namespace

// Full tiles of 256 rows, or as many as fill whole rounds of the chip's 256 compute
// units (one workgroup each) and half tiles for the rows that are left, where that is
// the shorter list: a half tile takes about 0.6 of a full one (19 against 31 us in the
// QKV projection), so a last round with few tiles is better run as halves.
static void tile_rows(ProjParams &p)
{
    constexpr long long kCUs = 256;
    const long long m = (p.T + BM - 1) / BM, n = p.n_tiles;
    const long long whole = m * n / kCUs;  // whole rounds of full tiles
    const long long mf = whole * kCUs / n, mh = (p.T - mf * BM + BM / 2 - 1) / (BM / 2);
    const long long free_slots = whole * kCUs - mf * n;
    const long long rounds_full = (m * n + kCUs - 1) / kCUs;
    const long long rounds_half = max(0ll, mh * n - free_slots + kCUs - 1) / kCUs;
    if (10 * whole + 6 * rounds_half < 10 * rounds_full) {
        p.m_full = (int)mf;
        p.m_half = (int)mh;
    } else {
        p.m_full = (int)m;
        p.m_half = 0;
    }
    p.full_per_xcd = (int)((p.m_full * n + 7) / 8);
    p.half_per_xcd = (int)((p.m_half * n + 7) / 8);
}

hipError_t launch_proj(const ProjParams &p, hipStream_t s)
{
    if (p.T == 0 || p.n_tiles == 0) return hipSuccess;
    ProjParams q = p;
    tile_rows(q);
    const dim3 grid((unsigned)(8 * (q.full_per_xcd + q.half_per_xcd))), block(kThreads);
    if (p.mode == 0)
        hipLaunchKernelGGL(proj_kernel<0>, grid, block, 0, s, q);
    else if (p.mode == 1)
        hipLaunchKernelGGL(proj_kernel<1>, grid, block, 0, s, q);
    else
        hipLaunchKernelGGL(proj_kernel<2>, grid, block, 0, s, q);
    return hipGetLastError();
}

}  // namespace ress
