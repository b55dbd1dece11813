// The change that masking makes in what attention writes into the residual
// stream, per query block (the reference measurement of Sec. 3, "Testing the
// Probability Assumption"): out[h][i] = sum over the block's tokens t of
// x_t^T M_h x_t = ||W_O^h x_t||^2, with x_t = a_t - b_t the difference of two
// float32 attention outputs of the same queries.
//
// One workgroup of 4 waves per (head, query block); wave w takes the block's
// 16-token tiles w, w + 4. A tile is a float64 matrix product on the matrix cores
// (16x16x4 steps), U^T = M X^T, with everything a lane needs already in its
// registers:
//  - lane l holds channels 16 u + 4 g + e (u, e = 0..3, g = l / 16) of token l % 16
//    as 16 float64 values (the difference of two float32 values is exact): four
//    16-byte loads per input, each covering 64 contiguous bytes of 16 tokens. They
//    are the B operands of the steps (u, e) as they lie;
//  - row r of the product's 16-row block nt stands for channel 16 nt + 4 (r % 4) +
//    r / 4, so result register v of lane l (row 4 v + g) is channel 16 nt + 4 g + v,
//    the x value the lane holds as (u = nt, e = v): x . (M x) needs no exchange;
//  - the quadratic form folds M's off-diagonal 16 x 16 blocks (nt, u) and (u, nt)
//    into one (M + M^T, exact or once rounded in float64), so 10 of the 16 blocks
//    are multiplied. Their A operands, 40 float64 values a lane, are read once per
//    wave and stay in registers.
// Roofline: 0.90 GFLOP of float64 matrix steps (40 a tile) and 90 MB (two float32 inputs)
// at 16 heads x 10,992 tokens, 11.5 and 18 us at 78.6 TFLOP/s and 5.1 TB/s. Measured there:
// 28 us (one lane per channel with M and x read from LDS for every token: 145 us).
#include "ress_internal.h"

namespace ress {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

__device__ __forceinline__ double wave_sum(double x)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

__global__ void __launch_bounds__(kThreads, 2) drift_sq_kernel(const DriftSqParams p)
{
    __shared__ double part[kWaves];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = blockIdx.x / p.n_qb, i = blockIdx.x % p.n_qb;
    const int t0 = i * p.bq, t1 = min(t0 + p.bq, p.N);
    const int g = lane >> 4, col = lane & 15;
    const float *Mh = p.gram + (size_t)h * kD * kD;

    // The two inputs' 16 channels of this lane's token (rows past the block repeat its
    // last row and are left out of the sum).
    auto load = [&](int t, float4 (&xa)[4], float4 (&xb)[4]) __attribute__((always_inline)) {
        const size_t off = ((size_t)h * p.N + min(t + col, t1 - 1)) * kD + 4 * g;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            xa[u] = *reinterpret_cast<const float4 *>(p.a + off + 16 * u);
            xb[u] = *reinterpret_cast<const float4 *>(p.b + off + 16 * u);
        }
    };
    float4 xa[4], xb[4];
    int t = t0 + 16 * wave;
    if (t < t1) load(t, xa, xb);

    double m[4][4][4];  // A operand of block (nt, u >= nt), step e
    if (t < t1) {
        const int chan = 4 * (col & 3) + (col >> 2);  // channel of row `col` within its block
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int u = nt; u < 4; ++u) {
                const int row = 16 * nt + chan, c0 = 16 * u + 4 * g;
                const float4 v = *reinterpret_cast<const float4 *>(Mh + row * kD + c0);
                const float w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    m[nt][u][e] = u == nt ? (double)w[e] : (double)w[e] + (double)Mh[(c0 + e) * kD + row];
            }
    }

    double acc = 0.0;
    for (; t < t1; t += 16 * kWaves) {
        double x[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x[u][0] = (double)xa[u].x - (double)xb[u].x;
            x[u][1] = (double)xa[u].y - (double)xb[u].y;
            x[u][2] = (double)xa[u].z - (double)xb[u].z;
            x[u][3] = (double)xa[u].w - (double)xb[u].w;
        }
        const bool in = t + col < t1;
        if (t + 16 * kWaves < t1) load(t + 16 * kWaves, xa, xb);
        v4d c[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) c[nt] = v4d{0.0, 0.0, 0.0, 0.0};
        // Independent chains of the four row blocks side by side.
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int nt = 0; nt <= u; ++nt)
                    c[nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(m[nt][u][e], x[u][e], c[nt], 0, 0, 0);
        // (A zero x would not do for the rows past the block: M need not be finite.)
        double with = acc;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) with = fma(x[nt][v], c[nt][v], with);
        acc = in ? with : acc;
    }
    acc = wave_sum(acc);
    if (lane == 0) part[wave] = acc;
    __syncthreads();
    if (tid == 0) {
        double s = 0.0;
        for (int w = 0; w < kWaves; ++w) s += part[w];
        p.out[(size_t)h * p.n_qb + i] = s;
    }
}

}  // namespace

hipError_t launch_drift_sq(const DriftSqParams &p, hipStream_t s)
{
    const long long blocks = (long long)p.H * p.n_qb;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(drift_sq_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

}  // namespace ress
