// The segment-proposal network (an addition to the paper's method): 12 -> 64 -> 64 -> 2,
// ReLU hidden layers, sigmoid outputs (alpha_lo, alpha_hi), trained with a pinball loss.
//
// GEMMs run on the matrix cores, fp16 operands and fp32 accumulation: the 16x16x16 shape for
// layer 1 (K = 16, the 12 inputs padded), gfx950's 16x16x32 shape for every K = 64 product
// (operand layouts in amr_mlp.h).
// Parameters are fp32 masters packed as W1 [12][64], b1 [64], W2 [64][64], b2 [64],
// W3 [64][2], b3 [2] (input-major); the fp16 operands are rounded from them.
#include <hip/hip_runtime.h>

#include "amr_mlp.h"

namespace amr {

// Stage the fp16 operand copies of the weights in LDS, in the layouts the MFMA loads want.
__device__ inline void stage_weights(const float *W, MlpLds &s) {
    const float *W1 = W + kOffW1, *W2 = W + kOffW2, *W3 = W + kOffW3;
    for (int i = threadIdx.x; i < 64 * 16; i += blockDim.x) {       // W1T[u][i], i >= 12 zero
        int u = i / 16, k = i % 16;
        s.w1t[i] = (_Float16)(k < kIn ? W1[k * 64 + u] : 0.f);
    }
    for (int i = threadIdx.x; i < 64 * 64; i += blockDim.x) {
        int a = i / 64, b = i % 64;
        s.w2t[i] = (_Float16)W2[b * 64 + a];                          // W2T[v][u] = W2[u][v]
        s.w2[i] = (_Float16)W2[i];                                    // W2[u][v]
    }
    for (int i = threadIdx.x; i < 16 * 64; i += blockDim.x) {       // W3T[j][u], j >= 2 zero
        int j = i / 64, u = i % 64;
        s.w3t[i] = (_Float16)(j < kOut ? W3[u * 2 + j] : 0.f);
    }
    for (int i = threadIdx.x; i < 64; i += blockDim.x) {
        s.b1[i] = W[kOffB1 + i];
        s.b2[i] = W[kOffB2 + i];
    }
    if (threadIdx.x < 2) s.b3[threadIdx.x] = W[kOffB3 + threadIdx.x];
}

__device__ inline float sigmoidf_(float z) { return 1.f / (1.f + __expf(-z)); }

// The training kernels: 512 threads, eight waves, each taking tiles of 32 rows: 65536 rows are 256
// blocks' worth of one tile per wave.  Both kernels are chains (weights, inputs, layers, results), so
// a tile is small and a CU holds eight of them to overlap.
constexpr int kTile = 32;
constexpr int kWaves = 8;
// LDS rows are padded to a multiple of 16 bytes that is not one of 128: the matrix-core operand
// reads take 16 bytes from each of 16 rows, which at 128 bytes all fall into the same banks.
constexpr int kRow = 72;              // rows of 64 units
constexpr int kCol = 40;              // rows of kTile tile rows

struct FwdLds {
    _Float16 w1t[64 * 16];           // [u][i], i >= 12 zero
    _Float16 w2t[64 * kRow];         // [v][u]
    _Float16 w3t[16 * kRow];         // [j][u], j >= 2 zero
    float b1[64], b2[64], b3[4];
    _Float16 x[kWaves][kTile * 16];  // per wave: the tile's inputs, zero padded
    _Float16 h[kWaves][kTile * kRow];  // per wave: layer 1's activations, then layer 2's
};

// Forward.  Its floor is the activations it writes for the backward pass (512 bytes a row, 33.5 MB at
// 65536 rows, 6.5 us at the copy rate); they leave as whole rows, 16 bytes per lane.  The layers
// share one activation buffer per wave: a layer's operand rows are in registers before its
// results overwrite them.  65536 rows: 14 us (four waves a block on 64-row tiles: 22 us).
__global__ __launch_bounds__(64 * kWaves) void mlp_forward_kernel(const float *X, const float *W, float *Y, float *H,
                                                                 int64_t n) {
    __shared__ __attribute__((aligned(16))) FwdLds s;
    const int tid = threadIdx.x;
    {   // every load of the weights in flight before the first is used
        float w1[2], w2[8], w3[2], bias = 0.f;
        #pragma unroll
        for (int i = 0; i < 2; i++) {
            const int e = tid + 512 * i;
            w1[i] = (e >> 6) < kIn ? W[kOffW1 + e] : 0.f;                   // W1[k][u], k >= 12 zero
            w3[i] = (e & 15) < kOut ? W[kOffW3 + (e >> 4) * kOut + (e & 15)] : 0.f;
        }
        #pragma unroll
        for (int i = 0; i < 8; i++) w2[i] = W[kOffW2 + tid + 512 * i];
        if (tid < 64) bias = W[kOffB1 + tid];
        else if (tid < 128) bias = W[kOffB2 + tid - 64];
        else if (tid < 128 + kOut) bias = W[kOffB3 + tid - 128];
        #pragma unroll
        for (int i = 0; i < 2; i++) {
            const int e = tid + 512 * i;
            s.w1t[(e & 63) * 16 + (e >> 6)] = (_Float16)w1[i];
            s.w3t[(e & 15) * kRow + (e >> 4)] = (_Float16)w3[i];
        }
        #pragma unroll
        for (int i = 0; i < 8; i++) {
            const int e = tid + 512 * i;
            s.w2t[(e & 63) * kRow + (e >> 6)] = (_Float16)w2[i];
        }
        if (tid < 64) s.b1[tid] = bias;
        else if (tid < 128) s.b2[tid - 64] = bias;
        else if (tid < 128 + kOut) s.b3[tid - 128] = bias;
    }
    __syncthreads();
    const int wave = tid >> 6, lane = tid & 63;
    const int lr = lane & 15, lq = lane >> 4;
    _Float16 *x = s.x[wave], *h = s.h[wave];
    const bool wide = (reinterpret_cast<uintptr_t>(H) & 15u) == 0;
    const int64_t ntiles = (n + kTile - 1) / kTile;
    for (int64_t t = (int64_t)blockIdx.x * kWaves + wave; t < ntiles; t += (int64_t)gridDim.x * kWaves) {
        const int64_t row0 = t * kTile;
        #pragma unroll
        for (int i = 0; i < kTile * kIn / 64; i++) {     // rows of 12 values, contiguous
            const int e = i * 64 + lane;
            const int64_t g = row0 * kIn + e;
            x[(e / kIn) * 16 + e % kIn] = (_Float16)(g < n * kIn ? X[g] : 0.f);
        }
        if (lane < kTile) *reinterpret_cast<half4 *>(x + lane * 16 + 12) = half4{0, 0, 0, 0};
        __builtin_amdgcn_wave_barrier();
        // activations of one layer to H (part 0: layer 1, 1: layer 2), whole rows
        auto keep = [&](int part) {
            if (!H) return;
            #pragma unroll
            for (int i = 0; i < kTile / 4; i++) {
                const int row = i * 4 + lq;
                const half4 v = *reinterpret_cast<const half4 *>(h + row * kRow + 4 * lr);
                float *out = H + (row0 + row) * 128 + part * 64 + 4 * lr;
                if (row0 + row >= n) continue;
                if (wide) {
                    *reinterpret_cast<float4 *>(out) = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
                } else {
                    #pragma unroll
                    for (int j = 0; j < 4; j++) out[j] = (float)v[j];
                }
            }
        };
        // layer 1: [32 x 16] . [16 x 64]
        #pragma unroll
        for (int rt = 0; rt < kTile / 16; rt++) {
            const half4 a = *reinterpret_cast<const half4 *>(x + (rt * 16 + lr) * 16 + 4 * lq);
            #pragma unroll
            for (int ct = 0; ct < 4; ct++) {
                const half4 b = *reinterpret_cast<const half4 *>(s.w1t + (ct * 16 + lr) * 16 + 4 * lq);
                float4v acc = {0.f, 0.f, 0.f, 0.f};
                acc = mfma_k16(a, b, acc);
                #pragma unroll
                for (int j = 0; j < 4; j++)
                    h[(rt * 16 + 4 * lq + j) * kRow + ct * 16 + lr] = (_Float16)fmaxf(acc[j] + s.b1[ct * 16 + lr], 0.f);
            }
        }
        __builtin_amdgcn_wave_barrier();
        keep(0);
        // layer 2: [32 x 64] . [64 x 64]
        half8 a2[kTile / 16][2];
        #pragma unroll
        for (int rt = 0; rt < kTile / 16; rt++)
            #pragma unroll
            for (int ks = 0; ks < 2; ks++)
                a2[rt][ks] = *reinterpret_cast<const half8 *>(h + (rt * 16 + lr) * kRow + ks * 32 + 8 * lq);
        __builtin_amdgcn_wave_barrier();
        #pragma unroll
        for (int ct = 0; ct < 4; ct++) {
            half8 b[2];
            #pragma unroll
            for (int ks = 0; ks < 2; ks++)
                b[ks] = *reinterpret_cast<const half8 *>(s.w2t + (ct * 16 + lr) * kRow + ks * 32 + 8 * lq);
            #pragma unroll
            for (int rt = 0; rt < kTile / 16; rt++) {
                float4v acc = {0.f, 0.f, 0.f, 0.f};
                acc = mfma_k32(a2[rt][0], b[0], acc);
                acc = mfma_k32(a2[rt][1], b[1], acc);
                #pragma unroll
                for (int j = 0; j < 4; j++)
                    h[(rt * 16 + 4 * lq + j) * kRow + ct * 16 + lr] = (_Float16)fmaxf(acc[j] + s.b2[ct * 16 + lr], 0.f);
            }
        }
        __builtin_amdgcn_wave_barrier();
        keep(1);
        // layer 3: [32 x 64] . [64 x 16] (two valid columns)
        half8 b3[2];
        #pragma unroll
        for (int ks = 0; ks < 2; ks++) b3[ks] = *reinterpret_cast<const half8 *>(s.w3t + lr * kRow + ks * 32 + 8 * lq);
        #pragma unroll
        for (int rt = 0; rt < kTile / 16; rt++) {
            float4v acc = {0.f, 0.f, 0.f, 0.f};
            #pragma unroll
            for (int ks = 0; ks < 2; ks++)
                acc = mfma_k32(*reinterpret_cast<const half8 *>(h + (rt * 16 + lr) * kRow + ks * 32 + 8 * lq), b3[ks], acc);
            #pragma unroll
            for (int j = 0; j < 4; j++) {
                const int64_t g = row0 + rt * 16 + 4 * lq + j;
                if (lr < kOut && g < n) Y[g * 2 + lr] = sigmoidf_(acc[j] + s.b3[lr]);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

constexpr int kSums = 88;            // sums that a lane holds: dW2 64, dW1 16, db2, dW3 2, db3 2, loss, 2 unused

struct BwdTile {                     // per wave
    _Float16 h1t[64 * kCol];         // [u][row]: layer 1's activations
    _Float16 dzt[64 * kCol];         // [v][row]: dZ2, then [u][row]: dZ1
    _Float16 dz2[kTile * kRow];      // [row][v]: dZ2
    float2 dz3[kTile];               // the rows' output derivatives
};
struct BwdLds {
    _Float16 w2[64 * kRow];          // [u][v]
    union {
        BwdTile tile[kWaves];
        float4 sums[kWaves / 2][kSums / 4][64];   // after the last tile: the upper waves' sums, per lane
    };
};

// Backward of the mean pinball loss.  dZ values are kept unscaled (no 1/n) through the fp16
// products and scaled at the end, so they stay in fp16's normal range.
// Of a tile: the rows' output derivatives, one per lane; then, lane = hidden unit, dZ2 of the rows,
// H read as whole rows, all of them in flight together; the products on the matrix cores from
// operands laid out so that each is read as 16 bytes per lane (dZ2 by row and by unit, H1 by unit).
// dW1 and db1 are one product too, on the fp32 matrix instruction, as the inputs are fp32 of any
// magnitude (two fp16 terms in their place held 22 bits between 1/8 and 65504, and none of a value
// below 3e-8); a row of ones gives db1.  A call (mlp_zero and the binding's allocations included, 20 us of
// it at any size) takes 35.2 us at 65536 rows and 132 us at 1048576; with the two fp16 terms 33.7 and
// 166 us on 128 blocks; with serial row loops, operands gathered by halves and sums in LDS by atomics
// 107 and 1323 us.
// Blocks: one fits a CU (130 KB of LDS), a tile takes some 5 us and a block's 5058 atomic sums 0.06, so
// few blocks while a wave has few tiles, every CU when it has many.  65536 rows: 128 blocks 36.4, 160
// 35.2, 192 35.5, 256 39.7 us; 100003: 41.8, 39.4, 41.6, 39.5; 262144: 67.2, 60.5, 57.2, 56.4; 1048576:
// 204, 173, 154, 132.
constexpr int64_t bwd_blocks(int64_t tiles) {
    const int64_t full = (tiles + kWaves - 1) / kWaves;          // a tile per wave
    return std::min<int64_t>(full, full < 1024 ? 160 : 256);
}
// The rows that fill up the last tile: an infinity of some row's in their place, times their zero, would
// count.
__device__ const float kNoRow[128] = {};

__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void mlp_backward_kernel(const float *X, const float *W, const float *H,
                                                                  const float *Y, const float *Tg, int64_t n,
                                                                  float q_lo, float q_hi, float *dW, float *loss) {
    __shared__ __attribute__((aligned(16))) BwdLds s;
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int lr = lane & 15, lq = lane >> 4;
    {
        float w2[8];
        #pragma unroll
        for (int i = 0; i < 8; i++) w2[i] = W[kOffW2 + tid + 512 * i];
        #pragma unroll
        for (int i = 0; i < 8; i++) {
            const int e = tid + 512 * i;
            s.w2[(e >> 6) * kRow + (e & 63)] = (_Float16)w2[i];
        }
    }
    const float w3u0 = W[kOffW3 + lane * 2], w3u1 = W[kOffW3 + lane * 2 + 1];   // lane = hidden unit u
    __syncthreads();
    BwdTile &b = s.tile[wave];
    const int64_t ntiles = (n + kTile - 1) / kTile;
    // per-lane fp32 accumulators: dW2 and dW1 tiles (MFMA D layout) and the VALU parts
    float4v dw2[4][4], dw1[4];
    #pragma unroll
    for (int i = 0; i < 4; i++) {
        dw1[i] = float4v{0.f, 0.f, 0.f, 0.f};
        #pragma unroll
        for (int j = 0; j < 4; j++) dw2[i][j] = float4v{0.f, 0.f, 0.f, 0.f};
    }
    float db2 = 0.f, dw3[2] = {0.f, 0.f}, db3[2] = {0.f, 0.f}, lsum = 0.f;
    for (int64_t t = (int64_t)blockIdx.x * kWaves + wave; t < ntiles; t += (int64_t)gridDim.x * kWaves) {
        const int64_t row0 = t * kTile;
        float h1[kTile], h2[kTile], x[8];
        #pragma unroll
        for (int r = 0; r < kTile; r++) {
            const float *h = row0 + r < n ? H + (row0 + r) * 128 : kNoRow;
            h1[r] = h[lane];
            h2[r] = h[64 + lane];
        }
        // dW1's operand rows: input lr (row 12: ones) of tile rows 8 lq .. 8 lq + 7
        #pragma unroll
        for (int j = 0; j < 8; j++) {
            const int64_t g = row0 + 8 * lq + j;
            x[j] = lr < kIn && g < n ? X[g * kIn + lr] : (lr == kIn ? 1.f : 0.f);
        }
        // lane = row: the output derivatives (zero past the last row, which keeps such a row out of
        // every product below) and the loss
        if (lane < kTile) {
            const int64_t g = row0 + lane;
            float2 d = make_float2(0.f, 0.f);
            if (g < n) {
                const float y0 = Y[g * 2], y1 = Y[g * 2 + 1], tg = Tg[g];
                const float d0 = tg > y0 ? -q_lo : 1.f - q_lo;
                const float d1 = tg > y1 ? -q_hi : 1.f - q_hi;
                const float r0 = tg - y0, r1 = tg - y1;
                lsum += fmaxf(q_lo * r0, (q_lo - 1.f) * r0) + fmaxf(q_hi * r1, (q_hi - 1.f) * r1);
                d = make_float2(d0 * y0 * (1.f - y0), d1 * y1 * (1.f - y1));
            }
            db3[0] += d.x;
            db3[1] += d.y;
            b.dz3[lane] = d;
        }
        __builtin_amdgcn_wave_barrier();
        // lane = hidden unit: dZ2's column for the tile's rows; dW3 and db2 on the VALU
        #pragma unroll
        for (int r8 = 0; r8 < kTile; r8 += 8) {
            half8 hv, dv;
            #pragma unroll
            for (int i = 0; i < 8; i++) {
                const float2 d = b.dz3[r8 + i];
                dw3[0] += h2[r8 + i] * d.x;
                dw3[1] += h2[r8 + i] * d.y;
                const float dz2 = h2[r8 + i] > 0.f ? d.x * w3u0 + d.y * w3u1 : 0.f;
                db2 += dz2;
                hv[i] = (_Float16)h1[r8 + i];
                dv[i] = (_Float16)dz2;
                b.dz2[(r8 + i) * kRow + lane] = dv[i];
            }
            *reinterpret_cast<half8 *>(b.h1t + lane * kCol + r8) = hv;
            *reinterpret_cast<half8 *>(b.dzt + lane * kCol + r8) = dv;
        }
        __builtin_amdgcn_wave_barrier();
        // dW2 += H1^T dZ2: M = unit u, K = row, N = unit v
        {
            half8 a[4];
            #pragma unroll
            for (int mt = 0; mt < 4; mt++) a[mt] = *reinterpret_cast<const half8 *>(b.h1t + (mt * 16 + lr) * kCol + 8 * lq);
            #pragma unroll
            for (int nt = 0; nt < 4; nt++) {
                const half8 d = *reinterpret_cast<const half8 *>(b.dzt + (nt * 16 + lr) * kCol + 8 * lq);
                #pragma unroll
                for (int mt = 0; mt < 4; mt++) dw2[mt][nt] = mfma_k32(a[mt], d, dw2[mt][nt]);
            }
        }
        __builtin_amdgcn_wave_barrier();
        // dH1 = dZ2 W2^T (M = row, K = unit v, N = unit u), then dZ1 = dH1 (H1 > 0), by unit
        half8 a[kTile / 16][2];
        #pragma unroll
        for (int rt = 0; rt < kTile / 16; rt++)
            #pragma unroll
            for (int ks = 0; ks < 2; ks++)
                a[rt][ks] = *reinterpret_cast<const half8 *>(b.dz2 + (rt * 16 + lr) * kRow + ks * 32 + 8 * lq);
        #pragma unroll
        for (int ct = 0; ct < 4; ct++) {
            half8 w[2];
            #pragma unroll
            for (int ks = 0; ks < 2; ks++) w[ks] = *reinterpret_cast<const half8 *>(s.w2 + (ct * 16 + lr) * kRow + ks * 32 + 8 * lq);
            #pragma unroll
            for (int rt = 0; rt < kTile / 16; rt++) {
                float4v acc = {0.f, 0.f, 0.f, 0.f};
                acc = mfma_k32(a[rt][0], w[0], acc);
                acc = mfma_k32(a[rt][1], w[1], acc);
                const int at = (ct * 16 + lr) * kCol + rt * 16 + 4 * lq;
                const half4 hs = *reinterpret_cast<const half4 *>(b.h1t + at);
                half4 d;
                #pragma unroll
                for (int j = 0; j < 4; j++) d[j] = (_Float16)((float)hs[j] > 0.f ? acc[j] : 0.f);
                *reinterpret_cast<half4 *>(b.dzt + at) = d;
            }
        }
        __builtin_amdgcn_wave_barrier();
        // dW1 += X^T dZ1 (M = input, K = row, N = unit u), both operands fp32; of step j's four rows a lane
        // holds 8 lq + j, which is the order that x and dzt are in
        #pragma unroll
        for (int nt = 0; nt < 4; nt++) {
            const half8 d = *reinterpret_cast<const half8 *>(b.dzt + (nt * 16 + lr) * kCol + 8 * lq);
            #pragma unroll
            for (int j = 0; j < 8; j++) dw1[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], (float)d[j], dw1[nt], 0, 0, 0);
        }
        __builtin_amdgcn_wave_barrier();
    }
    for (int o = 32; o > 0; o >>= 1) {
        db3[0] += __shfl_xor(db3[0], o, 64);
        db3[1] += __shfl_xor(db3[1], o, 64);
        lsum += __shfl_xor(lsum, o, 64);
    }
    // the block's sums: the upper half of the waves hands its sums to the lower, three times; then
    // one global atomic per parameter and block (adding to one LDS copy by atomics took 6.6 us per
    // wave)
    float sum[kSums];
    #pragma unroll
    for (int i = 0; i < 4; i++) {
        #pragma unroll
        for (int k = 0; k < 4; k++)
            #pragma unroll
            for (int j = 0; j < 4; j++) sum[16 * i + 4 * k + j] = dw2[i][k][j];
        #pragma unroll
        for (int j = 0; j < 4; j++) sum[64 + 4 * i + j] = dw1[i][j];
    }
    sum[80] = db2;
    sum[81] = dw3[0];
    sum[82] = dw3[1];
    sum[83] = db3[0];
    sum[84] = db3[1];
    sum[85] = lsum;
    sum[86] = sum[87] = 0.f;
    #pragma unroll
    for (int half = kWaves / 2; half >= 1; half /= 2) {
        __syncthreads();
        if (wave >= half && wave < 2 * half) {
            #pragma unroll
            for (int i = 0; i < kSums / 4; i++)
                s.sums[wave - half][i][lane] = make_float4(sum[4 * i], sum[4 * i + 1], sum[4 * i + 2], sum[4 * i + 3]);
        }
        __syncthreads();
        if (wave < half) {
            #pragma unroll
            for (int i = 0; i < kSums / 4; i++) {
                const float4 v = s.sums[wave][i][lane];
                sum[4 * i] += v.x;
                sum[4 * i + 1] += v.y;
                sum[4 * i + 2] += v.z;
                sum[4 * i + 3] += v.w;
            }
        }
    }
    if (wave) return;
    const float inv_n = 1.f / (float)n;
    #pragma unroll
    for (int mt = 0; mt < 4; mt++)
        #pragma unroll
        for (int nt = 0; nt < 4; nt++)
            #pragma unroll
            for (int j = 0; j < 4; j++)
                atomicAdd(&dW[kOffW2 + (mt * 16 + 4 * lq + j) * 64 + nt * 16 + lr], sum[16 * mt + 4 * nt + j] * inv_n);
    #pragma unroll
    for (int nt = 0; nt < 4; nt++)
        #pragma unroll
        for (int j = 0; j < 4; j++) {
            const int k = 4 * lq + j, u = nt * 16 + lr;       // input (12: the bias), unit
            if (k < kIn) atomicAdd(&dW[kOffW1 + k * 64 + u], sum[64 + 4 * nt + j] * inv_n);
            else if (k == kIn) atomicAdd(&dW[kOffB1 + u], sum[64 + 4 * nt + j] * inv_n);
        }
    atomicAdd(&dW[kOffB2 + lane], sum[80] * inv_n);
    atomicAdd(&dW[kOffW3 + lane * 2], sum[81] * inv_n);
    atomicAdd(&dW[kOffW3 + lane * 2 + 1], sum[82] * inv_n);
    if (lane < 3) atomicAdd(lane == 2 ? loss : &dW[kOffB3 + lane], (lane == 0 ? sum[83] : (lane == 1 ? sum[84] : sum[85])) * inv_n);
}

__global__ void mlp_zero(float *dW, float *loss) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kParams) dW[i] = 0.f;
    if (i == kParams) *loss = 0.f;
}

__global__ void mlp_adam_kernel(float *W, const float *dW, float *M, float *V, int n, float lr, float b1, float b2,
                                float eps, float c1, float c2) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float g = dW[i];
    float m = b1 * M[i] + (1.f - b1) * g;
    float v = b2 * V[i] + (1.f - b2) * g * g;
    M[i] = m;
    V[i] = v;
    W[i] -= lr * (m / c1) / (sqrtf(v / c2) + eps);
}

// Packed inference layout: the LDS image of MlpLds (fp16 operand copies + fp32 biases).
__global__ void mlp_pack_kernel(const float *W, MlpLds *out) {
    __shared__ MlpLds s;
    stage_weights(W, s);
    __syncthreads();
    const uint32_t *src = reinterpret_cast<const uint32_t *>(&s);
    uint32_t *dst = reinterpret_cast<uint32_t *>(out);
    for (int i = threadIdx.x; i < (int)(sizeof(MlpLds) / 4); i += blockDim.x) dst[i] = src[i];
}

}  // namespace amr

using namespace amr;

extern "C" {

int32_t amr_mlp_param_count(void) { return kParams; }
int64_t amr_mlp_packed_bytes(void) { return (int64_t)sizeof(MlpLds); }

int amr_mlp_forward(const float *X, const float *W, float *Y, float *H, int64_t n, void *stream) {
    if (!X || !W || !Y || n <= 0) { set_error("amr_mlp_forward: null argument or n <= 0"); return AMR_EINVAL; }
    const int64_t tiles = (n + kTile - 1) / kTile;
    const int grid = (int)std::min<int64_t>((tiles + kWaves - 1) / kWaves, 2048);
    hipLaunchKernelGGL(mlp_forward_kernel, dim3(grid), dim3(64 * kWaves), 0, (hipStream_t)stream, X, W, Y, H, n);
    return check_hip_mlp(hipGetLastError(), "mlp_forward launch");
}

int amr_mlp_backward(const float *X, const float *W, const float *H, const float *Y, const float *T, int64_t n,
                     float q_lo, float q_hi, float *dW, float *loss, void *stream) {
    if (!X || !W || !H || !Y || !T || !dW || !loss || n <= 0) {
        set_error("amr_mlp_backward: null argument or n <= 0");
        return AMR_EINVAL;
    }
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(mlp_zero, dim3((kParams + 256) / 256), dim3(256), 0, s, dW, loss);
    const int64_t tiles = (n + kTile - 1) / kTile;
    const int grid = (int)bwd_blocks(tiles);
    hipLaunchKernelGGL(mlp_backward_kernel, dim3(grid), dim3(64 * kWaves), 0, s, X, W, H, Y, T, n, q_lo, q_hi, dW, loss);
    return check_hip_mlp(hipGetLastError(), "mlp_backward launch");
}

int amr_mlp_adam_step(float *W, const float *dW, float *M, float *V, int32_t t, float lr, float beta1, float beta2,
                      float eps, void *stream) {
    if (!W || !dW || !M || !V || t < 1) { set_error("amr_mlp_adam_step: null argument or t < 1"); return AMR_EINVAL; }
    float c1 = 1.f - powf(beta1, (float)t), c2 = 1.f - powf(beta2, (float)t);
    hipLaunchKernelGGL(mlp_adam_kernel, dim3((kParams + 255) / 256), dim3(256), 0, (hipStream_t)stream, W, dW, M, V,
                       kParams, lr, beta1, beta2, eps, c1, c2);
    return check_hip_mlp(hipGetLastError(), "mlp_adam launch");
}

int amr_mlp_pack(const float *W, void *d_out, void *stream) {
    if (!W || !d_out) { set_error("amr_mlp_pack: null argument"); return AMR_EINVAL; }
    if (reinterpret_cast<uintptr_t>(d_out) & 15u) { set_error("amr_mlp_pack: d_out must be 16-byte aligned"); return AMR_EINVAL; }
    hipLaunchKernelGGL(mlp_pack_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, W, (MlpLds *)d_out);
    return check_hip_mlp(hipGetLastError(), "mlp_pack launch");
}

}  // extern "C"
