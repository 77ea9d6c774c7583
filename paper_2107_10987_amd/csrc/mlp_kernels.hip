// Learned reconstruction on gfx950: a 34-64-64-26 tanh-GELU network on
// normalised 3x3x3 neighbourhoods, bfloat16 operands and FP32 accumulation on
// MFMA (training: v_mfma_f32_16x16x16_bf16; inference:
// v_mfma_f32_16x16x32_bf16), with every value that reaches the FP64 scheme
// checked in FP64 (neighbour bounds, per-line PPM monotonicity, positivity).
//
// Parameter vector (float32 masters, 8090 values): W1[64][34], b1[64],
// W2[64][64], b2[64], W3[26][64], b3[26].  The MFMA copies are bfloat16,
// zero-padded to W1p[64][64] and W3p[32][64].
//
// MFMA operand layout of the 16x16x16 bf16 instruction (lane l, q = l / 16):
//   A[m][k]: lane holds m = l % 16, k = 4q .. 4q+3
//   B[k][n]: lane holds n = l % 16, k = 4q .. 4q+3
//   D[m][n]: lane holds n = l % 16, m = 4q .. 4q+3

#include "hydro_common.h"
#include "mlp_common.h"

#include <math.h>

using namespace hydro;
using namespace hydro::mlp;

namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Forward and training kernels: four waves hold 16 rows, wave c the columns
// 16 c .. 16 c + 15 of every layer.  LDS staging of the bf16 rows of 64, padded
// to a 68-element (136 B) stride: rows written by columns then fall in
// different banks, and the 8-byte MFMA operand loads stay aligned.
constexpr int LDA = 68;
constexpr int STAGE_ELEMS = 16 * LDA;   // bf16 elements of 16 rows

__device__ __forceinline__ v4f mfma(v4s a, v4s b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// binary32 -> bfloat16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ uint16_t bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_float(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

constexpr float GELU_C = 0.7978845608028654f;
constexpr float GELU_A = 0.044715f;

__device__ __forceinline__ float gelu_tanh(float z) { return tanhf(GELU_C * (z + GELU_A * z * z * z)); }
__device__ __forceinline__ float gelu(float z, float t) { return 0.5f * z * (1.0f + t); }
__device__ __forceinline__ float gelu_grad(float z, float t) {
    return 0.5f * (1.0f + t) + 0.5f * z * (1.0f - t * t) * GELU_C * (1.0f + 3.0f * GELU_A * z * z);
}

// Four values of D-layout rows 4q .. 4q + 3 as bfloat16: rows of one column,
// which is also how an MFMA operand holds them when the rows are contracted.
__device__ __forceinline__ v4s pack4(const float v[4]) {
    v4s r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = (short)bf16_bits(v[i]);
    return r;
}

// A wave's operands of one layer's weights W bf16 [..][64], columns 16 c ..,
// k below 16 KB.
template <int KB>
__device__ __forceinline__ void weights(const uint16_t *W, int c, int lane, v4s b[KB]) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) b[kb] = *(const v4s *)(W + (16 * c + (lane & 15)) * 64 + 16 * kb + 4 * (lane >> 4));
}

// Z[r][n] = sum_k A[r][k] W[n][k] for 16 rows and the wave's 16 columns, A in
// LDS (bf16, row stride LDA).  D layout: z holds rows 4q + i, column l % 16.
template <int KB>
__device__ __forceinline__ v4f layer(const uint16_t *A, const v4s b[KB], int lane) {
    v4f z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
        z = mfma(*(const v4s *)(A + (lane & 15) * LDA + 16 * kb + 4 * (lane >> 4)), b[kb], z);
    return z;
}

// The wave's columns 16 c .. of the rows into the staging buffer.
__device__ __forceinline__ void stage_col(uint16_t *S, int c, int lane, v4s v) {
    const int r = lane & 15, q = lane >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) S[(4 * q + i) * LDA + 16 * c + r] = (uint16_t)v[i];
}

// The forward pass's weights and biases of a wave's columns: loaded before the
// first layer, so a call waits for them once.
struct Net {
    v4s w1[3], w2[4], w3[4];
    float b1, b2, b3;
    __device__ __forceinline__ Net(const MlpTrain &t, int c, int lane) {
        const int n = 16 * c + (lane & 15);
        weights<3>(t.wb + WB_W1, c, lane, w1);
        weights<4>(t.wb + WB_W2, c, lane, w2);
        if (c < 2) weights<4>(t.wb + WB_W3, c, lane, w3);
        b1 = t.par[P_B1 + n];
        b2 = t.par[P_B2 + n];
        b3 = n < OUT ? t.par[P_B3 + n] : 0.f;
    }
};

// Forward pass of the 16 rows row0 .. of X [B][34] (float32; rows past nrows
// are zero): z and tanh of the two hidden layers, their bf16 activations, and
// in the waves of columns 0 .. 31 the output layer in y (bias added).  S0 and
// S1 are the rows' staging buffers; a barrier before each layer.  xcol: where
// the inputs' columns go as operands of the rows' contraction, or null.
struct Forward {
    v4f z1, z2, y;
    float t1[4], t2[4];
    v4s a1, a2;
};
__device__ __forceinline__ void activate(v4f &z, float b, float t[4], v4s &a, uint16_t *S, int c, int lane) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        z[i] += b;
        t[i] = gelu_tanh(z[i]);
        v[i] = gelu(z[i], t[i]);
    }
    a = pack4(v);
    stage_col(S, c, lane, a);
}
__device__ __forceinline__ void forward16(const float *X, int row0, int nrows, const Net &net, uint16_t *S0,
                                          uint16_t *S1, int c, int lane, Forward &o, v4s *xcol = nullptr, int xstep = 0) {
    const int r = lane & 15, q = lane >> 4;
    if (c < 3) {   // the first layer's inputs 16 c + 4q + i of row r
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = 16 * c + 4 * q + i;
            v[i] = (r < nrows && k < IN) ? X[(size_t)(row0 + r) * IN + k] : 0.f;
        }
        *(v4s *)(S0 + r * LDA + 16 * c + 4 * q) = pack4(v);
    }
    __syncthreads();
    if (xcol && c < 3) {
        v4s v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (short)S0[(4 * q + i) * LDA + 16 * c + r];
        xcol[c * xstep] = v;
    }
    o.z1 = layer<3>(S0, net.w1, lane);
    activate(o.z1, net.b1, o.t1, o.a1, S1, c, lane);
    __syncthreads();
    o.z2 = layer<4>(S1, net.w2, lane);
    activate(o.z2, net.b2, o.t2, o.a2, S0, c, lane);
    __syncthreads();
    if (c < 2) {
        o.y = layer<4>(S0, net.w3, lane);
#pragma unroll
        for (int i = 0; i < 4; ++i) o.y[i] += net.b3;
    }
}

// GELU for inference: 0.5 z (1 + tanh u) = z / (1 + exp(-2u)),
// u = C (z + A z^3) = z (C + C A z^2), with the hardware exp2 and reciprocal
// (relative error ~1e-7, far below the bfloat16 rounding that follows).
__device__ __forceinline__ float gelu_fast(float z) {
    constexpr float K = -2.0f * 1.4426950408889634f;   // exp(-2u) = exp2(K u)
    const float e = __builtin_amdgcn_exp2f(z * __builtin_fmaf(z * z, K * GELU_C * GELU_A, K * GELU_C));
    return z * __builtin_amdgcn_rcpf(1.0f + e);
}

}  // namespace

// ---------------------------------------------------------------------------
// Training
// ---------------------------------------------------------------------------

// Network outputs Y [B][26] of B rows of X [B][34], a workgroup per 16 rows.
// Bound by the latency of its chain of layers, most of it the 32 tanh a row's
// lanes have in turn where one wave holds the rows: four waves have eight each
// (a call on 1003 rows: 7.9 us with one, 5.4 with four).
__global__ void __launch_bounds__(256) mlp_forward(MlpTrain t, const float *X, int B, float *Y) {
    __shared__ __attribute__((aligned(16))) uint16_t S[2][STAGE_ELEMS];
    const int c = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int row0 = blockIdx.x * 16;
    const Net net(t, c, lane);
    Forward o;
    forward16(X, row0, B - row0, net, S[0], S[1], c, lane, o);
    if (c < 2)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = row0 + 4 * q + i, col = 16 * c + r;
            if (row < B && col < OUT) Y[(size_t)row * OUT + col] = o.y[i];
        }
}

// Forward, backward and the partial weight gradients of groups of 32 rows in
// one pass, four waves per 16 rows: dY = 2 (y - T) / (B * 26);
// dZ2 = (dY W3) * gelu'(z2); dZ1 = (dZ2 W2) * gelu'(z1).  Everything stays in
// registers and LDS.  An MFMA result holds, per lane, four rows of a column,
// which is an operand of the products dZ^T A over the rows: the waves lay
// those operands down in LDS (21 KB) and share the 36 gradient tiles over the
// group's rows, and over the groups group, group + grid, ...; the workgroup's
// sums go to its slice of gpart, where mlp_reduce adds the slices in order
// (deterministic).  A batch of 4096 is 128 workgroups, bound by the latency of
// one group: with a wave per 16 rows, whose lanes have 32 tanh in turn and
// whose weights are loaded layer by layer, 20 us; with four waves, 15 in groups
// of 64 rows (four waves' tanh on a SIMD) and 12 in groups of 32.  Groups of
// 16 leave more slices to add than they save: a step and a gradient 36.6, 30.5
// and 38.6 us in groups of 64, 32 and 16.
constexpr int OP_DY = 0, OP_DZ2 = 2, OP_DZ1 = 6, OP_A2 = 10, OP_A1 = 14, OP_X = 18, OPS = 21;
constexpr int ROW_WAVES = TRAIN_ROWS / 16, TRAIN_WAVES = 4 * ROW_WAVES;
constexpr int WAVE_TILES = (WG_TILES + TRAIN_WAVES - 1) / TRAIN_WAVES;

__global__ void __launch_bounds__(64 * TRAIN_WAVES) mlp_train_rows(MlpTrain t, const float *X, const float *T, int B) {
    __shared__ __attribute__((aligned(16))) uint16_t stage[ROW_WAVES][2][STAGE_ELEMS];
    __shared__ v4s op[OPS][ROW_WAVES][64];
    __shared__ float red[ROW_WAVES][160];
    int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = wave >> 2, c = wave & 3;   // 16 rows of the group, 16 of their columns
    uint16_t *S0 = stage[w][0], *S1 = stage[w][1];
    const float scale = 2.0f / ((float)B * OUT);
    const Net net(t, c, lane);
    v4s w3t[2], w2t[4];
    weights<2>(t.wbT + WB_W3T, c, lane, w3t);
    weights<4>(t.wbT + WB_W2T, c, lane, w2t);
    v4f acc[WAVE_TILES];
#pragma unroll
    for (int j = 0; j < WAVE_TILES; ++j) acc[j] = v4f{0.f, 0.f, 0.f, 0.f};
    float db1 = 0.f, db2 = 0.f, db3 = 0.f, loss = 0.f;
    for (int g = blockIdx.x; TRAIN_ROWS * g < B; g += gridDim.x) {
        const int row0 = TRAIN_ROWS * g + 16 * w, nrows = min(16, B - row0);   // nrows <= 0: no rows left
        asm volatile("" : "+v"(lane));   // addresses are formed here, not kept from before the loop
        const int r = lane & 15, q = lane >> 4;
        float tgt[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 4 * q + i, col = 16 * c + r;
            tgt[i] = row < nrows && col < OUT ? T[(size_t)(row0 + row) * OUT + col] : 0.f;
        }
        Forward o;
        forward16(X, row0, nrows, net, S0, S1, c, lane, o, &op[OP_X][w][lane], ROW_WAVES * 64);
        if (c < 2) {   // dY, its bias sums and the loss (columns 26..31 are zero)
            float d[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                d[i] = 0.f;
                if (4 * q + i < nrows && 16 * c + r < OUT) {
                    const float e = o.y[i] - tgt[i];
                    loss += e * e;
                    d[i] = scale * e;
                }
                db3 += d[i];
            }
            const v4s v = pack4(d);
            stage_col(S1, c, lane, v);
            op[OP_DY + c][w][lane] = v;
        }
        __syncthreads();
        {   // dA2[r][h] = sum_o dY[r][o] W3[o][h]
            const v4f z = layer<2>(S1, w3t, lane);
            float d[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                d[i] = 4 * q + i < nrows ? z[i] * gelu_grad(o.z2[i], o.t2[i]) : 0.f;
                db2 += d[i];
            }
            const v4s v = pack4(d);
            stage_col(S0, c, lane, v);
            op[OP_DZ2 + c][w][lane] = v;
        }
        __syncthreads();
        {
            const v4f z = layer<4>(S0, w2t, lane);
            float d[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool in = 4 * q + i < nrows;
                d[i] = in ? z[i] * gelu_grad(o.z1[i], o.t1[i]) : 0.f;
                db1 += d[i];
                if (!in) o.a1[i] = o.a2[i] = 0;
            }
            op[OP_DZ1 + c][w][lane] = pack4(d);
            op[OP_A1 + c][w][lane] = o.a1;
            op[OP_A2 + c][w][lane] = o.a2;
        }
        __syncthreads();
        // tiles wave, wave + 8, ...: 0..7 W3 (2 x 4), 8..23 W2 (4 x 4), 24..35 W1 (4 x 3)
#pragma unroll
        for (int j = 0; j < WAVE_TILES; ++j) {
            const int tile = TRAIN_WAVES * j + wave;
            if (tile >= WG_TILES) break;
            const int oa = tile < 8 ? OP_DY + tile / 4 : (tile < 24 ? OP_DZ2 + (tile - 8) / 4 : OP_DZ1 + (tile - 24) / 3);
            const int ob = tile < 8 ? OP_A2 + tile % 4 : (tile < 24 ? OP_A1 + tile % 4 : OP_X + (tile - 24) % 3);
#pragma unroll
            for (int k = 0; k < ROW_WAVES; ++k) acc[j] = mfma(op[oa][k][lane], op[ob][k][lane], acc[j]);
        }
        __syncthreads();   // the operands are replaced by the next group's
    }
    float *gp = t.gpart + (size_t)blockIdx.x * GP_STRIDE;
    const int r = lane & 15, q = lane >> 4;
#pragma unroll
    for (int j = 0; j < WAVE_TILES; ++j) {
        const int tile = TRAIN_WAVES * j + wave;
        if (tile >= WG_TILES) break;
        const int mt = tile < 8 ? tile / 4 : (tile < 24 ? (tile - 8) / 4 : (tile - 24) / 3);
        const int nt = tile < 24 ? tile % 4 : (tile - 24) % 3;
        const int ofs = tile < 8 ? P_W3 : (tile < 24 ? P_W2 : P_W1);
        const int rows = tile < 8 ? OUT : HID, cols = tile < 24 ? HID : IN;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int m = 16 * mt + 4 * q + i, n = 16 * nt + r;
            if (m < rows && n < cols) gp[ofs + m * cols + n] = acc[j][i];
        }
    }
    // bias sums and the loss (two waves' columns): over the lane groups, then
    // over the rows' waves in order
    auto over_rows = [](float v) {
        v += __shfl_xor(v, 16, 64);
        return v + __shfl_xor(v, 32, 64);
    };
    const float s1 = over_rows(db1), s2 = over_rows(db2), s3 = over_rows(db3);
    if (q == 0) {
        red[w][16 * c + r] = s1;
        red[w][64 + 16 * c + r] = s2;
        if (16 * c + r < OUT) red[w][128 + 16 * c + r] = s3;
    }
    for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o, 64);
    if (lane == 0 && c < 2) red[w][128 + OUT + c] = loss;
    __syncthreads();
    const int i = threadIdx.x;
    if (i < 128 + OUT + 1) {
        float v = red[0][i];
#pragma unroll
        for (int k = 1; k < ROW_WAVES; ++k) v += red[k][i];
        if (i == 128 + OUT)
#pragma unroll
            for (int k = 0; k < ROW_WAVES; ++k) v += red[k][i + 1];
        gp[i < 64 ? P_B1 + i : (i < 128 ? P_B2 + i - 64 : (i < 128 + OUT ? P_B3 + i - 128 : NPAR))] = v;
    }
}

// ---------------------------------------------------------------------------
// Inference weight image
// ---------------------------------------------------------------------------
//
// Inference runs the network transposed, Z^T = W X^T: the weights are the A
// operand of v_mfma_f32_16x16x32_bf16 (lane l holds unit 16 mt + l % 16 and
// eight consecutive k), the 16 rows of a tile the B operand (lane l holds row
// l % 16 and the same eight k), so a layer's result lands with lane l holding
// row l % 16, units 16 mt + 4 (l / 16) + i.  Those sixteen values are exactly
// the B operand of the next layer if its k order lists, per 32-unit block kb
// and lane group q, units 32 kb + 4q + 0..3 and then 32 kb + 16 + 4q + 0..3:
// the image stores the next layer's weight columns in that order, and no
// activation ever goes through LDS.  The output layer's rows are ordered so
// that output position 16 e + 4q + t is end e (0: +d, 1: -d) of line 4q + t:
// the lanes of a row's group q hold both ends of up to four lines.

namespace {

// the +d direction (index into the 3x3x3 neighbourhood, 13 = centre) of the
// 13 lines in the network's output order
__constant__ int c_lines[13] = {LINE_DIR[0], LINE_DIR[1], LINE_DIR[2],  LINE_DIR[3],  LINE_DIR[4],
                                LINE_DIR[5], LINE_DIR[6], LINE_DIR[7],  LINE_DIR[8],  LINE_DIR[9],
                                LINE_DIR[10], LINE_DIR[11], LINE_DIR[12]};

// hidden unit at k position kap of a 64-wide layer input
__device__ __forceinline__ int hidden_of(int kap) {
    const int kb = kap >> 5, q = (kap >> 3) & 3, j = kap & 7;
    return 32 * kb + (j < 4 ? 4 * q + j : 16 + 4 * q + j - 4);
}

// network output (0..25) at output position o of the image, -1 for padding
__device__ __forceinline__ int output_of(int o) {
    const int e = o >> 4, lam = o & 15;
    if (lam >= 13) return -1;
    const int d = e == 0 ? c_lines[lam] : 26 - c_lines[lam];
    return d < 13 ? d : d - 1;
}

}  // namespace

// bf16 copies of the weights: W1p[64][64], W2[64][64], W3p[32][64] and the
// transposes used by the backward pass, W2T[64][64], W3T[64][64] (k = output);
// the inference image (W1i, W2i, W3i as MFMA A-operand fragments) and its
// biases (the first layer's per field: the one-hot input's weight folded in).
__global__ void __launch_bounds__(256) mlp_pack(MlpTrain t) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= 64 * 64) return;
    const int n = i / 64, k = i % 64;
    t.wb[WB_W1 + i] = bf16_bits(k < IN ? t.par[P_W1 + n * IN + k] : 0.f);
    t.wb[WB_W2 + i] = bf16_bits(t.par[P_W2 + n * HID + k]);
    if (n < 32) t.wb[WB_W3 + i] = bf16_bits(n < OUT ? t.par[P_W3 + n * HID + k] : 0.f);
    // transposes: W2T[h][k2] = W2[k2][h]; W3T[h][o] = W3[o][h] (o < 26, else 0)
    t.wbT[WB_W2T + i] = bf16_bits(t.par[P_W2 + k * HID + n]);
    t.wbT[WB_W3T + i] = bf16_bits(k < OUT ? t.par[P_W3 + k * HID + n] : 0.f);
    // inference image, fragment by fragment (see infer_frag)
    for (int e = i; e < WBI_SIZE; e += 64 * 64) {
        const int F = e >> 9, lane = (e >> 3) & 63, j = e & 7, r = lane & 15, kq = 8 * (lane >> 4) + j;
        float w = 0.f;
        if (F < 4) {                       // W1i, m-tile F
            if (kq < NNB) w = t.par[P_W1 + (16 * F + r) * IN + kq];
        } else if (F < 12) {               // W2i, m-tile (F - 4) / 2, k block (F - 4) % 2
            const int mt = (F - 4) >> 1, kb = (F - 4) & 1;
            w = t.par[P_W2 + (16 * mt + r) * HID + hidden_of(32 * kb + kq)];
        } else {                           // W3i, end (F - 12) / 2, k block (F - 12) % 2
            const int en = (F - 12) >> 1, kb = (F - 12) & 1, o = output_of(16 * en + r);
            if (o >= 0) w = t.par[P_W3 + o * HID + hidden_of(32 * kb + kq)];
        }
        t.wbi[e] = bf16_bits(w);
    }
    if (i < NF * HID) {
        const int f = i / HID, u = i % HID;
        t.bi[BI_B1 + i] = t.par[P_B1 + u] + bf16_float(bf16_bits(t.par[P_W1 + u * IN + NNB + f]));
    }
    if (i < HID) t.bi[BI_B2 + i] = t.par[P_B2 + i];
    if (i < 32) {
        const int o = output_of(i);
        t.bi[BI_B3 + i] = o >= 0 ? t.par[P_B3 + o] : 0.f;
    }
}

namespace {

// Hidden unit h's place among the inference image's columns: k block, lane
// group and element (the inverse of hidden_of).
struct HiddenPlace {
    int kb, q, j;
    __device__ explicit HiddenPlace(int h) : kb(h >> 5), q((h >> 2) & 3), j((h & 3) + ((h >> 4) & 1) * 4) {}
};

// Output o's line (0..12), + 16 where it is the line's -d end.
__constant__ LineOfDir c_line_of = make_line_of_dir();

// A new value x of parameter i into the bf16 copies and the image (mlp_pack's
// entries of i), except the image's first bias.
__device__ __forceinline__ void repack(const MlpTrain &t, int i, float x) {
    const uint16_t b = bf16_bits(x);
    if (i < P_B1) {
        const int n = i / IN, k = i % IN;
        t.wb[WB_W1 + n * 64 + k] = b;
        if (k < NNB) t.wbi[512 * (n >> 4) + 8 * (16 * (k >> 3) + (n & 15)) + (k & 7)] = b;
    } else if (i < P_W2) {   // the first bias
    } else if (i < P_B2) {
        const int n = (i - P_W2) / HID, k = (i - P_W2) % HID;
        const HiddenPlace h(k);
        t.wb[WB_W2 + n * 64 + k] = b;
        t.wbT[WB_W2T + k * 64 + n] = b;
        t.wbi[512 * (4 + 2 * (n >> 4) + h.kb) + 8 * (16 * h.q + (n & 15)) + h.j] = b;
    } else if (i < P_W3) {
        t.bi[BI_B2 + i - P_B2] = x;
    } else if (i < P_B3) {
        const int n = (i - P_W3) / HID, k = (i - P_W3) % HID, lt = c_line_of.v[n < 13 ? n : n + 1];
        const HiddenPlace h(k);
        t.wb[WB_W3 + n * 64 + k] = b;
        t.wbT[WB_W3T + k * 64 + n] = b;
        t.wbi[512 * (12 + 2 * (lt >> 4) + h.kb) + 8 * (16 * h.q + (lt & 15)) + h.j] = b;
    } else {
        const int n = i - P_B3;
        t.bi[BI_B3 + c_line_of.v[n < 13 ? n : n + 1]] = x;
    }
}

// Parameter of the reduction's place l: the first 512 places hold, eight to a
// hidden unit, its seven one-hot weights and its first bias, which the image's
// first bias adds up; then the other first weights; then the rest in order.
constexpr int COUPLED = 8 * HID;
__device__ __forceinline__ int param_of(int l) {
    if (l < COUPLED) return (l & 7) < NF ? P_W1 + (l >> 3) * IN + NNB + (l & 7) : P_B1 + (l >> 3);
    if (l < P_W2) return P_W1 + (l - COUPLED) / NNB * IN + (l - COUPLED) % NNB;
    return l;
}
static_assert(COUPLED + HID * NNB == P_W2, "places and parameters");

}  // namespace

// The slices' sums added in order (four threads a quarter of the slices each,
// then the quarters), into grad, or into an Adam step of the float32 masters
// and of their bf16 copies (a launch of mlp_pack after it took 4 us of a
// step's 24); the value after the parameters is the loss, the sum of squares /
// (B * 26).
struct Adam {
    float lr, b1, b2, eps, c1, c2;
};
__global__ void __launch_bounds__(256) mlp_reduce(MlpTrain t, int slices, int B, float *grad, Adam ad, float *loss) {
    __shared__ float part[4][64];
    const int l = threadIdx.x & 63, s0 = threadIdx.x >> 6, place = blockIdx.x * 64 + l;
    const int i = place <= NPAR ? param_of(place) : place;
    float s = 0.f;
    if (i <= NPAR) {
        float v[WG_SLICES / 4];
#pragma unroll
        for (int k = 0; k < WG_SLICES / 4; ++k) {
            const int sl = WG_SLICES / 4 * s0 + k;
            v[k] = sl < slices ? t.gpart[(size_t)sl * GP_STRIDE + i] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < WG_SLICES / 4; ++k) s += v[k];
    }
    part[s0][l] = s;
    __syncthreads();
    if (s0 || i > NPAR) return;
    const float g = ((part[0][l] + part[1][l]) + part[2][l]) + part[3][l];
    if (i == NPAR) {
        if (loss) *loss = g / ((float)B * OUT);
    } else if (grad) {
        grad[i] = g;
    } else {
        const float m = ad.b1 * t.m[i] + (1.f - ad.b1) * g;
        const float v = ad.b2 * t.v[i] + (1.f - ad.b2) * g * g;
        const float x = t.par[i] - ad.lr * (m / ad.c1) / (sqrtf(v / ad.c2) + ad.eps);
        t.m[i] = m;
        t.v[i] = v;
        t.par[i] = x;
        repack(t, i, x);
        if (place < COUPLED) {   // a whole wave: this block is all one-hot weights and first biases
            const float b1 = __shfl(x, l | 7, 64);
            const int f = l & 7, u = place >> 3;
            if (f < NF) t.bi[BI_B1 + HID * f + u] = b1 + bf16_float(bf16_bits(x));
        }
    }
}

// ---------------------------------------------------------------------------
// Inference pre-pass of a stage: every needed cell of every block
// ---------------------------------------------------------------------------

namespace {

typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int ICHUNK = NSLOT / 64;    // 14 workgroups per block, 64 needed cells each
constexpr int BOX = 300;              // 3 x 10 x 10 cells: the neighbourhoods of a chunk

__constant__ int16_t c_pad_ghost[NP];   // padded index -> ghost slot (-1 for interior cells)

__device__ __forceinline__ v4f mfma32(v8bf a, v8bf b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// A-operand fragment F of the inference image for this lane: fragments are
// stored lane by lane (64 x 8 bf16, 1 KB), so a wave reads 1 KB of
// consecutive LDS without bank conflicts.  F 0..3: W1i m-tile F; 4..11: W2i
// m-tile (F-4)/2, k block (F-4)%2; 12..15: W3i end (F-12)/2, k block (F-12)%2.
__device__ __forceinline__ v8bf infer_frag(const uint16_t *W, int F, int lane) {
    return *(const v8bf *)(W + 512 * F + 8 * lane);
}

// The plain limiter and the FP64 check on one line of a row, on its two
// predicted values R (at +d) and L (at -d): each value clamped between the
// cell and its neighbour in that direction, the pair put through the PPM
// monotonicity constraint and kept as binary32 offsets oR, oL from qc (see
// learned_limit), then the point values qc + offset are checked in FP64
// (bounds, positivity of rho, E, tau, non-negative X, the monotonicity
// conditions with a rounding slack of 1e-13 |D| (|L| + |q| + |R|); qc, nbR and
// nbL are no signalling NaN).  Limiter
// and check only ever couple the two ends of one line, so a row is processed
// line by line.  nbR / nbL are the neighbours in those directions.  Returns
// whether the line passes.  Written without branches: min/max clamps (a NaN
// prediction, which they would turn into a bound, fails explicitly) and
// selects for the constraint's cases.
__device__ __forceinline__ bool limit_check_line(double qc, double nbR, double nbL, int f, double R, double L,
                                                 float &oR, float &oL) {
    bool ok = (R == R) & (L == L);
    const double loR = min_of(qc, nbR), hiR = max_of(qc, nbR);
    const double loL = min_of(qc, nbL), hiL = max_of(qc, nbL);
    learned_limit(qc, min_of(max_of(R, loR), hiR), min_of(max_of(L, loL), hiL), oR, oL);
    const double r = qc + (double)oR, l = qc + (double)oL;
    ok = ok & (r >= loR) & (r <= hiR) & (l >= loL) & (l <= hiL);
    if (f == RHO || f == EGAS || f == TAU) ok = ok & (r > 0.0) & (l > 0.0);
    if (f == SPC) ok = ok & (r >= 0.0) & (l >= 0.0);
    {
        const double D = r - l, M6 = 6.0 * __builtin_fma(-0.5, l + r, qc), DM = D * M6;
        const double lim = __builtin_fma(1e-13 * fabs(D), fabs(l) + fabs(qc) + fabs(r), D * D);
        const bool mono = ((r - qc) * (qc - l) > 0.0) & !(fabs(DM) > lim);
        ok = ok & (((l == qc) & (r == qc)) | mono);
    }
    return ok;
}

__device__ __forceinline__ double shfl_xor_d(double v, int m) {
    return __shfl_xor(v, m, 64);
}

}  // namespace

// Workgroup (block, chunk): the chunk's 64 needed cells are one 8 x 8 layer of
// cells, normal to axis A at layer Lc (interior layers 0..7 along z, then the
// face-adjacent ghost slabs x-, x+, y-, y+, z-, z+); their 3x3x3
// neighbourhoods fill a 3 x 10 x 10 box, staged in LDS for all seven fields
// (one thread per box cell) next to the inference weight image.  Wave f then
// takes field f: four tiles of 16 cells, each lane group q of a tile computing
// features 8q .. 8q+7 of its cell (sigma and the density contrast combined
// over the group by lane exchange), the three layers on MFMA, and the limiter
// and FP64 check for its lines.  Point values go out as val[block][field]
// [dir][slot]; a cell passes when all seven of its rows pass.
// VAL64: the point values go out in FP64 to m.val (inspection), else as the
// binary32 offsets the stage reads to m.off.
// Bound by vector instructions (busy three quarters of the time): the GELUs'
// seven each, two of them transcendental, and the lines' limiter and check.
// Hence the box holds no signalling NaN (min and max need not quiet their
// operands), only the density's wave looks for the extremes, the features are
// formed without branches, and the tables are made by the wave that has
// nothing to load: 668 before, 633 us now for 1576 blocks.
template <bool VAL64>
__global__ void __launch_bounds__(64 * NF) __attribute__((amdgpu_waves_per_eu(7))) mlp_infer_kernel(MlpInfer m) {
    __shared__ double box[NF][BOX];                               // 16,800 B
    __shared__ __attribute__((aligned(16))) uint16_t W[WBI_SIZE];  // 16,384 B
    __shared__ __attribute__((aligned(16))) float bias[BI_SIZE];   //  2,176 B
    __shared__ unsigned long long fails[NF];
    __shared__ int4 otab[4][4];
    __shared__ int shared_s;
    const int item = xcd_leaf(blockIdx.x, gridDim.x);
    const int blk = m.leaf0 + item / ICHUNK, chunk = item % ICHUNK;
    const int tid = threadIdx.x, lane = tid & 63, f = tid >> 6;
    if (!VAL64 && m.alias && chunk >= NX) {
        // a ghost slab whose every cell shares its row with a block of this
        // launch (whose pre-pass computes it as an interior cell) is skipped:
        // the stage reads those rows there
        if (tid < 64) {
            const int al = m.alias[(size_t)blk * (NSLOT - NC) + 64 * (chunk - NX) + tid];
            const int tb = al / NSLOT;
            const bool in = al >= 0 && tb >= m.leaf0 && tb < m.leaf0 + (int)(gridDim.x / ICHUNK);
            const bool all = __all(in);
            if (tid == 0) shared_s = all;
        }
        __syncthreads();
        if (shared_s) return;
    }
    for (int i = tid; i < WBI_SIZE / 8; i += 64 * NF) ((uint4 *)W)[i] = ((const uint4 *)m.wbi)[i];
    for (int i = tid; i < BI_SIZE; i += 64 * NF) bias[i] = m.bi[i];
    // chunk geometry: box origin (o0, o1, o2), extents (d0, d1, 3 or 10)
    const int A = chunk < NX ? 2 : (chunk - NX) >> 1;
    const int Lc = chunk < NX ? chunk : (((chunk - NX) & 1) ? NX : -1);
    const int d0 = A == 0 ? 3 : 10, d1 = A == 1 ? 3 : 10;
    const int o0 = A == 0 ? Lc - 1 : -1, o1 = A == 1 ? Lc - 1 : -1, o2 = A == 2 ? Lc - 1 : -1;
    const int s1 = d0, s2 = d0 * d1;
    // per lane group q: neighbour offsets in the box of features 8q .. 8q+7
    // (k < 27), +d offsets of lines 4q .. 4q+3 and the output rows of their
    // two ends; read in each tile (kept live, they would cost 16 registers).
    // The last wave has no box cell to load and makes them meanwhile.
    static_assert(BOX <= 64 * (NF - 1), "a wave without box cells");
    if (tid >= 64 * (NF - 1) && tid < 64 * (NF - 1) + 4) {
        const int qq = lane;
        int ko[8], lo4[4], lr4[4];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = 8 * qq + j < NNB ? 8 * qq + j : 13;
            ko[j] = (k % 3 - 1) + s1 * ((k / 3) % 3 - 1) + s2 * (k / 9 - 1);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int lam = 4 * qq + t < 13 ? 4 * qq + t : 0;
            const int op = c_lines[lam], om = 26 - op;
            lo4[t] = (op % 3 - 1) + s1 * ((op / 3) % 3 - 1) + s2 * (op / 9 - 1);
            lr4[t] = (op < 13 ? op : op - 1) | ((om < 13 ? om : om - 1) << 8);
        }
        otab[qq][0] = int4{ko[0], ko[1], ko[2], ko[3]};
        otab[qq][1] = int4{ko[4], ko[5], ko[6], ko[7]};
        otab[qq][2] = int4{lo4[0], lo4[1], lo4[2], lo4[3]};
        otab[qq][3] = int4{lr4[0], lr4[1], lr4[2], lr4[3]};
    }
    {
        const double *Ub = m.U + block_base(blk, m.ts, m.lg);
        const size_t fs = (size_t)1 << (3 * m.lg);
        const int32_t *gm = m.gmap + (size_t)blk * NG;
        for (int c = tid; c < BOX; c += 64 * NF) {
            const int x = o0 + c % d0, y = o1 + (c / d0) % d1, z = o2 + c / s2;
            if (x >= 0 && x < NX && y >= 0 && y < NX && z >= 0 && z < NX) {
                const double *p = Ub + block_cell((z * NX + y) * NX + x, m.lg);
#pragma unroll
                for (int ff = 0; ff < NF; ++ff) box[ff][c] = __builtin_canonicalize(p[ff * fs]);
            } else {
                const int src = gm[c_pad_ghost[((z + GW) * PB + (y + GW)) * PB + (x + GW)]];
                double gs[NF];
                ghost_values(m.U, src, m.lg, m.prolong, m.n_prolong, gs);
#pragma unroll
                for (int ff = 0; ff < NF; ++ff) box[ff][c] = __builtin_canonicalize(gs[ff]);
            }
        }
    }
    __syncthreads();
    const int r = lane & 15, q = lane >> 4;
    const double *bx = box[f];
    float2 *oout = VAL64 ? nullptr : (float2 *)m.off + ((size_t)blk * NF + f) * 13 * NSLOT;
    double *vout = VAL64 ? m.val + ((size_t)blk * NF + f) * 26 * NSLOT : nullptr;
    unsigned long long wfail = 0;
#pragma unroll 1
    for (int tt = 0; tt < 4; ++tt) {
        const int s = 16 * tt + r, slot = 64 * chunk + s;
        const int u = s & 7, v = s >> 3;
        const int cx = A == 0 ? Lc : u, cy = A == 1 ? Lc : (A == 0 ? u : v), cz = A == 2 ? Lc : v;
        const int cb = (cx - o0) + s1 * (cy - o1) + s2 * (cz - o2);
        const double qc = bx[cb];
        int oz = 0;
        asm volatile("" : "+s"(oz));
        const int4 ka = otab[q + oz][0], kb4 = otab[q + oz][1];
        const int koff[8] = {ka.x, ka.y, ka.z, ka.w, kb4.x, kb4.y, kb4.z, kb4.w};
        double sig = 0.0;
#pragma unroll
        for (int j = 0; j < 8; ++j) sig = fmax(sig, fabs(bx[cb + koff[j]] - qc));   // (fmax passes over a NaN)
        // over the row's four lane groups
        sig = max_of(sig, shfl_xor_d(sig, 16));
        sig = max_of(sig, shfl_xor_d(sig, 32));
        const bool flat = !(sig > 0.0);
        if (__all(flat)) {
            // sixteen flat cells (sigma = 0 in this field): every point value
            // is the cell value, exactly, every row passes, and the network
            // is not evaluated
            const int4 lb = otab[q + oz][3];
            const int lrow[4] = {lb.x, lb.y, lb.z, lb.w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (4 * q + t >= 13) continue;
                if (VAL64) {
                    vout[(size_t)(lrow[t] & 255) * NSLOT + slot] = qc;
                    vout[(size_t)(lrow[t] >> 8) * NSLOT + slot] = qc;
                } else {
                    oout[(size_t)(4 * q + t) * NSLOT + slot] = float2{0.0f, 0.0f};
                }
            }
            continue;
        }
        // the network's error is a few percent of sigma: where the density
        // spans more than a factor 8 over the neighbourhood, the low side's
        // point values (and s / rho from them) would be off by order one
        bool ok = true;
        if (f == RHO) {
            asm volatile("" ::: "memory");   // this wave's alone: read here
            double lo = qc, hi = qc;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const double nvj = bx[cb + koff[j]];
                lo = min_of(lo, nvj);
                hi = max_of(hi, nvj);
            }
            lo = min_of(lo, shfl_xor_d(lo, 16));
            lo = min_of(lo, shfl_xor_d(lo, 32));
            hi = max_of(hi, shfl_xor_d(hi, 16));
            hi = max_of(hi, shfl_xor_d(hi, 32));
            ok = flat || hi <= 8.0 * lo;
        }
        const double rs = flat ? 0.0 : 1.0 / sig;
        asm volatile("" ::: "memory");   // re-read the neighbours rather than keep them live
        // (the padding's features are the cell's own: 0, or NaN where the row's are)
        v8bf x;
        {
            v4u xb;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v2bf t;
                t[0] = (__bf16)(float)((bx[cb + koff[2 * j]] - qc) * rs);
                t[1] = (__bf16)(float)((bx[cb + koff[2 * j + 1]] - qc) * rs);
                unsigned b = __builtin_bit_cast(unsigned, t);
                asm volatile("" : "+v"(b));   // computed by all lanes: a select, not a branch
                xb[j] = flat ? 0u : b;
            }
            x = __builtin_bit_cast(v8bf, xb);
        }
        // an opaque zero offset: the weight and bias fragments are then read
        // from LDS in every tile rather than hoisted out of the loop, where
        // they would hold 104 registers
        int wz = 0;
        asm volatile("" : "+s"(wz));
        const uint16_t *Wt = W + wz;
        const float *bt = bias + wz;
        // layer 1 (K = 32: the 27 neighbourhood features, zero padded)
        v4f z[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
            z[mt] = mfma32(infer_frag(Wt, mt, lane), x,
                           *(const v4f *)(bt + BI_B1 + HID * f + 16 * mt + 4 * q));
        v8bf h[2];
#pragma unroll
        for (int j = 0; j < 16; ++j) h[j >> 3][j & 7] = (__bf16)gelu_fast(z[(j >> 3) * 2 + ((j >> 2) & 1)][j & 3]);
        // layer 2
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            v4f c = *(const v4f *)(bt + BI_B2 + 16 * mt + 4 * q);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                c = mfma32(infer_frag(Wt, 4 + 2 * mt + kb, lane), h[kb], c);
            z[mt] = c;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) h[j >> 3][j & 7] = (__bf16)gelu_fast(z[(j >> 3) * 2 + ((j >> 2) & 1)][j & 3]);
        // output layer: y[e][t] = end e of line 4q + t
        v4f y[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            v4f c = *(const v4f *)(bt + BI_B3 + 16 * e + 4 * q);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
                c = mfma32(infer_frag(Wt, 12 + 2 * e + kb, lane), h[kb], c);
            y[e] = c;
        }
        // this lane's lines: denormalise, limit, check, store
        const int4 la = otab[q + wz][2], lb = otab[q + wz][3];
        const int loff[4] = {la.x, la.y, la.z, la.w}, lrow[4] = {lb.x, lb.y, lb.z, lb.w};
        float *yr = m.yraw ? m.yraw + (((size_t)blk * NF + f) * NSLOT + slot) * 26 : nullptr;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (4 * q + t >= 13) continue;
            if (yr) {
                yr[lrow[t] & 255] = y[0][t];
                yr[lrow[t] >> 8] = y[1][t];
            }
            float oR = 0.0f, oL = 0.0f;
            if (!flat) {
                const double R = qc + sig * (double)y[0][t];
                const double L = qc + sig * (double)y[1][t];
                ok = limit_check_line(qc, bx[cb + loff[t]], bx[cb - loff[t]], f, R, L, oR, oL) && ok;
            }
            if (VAL64) {
                vout[(size_t)(lrow[t] & 255) * NSLOT + slot] = qc + (double)oR;
                vout[(size_t)(lrow[t] >> 8) * NSLOT + slot] = qc + (double)oL;
            } else {
                oout[(size_t)(4 * q + t) * NSLOT + slot] = float2{oR, oL};
            }
        }
        const unsigned long long bad = __ballot(!ok);
        wfail |= ((bad | (bad >> 16) | (bad >> 32) | (bad >> 48)) & 0xffffull) << (16 * tt);
    }
    if (lane == 0) fails[f] = wfail;
    __syncthreads();
    // verdicts of the chunk's cells, and the count of those that fall back
    if (tid < 64) {
        unsigned long long any = 0;
#pragma unroll
        for (int ff = 0; ff < NF; ++ff) any |= fails[ff];
        const bool bad = (any >> tid) & 1ull;
        m.cell_ok[(size_t)blk * NSLOT + 64 * chunk + tid] = bad ? 0 : 1;
        // statistics count each block's interior cells (a ghost-slab cell is
        // counted in the block it belongs to)
        if (tid == 0 && any && chunk < NX) atomicAdd(m.fb_count, (unsigned long long)__popcll(any));
    }
}

hipError_t hydro_mlp_upload_pad_ghost(const int16_t *pad_ghost) {
    return hipMemcpyToSymbol(HIP_SYMBOL(c_pad_ghost), pad_ghost, sizeof(int16_t) * NP);
}

hipError_t hydro_mlp_launch_infer(const MlpInfer &m, int nleaf, hipStream_t s) {
    if (nleaf <= 0) return hipSuccess;
    if (m.val)
        hipLaunchKernelGGL(mlp_infer_kernel<true>, dim3(nleaf * ICHUNK), dim3(64 * NF), 0, s, m);
    else
        hipLaunchKernelGGL(mlp_infer_kernel<false>, dim3(nleaf * ICHUNK), dim3(64 * NF), 0, s, m);
    return hipGetLastError();
}

hipError_t hydro_mlp_launch_pack(const MlpTrain &t, hipStream_t s) {
    hipLaunchKernelGGL(mlp_pack, dim3(16), dim3(256), 0, s, t);
    return hipGetLastError();
}

hipError_t hydro_mlp_launch_forward(const MlpTrain &t, const float *X, int B, float *Y, hipStream_t s) {
    hipLaunchKernelGGL(mlp_forward, dim3((B + 15) / 16), dim3(256), 0, s, t, X, B, Y);
    return hipGetLastError();
}

static hipError_t launch_rows(const MlpTrain &t, const float *X, const float *T, int B, float *grad, const Adam &ad,
                              float *loss, hipStream_t s) {
    const int groups = (B + TRAIN_ROWS - 1) / TRAIN_ROWS, slices = groups < WG_SLICES ? groups : WG_SLICES;
    hipLaunchKernelGGL(mlp_train_rows, dim3(slices), dim3(64 * TRAIN_WAVES), 0, s, t, X, T, B);
    hipLaunchKernelGGL(mlp_reduce, dim3((NPAR + 64) / 64), dim3(256), 0, s, t, slices, B, grad, ad, loss);
    return hipGetLastError();
}

hipError_t hydro_mlp_launch_grad(const MlpTrain &t, const float *X, const float *T, int B, float *grad, float *loss,
                                 hipStream_t s) {
    return launch_rows(t, X, T, B, grad, Adam{}, loss, s);
}

hipError_t hydro_mlp_launch_step(const MlpTrain &t, const float *X, const float *T, int B, float lr, float b1, float b2,
                                 float eps, float c1, float c2, float *loss, hipStream_t s) {
    return launch_rows(t, X, T, B, nullptr, Adam{lr, b1, b2, eps, c1, c2}, loss, s);
}
