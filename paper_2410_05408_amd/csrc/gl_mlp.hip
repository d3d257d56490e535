// gl_mlp.hip -- the residual surrogate network on the GPU: BF16 matrix-core
// (MFMA) GEMMs with FP32 accumulation, fused bias/GELU epilogues, backward
// pass, MSE loss and Adam on FP32 master weights.
//
// Network: x[n][16] -> [Linear -> GELU] x 4 (width 256) -> Linear -> y[n]
// (input width 16: the encoded features, zero-padded).  Activations and the
// weights fed to the matrix cores are BF16; accumulation, biases, the output
// layer, the loss, gradients of the output layer and the optimizer are FP32.
// All reductions run in a fixed order (no floating-point atomics).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "gl.h"
#include "gl_internal.h"

namespace {

constexpr int D_IN = GL_MLP_DIN;   // 16
constexpr int W = GL_MLP_WIDTH;    // 256
constexpr int DEPTH = 4;           // hidden layers

using bf16 = unsigned short;

__device__ __forceinline__ bf16 f2bf(float f)
{
    unsigned int u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
    return (bf16)(u >> 16);
}
__device__ __forceinline__ float bf2f(bf16 h) { return __uint_as_float(((unsigned int)h) << 16); }

constexpr float kGeluC = 0.7978845608028654f;  // sqrt(2/pi)

// tanh(u) = 1 - 2 / (exp(2u) + 1) from the hardware exponential and
// reciprocal (relative error ~1e-6, far below the BF16 rounding of the
// activations; exp overflow gives exactly 1, underflow exactly -1)
__device__ __forceinline__ float tanh_fast(float u)
{
    return 1.0f - 2.0f * __builtin_amdgcn_rcpf(__expf(2.0f * u) + 1.0f);
}

__device__ __forceinline__ float gelu(float z)
{
    return 0.5f * z * (1.0f + tanh_fast(kGeluC * (z + 0.044715f * z * z * z)));
}
__device__ __forceinline__ float gelu_grad(float z)
{
    const float th = tanh_fast(kGeluC * (z + 0.044715f * z * z * z));
    const float du = kGeluC * (1.0f + 3.0f * 0.044715f * z * z);
    return 0.5f * (1.0f + th) + 0.5f * z * (1.0f - th * th) * du;
}

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8_t as_bf8(u32x4_t v) { return __builtin_bit_cast(bf16x8_t, v); }
// BF16 values are handled as 16-bit halves of 32-bit words (element j in
// word j/2, low half first); single elements are never read out of a bf16x8_t
__device__ __forceinline__ bf16 half_of(u32x4_t v, int j) { return (bf16)(v[j >> 1] >> (16 * (j & 1))); }
__device__ __forceinline__ unsigned pack2(bf16 lo, bf16 hi) { return (unsigned)lo | ((unsigned)hi << 16); }

// MFMA 16x16x32 BF16 (gfx950), FP32 accumulate.  Lane l holds row l%16 of A
// and column l%16 of B, each with 8 values of the K dimension (lane group
// l/16 picks which 8: the same choice for both operands, so the K order in
// which values are laid out only has to agree between A and B); the result
// D[4(l/16)+i][l%16], i < 4, lands in lane l.
__device__ __forceinline__ float4_t mfma32(bf16x8_t a, bf16x8_t b, float4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// x (fp32 [n][16]) -> bf16
__global__ void k_to_bf16(const float* __restrict__ x, bf16* __restrict__ y, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = f2bf(x[i]);
}

// Training batch: rows perm(step * batch + i) of X / T, where perm(j) =
// (a j + c) mod n for a coprime to n (a fresh permutation every epoch).
__global__ void k_gather_rows(const bf16* __restrict__ Xall, const float* __restrict__ Tall, int64_t n,
                              uint64_t a, uint64_t c, int64_t j0, int batch, bf16* __restrict__ X,
                              float* __restrict__ T)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)batch * D_IN) return;
    const int64_t i = e / D_IN, f = e % D_IN;
    const uint64_t r = ((unsigned __int128)a * (uint64_t)(j0 + i) + c) % (uint64_t)n;
    X[e] = Xall[r * D_IN + f];
    if (f == 0) T[i] = Tall[r];
}

// hist[0] += loss[0] / n (one thread: the epoch's mean squared error)
__global__ void k_add_loss(const float* __restrict__ loss, float inv_n, float* __restrict__ hist)
{
    hist[0] += loss[0] * inv_n;
}

// packed parameter layout (FP32): W0[16][256] b0[256] W1[256][256] b1 W2 b2 W3 b3 w4[256] b4[1]
constexpr int64_t kSizeW0 = (int64_t)D_IN * W;
constexpr int64_t kSizeWh = (int64_t)W * W;
constexpr int64_t kOffW4 = kSizeW0 + W + 3 * (kSizeWh + W);
constexpr int64_t kOffB4 = kOffW4 + W;
constexpr int64_t kNParam = kOffB4 + 1;

__host__ __device__ constexpr int64_t off_w(int l) { return l == 0 ? 0 : kSizeW0 + W + (int64_t)(l - 1) * (kSizeWh + W); }
__host__ __device__ constexpr int64_t off_b(int l) { return off_w(l) + (l == 0 ? kSizeW0 : kSizeWh); }
constexpr int64_t in_dim(int l) { return l == 0 ? D_IN : W; }

// ---------------------------------------------------------------- training step
// One step is three launches:
//   k_train_rows    forward, loss gradient and the backward chain of a block of
//                   rows, activations in registers and LDS throughout;
//   k_train_sums    everything summed over the batch: weight gradients (matrix
//                   cores, split over row chunks), bias and output-layer
//                   column sums, loss;
//   k_train_update  the partial sums in order, then Adam.
// Between them lie the layer inputs and the dL/dZ of every layer, stored the
// way the matrix cores take them when rows are the contraction: per 32 rows a
// tile [feature][32 rows], so that a wavefront's operand (16 features x 32 rows)
// is one contiguous kilobyte.  (One GEMM, reduction or elementwise kernel per
// layer and direction, 29 launches through row-major activations and transposed
// LDS stores, took 314 us a step at 8192 rows, these three 59; every sum is in the
// same order.)
constexpr int kTR = 32;             // rows per tile and per block of k_train_rows
constexpr int kTrWaves = 8;         // each 32 of the 256 features
constexpr int kTP = W + 8;          // LDS row pitch (bf16): the 16 rows of an operand fall on different banks
constexpr int64_t kTile = (int64_t)W * kTR;  // elements of a tile of W features

// BF16 weights in the order in which the matrix cores take them: for 16
// features of one side and 32 of the contraction, lane l holds feature l % 16
// and 8 (l / 16) .. + 7 of the contraction, a contiguous kilobyte.  Forward
// (contraction over inputs; layer 0's 16 inputs: the first 32 lanes only) and,
// for layers 1..3, backward (contraction over outputs).
__host__ __device__ constexpr int64_t off_f(int l) { return l == 0 ? 0 : kSizeW0 + (int64_t)(l - 1) * kSizeWh; }
__host__ __device__ constexpr int64_t off_r(int l) { return (int64_t)(l - 1) * kSizeWh; }
constexpr int64_t kSizeF = kSizeW0 + 3 * kSizeWh, kSizeR = 3 * kSizeWh;

__device__ __forceinline__ int frag_pos(int f, int c) { return ((f >> 4) * (W / 32) + (c >> 5)) * 512 + ((c >> 3) & 3) * 128 + (f & 15) * 8 + (c & 7); }
// positions of weight (k, n) of layer l
__device__ __forceinline__ int64_t f_pos(int l, int k, int n)
{
    return l == 0 ? (n >> 4) * 256 + (k >> 3) * 128 + (n & 15) * 8 + (k & 7) : off_f(l) + frag_pos(n, k);
}
__device__ __forceinline__ int64_t r_pos(int l, int k, int n) { return off_r(l) + frag_pos(k, n); }

struct TrainBufs {
    const float* p;      // master parameters
    const bf16 *wf, *wr; // BF16 weights, forward and backward order
    bf16* in[DEPTH];     // layer inputs (x, H0, H1, H2) in tiles
    bf16* h;             // last hidden layer's output in tiles
    bf16* dz[DEPTH];     // dL/dZ in tiles
    float *dy, *sq;      // per row: dL/dy, squared residual
};

__device__ __forceinline__ bf16x8_t load_op(const bf16* p) { return *reinterpret_cast<const bf16x8_t*>(p); }

// Bound by the latency of its nine dependent stages and, below that, by the
// 0.8 MB of weights each block pulls from L2 (64 bytes a clock: 5 us); a
// stage's weights are loaded while the stage before is finished.  32 rows per
// block give 256 blocks at 8192 rows, one per CU: 26 us (41 with the weights
// row-major, where an operand touches 16 half lines).
__global__ void __launch_bounds__(kTrWaves * 64)
k_train_rows(const float* __restrict__ xf, const bf16* __restrict__ xb, const float* __restrict__ t, int n, TrainBufs B)
{
    __shared__ __align__(16) bf16 Hs[2][kTR][kTP];
    __shared__ __align__(16) bf16 Xs[kTR][D_IN + 8];
    __shared__ __align__(16) float w4s[W];
    __shared__ float dys[kTR];
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t tile = blockIdx.x;
    const int r0 = (int)(tile * kTR);
    const int f0 = wave * 32;  // this wavefront's features
    bf16x8_t wf[2][W / 32];    // a stage's weights: feature f0 + 16 c + lr, K 32 kb + 8 lg ...
    auto weights = [&](const bf16* src) {
        __builtin_amdgcn_sched_barrier(0);  // not before the last product has read wf
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int kb = 0; kb < W / 32; ++kb)
                wf[c][kb] = load_op(src + ((2 * wave + c) * (W / 32) + kb) * 512 + lane * 8);
    };
    const bf16x8_t zero8 = as_bf8(u32x4_t{0u, 0u, 0u, 0u});
    bf16x8_t w0[2];
    float bias[DEPTH][2];
    for (int c = 0; c < 2; ++c) {
        w0[c] = lg < 2 ? load_op(B.wf + (2 * wave + c) * 256 + lane * 8) : zero8;
#pragma unroll
        for (int l = 0; l < DEPTH; ++l) bias[l][c] = B.p[off_b(l) + f0 + 16 * c + lr];
    }
    const float target = tid < kTR && r0 + tid < n ? t[r0 + tid] : 0.f;
    {
        // one input element per thread
        const int r = tid >> 4, f = tid & 15;
        bf16 v = 0;
        if (r0 + r < n) v = xf ? f2bf(xf[(int64_t)(r0 + r) * D_IN + f]) : xb[(int64_t)(r0 + r) * D_IN + f];
        Xs[r][f] = v;
        if (tid < W) w4s[tid] = B.p[kOffW4 + tid];
    }
    weights(B.wf + off_f(1));
    __syncthreads();
    B.in[0][tile * (D_IN * kTR) + tid] = Xs[tid & 31][tid >> 5];  // [feature][row]
    float4_t acc[2][2];  // [row tile][feature tile]: rows 16 a + 4 lg + i, feature f0 + 16 c + lr
    unsigned z[DEPTH][2][2][2];  // bf16(Z) of each layer, pairs of rows
    auto clear = [&] {
        for (int a = 0; a < 2; ++a)
            for (int c = 0; c < 2; ++c) acc[a][c] = float4_t{0.f, 0.f, 0.f, 0.f};
    };
    auto product = [&](int buf) {
        clear();
#pragma unroll
        for (int kb = 0; kb < W / 32; ++kb) {
            bf16x8_t x[2];
            for (int a = 0; a < 2; ++a) x[a] = load_op(&Hs[buf][16 * a + lr][32 * kb + 8 * lg]);
            for (int a = 0; a < 2; ++a)
                for (int c = 0; c < 2; ++c) acc[a][c] = mfma32(x[a], wf[c][kb], acc[a][c]);
        }
    };
    // four rows' values of a feature to LDS (row-major) and to the tile in
    // memory (rows beyond the batch as zero)
    auto put = [&](int buf, bf16* dst, int a, int c, const bf16* v) {
        const int f = f0 + 16 * c + lr, r = 16 * a + 4 * lg;
        bf16 q[4];
        for (int i = 0; i < 4; ++i) {
            Hs[buf][r + i][f] = v[i];
            q[i] = r0 + r + i < n ? v[i] : (bf16)0;
        }
        uint2 u;
        u.x = pack2(q[0], q[1]);
        u.y = pack2(q[2], q[3]);
        *reinterpret_cast<uint2*>(dst + tile * kTile + f * kTR + r) = u;
    };
    int buf = 0;
#pragma unroll
    for (int l = 0; l < DEPTH; ++l) {
        if (l == 0) {
            clear();
            for (int a = 0; a < 2; ++a) {
                const bf16x8_t x = lg < 2 ? load_op(&Xs[16 * a + lr][8 * lg]) : zero8;
                for (int c = 0; c < 2; ++c) acc[a][c] = mfma32(x, w0[c], acc[a][c]);
            }
        } else {
            product(buf);
            buf ^= 1;
            weights(l + 1 < DEPTH ? B.wf + off_f(l + 1) : B.wr + off_r(DEPTH - 1));
        }
        bf16* dst = l + 1 < DEPTH ? B.in[l + 1] : B.h;
        for (int c = 0; c < 2; ++c) {
            for (int a = 0; a < 2; ++a) {
                bf16 h[4], zz[4];
                for (int i = 0; i < 4; ++i) {
                    const float v = acc[a][c][i] + bias[l][c];
                    zz[i] = f2bf(v);
                    h[i] = f2bf(gelu(v));
                }
                z[l][a][c][0] = pack2(zz[0], zz[1]);
                z[l][a][c][1] = pack2(zz[2], zz[3]);
                put(buf, dst, a, c, h);
            }
        }
        __syncthreads();
    }
    // output layer (FP32, k in order) and the loss: a row per lane
    if (tid < kTR) {
        const int m = r0 + tid;
        float s = 0.f;
#pragma unroll 4
        for (int k = 0; k < W; k += 8) {
            const u32x4_t v = *reinterpret_cast<const u32x4_t*>(&Hs[buf][tid][k]);
            const float4_t wa = *reinterpret_cast<const float4_t*>(&w4s[k]), wb = *reinterpret_cast<const float4_t*>(&w4s[k + 4]);
            for (int j = 0; j < 8; ++j) s = fmaf(bf2f(half_of(v, j)), j < 4 ? wa[j] : wb[j - 4], s);
        }
        const float y = s + B.p[kOffB4];
        float d = 0.f;
        if (m < n) {
            const float r = y - target;
            d = 2.0f * r / (float)n;
            B.dy[m] = d;
            B.sq[m] = r * r;
        }
        dys[tid] = d;
    }
    __syncthreads();
    // dZ of the last hidden layer, then down the layers
    buf ^= 1;
    for (int c = 0; c < 2; ++c) {
        const float w4 = w4s[f0 + 16 * c + lr];
        for (int a = 0; a < 2; ++a) {
            bf16 v[4];
            for (int i = 0; i < 4; ++i) {
                const unsigned zz = z[DEPTH - 1][a][c][i >> 1];
                v[i] = f2bf(dys[16 * a + 4 * lg + i] * w4 * gelu_grad(bf2f((bf16)(zz >> (16 * (i & 1))))));
            }
            put(buf, B.dz[DEPTH - 1], a, c, v);
        }
    }
    __syncthreads();
#pragma unroll
    for (int l = DEPTH - 1; l > 0; --l) {
        product(buf);
        buf ^= 1;
        if (l > 1) weights(B.wr + off_r(l - 1));
        for (int c = 0; c < 2; ++c)
            for (int a = 0; a < 2; ++a) {
                bf16 v[4];
                for (int i = 0; i < 4; ++i) {
                    const unsigned zz = z[l - 1][a][c][i >> 1];
                    v[i] = f2bf(acc[a][c][i] * gelu_grad(bf2f((bf16)(zz >> (16 * (i & 1))))));
                }
                put(buf, B.dz[l - 1], a, c, v);
            }
        __syncthreads();
    }
}

// Row chunks of the weight gradients: chunk rows (a multiple of 32) and count.
struct Split {
    int rows, count;
};

// Workgroups of k_train_sums, in this order: the two vector sums (the longest
// chains), column sums, weight gradients of layers 3..1 and of layer 0.
struct SumArgs {
    int n, groups;        // rows, column-sum groups of kColRows rows
    Split hid, first;     // layers 1..3, layer 0
    TrainBufs B;
    float* dw[DEPTH];     // partial weight gradients: [chunk][16 x 16 tile][lane][4]
    float* col;           // partial column sums: [DEPTH + 1][group][W] (dZ of each layer, then H3 dy)
    float* vec;           // sums of dy and of sq
};

constexpr int kColRows = 256;  // rows per column-sum partial

// A wavefront's [16 nk x 64] piece of the gradient over the tiles [t0, t1):
// the operands straight from memory, the D tile as lane l: in-feature l % 16,
// out-features 4 (l / 16) + i.
template <int NK>
__device__ __forceinline__ void grad_piece(const bf16* __restrict__ in, int64_t in_tile, const bf16* __restrict__ dz,
                                           int t0, int t1, int k0, int n0, int lane, float* __restrict__ out)
{
    const int lr = lane & 15, lg = lane >> 4;
    float4_t acc[NK][4];
    for (int i = 0; i < NK; ++i)
        for (int j = 0; j < 4; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
    bf16x8_t a[3][NK], b[3][4];
    auto fetch = [&](int s, int t) {
        for (int i = 0; i < NK; ++i) a[s][i] = load_op(in + t * in_tile + (k0 + 16 * i + lr) * kTR + 8 * lg);
        for (int j = 0; j < 4; ++j) b[s][j] = load_op(dz + t * kTile + (n0 + 16 * j + lr) * kTR + 8 * lg);
    };
    auto mul = [&](int s) {
        for (int i = 0; i < NK; ++i)
            for (int j = 0; j < 4; ++j) acc[i][j] = mfma32(b[s][j], a[s][i], acc[i][j]);
    };
    // two tiles ahead
    fetch(0, t0);
    if (t0 + 1 < t1) fetch(1, t0 + 1);
    for (int t = t0; t < t1; t += 3) {
        if (t + 2 < t1) fetch(2, t + 2);
        mul(0);
        if (t + 3 < t1) fetch(0, t + 3);
        if (t + 1 < t1) mul(1);
        if (t + 4 < t1) fetch(1, t + 4);
        if (t + 2 < t1) mul(2);
    }
    for (int i = 0; i < NK; ++i)
        for (int j = 0; j < 4; ++j) {
            const int tile = (k0 / 16 + i) * (W / 16) + n0 / 16 + j;
            *reinterpret_cast<float4_t*>(out + ((int64_t)tile * 64 + lane) * 4) = acc[i][j];
        }
}

// Bound by reading the 33 MB of tiles and writing 26 MB of partials (8192
// rows): 15 us.  A wavefront takes a 64 x 64 piece of a gradient over one row chunk:
// 8 operands for 16 matrix instructions, none through LDS.
__global__ void __launch_bounds__(256) k_train_sums(SumArgs A)
{
    __shared__ float red[256];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int b = blockIdx.x;
    if (b < 2) {
        // a vector sum: rows in 256 phases, then a tree
        const float* x = b == 0 ? A.B.dy : A.B.sq;
        float acc = 0.f;
#pragma unroll 16
        for (int m = tid; m < A.n; m += 256) acc += x[m];
        red[tid] = acc;
        __syncthreads();
        for (int d = 128; d >= 1; d >>= 1) {
            if (tid < d) red[tid] += red[tid + d];
            __syncthreads();
        }
        if (tid == 0) A.vec[b] = red[0];
        return;
    }
    b -= 2;
    if (b < (DEPTH + 1) * A.groups) {
        // column sums of a group: a column per thread, its rows in four phases
        const int which = b / A.groups, grp = b - which * A.groups;
        const bf16* src = (which < DEPTH ? A.B.dz[which] : A.B.h) + tid * kTR;
        red[tid] = which == DEPTH && grp * kColRows + tid < A.n ? A.B.dy[grp * kColRows + tid] : 0.f;
        __syncthreads();
        // (rows beyond the batch are zero)
        const int t0 = grp * (kColRows / kTR), nt = min((A.n + kTR - 1) / kTR - t0, kColRows / kTR);
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        // (all of a thread's loads first: its sums are one chain, and a load
        // per link took 17 us)
        u32x4_t v[kColRows / kTR][4];
#pragma unroll
        for (int t = 0; t < kColRows / kTR; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v[t][q] = *reinterpret_cast<const u32x4_t*>(src + (t0 + min(t, nt - 1)) * kTile + 8 * q);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < kColRows / kTR; ++t) {
            if (t >= nt) break;
#pragma unroll
            for (int r = 0; r < kTR; ++r) {
                const float x = bf2f(half_of(v[t][r >> 3], r & 7));
                acc[r & 3] = which == DEPTH ? fmaf(x, red[t * kTR + r], acc[r & 3]) : acc[r & 3] + x;
            }
        }
        A.col[((int64_t)which * A.groups + grp) * W + tid] = ((acc[0] + acc[1]) + acc[2]) + acc[3];
        return;
    }
    b -= (DEPTH + 1) * A.groups;
    const int tiles = (A.n + kTR - 1) / kTR;
    if (b < 3 * 4 * A.hid.count) {
        const int l = 1 + b / (4 * A.hid.count), r = b % (4 * A.hid.count);
        // (chunks fastest: the four workgroups of one chunk, which read the same
        // dZ, then mostly share an XCD's L2)
        const int q = r / A.hid.count, s = r - q * A.hid.count;
        const int t0 = s * (A.hid.rows / kTR), t1 = min(tiles, t0 + A.hid.rows / kTR);
        grad_piece<4>(A.B.in[l], kTile, A.B.dz[l], t0, t1, q * 64, wave * 64, lane,
                      A.dw[l] + (int64_t)s * kSizeWh);
        return;
    }
    const int s = b - 3 * 4 * A.hid.count;
    const int t0 = s * (A.first.rows / kTR), t1 = min(tiles, t0 + A.first.rows / kTR);
    grad_piece<1>(A.B.in[0], D_IN * kTR, A.B.dz[0], t0, t1, 0, wave * 64, lane, A.dw[0] + (int64_t)s * kSizeW0);
}

struct UpdateArgs {
    SumArgs S;
    float *p, *g, *m, *v;
    bf16 *wf, *wr;
    float lr, c1, c2;
    float* loss;       // the batch's sum of squared residuals goes here too, if given
};

// Adam on FP32 master weights and their BF16 copies.
// c1 = 1 - b1^step and c2 = 1 - b2^step come from the host in FP64 (in FP32,
// 1 - 0.999^step loses ~1e-5 to cancellation), and 1 - b1, 1 - b2 are the
// FP32 roundings of 0.1 and 0.001 rather than differences of rounded betas.
__device__ __forceinline__ float adam(const UpdateArgs& U, float w, float gi, float& m, float& v)
{
    const float b1 = 0.9f, b2 = 0.999f, omb1 = 0.1f, omb2 = 0.001f, eps = 1e-8f;
    const float mi = b1 * m + omb1 * gi;
    const float vi = b2 * v + omb2 * gi * gi;
    m = mi;
    v = vi;
    return w - U.lr * (mi / U.c1) / (sqrtf(vi / U.c2) + eps);
}

// Gradients from the partials, in order of the chunks; GRADS: into g,
// otherwise straight into Adam.  Threads: four out-features of a weight row
// each (the partials' layout), then the biases, the output layer and the loss.
// Bound by reading the partials: 8 us at 8192 rows.
constexpr int kUpThreadsW = (int)((kSizeW0 + 3 * kSizeWh) / 4);
constexpr int kUpThreads = kUpThreadsW + (DEPTH + 1) * W + 2;
template <bool GRADS>
__global__ void __launch_bounds__(256) k_train_update(UpdateArgs U)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < kUpThreadsW) {
        const int l = i < kSizeW0 / 4 ? 0 : 1 + (i - (int)(kSizeW0 / 4)) / (int)(kSizeWh / 4);
        const int e = l == 0 ? i : (i - (int)(kSizeW0 / 4)) % (int)(kSizeWh / 4);
        const int S = l == 0 ? U.S.first.count : U.S.hid.count;
        const int64_t step = l == 0 ? kSizeW0 : kSizeWh;
        const float* src = U.S.dw[l] + (int64_t)e * 4;
        const int tile = e >> 6, lane = e & 63;
        const int k = 16 * (tile / (W / 16)) + (lane & 15), nn = 16 * (tile % (W / 16)) + 4 * (lane >> 4);
        const int64_t o = off_w(l) + (int64_t)k * W + nn;
        float4_t w = *reinterpret_cast<const float4_t*>(U.p + o), m = *reinterpret_cast<const float4_t*>(U.m + o),
                 v = *reinterpret_cast<const float4_t*>(U.v + o);
        float4_t g = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 16
        for (int s = 0; s < S; ++s) {
            const float4_t x = *reinterpret_cast<const float4_t*>(src + s * step);
            for (int j = 0; j < 4; ++j) g[j] += x[j];
        }
        if (GRADS) {
            *reinterpret_cast<float4_t*>(U.g + o) = g;
            return;
        }
        bf16 q[4];
        for (int j = 0; j < 4; ++j) {
            float mj = m[j], vj = v[j];
            const float wj = adam(U, w[j], g[j], mj, vj);
            m[j] = mj;
            v[j] = vj;
            w[j] = wj;
            q[j] = f2bf(wj);
            U.wf[f_pos(l, k, nn + j)] = q[j];
        }
        *reinterpret_cast<float4_t*>(U.p + o) = w;
        *reinterpret_cast<float4_t*>(U.m + o) = m;
        *reinterpret_cast<float4_t*>(U.v + o) = v;
        if (l > 0) {
            uint2 u;
            u.x = pack2(q[0], q[1]);
            u.y = pack2(q[2], q[3]);
            *reinterpret_cast<uint2*>(U.wr + r_pos(l, k, nn)) = u;
        }
        return;
    }
    const int c = i - kUpThreadsW;
    if (c >= (DEPTH + 1) * W + 2) return;
    if (c == (DEPTH + 1) * W + 1) {
        if (U.loss) U.loss[0] = U.S.vec[1];
        return;
    }
    float g = 0.f;
    int64_t o = kOffB4;
    if (c < (DEPTH + 1) * W) {
        const int which = c / W, f = c % W;
        o = which < DEPTH ? off_b(which) + f : kOffW4 + f;
#pragma unroll 8
        for (int s = 0; s < U.S.groups; ++s) g += U.S.col[((int64_t)which * U.S.groups + s) * W + f];
    } else {
        g = U.S.vec[0];
    }
    if (GRADS) {
        U.g[o] = g;
        return;
    }
    float m = U.m[o], v = U.v[o];
    const float w = adam(U, U.p[o], g, m, v);
    U.p[o] = w;
    U.m[o] = m;
    U.v[o] = v;
}

// BF16 weights of new parameters in the training step's two orders
__global__ void k_refresh_bf16(const float* __restrict__ w, bf16* __restrict__ wf, bf16* __restrict__ wr)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kNParam) return;
    const bf16 v = f2bf(w[i]);
    for (int l = 0; l < DEPTH; ++l) {
        const int64_t e = i - off_w(l);
        if (e < 0 || i >= off_b(l)) continue;
        wf[f_pos(l, (int)(e / W), (int)(e % W))] = v;
        if (l > 0) wr[r_pos(l, (int)(e / W), (int)(e % W))] = v;
    }
}

// ---------------------------------------------------------------- fused inference
// The whole network for a block of rows in one kernel, activations kept in
// registers from layer to layer.  Each layer is computed transposed,
// H^T[out][row] = W^T[out][in] X^T[in][row], with the weights as the MFMA A
// operand (from LDS) and the activations as the B operand: lane l holds sample
// l%16.  The accumulator tiles of one layer are then the B operands of the next
// with no data movement: the two 16-feature tiles 2kb and 2kb+1 give lane group
// g the features {32kb + 4g + i} and {32kb + 16 + 4g + i} (i < 4), which become
// the 8 K values of K block kb when the next layer's weights are stored with
// their input features in that order (kInK below).
constexpr int kInferWaves = 8;                              // two wavefronts per SIMD (256 registers each)
constexpr int kInferTiles = 2;                              // 16-sample tiles per wavefront
constexpr int kInferRows = kInferWaves * kInferTiles * 16;  // rows per block and round
constexpr int kW0K = 32;                                    // layer-0 K (16 features, zero-padded)
constexpr int64_t kInferW = (int64_t)W * kW0K + 3 * (int64_t)W * W;  // prepared weights (bf16)
// The weights pass through LDS in pieces of 64 output features (layer 0: all
// 256), 32 KB, two buffers: a piece is loaded into registers while the one
// before it is worked on.
constexpr int kPiece = 64 * W;                 // bf16 elements
constexpr int kPieces = 1 + 3 * (W / 64);      // per round
constexpr int kInferStage = kPiece / 8 / (kInferWaves * 64);  // 16-byte loads per thread
static_assert(W * kW0K <= kPiece && W * kW0K / 8 <= kInferStage * kInferWaves * 64, "layer 0 is one piece");

// input feature at position kp of the permuted K order of a hidden layer
__host__ __device__ constexpr int kInK(int kp)
{
    return 32 * (kp / 32) + 4 * ((kp % 32) / 8) + ((kp % 8) < 4 ? (kp % 8) : 12 + (kp % 8));
}

// prepared weights, operand by operand (16 outputs x 32 K, lane by lane: a
// contiguous kilobyte): layer 0 [16 output tiles] (k >= 16 zero), layers 1..3
// [16 output tiles][8 K blocks] with input feature kInK(k') at position k'
__global__ void k_prep_infer(const float* __restrict__ p, bf16* __restrict__ wt)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kInferW) return;
    const int j = (int)(i & 7), lane = (int)(i >> 3) & 63;
    if (i < (int64_t)W * kW0K) {
        const int out = (int)(i >> 9) * 16 + (lane & 15), k = 8 * (lane >> 4) + j;
        wt[i] = k < D_IN ? f2bf(p[(int64_t)k * W + out]) : (bf16)0;
        return;
    }
    const int64_t e = i - (int64_t)W * kW0K;
    const int l = 1 + (int)(e / ((int64_t)W * W));
    const int op = (int)(e % ((int64_t)W * W)) >> 9;  // operand: output tile, K block
    const int out = (op / (W / 32)) * 16 + (lane & 15), kp = 32 * (op % (W / 32)) + 8 * (lane >> 4) + j;
    wt[i] = f2bf(p[off_w(l) + (int64_t)kInK(kp) * W + out]);
}

// GELU (tanh form) as z times a logistic function: z / (1 + exp(-2u)) with
// u = sqrt(2/pi) (z + 0.044715 z^3).  One exponential and one reciprocal, and
// no difference of nearly equal numbers for negative z.
__device__ __forceinline__ float gelu_logistic(float z)
{
    constexpr float k1 = -2.0f * kGeluC * 1.4426950408889634f, k3 = 0.044715f * k1;
    return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(z * fmaf(k3, z * z, k1)));
}

// two floats to a BF16 pair, rounded to nearest even
__device__ __forceinline__ unsigned cvt2bf(float lo, float hi)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f2{lo, hi}, b2));
}

// A value the optimiser does not know: addresses computed from it are computed
// again where they are used rather than held in registers across the loop.
__device__ __forceinline__ int fresh_v(int i)
{
    asm volatile("" : "+v"(i));
    return i;
}

// y[r] = network(X[r]) for r < n, n = min(n_cap, *n_dev) (or n_cap); X BF16
// [rows][16]; persistent over blocks of kInferRows rows.
// Bound by the vector units (10 instructions per GELU, two of them at a quarter
// of the rate, 70 % of the cycles); the matrix units' 32 % run beside them,
// with the GELUs of one pair of tiles between the matrix instructions of the
// next.  99 k rows: 187 us with 35 vector instructions per GELU, one wavefront
// per SIMD and the matrix instructions before the GELUs; 118 with these GELUs
// and two wavefronts, 74 interleaved, 63 with a last round of one tile per
// wavefront where that holds the rows left (a round of 65536 rows 37 us, of
// 32768 24; a call of 1000 rows 36 -> 25 us).
__global__ void __launch_bounds__(kInferWaves * 64)
k_mlp_infer(const bf16* __restrict__ X, int64_t n_cap, const unsigned long long* __restrict__ n_dev,
            const bf16* __restrict__ wt, const float* __restrict__ p, float* __restrict__ y)
{
    __shared__ __align__(16) bf16 Wl[2][kPiece];
    __shared__ __align__(16) float bl[DEPTH][W];
    __shared__ __align__(16) float w4[W];
    const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int64_t n = n_cap;
    if (n_dev) n = min(n, (int64_t)*n_dev);
    // rows per block of the round that starts at row `base`: all, or half of
    // them (one tile per wavefront) where that takes every row left
    auto share = [&](int64_t base) { return n - base <= (int64_t)gridDim.x * (kInferRows / 2) ? kInferRows / 2 : kInferRows; };
    int64_t base = 0;
    if ((int64_t)blockIdx.x * share(base) >= n) return;
    for (int i = tid; i < DEPTH * W; i += kInferWaves * 64) bl[i / W][i % W] = p[off_b(i / W) + i % W];
    if (tid < W) w4[tid] = p[kOffW4 + tid];
    const float b4 = p[kOffB4];
    u32x4_t st[kInferStage];
    // piece q of a round: layer 0 (and what follows it), then four of each hidden layer
    auto fetch = [&](int q) {
        const bf16* src = q == 0 ? wt : wt + (int64_t)W * kW0K + (int64_t)(q - 1) * kPiece;
        const int tid = fresh_v(threadIdx.x);
#pragma unroll
        for (int j = 0; j < kInferStage; ++j) {
            st[j] = *reinterpret_cast<const u32x4_t*>(src + (j * kInferWaves * 64 + tid) * 8);
        }
    };
    auto stash = [&](int buf) {
        const int tid = fresh_v(threadIdx.x);
#pragma unroll
        for (int j = 0; j < kInferStage; ++j)
            *reinterpret_cast<u32x4_t*>(&Wl[buf][(j * kInferWaves * 64 + tid) * 8]) = st[j];
    };
    bf16x8_t xb[kInferTiles];
    // K values 8 lg .. 8 lg + 7 of sample lr (features >= 16 are zero)
    auto rows = [&](int64_t base) {
        const int lane = fresh_v(threadIdx.x) & 63, lr = lane & 15, lg = lane >> 4, per = share(base);
        for (int s = 0; s < kInferTiles; ++s) {
            const int at = per == kInferRows ? (wave * kInferTiles + s) * 16 : wave * 16;
            const int64_t row = base + (int64_t)blockIdx.x * per + at + lr;
            const bool has = lg < 2 && row < n;
            u32x4_t v = *reinterpret_cast<const u32x4_t*>(X + (has ? row * D_IN + 8 * lg : 0));
            for (int i = 0; i < 4; ++i) v[i] = has ? v[i] : 0u;
            xb[s] = as_bf8(v);
        }
    };
    fetch(0);
    rows(base);
    stash(0);
    __syncthreads();
    int buf = 0;
    u32x4_t hb[kInferTiles][W / 32], hn[kInferTiles][W / 32];  // B operands: this layer's, the next one's
    float4_t pend[kInferTiles][2];  // a pair of output tiles before bias and GELU
    // two features of the pending pair (q of 4 per sample tile) to BF16
    auto gelu2 = [&](u32x4_t& h, int s, int q, const float4_t& b) {
        const int i = 2 * (q & 1);
        unsigned v = cvt2bf(gelu_logistic(pend[s][q >> 1][i] + b[i]), gelu_logistic(pend[s][q >> 1][i + 1] + b[i + 1]));
        asm volatile("" : "+v"(v));  // here, not where it is used (a layer later)
        h[q] = v;
    };
    auto bias = [&](int l, int kb, int u) { return *reinterpret_cast<const float4_t*>(&bl[l][32 * kb + 16 * u + 4 * lg]); };
    auto finish = [&](auto tiles, u32x4_t (&dst)[kInferTiles][W / 32], int l, int kb) {
        constexpr int T = decltype(tiles)::value;
        const float4_t b[2] = {bias(l, kb, 0), bias(l, kb, 1)};
        for (int s = 0; s < T; ++s)
            for (int q = 0; q < 4; ++q) gelu2(dst[s][kb], s, q, b[q >> 1]);
    };
    // A pair of output tiles of a hidden layer from the h-th half of a piece,
    // the pending pair's GELUs (K block kp of layer lp, into dst) a few at a
    // time between the matrix instructions of each K block, all before the
    // last one, which may need them
    auto pair = [&](auto tiles, int h, u32x4_t (&dst)[kInferTiles][W / 32], int lp, int kp) {
        constexpr int T = decltype(tiles)::value;
        float4_t acc[T][2];
        const float4_t b[2] = {bias(lp, kp, 0), bias(lp, kp, 1)};
        auto operand = [&](int u, int kb) {
            return *reinterpret_cast<const bf16x8_t*>(&Wl[buf][((2 * h + u) * (W / 32) + kb) * 512 + lane * 8]);
        };
        bf16x8_t a[2] = {operand(0, 0), operand(1, 0)};
        int g = 0;
#pragma unroll
        for (int kb = 0; kb < W / 32; ++kb) {
            const bf16x8_t a0 = a[0], a1 = a[1];
            if (kb + 1 < W / 32) {
                a[0] = operand(0, kb + 1);
                a[1] = operand(1, kb + 1);
            }
            for (int s = 0; s < T; ++s) {
                const bf16x8_t x = as_bf8(hb[s][kb]);
                acc[s][0] = mfma32(a0, x, kb ? acc[s][0] : float4_t{0.f, 0.f, 0.f, 0.f});
                acc[s][1] = mfma32(a1, x, kb ? acc[s][1] : float4_t{0.f, 0.f, 0.f, 0.f});
            }
            for (int r = 0; r < (kb == 0 ? 2 : 1) && g < 4 * T; ++r, ++g) gelu2(dst[g >> 2][kp], g >> 2, g & 3, b[(g >> 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int s = 0; s < T; ++s)
            for (int u = 0; u < 2; ++u) pend[s][u] = acc[s][u];
    };
    // one round: T tiles of 16 rows per wavefront from the block's first row r0
    auto round = [&](auto tiles, int64_t r0, int64_t next) {
        constexpr int T = decltype(tiles)::value;
        fetch(1);
#pragma unroll
        for (int kb = 0; kb < W / 32; ++kb) {
            if (kb) finish(tiles, hn, 0, kb - 1);
            for (int u = 0; u < 2; ++u) {
                const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(&Wl[buf][(2 * kb + u) * 512 + lane * 8]);
                for (int s = 0; s < T; ++s) pend[s][u] = mfma32(a, xb[s], float4_t{0.f, 0.f, 0.f, 0.f});
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        stash(buf ^ 1);
        __syncthreads();
        buf ^= 1;
        for (int l = 1; l < DEPTH; ++l) {
            for (int s = 0; s < T; ++s)
                for (int kb = 0; kb < W / 32 - 1; ++kb) hb[s][kb] = hn[s][kb];
#pragma unroll
            for (int c = 0; c < W / 64; ++c) {
                const int q = 1 + (l - 1) * (W / 64) + c;
                // the next piece (after the last one, the next round's first)
                fetch(q + 1 < kPieces ? q + 1 : 0);
                if (c == 0) pair(tiles, 0, hb, l - 1, W / 32 - 1);
                else pair(tiles, 0, hn, l, 2 * c - 1);
                pair(tiles, 1, hn, l, 2 * c);
                if (c == W / 64 - 1 && l == DEPTH - 1 && next < n) rows(next);
                stash(buf ^ 1);
                __syncthreads();
                buf ^= 1;
            }
        }
        finish(tiles, hn, DEPTH - 1, W / 32 - 1);
        // output layer in FP32 on the BF16 activations, features summed over
        // the four lane groups
        const int lane = fresh_v(threadIdx.x) & 63, lr = lane & 15, lg = lane >> 4;
        for (int s = 0; s < T; ++s) {
            float a = 0.f;
            for (int kb = 0; kb < W / 32; ++kb) {
                const float4_t wa = *reinterpret_cast<const float4_t*>(&w4[32 * kb + 4 * lg]),
                               wb = *reinterpret_cast<const float4_t*>(&w4[32 * kb + 16 + 4 * lg]);
                for (int j = 0; j < 8; ++j) a = fmaf(bf2f(half_of(hn[s][kb], j)), j < 4 ? wa[j] : wb[j - 4], a);
            }
            a += __shfl_xor(a, 16);
            a += __shfl_xor(a, 32);
            const int64_t row = r0 + (int64_t)(wave * T + s) * 16 + lr;
            if (lg == 0 && row < n) y[row] = a + b4;
        }
    };
    while (base < n) {
        const int per = share(base);
        const int64_t r0 = base + (int64_t)blockIdx.x * per, next = base + (int64_t)gridDim.x * per;
        if (r0 >= n) return;
        if (per == kInferRows) round(std::integral_constant<int, kInferTiles>(), r0, next);
        else round(std::integral_constant<int, kInferTiles / 2>(), r0, next);
        base = next;
    }
}

}  // namespace

struct gl_mlp {
    int device = 0;
    int max_batch = 0;
    int64_t step = 0;
    std::string err;
    float *p = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;  // master, grad, Adam
    bf16 *wf = nullptr, *wr = nullptr;                              // BF16 weights (TrainBufs)
    bf16* X = nullptr;                                              // BF16 input rows
    bf16 *in[DEPTH] = {}, *h = nullptr, *dz[DEPTH] = {};            // training: tiles (TrainBufs)
    float *t = nullptr, *dy = nullptr, *sq = nullptr;               // a batch's targets, dL/dy, squares
    float* vec = nullptr;       // sums of dy and sq
    float *dw[DEPTH] = {}, *col = nullptr;  // partial sums
    bf16* wt = nullptr;         // weights prepared for the fused inference kernel
    bool wt_stale = true;       // master weights changed since wt was prepared
    int n_cu = 256;
};

namespace {

gl_status mfail(gl_mlp* m, gl_status st, const char* what, hipError_t e = hipSuccess)
{
    if (m) {
        m->err = what;
        if (e != hipSuccess) {
            m->err += ": ";
            m->err += hipGetErrorString(e);
        }
    }
    return st;
}

#define GM_HIP(call, what)                                                 \
    do {                                                                   \
        hipError_t e_ = (call);                                            \
        if (e_ != hipSuccess) return mfail(mm, GL_ERR_DEVICE, what, e_);   \
    } while (0)

unsigned blocks(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// Row chunks of a weight gradient [K][W] over n rows: enough for two
// wavefronts per SIMD when the pieces were 64 x 64, at most 64.
Split split_of(const gl_mlp* mm, int K, int64_t n)
{
    const int tiles = (K + 63) / 64 * (W / 64);
    const int64_t S = std::max(1, std::min(64, (2 * mm->n_cu + tiles - 1) / tiles));
    const int64_t rows = ((n + S - 1) / S + kTR - 1) / kTR * kTR;
    return {(int)rows, (int)((n + rows - 1) / rows)};
}

// One step on n <= max_batch rows: x (FP32, else the BF16 rows of mm->X) and
// targets t; gradients into mm->g, or Adam when u is given.
void train_pass(gl_mlp* mm, const float* x, const float* t, int n, const UpdateArgs* u, float* loss, hipStream_t s)
{
    UpdateArgs U{};
    if (u) U = *u;
    U.p = mm->p;
    U.g = mm->g;
    U.m = mm->m;
    U.v = mm->v;
    U.wf = mm->wf;
    U.wr = mm->wr;
    U.loss = loss;
    SumArgs& A = U.S;
    A.n = n;
    A.groups = (n + kColRows - 1) / kColRows;
    A.hid = split_of(mm, W, n);
    A.first = split_of(mm, D_IN, n);
    TrainBufs& B = A.B;
    B.p = mm->p;
    B.wf = mm->wf;
    B.wr = mm->wr;
    for (int l = 0; l < DEPTH; ++l) {
        B.in[l] = mm->in[l];
        B.dz[l] = mm->dz[l];
        A.dw[l] = mm->dw[l];
    }
    B.h = mm->h;
    B.dy = mm->dy;
    B.sq = mm->sq;
    A.col = mm->col;
    A.vec = mm->vec;
    hipLaunchKernelGGL(k_train_rows, dim3((n + kTR - 1) / kTR), dim3(kTrWaves * 64), 0, s, x, mm->X, t, n, B);
    const int sums = 2 + (DEPTH + 1) * A.groups + 12 * A.hid.count + A.first.count;
    hipLaunchKernelGGL(k_train_sums, dim3(sums), dim3(256), 0, s, A);
    if (u) hipLaunchKernelGGL(k_train_update<false>, dim3(blocks(kUpThreads)), dim3(256), 0, s, U);
    else hipLaunchKernelGGL(k_train_update<true>, dim3(blocks(kUpThreads)), dim3(256), 0, s, U);
}

// Adam's factors of the step after mm->step steps
UpdateArgs next_step(gl_mlp* mm, float lr)
{
    mm->step += 1;
    UpdateArgs U{};
    U.lr = lr;
    U.c1 = (float)(1.0 - std::pow(0.9, (double)mm->step));
    U.c2 = (float)(1.0 - std::pow(0.999, (double)mm->step));
    return U;
}

// refreshes the fused kernel's prepared weights if the masters changed
void prepare_infer(gl_mlp* mm, hipStream_t s)
{
    if (!mm->wt_stale) return;
    hipLaunchKernelGGL(k_prep_infer, dim3(blocks(kInferW)), dim3(256), 0, s, mm->p, mm->wt);
    mm->wt_stale = false;
}

void launch_infer(gl_mlp* mm, const bf16* X, int64_t n_cap, const unsigned long long* n_dev, float* y,
                  hipStream_t s)
{
    prepare_infer(mm, s);
    const int64_t rounds = (n_cap + kInferRows / 2 - 1) / (kInferRows / 2);  // of half the rows, see k_mlp_infer
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(rounds, mm->n_cu));
    hipLaunchKernelGGL(k_mlp_infer, dim3(grid), dim3(kInferWaves * 64), 0, s, X, n_cap, n_dev, mm->wt, mm->p, y);
}

}  // namespace

extern "C" {

int gl_mlp_num_params(void) { return (int)kNParam; }

gl_status gl_mlp_create(gl_mlp** out, int device, int max_batch)
{
    if (!out) return GL_ERR_NULL;
    *out = nullptr;
    if (max_batch < 64 || max_batch > (1 << 22) || max_batch % 64) return GL_ERR_SIZE;
    if (hipSetDevice(device) != hipSuccess) return GL_ERR_DEVICE;
    gl_mlp* mm = new (std::nothrow) gl_mlp();
    if (!mm) return GL_ERR_NOMEM;
    mm->device = device;
    mm->max_batch = max_batch;
    bool ok = true;
    auto al = [&](void** pp, size_t bytes) {
        if (hipMalloc(pp, bytes) != hipSuccess) ok = false;
    };
    al((void**)&mm->p, sizeof(float) * kNParam);
    al((void**)&mm->g, sizeof(float) * kNParam);
    al((void**)&mm->m, sizeof(float) * kNParam);
    al((void**)&mm->v, sizeof(float) * kNParam);
    al((void**)&mm->wf, sizeof(bf16) * kSizeF);
    al((void**)&mm->wr, sizeof(bf16) * kSizeR);
    al((void**)&mm->X, sizeof(bf16) * (size_t)max_batch * D_IN);
    for (int l = 0; l < DEPTH; ++l) {
        al((void**)&mm->in[l], sizeof(bf16) * (size_t)max_batch * in_dim(l));
        al((void**)&mm->dz[l], sizeof(bf16) * (size_t)max_batch * W);
    }
    al((void**)&mm->h, sizeof(bf16) * (size_t)max_batch * W);
    al((void**)&mm->t, sizeof(float) * (size_t)max_batch);
    al((void**)&mm->dy, sizeof(float) * max_batch);
    al((void**)&mm->sq, sizeof(float) * max_batch);
    al((void**)&mm->vec, sizeof(float) * 4);
    // (at most 64 chunks, and none shorter than 32 rows)
    const size_t chunks = std::min<size_t>(64, (size_t)max_batch / kTR);
    for (int l = 0; l < DEPTH; ++l) al((void**)&mm->dw[l], sizeof(float) * chunks * (size_t)(l == 0 ? kSizeW0 : kSizeWh));
    al((void**)&mm->col, sizeof(float) * (DEPTH + 1) * W * (size_t)((max_batch + kColRows - 1) / kColRows));
    al((void**)&mm->wt, sizeof(bf16) * kInferW);
    int ncu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && ncu > 0)
        mm->n_cu = ncu;
    if (ok) {
        ok = hipMemset(mm->p, 0, sizeof(float) * kNParam) == hipSuccess &&
             hipMemset(mm->g, 0, sizeof(float) * kNParam) == hipSuccess &&
             hipMemset(mm->m, 0, sizeof(float) * kNParam) == hipSuccess &&
             hipMemset(mm->v, 0, sizeof(float) * kNParam) == hipSuccess &&
             hipMemset(mm->wf, 0, sizeof(bf16) * kSizeF) == hipSuccess &&
             hipMemset(mm->wr, 0, sizeof(bf16) * kSizeR) == hipSuccess &&
             hipDeviceSynchronize() == hipSuccess;
    }
    if (!ok) {
        gl_mlp_destroy(mm);
        return GL_ERR_NOMEM;
    }
    *out = mm;
    return GL_OK;
}

void gl_mlp_destroy(gl_mlp* mm)
{
    if (!mm) return;
    (void)hipSetDevice(mm->device);
    (void)hipDeviceSynchronize();
    void* bufs[] = {mm->p, mm->g, mm->m, mm->v, mm->wf, mm->wr, mm->X, mm->h, mm->t, mm->dy, mm->sq, mm->vec, mm->col,
                    mm->wt};
    for (void* b : bufs) (void)hipFree(b);
    for (int l = 0; l < DEPTH; ++l) {
        (void)hipFree(mm->in[l]);
        (void)hipFree(mm->dz[l]);
        (void)hipFree(mm->dw[l]);
    }
    delete mm;
}

const char* gl_mlp_last_error(const gl_mlp* mm) { return mm ? mm->err.c_str() : "null network"; }

gl_status gl_mlp_set_weights(gl_mlp* mm, const float* host, int64_t n)
{
    if (!mm || !host) return GL_ERR_NULL;
    if (n != kNParam) return mfail(mm, GL_ERR_SIZE, "parameter count");
    GM_HIP(hipSetDevice(mm->device), "hipSetDevice");
    GM_HIP(hipMemcpy(mm->p, host, sizeof(float) * kNParam, hipMemcpyHostToDevice), "hipMemcpy");
    GM_HIP(hipMemset(mm->m, 0, sizeof(float) * kNParam), "hipMemset");
    GM_HIP(hipMemset(mm->v, 0, sizeof(float) * kNParam), "hipMemset");
    hipLaunchKernelGGL(k_refresh_bf16, dim3(blocks(kNParam)), dim3(256), 0, 0, mm->p, mm->wf, mm->wr);
    mm->wt_stale = true;
    prepare_infer(mm, 0);
    GM_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
    mm->step = 0;
    return GL_OK;
}

gl_status gl_mlp_get_weights(const gl_mlp* mmc, float* host, int64_t n)
{
    gl_mlp* mm = const_cast<gl_mlp*>(mmc);
    if (!mm || !host) return GL_ERR_NULL;
    if (n != kNParam) return mfail(mm, GL_ERR_SIZE, "parameter count");
    GM_HIP(hipSetDevice(mm->device), "hipSetDevice");
    GM_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
    GM_HIP(hipMemcpy(host, mm->p, sizeof(float) * kNParam, hipMemcpyDeviceToHost), "hipMemcpy");
    return GL_OK;
}

gl_status gl_mlp_forward(gl_mlp* mm, const float* x, int64_t n, float* y, void* stream)
{
    if (!mm || !x || !y) return GL_ERR_NULL;
    if (n < 0) return mfail(mm, GL_ERR_SIZE, "n < 0");
    GM_HIP(hipSetDevice(mm->device), "hipSetDevice");
    hipStream_t s = (hipStream_t)stream;
    // fused kernel over chunks of max_batch rows converted to BF16
    for (int64_t r0 = 0; r0 < n; r0 += mm->max_batch) {
        const int nb = (int)std::min<int64_t>(mm->max_batch, n - r0);
        hipLaunchKernelGGL(k_to_bf16, dim3(blocks((int64_t)nb * D_IN)), dim3(256), 0, s,
                           x + r0 * D_IN, mm->X, (int64_t)nb * D_IN);
        launch_infer(mm, mm->X, nb, nullptr, y + r0, s);
    }
    GM_HIP(hipGetLastError(), "kernel launch");
    return GL_OK;
}

gl_status gl_mlp_grads(gl_mlp* mm, const float* x, const float* t, int64_t n, float* host_grads,
                       float* host_loss, void* stream)
{
    if (!mm || !x || !t || !host_grads) return GL_ERR_NULL;
    if (n < 1 || n > mm->max_batch) return mfail(mm, GL_ERR_SIZE, "1 <= n <= max_batch");
    GM_HIP(hipSetDevice(mm->device), "hipSetDevice");
    hipStream_t s = (hipStream_t)stream;
    train_pass(mm, x, t, (int)n, nullptr, nullptr, s);
    GM_HIP(hipGetLastError(), "kernel launch");
    GM_HIP(hipStreamSynchronize(s), "hipStreamSynchronize");
    GM_HIP(hipMemcpy(host_grads, mm->g, sizeof(float) * kNParam, hipMemcpyDeviceToHost), "hipMemcpy");
    if (host_loss) {
        float l = 0.f;
        GM_HIP(hipMemcpy(&l, mm->vec + 1, sizeof(float), hipMemcpyDeviceToHost), "hipMemcpy");
        *host_loss = l / (float)n;
    }
    return GL_OK;
}

// loss_dev (device, optional) receives the batch's sum of squared residuals
gl_status gl_mlp_train_step(gl_mlp* mm, const float* x, const float* t, int64_t n, float lr,
                            float* loss_dev, void* stream)
{
    if (!mm || !x || !t) return GL_ERR_NULL;
    if (n < 1 || n > mm->max_batch) return mfail(mm, GL_ERR_SIZE, "1 <= n <= max_batch");
    hipStream_t s = (hipStream_t)stream;
    const UpdateArgs U = next_step(mm, lr);
    // the last kernel stores the loss itself where it can reach it (a copy of
    // four bytes costs a launch of its own)
    hipPointerAttribute_t at{};
    const bool store = loss_dev && (uintptr_t)loss_dev % sizeof(float) == 0 &&
                       hipPointerGetAttributes(&at, loss_dev) == hipSuccess && at.type == hipMemoryTypeDevice &&
                       at.device == mm->device;
    if (loss_dev && !store) (void)hipGetLastError();  // (an unknown pointer leaves an error)
    train_pass(mm, x, t, (int)n, &U, store ? loss_dev : nullptr, s);
    mm->wt_stale = true;
    if (loss_dev && !store)
        GM_HIP(hipMemcpyAsync(loss_dev, mm->vec + 1, sizeof(float), hipMemcpyDeviceToDevice, s),
               "hipMemcpyAsync");
    GM_HIP(hipGetLastError(), "kernel launch");
    return GL_OK;
}

}  // extern "C"

// ---------------------------------------------------------------- internal calls
namespace gl_net {

namespace {
uint64_t mix64(uint64_t z)
{
    z += 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}
uint64_t gcd64(uint64_t a, uint64_t b)
{
    while (b) {
        const uint64_t t = a % b;
        a = b;
        b = t;
    }
    return a;
}
}  // namespace

int max_batch(const gl_mlp* mm) { return mm->max_batch; }

gl_status train_rows(gl_mlp* mm, const uint16_t* X, const float* T, int64_t n, int epochs, int batch,
                     float lr, float lr_final, uint64_t seed, float* hist_dev, hipStream_t s)
{
    if (!mm || !X || !T) return GL_ERR_NULL;
    if (batch < 64 || batch > mm->max_batch || n < batch || epochs < 1) return mfail(mm, GL_ERR_SIZE, "training sizes");
    GM_HIP(hipSetDevice(mm->device), "hipSetDevice");
    const int64_t per_epoch = n / batch;
    const int64_t steps = per_epoch * epochs;
    int64_t step = 0;
    for (int ep = 0; ep < epochs; ++ep) {
        // a fresh permutation j -> (a j + c) mod n
        uint64_t a = (mix64(seed * 1315423911ull + (uint64_t)ep) % (uint64_t)n) | 1ull;
        while (gcd64(a, (uint64_t)n) != 1ull) a += 2;
        const uint64_t c = mix64(seed + 7919ull * (uint64_t)(ep + 1)) % (uint64_t)n;
        for (int64_t b = 0; b < per_epoch; ++b, ++step) {
            hipLaunchKernelGGL(k_gather_rows, dim3(blocks((int64_t)batch * D_IN)), dim3(256), 0, s, (const bf16*)X, T, n,
                               a % (uint64_t)n, c, b * batch, batch, mm->X, mm->t);
            const float lr_s = (float)((double)lr * std::pow((double)lr_final / (double)lr,
                                                             (double)step / (double)std::max<int64_t>(1, steps - 1)));
            const UpdateArgs U = next_step(mm, lr_s);
            train_pass(mm, nullptr, mm->t, batch, &U, nullptr, s);
            if (hist_dev)
                hipLaunchKernelGGL(k_add_loss, dim3(1), dim3(1), 0, s, mm->vec + 1, 1.0f / (float)(per_epoch * batch),
                                   hist_dev + ep);
        }
    }
    mm->wt_stale = true;
    GM_HIP(hipGetLastError(), "kernel launch");
    return GL_OK;
}

void infer(gl_mlp* mm, const uint16_t* X, int64_t n_cap, const unsigned long long* n_dev, float* y, hipStream_t s)
{
    launch_infer(mm, (const bf16*)X, n_cap, n_dev, y, s);
}

gl_status get_state(const gl_mlp* mmc, float* m, float* v, int64_t* step)
{
    gl_mlp* mm = const_cast<gl_mlp*>(mmc);
    if (!mm || !m || !v || !step) return GL_ERR_NULL;
    GM_HIP(hipSetDevice(mm->device), "hipSetDevice");
    GM_HIP(hipDeviceSynchronize(), "hipDeviceSynchronize");
    GM_HIP(hipMemcpy(m, mm->m, sizeof(float) * kNParam, hipMemcpyDeviceToHost), "hipMemcpy");
    GM_HIP(hipMemcpy(v, mm->v, sizeof(float) * kNParam, hipMemcpyDeviceToHost), "hipMemcpy");
    *step = mm->step;
    return GL_OK;
}

gl_status set_state(gl_mlp* mm, const float* m, const float* v, int64_t step)
{
    if (!mm || !m || !v) return GL_ERR_NULL;
    GM_HIP(hipSetDevice(mm->device), "hipSetDevice");
    GM_HIP(hipMemcpy(mm->m, m, sizeof(float) * kNParam, hipMemcpyHostToDevice), "hipMemcpy");
    GM_HIP(hipMemcpy(mm->v, v, sizeof(float) * kNParam, hipMemcpyHostToDevice), "hipMemcpy");
    mm->step = step;
    return GL_OK;
}

}  // namespace gl_net
