// mlp.hip -- the warm-start network on gfx950: 4 -> 256 -> 256 -> 256 -> 1792,
// ReLU after the hidden layers.  Weights, biases, inputs and stored
// activations are BF16 (round to nearest even from FP32); products
// accumulate in FP32 on the matrix cores (v_mfma_f32_16x16x32_bf16).  The
// forward pass is one launch, the backward pass one launch per layer.
// Training: backward on the same BF16 operands (output and hidden gradients
// rounded to BF16 before each product), FP32 weight gradients, Adam on an FP32
// master copy.
//
// Parameter vector (element offsets, identical in the BF16 and FP32 copies):
// W1 [256][4], b1 [256], W2 [256][256], b2, W3 [256][256], b3,
// W4 [1792][256], b4 [1792].
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "slpic.h"

namespace slpic_mlp {

constexpr int kIn = SLPIC_MLP_IN, kHid = SLPIC_MLP_HIDDEN, kOut = SLPIC_MLP_OUT;
constexpr int64_t oW1 = 0, ob1 = oW1 + kHid * kIn;
constexpr int64_t oW2 = ob1 + kHid, ob2 = oW2 + kHid * kHid;
constexpr int64_t oW3 = ob2 + kHid, ob3 = oW3 + kHid * kHid;
constexpr int64_t oW4 = ob3 + kHid, ob4 = oW4 + (int64_t)kOut * kHid;
static_assert(ob4 + kOut == SLPIC_MLP_PARAMS, "parameter layout");

using bf16 = uint16_t;
typedef float v4f32 __attribute__((ext_vector_type(4)));

// FP32 -> BF16, round to nearest even (finite values)
__device__ __forceinline__ bf16 to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16)(u >> 16);
}
__device__ __forceinline__ float from_bf16(bf16 h) { return __uint_as_float((uint32_t)h << 16); }

// Orders a wave's LDS accesses (every lane's earlier ones before any later one).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

typedef __bf16 v8bf16 __attribute__((ext_vector_type(8)));
typedef float f32x4a __attribute__((ext_vector_type(4), aligned(4)));  // of caller arrays: FP32 alignment only

// ---------------------------------------------------------------------------
// Forward pass in one launch.  A workgroup of 16 wavefronts takes 16 RT batch
// rows and 256 CB of the 1792 outputs; it computes the three hidden layers of
// its rows itself (with CB = 1 7 workgroups repeat them for one row block; with
// CB = 7 one walks all the outputs, for large batches), wavefront w
// the columns 16 w .. 16 w + 15 of every layer with gfx950's
// v_mfma_f32_16x16x32_bf16 (lane l holds A row l % 16 and B column l % 16 at
// k = 8 (l / 16) + 0..7; the accumulator holds rows 4 (l / 16) + 0..3 of
// column l % 16).  The weights depend on nothing computed here: every
// wavefront loads its fragments (k is contiguous in a weight row) straight
// into registers, two layers ahead; the activations stay in one LDS block.
// What bounds it is the weights' way into a CU, 384 KB per workgroup: loads
// in fragment order, which touch half of 16 cache lines at a time, took 13.9
// us a call at batch 256, whole lines exchanged through LDS 10.0 us, one
// launch per layer 18.2 us.
// The workgroups of column block 0 also store the activations the backward
// pass reads (act, null: not wanted).
// ---------------------------------------------------------------------------
constexpr int kFwdCols = 256, kFwdThreads = 1024;
constexpr int kFwdLdsRow = kHid + 8;  // 528 B: 16-byte aligned rows, 4 banks apart
constexpr int kFrags = kHid / 32;     // k slices of 32
static_assert(kFwdCols == kFwdThreads / 64 * 16 && kHid == kFwdCols && kOut % kFwdCols == 0, "16 columns per wave");

// A wavefront's 16 weight rows (8 KB), as loaded: piece 2 q + h holds the k
// range [64 q, 64 q + 64) of rows 8 h + lane / 8, 16 bytes per lane at 8 (lane %
// 8), so that an instruction reads whole 128-byte lines ...
__device__ __forceinline__ void load_rows(const bf16* __restrict__ W, int row0, int lane, v8bf16 (&f)[kFrags]) {
#pragma unroll
    for (int p = 0; p < kFrags; ++p)
        f[p] = *(const v8bf16*)(W + (int64_t)(row0 + 8 * (p & 1) + (lane >> 3)) * kHid + 64 * (p >> 1) + 8 * (lane & 7));
}
// ... and as the matrix cores want it, fragment k / 32 with lane l holding row
// l % 16 at 8 (l / 16) of the slice: exchanged through 2.25 KB of LDS that
// belong to the wavefront.
constexpr int kXRow = 64 + 8;
__device__ __forceinline__ void to_fragments(bf16 (*X)[kXRow], int lane, v8bf16 (&f)[kFrags]) {
#pragma unroll
    for (int q = 0; q < kFrags / 2; ++q) {
        *(v8bf16*)&X[lane >> 3][8 * (lane & 7)] = f[2 * q];
        *(v8bf16*)&X[8 + (lane >> 3)][8 * (lane & 7)] = f[2 * q + 1];
        wave_sync();
        f[2 * q] = *(const v8bf16*)&X[lane & 15][8 * (lane >> 4)];
        f[2 * q + 1] = *(const v8bf16*)&X[lane & 15][32 + 8 * (lane >> 4)];
        wave_sync();
    }
}
template <int RT>
__device__ __forceinline__ void row_products(const bf16 (*H)[kFwdLdsRow], int i, int kq, const v8bf16 (&f)[kFrags],
                                             v4f32 (&acc)[RT]) {
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = v4f32{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < kFrags; ++k)
#pragma unroll
        for (int t = 0; t < RT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(const v8bf16*)&H[16 * t + i][32 * k + 8 * kq], f[k],
                                                             acc[t], 0, 0, 0);
}

template <int RT, int CB>
__global__ __launch_bounds__(kFwdThreads) void k_forward(const bf16* __restrict__ P, const float* __restrict__ x,
                                                         float* __restrict__ y, int batch, bf16* __restrict__ act) {
    constexpr int kRows = 16 * RT;
    __shared__ __align__(16) bf16 H[kRows][kFwdLdsRow];
    __shared__ __align__(16) bf16 X[kFwdThreads / 64][16][kXRow];
    __shared__ float xs[kRows][kIn];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = lane & 15, kq = lane >> 4;
    constexpr int kGroups = kOut / kFwdCols / CB;  // workgroups of a row block
    static_assert(kGroups * CB * kFwdCols == kOut, "whole column blocks");
    const int b0 = (int)(blockIdx.x / kGroups) * kRows, c0 = (int)(blockIdx.x % kGroups) * CB * kFwdCols;
    const int rows = min(kRows, batch - b0);
    const int n = 16 * w + i;  // this lane's column of every layer
    const int j1 = threadIdx.x & (kHid - 1), r1 = threadIdx.x / kHid;  // layer 1: one column, every fourth row
    bf16* hg = act + (int64_t)batch * kIn;  // the three hidden activations, [batch][256] each
    const bool keep = act && c0 == 0;       // workgroup-uniform
    // a read behind a store of another array would wait for its own round
    // trip: every read of a phase comes before its stores
    const float xv = (int)threadIdx.x < rows * kIn ? x[(int64_t)b0 * kIn + threadIdx.x] : 0.f;
    float w1[kIn];
#pragma unroll
    for (int k = 0; k < kIn; ++k) w1[k] = from_bf16(P[oW1 + j1 * kIn + k]);
    const float bias1 = from_bf16(P[ob1 + j1]);
    v8bf16 f[2][kFrags];
    load_rows(P + oW2, 16 * w, lane, f[0]);
    load_rows(P + oW3, 16 * w, lane, f[1]);
    const float bias[3] = {from_bf16(P[ob2 + n]), from_bf16(P[ob3 + n]), from_bf16(P[ob4 + c0 + n])};
    if ((int)threadIdx.x < kRows * kIn) ((float*)xs)[threadIdx.x] = xv;
    if (keep && (int)threadIdx.x < rows * kIn) act[(int64_t)b0 * kIn + threadIdx.x] = to_bf16(xv);
    __syncthreads();
#pragma unroll
    for (int r = r1; r < kRows; r += kFwdThreads / kHid) {  // layer 1: x -> bf16(x), h1 = bf16(max(x W1^T + b1, 0))
        float acc = 0.f;
#pragma unroll
        for (int k = 0; k < kIn; ++k) acc = fmaf(from_bf16(to_bf16(xs[r][k])), w1[k], acc);
        const bf16 h = to_bf16(fmaxf(acc + bias1, 0.f));
        H[r][j1] = h;
        if (keep && r < rows) hg[(int64_t)(b0 + r) * kHid + j1] = h;
    }
    to_fragments(X[w], lane, f[0]);
    to_fragments(X[w], lane, f[1]);
    v4f32 acc[RT];
#pragma unroll
    for (int l = 0; l < 2; ++l) {  // layers 2 and 3
        __syncthreads();
        row_products<RT>(H, i, kq, f[l], acc);
        if (l == 0) load_rows(P + oW4, c0 + 16 * w, lane, f[0]);
        __syncthreads();
        bf16* ho = hg + (int64_t)(l + 1) * batch * kHid;
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * t + 4 * kq + r;
                const bf16 h = to_bf16(fmaxf(acc[t][r] + bias[l], 0.f));
                H[row][n] = h;
                if (keep && row < rows) ho[(int64_t)(b0 + row) * kHid + n] = h;
            }
    }
    float b4 = bias[2];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {  // the output layer, a column block after the other
        const int c = c0 + cb * kFwdCols;
        float next = 0.f;
        if (cb + 1 < CB) {
            load_rows(P + oW4, c + kFwdCols + 16 * w, lane, f[(cb + 1) & 1]);
            next = from_bf16(P[ob4 + c + kFwdCols + n]);
        }
        to_fragments(X[w], lane, f[cb & 1]);
        if (cb == 0) __syncthreads();
        row_products<RT>(H, i, kq, f[cb & 1], acc);
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * t + 4 * kq + r;
                if (row < rows) y[(int64_t)(b0 + row) * kOut + c + n] = acc[t][r] + b4;
            }
        b4 = next;
    }
}

// ---------------------------------------------------------------------------
// Products of the backward pass: C[m][n] = sum_k A(m, k) B(k, n) with A(m, k)
// = A[m sam + k sak] (BF16, or FP32 rounded to BF16 when read: the output
// gradient) and B(k, n) = B[k ldb + n] (BF16); one of sam, sak is 1, M, N and
// K are multiples of 16.  A workgroup of four wavefronts computes a 32 x 32
// block of C, wavefront w the 16 x 16 tile at rows 16 (w / 2), columns
// 16 (w % 2), with the matrix-core layout above.  Each step of 64 k stages the
// A block [32 m][64 k] and the B block [32 n][64 k] in LDS, k contiguous in
// both, from one 16-byte load per thread and operand along whichever index is
// contiguous in memory; rows past M or N and k past K are zero.  kAhead steps
// of loads are in flight and two LDS buffers alternate, so a step costs one
// barrier and no memory round trip; what bounds the longest product (K = 1792,
// 64 workgroups at batch 256) is then the 2-byte LDS writes of the transposed
// operand, 0.6 us a step.  With the loads waited for in every step it took 25
// us by itself; the output layer's launch, both products, takes 18 us.  Epilogues:
//   masked: out_bf16[m][n] = bf16(h[m][n] > 0 ? acc : 0)
//   grad:   out_f32[m][n]  = acc, and the first column block adds up
//           db[m] = sum_k A(m, k): the bias gradient of the layer
// ---------------------------------------------------------------------------
constexpr int kBlk = 32;            // block tile side (m and n)
constexpr int kKs = 64;             // k per staged step
constexpr int kAhead = 4;           // steps whose loads are in flight (even: two LDS buffers alternate)
constexpr int kLdsRow = kKs + 8;    // padded LDS row (bf16): 144 B, rows start 16 B apart mod 128

struct Gemm {
    const void* A;
    int64_t sam, sak;
    const bf16* B;
    int64_t ldb;
    int M, N, K;
    const bf16* h;  // masked: the activations
    void* out;
    int64_t ldo;
    float* db;  // grad: the bias gradient
    int blocks;  // of C
};

// This thread's eight elements of an operand block (256 threads): rows r of
// the operand are X[(r0 + r) srow + (k0 + k) sk]; FP32 elements are rounded to
// BF16 when they are used, so that nothing waits for the load here.
template <bool F32> struct Oct;
template <> struct Oct<true> {
    f32x4a lo, hi;
    __device__ __forceinline__ void load(const void* X, int64_t at) {
        lo = *(const f32x4a*)((const float*)X + at);
        hi = *(const f32x4a*)((const float*)X + at + 4);
    }
    __device__ __forceinline__ void zero() { lo = hi = f32x4a{0.f, 0.f, 0.f, 0.f}; }
    __device__ __forceinline__ uint4 bits() const {
        union { uint4 v; bf16 e[8]; } u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            u.e[j] = to_bf16(lo[j]);
            u.e[4 + j] = to_bf16(hi[j]);
        }
        return u.v;
    }
};
template <> struct Oct<false> {
    uint4 v;
    __device__ __forceinline__ void load(const void* X, int64_t at) { v = *(const uint4*)((const bf16*)X + at); }
    __device__ __forceinline__ void zero() { v = make_uint4(0u, 0u, 0u, 0u); }
    __device__ __forceinline__ uint4 bits() const { return v; }
};
template <typename O>
__device__ __forceinline__ void fetch_oct(O& o, const void* X, int64_t srow, int64_t sk, int r0, int rows, int k0, int K) {
    const int t = threadIdx.x;
    const int r = sk == 1 ? t >> 3 : (t & 3) * 8, k = sk == 1 ? (t & 7) * 8 : t >> 2;
    if (r0 + r >= rows || k0 + k >= K) o.zero();
    else o.load(X, (int64_t)(r0 + r) * srow + (int64_t)(k0 + k) * sk);
}
__device__ __forceinline__ void put(const uint4& v, bool kcont, bf16 (*L)[kLdsRow]) {
    const int t = threadIdx.x;
    if (kcont) {
        *(uint4*)&L[t >> 3][(t & 7) * 8] = v;
    } else {
        const union { uint4 v; bf16 e[8]; } u{v};
#pragma unroll
        for (int j = 0; j < 8; ++j) L[(t & 3) * 8 + j][t >> 2] = u.e[j];
    }
}

template <bool GRAD, bool AF32>
__device__ __forceinline__ void gemm_block(const Gemm& g, int block, bf16 (*As)[kBlk][kLdsRow],
                                           bf16 (*Bs)[kBlk][kLdsRow]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int bn_count = (g.N + kBlk - 1) / kBlk;
    const int bm = (block / bn_count) * kBlk, bn = (block % bn_count) * kBlk;
    const int i = lane & 15, kq = lane >> 4;
    const int ar = 16 * (w >> 1) + i, bc = 16 * (w & 1) + i;  // this lane's A row and B column in the block
    const bool kc = g.sak == 1, sums = GRAD && bn == 0;
    v4f32 acc = {0.f, 0.f, 0.f, 0.f};
    float rs[8] = {};  // grad: this thread's part of the row sums of A
    Oct<AF32> va[kAhead];
    Oct<false> vb[kAhead];
#pragma unroll
    for (int d = 0; d < kAhead; ++d) {
        fetch_oct(va[d], g.A, g.sam, g.sak, bm, g.M, d * kKs, g.K);
        fetch_oct(vb[d], g.B, 1, g.ldb, bn, g.N, d * kKs, g.K);
    }
    for (int k0 = 0; k0 < g.K; k0 += kAhead * kKs) {
#pragma unroll
        for (int d = 0; d < kAhead; ++d) {  // steps past K multiply zeros
            const int p = d & 1;
            const uint4 a8 = va[d].bits();
            put(a8, kc, As[p]);
            put(vb[d].bits(), false, Bs[p]);
            if (sums) {
                const union { uint4 v; bf16 e[8]; } u{a8};
#pragma unroll
                for (int j = 0; j < 8; ++j) rs[j] += from_bf16(u.e[j]);
            }
            __syncthreads();  // the other buffer's readers passed the barrier before
            fetch_oct(va[d], g.A, g.sam, g.sak, bm, g.M, k0 + (kAhead + d) * kKs, g.K);
            fetch_oct(vb[d], g.B, 1, g.ldb, bn, g.N, k0 + (kAhead + d) * kKs, g.K);
#pragma unroll
            for (int kk = 0; kk < kKs; kk += 32) {
                const v8bf16 a = *(const v8bf16*)&As[p][ar][kk + 8 * kq];
                const v8bf16 b = *(const v8bf16*)&Bs[p][bc][kk + 8 * kq];
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
            }
        }
    }
    if (sums) {  // thread t holds rows 8 (t % 4) + 0..7 at k = t / 4 of every step
        __syncthreads();
        float* R = (float*)As;  // [32][64]
        const int t = threadIdx.x;
#pragma unroll
        for (int j = 0; j < 8; ++j) R[((t & 3) * 8 + j) * 64 + (t >> 2)] = rs[j];
        __syncthreads();
        float v = 0.f;  // eight threads per row, eight values each
#pragma unroll
        for (int j = 0; j < 8; ++j) v += R[(t >> 3) * 64 + (t & 7) + 8 * j];
        for (int o = 4; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((t & 7) == 0 && bm + (t >> 3) < g.M) g.db[bm + (t >> 3)] = v;
    }
    const int col = bn + 16 * (w & 1) + i;
    if (col >= g.N) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = bm + 16 * (w >> 1) + 4 * kq + r;
        if (row >= g.M) continue;
        const int64_t o = (int64_t)row * g.ldo + col;
        if (GRAD) ((float*)g.out)[o] = acc[r];
        else ((bf16*)g.out)[o] = to_bf16(from_bf16(g.h[o]) > 0.f ? acc[r] : 0.f);
    }
}

// A layer's two products, which both need its output gradient D: the input
// gradient (masked) in the first blocks, the weight and bias gradients after
// them.  AF32: D is the caller's FP32 gradient of the output layer.
template <bool AF32>
__global__ __launch_bounds__(256) void k_backward_layer(Gemm masked, Gemm grad) {
    __shared__ __align__(16) bf16 As[2][kBlk][kLdsRow];
    __shared__ __align__(16) bf16 Bs[2][kBlk][kLdsRow];
    static_assert(sizeof As >= 32 * 64 * sizeof(float), "the row sums reuse the A buffers");
    if ((int)blockIdx.x < masked.blocks) gemm_block<false, AF32>(masked, blockIdx.x, As, Bs);
    else gemm_block<true, AF32>(grad, blockIdx.x - masked.blocks, As, Bs);
}

// Layer of fan-out O: D [batch][O] (ldd = O), weights W [O][256], input
// activations h [batch][256]; din = (D W) * (h > 0), dW = D^T h, db.
template <bool AF32>
void backward_layer(const void* D, int O, const bf16* W, const bf16* h, int batch, bf16* din, float* dW, float* db,
                    hipStream_t s) {
    auto blocks = [](int M, int N) { return ((M + kBlk - 1) / kBlk) * ((N + kBlk - 1) / kBlk); };
    const Gemm masked{D, O, 1, W, kHid, batch, kHid, O, h, din, kHid, nullptr, blocks(batch, kHid)};
    const Gemm grad{D, 1, O, h, kHid, O, kHid, batch, nullptr, dW, kHid, db, blocks(O, kHid)};
    hipLaunchKernelGGL(k_backward_layer<AF32>, dim3((unsigned)(masked.blocks + grad.blocks)), dim3(256), 0, s, masked,
                       grad);
}

// First layer: dW1[j][k] = sum_b d1[b][j] x[b][k] (K = 4) and db1[j] = sum_b
// d1[b][j].  A workgroup takes 32 columns j, 32 threads each striding over the
// batch (one thread per gradient walking the whole batch took 65 us at batch
// 256: a chain of 256 reads).
constexpr int kG1Cols = 32, kG1Rows = 32;
__global__ __launch_bounds__(kG1Cols * kG1Rows) void k_grad_layer1(const bf16* __restrict__ d1,
                                                                   const bf16* __restrict__ xr, int batch,
                                                                   float* __restrict__ g) {
    __shared__ float S[kG1Rows][kG1Cols][kIn + 1];
    const int c = threadIdx.x % kG1Cols, r = threadIdx.x / kG1Cols;
    const int j = blockIdx.x * kG1Cols + c;
    float acc[kIn + 1] = {};
    for (int b = r; b < batch; b += kG1Rows) {
        const float d = from_bf16(d1[(int64_t)b * kHid + j]);
#pragma unroll
        for (int k = 0; k < kIn; ++k) acc[k] = fmaf(d, from_bf16(xr[b * kIn + k]), acc[k]);
        acc[kIn] += d;
    }
#pragma unroll
    for (int k = 0; k <= kIn; ++k) S[r][c][k] = acc[k];
    __syncthreads();
    if (threadIdx.x >= kG1Cols * (kIn + 1)) return;
    const int cc = threadIdx.x / (kIn + 1), k = threadIdx.x % (kIn + 1), jj = blockIdx.x * kG1Cols + cc;
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < kG1Rows; ++q) v += S[q][cc][k];
    if (k < kIn) g[oW1 + jj * kIn + k] = v;
    else g[ob1 + jj] = v;
}

__global__ void k_round(const float* __restrict__ in, bf16* __restrict__ out, int64_t n) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) out[t] = to_bf16(in[t]);
}

// Adam: m, v moving averages of g and g^2; p -= lr (m / c1) / (sqrt(v / c2) + eps)
// with the bias corrections c1 = 1 - beta1^t, c2 = 1 - beta2^t.
__global__ void k_adam(float* __restrict__ p, bf16* __restrict__ pb, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, int64_t n, float b1, float b2, float c1, float c2, float lr,
                       float eps) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const float gt = g[t];
    const float mt = b1 * m[t] + (1.f - b1) * gt;
    const float vt = b2 * v[t] + (1.f - b2) * gt * gt;
    m[t] = mt;
    v[t] = vt;
    const float pt = p[t] - lr * (mt / c1) / (sqrtf(vt / c2) + eps);
    p[t] = pt;
    pb[t] = to_bf16(pt);
}

// Mean squared error over n outputs: dy = 2 (y - t) / n, and the loss
// sum (y - t)^2 / n added to *loss (per-block partial sums, one atomic each).
// At most kMseBlocks workgroups stride over the outputs: atomics on one
// address are taken one after another (one workgroup per 256 outputs, 1792
// atomics at batch 256: 25 us).
constexpr int kMseBlocks = 256, kMseUnroll = 4;
__global__ __launch_bounds__(256) void k_mse(const float* __restrict__ y, const float* __restrict__ t,
                                             float* __restrict__ dy, int64_t n, float* __restrict__ loss) {
    __shared__ float part[4];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    float e2 = 0.f;
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < n; i0 += kMseUnroll * stride) {
        float d[kMseUnroll];
#pragma unroll
        for (int q = 0; q < kMseUnroll; ++q) {
            const int64_t i = min(i0 + q * stride, n - 1);
            d[q] = y[i] - t[i];
        }
#pragma unroll
        for (int q = 0; q < kMseUnroll; ++q) {
            const int64_t i = i0 + q * stride;
            if (i >= n) break;
            dy[i] = 2.f * d[q] / (float)n;
            e2 += d[q] * d[q];
        }
    }
    for (int o = 32; o >= 1; o >>= 1) e2 += __shfl_xor(e2, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = e2;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(loss, (part[0] + part[1] + part[2] + part[3]) / (float)n);
}

}  // namespace slpic_mlp

using namespace slpic_mlp;

static int last_error() { return hipGetLastError() == hipSuccess ? SLPIC_OK : SLPIC_EHIP; }

// The forward pass on caller buffers: BF16 inputs and the three hidden
// activations go to act ([batch][4 + 3 * 256] BF16; null: not stored), the
// output to y.
static int forward_impl(const bf16* P, const float* x, float* y, int32_t batch, bf16* act, hipStream_t s) {
    // The variant that repeats the least work among those whose workgroups all
    // fit the chip's 256 CUs at once (one fits a CU): a second round costs as much
    // as the first.  us a call with <rows / 16, output blocks per workgroup> <1, 1>,
    // <2, 1>, <1, 7>, <2, 7>: batch 512 11.2, 13.3, 20.2, 25.3; 1024 19.9, 14.2, 20.7,
    // 26.0; 1184 27.8, 24.1, 20.9, 26.0; 4096 62.0, 46.1, 23.6, 28.3; 8192 122, 80,
    // 41.9, 29.7; 16384 242, 157, 80, 53 (a launch per layer 19.6, 22.4, 24.5, 41.8,
    // 66.8, 120)
    constexpr int kCus = 256, kBlocks = kOut / kFwdCols;
    auto rows = [&](int rt) { return (batch + 16 * rt - 1) / (16 * rt); };
    auto launch = [&](auto kernel, int groups) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3(kFwdThreads), 0, s, P, x, y, batch, act);
    };
    if ((int64_t)rows(1) * kBlocks <= kCus) launch(k_forward<1, 1>, rows(1) * kBlocks);
    else if ((int64_t)rows(2) * kBlocks <= kCus) launch(k_forward<2, 1>, rows(2) * kBlocks);
    else if (rows(1) <= kCus) launch(k_forward<1, kBlocks>, rows(1));
    else launch(k_forward<2, kBlocks>, rows(2));
    return last_error();
}

extern "C" {

size_t slpic_mlp_act_bytes(int32_t batch) {
    return batch > 0 ? (size_t)batch * (kIn + 3 * kHid) * sizeof(bf16) : 0;
}
size_t slpic_mlp_work_bytes(int32_t batch) {
    return batch > 0 ? (size_t)batch * 3 * kHid * sizeof(bf16) : 0;
}

int slpic_mlp_to_bf16(const float* d_params_fp32, void* d_params_bf16, void* stream) {
    if (!d_params_fp32 || !d_params_bf16) return SLPIC_EINVAL;
    const int64_t n = SLPIC_MLP_PARAMS;
    hipLaunchKernelGGL(k_round, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, d_params_fp32,
                       (bf16*)d_params_bf16, n);
    return last_error();
}

int slpic_mlp_forward(const void* d_params_bf16, const float* d_x, float* d_y, int32_t batch, void* d_act,
                      void* stream) {
    if (!d_params_bf16 || !d_x || !d_y || !d_act || batch <= 0 || batch % 16) return SLPIC_EINVAL;
    return forward_impl((const bf16*)d_params_bf16, d_x, d_y, batch, (bf16*)d_act, (hipStream_t)stream);
}

int slpic_mlp_forward_noalloc(const void* d_params_bf16, const float* d_x, float* d_y, int32_t batch,
                              void* stream) {
    if (!d_params_bf16 || !d_x || !d_y || batch <= 0 || batch % 16) return SLPIC_EINVAL;
    if (batch > SLPIC_MLP_NOALLOC_MAX_BATCH) return SLPIC_ELIMIT;
    return forward_impl((const bf16*)d_params_bf16, d_x, d_y, batch, nullptr, (hipStream_t)stream);
}

int slpic_mlp_backward(const void* d_params_bf16, const void* d_act, const float* d_dy, float* d_grads,
                       int32_t batch, void* d_work, void* stream) {
    if (!d_params_bf16 || !d_act || !d_dy || !d_grads || !d_work || batch <= 0 || batch % 16) return SLPIC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    const bf16* P = (const bf16*)d_params_bf16;
    const bf16* xr = (const bf16*)d_act;
    const bf16* h1 = xr + (int64_t)batch * kIn;
    const bf16* h2 = h1 + (int64_t)batch * kHid;
    const bf16* h3 = h2 + (int64_t)batch * kHid;
    bf16* d3 = (bf16*)d_work;
    bf16* d2 = d3 + (int64_t)batch * kHid;
    bf16* d1 = d2 + (int64_t)batch * kHid;
    float* g = d_grads;
    backward_layer<true>(d_dy, kOut, P + oW4, h3, batch, d3, g + oW4, g + ob4, s);
    backward_layer<false>(d3, kHid, P + oW3, h2, batch, d2, g + oW3, g + ob3, s);
    backward_layer<false>(d2, kHid, P + oW2, h1, batch, d1, g + oW2, g + ob2, s);
    hipLaunchKernelGGL(k_grad_layer1, dim3(kHid / kG1Cols), dim3(kG1Cols * kG1Rows), 0, s, d1, xr, batch, g);
    return last_error();
}

int slpic_mlp_mse(const float* d_y, const float* d_t, float* d_dy, int64_t n, float* d_loss, void* stream) {
    if (!d_y || !d_t || !d_dy || !d_loss || n <= 0) return SLPIC_EINVAL;
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_mse, dim3((unsigned)(blocks < kMseBlocks ? blocks : kMseBlocks)), dim3(256), 0,
                       (hipStream_t)stream, d_y, d_t, d_dy, n, d_loss);
    return last_error();
}

int slpic_mlp_adam(float* d_params_fp32, void* d_params_bf16, float* d_m, float* d_v, const float* d_grads,
                   float lr, float beta1, float beta2, float eps, int32_t step, void* stream) {
    if (!d_params_fp32 || !d_params_bf16 || !d_m || !d_v || !d_grads || step < 1) return SLPIC_EINVAL;
    const int64_t n = SLPIC_MLP_PARAMS;
    const double c1 = 1.0 - std::pow((double)beta1, step), c2 = 1.0 - std::pow((double)beta2, step);
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, d_params_fp32,
                       (bf16*)d_params_bf16, d_m, d_v, d_grads, n, beta1, beta2, (float)c1, (float)c2, lr, eps);
    return last_error();
}

}  // extern "C"
