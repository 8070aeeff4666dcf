// Kernels of the learned initial-particle proposal: a point-set network that
// maps a (source, reference) cloud pair to K pose particles which then seed
// Stein ICP in place of the uniform draw of the particles (Sec. V).
//
// Network: a shared per-point MLP 3 -> 64 -> 128 -> 256 (ReLU after each
// layer) runs on every point of both clouds; each cloud is max-pooled to a
// 256-vector; the two vectors are concatenated (source first) and mapped by
// 512 -> 256 (ReLU) -> 6K, read as K row-major particles (x, y, z, roll,
// pitch, yaw).
//
// Precision: every matrix product rounds both operands to BF16 (round to
// nearest even) as it stages them into LDS and accumulates in FP32 on the
// matrix cores; master weights, activations, gradients and Adam moments are
// FP32; the set loss is evaluated in FP64.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sicp {
namespace prop {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint16_t u16x8_t __attribute__((ext_vector_type(8)));

// FP32 -> BF16 bits, round to nearest even; infinities and NaNs keep their
// class (a NaN stays a NaN). One instruction per two values (gfx950's
// v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint16_t to_bf16(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

// ------------------------------------------------------------------- GEMM
// C = op(A) op(B) [+ bias] [ReLU] [+ C]   (M x N, FP32, row-major, ldc)
// and, with `gate` (M x N, as C), zero where gate is not > 0: the backward of
// the ReLU that produced it (a pass of its own took 1.8 to 5.7 us)
//   op(A) = A   with A row-major M x K (lda)   when ta == 0,
//         = A^T with A row-major K x M (lda)   when ta == 1;
//   op(B) = B   with B row-major K x N (ldb)   when tb == 0,
//         = B^T with B row-major N x K (ldb)   when tb == 1.
// Split K: slice z covers K range [z kper, (z + 1) kper) and writes its
// partial product, without bias, ReLU or accumulation, to C + z c_split
// (the caller then sums the splits with splitk_reduce_kernel).
// Pooled epilogue (pool_keys != nullptr, one K slice, ReLU on, rows in
// clouds of pool_P points with pool_P % 64 == 0 so that a 64-row tile lies
// in one cloud): C is not written; instead the maximum of every column over
// each cloud's rows, with its first row, is folded into
// pool_keys[cloud N + n] as the key (value bits << 32) | ~row_in_cloud
// (values are >= +0, whose bit patterns order like the values; a larger key
// is a larger value, or the same value at a smaller row).
struct GemmArgs {
    const float* A;
    const float* B;
    float* C;
    const float* bias;
    const float* gate;
    int64_t M, N, K, lda, ldb, ldc;
    int64_t kper, c_split;
    int32_t ta, tb, relu, accumulate, by_slice, splits;
    unsigned long long* pool_keys;
    int64_t pool_P;
};

constexpr int kGT = 64;    // output tile edge
constexpr int kGK = 32;    // K step (one MFMA 16x16x32 deep)
constexpr int kLdsPad = 8; // BF16 pad per LDS row: spreads banks, keeps 16-byte rows aligned

constexpr int kXcds = 8;   // workgroups are dealt to the 8 XCDs round robin

// Tile and K slice of workgroup (b, z): workgroups b, b + 8, b + 16, ... land on
// the same XCD, and are given what shares operand rows: the Nt column tiles of
// one row tile (ceil(Mt / 8) * 8 * Nt x splits workgroups; Mt, Nt: row and
// column tiles), or by_slice all tiles of one K slice (ceil(splits / 8) * 8 Mt
// Nt workgroups). The second is for eight slices and more of fewer than eight
// row tiles, which by rows would leave the other XCDs idle: the 128 x 256 weight
// gradient over 16,384 rows (two row tiles, 64 slices) takes 12.4 us, 28.4 by
// rows. Fewer slices of few row tiles stay on one XCD: spread over all, the
// head's products and their sums took 1 us more (64 pairs 84.3 us a forward
// pass, 83.3 so).
__device__ __forceinline__ bool gemm_tile(int32_t by_slice, int64_t b, int64_t splits, int64_t Mt, int64_t Nt,
                                          int64_t& mt, int64_t& nt, int64_t& z)
{
    if (by_slice) {
        const int64_t tile = b / kXcds % (Mt * Nt);
        z = b / (kXcds * Mt * Nt) * kXcds + b % kXcds;
        mt = tile / Nt;
        nt = tile % Nt;
        return z < splits;
    }
    const int64_t grp = b / (kXcds * Nt), r = b % (kXcds * Nt);
    mt = grp * kXcds + r % kXcds;
    nt = r / kXcds;
    return mt < Mt;
}

// Eight consecutive k of one row (or column) of an operand tile, zero outside
// the matrix. kc: k is the contiguous dimension of global memory (two 16-byte
// loads where `vec`, the whole operand's rows are aligned to 16 bytes), else
// rows are (a load takes the same k of 64 consecutive rows).
__device__ __forceinline__ void gemm_load(const float* __restrict__ A, bool kc, bool vec, int64_t ld, int64_t row,
                                          bool in, int64_t k, int64_t kend, float (&v)[8])
{
    if (in && k + 8 <= kend) {
        if (kc && vec) {
            const float4 x = *reinterpret_cast<const float4*>(A + row * ld + k);
            const float4 y = *reinterpret_cast<const float4*>(A + row * ld + k + 4);
            v[0] = x.x;
            v[1] = x.y;
            v[2] = x.z;
            v[3] = x.w;
            v[4] = y.x;
            v[5] = y.y;
            v[6] = y.z;
            v[7] = y.w;
        } else {
            const float* a = A + (kc ? row * ld + k : k * ld + row);
            const int64_t st = kc ? 1 : ld;
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = a[u * st];
        }
        return;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = in && k + u < kend ? A[kc ? row * ld + k + u : (k + u) * ld + row] : 0.f;
}

// 256 threads, 64 x 64 output tile; wavefront w owns the 32 x 32 quarter
// (w / 2, w % 2) as 2 x 2 MFMA tiles. Both LDS tiles are K-contiguous
// ([row][k] and [col][k]), so a lane reads the eight K values of its
// fragment (row lane % 16, K slice 8 (lane / 16)) in one 16-byte load, and a
// thread stages the eight K values of one row of each operand in one 16-byte
// store. The next step's values are loaded while this one is multiplied, into
// the other of two LDS tiles. Bound by load latency and launch at this model's
// sizes: the thirteen products of a training step at batch 32 average 8.6 us
// (36 with a 2-byte store per element and the loads between two barriers).
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmArgs g)
{
    __shared__ __attribute__((aligned(16))) uint16_t As[2][kGT][kGK + kLdsPad];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][kGT][kGK + kLdsPad];
    int64_t mt, nt;
    int64_t z = blockIdx.z;
    if (!gemm_tile(g.by_slice, blockIdx.x, g.splits, (g.M + kGT - 1) / kGT, (g.N + kGT - 1) / kGT, mt, nt, z))
        return;   // whole workgroup
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t m0 = mt * kGT, n0 = nt * kGT;
    const int64_t kbeg = z * g.kper;
    const int64_t kend = min(g.K, kbeg + g.kper);
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    f32x4_t acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

    // this thread's row of each operand tile and its eight k of a step: the
    // threads of a wavefront run along the contiguous dimension
    const bool akc = !g.ta, bkc = g.tb != 0;
    const int ar = akc ? tid / 4 : tid % 64, ak = 8 * (akc ? tid % 4 : tid / 64);
    const int br = bkc ? tid / 4 : tid % 64, bk = 8 * (bkc ? tid % 4 : tid / 64);
    const bool av = ((uintptr_t)g.A & 15) == 0 && g.lda % 4 == 0, bv = ((uintptr_t)g.B & 15) == 0 && g.ldb % 4 == 0;
    const bool ain = m0 + ar < g.M, bin = n0 + br < g.N;
    float va[8], vb[8];
    auto load = [&](int64_t k0) {
        gemm_load(g.A, akc, av, g.lda, m0 + ar, ain, k0 + ak, kend, va);
        gemm_load(g.B, bkc, bv, g.ldb, n0 + br, bin, k0 + bk, kend, vb);
    };
    if (kbeg < kend) load(kbeg);
    int cur = 0;
    for (int64_t k0 = kbeg; k0 < kend; k0 += kGK, cur ^= 1) {
        u16x8_t ha, hb;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            ha[u] = to_bf16(va[u]);
            hb[u] = to_bf16(vb[u]);
        }
        *reinterpret_cast<u16x8_t*>(&As[cur][ar][ak]) = ha;
        *reinterpret_cast<u16x8_t*>(&Bs[cur][br][bk]) = hb;
        if (k0 + kGK < kend) load(k0 + kGK);
        __syncthreads();
        const int fr = lane & 15, fk = 8 * (lane >> 4);
        bf16x8_t af[2], bfr[2];
#pragma unroll
        for (int a = 0; a < 2; ++a)
            af[a] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u16x8_t*>(&As[cur][wm + 16 * a + fr][fk]));
#pragma unroll
        for (int b = 0; b < 2; ++b)
            bfr[b] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u16x8_t*>(&Bs[cur][wn + 16 * b + fr][fk]));
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a], bfr[b], acc[a][b], 0, 0, 0);
        // the other tile is written next: its readers have passed this step's barrier
    }
    // lane holds column lane % 16 and rows 4 (lane / 16) .. +3 of each tile
    if (g.pool_keys) {
        const int64_t cloud = m0 / g.pool_P;
        const int64_t rbase = m0 - cloud * g.pool_P + wm;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int64_t gn = n0 + wn + 16 * b + (lane & 15);
            const float bias = (g.bias && gn < g.N) ? g.bias[gn] : 0.f;
            unsigned long long best = 0ull;
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float v = acc[a][b][t] + bias;
                    const float r = v > 0.f ? v : 0.f;   // ReLU, canonical +0
                    const uint32_t row = (uint32_t)(rbase + 16 * a + 4 * (lane >> 4) + t);
                    const unsigned long long key =
                        ((unsigned long long)__float_as_uint(r) << 32) | (unsigned long long)(~row);
                    best = key > best ? key : best;
                }
            // the four lanes of a column hold rows 4 (lane / 16) .. +3 of the wavefront's 32
            unsigned long long o = __shfl_xor(best, 16);
            best = o > best ? o : best;
            o = __shfl_xor(best, 32);
            best = o > best ? o : best;
            if (lane < 16 && gn < g.N) atomicMax(g.pool_keys + cloud * g.N + gn, best);
        }
        return;
    }
    float* Cz = g.C + z * g.c_split;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int64_t gm = m0 + wm + 16 * a + 4 * (lane >> 4) + t;
                const int64_t gn = n0 + wn + 16 * b + (lane & 15);
                if (gm < g.M && gn < g.N) {
                    float v = acc[a][b][t];
                    if (g.bias) v += g.bias[gn];
                    if (g.relu) v = fmaxf(v, 0.f);
                    if (g.gate && !(g.gate[gm * g.ldc + gn] > 0.f)) v = 0.f;
                    float* dst = Cz + gm * g.ldc + gn;
                    *dst = g.accumulate ? *dst + v : v;
                }
            }
}

// -------------------------------------------------- fused per-point MLP
// The three per-point layers and the max-pool of one 64-point tile in one
// workgroup: h1 = relu(x W1 + b1), h2 = relu(h1 W2 + b2), h3 = relu(h2 W3 +
// b3), folded into the pool keys as in the pooled GEMM epilogue. Every
// product is a chain of v_mfma_f32_16x16x32_bf16 over K steps of 32 in
// increasing order, from zero, with the bias added to the FP32 sum and ReLU
// after it -- the arithmetic of gemm_bf16_kernel, so a row recomputed by
// that kernel has the same bits. Activations pass between the layers through
// LDS as BF16 and never reach HBM. The weights are staged once per workgroup
// as BF16, column-major with padded rows (the B-operand layout of the GEMM).
// Bound by the vector instructions between the matrix ones (activations and
// pooling): 524,288 points (64 pairs) take 64 us, 0.70 PFLOP/s, 8,192 points
// 9.2 us, against 129 and 22.6 with the conversion in integer steps, 2-byte
// activation stores and a 64-bit key maximum over every output of every tile.
struct MlpArgs {
    const float* X;   // rows x 3
    const float *W1, *b1, *W2, *b2, *W3, *b3;
    unsigned long long* keys;   // clouds x 256
    int64_t rows, P;            // P % 64 == 0
};

constexpr int kMT = 64;                 // points per tile
constexpr int kLd1 = 32 + kLdsPad;      // K stride of x and W1 (K = 3 padded to 32)
constexpr int kLd2 = 64 + kLdsPad;      // K stride of h1 and W2
constexpr int kLd3 = 128 + kLdsPad;     // K stride of h2 and W3
// LDS layout in BF16 elements
constexpr int kOffW1 = 0;
constexpr int kOffW2 = kOffW1 + 64 * kLd1;
constexpr int kOffW3 = kOffW2 + 128 * kLd2;
constexpr int kOffU = kOffW3 + 256 * kLd3;   // h2 tile (one per tile in flight, as the next two)
constexpr int kOffH1 = kOffU + 2 * kMT * kLd3;
constexpr int kOffX = kOffH1 + 2 * kMT * kLd2;   // x tile
constexpr int kMlpLdsElems = kOffX + 2 * kMT * kLd1;
constexpr int kMlpThreads = 512;              // two tiles at a time, four wavefronts each
constexpr size_t kMlpLdsBytes = 2 * (size_t)kMlpLdsElems;

__device__ __forceinline__ bf16x8_t lds_frag(const uint16_t* base, int row, int ld, int k)
{
    return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u16x8_t*>(base + row * ld + k));
}

// Four outputs of a layer that passes its activations on: bias, ReLU, BF16.
__device__ __forceinline__ void store_act(uint16_t* dst, f32x4_t acc, const float4 bias)
{
    const float b[4] = {bias.x, bias.y, bias.z, bias.w};
    ushort4 h;
    h.x = to_bf16(fmaxf(acc[0] + b[0], 0.f));
    h.y = to_bf16(fmaxf(acc[1] + b[1], 0.f));
    h.z = to_bf16(fmaxf(acc[2] + b[2], 0.f));
    h.w = to_bf16(fmaxf(acc[3] + b[3], 0.f));
    *reinterpret_cast<ushort4*>(dst) = h;
}

__global__ __launch_bounds__(kMlpThreads) void mlp_pool_kernel(MlpArgs g)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t sm16[];
    uint16_t* W1s = sm16 + kOffW1;
    uint16_t* W2s = sm16 + kOffW2;
    uint16_t* W3s = sm16 + kOffW3;
    const int half = threadIdx.x >> 8;           // which of the two tiles in flight
    const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;
    uint16_t* U = sm16 + kOffU + half * kMT * kLd3;
    uint16_t* H1s = sm16 + kOffH1 + half * kMT * kLd2;
    uint16_t* Xs = sm16 + kOffX + half * kMT * kLd1;
    const int fr = lane & 15, fk = 8 * (lane >> 4), f4 = 4 * (lane >> 4);
    // weights, transposed to [column][k] BF16: a thread takes eight k of one
    // column (its loads run along the rows with its neighbours')
    for (int e = threadIdx.x; e < 64 * 32; e += kMlpThreads) {
        const int n = e % 64, k = e / 64;
        W1s[n * kLd1 + k] = to_bf16(k < 3 ? g.W1[k * 64 + n] : 0.f);
    }
    auto stage = [&](const float* __restrict__ W, int N, int K, uint16_t* dst, int ld) {
        for (int e = threadIdx.x; e < N * K / 8; e += kMlpThreads) {
            const int n = e % N, k = e / N * 8;
            u16x8_t v;
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = to_bf16(W[(k + u) * N + n]);
            *reinterpret_cast<u16x8_t*>(dst + n * ld + k) = v;
        }
    };
    stage(g.W2, 128, 64, W2s, kLd2);
    stage(g.W3, 256, 128, W3s, kLd3);
    const int64_t ntiles = g.rows / kMT;
    // each workgroup takes a run of consecutive tiles, so of few clouds; its
    // halves take them in turn. The loop count is the same for all threads
    // (the barriers are workgroup-wide) and a half without a tile skips the
    // work. The tile's 64 x 3 inputs, one value per thread below 192, are
    // loaded a round ahead.
    const int64_t first = ntiles * blockIdx.x / gridDim.x, last = ntiles * (blockIdx.x + 1) / gridDim.x;
    int64_t base = first;
    float xv = (base + half < last && tid < 3 * kMT) ? g.X[(base + half) * kMT * 3 + tid] : 0.f;
    // this lane's largest value and its first row, of the columns
    // 16 (4 wave + c) + fr, since the cloud's first tile here
    float best[4];
    uint32_t brow[4];
    int64_t cloud = -1;
    auto flush = [&] {   // fold the cloud's maxima into its keys
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            unsigned long long key =
                ((unsigned long long)__float_as_uint(best[c]) << 32) | (unsigned long long)(~brow[c]);
            unsigned long long o = __shfl_xor(key, 16);
            key = o > key ? o : key;
            o = __shfl_xor(key, 32);
            key = o > key ? o : key;
            if (lane < 16) atomicMax(g.keys + cloud * 256 + 16 * (4 * wave + c) + fr, key);
        }
    };
    const float4 bias1 = *reinterpret_cast<const float4*>(g.b1 + 16 * wave + f4);
    const float4 bias2[2] = {*reinterpret_cast<const float4*>(g.b2 + 32 * wave + f4),
                             *reinterpret_cast<const float4*>(g.b2 + 32 * wave + 16 + f4)};
    float bias3[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) bias3[c] = g.b3[16 * (4 * wave + c) + fr];
    for (int e = tid; e < kMT * 32; e += 256)   // the inputs, zero past their three columns
        if (e % 32 >= 3) Xs[e / 32 * kLd1 + e % 32] = 0;
    if (tid < 3 * kMT) Xs[(tid / 3) * kLd1 + tid % 3] = to_bf16(xv);
    for (; base < last; base += 2) {
        const int64_t tile = base + half;
        const bool live = tile < last;
        const int64_t m0 = tile * kMT;
        const int64_t next = tile + 2;
        if (next < last && tid < 3 * kMT) xv = g.X[next * kMT * 3 + tid];
        __syncthreads();   // the inputs (and, before the first tile, the weights) are staged
        // layers 1 and 2 with the operands exchanged (the same products and
        // sums): a lane holds four consecutive features of a point, one
        // 8-byte LDS store. Layer 1: wavefront w owns features 16 w .. + 15
        {
            const bf16x8_t b = lds_frag(W1s, 16 * wave + fr, kLd1, fk);
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) {
                f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, lds_frag(Xs, 16 * rb + fr, kLd1, fk), acc, 0, 0, 0);
                store_act(H1s + (16 * rb + fr) * kLd2 + 16 * wave + f4, acc, bias1);
            }
        }
        __syncthreads();
        // layer 2: wavefront w owns features 32 w .. + 31
        {
            f32x4_t acc[4][2];
#pragma unroll
            for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                for (int c = 0; c < 2; ++c) acc[rb][c] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                bf16x8_t a[4], b[2];
#pragma unroll
                for (int rb = 0; rb < 4; ++rb) a[rb] = lds_frag(H1s, 16 * rb + fr, kLd2, 32 * ks + fk);
#pragma unroll
                for (int c = 0; c < 2; ++c) b[c] = lds_frag(W2s, 16 * (2 * wave + c) + fr, kLd2, 32 * ks + fk);
#pragma unroll
                for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        acc[rb][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[c], a[rb], acc[rb][c], 0, 0, 0);
            }
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int rb = 0; rb < 4; ++rb)
                    store_act(U + (16 * rb + fr) * kLd3 + 16 * (2 * wave + c) + f4, acc[rb][c], bias2[c]);
        }
        __syncthreads();
        // layer 3: wavefront w owns column blocks 4w .. 4w + 3; the columns'
        // maxima over the run's tiles of a cloud stay in registers
        {
            f32x4_t acc[4][4];
#pragma unroll
            for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[rb][c] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                bf16x8_t a[4], b[4];
#pragma unroll
                for (int rb = 0; rb < 4; ++rb) a[rb] = lds_frag(U, 16 * rb + fr, kLd3, 32 * ks + fk);
#pragma unroll
                for (int c = 0; c < 4; ++c) b[c] = lds_frag(W3s, 16 * (4 * wave + c) + fr, kLd3, 32 * ks + fk);
#pragma unroll
                for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        acc[rb][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rb], b[c], acc[rb][c], 0, 0, 0);
            }
            const int64_t here = m0 / g.P;
            const uint32_t row0 = (uint32_t)(m0 - here * g.P) + f4;
            if (live) {
                if (here != cloud) {   // the same for the whole half
                    if (cloud >= 0) flush();
                    cloud = here;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        best[c] = 0.f;   // ReLU: no value is below
                        brow[c] = row0;
                    }
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float m = 0.f;
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            acc[rb][c][t] += bias3[c];
                            m = fmaxf(m, acc[rb][c][t]);
                        }
                    if (m > best[c]) {   // rows ascend: a later tile's equal value is not the first
                        best[c] = m;
                        uint32_t r = 0;
#pragma unroll
                        for (int rb = 3; rb >= 0; --rb)
#pragma unroll
                            for (int t = 3; t >= 0; --t)
                                if (acc[rb][c][t] == m) r = 16 * rb + t;
                        brow[c] = row0 + r;
                    }
                }
            }
        }
        // every wavefront has left layer 1: the next inputs may follow. The
        // second layer's tile is next written after two more barriers
        if (tid < 3 * kMT) Xs[(tid / 3) * kLd1 + tid % 3] = to_bf16(xv);
    }
    if (cloud >= 0) flush();
}

// C[m][n] (+)= sum_{z < S} W[z][m][n] (+ bias[n]) (ReLU) (gate), z in order.
__global__ void splitk_reduce_kernel(const float* __restrict__ W, int32_t S, int64_t M, int64_t N,
                                     float* __restrict__ C, int64_t ldc, const float* __restrict__ bias,
                                     const float* __restrict__ gate, int32_t relu, int32_t accumulate)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M * N) return;
    const int64_t m = i / N, n = i % N;
    float s = 0.f;
#pragma unroll 16   // loads in flight; the sum keeps its order
    for (int32_t z = 0; z < S; ++z) s += W[(int64_t)z * M * N + i];
    if (bias) s += bias[n];
    if (relu) s = fmaxf(s, 0.f);
    if (gate && !(gate[m * ldc + n] > 0.f)) s = 0.f;
    float* dst = C + m * ldc + n;
    *dst = accumulate ? *dst + s : s;
}

// --------------------------------------------------------------- max-pool
// H holds `clouds` clouds of P points, F features each: row c P + p.
// Stage 1, grid (clouds, chunks): maximum and its first index over the
// chunk's points, per feature.
__global__ void maxpool_partial_kernel(const float* __restrict__ H, int64_t P, int64_t F, int64_t chunk,
                                       float* __restrict__ pv, int32_t* __restrict__ pi)
{
    const int64_t c = blockIdx.x, ch = blockIdx.y, nch = gridDim.y;
    const int64_t p0 = ch * chunk, p1 = min(P, p0 + chunk);
    for (int64_t f = threadIdx.x; f < F; f += blockDim.x) {
        float best = -__builtin_inff();
        int32_t bi = (int32_t)p0;
        for (int64_t p = p0; p < p1; ++p) {
            const float v = H[(c * P + p) * F + f];
            if (v > best) {
                best = v;
                bi = (int32_t)p;
            }
        }
        pv[(c * nch + ch) * F + f] = best;
        pi[(c * nch + ch) * F + f] = bi;
    }
}

// Stage 2, one thread per (cloud, feature): merge the chunks in order (the
// first maximum wins). Pair layout: clouds 2b (source) and 2b + 1
// (reference) fill columns [0, F) and [F, 2F) of row b of `out`.
__global__ void maxpool_merge_kernel(const float* __restrict__ pv, const int32_t* __restrict__ pi, int64_t clouds,
                                     int64_t nch, int64_t F, float* __restrict__ out, int64_t ld_out,
                                     int32_t* __restrict__ arg)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= clouds * F) return;
    const int64_t c = i / F, f = i % F;
    float best = pv[(c * nch) * F + f];
    int32_t bi = pi[(c * nch) * F + f];
    for (int64_t ch = 1; ch < nch; ++ch) {
        const float v = pv[(c * nch + ch) * F + f];
        if (v > best) {
            best = v;
            bi = pi[(c * nch + ch) * F + f];
        }
    }
    out[(c / 2) * ld_out + (c % 2) * F + f] = best;
    arg[i] = bi;
}

// Keys of the pooled epilogue to the pooled features (pair layout as in
// maxpool_merge_kernel) and the winning rows. One thread per (cloud, feature).
__global__ void pool_keys_finish_kernel(const unsigned long long* __restrict__ keys, int64_t clouds, int64_t F,
                                        float* __restrict__ out, int64_t ld_out, int32_t* __restrict__ arg)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= clouds * F) return;
    const int64_t c = i / F, f = i % F;
    const unsigned long long k = keys[i];
    out[(c / 2) * ld_out + (c % 2) * F + f] = __uint_as_float((uint32_t)(k >> 32));
    arg[i] = (int32_t)(~(uint32_t)k);
}

// Below the max-pool only the points that won a pooled feature receive
// gradient. winner_rows_kernel gives each cloud F3 rows: its distinct
// winning points first (in order of the first feature each wins), then zero
// rows. Row u holds the point's input (G0) and the pooled gradients of the
// features it wins (dA3[u][f] = dF[c][f] where F[c][f] > 0, else 0): the
// dense backward's nonzero rows, so every product below is the dense chain
// rule's product restricted to them (zero rows add exact zeros).
// grid: (clouds, kWinnerParts): the workgroups of a cloud number its winners
// alike and write a share of the rows each. F3 threads: one per feature to
// number, then four features of one row per 16-byte store (every element is
// written once, value or zero). Bound by its stores, 16 MB at 32 pairs: 11.6 us
// there; 33.5 with one workgroup a cloud, 4-byte stores and a serial search
// for the first feature.
constexpr int kWinnerParts = 4;

template <int F3>
__global__ __launch_bounds__(F3) void winner_rows_kernel(const float* __restrict__ X, const int32_t* __restrict__ arg,
                                                         const float* __restrict__ F, const float* __restrict__ dF,
                                                         int64_t ld_f, int64_t P, float* __restrict__ G0,
                                                         float* __restrict__ dA3)
{
    constexpr int kW = 64;   // wavefront width
    constexpr int kRows = F3 / kWinnerParts, kQuads = F3 / 4;
    static_assert(F3 % kW == 0 && kRows % 4 == 0, "one thread per feature, whole wavefronts; four rows a pass");
    __shared__ __attribute__((aligned(16))) int32_t pt[F3];
    __shared__ __attribute__((aligned(16))) int32_t row[F3];
    __shared__ __attribute__((aligned(16))) float val[F3];
    __shared__ int32_t wtot[F3 / kW];
    const int64_t c = blockIdx.x;
    const int f = threadIdx.x, lane = f % kW, wv = f / kW;
    const int32_t p = min(max(arg[c * F3 + f], 0), (int32_t)(P - 1));   // arg is in range; clamp anyway
    pt[f] = p;
    const int64_t e = (c / 2) * ld_f + (c % 2) * F3 + f;
    val[f] = F[e] > 0.f ? dF[e] : 0.f;
    __syncthreads();
    int first = f;   // first feature won by the same point
#pragma unroll 8
    for (int j = kQuads - 1; j >= 0; --j) {
        const int4 q = reinterpret_cast<const int4*>(pt)[j];
        first = q.w == p ? 4 * j + 3 : first;
        first = q.z == p ? 4 * j + 2 : first;
        first = q.y == p ? 4 * j + 1 : first;
        first = q.x == p ? 4 * j : first;
    }
    const bool owner = first == f;
    const unsigned long long ob = __ballot(owner);
    if (lane == 0) wtot[wv] = __popcll(ob);
    __syncthreads();
    int r = __popcll(ob & ((1ull << lane) - 1ull)), rows = 0;
    for (int w = 0; w < F3 / kW; ++w) {
        r += w < wv ? wtot[w] : 0;
        rows += wtot[w];
    }
    if (owner) row[f] = r;
    __syncthreads();
    const int mine = row[first];
    __syncthreads();
    row[f] = mine;   // the row of every feature, not of the owners only
    const int r0 = (int)blockIdx.y * kRows, r1 = r0 + kRows;
    float* __restrict__ Gc = G0 + c * F3 * 3;
    if (owner && r >= r0 && r < r1) {
        const float* x = X + (c * P + p) * 3;
        Gc[3 * r] = x[0];
        Gc[3 * r + 1] = x[1];
        Gc[3 * r + 2] = x[2];
    }
    if (f >= rows && f >= r0 && f < r1) Gc[3 * f] = Gc[3 * f + 1] = Gc[3 * f + 2] = 0.f;
    __syncthreads();
    const int q = f % kQuads;
    const int4 rq = reinterpret_cast<const int4*>(row)[q];
    const float4 vq = reinterpret_cast<const float4*>(val)[q];
    float4* __restrict__ Dc = reinterpret_cast<float4*>(dA3 + c * F3 * F3);
    for (int u = r0 + f / kQuads; u < r1; u += 4)
        Dc[u * kQuads + q] = make_float4(rq.x == u ? vq.x : 0.f, rq.y == u ? vq.y : 0.f, rq.z == u ? vq.z : 0.f,
                                         rq.w == u ? vq.w : 0.f);
}

// ------------------------------------------------------------ elementwise
__global__ void fill_f32_kernel(float* __restrict__ x, int64_t n, float v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = v;
}

// Column sums of several matrices X (rows x N) in two launches of fixed-order
// stages: partial sums over row chunks, then over chunks. A workgroup takes
// 256 columns of one chunk; it finds its matrix by the first workgroups of
// each (a launch of either stage per matrix, ten a training step, took 3 us
// each; the two take 13.5 together at 32 pairs).
constexpr int kColMats = 5;
struct ColSums {
    const float* X[kColMats];
    float* out[kColMats];
    float* part[kColMats];
    int64_t rows[kColMats], N[kColMats];
    uint32_t first[kColMats];    // first workgroup of the partial sums
    uint32_t mfirst[kColMats];   // and of the merge
    int64_t chunk;
    int32_t n;
};

__global__ void colsum_partial_kernel(ColSums a)
{
    int i = a.n - 1;
    while (i > 0 && blockIdx.x < a.first[i]) --i;
    const float* __restrict__ X = a.X[i];
    const int64_t N = a.N[i], nb = (N + 255) / 256, b = blockIdx.x - a.first[i];
    const int64_t n = (b % nb) * 256 + threadIdx.x, ch = b / nb;
    if (n >= N) return;
    const int64_t r0 = ch * a.chunk, r1 = min(a.rows[i], r0 + a.chunk);
    float s = 0.f;
#pragma unroll 16   // loads in flight; the sum keeps its order
    for (int64_t r = r0; r < r1; ++r) s += X[r * N + n];
    a.part[i][ch * N + n] = s;
}

__global__ void colsum_merge_kernel(ColSums a)
{
    int i = a.n - 1;
    while (i > 0 && blockIdx.x < a.mfirst[i]) --i;
    const float* __restrict__ part = a.part[i];
    const int64_t N = a.N[i], nch = (a.rows[i] + a.chunk - 1) / a.chunk;
    const int64_t n = (int64_t)(blockIdx.x - a.mfirst[i]) * 256 + threadIdx.x;
    if (n >= N) return;
    float s = 0.f;
#pragma unroll 32   // loads in flight; the sum keeps its order
    for (int64_t c = 0; c < nch; ++c) s += part[c * N + n];
    a.out[i][n] = s;
}

// ------------------------------------------------------------- set loss
constexpr int kMaxLossScales = 4;
struct MmdScales {
    int32_t ns;
    double inv[kMaxLossScales][6];   // 1 / sigma per scale and coordinate
};

__device__ __forceinline__ double wrap_angle_diff(double t)
{
    constexpr double two_pi = 6.283185307179586476925286766559;
    return t - rint(t / two_pi) * two_pi;
}

// Multi-scale Gaussian kernel between particles u and v (6 coordinates;
// angle differences wrapped to [-pi, pi]) and, when du != nullptr, its
// gradient with respect to u.
__device__ __forceinline__ double mmd_k(const MmdScales& sc, const double* u, const double* v, double* du)
{
    double d[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) d[c] = c < 3 ? u[c] - v[c] : wrap_angle_diff(u[c] - v[c]);
    double k = 0.0;
    if (du)
#pragma unroll
        for (int c = 0; c < 6; ++c) du[c] = 0.0;
    for (int s = 0; s < sc.ns; ++s) {
        double q = 0.0;
#pragma unroll
        for (int c = 0; c < 6; ++c) q += (d[c] * sc.inv[s][c]) * (d[c] * sc.inv[s][c]);
        const double e = exp(-0.5 * q);
        k += e;
        if (du)
#pragma unroll
            for (int c = 0; c < 6; ++c) du[c] -= e * d[c] * sc.inv[s][c] * sc.inv[s][c];
    }
    return k;
}

// X[b] (K x 6, FP32 network output, or FP64 when Xd is given) against the
// target set Y[b] (FP64):
//   loss[b] = (1 / K^2) sum_ij [k(x_i, x_j) + k(y_i, y_j) - 2 k(x_i, y_j)]
// (the biased MMD^2 estimate) and, when dX != nullptr,
//   dX[b] = gscale * d loss[b] / d X[b]
//         = gscale (2 / K^2) sum_j [grad_u k(x_i, x_j) - grad_u k(x_i, y_j)].
// Workgroup (b, r) takes the rows i of part r of gridDim.y, 256 at a time (G =
// max(1, 256 / rows) threads to a row, each with a range of j; their sums are
// added in order), and writes its share of the loss to
// part[b gridDim.y + r]; mmd_loss_kernel adds the shares (a sample's only
// workgroup writes the loss itself). Bound by the FP64
// exponentials: 32 samples of 100 particles took 115 us with one workgroup a
// sample, which leaves most of the chip idle, 20 with kMmdParts.
constexpr int kMmdParts = 16;
__global__ __launch_bounds__(256) void mmd_kernel(const float* __restrict__ Xf, const double* __restrict__ Xd,
                                                  const double* __restrict__ Y, int32_t K, MmdScales sc,
                                                  double gscale, float* __restrict__ dX, double* __restrict__ part)
{
    extern __shared__ double sm[];   // X, Y (K x 6 each), then 256 x 6 gradient partials
    const int64_t b = blockIdx.x;
    const int i0 = (int)((int64_t)K * blockIdx.y / gridDim.y), i1 = (int)((int64_t)K * (blockIdx.y + 1) / gridDim.y);
    double* x = sm;
    double* y = sm + 6 * K;
    double* gp = sm + 12 * K;
    for (int e = threadIdx.x; e < 6 * K; e += blockDim.x) {
        x[e] = Xd ? Xd[b * 6 * K + e] : (double)Xf[b * 6 * K + e];
        y[e] = Y[b * 6 * K + e];
    }
    __syncthreads();
    __shared__ double red[256];
    double sum = 0.0;
    const int t = threadIdx.x;
    const double w = gscale * 2.0 / ((double)K * K);
    for (int r0 = i0; r0 < i1; r0 += 256) {
        const int rows = min(256, i1 - r0), G = 256 / rows;
        if (t < G * rows) {
            const int row = t % rows, grp = t / rows, i = r0 + row;
            double g[6] = {0, 0, 0, 0, 0, 0}, du[6];
            const int j0 = (int)((int64_t)K * grp / G), j1 = (int)((int64_t)K * (grp + 1) / G);
            for (int j = j0; j < j1; ++j) {
                const double kxx = mmd_k(sc, x + 6 * i, x + 6 * j, du);
#pragma unroll
                for (int c = 0; c < 6; ++c) g[c] += du[c];
                const double kxy = mmd_k(sc, x + 6 * i, y + 6 * j, du);
#pragma unroll
                for (int c = 0; c < 6; ++c) g[c] -= du[c];
                sum += kxx + mmd_k(sc, y + 6 * i, y + 6 * j, nullptr) - 2.0 * kxy;
            }
            if (dX)
#pragma unroll
                for (int c = 0; c < 6; ++c) gp[t * 6 + c] = g[c];
        }
        __syncthreads();
        if (dX)
            for (int e = t; e < 6 * rows; e += blockDim.x) {
                double s = 0.0;
                for (int q = 0; q < G; ++q) s += gp[q * 6 * rows + e];
                dX[(b * K + r0) * 6 + e] = (float)(w * s);
            }
        __syncthreads();
    }
    red[t] = sum;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (t < s) red[t] += red[t + s];
        __syncthreads();
    }
    if (t == 0) part[b * gridDim.y + blockIdx.y] = gridDim.y == 1 ? red[0] / ((double)K * K) : red[0];
}

// loss[b] = (sum of its shares, in order) / K^2.
__global__ void mmd_loss_kernel(const double* __restrict__ part, int64_t B, int32_t parts, int32_t K,
                                double* __restrict__ loss)
{
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    double s = 0.0;
    for (int r = 0; r < parts; ++r) s += part[b * parts + r];
    loss[b] = s / ((double)K * K);
}

// ------------------------------------------------------------- optimiser
// Adam on FP32 parameters, bias corrections bc1 = 1 - b1^t, bc2 = 1 - b2^t
// (the moments are stored in FP32, the update is evaluated in FP64).
__global__ void adam_kernel(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, int64_t n, double lr, double b1, double b2, double eps,
                            double bc1, double bc2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double gi = g[i];
    const double mm = b1 * (double)m[i] + (1.0 - b1) * gi;
    const double vv = b2 * (double)v[i] + (1.0 - b2) * gi * gi;
    m[i] = (float)mm;
    v[i] = (float)vv;
    w[i] = (float)((double)w[i] - lr * (mm / bc1) / (sqrt(vv / bc2) + eps));
}

// --------------------------------------------------------------- in / out
// Network output (FP32, pairs of `per` values) to particles (FP64);
// bad[i / per] = 1 where a value is not finite (bad cleared by the caller).
__global__ void output_particles_kernel(const float* __restrict__ Y, int64_t n, int64_t per, double* __restrict__ out,
                                        int32_t* __restrict__ bad)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float v = Y[i];
    if (!isfinite(v)) bad[i / per] = 1;
    out[i] = (double)v;
}

__global__ void fill_i32_kernel(int32_t* __restrict__ x, int64_t n, int32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = v;
}

__global__ void fill_u64_kernel(unsigned long long* __restrict__ x, int64_t n, unsigned long long v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = v;
}

// Network input of one cloud: point p of P takes cloud point floor(p n / P)
// (each point once when n == P, evenly repeated when n < P).
__global__ void subsample_kernel(const float* __restrict__ xyz, int64_t n, int64_t P, float* __restrict__ out)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    const int64_t s = (p * n) / P;
    out[3 * p] = xyz[3 * s];
    out[3 * p + 1] = xyz[3 * s + 1];
    out[3 * p + 2] = xyz[3 * s + 2];
}

}  // namespace prop
}  // namespace sicp
