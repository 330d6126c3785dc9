// mlp_kernels.hip -- the warm-start scoring network (20 -> 256 -> 256 -> 120,
// ReLU) on the matrix cores: BF16 operands, FP32 accumulation.
//
// All products run on v_mfma_f32_16x16x16_bf16 tiles.  Inference is one kernel
// (all layers and the top-k of a tile of 64 directions).  A training step's
// gradients are two: everything that is local to a row of the batch -- forward
// pass, loss, dS, dZ2, dZ1 -- for a tile of sixteen rows in one workgroup with
// the activations in LDS (mlp_rows_kernel), and everything that sums over the
// batch -- dW, bias gradients, mean loss (mlp_sums_kernel).  Every reduction
// runs in a fixed order, so a training step is deterministic.
//
// The remaining kernel: AdamW on the FP32 master weights with a fresh BF16 copy.
#include <math.h>
#include <stdint.h>

#include "internal.h"

namespace lpb {
namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// FP32 -> bfloat16 bits, round to nearest, ties to even (finite inputs).
__device__ __forceinline__ uint16_t to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}

// AdamW on the FP32 master copy; decay[i] = 1 for weights, 0 for biases.
__global__ void adamw_kernel(float *w, const float *g, float *m, float *v, uint16_t *w16, int64_t count,
                             MlpAdam h, int64_t decay_lo0, int64_t decay_hi0, int64_t decay_lo1,
                             int64_t decay_hi1, int64_t decay_lo2, int64_t decay_hi2)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const bool decay = (i >= decay_lo0 && i < decay_hi0) || (i >= decay_lo1 && i < decay_hi1) ||
                       (i >= decay_lo2 && i < decay_hi2);
    const float gi = g[i];
    const float mi = h.beta1 * m[i] + (1.f - h.beta1) * gi;
    const float vi = h.beta2 * v[i] + (1.f - h.beta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float mhat = mi / h.bc1;
    const float vhat = vi / h.bc2;
    float wi = w[i];
    wi = wi - h.lr * mhat / (sqrtf(vhat) + h.eps) - (decay ? h.lr * h.wd * w[i] : 0.f);
    w[i] = wi;
    w16[i] = to_bf16(wi);
}

__global__ void cast_params_kernel(const float *w, uint16_t *w16, int64_t count)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < count) w16[i] = to_bf16(w[i]);
}


// ---- Fused inference --------------------------------------------------------
// All three layers and the top-k for a tile of 64 directions in one workgroup
// of four wavefronts: the input tile and both hidden activations stay in LDS
// (BF16), the weights stream from L2 as MFMA fragments.  The products, their
// k order and the epilogues are those of the training forward pass, so the
// scores are the same bits.

// ---- Top-k by a bitonic sort over the wavefront ------------------------------
// Key of entry t with score v: the score's bits mapped to an order-preserving
// unsigned integer (-0 taken as +0, so equal scores give equal keys) above
// 127 - t, so that descending key order is descending score with equal scores
// in ascending entry order.
__device__ __forceinline__ uint64_t topk_key(float v, int t)
{
    const uint32_t u = __float_as_uint(v + 0.0f);
    const uint32_t mono = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return (uint64_t(mono) << 32) | uint32_t(127 - t);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t v)
{
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, 0xf, 0xf, false));
}

// Value of lane (lane ^ J).  DPP patterns: quad_perm [1,0,3,2] (0xB1) and
// [2,3,0,1] (0x4E) swap at distance 1 and 2; [3,2,1,0] (0x1B) after
// row_half_mirror (0x141, i -> i ^ 7 in each group of 8) gives i ^ 4;
// row_half_mirror after row_mirror (0x140, i -> i ^ 15 in each row of 16) gives
// i ^ 8; the permlane swaps exchange rows (16) and halves (32).
template <int J>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v)
{
    const int lane = threadIdx.x & 63;
    if constexpr (J == 1) return dpp32<0xB1>(v);
    else if constexpr (J == 2) return dpp32<0x4E>(v);
    else if constexpr (J == 4) return dpp32<0x1B>(dpp32<0x141>(v));
    else if constexpr (J == 8) return dpp32<0x141>(dpp32<0x140>(v));
    else if constexpr (J == 16) {
        auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return ((lane >> 4) & 1) ? uint32_t(p[0]) : uint32_t(p[1]);
    } else {
        auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (lane >> 5) ? uint32_t(p[0]) : uint32_t(p[1]);
    }
}

template <int J>
__device__ __forceinline__ uint64_t xor_lane64(uint64_t v)
{
    return (uint64_t(xor_lane<J>(uint32_t(v >> 32))) << 32) | xor_lane<J>(uint32_t(v));
}

// One compare-exchange step (block size SZ, distance J < 64) on both halves:
// element e keeps the larger key when bit J of e is clear exactly when bit SZ
// of e is clear (descending blocks), the smaller otherwise.
template <int SZ, int J>
__device__ __forceinline__ void bitonic_step(uint64_t &k0, uint64_t &k1)
{
    const int lane = threadIdx.x & 63;
    const uint64_t p0 = xor_lane64<J>(k0), p1 = xor_lane64<J>(k1);
    const bool lower = (lane & J) == 0;
    const bool up0 = ((lane + 0) & SZ) == 0, up1 = ((lane + 64) & SZ) == 0;
    const bool max0 = lower == up0, max1 = lower == up1;
    // Take the partner's key when it is larger and this element keeps the
    // larger, or it is not larger and this element keeps the smaller.
    k0 = ((p0 > k0) == max0) ? p0 : k0;
    k1 = ((p1 > k1) == max1) ? p1 : k1;
}

template <int SZ, int J>
__device__ __forceinline__ void bitonic_merge2(uint64_t &a0, uint64_t &a1, uint64_t &b0, uint64_t &b1)
{
    if constexpr (J == 64) {
        const uint64_t ah = a0 > a1 ? a0 : a1, al = a0 > a1 ? a1 : a0;
        const uint64_t bh = b0 > b1 ? b0 : b1, bl = b0 > b1 ? b1 : b0;
        a0 = ah; a1 = al; b0 = bh; b1 = bl;
    } else {
        bitonic_step<SZ, J>(a0, a1);
        bitonic_step<SZ, J>(b0, b1);
    }
    if constexpr (J > 1) bitonic_merge2<SZ, J / 2>(a0, a1, b0, b1);
}

template <int SZ>
__device__ __forceinline__ void bitonic_stage2(uint64_t &a0, uint64_t &a1, uint64_t &b0, uint64_t &b1)
{
    bitonic_merge2<SZ, SZ / 2>(a0, a1, b0, b1);
    if constexpr (SZ < 128) bitonic_stage2<SZ * 2>(a0, a1, b0, b1);
}

// Sorts two independent sets of 128 keys, (a0, a1) and (b0, b1), each in
// descending order over positions lane (x0) and lane + 64 (x1); all 64
// lanes must be active.
__device__ __forceinline__ void bitonic_desc128x2(uint64_t &a0, uint64_t &a1, uint64_t &b0, uint64_t &b1)
{
    bitonic_stage2<2>(a0, a1, b0, b1);
}

constexpr int kTile = 64;
constexpr int kIn = 20, kHid = 256, kOut = 120;
constexpr int64_t kOW1 = 0, kOB1 = kOW1 + int64_t(kHid) * kIn, kOW2 = kOB1 + kHid,
                  kOB2 = kOW2 + int64_t(kHid) * kHid, kOW3 = kOB2 + kHid, kOB3 = kOW3 + int64_t(kOut) * kHid;

// Row strides (BF16 elements) of the LDS tiles, padded so that the sixteen
// rows one MFMA fragment load touches fall in different LDS banks.
constexpr int kLdx = 40, kLdh = kHid + 8;

__host__ __device__ constexpr int64_t infer_lds_bytes()
{
    return int64_t(kTile) * kLdx * 2 + 2 * int64_t(kTile) * kLdh * 2;
}

// Weight fragment: row n of a [rows][K] BF16 matrix, k = k0 .. k0+3 (zero past K or rows).
__device__ __forceinline__ s16x4 wfrag(const uint16_t *w, int n, int rows, int K, int k0)
{
    s16x4 v = {0, 0, 0, 0};
    if (n >= rows) return v;
    if (k0 + 3 < K) {
        const uint2 q = *reinterpret_cast<const uint2 *>(w + int64_t(n) * K + k0);
        v[0] = short(q.x & 0xFFFF);
        v[1] = short(q.x >> 16);
        v[2] = short(q.y & 0xFFFF);
        v[3] = short(q.y >> 16);
        return v;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (k0 + t < K) v[t] = short(w[int64_t(n) * K + k0 + t]);
    return v;
}

// One layer on the tile: out[64][NT*16*4 waves] = act[64][K] * W^T (+ bias),
// this wavefront taking N tiles NT*wave .. NT*wave + NT-1.  Epilogue: BF16
// ReLU activations (h16, row stride kLdh) or FP32 scores (s32, row stride 128).
template <int NT>
__device__ __forceinline__ void tile_layer(const uint16_t *act, int lda, int K, const uint16_t *w, int rows,
                                           const float *bias, uint16_t *h16, float *s32)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, kq = (lane >> 4) * 4;
    f32x4 acc[4][NT];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[a][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Weight fragments are loaded one k step ahead of their use.
    s16x4 fbn[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) fbn[j] = wfrag(w, (NT * wave + j) * 16 + r16, rows, K, kq);
    for (int k0 = 0; k0 < K; k0 += 16) {
        s16x4 fa[4], fb[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) fb[j] = fbn[j];
        if (k0 + 16 < K) {
#pragma unroll
            for (int j = 0; j < NT; ++j) fbn[j] = wfrag(w, (NT * wave + j) * 16 + r16, rows, K, k0 + 16 + kq);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) fa[a] = *reinterpret_cast<const s16x4 *>(act + (16 * a + r16) * lda + k0 + kq);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[a][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa[a], fb[j], acc[a][j], 0, 0, 0);
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int col = (NT * wave + j) * 16 + r16;
            const float bj = col < rows ? bias[col] : 0.f;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int row = 16 * a + kq + t;
                const float v = acc[a][j][t] + bj;
                if (h16) h16[row * kLdh + col] = to_bf16(fmaxf(v, 0.f));
                else s32[row * 128 + col] = v;
            }
        }
}

__global__ __launch_bounds__(256) void mlp_infer_kernel(const float *dirs, int64_t B, const uint16_t *w16,
                                                        const float *w32, float *scores, int32_t *topk, int k)
{
    extern __shared__ __align__(16) char smem[];
    uint16_t *x16 = reinterpret_cast<uint16_t *>(smem);                         // [64][kLdx]
    uint16_t *h1 = reinterpret_cast<uint16_t *>(smem + kTile * kLdx * 2);       // [64][kLdh]
    uint16_t *h2 = h1 + kTile * kLdh;                                             // [64][kLdh]
    float *sc = reinterpret_cast<float *>(h1);                                    // [64][128], after layer 2
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t b0 = int64_t(blockIdx.x) * kTile;
    for (int e = tid; e < kTile * 32; e += 256) {
        const int r = e >> 5, kk = e & 31;
        const int64_t b = b0 + r;
        x16[r * kLdx + kk] = to_bf16((b < B && kk < kIn) ? dirs[b * kIn + kk] : 0.f);
    }
    __syncthreads();
    tile_layer<4>(x16, kLdx, kIn, w16 + kOW1, kHid, w32 + kOB1, h1, nullptr);
    __syncthreads();
    tile_layer<4>(h1, kLdh, kHid, w16 + kOW2, kHid, w32 + kOB2, h2, nullptr);
    __syncthreads();
    tile_layer<2>(h2, kLdh, kHid, w16 + kOW3, kOut, w32 + kOB3, nullptr, sc);
    __syncthreads();
    // Scores out, and the top-k of every row by rank counting (one wavefront
    // per sixteen rows; lanes hold entries lane and lane + 64).
    // Two rows per step, so that the two sorts' independent instruction
    // chains interleave.
    for (int rr = 0; rr < kTile / 4; rr += 2) {
        const int row = wave * (kTile / 4) + rr;
        const int64_t b = b0 + row;
        if (b >= B) break;
        const bool two = b + 1 < B;
        float s0[2], s1[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            s0[q] = sc[(row + q) * 128 + lane];
            s1[q] = (lane + 64 < kOut) ? sc[(row + q) * 128 + lane + 64] : 0.f;
        }
        if (scores) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (q == 1 && !two) break;
                scores[(b + q) * kOut + lane] = s0[q];
                if (lane + 64 < kOut) scores[(b + q) * kOut + lane + 64] = s1[q];
            }
        }
        if (topk) {
            // Sort each row's 120 keys (and 8 padding keys below every real
            // one) in descending order; position e = lane + 64 h then holds
            // the entry of rank e.
            uint64_t ka0 = topk_key(s0[0], lane), kb0 = topk_key(s0[1], lane);
            uint64_t ka1 = (lane + 64 < kOut) ? topk_key(s1[0], lane + 64) : 0;
            uint64_t kb1 = (lane + 64 < kOut) ? topk_key(s1[1], lane + 64) : 0;
            bitonic_desc128x2(ka0, ka1, kb0, kb1);
            if (lane < k) topk[b * k + lane] = 127 - int(uint32_t(ka0));
            if (lane + 64 < k) topk[b * k + lane + 64] = 127 - int(uint32_t(ka1));
            if (two) {
                if (lane < k) topk[(b + 1) * k + lane] = 127 - int(uint32_t(kb0));
                if (lane + 64 < k) topk[(b + 1) * k + lane + 64] = 127 - int(uint32_t(kb1));
            }
        }
    }
}

// ---- Training: gradients of a batch ---------------------------------------------
// What limited the layer-by-layer form (one launch per product, elementwise step
// and column sum, fifteen in all) was latency: the dW products ran on 8 to 64
// wavefronts whose lanes gathered every operand two bytes at a time, 100 us
// each for 512 rows.  The row kernel writes the BF16 operands of the dW
// products transposed (the rows of a tile are neighbours in a lane's
// accumulators, so that is one 8-byte store), and both kernels load several k
// steps ahead.  512 rows: 410 us before, 37 us now (25 and 14 us in a kernel trace).

// Weight fragment of a product that contracts over a weight matrix's rows:
// column j of a [K][cols] BF16 matrix, k = k0 .. k0+3 (zero past K).
__device__ __forceinline__ s16x4 wfrag_t(const uint16_t *w, int j, int cols, int K, int k0)
{
    s16x4 v = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (k0 + t < K) v[t] = short(w[int64_t(k0 + t) * cols + j]);
    return v;
}

constexpr int kRowsT = 16;  // batch rows of a workgroup
constexpr int kWavesT = 8;  // wavefronts of a workgroup
constexpr int kNT = kHid / 16 / kWavesT;  // column tiles of a hidden layer per wavefront
static_assert(16 * kWavesT >= kOut, "one column tile of the scores per wavefront");
constexpr int kLdo = 136;   // row stride of the dS tile: 120 columns, 0 up to 128

// acc[j] = the wavefront's NT column tiles of act[16][K] * W, fragments by
// frag(column tile, k0), eight k steps loaded ahead.
template <int NT, int K, typename F>
__device__ __forceinline__ void rows_product(const uint16_t *act, int lda, F frag, f32x4 (&acc)[NT])
{
    constexpr int STEPS = (K + 15) / 16, U = 8;
    const int lane = threadIdx.x & 63, r16 = lane & 15, kq = (lane >> 4) * 4;
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s0 = 0; s0 < STEPS; s0 += U) {
        s16x4 fb[U][NT];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < NT; ++j)
                if (s0 + u < STEPS) fb[u][j] = frag(j, 16 * (s0 + u) + kq);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + u >= STEPS) continue;
            const s16x4 fa = *reinterpret_cast<const s16x4 *>(act + r16 * lda + 16 * (s0 + u) + kq);
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa, fb[u][j], acc[j], 0, 0, 0);
        }
    }
}

__device__ __forceinline__ s16x4 pack4(const float (&v)[4])
{
    return s16x4{short(to_bf16(v[0])), short(to_bf16(v[1])), short(to_bf16(v[2])), short(to_bf16(v[3]))};
}

// Rows b0 .. b0 + 15 of the batch.  D layout of a tile: lane holds column
// lane % 16 and rows 4 (lane / 16) + t, so the masks of the backward pass stay
// in the lanes that computed Z1 and Z2.
__global__ __launch_bounds__(64 * kWavesT) void mlp_rows_kernel(MlpTrain g)
{
    __shared__ __align__(16) uint16_t x16[kRowsT * kLdx];
    __shared__ __align__(16) uint16_t ha[kRowsT * kLdh];   // H1, then dZ2
    __shared__ __align__(16) uint16_t hb[kRowsT * kLdh];   // H2
    __shared__ __align__(16) uint16_t d16[kRowsT * kLdo];  // dS
    __shared__ __align__(16) float sc[kRowsT * 128];       // S
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, kq = (lane >> 4) * 4;
    const int64_t B = g.B, b0 = int64_t(blockIdx.x) * kRowsT;
    const uint16_t *w16 = g.w16;
    const float *w32 = g.w32;
    for (int e = tid; e < kRowsT * 32; e += 64 * kWavesT) {
        const int r = e >> 5, k = e & 31;
        x16[r * kLdx + k] = to_bf16((b0 + r < B && k < kIn) ? g.dirs[(b0 + r) * kIn + k] : 0.f);
    }
    for (int e = tid; e < kRowsT * kLdo; e += 64 * kWavesT) d16[e] = 0;
    __syncthreads();
    // Four rows of column c of a BF16 tile into the transposed array (rows past
    // the batch stay within its padding and are not read).
    const int64_t bt = b0 + kq;
    auto put_t = [&](uint16_t *t, int c, s16x4 v) { *reinterpret_cast<s16x4 *>(t + c * g.ldt + bt) = v; };
    if (tid < 4 * kIn) {
        const int c = tid >> 2, q = (tid & 3) * 4;
        s16x4 v;
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = short(x16[(q + t) * kLdx + c]);
        *reinterpret_cast<s16x4 *>(g.xt + c * g.ldt + b0 + q) = v;
    }
    // A hidden layer's epilogue: bias, ReLU, BF16; returns which values pass.
    auto hidden = [&](const f32x4 (&acc)[kNT], const float *bias, uint16_t *h, uint16_t *ht) {
        uint32_t pass = 0;
#pragma unroll
        for (int j = 0; j < kNT; ++j) {
            const int c = (kNT * wave + j) * 16 + r16;
            float v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float z = acc[j][t] + bias[c];
                pass |= uint32_t(z > 0.f) << (4 * j + t);
                v[t] = fmaxf(z, 0.f);
                h[(kq + t) * kLdh + c] = to_bf16(v[t]);
            }
            put_t(ht, c, pack4(v));
        }
        return pass;
    };
    f32x4 acc[kNT];
    rows_product<kNT, kIn>(x16, kLdx, [&](int j, int k0) { return wfrag(w16 + kOW1, (kNT * wave + j) * 16 + r16, kHid, kIn, k0); }, acc);
    const uint32_t pass1 = hidden(acc, w32 + kOB1, ha, g.h1t);
    __syncthreads();
    rows_product<kNT, kHid>(ha, kLdh, [&](int j, int k0) { return wfrag(w16 + kOW2, (kNT * wave + j) * 16 + r16, kHid, kHid, k0); }, acc);
    const uint32_t pass2 = hidden(acc, w32 + kOB2, hb, g.h2t);
    __syncthreads();
    {
        f32x4 s[1];
        rows_product<1, kHid>(hb, kLdh, [&](int j, int k0) { return wfrag(w16 + kOW3, (wave + j) * 16 + r16, kOut, kHid, k0); }, s);
        const int c = wave * 16 + r16;
#pragma unroll
        for (int t = 0; t < 4; ++t) sc[(kq + t) * 128 + c] = s[0][t] + (c < kOut ? w32[kOB3 + c] : 0.f);
    }
    __syncthreads();
    // Loss and dS = (sigmoid(S) - Y) / (B * O): one wavefront per row, lane j
    // takes outputs j and j + 64, the row's loss by a fixed butterfly.
    const float inv = 1.0f / (float(B) * float(kOut));
    for (int r = wave; r < kRowsT; r += kWavesT) {
        const int64_t b = b0 + r;
        if (b >= B) break;
        float loss = 0.f;
        for (int j = lane; j < kOut; j += 64) {
            const float s = sc[r * 128 + j];
            const float y = g.tight[b * kOut + j] ? 1.f : 0.f;
            const float sp = fmaxf(s, 0.f) + log1pf(expf(-fabsf(s)));
            loss += sp - y * s;
            const float sg = 1.f / (1.f + expf(-s));
            const float d = (sg - y) * inv;
            g.ds[b * kOut + j] = d;
            d16[r * kLdo + j] = to_bf16(d);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off);
        if (lane == 0) g.row_loss[b] = loss;
    }
    __syncthreads();
    for (int e = tid; e < 4 * kOut; e += 64 * kWavesT) {
        const int c = e >> 2, q = (e & 3) * 4;
        s16x4 v;
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = short(d16[(q + t) * kLdo + c]);
        *reinterpret_cast<s16x4 *>(g.dst + c * g.ldt + b0 + q) = v;
    }
    // dZ = (upstream * W) where the ReLU passed: FP32 for the bias gradient,
    // BF16 for the products.
    auto masked = [&](const f32x4 (&a)[kNT], uint32_t pass, float *z32, uint16_t *z, uint16_t *zt) {
#pragma unroll
        for (int j = 0; j < kNT; ++j) {
            const int c = (kNT * wave + j) * 16 + r16;
            float v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                v[t] = (pass >> (4 * j + t)) & 1 ? a[j][t] + 0.f : 0.f;
                if (bt + t < B) z32[(bt + t) * kHid + c] = v[t];
                if (z) z[(kq + t) * kLdh + c] = to_bf16(v[t]);
            }
            put_t(zt, c, pack4(v));
        }
    };
    rows_product<kNT, kOut>(d16, kLdo, [&](int j, int k0) { return wfrag_t(w16 + kOW3, (kNT * wave + j) * 16 + r16, kHid, kOut, k0); }, acc);
    masked(acc, pass2, g.dz2, ha, g.dz2t);
    __syncthreads();
    rows_product<kNT, kHid>(ha, kLdh, [&](int j, int k0) { return wfrag_t(w16 + kOW2, (kNT * wave + j) * 16 + r16, kHid, kHid, k0); }, acc);
    masked(acc, pass1, g.dz1, nullptr, g.dz1t);
}

// One 16 x 16 tile of a dW product over the batch: C[i][j] = sum_b a[i][b] w[j][b]
// with both operands transposed ([rows][ldt], b contiguous), in order of b.
__device__ __forceinline__ void dw_tile(const uint16_t *a, int M, const uint16_t *w, int N, int64_t ldt, int64_t B,
                                        int ti, int tj, float *C)
{
    const int lane = threadIdx.x & 63, r16 = lane & 15, kq = (lane >> 4) * 4;
    const int i = 16 * ti + r16, j = 16 * tj + r16;
    const uint16_t *pa = a + int64_t(i < M ? i : M - 1) * ldt, *pw = w + int64_t(j < N ? j : N - 1) * ldt;
    // Past the batch: whole groups of four are skipped, a last partial one masked.
    auto frag = [&](const uint16_t *p, int64_t k) {
        s16x4 v = {0, 0, 0, 0};
        if (k < B) v = *reinterpret_cast<const s16x4 *>(p + k);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (k + t >= B) v[t] = 0;
        return v;
    };
    constexpr int U = 8;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int64_t k0 = 0; k0 < B; k0 += 16 * U) {
        s16x4 fa[U], fw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            fa[u] = frag(pa, k0 + 16 * u + kq);
            fw[u] = frag(pw, k0 + 16 * u + kq);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k0 + 16 * u < B) acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa[u], fw[u], acc, 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int row = 16 * ti + kq + t;
        if (row < M && j < N) C[int64_t(row) * N + j] = acc[t] + 0.f;
    }
}

// db[j] = sum_b dZ[b][j] for 64 columns: sixteen partial sums over rows p, p + 16,
// ... in order, then the partial sums in order of p.
__device__ __forceinline__ void column_sums(const float *dZ, int64_t B, int N, int j0, float *db, float (&part)[16][64])
{
    const int c = threadIdx.x & 63, j = j0 + c;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    const int p0 = (threadIdx.x >> 6) * 4;
    constexpr int U = 8;  // sixteen-row steps loaded ahead
    if (j < N)
        for (int64_t b0 = p0; b0 < B; b0 += 16 * U) {
            float v[U][4];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t b = b0 + 16 * u + q;
                    v[u][q] = dZ[(b < B ? b : B - 1) * N + j];
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (b0 + 16 * u + q < B) s[q] += v[u][q];
        }
#pragma unroll
    for (int q = 0; q < 4; ++q) part[p0 + q][c] = s[q];
    __syncthreads();
    if (threadIdx.x < 64 && j < N) {
        float t = part[0][c];
#pragma unroll
        for (int q = 1; q < 16; ++q) t += part[q][c];
        db[j] = t;
    }
}

// Tiles of the three dW products (four wavefronts to a workgroup), then the bias
// gradients (64 columns to a workgroup), then the mean loss.
constexpr int kTilesH = kHid / 16, kTilesO = (kOut + 15) / 16, kTilesI = (kIn + 15) / 16;
constexpr int kDw2 = kTilesH * kTilesH, kDw3 = kTilesO * kTilesH, kDw1 = kTilesH * kTilesI;
constexpr int kDwBlocks = (kDw2 + kDw3 + kDw1) / 4;
constexpr int kColsH = kHid / 64, kColsO = (kOut + 63) / 64;
static_assert((kDw2 + kDw3 + kDw1) % 4 == 0 && kHid % 64 == 0, "whole workgroups of tiles");

__global__ __launch_bounds__(256) void mlp_sums_kernel(MlpTrain g)
{
    __shared__ union {
        float cols[16][64];
        double mean[256];
    } sh;
    const int tid = threadIdx.x;
    int blk = blockIdx.x;
    if (blk < kDwBlocks) {
        int t = 4 * blk + (tid >> 6);
        if (t < kDw2) dw_tile(g.dz2t, kHid, g.h1t, kHid, g.ldt, g.B, t / kTilesH, t % kTilesH, g.grad + kOW2);
        else if ((t -= kDw2) < kDw3) dw_tile(g.dst, kOut, g.h2t, kHid, g.ldt, g.B, t / kTilesH, t % kTilesH, g.grad + kOW3);
        else {
            t -= kDw3;
            dw_tile(g.dz1t, kHid, g.xt, kIn, g.ldt, g.B, t / kTilesI, t % kTilesI, g.grad + kOW1);
        }
        return;
    }
    blk -= kDwBlocks;
    if (blk < kColsH) return column_sums(g.dz2, g.B, kHid, 64 * blk, g.grad + kOB2, sh.cols);
    blk -= kColsH;
    if (blk < kColsH) return column_sums(g.dz1, g.B, kHid, 64 * blk, g.grad + kOB1, sh.cols);
    blk -= kColsH;
    if (blk < kColsO) return column_sums(g.ds, g.B, kOut, 64 * blk, g.grad + kOB3, sh.cols);
    // Mean of the row losses: each thread sums a strided slice, then a tree.
    double s = 0.0;
    for (int64_t b = tid; b < g.B; b += 256) s += double(g.row_loss[b]);
    sh.mean[tid] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) sh.mean[tid] += sh.mean[tid + w];
        __syncthreads();
    }
    if (tid == 0) *g.loss = float(sh.mean[0] / (double(g.B) * kOut));
}

}  // namespace

hipError_t launch_mlp_grads(const MlpTrain &g, hipStream_t s)
{
    hipLaunchKernelGGL(mlp_rows_kernel, dim3(unsigned((g.B + kRowsT - 1) / kRowsT)), dim3(64 * kWavesT), 0, s,
                       g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mlp_sums_kernel, dim3(kDwBlocks + 2 * kColsH + kColsO + 1), dim3(256), 0, s, g);
    return hipGetLastError();
}

hipError_t launch_adamw(float *w, const float *g, float *m, float *v, uint16_t *w16, int64_t count,
                        const MlpAdam &h, const int64_t (&decay)[6], hipStream_t s)
{
    hipLaunchKernelGGL(adamw_kernel, dim3(unsigned((count + 255) / 256)), dim3(256), 0, s, w, g, m, v, w16,
                       count, h, decay[0], decay[1], decay[2], decay[3], decay[4], decay[5]);
    return hipGetLastError();
}

hipError_t launch_cast_params(const float *w, uint16_t *w16, int64_t count, hipStream_t s)
{
    hipLaunchKernelGGL(cast_params_kernel, dim3(unsigned((count + 255) / 256)), dim3(256), 0, s, w, w16, count);
    return hipGetLastError();
}

hipError_t launch_mlp_infer(const float *dirs, int64_t B, const uint16_t *w16, const float *w32, float *scores,
                            int32_t *topk, int k, hipStream_t s)
{
    if (B <= 0) return hipSuccess;
    hipLaunchKernelGGL(mlp_infer_kernel, dim3(unsigned((B + kTile - 1) / kTile)), dim3(256), size_t(infer_lds_bytes()), s,
                       dirs, B, w16, w32, scores, topk, k);
    return hipGetLastError();
}

hipError_t mlp_configure()
{
    return hipFuncSetAttribute((const void *)mlp_infer_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               int(infer_lds_bytes()));
}

}  // namespace lpb
