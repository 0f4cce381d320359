// tsat_learned.hip -- gfx950 kernels of the learned proposal: per-variable
// features with signed neighbour aggregation over the occurrence store, and a
// per-variable MLP 16 -> 128 -> 128 -> 1 whose dense layers run on MFMA
// (BF16 operands with FP32 accumulation forward, FP32 operands backward),
// with a deterministic split reduction of the gradient fused with Adam.
//
// The network and its features are not part of the paper: they implement
// the learned initialiser that proposes soft assignments to the
// gradient-based search of Sec. IV-A in place of its N(0,1) start.
#include <hip/hip_runtime.h>

#include "tsat_learned.h"

namespace tsat {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// features
// ---------------------------------------------------------------------------

// Four lanes per variable walk its occurrence records (positive occurrences
// first, then negative ones; each record lists the other literals of the
// clause in clause order).  Clauses holding a variable and its negation are
// skipped.  Round 0 counts and writes the base features and the channels h0;
// round r (1..3) sums sgn(l_v) sgn(l_u) h_{r-1}[u] over co-literals, lane c
// of a variable in channel c, in record order.
//
// A chain of dependent loads (record, then channels) per record: the four
// lanes read one 16-byte channel group together and quadruple the waves that
// hide it, and records of known width (uniform stores) are taken kBatch at a
// time, all their loads in flight before the first sum.  V = 1e5, C = 4.1e5,
// 3-SAT: 36 us per round with a thread per variable and a record at a
// time, 17 us.
constexpr int kBatch = 4;

// sum over one record's co-literals of the signed channel value; false for a
// tautology.  K1: co-literals (code[0 .. K1)).
template <int K1>
__device__ __forceinline__ bool feature_taut(const uint32_t (&code)[K1], uint32_t v)
{
    bool taut = false;
#pragma unroll
    for (int j = 0; j < K1; ++j) taut |= (code[j] >> 1) == v || (j > 0 && (code[j] >> 1) == (code[j - 1] >> 1));
    return taut;
}

template <int K1>
__device__ __forceinline__ void feature_records(const FeatArgs& a, uint32_t v, uint32_t ch, uint32_t beg, uint32_t mid,
                                                uint32_t end, int32_t (&cnt)[2], float& acc)
{
    const float* h = (const float*)a.h_prev;
    for (uint32_t w = beg; w < end; w += kBatch) {
        uint32_t code[kBatch][K1];
        float x[kBatch][K1];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            const size_t rec = w + q < end ? w + q : end - 1;
#pragma unroll
            for (int j = 0; j < K1; ++j) code[q][j] = a.occ_data[rec * K1 + j];
        }
        if (a.round > 0) {
#pragma unroll
            for (int q = 0; q < kBatch; ++q)
#pragma unroll
                for (int j = 0; j < K1; ++j) x[q][j] = h[(size_t)(code[q][j] >> 1) * 4 + ch];
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            if (w + q >= end || feature_taut<K1>(code[q], v)) continue;
            const int neg = w + q >= mid;
            cnt[neg] += 1;
            if (a.round == 0) continue;
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < K1; ++j) s = (code[q][j] & 1u) ? s - x[q][j] : s + x[q][j];
            acc = neg ? acc - s : acc + s;
        }
    }
}

__global__ __launch_bounds__(256) void features_kernel(FeatArgs a)
{
    const uint32_t v = blockIdx.x * 64u + threadIdx.x / 4u, ch = threadIdx.x & 3u;
    if (v >= (uint32_t)a.V) return;
    const uint32_t beg = a.occ_off[v], end = a.occ_off[v + 1], mid = a.occ_mid[v];
    int32_t cnt[2] = {0, 0}, wsum = 0, z = 0; // occurrences by sign, their widths, co-literals
    float acc = 0.f;
    if (a.pure_k) {
        switch (a.pure_k) {
        case 2: feature_records<1>(a, v, ch, beg, mid, end, cnt, acc); break;
        case 3: feature_records<2>(a, v, ch, beg, mid, end, cnt, acc); break;
        default: feature_records<3>(a, v, ch, beg, mid, end, cnt, acc); break;
        }
        wsum = (cnt[0] + cnt[1]) * a.pure_k;
        z = (cnt[0] + cnt[1]) * (a.pure_k - 1);
    } else {
        const float* hp = (const float*)a.h_prev;
        uint32_t w = beg;
        while (w < end) {
            const bool negv = w >= mid;
            const uint32_t km1 = a.occ_data[w], base = w + 1;
            w += 1 + km1;
            bool taut = false;
            uint32_t prev_var = 0xffffffffu;
            float s = 0.f;
            for (uint32_t j = 0; j < km1; ++j) {
                const uint32_t c = a.occ_data[base + j], u = c >> 1;
                taut |= (u == v) | (u == prev_var);
                prev_var = u;
                if (a.round > 0) {
                    const float h = hp[(size_t)u * 4 + ch];
                    s = (c & 1u) ? s - h : s + h;
                }
            }
            if (taut) continue;
            cnt[negv] += 1;
            wsum += (int32_t)km1 + 1;
            z += (int32_t)km1;
            acc = negv ? acc - s : acc + s;
        }
    }
    float* x = a.X + (int64_t)v * kFeat;
    if (a.round == 0) {
        const int32_t pos = cnt[0], neg = cnt[1], deg = pos + neg;
        const float f0 = log1pf((float)pos), f1 = log1pf((float)neg);
        const float bias = (float)(pos - neg) / (float)(deg > 1 ? deg : 1);
        const float width = deg > 0 ? (float)wsum / (float)deg * 0.25f : 0.f;
        const float norm = (float)(pos - neg) / sqrtf((float)(deg > 1 ? deg : 1));
        x[ch] = ch == 0 ? f0 : (ch == 1 ? f1 : (ch == 2 ? bias : width));
        ((float*)a.h_next)[(size_t)v * 4 + ch] = ch == 0 ? bias : (ch == 1 ? norm : (ch == 2 ? f0 - f1 : 1.f));
        if (ch == 0) a.zinv[v] = 1.f / (float)(z > 1 ? z : 1);
    } else {
        const float h = acc * a.zinv[v];
        ((float*)a.h_next)[(size_t)v * 4 + ch] = h;
        x[4 * a.round + ch] = h;
    }
}

hipError_t launch_features(const FeatArgs& a, hipStream_t st)
{
    if (a.V <= 0) return hipSuccess;
    hipLaunchKernelGGL(features_kernel, dim3((unsigned)((a.V + 63) / 64)), dim3(256), 0, st, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// MLP helpers
// ---------------------------------------------------------------------------

// round to nearest bfloat16, ties to even (finite inputs)
__device__ __forceinline__ uint32_t bf16_bits(float x)
{
    const uint32_t u = __float_as_uint(x);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ float bf16_value(uint32_t h) { return __uint_as_float(h << 16); }

// v_mfma_f32_16x16x16_bf16: A[i][k] from lane i + 16*(k/4), element k%4;
// B[k][j] from lane j + 16*(k/4), element k%4; D[i][j] in lane j + 16*(i/4),
// element i%4.
__device__ __forceinline__ v4f mfma_bf16(uint2 a, uint2 b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(v4s, a), __builtin_bit_cast(v4s, b), c, 0,
                                                      0, 0);
}
// v_mfma_f32_16x16x4_f32: A[i][k] from lane i + 16*k, B[k][j] from lane
// j + 16*k, D as above.
__device__ __forceinline__ v4f mfma_f32(float a, float b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// BF16 slot of W1[f][c] among the layer-1 B operands: column tile c/16,
// lane c%16 + 16*(f/4), element f%4
__device__ __forceinline__ int w1_slot(int f, int c) { return ((c >> 4) * 64 + (c & 15) + 16 * (f >> 2)) * 4 + (f & 3); }
// BF16 slot of W2[k][c] among the layer-2 B operands: k-step k/16, column
// tile c/16, lane c%16 + 16*((k%16)/4), element k%4
__device__ __forceinline__ int w2_slot(int k, int c)
{
    return (((k >> 4) * 8 + (c >> 4)) * 64 + (c & 15) + 16 * ((k & 15) >> 2)) * 4 + (k & 3);
}

// BF16 slot of W2[k][c] among the operands of the transposed product
// (da2 W2^T): c-step c/16, column tile k/16, lane k%16 + 16*((c%16)/4),
// element c%4
__device__ __forceinline__ int w2t_slot(int k, int c)
{
    return (((c >> 4) * 8 + (k >> 4)) * 64 + (k & 15) + 16 * ((c & 15) >> 2)) * 4 + (c & 3);
}

// Four FP32 values as three BF16 operands each, x = s[0] + s[1] + s[2]: each
// part is the rounded rest of the ones before it, 8 significant bits a part,
// so the sum is x itself for magnitudes of 2^-102 (below, the last part leaves
// the normal numbers) up to 2^127 (above, the first may round to infinity).
// An infinity's rest, and a NaN's, is some finite number, which changes nothing
// beside them.  Products with BF16 operands are then exact in the FP32
// accumulation, as FP32 operands would be, at the BF16 matrix rate.
__device__ __forceinline__ void split_bf16(const float (&x)[4], uint2 (&s)[3])
{
    float r[4] = {x[0], x[1], x[2], x[3]};
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        uint32_t h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            h[e] = bf16_bits(r[e]);
            r[e] -= bf16_value(h[e]);
            if (p == 0) r[e] = fmaxf(r[e], -0x1p120f);
        }
        s[p] = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
    }
}

__device__ __forceinline__ void write_operand(const MlpDev& d, int e, float p)
{
    if (e < kOffB1) {
        reinterpret_cast<uint16_t*>(d.w1op)[w1_slot(e / kHid, e % kHid)] = (uint16_t)bf16_bits(p);
    } else if (e >= kOffW2 && e < kOffB2) {
        const int k = (e - kOffW2) / kHid, c = (e - kOffW2) % kHid;
        reinterpret_cast<uint16_t*>(d.w2op)[w2_slot(k, c)] = (uint16_t)bf16_bits(p);
        reinterpret_cast<uint16_t*>(d.w2t)[w2t_slot(k, c)] = (uint16_t)bf16_bits(p);
    } else if (e >= kOffW3 && e < kOffB3) {
        d.w3q[e - kOffW3] = bf16_value(bf16_bits(p));
    }
}

__global__ void mlp_quantize_kernel(MlpDev d)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < kNumParams) write_operand(d, e, d.params[e]);
}

constexpr int kH1S = 136; // BF16 row stride of an h1 tile
constexpr int kDS = 132;  // FP32 row stride of a da tile
constexpr int kXS = 20;   // FP32 row stride of the rounded-input tile
constexpr int kRed = 3 * kHid + 2;

// ---------------------------------------------------------------------------
// MLP forward / backward
// ---------------------------------------------------------------------------

// A block of 4 waves takes 64 rows at a time (16 per wave).  Layer 1 is one
// MFMA per 16-column tile (K = 16); its rounded ReLU output goes through LDS
// into the A layout of layer 2 (8 K-steps x 8 column tiles against the W2
// operands held in LDS); layer 3 is a dot product per row.  With TRAIN, the
// block then forms dLoss/da2 per row and accumulates, over all its rows,
//   dW2 = h1q^T da2   (each wave 2 of the 8 row tiles of dW2),
//   dh1 = da2 W2q^T   (each wave its own 16 rows),
//   dW1 = xq^T da1    (each wave 2 of the 8 column tiles, FP32 MFMA),
// and the bias / w3 gradients, in a fixed order; its sums go to one slot of
// the partial buffer, which mlp_reduce_kernel adds up in block order.
// In dW2 and dh1 one factor is BF16 already (h1q, W2q) and da2 is split into
// three BF16 parts, so they run at the BF16 rate with nothing rounded: dLoss/dout
// and what follows from it are held at 2^24 times their size, so that the parts
// of small ones stay normal numbers, or at 2^-24 where the block's row weights,
// labels or w3 allow a da2 past 2^76 or are not finite (error
// of the gradient against FP64, four seeds: B = 16384 1.3e-7 .. 2.1e-6,
// FP32 operands 2.8e-7 .. 2.1e-6; B = 60000 1.6e-7 .. 1.0e-6 and 2.9e-7 ..
// 1.1e-6; the upper ends are rounding decisions of h1 that FP32 and FP64 take
// differently).  The
// accumulator layout of the forward is the operand layout of dW2 (lane r + 16 q
// holds rows 4 q .. 4 q + 3 of column r), so each wave hands its h1 and da2
// parts over in lane order, without a transpose.  B = 16384, one block per CU:
// 35.4 us with FP32 operands read element by element from LDS, 28.6 us so, 29.0
// with the scale.
template <bool TRAIN>
__global__ __launch_bounds__(256) void mlp_kernel(MlpDev d, const float* __restrict__ X, const float* __restrict__ y,
                                                  const float* __restrict__ wt, int64_t B,
                                                  float* __restrict__ logits, float* __restrict__ probs)
{
    __shared__ uint2 s_w2[8 * 8 * 64];
    __shared__ __align__(16) uint16_t s_h1[4][16 * kH1S];
    __shared__ __align__(16) float s_da[TRAIN ? 4 : 1][TRAIN ? 16 * kDS : 1];
    __shared__ __align__(16) float s_xq[TRAIN ? 64 * kXS : 1];
    __shared__ float s_red[TRAIN ? 4 * kRed : 1];
    __shared__ uint2 s_opA[TRAIN ? 4 : 1][TRAIN ? 8 * 64 : 1];     // h1 of a wave's rows, [tile][lane]
    __shared__ uint2 s_opB[TRAIN ? 4 : 1][TRAIN ? 3 * 8 * 64 : 1]; // da2 parts, [part][tile][lane]
    __shared__ int s_large[4];                                     // a da2 may pass 2^76, by wave

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, r = lane & 15, q = lane >> 4;
    // |dLoss/dout| <= |weight| (1 + |label|) / B; a NaN stays
    float reach = 0.f;
    if (TRAIN) {
        for (int64_t i = ((int64_t)wv * gridDim.x + blockIdx.x) * 64 + lane; i < B; i += (int64_t)gridDim.x * 256) {
            const float x = (wt ? fabsf(wt[i]) : 1.f) * (1.f + fabsf(y[i]));
            reach = x <= reach ? reach : x;
        }
    }
    for (int e = tid; e < 8 * 8 * 64; e += 256) s_w2[e] = d.w2op[e];
    uint2 w1[8];
    float b1c[8], b2c[8], w3c[8];
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        w1[n] = d.w1op[n * 64 + lane];
        b1c[n] = d.params[kOffB1 + 16 * n + r];
        b2c[n] = d.params[kOffB2 + 16 * n + r];
        w3c[n] = d.w3q[16 * n + r];
    }
    const float b3 = d.params[kOffB3];
    const float invB = 1.f / (float)B;
    float scale = 0x1p24f;
    if (TRAIN) {
        float w3top = 0.f;
#pragma unroll
        for (int n = 0; n < 8; ++n) w3top = fmaxf(w3top, fabsf(w3c[n]));
        const uint64_t large = __ballot(!(reach * invB < 0x1p50f && w3top < 0x1p26f));
        if (lane == 0) s_large[wv] = large != 0;
    }
    __syncthreads();
    // everything from dLoss/dout on carries the scale
    if (TRAIN && (s_large[0] | s_large[1] | s_large[2] | s_large[3])) scale = 0x1p-24f;

    const v4f zero = {0.f, 0.f, 0.f, 0.f};
    v4f gW2[2][8], gW1[2];
    float gb1[8], gb2[8], gw3[8], gb3 = 0.f, gloss = 0.f;
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        gW2[0][n] = zero;
        gW2[1][n] = zero;
        gb1[n] = gb2[n] = gw3[n] = 0.f;
    }
    gW1[0] = gW1[1] = zero;
    const int64_t nsuper = (B + 63) / 64;
    uint16_t* h1 = s_h1[wv];
    float* da = s_da[TRAIN ? wv : 0];

    for (int64_t sup = blockIdx.x; sup < nsuper; sup += gridDim.x) {
        const int64_t row0 = sup * 64 + wv * 16;
        const int64_t row = row0 + r;
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row < B) x = *reinterpret_cast<const float4*>(X + row * kFeat + 4 * q);
        const uint32_t e0 = bf16_bits(x.x), e1 = bf16_bits(x.y), e2 = bf16_bits(x.z), e3 = bf16_bits(x.w);
        const uint2 ax = make_uint2(e0 | (e1 << 16), e2 | (e3 << 16));
        if (TRAIN)
            *reinterpret_cast<float4*>(&s_xq[(wv * 16 + r) * kXS + 4 * q]) =
                make_float4(bf16_value(e0), bf16_value(e1), bf16_value(e2), bf16_value(e3));
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const v4f c = mfma_bf16(ax, w1[n], zero);
            uint32_t hb[4];
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                hb[rr] = bf16_bits(fmaxf(c[rr] + b1c[n], 0.f));
                h1[(4 * q + rr) * kH1S + 16 * n + r] = (uint16_t)hb[rr];
            }
            if (TRAIN) s_opA[TRAIN ? wv : 0][TRAIN ? n * 64 + lane : 0] = make_uint2(hb[0] | (hb[1] << 16), hb[2] | (hb[3] << 16));
        }
        __syncthreads();
        v4f acc[8];
#pragma unroll
        for (int n = 0; n < 8; ++n) acc[n] = zero;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const uint2 ah = *reinterpret_cast<const uint2*>(&h1[r * kH1S + 16 * s + 4 * q]);
            uint2 b2[8];
#pragma unroll
            for (int n = 0; n < 8; ++n) b2[n] = s_w2[(s * 8 + n) * 64 + lane];
#pragma unroll
            for (int n = 0; n < 8; ++n) acc[n] = mfma_bf16(ah, b2[n], acc[n]);
            // five LDS reads, then eight products: left to itself the scheduler
            // waits for each pair of operands (3e5 rows: 238 us a step, 224)
            __builtin_amdgcn_sched_group_barrier(0x100, 5, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
        }
        float out[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int n = 0; n < 8; ++n)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) out[rr] += fmaxf(acc[n][rr] + b2c[n], 0.f) * w3c[n];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            out[rr] += __shfl_xor(out[rr], 1);
            out[rr] += __shfl_xor(out[rr], 2);
            out[rr] += __shfl_xor(out[rr], 4);
            out[rr] += __shfl_xor(out[rr], 8);
            out[rr] += b3;
        }
        if (!TRAIN) {
            if (r == 0) {
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const int64_t ro = row0 + 4 * q + rr;
                    if (ro < B) {
                        if (logits) logits[ro] = out[rr];
                        if (probs) probs[ro] = 1.f / (1.f + expf(-out[rr]));
                    }
                }
            }
            __syncthreads(); // the next iteration rewrites the h1 tiles
            continue;
        }
        // ---- backward ----
        float dout[4];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int64_t ro = row0 + 4 * q + rr;
            dout[rr] = 0.f;
            if (ro < B) {
                const float yy = y[ro], ww = wt ? wt[ro] : 1.f, z = out[rr];
                dout[rr] = ww * (1.f / (1.f + expf(-z)) - yy) * invB;
                if (r == 0) gloss += ww * (fmaxf(z, 0.f) + log1pf(expf(-fabsf(z))) - yy * z) * invB;
            }
        }
        // a NaN as the one whose upper half is a NaN
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) dout[rr] = dout[rr] == dout[rr] ? dout[rr] * scale : __builtin_nanf("");
        if (r == 0) gb3 += (dout[0] + dout[1]) + (dout[2] + dout[3]);
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            float g4[4];
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const float a2 = acc[n][rr] + b2c[n];
                const float g = a2 > 0.f ? dout[rr] * w3c[n] : 0.f;
                g4[rr] = g;
                da[(4 * q + rr) * kDS + 16 * n + r] = g;
                gb2[n] += g;
                gw3[n] += fmaxf(a2, 0.f) * dout[rr];
            }
            uint2 part[3];
            split_bf16(g4, part);
#pragma unroll
            for (int p = 0; p < 3; ++p) s_opB[TRAIN ? wv : 0][TRAIN ? (p * 8 + n) * 64 + lane : 0] = part[p];
        }
        __syncthreads();
        // dW2 row tiles 2*wv and 2*wv+1 over the four waves' rows, smallest
        // parts first
        for (int sw = 0; sw < 4; ++sw) {
            const uint2 a0 = s_opA[TRAIN ? sw : 0][TRAIN ? (2 * wv) * 64 + lane : 0];
            const uint2 a1 = s_opA[TRAIN ? sw : 0][TRAIN ? (2 * wv + 1) * 64 + lane : 0];
#pragma unroll
            for (int n = 0; n < 8; ++n)
#pragma unroll
                for (int p = 2; p >= 0; --p) {
                    const uint2 b = s_opB[TRAIN ? sw : 0][TRAIN ? (p * 8 + n) * 64 + lane : 0];
                    gW2[0][n] = mfma_bf16(a0, b, gW2[0][n]);
                    gW2[1][n] = mfma_bf16(a1, b, gW2[1][n]);
                }
        }
        // dh1 of this wave's rows: sum over columns of da2 * W2q
        v4f dh[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) dh[m] = zero;
#pragma unroll 2
        for (int st = 0; st < 8; ++st) {
            const float4 f = *reinterpret_cast<const float4*>(&da[r * kDS + 16 * st + 4 * q]);
            const float x4[4] = {f.x, f.y, f.z, f.w};
            uint2 part[3];
            split_bf16(x4, part);
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const uint2 b = d.w2t[(st * 8 + m) * 64 + lane];
#pragma unroll
                for (int p = 2; p >= 0; --p) dh[m] = mfma_bf16(part[p], b, dh[m]);
            }
        }
        __syncthreads(); // every wave is done with the da2 tiles
#pragma unroll
        for (int m = 0; m < 8; ++m)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int kk = 16 * m + r;
                const float g = bf16_value(h1[(4 * q + rr) * kH1S + kk]) > 0.f ? dh[m][rr] : 0.f;
                da[(4 * q + rr) * kDS + kk] = g;
                gb1[m] += g;
            }
        __syncthreads();
        // dW1 column tiles 2*wv and 2*wv+1 over the 64 rows
        for (int t = 0; t < 16; ++t) {
            const int rw = 4 * t + q, sw = rw >> 4, lr = rw & 15;
            const float xa = s_xq[rw * kXS + r];
#pragma unroll
            for (int mm = 0; mm < 2; ++mm)
                gW1[mm] = mfma_f32(xa, s_da[TRAIN ? sw : 0][lr * kDS + 16 * (2 * wv + mm) + r], gW1[mm]);
        }
        __syncthreads(); // the next super-tile rewrites every tile
    }
    if (!TRAIN) return;

    const float unscale = 1.f / scale;
    float* P = d.partial + (int64_t)blockIdx.x * kPartialStride;
#pragma unroll
    for (int mm = 0; mm < 2; ++mm) {
#pragma unroll
        for (int n = 0; n < 8; ++n)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
                P[kOffW2 + (16 * (2 * wv + mm) + 4 * q + rr) * kHid + 16 * n + r] = gW2[mm][n][rr] * unscale;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) P[kOffW1 + (4 * q + rr) * kHid + 16 * (2 * wv + mm) + r] = gW1[mm][rr] * unscale;
    }
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        gb1[n] += __shfl_xor(gb1[n], 16);
        gb1[n] += __shfl_xor(gb1[n], 32);
        gb2[n] += __shfl_xor(gb2[n], 16);
        gb2[n] += __shfl_xor(gb2[n], 32);
        gw3[n] += __shfl_xor(gw3[n], 16);
        gw3[n] += __shfl_xor(gw3[n], 32);
    }
    gb3 += __shfl_xor(gb3, 16);
    gb3 += __shfl_xor(gb3, 32);
    gloss += __shfl_xor(gloss, 16);
    gloss += __shfl_xor(gloss, 32);
    if (q == 0) {
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            s_red[wv * kRed + 16 * n + r] = gb1[n] * unscale;
            s_red[wv * kRed + kHid + 16 * n + r] = gb2[n] * unscale;
            s_red[wv * kRed + 2 * kHid + 16 * n + r] = gw3[n] * unscale;
        }
    }
    if (lane == 0) {
        s_red[wv * kRed + 3 * kHid] = gb3 * unscale;
        s_red[wv * kRed + 3 * kHid + 1] = gloss;
    }
    __syncthreads();
    for (int e = tid; e < kRed; e += 256) {
        const float sum = ((s_red[e] + s_red[kRed + e]) + s_red[2 * kRed + e]) + s_red[3 * kRed + e];
        int dst;
        if (e < kHid) dst = kOffB1 + e;
        else if (e < 2 * kHid) dst = kOffB2 + e - kHid;
        else if (e < 3 * kHid) dst = kOffW3 + e - 2 * kHid;
        else if (e == 3 * kHid) dst = kOffB3;
        else dst = kNumParams; // loss
        P[dst] = sum;
    }
}

// Sum of the blocks' partial gradients in a fixed order, then Adam.  A block
// takes kRedCols parameters: its kRedSegs thread groups each add a run of
// consecutive blocks, eight loads in flight, and the runs are added in order.
// (One thread per parameter adding all blocks one after the other waits for
// memory 256 times: 61 us for 256 blocks; 7.7 us this way, 19 MB.)
constexpr int kRedCols = 32, kRedSegs = 8;

__global__ __launch_bounds__(256) void mlp_reduce_kernel(MlpDev d, int blocks, int adam, float lr, float beta1,
                                                         float beta2, float eps, float bc1, float bc2)
{
    __shared__ float s_sum[kRedSegs][kRedCols];
    const int col = threadIdx.x % kRedCols, seg = threadIdx.x / kRedCols;
    const int e = blockIdx.x * kRedCols + col;
    const int run = (blocks + kRedSegs - 1) / kRedSegs;
    const int b0 = seg * run, b1 = min(blocks, b0 + run);
    float sum = 0.f;
    if (e <= kNumParams) {
        const float* p = d.partial + e;
        for (int b = b0; b < b1; b += 8) {
            float x[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = b + q < b1 ? p[(int64_t)(b + q) * kPartialStride] : 0.f;
#pragma unroll
            for (int q = 0; q < 8; ++q) sum += x[q];
        }
    }
    s_sum[seg][col] = sum;
    __syncthreads();
    if (seg != 0 || e > kNumParams) return;
    float g = 0.f;
#pragma unroll
    for (int q = 0; q < kRedSegs; ++q) g += s_sum[q][col];
    if (e == kNumParams) {
        *d.loss = g;
        return;
    }
    d.grad[e] = g;
    if (!adam) return;
    const float m = beta1 * d.m[e] + (1.f - beta1) * g;
    const float v = beta2 * d.v[e] + (1.f - beta2) * g * g;
    d.m[e] = m;
    d.v[e] = v;
    const float p = d.params[e] - lr * (m / bc1) / (sqrtf(v / bc2) + eps);
    d.params[e] = p;
    write_operand(d, e, p);
}

hipError_t launch_mlp_forward(const MlpDev& d, const float* X, int64_t B, float* logits, float* probs,
                              hipStream_t st)
{
    if (B <= 0) return hipSuccess;
    const int64_t nsuper = (B + 63) / 64;
    const int blocks = (int)(nsuper < 768 ? nsuper : 768);
    hipLaunchKernelGGL(mlp_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, st, d, X, (const float*)nullptr,
                       (const float*)nullptr, B, logits, probs);
    return hipGetLastError();
}

int mlp_train_blocks(int64_t B)
{
    const int64_t nsuper = (B + 63) / 64;
    return (int)(nsuper < 256 ? (nsuper > 0 ? nsuper : 1) : 256);
}

hipError_t launch_mlp_backward(const MlpDev& d, const float* X, const float* y, const float* w, int64_t B,
                               hipStream_t st)
{
    hipLaunchKernelGGL(mlp_kernel<true>, dim3((unsigned)mlp_train_blocks(B)), dim3(256), 0, st, d, X, y, w, B,
                       (float*)nullptr, (float*)nullptr);
    return hipGetLastError();
}

hipError_t launch_mlp_reduce(const MlpDev& d, int blocks, int adam, float lr, float beta1, float beta2, float eps,
                             float bc1, float bc2, hipStream_t st)
{
    hipLaunchKernelGGL(mlp_reduce_kernel, dim3((kNumParams + kRedCols) / kRedCols), dim3(256), 0, st, d, blocks, adam, lr,
                       beta1, beta2, eps, bc1, bc2);
    return hipGetLastError();
}

hipError_t launch_mlp_quantize(const MlpDev& d, hipStream_t st)
{
    hipLaunchKernelGGL(mlp_quantize_kernel, dim3((kNumParams + 255) / 256), dim3(256), 0, st, d);
    return hipGetLastError();
}

} // namespace tsat
