// The refinement network: 12 -> 64 -> 64 -> 1 with ReLU between layers and a
// logit out, BF16 weights and activations on the matrix cores with FP32
// accumulation (v_mfma_f32_32x32x8_bf16), FP32 master weights and Adam.  The
// hidden activations feeding the second layer are carried as two bf16 parts
// (value and residual, two products each): one bf16 rounding there moves
// pre-activations across the ReLU kink often enough to change gradients by
// percents, while the rounding of weights and back-propagated gradients
// costs about 2^-9.
//
// Parameters (FP32, 5057): W1 [12][64], b1 [64], W2 [64][64], b2 [64],
// W3 [64], b3; layer l computes h_l = relu(h_{l-1} W_l + b_l).
// Loss: mean_i [ w+ y_i softplus(-z_i) + (1 - y_i) softplus(z_i) ].
//
// One wavefront takes 32 samples.  Every product is a 32 x 32 block tile (one
// MFMA per 8 of the reduced dimension): lane l holds A(l % 32, 4 (l / 32) + t) and
// B(4 (l / 32) + t, l % 32), t < 4, read as 8 bytes along the reduced dimension.
#include <algorithm>

#include "cellfeat.hpp"
#include "dev.hpp"

namespace mlm {

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NP = 5057;
constexpr int OW1 = 0, OB1 = 768, OW2 = 832, OB2 = 4928, OW3 = 4992, OB3 = 5056;
constexpr int MB = 128;   // samples are padded to whole groups of so many

// float -> bf16, round to nearest even (finite inputs): one hardware
// conversion (v_cvt_pk_bf16_f32) in the default rounding mode
__device__ inline uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// row of accumulator element j of lane `lane` in a 32 x 32 tile (its column is
// lane % 32)
__device__ inline int acc_row(int j, int lane) { return 8 * (j >> 2) + 4 * (lane >> 5) + (j & 3); }

constexpr int PS = 68;    // padded row stride (bf16) of the 64-wide operands: 136 B, so rows fall in other banks
constexpr int XS = 20;    // and of the 16-wide input rows: 40 B

__device__ inline void wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline bf16x4 row4(const uint16_t *p) { return *reinterpret_cast<const bf16x4 *>(p); }
__device__ inline f32x16 mma32(bf16x4 a, bf16x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a, b, c, 0, 0, 0);
}

// Inference only.  The products are formed transposed (units by samples): what a
// lane then holds of a layer's result, units 8 q + 4 (lane / 32) + t of sample
// lane % 32, is just what it feeds the next layer's product, so the activations
// stay in registers, as the weights do (a lane's 224 bytes of them and 384 of
// biases, loaded once; a wavefront loops over the samples).  Same arithmetic as the
// training's forward pass (bf16 inputs, two-part bf16 hidden layer, FP32
// accumulation); the final 64-term sum runs in another order, through LDS.  Bound
// by vector issue (555 instructions per 32 cells beside the products): 4.7e8 cells
// in 21.0 ms, with every operand through LDS 23.7; the products alone would take 7.
struct PredictNet {
    bf16x4 w1[2][2], w2[2][8];
    float b1[2][16], b2[2][16], w3[2][16], b3;

    __device__ void load(const uint16_t *__restrict__ W1t, const uint16_t *__restrict__ W2t, const float *__restrict__ P,
                         int lane)
    {
        const int r = lane & 31, h4 = 4 * (lane >> 5);
#pragma unroll
        for (int nh = 0; nh < 2; ++nh) {
#pragma unroll
            for (int k = 0; k < 2; ++k) w1[nh][k] = row4(W1t + (nh * 32 + r) * 16 + 8 * k + h4);
#pragma unroll
            for (int k = 0; k < 8; ++k) w2[nh][k] = row4(W2t + (nh * 32 + r) * 64 + 8 * k + h4);
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int c = nh * 32 + acc_row(j, lane);
                b1[nh][j] = P[OB1 + c];
                b2[nh][j] = P[OB2 + c];
                w3[nh][j] = bf2f(f2bf(P[OW3 + c]));
            }
        }
        b3 = P[OB3];
    }

    // the terms of 32 samples' logits, of units j and 32 + j together, to zb
    // [sample][ZP], twice, so that they can be read from any of them on; x0, x1: this lane's inputs 4 (lane / 32) .. + 3 and 8 more on
    // of sample lane % 32
    static constexpr int ZP = 65;
    __device__ __forceinline__ void terms(bf16x4 x0, bf16x4 x1, float *zb, int lane) const
    {
        bf16x4 hi[8], lo[8];
#pragma unroll
        for (int nh = 0; nh < 2; ++nh) {
            f32x16 acc = {};
            acc = mma32(w1[nh][0], x0, acc);
            acc = mma32(w1[nh][1], x1, acc);
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const float h = fmaxf(acc[j] + b1[nh][j], 0.0f);
                const uint16_t v = f2bf(h);
                hi[nh * 4 + (j >> 2)][j & 3] = (short)v;
                lo[nh * 4 + (j >> 2)][j & 3] = (short)f2bf(h - bf2f(v));
            }
        }
        float part[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) part[j] = 0.0f;
#pragma unroll
        for (int nh = 0; nh < 2; ++nh) {
            f32x16 acc = {};
#pragma unroll
            for (int k = 0; k < 8; ++k) acc = mma32(w2[nh][k], hi[k], acc);
#pragma unroll
            for (int k = 0; k < 8; ++k) acc = mma32(w2[nh][k], lo[k], acc);
#pragma unroll
            for (int j = 0; j < 16; ++j) part[j] += fmaxf(acc[j] + b2[nh][j], 0.0f) * w3[nh][j];
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            float *to = zb + (lane & 31) * ZP + acc_row(j, lane);
            to[0] = part[j];
            to[32] = part[j];
        }
    }

    // the logit of sample `lane` of 64, from their terms, term lane % 32 first
    __device__ float logit(const float *zb, int lane) const
    {
        const float *from = zb + lane * ZP + (lane & 31);
        float z = b3;
#pragma unroll
        for (int q = 0; q < 32; ++q) z += from[q];
        return z;
    }
};
constexpr int PW = 4;   // wavefronts of an inference workgroup

__global__ __launch_bounds__(64 * PW) __attribute__((amdgpu_waves_per_eu(2))) void k_mlp_predict(const float *__restrict__ feats, int64_t n,
                                                         const uint16_t *__restrict__ W1t,
                                                         const uint16_t *__restrict__ W2t, const float *__restrict__ P,
                                                         float *__restrict__ logits)
{
    __shared__ float zs[PW][64 * PredictNet::ZP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 31, hh = lane >> 5;
    PredictNet net;
    net.load(W1t, W2t, P, lane);
    float *zb = zs[wave];
    const int64_t nblocks = (n + 63) / 64, nwaves = (int64_t)gridDim.x * PW;
    for (int64_t blk = (int64_t)blockIdx.x * PW + wave; blk < nblocks; blk += nwaves) {
        const int64_t s0 = blk * 64;
#pragma unroll 1
        for (int half = 0; half < 2; ++half) {
            const int64_t s = s0 + 32 * half + r;
            bf16x4 x0 = {}, x1 = {};
            if (s < n) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    x0[k] = (short)f2bf(feats[s * 12 + 4 * hh + k]);
                    if (hh == 0) x1[k] = (short)f2bf(feats[s * 12 + 8 + k]);
                }
            }
            net.terms(x0, x1, zb + 32 * half * PredictNet::ZP, lane);
        }
        wave_sync_lds();
        const float z = net.logit(zb, lane);
        if (s0 + lane < n) logits[s0 + lane] = z;
        wave_sync_lds();   // (the next samples overwrite zb)
    }
}

// The cells of a strip (cells [cb0, cb0 + ncells / (nr1 - 1)) of the grid,
// vertex rows from vb0 in `verts`) that the refinement tests: the network's
// logit above thr, or folded.  Features are formed from the mapped corners
// by the two lanes that feed them in (zero for a cell with a non-finite corner,
// which the test then leaves alone), so nothing per cell goes through memory but
// its bit in the block's mask.
__global__ __launch_bounds__(64 * PW) __attribute__((amdgpu_waves_per_eu(2))) void k_mlp_flag_cells(int64_t nr1, int64_t cb0, int64_t ncells, int64_t vb0,
                                                            const double2 *__restrict__ verts,
                                                            const uint16_t *__restrict__ W1t,
                                                            const uint16_t *__restrict__ W2t,
                                                            const float *__restrict__ P, float thr,
                                                            uint64_t *__restrict__ mask, int32_t *__restrict__ cnt)
{
    __shared__ float zs[PW][64 * PredictNet::ZP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 31, hh = lane >> 5;
    PredictNet net;
    net.load(W1t, W2t, P, lane);
    float *zb = zs[wave];
    const int64_t nblocks = (ncells + 63) / 64, nwaves = (int64_t)gridDim.x * PW;
    // (a strip's cells number fewer than 2^32)
    const uint32_t ncol = (uint32_t)(nr1 - 1);
    for (int64_t blk = (int64_t)blockIdx.x * PW + wave; blk < nblocks; blk += nwaves) {
        bool fold = false;
        // row and column of the block's first cell
        const uint32_t t0 = __builtin_amdgcn_readfirstlane((uint32_t)(blk * 64)), row0 = t0 / ncol, a0 = t0 - row0 * ncol;
#pragma unroll 1
        for (int half = 0; half < 2; ++half) {
            // cell r of the half, half hh of its features on this lane
            const uint32_t t = t0 + 32 * half + r;
            float f[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) f[k] = 0.0f;
            if ((int64_t)t < ncells) {
                uint32_t row = row0, a = a0 + 32 * half + r;
                while (a >= ncol) {   // (once at most, unless the grid is narrower than a block)
                    a -= ncol;
                    ++row;
                }
                const double2 *r0 = verts + (cb0 + row - vb0) * nr1 + a, *r1 = r0 + nr1;
                const double2 q[4] = {r0[0], r0[1], r1[1], r1[0]};
                const double u4[4] = {q[0].x, q[1].x, q[2].x, q[3].x}, v4[4] = {q[0].y, q[1].y, q[2].y, q[3].y};
                if (isfinite(u4[0]) && isfinite(u4[1]) && isfinite(u4[2]) && isfinite(u4[3]) && isfinite(v4[0]) &&
                    isfinite(v4[1]) && isfinite(v4[2]) && isfinite(v4[3]))
                    cell_features_half_f32(u4, v4, hh, f);
            }
            // the four ear signs (0 or +-1): this lane's two, and its partner's
            const float g4 = __shfl_xor(f[4], 32, 64), g5 = __shfl_xor(f[5], 32, 64);
            const bool flat = f[4] == f[5] && f[5] == g4 && g4 == g5;
            if (half == hh) fold = !flat;
            bf16x4 x0, x1 = {};
#pragma unroll
            for (int k = 0; k < 4; ++k) x0[k] = (short)f2bf(f[k]);
            if (hh == 0) x1 = bf16x4{(short)f2bf(f[4]), (short)f2bf(f[5]), (short)f2bf(g4), (short)f2bf(g5)};
            net.terms(x0, x1, zb + 32 * half * PredictNet::ZP, lane);
        }
        wave_sync_lds();
        const float z = net.logit(zb, lane);
        const uint64_t flags = __ballot(blk * 64 + lane < ncells && (z > thr || fold));
        if (lane == 0) {
            mask[blk] = flags;
            cnt[blk] = __popcll(flags);
        }
        wave_sync_lds();
    }
}

__device__ inline float softplus(float x) { return x > 0.0f ? x + log1pf(expf(-x)) : log1pf(expf(x)); }

// A training wavefront's LDS.  Every product reads its operands as rows along
// the reduced dimension, 8 bytes a lane and MFMA, so what enters products in
// both directions is stored both ways.
constexpr int TS = 36;    // row stride (bf16) of the operands reduced over the 32 samples: 72 B
constexpr int ZS = 33;    // and of the FP32 layer-2 activations
struct TrainLds {
    uint16_t x[32 * XS], xt[16 * TS];          // inputs [sample][feature] and [feature][sample]
    uint16_t h1[32 * PS], h1lo[32 * PS];       // layer-1 activations [sample][unit], two bf16 parts
    uint16_t h1t[64 * TS], h1lot[64 * TS];     // [unit][sample]
    uint16_t d2t[64 * TS];                     // gradient at layer-2 pre-activations [unit][sample]
    float h2t[64 * ZS];                        // layer-2 activations [unit][sample]
    float z[32], dz[32];
    // (re-used once what they held is spent)
    __device__ uint16_t *d2() { return h1; }                                      // [sample][unit]
    __device__ uint16_t *d1t() { return reinterpret_cast<uint16_t *>(h2t); }      // layer 1's, [unit][sample]
};

// forward and backward of samples idx[s] (s in [0, n)); each wavefront (32
// samples, a workgroup of its own, so that a batch's few wavefronts spread over
// the CUs) writes its whole gradient (FP32) and its part of the loss (at [NP]; the
// loss is divided by `norm`, the batch size) to its own row part[w * (NP + 1) ..],
// w = blockIdx.x, with no atomics: the rows are then added in a fixed order, so a
// batch's gradient is the same bits on every run.  The pass is one chain of
// latencies; the weights (W1t, W2t: transposed; W2b) are loaded to registers at
// its start, beside the samples (4096 samples: 11.8 us; through strided two-byte
// reads of LDS and memory, four wavefronts a workgroup, 26).
__global__ __launch_bounds__(64) void k_mlp_train(const float *__restrict__ feats_all, const uint8_t *__restrict__ y_all,
                                                  const int64_t *__restrict__ idx, int64_t n,
                                                  const uint16_t *__restrict__ W1t, const uint16_t *__restrict__ W2t,
                                                  const uint16_t *__restrict__ W2b, const float *__restrict__ P,
                                                  float pos_weight, float norm, float *__restrict__ part)
{
    __shared__ TrainLds L;
    const int lane = threadIdx.x, r = lane & 31, hh = lane >> 5, h4 = 4 * hh;
    const int64_t s0 = (int64_t)blockIdx.x * 32;
    float *g = part + (int64_t)blockIdx.x * (NP + 1);
    // sample r of the wavefront, half hh of its features on this lane
    const bool have = s0 + r < n;
    const int64_t row = have ? idx[s0 + r] : 0;
    bf16x4 w1[2][2], w2[2][8], w2n[2][8];
    float b1v[2], b2v[2];
#pragma unroll
    for (int nh = 0; nh < 2; ++nh) {
        const int c = nh * 32 + r;
#pragma unroll
        for (int k = 0; k < 2; ++k) w1[nh][k] = row4(W1t + c * 16 + 8 * k + h4);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            w2[nh][k] = row4(W2t + c * 64 + 8 * k + h4);
            w2n[nh][k] = row4(W2b + c * 64 + 8 * k + h4);
        }
        b1v[nh] = P[OB1 + c];
        b2v[nh] = P[OB2 + c];
    }
    const float w3 = bf2f(f2bf(P[OW3 + lane])), b3 = P[OB3];
    float f[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) f[k] = have ? feats_all[row * 12 + 6 * hh + k] : 0.0f;
    const float y = have ? (float)y_all[row] : 0.0f;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const uint16_t v = f2bf(f[k]);
        L.x[r * XS + 6 * hh + k] = v;
        L.xt[(6 * hh + k) * TS + r] = v;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        L.x[r * XS + 12 + 2 * hh + k] = 0;
        L.xt[(12 + 2 * hh + k) * TS + r] = 0;
    }
    wave_sync_lds();
    // layer 1
#pragma unroll
    for (int nh = 0; nh < 2; ++nh) {
        f32x16 acc = {};
#pragma unroll
        for (int k = 0; k < 2; ++k) acc = mma32(row4(L.x + r * XS + 8 * k + h4), w1[nh][k], acc);
        const int c = nh * 32 + r;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            bf16x4 hi4, lo4;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float h = fmaxf(acc[4 * q + t] + b1v[nh], 0.0f);
                const uint16_t hi = f2bf(h), lo = f2bf(h - bf2f(hi));
                L.h1[(8 * q + h4 + t) * PS + c] = hi;
                L.h1lo[(8 * q + h4 + t) * PS + c] = lo;
                hi4[t] = (short)hi;
                lo4[t] = (short)lo;
            }
            *reinterpret_cast<bf16x4 *>(L.h1t + c * TS + 8 * q + h4) = hi4;
            *reinterpret_cast<bf16x4 *>(L.h1lot + c * TS + 8 * q + h4) = lo4;
        }
    }
    wave_sync_lds();
    // layer 2
#pragma unroll
    for (int nh = 0; nh < 2; ++nh) {
        f32x16 acc = {};
#pragma unroll
        for (int k = 0; k < 8; ++k) acc = mma32(row4(L.h1 + r * PS + 8 * k + h4), w2[nh][k], acc);
#pragma unroll
        for (int k = 0; k < 8; ++k) acc = mma32(row4(L.h1lo + r * PS + 8 * k + h4), w2[nh][k], acc);
        const int c = nh * 32 + r;
#pragma unroll
        for (int j = 0; j < 16; ++j) L.h2t[c * ZS + acc_row(j, lane)] = fmaxf(acc[j] + b2v[nh], 0.0f);
    }
    wave_sync_lds();
    // layer 3, the loss and dL/dz (lanes of the first half: a sample each)
    {
        float z = b3;
#pragma unroll
        for (int c = 0; c < 64; ++c)
            z += L.h2t[c * ZS + r] * __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w3), c));
        float l = 0.0f;
        if (lane < 32) {
            float dz = 0.0f;
            if (have) {
                const float sg = 1.0f / (1.0f + expf(-z));
                l = pos_weight * y * softplus(-z) + (1.0f - y) * softplus(z);
                dz = (pos_weight * y * (sg - 1.0f) + (1.0f - y) * sg) / norm;
            }
            L.dz[lane] = dz;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) l += __shfl_xor(l, o, 64);
        if (lane == 0) g[NP] = l / norm;
    }
    wave_sync_lds();
    // layer 3: dW3, db3; gradient at layer-2 pre-activations (lane: a unit)
    {
        float gw = 0.0f, gb = 0.0f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            bf16x4 d4;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int m = 4 * q + t;
                const float h = L.h2t[lane * ZS + m], dz = L.dz[m];
                gw += dz * h;
                const float d = h > 0.0f ? dz * w3 : 0.0f;
                gb += d;
                const uint16_t v = f2bf(d);
                L.d2()[m * PS + lane] = v;
                d4[t] = (short)v;
            }
            *reinterpret_cast<bf16x4 *>(L.d2t + lane * TS + 4 * q) = d4;
        }
        g[OW3 + lane] = gw;
        g[OB2 + lane] = gb;
        if (lane == 0) {
            float s = 0.0f;
            for (int m = 0; m < 32; ++m) s += L.dz[m];
            g[OB3] = s;
        }
    }
    wave_sync_lds();
    // dW2 (64 x 64) = h1^T d2
#pragma unroll
    for (int ih = 0; ih < 2; ++ih)
#pragma unroll
        for (int jh = 0; jh < 2; ++jh) {
            f32x16 acc = {};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                acc = mma32(row4(L.h1t + (ih * 32 + r) * TS + 8 * k + h4), row4(L.d2t + (jh * 32 + r) * TS + 8 * k + h4), acc);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                acc = mma32(row4(L.h1lot + (ih * 32 + r) * TS + 8 * k + h4), row4(L.d2t + (jh * 32 + r) * TS + 8 * k + h4), acc);
#pragma unroll
            for (int j = 0; j < 16; ++j) g[OW2 + (ih * 32 + acc_row(j, lane)) * 64 + jh * 32 + r] = acc[j];
        }
    // gradient at layer-1 pre-activations: (d2 W2^T) masked
#pragma unroll
    for (int ih = 0; ih < 2; ++ih) {
        f32x16 acc = {};
#pragma unroll
        for (int k = 0; k < 8; ++k) acc = mma32(row4(L.d2() + r * PS + 8 * k + h4), w2n[ih][k], acc);
        const int c = ih * 32 + r;
        float b1 = 0.0f;   // db1 of unit c: this lane's rows, then the other half's
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bf16x4 h = row4(L.h1t + c * TS + 8 * q + h4);
            bf16x4 d4;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float d = h[t] != 0 ? acc[4 * q + t] : 0.0f;   // relu'(pre) = [h1 > 0]
                d4[t] = (short)f2bf(d);
                b1 += d;
            }
            *reinterpret_cast<bf16x4 *>(L.d1t() + c * TS + 8 * q + h4) = d4;
        }
        b1 += __shfl_xor(b1, 32, 64);
        if (lane < 32) g[OB1 + c] = b1;
    }
    wave_sync_lds();
    // dW1 (16 x 64, rows 12.. zero) = x^T d1
#pragma unroll
    for (int jh = 0; jh < 2; ++jh) {
        f32x16 acc = {};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            bf16x4 av = row4(L.xt + (r & 15) * TS + 8 * k + h4);
            if (r >= 16) av = bf16x4{0, 0, 0, 0};
            acc = mma32(av, row4(L.d1t() + (jh * 32 + r) * TS + 8 * k + h4), acc);
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int k = acc_row(j, lane);
            if (k < 12) g[OW1 + k * 64 + jh * 32 + r] = acc[j];
        }
    }
}

// grad[t] += the sum over the rows w = 0 .. nrows - 1 of part[w * (NP + 1) + t],
// in a fixed order: a workgroup takes 32 parameters; its thread (g, p) sums
// the rows g, g + GS_GROUPS, ... of parameter p in order, and the GS_GROUPS
// partial sums are then added in the order g = 0, 1, ...
constexpr int GS_GROUPS = 8;

__device__ inline float grad_rows(const float *__restrict__ part, int64_t nrows, int t, int g, int p,
                                  float (&ps)[GS_GROUPS][32])
{
    float s = 0.0f;
    if (t <= NP) {
        int64_t w = g;
        for (; w + 7 * GS_GROUPS < nrows; w += 8 * GS_GROUPS) {   // (eight loads in flight, added in order)
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = part[(w + k * GS_GROUPS) * (NP + 1) + t];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += v[k];
        }
        for (; w < nrows; w += GS_GROUPS) s += part[w * (NP + 1) + t];
    }
    ps[g][p] = s;
    __syncthreads();
    float a = 0.0f;
    if (g == 0) {
#pragma unroll
        for (int k = 0; k < GS_GROUPS; ++k) a += ps[k][p];
    }
    return a;
}

__global__ __launch_bounds__(32 * GS_GROUPS) void k_grad_sum(const float *__restrict__ part, int64_t nrows,
                                                             float *__restrict__ grad)
{
    __shared__ float ps[GS_GROUPS][32];
    const int p = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int t = blockIdx.x * 32 + p;
    const float a = grad_rows(part, nrows, t, g, p, ps);
    if (g == 0 && t <= NP) grad[t] += a;
}

// The bf16 copies of the weights in the layouts the kernels read, for parameter
// t of value v: W1t [64][16] (layer 1's transposed; columns 12 .. zero, set once),
// W2b [64][64] and behind it W2t, its transpose.
__device__ inline void pack_weight(int t, float v, uint16_t *W1t, uint16_t *W2b)
{
    if (t < OB1) {
        const int k = t >> 6, c = t & 63;
        W1t[c * 16 + k] = f2bf(v);
    } else if (t >= OW2 && t < OB2) {
        const int k = (t - OW2) >> 6, c = (t - OW2) & 63;
        W2b[t - OW2] = f2bf(v);
        W2b[64 * 64 + c * 64 + k] = f2bf(v);
    }
}

__global__ void k_mlp_pack(const float *__restrict__ P, uint16_t *__restrict__ W1t, uint16_t *__restrict__ W2b)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < NP) pack_weight(t, P[t], W1t, W2b);
    if (t < 4 * 64) W1t[(t >> 2) * 16 + 12 + (t & 3)] = 0;   // (no features 12 .. 15)
}

// The end of a step: the rows of the batch's (last) launch added to the gradient
// as in k_grad_sum, the Adam step (bias-corrected) on the FP32 master weights with
// their bf16 copies, the gradient cleared, and the batch's loss (the mean over its
// nb rows, at [NP]) times nb added to the epoch's sum.  One launch where four took
// 20 us a step.  The step number is read from the device (the steps taken before
// the epoch, tstep, and this one's place k in it), so a captured epoch replays
// with the right corrections.
__global__ __launch_bounds__(32 * GS_GROUPS) void k_grad_step(const float *__restrict__ part, int64_t nrows,
                                                              float *__restrict__ P, float *__restrict__ M,
                                                              float *__restrict__ V, float *__restrict__ grad, float lr,
                                                              float b1, float b2, float eps,
                                                              const int64_t *__restrict__ tstep, int k,
                                                              double *__restrict__ lacc, float nb,
                                                              uint16_t *__restrict__ W1t, uint16_t *__restrict__ W2b)
{
    __shared__ float ps[GS_GROUPS][32];
    const int p = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int t = blockIdx.x * 32 + p;
    const float a = grad_rows(part, nrows, t, g, p, ps);
    if (g != 0 || t > NP) return;
    const float gv = grad[t] + a;
    grad[t] = 0.0f;
    if (t == NP) {
        *lacc += (double)gv * (double)nb;
        return;
    }
    const float s = (float)(tstep[0] + k + 1);
    const float c1 = 1.0f - powf(b1, s), c2 = 1.0f - powf(b2, s);
    const float m = b1 * M[t] + (1.0f - b1) * gv, v = b2 * V[t] + (1.0f - b2) * gv * gv;
    M[t] = m;
    V[t] = v;
    const float w = P[t] - lr * (m / c1) / (sqrtf(v / c2) + eps);
    P[t] = w;
    pack_weight(t, w, W1t, W2b);
}

// after an epoch: its steps counted
__global__ void k_steps_taken(int64_t *__restrict__ tstep, int64_t steps)
{
    if (threadIdx.x == 0) *tstep += steps;
}

__global__ void k_step_reset(int64_t *__restrict__ tstep, double *__restrict__ lacc, int steps)
{
    if (threadIdx.x == 0) {
        if (steps) *tstep = 0;
        *lacc = 0.0;
    }
}

__global__ void k_zero_f32(float *p, int64_t n)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) p[t] = 0.0f;
}

}  // namespace

// host launchers (device pointers throughout)
void mlp_pack(const float *P, uint16_t *W1t, uint16_t *W2b, hipStream_t st)
{
    hipLaunchKernelGGL(k_mlp_pack, dim3((NP + 255) / 256), dim3(256), 0, st, P, W1t, W2b);
}

// a grid the device holds at once (two workgroups per CU at these registers), a
// few times over, each wavefront looping over blocks of 64 samples
static unsigned predict_grid(int64_t n)
{
    const int64_t blocks = (n + 63) / 64;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((blocks + PW - 1) / PW, 256 * 2 * 4));
}

void mlp_flag_cells(int64_t nr1, int64_t cb0, int64_t ncells, int64_t vb0, const double2 *verts, const uint16_t *W1t,
                    const uint16_t *W2b, const float *P, float thr, uint64_t *mask, int32_t *cnt, hipStream_t st)
{
    if (ncells > 0)
        hipLaunchKernelGGL(k_mlp_flag_cells, dim3(predict_grid(ncells)), dim3(64 * PW), 0, st, nr1, cb0, ncells, vb0, verts,
                           W1t, W2b + 64 * 64, P, thr, mask, cnt);
}

void mlp_predict(const float *feats, int64_t n, const uint16_t *W1t, const uint16_t *W2b, const float *P,
                 float *logits, hipStream_t st)
{
    if (n > 0)
        hipLaunchKernelGGL(k_mlp_predict, dim3(predict_grid(n)), dim3(64 * PW), 0, st, feats, n, W1t, W2b + 64 * 64, P,
                           logits);
}

int64_t mlp_part_rows(int64_t n) { return (n + MB - 1) / MB * 4; }

void mlp_train_batch(const float *feats, const uint8_t *y, const int64_t *idx, int64_t n, const uint16_t *W1t,
                     const uint16_t *W2b, const float *P, float pos_weight, float norm, float *part, hipStream_t st)
{
    if (n > 0)
        hipLaunchKernelGGL(k_mlp_train, dim3((unsigned)mlp_part_rows(n)), dim3(64), 0, st, feats, y, idx, n, W1t,
                           W2b + 64 * 64, W2b, P, pos_weight, norm, part);
}

void mlp_grad_sum(const float *part, int64_t n, float *grad, hipStream_t st)
{
    if (n > 0)
        hipLaunchKernelGGL(k_grad_sum, dim3((NP + 1 + 31) / 32), dim3(32 * GS_GROUPS), 0, st, part, mlp_part_rows(n), grad);
}

void mlp_grad_step(const float *part, int64_t n, float *P, float *M, float *V, float *grad, float lr,
                   const int64_t *tstep, int k, double *lacc, float nb, uint16_t *W1t, uint16_t *W2b, hipStream_t st)
{
    hipLaunchKernelGGL(k_grad_step, dim3((NP + 1 + 31) / 32), dim3(32 * GS_GROUPS), 0, st, part, mlp_part_rows(n), P, M, V,
                       grad, lr, 0.9f, 0.999f, 1e-8f, tstep, k, lacc, nb, W1t, W2b);
}

void mlp_steps_taken(int64_t *tstep, int64_t steps, hipStream_t st)
{
    hipLaunchKernelGGL(k_steps_taken, dim3(1), dim3(64), 0, st, tstep, steps);
}

void mlp_step_reset(int64_t *tstep, double *lacc, bool steps, hipStream_t st)
{
    hipLaunchKernelGGL(k_step_reset, dim3(1), dim3(64), 0, st, tstep, lacc, steps ? 1 : 0);
}

void mlp_zero(float *p, int64_t n, hipStream_t st)
{
    if (n > 0) hipLaunchKernelGGL(k_zero_f32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
}

}  // namespace mlm
