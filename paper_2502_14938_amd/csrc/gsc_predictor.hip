// Learned reuse predictor (an extension of the reuse decision of Section 4,
// Alg. 1): label generation from the library's own FP32 derivation, and
// training with the library's own forward, backward and Adam kernels.
//
// Network: Linear(6,64) - ReLU - Linear(64,64) - ReLU - Linear(64,1) - sigmoid,
// parameters packed W1[64,6] b1 W2[64,64] b2 W3[1,64] b3.  Loss: mean BCE
// with positive-class weight w:  -(w y log p + (1-y) log(1-p)).
//
//   k_pred_fwdbwd   one lane per unit, two rows per wave: forward,
//                   dLoss/dlogit (/ rows), back-propagated dZ2, dZ1; stores
//                   what the gradient sums read, in the layouts they read
//   k_pred_grads    one wave per column of a gradient, four columns a block: the batch sum of every
//                   parameter's gradient (row order, deterministic) and the
//                   batch loss, then (training) the bias-corrected Adam step
//                   and the BF16 inference copy of that parameter
//   k_pred_infer    BF16 weights and activations, FP32 accumulate (the form
//                   the cache lookup uses)
//   k_pred_labels   compare every candidate's fresh derivation with its line
#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <random>
#include <vector>

#include "gsc_common.h"
#include "gsc_ctx.h"
#include "gsc_derive_mfma.h"
#include "gsc_pred_bf16.h"

namespace gsc {

namespace {

constexpr int NT = 256;
constexpr int P = GSC_PRED_NPARAMS;
constexpr int oW1 = 0, ob1 = 64 * 6, oW2 = ob1 + 64, ob2 = oW2 + 64 * 64, oW3 = ob2 + 64, ob3 = oW3 + 64;
constexpr int kMaxRows = 4096;

__device__ __forceinline__ int64_t gstride() { return (int64_t)gridDim.x * blockDim.x; }
__device__ __forceinline__ int64_t gtid() { return (int64_t)blockIdx.x * blockDim.x + threadIdx.x; }

__device__ __forceinline__ float softplus(float x) { return x > 0.f ? x + log1pf(expf(-x)) : log1pf(expf(x)); }

__device__ __forceinline__ uint16_t to_bf16(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Batch buffers.  The gradient sums run one lane per row of a [rows][64]
// matrix's columns times a vector over the rows, so the matrices are
// row-major and the vectors (the other factor) contiguous over the rows.
struct Work {
    float* XT;   // [6][kMaxRows]
    float* H1T;  // [64][kMaxRows]
    float* H2;   // [B][64]
    float* DZ1;  // [B][64]
    float* DZ2;  // [B][64]
    float* DL;   // [B] dLoss/dlogit (already divided by B)
    float* LS;   // [B] loss terms
};

constexpr int kRowsWave = 2;                      // rows a wave takes together
constexpr int kRowsBlock = kRowsWave * (NT / 64);

// One lane per unit: lane j holds row j of W2 (forward) and column j of W2
// (backward) in registers, and the row's vector comes from LDS, four values
// a read, broadcast to the wave.  A batch of 1,024 rows is then 128 blocks
// of four waves instead of four blocks of one row per lane, whose 64-step
// chains and their scalar weight loads nothing overlapped: 61 -> 8 us.
// Every sum runs in the same order as one thread per row would run it (i
// and j ascending, one FMA each), so splitting the units over the lanes
// changes no result.
__global__ __launch_bounds__(NT) void k_pred_fwdbwd(const float* __restrict__ w, const float* __restrict__ Xin,
                                                    const float* __restrict__ yf, const uint8_t* __restrict__ yb,
                                                    const int32_t* __restrict__ idx, int rows, float pos_weight,
                                                    Work wk) {
    __shared__ __align__(16) float s_x[kRowsBlock][8];
    __shared__ __align__(16) float s_h1[kRowsBlock][kPredW];
    __shared__ float s_h2[kRowsBlock][kPredW + 1];
    __shared__ __align__(16) float s_dz2[kRowsBlock][kPredW];
    __shared__ float s_dl[kRowsBlock];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int row0 = blockIdx.x * kRowsBlock;
    const int nr = rows - row0 < kRowsBlock ? rows - row0 : kRowsBlock;
    if ((int)threadIdx.x < kRowsBlock * 8) {
        const int r = threadIdx.x >> 3, i = threadIdx.x & 7;
        float x = 0.f;
        if (r < nr && i < kPredIn) {
            const int64_t src = idx ? idx[row0 + r] : row0 + r;
            x = Xin[src * kPredIn + i];
        }
        s_x[r][i] = x;
    }
    float w1[kPredIn], w2r[kPredW], w2c[kPredW];
#pragma unroll
    for (int i = 0; i < kPredIn; ++i) w1[i] = w[oW1 + lane * kPredIn + i];
#pragma unroll
    for (int i = 0; i < kPredW; i += 4) {
        const float4 v = *reinterpret_cast<const float4*>(w + oW2 + lane * kPredW + i);
        w2r[i] = v.x; w2r[i + 1] = v.y; w2r[i + 2] = v.z; w2r[i + 3] = v.w;
    }
#pragma unroll
    for (int j = 0; j < kPredW; ++j) w2c[j] = w[oW2 + j * kPredW + lane];
    const float b1 = w[ob1 + lane], b2 = w[ob2 + lane], w3 = w[oW3 + lane];
    __syncthreads();
    const int q0 = wv * kRowsWave;
    float z1[kRowsWave], z2m[kRowsWave];
#pragma unroll
    for (int u = 0; u < kRowsWave; ++u) {
        float a = b1;
#pragma unroll
        for (int i = 0; i < kPredIn; ++i) a = fmaf(w1[i], s_x[q0 + u][i], a);
        z1[u] = a;
        s_h1[q0 + u][lane] = fmaxf(a, 0.f);
    }
    __builtin_amdgcn_wave_barrier();  // the wave reads only its own rows; its LDS accesses complete in order
    {
        float a[kRowsWave];
#pragma unroll
        for (int u = 0; u < kRowsWave; ++u) a[u] = b2;
#pragma unroll
        for (int i = 0; i < kPredW; i += 4)
#pragma unroll
            for (int u = 0; u < kRowsWave; ++u) {
                const float4 h = *reinterpret_cast<const float4*>(&s_h1[q0 + u][i]);
                a[u] = fmaf(w2r[i], h.x, a[u]);
                a[u] = fmaf(w2r[i + 1], h.y, a[u]);
                a[u] = fmaf(w2r[i + 2], h.z, a[u]);
                a[u] = fmaf(w2r[i + 3], h.w, a[u]);
            }
#pragma unroll
        for (int u = 0; u < kRowsWave; ++u) {
            const float h2 = fmaxf(a[u], 0.f);
            z2m[u] = a[u] > 0.f ? 1.f : 0.f;
            s_h2[q0 + u][lane] = h2;
            if (q0 + u < nr) wk.H2[(int64_t)(row0 + q0 + u) * kPredW + lane] = h2;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < nr) {  // one lane per row of the block: the output unit
        const int r = row0 + threadIdx.x;
        float logit = w[ob3];
#pragma unroll 16
        for (int j = 0; j < kPredW; ++j) logit = fmaf(w[oW3 + j], s_h2[threadIdx.x][j], logit);
        const int64_t src = idx ? idx[r] : r;
        const float y = yf ? yf[src] : (float)yb[src];
        const float p = 1.0f / (1.0f + expf(-logit));
        wk.LS[r] = pos_weight * y * softplus(-logit) + (1.0f - y) * softplus(logit);
        const float dl = (pos_weight * y * (p - 1.0f) + (1.0f - y) * p) / (float)rows;
        wk.DL[r] = dl;
        s_dl[threadIdx.x] = dl;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kRowsWave; ++u) {
        const float dz2 = q0 + u < nr ? s_dl[q0 + u] * w3 * z2m[u] : 0.f;
        s_dz2[q0 + u][lane] = dz2;
        if (q0 + u < nr) wk.DZ2[(int64_t)(row0 + q0 + u) * kPredW + lane] = dz2;
    }
    __builtin_amdgcn_wave_barrier();
    {
        float a[kRowsWave];
#pragma unroll
        for (int u = 0; u < kRowsWave; ++u) a[u] = 0.f;
#pragma unroll
        for (int j = 0; j < kPredW; j += 4)
#pragma unroll
            for (int u = 0; u < kRowsWave; ++u) {
                const float4 d = *reinterpret_cast<const float4*>(&s_dz2[q0 + u][j]);
                a[u] = fmaf(w2c[j], d.x, a[u]);
                a[u] = fmaf(w2c[j + 1], d.y, a[u]);
                a[u] = fmaf(w2c[j + 2], d.z, a[u]);
                a[u] = fmaf(w2c[j + 3], d.w, a[u]);
            }
#pragma unroll
        for (int u = 0; u < kRowsWave; ++u)
            if (q0 + u < nr) wk.DZ1[(int64_t)(row0 + q0 + u) * kPredW + lane] = z1[u] > 0.f ? a[u] : 0.f;
    }
    // the transposed factors, the block's rows of a unit side by side
    for (int i = threadIdx.x; i < kPredW * kRowsBlock; i += NT) {
        const int u = i / kRowsBlock, r = i % kRowsBlock;
        if (r < nr) wk.H1T[(int64_t)u * kMaxRows + row0 + r] = s_h1[r][u];
    }
    if ((int)threadIdx.x < kPredIn * kRowsBlock) {
        const int u = threadIdx.x / kRowsBlock, r = threadIdx.x % kRowsBlock;
        if (r < nr) wk.XT[(int64_t)u * kMaxRows + row0 + r] = s_x[r][u];
    }
}

// One parameter's Adam step (bias corrections bc1, bc2) and its BF16 copy.
struct AdamArgs {
    float* w;  // nullptr: gradients only, to `grads`
    float* m;
    float* v;
    uint16_t* wbf;
    float* loss;  // the epoch's loss: set by its first batch, added to by the others
    float lr, bc1, bc2;
    int first;
};

__device__ __forceinline__ void adam_step(const AdamArgs& a, int p, float gi) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float mi = b1 * a.m[p] + (1.f - b1) * gi;
    const float vi = b2 * a.v[p] + (1.f - b2) * gi * gi;
    a.m[p] = mi;
    a.v[p] = vi;
    const float nw = a.w[p] - a.lr * (mi / a.bc1) / (sqrtf(vi / a.bc2) + eps);
    a.w[p] = nw;
    a.wbf[p] = to_bf16(nw);
}

__device__ __forceinline__ float lane_value(float v, int lane) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), lane));
}

// Gradient sums.  A block's four waves take four columns of one gradient:
// column i of W2's is sum over r of DZ2[r][lane] H1[r][i], of W1's DZ1[r][lane]
// X[r][i], of W3's H2[r][lane] DL[r], of b1's and b2's DZ1 and DZ2 themselves;
// one more block sums DL and the losses.  Each parameter's sum keeps the row
// order of a serial loop, a chain of `rows` FMAs that a lane runs at about
// ten cycles a row (the matrix from LDS, the row's factor broadcast from the
// lane that holds it): ~4 us at 1,024 rows, which bounds the kernel beside
// the latency of one chunk's loads.  kGradRows rows of the matrix are staged
// at a time, read as whole lines by all four waves while the chunk before is
// summed.  One thread per parameter with two dependent loads a row, 19
// blocks in all, took 281 us for a batch of 1,024 rows, and the Adam step was
// a kernel of its own (5 us); a wave per column reading its rows itself took
// 27 us (at most 63 loads a wave are in flight); this takes 14.
constexpr int kGradRows = 256;
constexpr int kGradVec = kGradRows * kPredW / 4 / NT;  // 16-byte words a thread stages
constexpr int kGradW2 = kPredW / 4, kGradW1 = (kPredIn + 3) / 4;
constexpr int kGradBlocks = kGradW2 + kGradW1 + 4;     // W3, b1, b2, and the sums over rows alone
static_assert(2 * kMaxRows <= kGradRows * kPredW, "a batch's loss terms fit the staging array");

__global__ __launch_bounds__(NT) void k_pred_grads(Work wk, int rows, float* __restrict__ grads, AdamArgs ad) {
    __shared__ float4 s_m[kGradRows * kPredW / 4];
    const int t = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (t == kGradBlocks - 1) {  // b3 and the loss
        // lane 0 sums dLoss/dlogit, lane 1 the losses, both from LDS (kMaxRows of each fit)
        float* s_dl = reinterpret_cast<float*>(s_m);
        for (int r = threadIdx.x; r < rows; r += NT) {
            s_dl[2 * r] = wk.DL[r];
            s_dl[2 * r + 1] = wk.LS[r];
        }
        __syncthreads();
        if (wv) return;
        float acc = 0.f;
        const float* src = s_dl + (lane & 1);
#pragma unroll 16
        for (int r = 0; r < rows; ++r) acc += src[2 * r];
        const float d = lane_value(acc, 0), l = lane_value(acc, 1);
        const float loss = l / (float)rows;
        if (lane == 0) {
            if (ad.w) {
                adam_step(ad, ob3, d);
                *ad.loss = ad.first ? loss : *ad.loss + loss;
            } else {
                grads[ob3] = d;
                grads[P] = loss;
            }
        }
        return;
    }
    const float* M;
    const float* V = nullptr;  // (none: the matrix alone)
    int p;
    bool mine = true;  // this wave has a column
    if (t < kGradW2) {
        const int i = 4 * t + wv;
        M = wk.DZ2; V = wk.H1T + (int64_t)i * kMaxRows; p = oW2 + lane * kPredW + i;
    } else if (t < kGradW2 + kGradW1) {
        const int i = 4 * (t - kGradW2) + wv;
        mine = i < kPredIn;
        M = wk.DZ1; V = wk.XT + (int64_t)(mine ? i : 0) * kMaxRows; p = oW1 + lane * kPredIn + i;
    } else {
        mine = wv == 0;
        const int q = t - kGradW2 - kGradW1;
        M = q == 0 ? wk.H2 : (q == 1 ? wk.DZ1 : wk.DZ2);
        V = q == 0 ? wk.DL : nullptr;
        p = (q == 0 ? oW3 : (q == 1 ? ob1 : ob2)) + lane;
    }
    const float4* M4 = reinterpret_cast<const float4*>(M);
    const int total = rows * (kPredW / 4);
    float4 nx[kGradVec];
    float vn[kGradRows / 64];
    auto fetch = [&](int r0) {
#pragma unroll
        for (int q = 0; q < kGradVec; ++q) {
            const int i = r0 * (kPredW / 4) + q * NT + (int)threadIdx.x;
            nx[q] = i < total ? M4[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int q = 0; q < kGradRows / 64; ++q) {
            const int r = r0 + q * 64 + lane;
            vn[q] = V ? (r < rows ? V[r] : 0.f) : 1.f;
        }
    };
    float acc = 0.f;
    fetch(0);
    for (int r0 = 0; r0 < rows; r0 += kGradRows) {
        float v[kGradRows / 64];
#pragma unroll
        for (int q = 0; q < kGradVec; ++q) s_m[q * NT + (int)threadIdx.x] = nx[q];
#pragma unroll
        for (int q = 0; q < kGradRows / 64; ++q) v[q] = vn[q];
        __syncthreads();
        if (r0 + kGradRows < rows) fetch(r0 + kGradRows);
        if (mine) {
            const float* m = reinterpret_cast<const float*>(s_m) + lane;
#pragma unroll
            for (int q = 0; q < kGradRows / 64; ++q) {
                const int n = rows - r0 - q * 64;
                if (n >= 64) {
                    // groups of 16 rows: the factors of a group are read
                    // from their lanes together (an FMA right behind its own
                    // v_readlane waits for it), the next group's matrix
                    // values while this group is added
                    float mm[16];
#pragma unroll
                    for (int r = 0; r < 16; ++r) mm[r] = m[(q * 64 + r) * kPredW];
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        float x[16], cur[16];
#pragma unroll
                        for (int r = 0; r < 16; ++r) x[r] = lane_value(v[q], 16 * g + r);
#pragma unroll
                        for (int r = 0; r < 16; ++r) cur[r] = mm[r];
                        if (g < 3) {
#pragma unroll
                            for (int r = 0; r < 16; ++r) mm[r] = m[(q * 64 + 16 * (g + 1) + r) * kPredW];
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc = fmaf(cur[r], x[r], acc);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else if (n > 0) {
#pragma unroll 8
                    for (int r = 0; r < n; ++r) acc = fmaf(m[(q * 64 + r) * kPredW], lane_value(v[q], r), acc);
                }
            }
        }
        __syncthreads();  // the chunk is summed before the next one overwrites it
    }
    if (mine) {
        if (ad.w) adam_step(ad, p, acc);
        else grads[p] = acc;
    }
}

__global__ __launch_bounds__(NT) void k_pred_to_bf16(const float* __restrict__ w, uint16_t* __restrict__ wbf) {
    const int p = (int)gtid();
    if (p < P) wbf[p] = to_bf16(w[p]);
}


// One candidate per lane; the loop is uniform per wave (the predictor runs
// on the whole wave).  Bound by latency (inputs, scalar weights, LDS, matrix
// fragments, one after the other), so four waves a SIMD: 234,567 rows then
// are one round of waves.  15.9 -> 12.7 us.
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_pred_infer(const uint16_t* __restrict__ wb, const float* __restrict__ w32,
                                                   const float* __restrict__ X, int64_t n, float* __restrict__ out) {
    __shared__ uint32_t s_h[NT / 64][kPredLdsWave];
    const int lane = threadIdx.x & 63;
    for (int64_t w0 = gtid() - lane; w0 < n; w0 += gstride()) {
        // (the weights are loaded each time around: hoisted out of the loop,
        // they would take 260 scalar registers and spill)
        asm volatile("" : "+s"(wb), "+s"(w32));
        const int64_t r = w0 + lane;
        float x[kPredIn] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (r < n) {
#pragma unroll
            for (int i = 0; i < kPredIn; ++i) x[i] = X[r * kPredIn + i];
        }
        const float p = pred_prob_bf16_wave(wb, w32, x, s_h[threadIdx.x >> 6]);
        if (r < n) out[r] = p;
    }
}

__global__ __launch_bounds__(NT) void k_iota(int32_t* __restrict__ a, int64_t n) {
    for (int64_t i = gtid(); i < n; i += gstride()) a[i] = (int32_t)i;
}

// Label per candidate: 1 iff its fresh derivation (scratch line i) differs
// from its cached one (line slot_of[anchor]) by more than the thresholds.
// Label of one reuse candidate: 1 (re-derive) when its cached Gaussians have
// drifted visibly from a fresh derivation at this frame.  The drift of one
// Gaussian is the largest of its opacity change, its colour change weighted by
// its opacity, and half the relative change of its covariance (the relative
// change of its footprint radius) weighted by its opacity; the anchor's drift
// (largest over its k Gaussians) times its projected footprint area in pixels,
// max(1, size^2) with size = 2^feature[5] the projected voxel size, must stay
// below the change of a 4x4-pixel patch by one 8-bit level (16/255).
__global__ __launch_bounds__(NT) void k_pred_labels(const int32_t* __restrict__ cand, const int32_t* __restrict__ slot_of,
                                                    const Counters* cnt, int k, const float* __restrict__ feat,
                                                    const float4* __restrict__ F0, const float4* __restrict__ F1,
                                                    const float4* __restrict__ F2, const float* __restrict__ F3,
                                                    const float4* __restrict__ C0, const float4* __restrict__ C1,
                                                    const float4* __restrict__ C2, const float* __restrict__ C3,
                                                    uint8_t* __restrict__ y) {
    const int64_t n = cnt->n_cand;
    for (int64_t i = gtid(); i < n; i += gstride()) {
        const int64_t line = slot_of[cand[i]];
        if (line < 0) {
            y[i] = 1;
            continue;
        }
        float drift = 0.f;
        for (int j = 0; j < k; ++j) {
            const int64_t f = i * k + j, c = line * k + j;
            const float4 a0 = F0[f], a1 = F1[f], a2 = F2[f];
            const float a3 = F3[f];
            const float4 b0 = C0[c], b1 = C1[c], b2 = C2[c];
            const float b3 = C3[c];
            const float dc = fmaxf(fabsf(a2.z - b2.z), fmaxf(fabsf(a2.w - b2.w), fabsf(a3 - b3)));
            const float sa[6] = {a1.x, a1.y, a1.z, a1.w, a2.x, a2.y};
            const float sb[6] = {b1.x, b1.y, b1.z, b1.w, b2.x, b2.y};
            float dmax = 0.f, smax = 0.f;
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                dmax = fmaxf(dmax, fabsf(sa[q] - sb[q]));
                smax = fmaxf(smax, fabsf(sa[q]));
            }
            const float geo = smax > 0.f ? dmax / smax : (dmax > 0.f ? INFINITY : 0.f);
            const float am = fmaxf(fabsf(a0.w), fabsf(b0.w));
            drift = fmaxf(drift, fmaxf(fabsf(a0.w - b0.w), am * fmaxf(dc, 0.5f * geo)));
        }
        const float size = exp2f(feat[i * kPredIn + 5]);
        y[i] = drift * fmaxf(1.f, size * size) > 16.0f / 255.0f ? 1 : 0;
    }
}

int fail(gsc_ctx* c, int code, const char* msg) {
    c->err = msg;
    return code;
}

hipError_t ensure_pred(gsc_ctx* c) {
    if (c->pred_w) return hipSuccess;
    size_t b = 0;
    hipError_t e;
    if ((e = dalloc(c->pmem, b, &c->pred_w, P)) != hipSuccess || (e = dalloc(c->pmem, b, &c->pred_wbf, P)) != hipSuccess ||
        (e = dalloc(c->pmem, b, &c->pred_m, P)) != hipSuccess || (e = dalloc(c->pmem, b, &c->pred_v, P)) != hipSuccess ||
        (e = dalloc(c->pmem, b, &c->pred_g, P + 1)) != hipSuccess ||
        (e = dalloc(c->pmem, b, &c->pred_work, (size_t)kMaxRows * (kPredIn + 4 * kPredW + 2))) != hipSuccess) {
        return e;
    }
    return hipSuccess;
}

Work work_of(gsc_ctx* c) {
    Work w;
    float* p = c->pred_work;
    w.XT = p; p += (size_t)kMaxRows * kPredIn;
    w.H1T = p; p += (size_t)kMaxRows * kPredW;
    w.H2 = p; p += (size_t)kMaxRows * kPredW;
    w.DZ1 = p; p += (size_t)kMaxRows * kPredW;
    w.DZ2 = p; p += (size_t)kMaxRows * kPredW;
    w.DL = p; p += kMaxRows;
    w.LS = p;
    return w;
}

inline unsigned batch_blocks(int rows) { return (unsigned)((rows + kRowsBlock - 1) / kRowsBlock); }
inline unsigned blocks_for(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + NT - 1) / NT, kGridBlocks)); }

}  // namespace

void pred_free(gsc_ctx* c) {
    free_labels(c);
    if (c->pmem.empty()) return;
    (void)hipStreamSynchronize(c->stream);
    c->pmem.release();
    c->pred_w = nullptr;
    c->pred_wbf = nullptr;
    c->pred_m = c->pred_v = c->pred_g = c->pred_work = nullptr;
    c->pred_loaded = false;
}

}  // namespace gsc

using namespace gsc;

extern "C" {

int gsc_predictor_load(gsc_ctx* c, const float* params, int64_t n) {
    if (!c || !params) return c ? fail(c, GSC_E_INVALID_ARG, "gsc_predictor_load: null argument") : GSC_E_INVALID_ARG;
    if (n != P) return fail(c, GSC_E_INVALID_ARG, "gsc_predictor_load: wrong parameter count");
    if (ensure_pred(c) != hipSuccess) return fail(c, GSC_E_OOM, "gsc_predictor_load: device allocation");
    if (hipMemcpyAsync(c->pred_w, params, P * 4, hipMemcpyHostToDevice, c->stream) != hipSuccess ||
        hipMemsetAsync(c->pred_m, 0, P * 4, c->stream) != hipSuccess ||
        hipMemsetAsync(c->pred_v, 0, P * 4, c->stream) != hipSuccess)
        return fail(c, GSC_E_HIP, "gsc_predictor_load: copy failed");
    hipLaunchKernelGGL(k_pred_to_bf16, dim3(blocks_for(P)), dim3(NT), 0, c->stream, c->pred_w, c->pred_wbf);
    if (hipStreamSynchronize(c->stream) != hipSuccess) return fail(c, GSC_E_HIP, "gsc_predictor_load: sync failed");
    c->pred_step = 0;
    c->pred_loaded = true;
    return GSC_OK;
}

int gsc_predictor_get(gsc_ctx* c, float* params, int64_t n) {
    if (!c || !params) return c ? fail(c, GSC_E_INVALID_ARG, "gsc_predictor_get: null argument") : GSC_E_INVALID_ARG;
    if (n != P) return fail(c, GSC_E_INVALID_ARG, "gsc_predictor_get: wrong parameter count");
    if (!c->pred_loaded) return fail(c, GSC_E_NOT_LOADED, "gsc_predictor_get: no predictor loaded");
    if (hipStreamSynchronize(c->stream) != hipSuccess ||
        hipMemcpy(params, c->pred_w, P * 4, hipMemcpyDeviceToHost) != hipSuccess)
        return fail(c, GSC_E_HIP, "gsc_predictor_get: copy failed");
    return GSC_OK;
}

int gsc_predictor_collect(gsc_ctx* c, int enable) {
    if (!c) return GSC_E_INVALID_ARG;
    c->collect_features = enable ? 1 : 0;
    return GSC_OK;
}

int gsc_predictor_labels(gsc_ctx* c, float* X_out, uint8_t* y_out, int32_t* ids_out, int64_t cap, int64_t* n) {
    if (!c || !n) return c ? fail(c, GSC_E_INVALID_ARG, "gsc_predictor_labels: null argument") : GSC_E_INVALID_ARG;
    if (cap > 0 && (!X_out || !y_out)) return fail(c, GSC_E_INVALID_ARG, "gsc_predictor_labels: null output");
    if (!c->loaded || !c->derived || !c->collect_features)
        return fail(c, GSC_E_NOT_LOADED, "gsc_predictor_labels: needs a gsc_derive with collection enabled");
    if (!(c->cfg.flags & GSC_FLAG_REUSE) || c->nviews != 1)
        return fail(c, GSC_E_INVALID_ARG, "gsc_predictor_labels: needs reuse on and de-redundancy on");
    View& v = c->view[0];
    const Scene& sc = c->scene;
    hipStream_t st = c->stream;
    const int64_t E = sc.n * sc.k;
    if (c->lab_entries < E) {  // scratch lines for fresh derivations of the candidates
        free_labels(c);
        size_t b = 0;
        hipError_t e;
        if ((e = dalloc(c->lmem, b, &c->lab_L0, E)) != hipSuccess || (e = dalloc(c->lmem, b, &c->lab_L1, E)) != hipSuccess ||
            (e = dalloc(c->lmem, b, &c->lab_L2, E)) != hipSuccess || (e = dalloc(c->lmem, b, &c->lab_L3, E)) != hipSuccess ||
            (e = dalloc(c->lmem, b, &c->lab_iota, sc.n)) != hipSuccess || (e = dalloc(c->lmem, b, &c->lab_y, sc.n)) != hipSuccess) {
            free_labels(c);
            return fail(c, GSC_E_OOM, "gsc_predictor_labels: device allocation");
        }
        c->lab_entries = E;
        hipLaunchKernelGGL(k_iota, dim3(blocks_for(sc.n)), dim3(NT), 0, st, c->lab_iota, sc.n);
    }
    // derive every candidate again with this frame's unified camera, FP32
    MfmaDeriveArgs m;
    m.posr = sc.posr; m.feat = sc.feat; m.scale = sc.scale; m.offsets = sc.offsets; m.k = sc.k;
    MfmaView& mv = m.v[0];
    mv.visible = v.cand_id; mv.misses = c->lab_iota; mv.vslot = c->lab_iota;
    mv.L0 = c->lab_L0; mv.L1 = c->lab_L1; mv.L2 = c->lab_L2; mv.L3 = c->lab_L3; mv.line_mask = nullptr;
    for (int i = 0; i < 3; ++i) mv.cam_pos[i] = (float)c->unified.pos[i];
    m.inv_dist_unit = sc.dist_unit > 0.f ? 1.0f / sc.dist_unit : 0.f;
    mv.n_miss = &v.cnt->n_cand; m.mode = GSC_PREC_F32;
    m.fr.l1_f32 = sc.fr_l1_f32; m.fr.l2_f32 = sc.fr_l2_f32; m.fr.l1_bf16 = sc.fr_l1_bf16;
    m.fr.l2_bf16 = sc.fr_l2_bf16; m.fr.l1_fp8 = sc.fr_l1_fp8; m.fr.l2_fp8 = sc.fr_l2_fp8;
    m.fr.b1 = sc.fr_b1; m.fr.b2 = sc.fr_b2; m.fr.s1 = sc.fr_s1; m.fr.s2 = sc.fr_s2;
    m.fr.n_at = sc.n_at; m.fr.n_ct = sc.n_ct; m.fr.n_vt = sc.n_vt;
    if (derive_mfma(m, 1, sc.n, st) != hipSuccess) return fail(c, GSC_E_HIP, "gsc_predictor_labels: derive failed");
    hipLaunchKernelGGL(k_pred_labels, dim3(blocks_for(sc.n)), dim3(NT), 0, st, v.cand_id, v.slot_of, v.cnt, sc.k,
                       v.cand_feat, c->lab_L0, c->lab_L1, c->lab_L2, c->lab_L3, v.L0, v.L1, v.L2, v.L3, c->lab_y);
    if (hipStreamSynchronize(st) != hipSuccess) return fail(c, GSC_E_HIP, "gsc_predictor_labels: kernels failed");
    Counters k;
    if (hipMemcpy(&k, v.cnt, sizeof(k), hipMemcpyDeviceToHost) != hipSuccess)
        return fail(c, GSC_E_HIP, "gsc_predictor_labels: copy failed");
    *n = k.n_cand;
    const int64_t m_out = std::min<int64_t>(cap, k.n_cand);
    if (m_out > 0 && (hipMemcpy(X_out, v.cand_feat, m_out * kPredIn * 4, hipMemcpyDeviceToHost) != hipSuccess ||
                      hipMemcpy(y_out, c->lab_y, m_out, hipMemcpyDeviceToHost) != hipSuccess))
        return fail(c, GSC_E_HIP, "gsc_predictor_labels: copy failed");
    if (m_out > 0 && ids_out && hipMemcpy(ids_out, v.cand_id, m_out * 4, hipMemcpyDeviceToHost) != hipSuccess)
        return fail(c, GSC_E_HIP, "gsc_predictor_labels: copy failed");
    return GSC_OK;
}

int gsc_predictor_grad(gsc_ctx* c, const float* X, const float* y, int64_t n, float pos_weight, float* grads_out,
                       float* loss_out) {
    if (!c || !X || !y || !grads_out) return c ? fail(c, GSC_E_INVALID_ARG, "gsc_predictor_grad: null argument")
                                               : GSC_E_INVALID_ARG;
    if (n < 1 || n > kMaxRows) return fail(c, GSC_E_INVALID_ARG, "gsc_predictor_grad: n must be in [1, 4096]");
    if (!c->pred_loaded) return fail(c, GSC_E_NOT_LOADED, "gsc_predictor_grad: no predictor loaded");
    Work wk = work_of(c);
    hipLaunchKernelGGL(k_pred_fwdbwd, dim3(batch_blocks((int)n)), dim3(NT), 0, c->stream, c->pred_w, X, y, nullptr,
                       nullptr, (int)n, pos_weight, wk);
    hipLaunchKernelGGL(k_pred_grads, dim3(kGradBlocks), dim3(NT), 0, c->stream, wk, (int)n, c->pred_g, AdamArgs{});
    std::vector<float> g(P + 1);
    if (hipStreamSynchronize(c->stream) != hipSuccess ||
        hipMemcpy(g.data(), c->pred_g, (P + 1) * 4, hipMemcpyDeviceToHost) != hipSuccess)
        return fail(c, GSC_E_HIP, "gsc_predictor_grad: kernels failed");
    std::memcpy(grads_out, g.data(), P * 4);
    if (loss_out) *loss_out = g[P];
    return GSC_OK;
}

int gsc_predictor_train(gsc_ctx* c, const float* X, const uint8_t* y, int64_t n, int32_t batch, int32_t epochs,
                        float lr, float pos_weight, uint64_t seed, float* loss_out) {
    if (!c || !X || !y) return c ? fail(c, GSC_E_INVALID_ARG, "gsc_predictor_train: null argument") : GSC_E_INVALID_ARG;
    if (n < 1 || batch < 1 || batch > kMaxRows || epochs < 1 || !(lr > 0.f))
        return fail(c, GSC_E_INVALID_ARG, "gsc_predictor_train: bad sizes");
    if (!c->pred_loaded) return fail(c, GSC_E_NOT_LOADED, "gsc_predictor_train: load initial weights first");
    hipStream_t st = c->stream;
    // device copies of the rows, two permutations (device and pinned) and
    // the epochs' losses: the host shuffles the next epoch's order while the
    // device trains on this one's, and waits only at the end
    AllocSet tmp;
    size_t acct = 0;
    float* dX = nullptr;
    uint8_t* dy = nullptr;
    float* dloss = nullptr;
    int32_t* dperm[2] = {nullptr, nullptr};
    int32_t* hperm = nullptr;
    if (dalloc(tmp, acct, &dX, n * kPredIn) != hipSuccess || dalloc(tmp, acct, &dy, n) != hipSuccess ||
        dalloc(tmp, acct, &dloss, epochs) != hipSuccess || dalloc(tmp, acct, &dperm[0], n) != hipSuccess ||
        dalloc(tmp, acct, &dperm[1], n) != hipSuccess || halloc(tmp, &hperm, 2 * n) != hipSuccess) {
        tmp.release();
        return fail(c, GSC_E_OOM, "gsc_predictor_train: device allocation");
    }
    hipEvent_t copied[2] = {nullptr, nullptr};
    int rc = GSC_OK;
    for (int i = 0; i < 2 && rc == GSC_OK; ++i)
        if (hipEventCreateWithFlags(&copied[i], hipEventDisableTiming) != hipSuccess)
            rc = fail(c, GSC_E_HIP, "gsc_predictor_train: event creation");
    std::vector<int32_t> perm(n);
    std::iota(perm.begin(), perm.end(), 0);
    std::mt19937_64 rng(seed);
    Work wk = work_of(c);
    if (rc == GSC_OK && (hipMemcpyAsync(dX, X, n * kPredIn * 4, hipMemcpyHostToDevice, st) != hipSuccess ||
                         hipMemcpyAsync(dy, y, n, hipMemcpyHostToDevice, st) != hipSuccess))
        rc = fail(c, GSC_E_HIP, "gsc_predictor_train: upload failed");
    for (int ep = 0; ep < epochs && rc == GSC_OK; ++ep) {
        std::shuffle(perm.begin(), perm.end(), rng);
        const int set = ep & 1;
        int32_t* hp = hperm + (int64_t)set * n;
        // (the pinned half was last read by the copy of two epochs back)
        if (ep >= 2 && hipEventSynchronize(copied[set]) != hipSuccess) {
            rc = fail(c, GSC_E_HIP, "gsc_predictor_train: training kernels failed");
            break;
        }
        std::memcpy(hp, perm.data(), n * 4);
        if (hipMemcpyAsync(dperm[set], hp, n * 4, hipMemcpyHostToDevice, st) != hipSuccess ||
            hipEventRecord(copied[set], st) != hipSuccess) {
            rc = fail(c, GSC_E_HIP, "gsc_predictor_train: upload failed");
            break;
        }
        for (int64_t b0 = 0; b0 < n; b0 += batch) {
            const int rows = (int)std::min<int64_t>(batch, n - b0);
            hipLaunchKernelGGL(k_pred_fwdbwd, dim3(batch_blocks(rows)), dim3(NT), 0, st, c->pred_w, dX, nullptr, dy,
                               dperm[set] + b0, rows, pos_weight, wk);
            c->pred_step += 1;
            AdamArgs ad;
            ad.w = c->pred_w; ad.m = c->pred_m; ad.v = c->pred_v; ad.wbf = c->pred_wbf;
            ad.loss = dloss + ep; ad.first = b0 == 0 ? 1 : 0;
            ad.lr = lr;
            ad.bc1 = 1.0f - (float)std::pow(0.9, c->pred_step);
            ad.bc2 = 1.0f - (float)std::pow(0.999, c->pred_step);
            hipLaunchKernelGGL(k_pred_grads, dim3(kGradBlocks), dim3(NT), 0, st, wk, rows, c->pred_g, ad);
        }
    }
    if (rc == GSC_OK && (hipGetLastError() != hipSuccess || hipStreamSynchronize(st) != hipSuccess ||
                         (loss_out && hipMemcpy(loss_out, dloss, (size_t)epochs * 4, hipMemcpyDeviceToHost) != hipSuccess)))
        rc = fail(c, GSC_E_HIP, "gsc_predictor_train: training kernels failed");
    if (rc == GSC_OK && loss_out) {
        const int nb = (int)((n + batch - 1) / batch);
        for (int ep = 0; ep < epochs; ++ep) loss_out[ep] /= (float)nb;
    }
    (void)hipStreamSynchronize(st);
    for (int i = 0; i < 2; ++i)
        if (copied[i]) (void)hipEventDestroy(copied[i]);
    tmp.release();
    return rc;
}

int gsc_predictor_infer(gsc_ctx* c, const float* X, int64_t n, float* p_out) {
    if (!c || !X || !p_out) return c ? fail(c, GSC_E_INVALID_ARG, "gsc_predictor_infer: null argument")
                                     : GSC_E_INVALID_ARG;
    if (n < 0) return fail(c, GSC_E_INVALID_ARG, "gsc_predictor_infer: negative n");
    if (!c->pred_loaded) return fail(c, GSC_E_NOT_LOADED, "gsc_predictor_infer: no predictor loaded");
    if (n == 0) return GSC_OK;
    hipLaunchKernelGGL(k_pred_infer, dim3(blocks_for(n)), dim3(NT), 0, c->stream, c->pred_wbf, c->pred_w, X, n, p_out);
    if (hipGetLastError() != hipSuccess) return fail(c, GSC_E_HIP, "gsc_predictor_infer: launch failed");
    return GSC_OK;
}

}  // extern "C"
