// Derive stage of one frame of one viewer, or of a batch of viewers at once
// (Section 4, Alg. 1):
//   anchor indexing + filtering  -> k_select, k_visible (X_t, ascending)
//   cache scheduling             -> k_cache_* (invalidate at the reuse depth,
//                                   hit/miss, learned staleness, slot
//                                   allocation, eviction of outdated lines)
//   decode new anchors           -> derive_mfma (eq. 3, eq. 2; matrix cores)
//   configure the cache depth    -> depth_update (eq. 4, linear guide), in k_compose_reduce
//   update the render buffer     -> k_compose_* (opacity mask, Section 6)
// Every count stays on the device (Counters); the host only enqueues.
//
// Frames of a few thousand anchors and batches of viewers are bound by the
// launches (4 to 5 us each, whatever they do), so the flags of a compaction
// are made by the kernel that also adds them up, the compaction writes what
// the next stage starts from, and the kernels take a grid row per view:
// without a cache 5 launches in place of 7, with one line per anchor 6 in
// place of 9, and for eight viewers 6 in place of 72.
#include <cmath>

#include "gsc_blockscan.h"
#include "gsc_common.h"
#include "gsc_derive_mfma.h"
#include "gsc_pred_bf16.h"

namespace gsc {

namespace {

constexpr int NT = 256;

__device__ __forceinline__ int64_t gstride() { return (int64_t)gridDim.x * blockDim.x; }
__device__ __forceinline__ int64_t gtid() { return (int64_t)blockIdx.x * blockDim.x + threadIdx.x; }

// Per-frame counters reset, and the unified camera centre of frame t kept
// for the reuse features of later frames (run by the first block of the
// selection kernel).
__device__ __forceinline__ void frame_begin(Counters* cnt, float* pu_hist, int32_t t, const DeriveCam& cam) {
    if (threadIdx.x == 0) {
        cnt->n_cand = 0;
        cnt->overflow = 0;
        cnt->n_evict = 0;
        cnt->evict_short = 0;
    }
    if (threadIdx.x < 3) pu_hist[4 * (t & 63) + threadIdx.x] = cam.pos[threadIdx.x];
}

// ------------------------------------------------------------- selection
// Keep anchor a iff (level 0 or |x - p_u| <= d_ref 2^-level, or < 2 d_ref
// 2^-level with the fractional level transition) and its bounding sphere is
// not wholly outside any unified-frustum plane (4 sides + near).
// Direct-mapped cache (line_anchor non-null: line a can only hold anchor a):
// the invalidation of Alg. 1 is done here too, anchor a's line dropped when
// its age exceeds the current depth (the depth is the previous frame's
// update; starting the frame leaves it alone).

// What the kernels of the stage need of one view.
struct ViewStage {
    DeriveCam cam;
    Counters* cnt;
    float* pu_hist;
    int32_t *slot_of, *line_anchor, *line_tau, *line_last;
    int32_t *visible, *vslot, *misses;
    uint64_t* bits;   // a flag per anchor, then per visible position (64 to a word)
    uint32_t* sums;   // the flags' sum per block
    const uint16_t* line_mask;
    int32_t* G;
    int32_t t;
};
// the sums of the misses without a line, of the free lines, and of the lines at
// the eviction's threshold lie behind them
constexpr int kNeedSums = kScanBlocks, kFreeSums = 2 * kScanBlocks, kThrSums = 3 * kScanBlocks;
template <int V>
struct Views {
    ViewStage v[V];  // blockIdx.y: view
};

// Sum of the block's waves' counts, one value per wave (all its lanes alike).
__device__ __forceinline__ uint32_t waves_sum(uint32_t count, uint32_t* wsum) {
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = count;
    __syncthreads();
    uint32_t t = 0;
    for (int i = 0; i < NT / 64; ++i) t += wsum[i];
    return t;
}

// Signed distance of an anchor from a plane, n.x + w, its fused products
// written out (from n_x x or from n_y y on): the set of visible anchors does
// not depend on which ones the compiler would fuse.
__device__ __forceinline__ float plane_side(const float (&q)[4], const float4& p, bool from_x) {
#pragma clang fp contract(off)
    const float s = from_x ? fmaf(q[1], p.y, q[0] * p.x) : fmaf(q[0], p.x, q[1] * p.y);
    return fmaf(q[2], p.z, s) + q[3];
}

// Does anchor position p (bounding radius in w) at level l stay?
__device__ __forceinline__ bool keep_anchor(const DeriveCam& cam, const float4& p, int l) {
    bool keep = true;
    if (l != 0) {
        float vx = p.x - cam.pos[0], vy = p.y - cam.pos[1], vz = p.z - cam.pos[2];
        float lim = ldexpf(cam.d_ref, -l);
        float d2 = fmaf(vz, vz, fmaf(vx, vx, vy * vy));
        // with the fractional transition a level stays until its weight
        // clamp(2 - dist / d_l, 0, 1) reaches 0 (the weight is applied
        // by the rasteriser's preprocess)
        keep = cam.fade ? d2 < 4.f * lim * lim : d2 <= lim * lim;
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) keep = keep && (plane_side(cam.planes[i], p, i & 1) >= -p.w);
    return keep;
}

constexpr int kSelStep = 1024;  // anchors a block tests at a time, four per thread with their loads together

template <int V>
__global__ __launch_bounds__(NT) void k_select(Views<V> vs, const float4* __restrict__ posr,
                                               const uint8_t* __restrict__ level, int64_t n, int direct) {
    __shared__ uint32_t wsum[NT / 64];
    const ViewStage& v = vs.v[V == 1 ? 0 : blockIdx.y];
    if (blockIdx.x == 0) frame_begin(v.cnt, v.pu_hist, v.t, v.cam);
    const DeriveCam& cam = v.cam;
    const int32_t depth = v.cnt->depth, t = v.t;
    int64_t b0, b1;
    blockscan::chunk_of(n, kSelStep, b0, b1);
    uint32_t count = 0;
    for (int64_t base = b0; base < b1; base += kSelStep) {
        float4 pos[4];
        int lev[4], owner[4], tau[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t a = base + u * NT + threadIdx.x, at = a < n ? a : n - 1;
            pos[u] = posr[at];
            lev[u] = level[at];
            owner[u] = direct ? v.line_anchor[at] : -1;
            tau[u] = direct ? v.line_tau[at] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t a = base + u * NT + threadIdx.x;
            if (a < n && owner[u] >= 0 && t - tau[u] > depth) {
                v.slot_of[a] = -1;
                v.line_anchor[a] = -1;
            }
            const bool keep = a < n && keep_anchor(cam, pos[u], lev[u]);
            const uint64_t m = __ballot(keep);
            if ((threadIdx.x & 63) == 0 && a < b1) v.bits[a >> 6] = m;
            count += (uint32_t)__popcll(m);
        }
    }
    const uint32_t total = waves_sum(count, wsum);
    if (threadIdx.x == 0) v.sums[blockIdx.x] = total;
}

// A scene of at most kOneBlock anchors takes one block for the selection and
// one for the composition, each with its scan inside: two launches of 3.5 us
// less of the small stereo frame's 90.
constexpr int kOneBlock = 4096;
constexpr int NO = 1024;

// Exclusive prefix of v over the block of NO threads from carry on, which
// becomes the carry after them.
__device__ __forceinline__ uint32_t one_block_scan(uint32_t v, uint32_t& carry, uint32_t* wsum) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    uint32_t before = carry, all = carry;
    for (int i = 0; i < NO / 64; ++i) {
        before += i < w ? wsum[i] : 0u;
        all += wsum[i];
    }
    __syncthreads();
    carry = all;
    return before + x - v;
}

// k_select and k_visible of a small scene.
template <int V, bool kNoCache>
__global__ __launch_bounds__(NO) void k_select_small(Views<V> vs, const float4* __restrict__ posr,
                                                     const uint8_t* __restrict__ level, int n, int direct) {
    __shared__ uint32_t wsum[NO / 64];
    const ViewStage& v = vs.v[V == 1 ? 0 : blockIdx.y];
    frame_begin(v.cnt, v.pu_hist, v.t, v.cam);
    const int32_t depth = v.cnt->depth;
    uint32_t carry = 0;
    for (int base = 0; base < n; base += NO) {
        const int a = base + threadIdx.x;
        bool keep = false;
        if (a < n) {
            if (direct && v.line_anchor[a] >= 0 && v.t - v.line_tau[a] > depth) {
                v.slot_of[a] = -1;
                v.line_anchor[a] = -1;
            }
            keep = keep_anchor(v.cam, posr[a], level[a]);
        }
        const uint32_t e = one_block_scan(keep ? 1u : 0u, carry, wsum);
        if (keep) {
            v.visible[e] = a;
            if (kNoCache) {
                v.misses[e] = (int32_t)e;
                v.vslot[e] = (int32_t)e;
                v.line_anchor[e] = a;
            }
        }
    }
    if (threadIdx.x == 0) {
        v.cnt->n_visible = (int32_t)carry;
        if (kNoCache) v.cnt->n_miss = (int32_t)carry;
    }
}

// X_t from the flags, ascending.  Without a cache every visible anchor is a
// miss derived into line i, its visible position.
template <int V, bool kNoCache>
__global__ __launch_bounds__(NT) void k_visible(Views<V> vs, int64_t n) {
    __shared__ uint32_t wsum[NT / 64];
    const ViewStage& v = vs.v[V == 1 ? 0 : blockIdx.y];
    uint32_t carry = blockscan::block_carry(v.sums, wsum, &v.cnt->n_visible);
    if (kNoCache && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
        v.cnt->n_miss = (int32_t)(carry + v.sums[blockIdx.x]);
    int64_t b0, b1;
    blockscan::chunk_of(n, kSelStep, b0, b1);
    for (int64_t base = b0; base < b1; base += kSelStep) {
        const int64_t i0 = base + threadIdx.x * 4;
        const uint32_t f = i0 < b1 ? (uint32_t)(v.bits[i0 >> 6] >> (i0 & 63)) & 15u : 0u;
        uint32_t tot;
        uint32_t e = carry + blockscan::block_excl_scan((uint32_t)__popc(f), wsum, tot);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (!(f >> u & 1u)) continue;
            v.visible[e] = (int32_t)(i0 + u);
            if (kNoCache) {
                v.misses[e] = (int32_t)e;
                v.vslot[e] = (int32_t)e;
                v.line_anchor[e] = (int32_t)(i0 + u);
            }
            ++e;
        }
        carry += tot;
    }
}

// ------------------------------------------------------------- cache

// The free lines as flags (64 to a word) and their sum per block, from what
// each line's `free_line` says; all threads of the block take part.
template <class Fn>
__device__ __forceinline__ void free_flags(int64_t C, uint64_t* bits, uint32_t* sums, uint32_t* wsum, Fn&& free_line) {
    int64_t b0, b1;
    blockscan::chunk_of(C, kSelStep, b0, b1);
    uint32_t count = 0;
    for (int64_t base = b0; base < b1; base += NT) {
        const int64_t s = base + threadIdx.x;
        const uint64_t m = __ballot(s < b1 && free_line(s));
        if ((threadIdx.x & 63) == 0 && s < b1) bits[s >> 6] = m;
        count += (uint32_t)__popcll(m);
    }
    const uint32_t total = waves_sum(count, wsum);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// Alg. 1: invalidate every line whose age exceeds the current depth; flags the
// free lines and clears the eviction's histogram.
__global__ __launch_bounds__(NT) void k_cache_invalidate(int32_t* __restrict__ line_anchor, const int32_t* __restrict__ tau,
                                                         int32_t* __restrict__ slot_of, int64_t C, int32_t t,
                                                         Counters* cnt, uint32_t* __restrict__ evict_hist,
                                                         uint64_t* __restrict__ bits, uint32_t* __restrict__ sums) {
    __shared__ uint32_t wsum[NT / 64];
    const int32_t d = cnt->depth;
    if (blockIdx.x == 0 && threadIdx.x < 64) evict_hist[threadIdx.x] = 0u;
    free_flags(C, bits, sums, wsum, [&](int64_t s) {
        const int32_t a = line_anchor[s];
        if (a < 0) return true;
        if (t - tau[s] <= d) return false;
        slot_of[a] = -1;
        line_anchor[s] = -1;
        return true;
    });
}

// Learned staleness (reuse predictor): features of one candidate.
__device__ __forceinline__ void reuse_features(float4 p, int lvl, int lmax, const float* sc, const float* pu_now,
                                               const float* pu_then, int age, int dmax, float fx, float* f) {
    float vn[3] = {p.x - pu_now[0], p.y - pu_now[1], p.z - pu_now[2]};
    float vt[3] = {p.x - pu_then[0], p.y - pu_then[1], p.z - pu_then[2]};
    float dn = sqrtf(vn[0] * vn[0] + vn[1] * vn[1] + vn[2] * vn[2]);
    float dt = sqrtf(vt[0] * vt[0] + vt[1] * vt[1] + vt[2] * vt[2]);
    float c = (vn[0] * vt[0] + vn[1] * vt[1] + vn[2] * vt[2]) / (dn * dt);
    float du[3] = {pu_now[0] - pu_then[0], pu_now[1] - pu_then[1], pu_now[2] - pu_then[2]};
    float smax = fmaxf(sc[0], fmaxf(sc[1], sc[2]));
    f[0] = 1.0f - c;
    f[1] = logf(dn / dt);
    f[2] = (float)age / (float)dmax;
    f[3] = (float)lvl / (float)(lmax > 0 ? lmax : 1);
    f[4] = sqrtf(du[0] * du[0] + du[1] * du[1] + du[2] * du[2]) / dn;
    f[5] = log2f(smax * fx / dn);
}


struct LookupArgs {
    int32_t predictor;
    float thr;
    const float4* posr;
    const uint8_t* level;
    const float* scale;
    int32_t lmax, dmax;
    const uint16_t* pred_wbf;
    const float* pred_w32;
    float* cand_feat;      // optional: features of candidates (for label collection; one view)
    int32_t* cand_id;
    // direct-mapped cache: a miss takes line aid here, and every visible
    // anchor's render-buffer line is its own id
    int32_t direct;
};

// Direct-mapped lines, used when there is a line for every anchor: anchor a
// owns line a.  Free lines can then never run short, so there is no free
// list and no eviction, and the hit/miss decisions are the same as with any
// other choice of free line.  Misses (re)take their line at frame t (here,
// in the lookup); every visible anchor's buffer position points at its own
// line.
//
// Hit iff the anchor still owns a line (after invalidation every owned line
// has 1 <= t - tau <= d_t), reuse is on and the predictor does not flag it.
// Every visible owned line is stamped last_used = t.  The loop is uniform
// per wave: the predictor runs on the whole wave (matrix cores) whenever one
// of its lanes has a candidate.
// (at most 128 VGPRs: four waves per SIMD.  The lookup with the predictor in
// views high above the city took 25 us with three, 21 with four)
template <int V>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_cache_lookup(Views<V> vs, LookupArgs a) {
    __shared__ uint32_t s_h[NT / 64][kPredLdsWave];
    __shared__ uint32_t wsum[NT / 64];
    const ViewStage& v = vs.v[V == 1 ? 0 : blockIdx.y];
    const int32_t nv = v.cnt->n_visible, t = v.t;
    int64_t b0, b1;
    blockscan::chunk_of(nv, NT, b0, b1);
    uint32_t count = 0, need = 0;  // misses, and those without a line
    for (int64_t base = b0; base < b1; base += NT) {
        const int64_t i = base + threadIdx.x;
        const bool valid = i < nv;
        bool hit = false;
        float f[kPredIn] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        int32_t aid = 0, s = -1;
        if (valid) {
            aid = v.visible[i];
            s = v.slot_of[aid];
            hit = s >= 0;
            if (s >= 0) v.line_last[s] = t;
            if (hit && (a.predictor || a.cand_feat)) {
                const int32_t tau = v.line_tau[s];
                reuse_features(a.posr[aid], a.level[aid], a.lmax, a.scale + 6 * (int64_t)aid, v.cam.pos,
                               v.pu_hist + 4 * (tau & 63), t - tau, a.dmax, v.cam.fx, f);
                if (a.cand_feat) {
                    const int32_t c = atomicAdd(&v.cnt->n_cand, 1);
                    for (int q = 0; q < kPredIn; ++q) a.cand_feat[(int64_t)c * kPredIn + q] = f[q];
                    a.cand_id[c] = aid;
                }
            }
        }
        if (a.predictor && __any(hit)) {
            const float p = pred_prob_bf16_wave(a.pred_wbf, a.pred_w32, f, s_h[threadIdx.x >> 6]);
            if (hit && p > a.thr) hit = false;
        }
        const uint64_t m = __ballot(valid && !hit);
        if ((threadIdx.x & 63) == 0 && valid) v.bits[i >> 6] = m;
        count += (uint32_t)__popcll(m);
        need += (uint32_t)__popcll(__ballot(valid && !hit && s < 0));
        if (valid) v.vslot[i] = a.direct ? aid : s;  // (-1: k_assign finds it a line)
        if (valid && a.direct) {
            if (!hit) {  // derived this frame into line aid
                if (s < 0) {
                    v.slot_of[aid] = aid;
                    v.line_anchor[aid] = aid;
                    v.line_last[aid] = t;
                }
                v.line_tau[aid] = t;
            }
        }
    }
    const uint32_t total = waves_sum(count, wsum);
    if (threadIdx.x == 0) v.sums[blockIdx.x] = total;
    if (a.direct) return;
    __syncthreads();
    const uint32_t need_total = waves_sum(need, wsum);
    if (threadIdx.x == 0) v.sums[kNeedSums + blockIdx.x] = need_total;
}

// Misses, ascending visible position (= ascending anchor id).  With fewer
// lines than anchors (need_rank) also the rank of each miss that owns no line
// among those (kOwnsLine: it does), and the number of free lines.
constexpr uint32_t kOwnsLine = 0xffffffffu;
template <int V>
__global__ __launch_bounds__(NT) void k_misses(Views<V> vs, uint32_t* __restrict__ need_rank, int free_blocks) {
    __shared__ uint32_t wsum[NT / 64];
    const ViewStage& v = vs.v[V == 1 ? 0 : blockIdx.y];
    uint32_t carry = blockscan::block_carry(v.sums, wsum, &v.cnt->n_miss), carry2 = 0;
    if (need_rank) {
        carry2 = blockscan::block_carry(v.sums + kNeedSums, wsum, &v.cnt->n_need);
        if (blockIdx.x == 0) {
            uint32_t n = 0;
            for (int i = threadIdx.x; i < free_blocks; i += NT) n += v.sums[kFreeSums + i];
            n = blockscan::block_sum(n, wsum);
            if (threadIdx.x == 0) v.cnt->n_free = (int32_t)n;
        }
    }
    int64_t b0, b1;
    blockscan::chunk_of(v.cnt->n_visible, NT, b0, b1);
    for (int64_t base = b0; base < b1; base += NT) {
        const int64_t i = base + threadIdx.x;
        const uint32_t f = i < b1 ? (uint32_t)(v.bits[i >> 6] >> (i & 63)) & 1u : 0u;
        uint32_t tot;
        const uint32_t e = carry + blockscan::block_excl_scan(f, wsum, tot);
        if (f) v.misses[e] = (int32_t)i;
        carry += tot;
        if (!need_rank) continue;  // (block-uniform)
        const uint32_t need = f && v.vslot[i] < 0 ? 1u : 0u;
        const uint32_t rank = carry2 + blockscan::block_excl_scan(need, wsum, tot);
        if (f) need_rank[e] = need ? rank : kOwnsLine;
        carry2 += tot;
    }
}

// Eviction plan: lines not visible now (last_used < t) are candidates; take
// them in ascending (last_used, anchor).  last_used of a surviving line lies
// in [t - d_max, t - 1], so a d_max-bin histogram finds the threshold bin.
__global__ __launch_bounds__(NT) void k_evict_hist(const int32_t* __restrict__ line_anchor,
                                                   const int32_t* __restrict__ line_last, int64_t C, int32_t t,
                                                   int32_t dmax, Counters* cnt, uint32_t* __restrict__ hist) {
    if (cnt->n_need - cnt->n_free <= 0) return;
    __shared__ uint32_t h[64];
    if (threadIdx.x < 64) h[threadIdx.x] = 0u;
    __syncthreads();
    for (int64_t s = gtid(); s < C; s += gstride()) {
        int32_t lu = line_last[s];
        if (line_anchor[s] >= 0 && lu < t) {
            int b = lu - (t - dmax);
            b = b < 0 ? 0 : b;
            atomicAdd(&h[b], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < dmax && h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
}

// The plan (run by every block of the flags' kernel; the first one stores it).
struct EvictPlan {
    int32_t thr, left, n_evict, short_of;
    bool over;
};
__device__ __forceinline__ EvictPlan evict_plan(const uint32_t* hist, int32_t t, int32_t dmax, int32_t shortfall) {
    EvictPlan p{t, 0, 0, shortfall > 0 ? shortfall : 0, false};
    if (shortfall <= 0) return p;
    int32_t acc = 0;
    for (int b = 0; b < dmax; ++b) {
        int32_t h = (int32_t)hist[b];
        if (acc + h >= shortfall) {
            p.thr = (t - dmax) + b;
            p.left = shortfall - acc;
            p.n_evict = shortfall;
            return p;
        }
        acc += h;
    }
    p.over = true;  // fewer evictable lines than needed: evict every candidate
    p.n_evict = acc;
    return p;
}

// Anchors (ascending id) whose line sits in the threshold bin: flags and sums.
__global__ __launch_bounds__(NT) void k_evict_thr_flags(const int32_t* __restrict__ slot_of,
                                                        const int32_t* __restrict__ line_last,
                                                        const uint32_t* __restrict__ hist, int32_t t, int32_t dmax,
                                                        int64_t n, Counters* cnt, uint64_t* __restrict__ bits,
                                                        uint32_t* __restrict__ sums) {
    __shared__ uint32_t h[64];
    __shared__ uint32_t wsum[NT / 64];
    __shared__ EvictPlan s_plan;
    if (threadIdx.x < 64) h[threadIdx.x] = hist[threadIdx.x];
    __syncthreads();
    if (threadIdx.x == 0) s_plan = evict_plan(h, t, dmax, cnt->n_need - cnt->n_free);
    __syncthreads();
    const EvictPlan p = s_plan;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        cnt->evict_short = p.short_of;
        cnt->n_evict = p.n_evict;
        if (p.short_of > 0) {
            cnt->evict_thr = p.thr;
            cnt->evict_left = p.left;
        }
        if (p.over) cnt->overflow |= 2;  // the frame is marked overflowed
    }
    if (p.left <= 0) return;  // nothing evicted, or every candidate
    free_flags(n, bits, sums, wsum, [&](int64_t a) {
        const int32_t s = slot_of[a];
        return s >= 0 && line_last[s] == p.thr;
    });
}

// Evicts the lines of the anchors (ascending id) that the plan takes: those
// last used before the threshold, and the first `left` at it.
__global__ __launch_bounds__(NT) void k_evict_apply(int32_t* __restrict__ line_anchor, const int32_t* __restrict__ line_last,
                                                    int32_t* __restrict__ slot_of, const uint64_t* __restrict__ bits,
                                                    const uint32_t* __restrict__ sums, int64_t n, int32_t t, Counters* cnt) {
    __shared__ uint32_t wsum[NT / 64];
    if (cnt->evict_short <= 0) return;
    const int32_t thr = cnt->evict_thr, left = cnt->evict_left;
    uint32_t carry = left > 0 ? blockscan::block_carry<uint32_t>(sums, wsum) : 0u;
    int64_t b0, b1;
    blockscan::chunk_of(n, kSelStep, b0, b1);
    for (int64_t base = b0; base < b1; base += NT) {
        const int64_t a = base + threadIdx.x;
        const uint32_t at = left > 0 && a < b1 ? (uint32_t)(bits[a >> 6] >> (a & 63)) & 1u : 0u;
        uint32_t tot;
        const uint32_t rank = carry + blockscan::block_excl_scan(at, wsum, tot);
        carry += tot;
        const int32_t s = a < b1 ? slot_of[a] : -1;
        if (s < 0) continue;
        const int32_t lu = line_last[s];
        if (lu < t && (lu < thr || (at && (int32_t)rank < left))) {
            slot_of[a] = -1;
            line_anchor[s] = -1;
        }
    }
}

// The free lines again, if anything was evicted.
__global__ __launch_bounds__(NT) void k_free_flags(const int32_t* __restrict__ line_anchor, int64_t C, const Counters* cnt,
                                                   uint64_t* __restrict__ bits, uint32_t* __restrict__ sums) {
    __shared__ uint32_t wsum[NT / 64];
    if (cnt->evict_short <= 0) return;
    free_flags(C, bits, sums, wsum, [&](int64_t s) { return line_anchor[s] < 0; });
}

// And listed, ascending.
__global__ __launch_bounds__(NT) void k_free_list(const uint64_t* __restrict__ bits, const uint32_t* __restrict__ sums,
                                                  int64_t C, int32_t* __restrict__ free_list) {
    __shared__ uint32_t wsum[NT / 64];
    uint32_t carry = blockscan::block_carry<uint32_t>(sums, wsum);
    int64_t b0, b1;
    blockscan::chunk_of(C, kSelStep, b0, b1);
    for (int64_t base = b0; base < b1; base += kSelStep) {
        const int64_t i0 = base + threadIdx.x * 4;
        const uint32_t f = i0 < b1 ? (uint32_t)(bits[i0 >> 6] >> (i0 & 63)) & 15u : 0u;
        uint32_t tot;
        uint32_t e = carry + blockscan::block_excl_scan((uint32_t)__popc(f), wsum, tot);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (f >> u & 1u) free_list[e++] = (int32_t)(i0 + u);
        carry += tot;
    }
}

// Misses without a line take free lines in ascending order; every miss is
// re-derived now (tau = t).
__global__ __launch_bounds__(NT) void k_assign(const int32_t* __restrict__ misses, const int32_t* __restrict__ visible,
                                               int32_t* __restrict__ slot_of, int32_t* __restrict__ line_anchor,
                                               int32_t* __restrict__ line_tau, int32_t* __restrict__ line_last,
                                               const uint32_t* __restrict__ need_rank,
                                               const int32_t* __restrict__ free_list, int32_t t, int64_t C,
                                               Counters* cnt, int32_t* __restrict__ vslot) {
    int32_t nm = cnt->n_miss;
    for (int64_t j = gtid(); j < nm; j += gstride()) {
        int32_t aid = visible[misses[j]];
        int32_t s;
        const uint32_t r = need_rank[j];
        if (r != kOwnsLine) {
            if ((int64_t)r >= C || r >= (uint32_t)max(cnt->n_free + cnt->n_evict, 0)) {
                atomicOr(&cnt->overflow, 2);
                continue;
            }
            s = free_list[r];
            slot_of[aid] = s;
            line_anchor[s] = aid;
            line_last[s] = t;
            vslot[misses[j]] = s;
        } else {
            s = slot_of[aid];
        }
        line_tau[s] = t;
    }
}


// Eq. 4 with the linear guiding function on the update (miss) rate.
__device__ __forceinline__ void depth_update(Counters* cnt, int32_t dmax, int32_t guide) {
    int32_t nx = cnt->n_visible, nm = cnt->n_miss;
    cnt->depth_used = cnt->depth;
    if (guide == GSC_GUIDE_FIXED) {
        cnt->depth = dmax;
        return;
    }
    if (nx <= 0) return;
    int64_t d;
    if (guide == GSC_GUIDE_EXP) {
        const int64_t q = (8ll * nm) / nx;  // eighths of update rate
        d = q >= 31 ? 0 : ((int64_t)dmax >> q);
    } else if (guide == GSC_GUIDE_STAGED) {
        d = 8ll * nm < nx ? dmax : (8ll * nm < 3ll * nx ? dmax / 2 : 1);
    } else {  // linear: round_half_up(d_max (1 - r))
        d = (2ll * dmax * (nx - nm) + nx) / (2ll * nx);
    }
    cnt->depth = (int32_t)(d < 1 ? 1 : (d > dmax ? dmax : d));
}




// ------------------------------------------------------------- compose
// G_t = [(i, j) : i visible ascending, j ascending, alpha_ij > 0]; each entry
// is the cache entry (line * k + j).
static_assert(NT == blockscan::kThreads, "the fused compose scan uses the block-scan shape");

// Composition of the render buffer as one fused scan: visible anchor i
// contributes the Gaussians of its line whose opacity is positive (the
// line's mask, set by the derivation; none for an anchor left without a line
// at a capacity overflow), written to G in visible order at the exclusive
// prefix of the contributions.  The reduce pass sums each block's chunk and
// runs the depth update (eq. 4) from this frame's counts; the down-sweep
// writes the ids.
__device__ __forceinline__ uint32_t compose_mask(const int32_t* __restrict__ vslot,
                                                 const uint16_t* __restrict__ line_mask, int64_t i, int32_t& slot) {
    slot = vslot[i];
    return slot < 0 ? 0u : (uint32_t)line_mask[slot];
}

template <int V>
__global__ __launch_bounds__(NT) void k_compose_reduce(Views<V> vs, int32_t dmax, int32_t guide) {
    __shared__ uint32_t wsum[NT / 64];
    const ViewStage& v = vs.v[V == 1 ? 0 : blockIdx.y];
    if (gtid() == 0) depth_update(v.cnt, dmax, guide);  // eq. 4, from this frame's counts
    int64_t b0, b1;
    blockscan::chunk_of(v.cnt->n_visible, NT, b0, b1);
    uint32_t s = 0;
    for (int64_t i = b0 + threadIdx.x; i < b1; i += NT) {
        int32_t slot;
        s += (uint32_t)__popc(compose_mask(v.vslot, v.line_mask, i, slot));
    }
    const uint32_t t = blockscan::block_sum(s, wsum);
    if (threadIdx.x == 0) v.sums[blockIdx.x] = t;
}

template <int V>
__global__ __launch_bounds__(NT) void k_compose_scatter(Views<V> vs, int k) {
    __shared__ uint32_t wsum[NT / 64];
    const ViewStage& v = vs.v[V == 1 ? 0 : blockIdx.y];
    uint32_t carry = blockscan::block_carry(v.sums, wsum, &v.cnt->n_gauss);
    int64_t b0, b1;
    blockscan::chunk_of(v.cnt->n_visible, NT, b0, b1);
    for (int64_t base = b0; base < b1; base += NT) {
        const int64_t i = base + threadIdx.x;
        int32_t slot = -1;
        uint32_t m = i < b1 ? compose_mask(v.vslot, v.line_mask, i, slot) : 0u;
        uint32_t tot;
        uint32_t o = carry + blockscan::block_excl_scan((uint32_t)__popc(m), wsum, tot);
        const int64_t gb = (int64_t)slot * k;
        while (m) {
            const int j = __ffs(m) - 1;
            m &= m - 1u;
            v.G[o++] = (int32_t)(gb + j);
        }
        carry += tot;
    }
}

// k_compose_reduce and k_compose_scatter of a small scene.
template <int V>
__global__ __launch_bounds__(NO) void k_compose_small(Views<V> vs, int k, int32_t dmax, int32_t guide) {
    __shared__ uint32_t wsum[NO / 64];
    const ViewStage& v = vs.v[V == 1 ? 0 : blockIdx.y];
    if (threadIdx.x == 0) depth_update(v.cnt, dmax, guide);  // eq. 4, from this frame's counts
    const int nv = v.cnt->n_visible;
    uint32_t carry = 0;
    for (int base = 0; base < nv; base += NO) {
        const int i = base + threadIdx.x;
        int32_t slot = -1;
        uint32_t m = i < nv ? compose_mask(v.vslot, v.line_mask, i, slot) : 0u;
        uint32_t o = one_block_scan((uint32_t)__popc(m), carry, wsum);
        const int64_t gb = (int64_t)slot * k;
        while (m) {
            const int j = __ffs(m) - 1;
            m &= m - 1u;
            v.G[o++] = (int32_t)(gb + j);
        }
    }
    if (threadIdx.x == 0) v.cnt->n_gauss = (int32_t)carry;
}

}  // namespace

#define GSC_TRY(x)                              \
    do {                                        \
        hipError_t e_ = (x);                    \
        if (e_ != hipSuccess) return e_;        \
    } while (0)

namespace {

ViewStage view_stage(const DeriveArgs& a) {
    View& v = *a.v;
    ViewStage s;
    s.cam = a.cam; s.cnt = v.cnt; s.pu_hist = v.pu_hist; s.slot_of = v.slot_of; s.line_anchor = v.line_anchor;
    s.line_tau = v.line_tau; s.line_last = v.line_last; s.visible = v.visible; s.vslot = v.vslot; s.misses = v.misses;
    s.bits = reinterpret_cast<uint64_t*>(v.tmp_a); s.sums = v.block_sums; s.line_mask = v.line_mask; s.G = v.G;
    s.t = (int32_t)v.t;
    return s;
}

// The derive stage of nv views (V = 1 or kMaxViews): all of them without a
// cache, or with one line per anchor, or a single one.
template <int V>
hipError_t derive_stage(const DeriveArgs* views, int nv, hipStream_t st, Marks* mk) {
    const DeriveArgs& a = views[0];
    const Scene& sc = *a.sc;
    View& v = *a.v;
    const int64_t n = sc.n;
    const int32_t t = (int32_t)v.t;
    Counters* cnt = v.cnt;
    Views<V> vs;
    for (int i = 0; i < V; ++i) vs.v[i] = view_stage(views[i < nv ? i : 0]);
    mark(mk, 0, st);
    // anchor indexing and filtering -> X_t ascending (the first block also
    // starts the frame's counters)
    const bool reuse = (a.flags & GSC_FLAG_REUSE) != 0;
    const bool direct = reuse && v.C >= n;  // line a holds anchor a or nothing
    // a block per step of anchors (of visible ones), up to the sums' number
    auto blocks = [&](int step) {
        const int64_t b = (n + step - 1) / step;
        return dim3((unsigned)(b < kScanBlocks ? b : kScanBlocks), (unsigned)nv);
    };
    const bool small = n <= kOneBlock;
    const dim3 one(1, (unsigned)nv);
    if (small && !reuse) {
        hipLaunchKernelGGL((k_select_small<V, true>), one, dim3(NO), 0, st, vs, sc.posr, sc.level, (int)n, 0);
    } else if (small) {
        hipLaunchKernelGGL((k_select_small<V, false>), one, dim3(NO), 0, st, vs, sc.posr, sc.level, (int)n, direct ? 1 : 0);
    } else {
        hipLaunchKernelGGL(k_select<V>, blocks(kSelStep), dim3(NT), 0, st, vs, sc.posr, sc.level, n, direct ? 1 : 0);
        if (reuse) hipLaunchKernelGGL((k_visible<V, false>), blocks(kSelStep), dim3(NT), 0, st, vs, n);
        else hipLaunchKernelGGL((k_visible<V, true>), blocks(kSelStep), dim3(NT), 0, st, vs, n);
    }
    if (reuse) {
        const int64_t C = v.C;
        // free lines and eviction flags of a cache with fewer lines than anchors
        uint64_t* fbits = reinterpret_cast<uint64_t*>(v.tmp_c);
        uint64_t* tbits = reinterpret_cast<uint64_t*>(v.tmp_d);
        const int64_t cb = (C + kSelStep - 1) / kSelStep;
        const dim3 cblocks((unsigned)(cb < kScanBlocks ? cb : kScanBlocks));
        if (!direct)  // (direct: done in k_select)
            hipLaunchKernelGGL(k_cache_invalidate, cblocks, dim3(NT), 0, st, v.line_anchor, v.line_tau, v.slot_of, C, t, cnt,
                               v.evict_hist, fbits, v.block_sums + kFreeSums);
        LookupArgs la;
        la.predictor = (a.flags & GSC_FLAG_PREDICTOR) ? 1 : 0;
        la.thr = a.pred_thr; la.posr = sc.posr; la.level = sc.level; la.scale = sc.scale;
        la.lmax = sc.l_max; la.dmax = a.d_max; la.pred_wbf = a.pred_wbf; la.pred_w32 = a.pred_w;
        la.cand_feat = a.collect ? v.cand_feat : nullptr; la.cand_id = v.cand_id;
        la.direct = direct ? 1 : 0;
        hipLaunchKernelGGL(k_cache_lookup<V>, blocks(NT), dim3(NT), 0, st, vs, la);
        hipLaunchKernelGGL(k_misses<V>, blocks(NT), dim3(NT), 0, st, vs, direct ? nullptr : v.tmp_b, (int)cblocks.x);
        if (!direct) {
            // eviction of outdated lines when free lines are short
            const dim3 nblocks(blocks(kSelStep).x);
            hipLaunchKernelGGL(k_evict_hist, grid_fit(k_evict_hist, C), dim3(NT), 0, st, v.line_anchor, v.line_last, C, t, a.d_max,
                               cnt, v.evict_hist);
            hipLaunchKernelGGL(k_evict_thr_flags, nblocks, dim3(NT), 0, st, v.slot_of, v.line_last, v.evict_hist, t, a.d_max, n,
                               cnt, tbits, v.block_sums + kThrSums);
            hipLaunchKernelGGL(k_evict_apply, nblocks, dim3(NT), 0, st, v.line_anchor, v.line_last, v.slot_of, tbits,
                               v.block_sums + kThrSums, n, t, cnt);
            hipLaunchKernelGGL(k_free_flags, cblocks, dim3(NT), 0, st, v.line_anchor, C, cnt, fbits, v.block_sums + kFreeSums);
            hipLaunchKernelGGL(k_free_list, cblocks, dim3(NT), 0, st, fbits, v.block_sums + kFreeSums, C, v.free_list);
            hipLaunchKernelGGL(k_assign, grid_fit(k_assign, n), dim3(NT), 0, st, v.misses, v.visible, v.slot_of, v.line_anchor,
                               v.line_tau, v.line_last, v.tmp_b, v.free_list, t, C, cnt, v.vslot);
        }
    }
    // decode the misses on the matrix cores
    mark(mk, 1, st);
    {
        MfmaDeriveArgs m;
        m.posr = sc.posr; m.feat = sc.feat; m.scale = sc.scale; m.offsets = sc.offsets; m.k = sc.k;
        for (int i = 0; i < nv; ++i) m.v[i] = derive_view(*views[i].v, views[i].cam.pos);
        m.inv_dist_unit = sc.dist_unit > 0.f ? 1.0f / sc.dist_unit : 0.f;
        m.mode = a.precision;
        m.fr.l1_f32 = sc.fr_l1_f32; m.fr.l2_f32 = sc.fr_l2_f32; m.fr.l1_bf16 = sc.fr_l1_bf16;
        m.fr.l2_bf16 = sc.fr_l2_bf16; m.fr.l1_fp8 = sc.fr_l1_fp8; m.fr.l2_fp8 = sc.fr_l2_fp8;
        m.fr.b1 = sc.fr_b1; m.fr.b2 = sc.fr_b2; m.fr.s1 = sc.fr_s1; m.fr.s2 = sc.fr_s2;
        m.fr.n_at = sc.n_at; m.fr.n_ct = sc.n_ct; m.fr.n_vt = sc.n_vt;
        GSC_TRY(derive_mfma(m, nv, n, st));
    }
    mark(mk, 2, st);
    // compose the render buffer
    if (small) {
        hipLaunchKernelGGL(k_compose_small<V>, one, dim3(NO), 0, st, vs, sc.k, a.d_max, a.guide);
    } else {
        hipLaunchKernelGGL(k_compose_reduce<V>, blocks(NT), dim3(NT), 0, st, vs, a.d_max, a.guide);
        hipLaunchKernelGGL(k_compose_scatter<V>, blocks(NT), dim3(NT), 0, st, vs, sc.k);
    }
    mark(mk, 3, st);
    return hipGetLastError();
}

}  // namespace

hipError_t derive_frame(const DeriveArgs& a, hipStream_t st, Marks* mk) { return derive_stage<1>(&a, 1, st, mk); }

hipError_t derive_batch(const DeriveArgs* a, int n, hipStream_t st) {
    // views with fewer lines than anchors go one by one (their eviction plan
    // has a kernel per step and view)
    bool together = n > 1 && n <= kMaxViews;
    for (int i = 0; i < n; ++i) together = together && (!(a[i].flags & GSC_FLAG_REUSE) || a[i].v->C >= a[i].sc->n);
    if (together) return derive_stage<kMaxViews>(a, n, st, nullptr);
    for (int i = 0; i < n; ++i) GSC_TRY(derive_stage<1>(a + i, 1, st, nullptr));
    return hipSuccess;
}

}  // namespace gsc
