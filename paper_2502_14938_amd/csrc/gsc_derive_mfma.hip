// Derivation of missed anchors on the matrix cores (Section 3.1 eq. 3; the
// AnchorDecoder of Section 6: the anchor row is read once for all k offsets,
// both MLP layers run back to back without leaving registers, and every
// output attribute is written straight into its cache array).
//
// One wave handles 16 anchors.  Layer 1 is computed transposed,
// H^T[96 x 16] = W1[96 x 35] Z^T[35 x 16], so that each 16x16 output tile is
// already laid out as the B operand of layer 2, O^T = W2 H^T.  The 110
// outputs of the anchor (alpha k, colour 3k, covariance 7k) land in LDS and
// an epilogue turns them into the k Gaussians (activations, quaternion,
// Sigma = R S S^T R^T (eq. 2), mean = x + s * O_j).
//
// MODE GSC_PREC_F32: v_mfma_f32_16x16x4f32 (FP32 operands, FP32 accumulate).
// MODE GSC_PREC_BF16: v_mfma_f32_16x16x16bf16_1k, inputs and hidden
//   activations rounded to bfloat16 (nearest even), FP32 accumulate.
// MODE GSC_PREC_FP8: as BF16 with e4m3fn weights (exact in bfloat16) and a
//   per-output-row FP32 scale applied to the accumulator.
//
// What bounds it: per tile of 16 anchors (k = 10) 118 F32 matrix instructions
// of 32 cycles and some 1,400 vector instructions, most of them the
// epilogue's exponentials and divisions: 21 and 32 us of issue for the city's
// 217,503 anchors, 34 us of memory traffic, and before that the latency of
// loads that depend on each other (list of misses, anchor, its row).  So each
// wave asks for the next tile's row and the anchors of the one after while it
// computes, for the next output tile's weights while the matrix cores work on
// one, and for the next step's shape in the epilogue; the waves share nothing
// but the layer-1 weights and never wait for each other; and eight waves a
// block with one copy of those weights and outputs packed to 11 k words let
// 16 waves live on a CU (12 with the weights in registers).  City: 140 ->
// 85 us, 62,281 anchors 53 -> 26 us, 2,000 anchors 19 -> 11 us; BF16, the
// city's 34,246 misses 30 -> 23 us.
#include <cmath>
#include <cstring>

#include "gsc_derive_mfma.h"

namespace gsc {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));

constexpr int NT = 512;          // 8 waves share the layer-1 weights in LDS
constexpr int kMaxBlocks = 512;  // two per CU: 4 waves per SIMD

uint16_t h_bf16(float x) {
    uint32_t u;
    std::memcpy(&u, &x, 4);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

float h_from_bf16(uint16_t h) {
    uint32_t u = (uint32_t)h << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}

// e4m3fn value nearest to x (ties to even), saturating at 448.
double h_e4m3(double x) {
    if (x == 0.0) return 0.0;
    double a = std::fabs(x), r;
    if (a < std::ldexp(1.0, -6)) {
        r = std::nearbyint(a / std::ldexp(1.0, -9)) * std::ldexp(1.0, -9);
    } else {
        int e;
        std::frexp(a, &e);
        double q = std::ldexp(1.0, e - 4);
        r = std::nearbyint(a / q) * q;
    }
    if (r > 448.0) r = 448.0;
    return x < 0 ? -r : r;
}

// Four floats as bfloat16 (nearest even).
__device__ __forceinline__ shortx4 d_bf16x4(float a, float b, float c, float d) {
    const uint2 v = make_uint2(bf16_pair(a, b), bf16_pair(c, d));
    return __builtin_bit_cast(shortx4, v);
}

__device__ __forceinline__ float sigm(float x) { return 1.0f / (1.0f + expf(-x)); }

}  // namespace

HostFrags pack_frags(const gsc_mlp& mlp, int k, int n_in) {
    HostFrags f;
    const int c[3] = {1, 3, 7};
    f.n_at = (k + 15) / 16;
    f.n_ct = (3 * k + 15) / 16;
    f.n_vt = (7 * k + 15) / 16;
    const int nt = f.n_at + f.n_ct + f.n_vt;
    const int tile0[3] = {0, f.n_at, f.n_at + f.n_ct};
    // layer 1, padded [96][48]; scales per hidden row
    std::vector<double> W1p(96 * 48, 0.0), q1(96 * 48, 0.0);
    f.b1.assign(96, 0.f);
    f.s1.assign(96, 1.f);
    for (int h = 0; h < 3; ++h)
        for (int r = 0; r < 32; ++r) {
            int row = h * 32 + r;
            double amax = 0.0;
            for (int q = 0; q < n_in; ++q) {
                W1p[row * 48 + q] = mlp.W1[h][r * n_in + q];
                amax = std::fmax(amax, std::fabs(W1p[row * 48 + q]));
            }
            double s = amax > 0.0 ? amax / 448.0 : 1.0;
            f.s1[row] = (float)s;
            for (int q = 0; q < n_in; ++q) q1[row * 48 + q] = h_e4m3(W1p[row * 48 + q] / s);
            f.b1[row] = mlp.b1[h][r];
        }
    // layer 2, padded [16 nt][32] per tile's head
    std::vector<double> W2p(16 * nt * 32, 0.0), q2(16 * nt * 32, 0.0);
    f.b2.assign(16 * nt, 0.f);
    f.s2.assign(16 * nt, 1.f);
    for (int h = 0; h < 3; ++h)
        for (int o = 0; o < c[h] * k; ++o) {
            int row = 16 * tile0[h] + o;
            double amax = 0.0;
            for (int q = 0; q < 32; ++q) {
                W2p[row * 32 + q] = mlp.W2[h][o * 32 + q];
                amax = std::fmax(amax, std::fabs(W2p[row * 32 + q]));
            }
            double s = amax > 0.0 ? amax / 448.0 : 1.0;
            f.s2[row] = (float)s;
            for (int q = 0; q < 32; ++q) q2[row * 32 + q] = h_e4m3(W2p[row * 32 + q] / s);
            f.b2[row] = mlp.b2[h][o];
        }
    // F32 fragments
    f.l1_f32.assign(14 * 64 * 4, 0.f);
    for (int hb = 0; hb < 6; ++hb)
        for (int ks = 0; ks < 9; ++ks)
            for (int l = 0; l < 64; ++l) {
                int row = hb * 16 + (l & 15), col = 4 * ks + (l >> 4);
                const int i = ks * 6 + hb;
                f.l1_f32[((i >> 2) * 64 + l) * 4 + (i & 3)] = col < n_in ? (float)W1p[row * 48 + col] : 0.f;
            }
    f.l2_f32.assign(nt * 2 * 4 * 64, 0.f);
    for (int ot = 0; ot < nt; ++ot)
        for (int hb2 = 0; hb2 < 2; ++hb2)
            for (int s = 0; s < 4; ++s)
                for (int l = 0; l < 64; ++l) {
                    int row = ot * 16 + (l & 15), col = 16 * hb2 + 4 * (l >> 4) + s;
                    f.l2_f32[((ot * 2 + hb2) * 64 + l) * 4 + s] = (float)W2p[row * 32 + col];
                }
    // BF16 / FP8 fragments: 4 consecutive k per lane
    f.l1_bf16.assign(6 * 3 * 64 * 4, 0);
    f.l1_fp8.assign(6 * 3 * 64 * 4, 0);
    for (int hb = 0; hb < 6; ++hb)
        for (int kb = 0; kb < 3; ++kb)
            for (int l = 0; l < 64; ++l)
                for (int i = 0; i < 4; ++i) {
                    int row = hb * 16 + (l & 15), col = 16 * kb + 4 * (l >> 4) + i;
                    const int at2 = kb * 6 + hb;
                    size_t at = ((size_t)(at2 >> 1) * 64 + l) * 8 + 4 * (at2 & 1) + i;
                    f.l1_bf16[at] = h_bf16((float)W1p[row * 48 + col]);
                    f.l1_fp8[at] = h_bf16((float)q1[row * 48 + col]);
                }
    f.l2_bf16.assign(nt * 2 * 64 * 4, 0);
    f.l2_fp8.assign(nt * 2 * 64 * 4, 0);
    for (int ot = 0; ot < nt; ++ot)
        for (int kb = 0; kb < 2; ++kb)
            for (int l = 0; l < 64; ++l)
                for (int i = 0; i < 4; ++i) {
                    int row = ot * 16 + (l & 15), col = 16 * kb + 4 * (l >> 4) + i;
                    size_t at = ((size_t)ot * 64 + l) * 8 + 4 * kb + i;
                    f.l2_bf16[at] = h_bf16((float)W2p[row * 32 + col]);
                    f.l2_fp8[at] = h_bf16((float)q2[row * 32 + col]);
                }
    (void)h_from_bf16;
    return f;
}

namespace {

// Four bf16 operands of 16-byte word v: its low or high half.
__device__ __forceinline__ shortx4 half_of(const uint4& v, int half) {
    const uint32_t a = half ? v.z : v.x, b = half ? v.w : v.y;
    return shortx4{(short)(a & 0xffff), (short)(a >> 16), (short)(b & 0xffff), (short)(b >> 16)};
}

// A wave's layer-2 operands of one output tile: 8 (F32) or 2 x 4 (BF16) weights
// per lane and the bias of its four rows.
template <int MODE>
struct OutTile {
    uint4 w[MODE == GSC_PREC_F32 ? 2 : 1];
    float4 b;
};
template <int MODE>
__device__ __forceinline__ OutTile<MODE> load_out_tile(const MfmaFrags& fr, int ot, int lane) {
    OutTile<MODE> t;
    if (MODE == GSC_PREC_F32) {
        t.w[0] = reinterpret_cast<const uint4*>(fr.l2_f32)[(ot * 2) * 64 + lane];
        t.w[MODE == GSC_PREC_F32 ? 1 : 0] = reinterpret_cast<const uint4*>(fr.l2_f32)[(ot * 2 + 1) * 64 + lane];
    } else {
        t.w[0] = reinterpret_cast<const uint4*>(MODE == GSC_PREC_BF16 ? fr.l2_bf16 : fr.l2_fp8)[ot * 64 + lane];
    }
    t.b = reinterpret_cast<const float4*>(fr.b2)[ot * 4 + (lane >> 4)];
    return t;
}
__device__ __forceinline__ float comp(const float4& v, int i) {
    return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w));
}

// A lane's share of the layer-1 operands of its column's anchor: in F32 the
// inputs 4 s + q of steps s, else the eight features of its two k-blocks; and
// the anchor's position.
struct Inputs {
    float z[8];
    float4 x;
};
template <int MODE>
__device__ __forceinline__ Inputs load_inputs(const MfmaDeriveArgs& a, int32_t aid, int q) {
    Inputs v;
    const float* f = a.feat + (int64_t)aid * kF;
    if (MODE == GSC_PREC_F32) {
#pragma unroll
        for (int s = 0; s < 8; ++s) v.z[s] = f[4 * s + q];
    } else {
        const float4 lo = reinterpret_cast<const float4*>(f)[q], hi = reinterpret_cast<const float4*>(f)[4 + q];
        v.z[0] = lo.x; v.z[1] = lo.y; v.z[2] = lo.z; v.z[3] = lo.w;
        v.z[4] = hi.x; v.z[5] = hi.y; v.z[6] = hi.z; v.z[7] = hi.w;
    }
    v.x = a.posr[aid];
    return v;
}

// Sigma = R diag(v) R^T (upper triangle) of the unit quaternion (w, x, y, z).
// Every fused product is written out: the values do not depend on which ones
// the compiler would fuse.
__device__ __forceinline__ void covariance(float w, float x, float y, float z, float v0, float v1, float v2, float (&S)[6]) {
#pragma clang fp contract(off)
    const float xw = x * w, yw = y * w, zw = z * w, xx = x * x, yy = y * y;
    const float xy_m = fmaf(y, x, -zw), xy_p = fmaf(y, x, zw);
    const float xz_m = fmaf(z, x, -yw), xz_p = fmaf(z, x, yw);
    const float yz_m = fmaf(z, y, -xw), yz_p = fmaf(z, y, xw);
    const float R[3][3] = {{fmaf(fmaf(z, z, yy), -2.f, 1.f), xy_m + xy_m, xz_p + xz_p},
                           {xy_p + xy_p, fmaf(fmaf(z, z, xx), -2.f, 1.f), yz_m + yz_m},
                           {xz_m + xz_m, yz_p + yz_p, fmaf(fmaf(y, y, xx), -2.f, 1.f)}};
    int i = 0;
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int c = r; c < 3; ++c)
            S[i++] = fmaf(v2 * R[r][2], R[c][2], fmaf(v0 * R[r][0], R[c][0], (v1 * R[r][1]) * R[c][1]));
}

// What the epilogue reads of Gaussian j of an anchor.
struct Shape {
    float sc[6], off[3];
};
__device__ __forceinline__ Shape load_shape(const MfmaDeriveArgs& a, int32_t aid, int j) {
    Shape v;
    const float* sc = a.scale + (int64_t)aid * 6;
    const float* off = a.offsets + ((int64_t)aid * a.k + j) * 3;
#pragma unroll
    for (int i = 0; i < 6; ++i) v.sc[i] = sc[i];
#pragma unroll
    for (int i = 0; i < 3; ++i) v.off[i] = off[i];
    return v;
}

template <int MODE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_derive_mfma(MfmaDeriveArgs a) {
    // layer-1 weights, then the outputs of each wave's 16 anchors: k alphas,
    // 3 k colours, 7 k covariance words each, rows an odd number of words apart
    extern __shared__ __align__(16) float s_mem[];
    __shared__ int32_t sAid[NT / 64][16];
    __shared__ int32_t sLine[NT / 64][16];
    __shared__ uint32_t sMask[NT / 64][16];
    constexpr int kW1 = MODE == GSC_PREC_F32 ? 14 : 9;  // 16-byte words per lane
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int q = lane >> 4, col = lane & 15;
    const MfmaFrags& fr = a.fr;
    const MfmaView& v = a.v[blockIdx.y];
    const int nt = fr.n_at + fr.n_ct + fr.n_vt;
    const int k = a.k, pitch = (11 * k) | 1;
    float* O = s_mem + kW1 * 64 * 4 + w * 16 * pitch;
    const int32_t n = *v.n_miss;
    const int ntiles = (n + 15) / 16;
    if ((int)blockIdx.x >= ntiles) return;  // (block-uniform)
    // (consecutive tiles go to different blocks: few tiles spread over the chip)
    const int step = NT / 64 * gridDim.x;
    int tile = w * gridDim.x + blockIdx.x;
    auto anchor_of = [&](int t, int32_t& aid, int32_t& line) {
        const int m = t * 16 + col;
        const bool ok = t < ntiles && m < n;
        const int32_t pos = ok ? v.misses[m] : 0;
        aid = ok ? v.visible[pos] : 0;
        line = ok ? v.vslot[pos] : -1;
    };
    int32_t aid, line;
    anchor_of(tile, aid, line);
    uint4* s_w1 = reinterpret_cast<uint4*>(s_mem);
    {
        const uint4* src = MODE == GSC_PREC_F32 ? reinterpret_cast<const uint4*>(fr.l1_f32)
                                                : reinterpret_cast<const uint4*>(MODE == GSC_PREC_BF16 ? fr.l1_bf16 : fr.l1_fp8);
        for (int i = threadIdx.x; i < kW1 * 64; i += NT) s_w1[i] = src[i];
    }
    Inputs in = load_inputs<MODE>(a, aid, q);
    int32_t aid1, line1;  // the next tile's
    anchor_of(tile + step, aid1, line1);
    const uint32_t rk = (65536u + (uint32_t)k - 1u) / (uint32_t)k;  // g / k = g rk >> 16 for g < 16 k <= 256
    __syncthreads();
    for (; tile < ntiles; tile += step) {
        if (q == 0) {
            sAid[w][col] = aid;
            sLine[w][col] = line;
            sMask[w][col] = 0;
        }
        float vx = in.x.x - v.cam_pos[0], vy = in.x.y - v.cam_pos[1], vz = in.x.z - v.cam_pos[2];
        const float nv = sqrtf(fmaf(vz, vz, fmaf(vx, vx, vy * vy)));
        const float inv = 1.0f / nv;
        const float dv[3] = {vx * inv, vy * inv, vz * inv};
        // the optional distance input (column 35; its weights are zero without it)
        const float dn = a.inv_dist_unit > 0.f ? nv * a.inv_dist_unit : 0.f;
        // ---- layer 1: H^T = W1 Z^T, 6 tiles of 16 hidden units
        floatx4 acc[6];
#pragma unroll
        for (int hb = 0; hb < 6; ++hb) acc[hb] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (MODE == GSC_PREC_F32) {
            float b[9];
#pragma unroll
            for (int s = 0; s < 8; ++s) b[s] = in.z[s];
            b[8] = q == 0 ? dv[0] : (q == 1 ? dv[1] : (q == 2 ? dv[2] : dn));
#pragma unroll
            for (int i4 = 0; i4 < 14; ++i4) {
                const uint4 v = s_w1[i4 * 64 + lane];
                const float wv[4] = {__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = 4 * i4 + e;  // step i / 6 of hidden block i % 6
                    if (i < 54) acc[i % 6] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[e], b[i / 6], acc[i % 6], 0, 0, 0);
                }
            }
        } else {
            shortx4 b[3];
            b[0] = d_bf16x4(in.z[0], in.z[1], in.z[2], in.z[3]);
            b[1] = d_bf16x4(in.z[4], in.z[5], in.z[6], in.z[7]);
            b[2] = q == 0 ? d_bf16x4(dv[0], dv[1], dv[2], dn) : shortx4{0, 0, 0, 0};
#pragma unroll
            for (int i2 = 0; i2 < 9; ++i2) {
                const uint4 v = s_w1[i2 * 64 + lane];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int i = 2 * i2 + e;  // k-block i / 6 of hidden block i % 6
                    acc[i % 6] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(half_of(v, e), b[i / 6], acc[i % 6], 0, 0, 0);
                }
            }
        }
        // asked for before they are needed: the first output tile's weights,
        // what the epilogue's first step reads, the next tile's inputs and the
        // anchors of the one after
        OutTile<MODE> ld = load_out_tile<MODE>(fr, 0, lane);
        int al = (int)(((uint32_t)lane * rk) >> 16), j = lane - al * k;
        Shape shape = load_shape(a, __shfl(aid, al & 15), al < 16 ? j : 0);
        aid = aid1;
        line = line1;
        in = load_inputs<MODE>(a, aid, q);
        anchor_of(tile + 2 * step, aid1, line1);
        // bias + ReLU (rows hb*16 + 4q + i of H^T, column = this lane's anchor)
        float h[6][4];
        shortx4 hh[6];
#pragma unroll
        for (int hb = 0; hb < 6; ++hb) {
            const float4 b1 = reinterpret_cast<const float4*>(fr.b1)[hb * 4 + q];
            const float4 s1 = MODE == GSC_PREC_FP8 ? reinterpret_cast<const float4*>(fr.s1)[hb * 4 + q] : b1;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float v = acc[hb][i];
                if (MODE == GSC_PREC_FP8) v *= comp(s1, i);
                h[hb][i] = fmaxf(v + comp(b1, i), 0.f);
            }
            if (MODE != GSC_PREC_F32)
                hh[hb] = d_bf16x4(h[hb][0], h[hb][1], h[hb][2], h[hb][3]);
        }
        // ---- layer 2: O^T = W2 H^T per 16-output tile, head by head
        int ot = 0;
#pragma unroll
        for (int head = 0; head < 3; ++head) {
            const int nh = head == 0 ? fr.n_at : (head == 1 ? fr.n_ct : fr.n_vt);
            const int rows = head == 0 ? k : (head == 1 ? 3 * k : 7 * k), first = head == 0 ? 0 : (head == 1 ? k : 4 * k);
            for (int t = 0; t < nh; ++t, ++ot) {
                const OutTile<MODE> cur = ld;
                ld = load_out_tile<MODE>(fr, ot + 1 < nt ? ot + 1 : ot, lane);
                const float4 s2 = MODE == GSC_PREC_FP8 ? reinterpret_cast<const float4*>(fr.s2)[ot * 4 + q] : cur.b;
                floatx4 o = floatx4{0.f, 0.f, 0.f, 0.f};
                if (MODE == GSC_PREC_F32) {
#pragma unroll
                    for (int hb2 = 0; hb2 < 2; ++hb2) {
                        const uint4 v = cur.w[MODE == GSC_PREC_F32 ? hb2 : 0];
                        o = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(v.x), h[2 * head + hb2][0], o, 0, 0, 0);
                        o = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(v.y), h[2 * head + hb2][1], o, 0, 0, 0);
                        o = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(v.z), h[2 * head + hb2][2], o, 0, 0, 0);
                        o = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(v.w), h[2 * head + hb2][3], o, 0, 0, 0);
                    }
                } else {
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
                        o = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(half_of(cur.w[0], kb), hh[2 * head + kb], o, 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = 16 * t + 4 * q + i;
                    float v = o[i];
                    if (MODE == GSC_PREC_FP8) v *= comp(s2, i);
                    if (row < rows) O[col * pitch + first + row] = v + comp(cur.b, i);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();  // a wave's LDS accesses complete in order
        // ---- epilogue: one Gaussian per lane step
        for (int g = lane; g < 16 * k; g += 64) {
            const int m = tile * 16 + al, gl = sLine[w][al];
            const Shape sh = shape;
            const int al0 = al, j0 = j, g1 = g + 64;
            al = (int)(((uint32_t)g1 * rk) >> 16);
            j = g1 - al * k;
            if (g1 < 16 * k) shape = load_shape(a, sAid[w][al], j);
            if (m >= n || gl < 0) continue;
            const float* Ov = O + al0 * pitch;
            float alpha = tanhf(Ov[j0]);
            float r = sigm(Ov[k + 3 * j0]), gg = sigm(Ov[k + 3 * j0 + 1]), bb = sigm(Ov[k + 3 * j0 + 2]);
            const float* os = Ov + 4 * k + 7 * j0;
            float s0 = sh.sc[3] * sigm(os[0]), s1 = sh.sc[4] * sigm(os[1]), s2 = sh.sc[5] * sigm(os[2]);
            float qw = os[3], qx = os[4], qy = os[5], qz = os[6];
            float qn = sqrtf(fmaf(qz, qz, fmaf(qy, qy, fmaf(qw, qw, qx * qx))));
            if (qn > 0.f) {
                float iq = 1.0f / qn;
                qw *= iq; qx *= iq; qy *= iq; qz *= iq;
            } else {
                qw = 1.f; qx = qy = qz = 0.f;
            }
            float S[6];
            covariance(qw, qx, qy, qz, s0 * s0, s1 * s1, s2 * s2, S);
            const int64_t e = (int64_t)gl * k + j0;
            // position relative to the anchor (small, so FP32 keeps it to
            // ~1e-7 m); the rasteriser adds anchor - camera in FP64
            v.L0[e] = make_float4(sh.sc[0] * sh.off[0], sh.sc[1] * sh.off[1], sh.sc[2] * sh.off[2], alpha);
            v.L1[e] = make_float4(S[0], S[1], S[2], S[3]);
            v.L2[e] = make_float4(S[4], S[5], r, gg);
            v.L3[e] = bb;
            if (alpha > 0.f) atomicOr(&sMask[w][al0], 1u << j0);
        }
        __builtin_amdgcn_wave_barrier();
        // the line's mask of kept Gaussians (alpha > 0, the render buffer's
        // test), from the same alphas
        if (v.line_mask && lane < 16) {
            const int m = tile * 16 + lane, gl = sLine[w][lane];
            if (m < n && gl >= 0) v.line_mask[gl] = (uint16_t)sMask[w][lane];
        }
        __builtin_amdgcn_wave_barrier();
    }
}

}  // namespace

hipError_t derive_mfma(const MfmaDeriveArgs& a, int nv, int64_t n_max, hipStream_t st) {
    const int64_t tiles = (n_max + 15) / 16;
    const size_t lds = ((a.mode == GSC_PREC_F32 ? 14 : 9) * 64 * 4 + NT / 64 * 16 * (size_t)((11 * a.k) | 1)) * sizeof(float);
    // a wave per tile, up to what the chip holds at once (4 waves per SIMD),
    // shared by the views
    const int64_t most = kMaxBlocks / nv;
    const dim3 blocks((unsigned)(tiles < 1 ? 1 : (tiles < most ? tiles : most)), (unsigned)nv);
    switch (a.mode) {
        case GSC_PREC_F32:
            hipLaunchKernelGGL(k_derive_mfma<GSC_PREC_F32>, blocks, dim3(NT), lds, st, a);
            break;
        case GSC_PREC_BF16:
            hipLaunchKernelGGL(k_derive_mfma<GSC_PREC_BF16>, blocks, dim3(NT), lds, st, a);
            break;
        default:
            hipLaunchKernelGGL(k_derive_mfma<GSC_PREC_FP8>, blocks, dim3(NT), lds, st, a);
            break;
    }
    return hipGetLastError();
}

}  // namespace gsc
