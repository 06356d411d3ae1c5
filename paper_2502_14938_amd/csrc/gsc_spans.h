// What the preprocess leaves of a footprint and the binning reads: the
// per-entry record, the span words of its tile rows, and the super tiles they
// cover.
#pragma once
#include "gsc_common.h"

namespace gsc {

// Footprints taller than this many tile rows get one thread per row for
// their spans (k_tall_spans) and are binned by super rows; shorter ones keep
// their row spans in the record and are binned from them.
constexpr int kSmallRows = 4;

// Per-entry record, 4 x float4 (64 B, one cache line):
//   A = (mean2d.x, mean2d.y, conic a, conic b)
//   B = (conic c, alpha, r, g)
//   C = (b, bits: tile rows y0 | y1 << 16, bits: segment, bits: (super tile, entry) pair count)
//   D = bits: exact tile span lo | hi << 16 of each of up to kSmallRows rows
//       (footprints of at most kSmallRows tile rows; hi < lo: empty row)
constexpr int kRec = 4;
constexpr int kEntryChunk = 256;  // entries the preprocess projects (and lists tall ones of) together

// Span word of a tile row: lo | hi << 16, hi < lo (0xffff, 0) when empty.
constexpr uint32_t kEmptySpan = 0x0000ffffu;
__device__ __forceinline__ int span_lo(uint32_t sp) { return (int)(sp & 0xffffu); }
__device__ __forceinline__ int span_hi(uint32_t sp) { return (int)(sp >> 16); }

// Super-tile columns [x0, x1] of a super row from the spans of its two tile
// rows a (even) and b (odd), either possibly empty: the hull of the rows'
// super columns (a convex footprint's rows give adjacent or overlapping
// ranges; a column of the hull may have an empty mask).  Returns the column
// count (0: both rows empty).
__device__ __forceinline__ uint32_t sup_cols(uint32_t sa, uint32_t sb, int& x0) {
    int lo = 0x7fffffff, hi = -1;
    if (span_hi(sa) >= span_lo(sa)) { lo = span_lo(sa) >> kSupShift; hi = span_hi(sa) >> kSupShift; }
    if (span_hi(sb) >= span_lo(sb)) {
        lo = min(lo, span_lo(sb) >> kSupShift);
        hi = max(hi, span_hi(sb) >> kSupShift);
    }
    x0 = lo;
    return hi >= lo ? (uint32_t)(hi - lo + 1) : 0u;
}

// Mask of the tiles of super column x covered by tile rows a and b: bit
// 2 (ty & 1) + (tx & 1).
__device__ __forceinline__ uint32_t sup_mask(uint32_t sa, uint32_t sb, int x) {
    const int t0 = x << kSupShift, t1 = t0 + 1;
    const int la = span_lo(sa), ha = span_hi(sa), lb = span_lo(sb), hb = span_hi(sb);
    return (uint32_t)(la <= t0 && t0 <= ha) | ((uint32_t)(la <= t1 && t1 <= ha) << 1) |
           ((uint32_t)(lb <= t0 && t0 <= hb) << 2) | ((uint32_t)(lb <= t1 && t1 <= hb) << 3);
}

// Binning record of an entry (16 B, read once when counting and once when
// writing): the spans of a short footprint's up to kSmallRows tile rows (ten
// bits per end: an image has at most 1,024 tile columns), its first tile row,
// its segment, whether it is short and covers a tile, and the depth key.
struct BinRec {
    uint32_t sp[kSmallRows];
    int y0, seg;
    bool binned;
};
__device__ __forceinline__ uint4 pack_bin(const uint32_t (&sp)[kSmallRows], int y0, uint32_t seg, bool binned, uint32_t key) {
    uint32_t s[kSmallRows];
#pragma unroll
    for (int i = 0; i < kSmallRows; ++i)
        s[i] = span_hi(sp[i]) >= span_lo(sp[i]) ? (uint32_t)span_lo(sp[i]) | ((uint32_t)span_hi(sp[i]) << 10) : 1u;
    return make_uint4(s[0] | (s[1] << 20), (s[1] >> 12) | (s[2] << 8) | (s[3] << 28),
                      (s[3] >> 4) | ((uint32_t)y0 << 16) | (binned ? 1u << 26 : 0u) | (seg << 27), key);
}
__device__ __forceinline__ BinRec unpack_bin(const uint4& v) {
    const uint32_t s[kSmallRows] = {v.x & 0xfffffu, ((v.x >> 20) | (v.y << 12)) & 0xfffffu, (v.y >> 8) & 0xfffffu,
                                    ((v.y >> 28) | (v.z << 4)) & 0xfffffu};
    BinRec r;
#pragma unroll
    for (int i = 0; i < kSmallRows; ++i) r.sp[i] = (s[i] & 0x3ffu) | ((s[i] >> 10) << 16);
    r.y0 = (int)((v.z >> 16) & 0x3ffu);
    r.binned = (v.z >> 26) & 1u;
    r.seg = (int)((v.z >> 27) & 0xfu);
    return r;
}

// Word of a stored super row of a tall footprint: its Y | segment << kRowSegShift.
constexpr int kRowSegShift = 16;
constexpr uint32_t kRowMask = (1u << kRowSegShift) - 1u;
static_assert(kMaxSeg <= 16, "a binning record has four bits for the segment");

// Super-tile grid of one segment.
struct SupGeo {
    int32_t base;  // first global super-tile id
    int32_t nsx;   // super tiles per row
};

}  // namespace gsc
