// Binning of a raster batch: from the entries' tile spans to every super
// tile's depth-ordered list.
//
//   k_bin<false>   per block of entries, how many items each super tile gets
//                  (counters in LDS)
//   k_bin_columns  per super tile, the blocks' first positions and the total
//   k_bin<true>    every block writes its items (depth key, entry, tile mask)
//                  at its positions of each super tile's range; where the items
//                  are more than the buffers hold, the nearest ones (write_cut)
//   k_bin_split    the lists of more than kSortCap items, divided by depth
//                  into pieces that fit
//   k_bin_sort     every list and piece in the order (depth key, entry), one
//                  block each, in LDS
//   k_bin_merge    long lists whose depths no division separates: their
//                  chunks, which k_bin_sort sorted one by one
// Lists of more than kHugeList items, too many for one block to divide, are
// sorted by chunks in the same three launches: the chunks (k_bin_split), groups
// of chunks merged (k_bin_sort), the groups merged (k_bin_merge).
//
// One counting pass over the super tiles puts every item in its list, and
// what is left to sort are lists that fit a block's LDS: two passes over the
// items in place of a radix sort of the Gaussians by depth (four passes), of
// the items by super tile (two) and the scans between them, with 14 launches
// less in a frame.  The order within a list is that of the whole (super tile,
// depth) key with ties by entry, so it does not depend on the order in which
// the blocks' lanes take positions.
//
// Measured, a whole pass with the radix sorts and with this: 2,000 Gaussians
// at 256x256 134 and 54 us, 60,000 at 1000x560 185 and 102 us, 500,000 at
// 1920x1081 301 and 205 us, a stereo frame of 2 x 2048x1080 high above the
// city (6 M items) 659 and 595 us.  Of that last one's 203 us the writes take
// 75: they go to 4,352 lists at once, more than an XCD's L2 holds the ends of,
// so four of five 8-byte items leave it as a partial line of their own (195 MB
// for 48); the sort takes 56, the division of the long lists 40, the counts 20,
// their columns 7, the merge 5.
// With more lists the writes gather less and less, and the radix sorts, whose
// launches are spread over more items, win: batches of stereo images with 6,192
// super tiles take 588 us binned and 611 radix-sorted, with 13,392 1,031 and
// 979, with 33,400 2,546 and 2,080.  The line is drawn at kBinLists = 8,192,
// where a block's counters for all lists still leave room for two blocks a CU.
#include "gsc_common.h"
#include "gsc_spans.h"

namespace gsc {

namespace {

constexpr int NB = 1024;            // threads of a counting / writing block
constexpr int kColTile = 64;        // super tiles per block of k_bin_columns
constexpr int kColRows = 32;        // blocks' counts a thread of it adds
constexpr int kMaxBinBlocks = kColRows * (NB / kColTile);

struct BinArgs {
    SupGeo sg[kMaxSeg];
    RasterCounters* rc;
    const uint4* brec;        // binning record per entry
    const uint4* srow;        // super rows of the tall footprints (see k_tall_spans)
    const int32_t* srow_y;
    int64_t srow_cap;
    const float4* rec;        // the entries' records (a tall footprint's item count)
    uint32_t* hist;           // [blocks][stride] counts, then first positions, of each super tile
    uint32_t* total;          // [stride]
    uint32_t* kept;           // [2 stride] items that stay of each super tile and those placed, where some are left out
    uint64_t* items;          // depth key << 32 | entry << 4 | mask
    int32_t* ranges;
    int32_t* n_sort;
    int32_t* long_lists;      // super tiles with more than kSortCap items,
    int32_t* huge_lists;      // or more than kHugeList
    int64_t max_pairs;
    int32_t total_sup, stride;
    int32_t run;              // entries a block takes at a time: 16 waves of 16, 32 or 64
};

// Counting: a super row adds one to n neighbouring super tiles, i.e. +1 where
// it begins and -1 past its end, two updates whatever its width; a running
// sum over the super tiles then gives the counts.
__device__ __forceinline__ void count_row(uint32_t* s_cnt, int sup, int n, int total_sup) {
    atomicAdd(&s_cnt[sup], 1u);
    if (sup + n < total_sup) atomicAdd(&s_cnt[sup + n], 0xffffffffu);
}

// Writing: each item at its super tile's next position.
__device__ __forceinline__ void write_item(const BinArgs& a, uint32_t* s_cnt, int sup, uint32_t low, uint32_t depth) {
    const uint32_t pos = atomicAdd(&s_cnt[sup], 1u);
    if ((int64_t)pos < a.max_pairs) a.items[pos] = ((uint64_t)depth << 32) | low;
}

__device__ __forceinline__ uint32_t lane_word(uint32_t v, int lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

// A super row: n items from super tile sup (tile column pair x0) on, the
// spans sa, sb of its two tile rows.
struct Row {
    int n, sup, x0;
    uint32_t sa, sb;
};

// Items [from, r.n) of lane l's row r, written by the whole wave.
__device__ __forceinline__ void write_wide(const BinArgs& a, uint32_t* s_cnt, const Row& r, int l, int from,
                                           uint32_t entry, uint32_t depth) {
    const int n = (int)lane_word((uint32_t)r.n, l), x0 = (int)lane_word((uint32_t)r.x0, l);
    const int sup = (int)lane_word((uint32_t)r.sup, l);
    const uint32_t sa = lane_word(r.sa, l), sb = lane_word(r.sb, l);
    for (int k = max(from, 0) + (int)(threadIdx.x & 63); k < n; k += 64)
        write_item(a, s_cnt, sup + k, (entry << 4) | sup_mask(sa, sb, x0 + k), depth);
}

// Items of a short footprint's three super rows (n = 0: no such row), one
// footprint per lane: every lane writes its own first kOwnItems, four at a
// time with their positions asked for together; the rest of the wide ones
// are written by the whole wave.  All lanes of the wave take part.
constexpr int kOwnItems = 12;
__device__ __forceinline__ void write_rows(const BinArgs& a, uint32_t* s_cnt, uint32_t e, uint32_t depth, const Row& r0,
                                           const Row& r1, const Row& r2) {
    const int n01 = r0.n + r1.n, all = n01 + r2.n, own = min(all, kOwnItems);
    for (int t0 = 0; t0 < own; t0 += 4) {
        uint32_t pos[4], low[4];
        bool on[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int t = t0 + q;
            const bool p1 = t >= r0.n, p2 = t >= n01;  // past row 0, past row 1
            const int k = t - (p2 ? n01 : (p1 ? r0.n : 0));
            const int x = (p2 ? r2.x0 : (p1 ? r1.x0 : r0.x0)) + k, c = (p2 ? r2.sup : (p1 ? r1.sup : r0.sup)) + k;
            low[q] = (e << 4) | sup_mask(p2 ? r2.sa : (p1 ? r1.sa : r0.sa), p2 ? r2.sb : (p1 ? r1.sb : r0.sb), x);
            on[q] = t < own;
            pos[q] = on[q] ? atomicAdd(&s_cnt[c], 1u) : 0u;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (on[q] && (int64_t)pos[q] < a.max_pairs) a.items[pos[q]] = ((uint64_t)depth << 32) | low[q];
    }
    for (uint64_t wide = __ballot(all > kOwnItems); wide; wide &= wide - 1) {
        const int l = __ffsll((unsigned long long)wide) - 1;
        const uint32_t d = lane_word(depth, l), el = lane_word(e, l);
        const int n0 = (int)lane_word((uint32_t)r0.n, l), n1 = (int)lane_word((uint32_t)n01, l);
        write_wide(a, s_cnt, r0, l, kOwnItems, el, d);
        write_wide(a, s_cnt, r1, l, kOwnItems - n0, el, d);
        write_wide(a, s_cnt, r2, l, kOwnItems - n1, el, d);
    }
}

// A footprint's super row at row Y of its image from the spans of its two
// tile rows.
__device__ __forceinline__ Row make_row(const SupGeo& sg, int Y, uint32_t sa, uint32_t sb) {
    Row r;
    r.sa = sa;
    r.sb = sb;
    r.n = (int)sup_cols(sa, sb, r.x0);
    r.sup = sg.base + Y * sg.nsx + r.x0;
    return r;
}

// Where the items are more than the buffers hold, those of the nearest
// entries stay, in the order (depth key, entry), and of the entry at the cut
// the first `keep` (row by row): what sorting the entries by depth and
// emitting them up to the capacity leaves.
struct Cut {
    uint32_t depth, entry;
    int32_t keep;
};
constexpr int kKeepAll = 1 << 30;
__device__ __forceinline__ int items_left(const Cut& c, uint32_t depth, uint32_t e) {
    if (depth == c.depth && e == c.entry) return c.keep;
    return depth < c.depth || (depth == c.depth && e < c.entry) ? kKeepAll : 0;
}
__device__ __forceinline__ void trim_row(Row& r, int& left) {
    const int n = r.n;
    r.n = max(min(n, left), 0);
    left -= n;
}

// The super rows of a short footprint from its binning record.
__device__ __forceinline__ void footprint_rows(const BinRec& r, const SupGeo& sg, Row& r0, Row& r1, Row& r2) {
    // super row i is Y = y0 / 2 + i: tile rows (0, 1), (2, 3)
    // from an even y0; (-, 0), (1, 2), (3, -) from an odd one
    const bool odd = r.y0 & 1;
    const int Y = r.y0 >> kSupShift;
    r0 = make_row(sg, Y, odd ? kEmptySpan : r.sp[0], odd ? r.sp[0] : r.sp[1]);
    r1 = make_row(sg, Y + 1, odd ? r.sp[1] : r.sp[2], odd ? r.sp[2] : r.sp[3]);
    r2 = make_row(sg, Y + 2, odd ? r.sp[3] : kEmptySpan, kEmptySpan);
}

// Block b takes every nblk-th run of the entries, for their short footprints
// (from their binning records), and every nblk-th run of the stored super
// rows of the tall ones: entries come in anchor order, coarse levels first, so
// a contiguous share would give a few blocks all the wide footprints (264 us
// instead of 20 on the city).  The same runs when counting and when writing.
// kCut: only the items that `cut` leaves.
template <bool kWrite, bool kCut>
__device__ __forceinline__ void walk(const BinArgs& a, uint32_t* s_cnt, const SupGeo* s_sg, int b, int nblk, const Cut& cut) {
    // Sixteen lanes run / 16 entries apart (and up to four neighbours at each):
    // a Gaussian's eyes and an anchor's Gaussians, which fall on the same super
    // tiles, come together, and LDS adds to one address wait for each other.
    // (block-uniform loop: whole waves take part in the wide footprints' items)
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ne = a.rc->n_entries, near = a.run >> 8;
    const int place = (lane & 15) * (a.run >> 4) + wv * near + (lane >> 4);
    const bool here = (lane >> 4) < near;
    auto load = [&](int64_t e) {
        if (!here || e >= ne) return make_uint4(1u, 0u, 0u, 0u);  // (not binned)
        return a.brec[e];
    };
    uint4 next = load((int64_t)b * a.run + place);
    for (int64_t eb = (int64_t)b * a.run; eb < ne; eb += (int64_t)nblk * a.run) {
        const int64_t e = eb + place;
        Row r0{0, 0, 0, 0u, 0u}, r1 = r0, r2 = r0;
        uint32_t depth = 0;
        {
            // (the next run's record is on its way while this one's items are written)
            const uint4 w = next;
            next = load(e + (int64_t)nblk * a.run);
            const BinRec r = unpack_bin(w);
            if (r.binned) {
                depth = w.w;
                footprint_rows(r, s_sg[r.seg], r0, r1, r2);
                if (kCut) {
                    int left = items_left(cut, depth, (uint32_t)e);
                    trim_row(r0, left);
                    trim_row(r1, left);
                    trim_row(r2, left);
                }
            }
        }
        if (kWrite) {
            write_rows(a, s_cnt, (uint32_t)e, depth, r0, r1, r2);
        } else {
            if (r0.n) count_row(s_cnt, r0.sup, r0.n, a.total_sup);
            if (r1.n) count_row(s_cnt, r1.sup, r1.n, a.total_sup);
            if (r2.n) count_row(s_cnt, r2.sup, r2.n, a.total_sup);
        }
    }
    // the tall footprints' super rows, runs b, b + nblk, ... of kRowRun: a
    // lane per row of several runs when counting (two updates a row), eight
    // lanes per row of one run when writing (a lane per item, or nearly: a
    // lane per row writes the city's in 103 us instead of 76)
    constexpr int kRowLanes = kWrite ? 8 : 1, kRowRun = NB / 8, kRuns = 8 / kRowLanes;
    const int64_t nsr = min((int64_t)a.rc->n_srows, a.srow_cap);
    const int sub = threadIdx.x % kRowLanes, at = threadIdx.x / kRowLanes;
    for (int64_t q = ((int64_t)b + (at / kRowRun) * nblk) * kRowRun + at % kRowRun; q < nsr;
         q += (int64_t)nblk * kRowRun * kRuns) {
        const uint4 sr = a.srow[q];
        const uint32_t e = sr.z, ys = (uint32_t)a.srow_y[q];
        int x0;
        int n = (int)sup_cols(sr.x, sr.y, x0);
        if (sub >= n) continue;
        const SupGeo sg = s_sg[(ys >> kRowSegShift) % kMaxSeg];
        const int64_t sup = sg.base + (int64_t)(ys & kRowMask) * sg.nsx + x0;
        // (a row that a capacity overflow left unwritten may hold anything)
        if (e >= (uint32_t)ne || sup < 0 || sup + n > a.total_sup) continue;
        uint32_t depth = 0;
        if (kWrite || kCut) depth = a.brec[e].w;
        if (kCut) n = (int)max(min((int64_t)n, (int64_t)items_left(cut, depth, e) - sr.w), (int64_t)0);
        if (!kWrite) {
            if (n) count_row(s_cnt, (int)sup, n, a.total_sup);
            continue;
        }
        for (int k = sub; k < n; k += kRowLanes)
            write_item(a, s_cnt, (int)sup + k, (e << 4) | sup_mask(sr.x, sr.y, x0 + k), depth);
    }
}

constexpr int kListsThread = kBinLists / NB;  // super tiles of a thread, in a row

// The counts of the thread's super tiles (c0 on) from what counting left in
// s_cnt (a running sum); all threads of the block take part.
__device__ __forceinline__ void list_counts(const uint32_t* s_cnt, uint32_t* s_part, int total_sup, int stride, int c0,
                                            uint32_t (&n)[kListsThread]) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    __syncthreads();
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kListsThread; ++i) {
        const int c = c0 + i;
        sum += c < stride ? s_cnt[c] : 0u;
        n[i] = sum;
    }
    uint32_t x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = __shfl_up(x, o, 64);
        if (lane >= o) x += v;
    }
    if (lane == 63) s_part[wv] = x;
    __syncthreads();
    uint32_t before = x - sum;
    for (int i = 0; i < wv; ++i) before += s_part[i];
#pragma unroll
    for (int i = 0; i < kListsThread; ++i) {
        const int c = c0 + i;
        n[i] = c < total_sup ? before + n[i] : 0u;
    }
}

// Exclusive prefix of v over the block; s: 16 words, free again after the next
// barrier.  32-bit sums saturate: all that lies past 2^32 - 1 is past every capacity.
__device__ __forceinline__ uint32_t add_sat(uint32_t x, uint32_t y) { return __builtin_elementwise_add_sat(x, y); }
__device__ __forceinline__ uint64_t add_sat(uint64_t x, uint64_t y) { return x + y; }  // (2^28 entries of 2^13 items at most)
template <typename T>
__device__ __forceinline__ T block_prefix(T v, T* s) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    T x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T y = __shfl_up(x, o, 64);
        if (lane >= o) x = add_sat(x, y);
    }
    if (lane == 63) s[wv] = x;
    T before = __shfl_up(x, 1, 64);
    if (lane == 0) before = 0;
    __syncthreads();
    for (int i = 0; i < wv; ++i) before = add_sat(before, s[i]);
    return before;
}

// The ranges of the thread's super tiles (c0 on) from their counts t and first
// positions, within the capacity, and the longer ones' lists; all threads of
// the block take part.  The long ones are listed in super-tile order:
// neighbours, which are about as long, go to different blocks of k_bin_split
// (66 -> 55 us over the fly-through, from the order that atomic adds left).
__device__ __forceinline__ void put_ranges(const BinArgs& a, int c0, const uint32_t (&t)[kListsThread], uint32_t first,
                                           uint32_t* s_part) {
    const uint32_t cap = (uint32_t)a.max_pairs;  // (at most 2^31 - 1)
    auto items = [&](int i, uint32_t at) { return (int)(min(at + t[i], cap) - min(at, cap)); };
    uint32_t longs = 0, f = first;
#pragma unroll
    for (int i = 0; i < kListsThread; ++i) {
        const int n = items(i, f);
        longs += n > kSortCap && n <= kHugeList ? 1u : 0u;
        f += t[i];
    }
    __syncthreads();
    uint32_t at = block_prefix(longs, s_part);
#pragma unroll
    for (int i = 0; i < kListsThread; ++i) {
        const int c = c0 + i, n = items(i, first);
        if (c < a.total_sup) {
            a.ranges[2 * c] = n ? (int32_t)first : 0;
            a.ranges[2 * c + 1] = n ? (int32_t)first + n : 0;
            if (n > kSortCap && n <= kHugeList) a.long_lists[at++] = c;
            if (n > kHugeList) a.huge_lists[atomicAdd(&a.rc->n_huge, 1)] = c;
        }
        first += t[i];
    }
    if (threadIdx.x == NB - 1) {  // (`first` and `at` are now the totals)
        *a.n_sort = (int32_t)min(first, cap);
        a.rc->n_long = (int32_t)at;
    }
}

// ------------------------------------------- items over the capacity
// Blocks of one launch that work together with barriers between them: those
// that have started when the first one closes the team (it waits a while for
// the rest, up to kTeamMost; whoever comes later leaves).  Every member is
// running, so every wait for the others ends, whatever else is on the device.
// What the members share within the launch they read and write by device-scope
// atomics alone, so a barrier waits for those and needs no cache write-back.
struct Team {
    RasterCounters* rc;
    int part, size;  // size 0: not a member
    uint32_t met;    // barriers passed
};
constexpr uint32_t kTeamMost = 128, kTeamClosed = 1u << 31;
template <typename T>
__device__ __forceinline__ T agent_load(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ void agent_store(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ T agent_add(T* p, T v) { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// (all threads of the block; s: two words)
__device__ __forceinline__ Team join_team(RasterCounters* rc, uint32_t blocks, uint32_t* s) {
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t at = agent_add(&rc->team, 1u), most = min(blocks, kTeamMost);
        if (at == 0) {
            for (int i = 0; i < 1024 && agent_load(&rc->team) < most; ++i) __builtin_amdgcn_s_sleep(8);
            const uint32_t n = __hip_atomic_fetch_or(&rc->team, kTeamClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            agent_store(&rc->team_size, min(n, most));
        }
        uint32_t size = 0;
        if (at < most)  // (not closed yet)
            while ((size = agent_load(&rc->team_size)) == 0) __builtin_amdgcn_s_sleep(8);
        s[0] = at;
        s[1] = at < size ? size : 0u;
    }
    __syncthreads();
    const Team t{rc, __builtin_amdgcn_readfirstlane((int)s[0]), __builtin_amdgcn_readfirstlane((int)s[1]), 0u};
    __syncthreads();
    return t;
}
__device__ __forceinline__ void team_barrier(Team& t) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's atomics are done
    __syncthreads();
    ++t.met;
    if (threadIdx.x == 0) {
        agent_add(&t.rc->team_met, 1u);
        while (agent_load(&t.rc->team_met) < t.met * (uint32_t)t.size) __builtin_amdgcn_s_sleep(8);
    }
    __syncthreads();
}

// The writing when there are more items than the buffers hold: finds the
// entry at the cut by its 60-bit (depth key, entry), twelve bits a pass (how
// many items the entries of each value have), counts the items that stay, and
// writes those.  A frame of 940,000 entries cut to 100,000 and to 500,000 items
// takes 340 and 389 us, with the radix sorts, which emit in depth order, 376
// and 389 (the cut found by one block: 3,517; by all blocks, with cache
// write-backs at every barrier: 799 and 1,962).
constexpr int kCutBits = 12, kCutPasses = 5, kCutValues = 1 << kCutBits;
__device__ __forceinline__ void write_cut(const BinArgs& a, uint32_t all, uint32_t* s_cnt, const SupGeo* s_sg,
                                          uint32_t* s_part) {
    constexpr int PER = kCutValues / NB, kAhead = 2;
    static_assert(kCutValues * 2 <= kBinLists && kCutBits * kCutPasses >= 32 + kMaskShift, "the counts fit, and the key");
    static_assert(kCutPasses * kCutValues * 2 <= 256 * kSortBlocks, "the passes' counts fit the blocks' counts");
    __shared__ int s_value;
    __shared__ uint64_t s_left;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // (addresses made here, not kept from the kernel's start on)
    Team team = join_team(a.rc, gridDim.x, s_part);
    if (!team.size) return;
    typedef unsigned long long u64;
    u64* s_w = reinterpret_cast<u64*>(s_cnt);
    u64* count = reinterpret_cast<u64*>(a.hist);  // [pass][value], in the place of the blocks' counts
    const int64_t step = (int64_t)team.size * NB, me = (int64_t)team.part * NB + tid;
    for (int64_t i = me; i < kCutPasses * kCutValues; i += step)
        agent_store(&count[i], (u64)0);
    for (int64_t i = me; i < 2 * a.stride; i += step)
        agent_store(&a.kept[i], 0u);
    team_barrier(team);
    const int64_t ne = a.rc->n_entries;
    uint64_t high = 0, left = (uint64_t)a.max_pairs;
    bool found = true;
    for (int pass = 0; pass < kCutPasses && found; ++pass, count += kCutValues) {  // (the same in every member)
        const int shift = kCutBits * (kCutPasses - 1 - pass);
        for (int i = tid; i < kCutValues; i += NB) s_w[i] = 0;
        if (tid == 0) s_value = -1;
        __syncthreads();
        for (int64_t e0 = me; e0 < ne; e0 += kAhead * step) {
            uint4 w[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int64_t e = e0 + u * step;
                w[u] = e < ne ? a.brec[e] : make_uint4(1u, 0u, 0u, 0u);  // (no items)
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int64_t e = e0 + u * step;
                const uint64_t key = ((uint64_t)w[u].w << kMaskShift) | (uint64_t)e;
                if (pass && key >> (shift + kCutBits) != high) continue;
                const BinRec r = unpack_bin(w[u]);
                uint32_t n;
                if (r.binned) {
                    Row r0, r1, r2;
                    footprint_rows(r, s_sg[r.seg], r0, r1, r2);
                    n = (uint32_t)(r0.n + r1.n + r2.n);
                } else {
                    n = w[u].w ? __float_as_uint(a.rec[kRec * e + 2].w) : 0u;  // (a tall one, or without items)
                }
                if (n) atomicAdd(&s_w[(key >> shift) & (kCutValues - 1)], (u64)n);
            }
        }
        __syncthreads();
        for (int i = tid; i < kCutValues; i += NB)
            if (s_w[i]) agent_add(&count[i], s_w[i]);
        team_barrier(team);
        uint64_t v[PER], sum = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            v[i] = agent_load(&count[tid * PER + i]);
            sum += v[i];
        }
        uint64_t before = block_prefix(sum, reinterpret_cast<uint64_t*>(s_part));
        if (before <= left && left < before + sum) {  // (at most one thread)
            int i = 0;
            while (left >= before + v[i]) before += v[i++];
            s_value = tid * PER + i;
            s_left = left - before;
        }
        __syncthreads();
        found = s_value >= 0;
        if (found) {
            high = (high << kCutBits) | (uint64_t)s_value;
            left = s_left;
        }
        __syncthreads();
    }
    // (not found: super rows that an overflow of theirs left unwritten were counted)
    Cut cut = found ? Cut{(uint32_t)(high >> kMaskShift), (uint32_t)high & kEntryMask, (int32_t)left}
                    : Cut{0xffffffffu, 0xffffffffu, 0};
    cut.depth = (uint32_t)__builtin_amdgcn_readfirstlane((int)cut.depth);  // (the same in every lane)
    cut.entry = (uint32_t)__builtin_amdgcn_readfirstlane((int)cut.entry);
    cut.keep = __builtin_amdgcn_readfirstlane(cut.keep);
    for (int c = tid; c < a.stride; c += NB) s_cnt[c] = 0u;
    __syncthreads();
    walk<false, true>(a, s_cnt, s_sg, team.part, team.size, cut);
    const int c0 = tid * kListsThread;
    uint32_t t[kListsThread], sum = 0;
    list_counts(s_cnt, s_part, a.total_sup, a.stride, c0, t);
#pragma unroll
    for (int i = 0; i < kListsThread; ++i) {
        const int c = c0 + i;
        s_cnt[c] = t[i];
        if (t[i]) agent_add(&a.kept[c], t[i]);
    }
    team_barrier(team);
#pragma unroll
    for (int i = 0; i < kListsThread; ++i) {
        const int c = c0 + i;
        t[i] = c < a.stride ? agent_load(&a.kept[c]) : 0u;
        sum += t[i];
    }
    uint32_t first = block_prefix(sum, s_part);
    if (team.part == 0) {
        put_ranges(a, c0, t, first, s_part);
        if (tid == 0) {
            a.rc->n_pairs = (int32_t)min(all, 0x7fffffffu);
            atomicOr(&a.rc->overflow, 1);
        }
    }
#pragma unroll
    for (int i = 0; i < kListsThread; ++i) {
        const int c = c0 + i;
        const uint32_t mine = s_cnt[c];
        if (mine)
            s_cnt[c] = first + agent_add(&a.kept[a.stride + c], mine);
        first += t[i];
    }
    __syncthreads();
    walk<true, true>(a, s_cnt, s_sg, team.part, team.size, cut);
}

// Blocks go to the XCDs round-robin, so blocks whose items land side by side
// in every list are given to one XCD: its L2 then completes most of the lines
// that they write parts of.
template <bool kWrite>
__global__ __launch_bounds__(NB) __attribute__((amdgpu_waves_per_eu(8))) void k_bin(BinArgs a) {
    __shared__ __align__(16) uint32_t s_cnt[kBinLists];
    __shared__ __align__(16) uint32_t s_part[2 * NB / 64];
    __shared__ uint32_t s_all;
    __shared__ SupGeo s_sg[kMaxSeg];
    constexpr int PER = kListsThread;
    const int nblk = gridDim.x;
    const int b = nblk % 8 == 0 ? (int)(blockIdx.x % 8) * (nblk / 8) + (int)(blockIdx.x / 8) : (int)blockIdx.x;
    uint32_t* row = a.hist + (int64_t)b * a.stride;
    if (threadIdx.x < kMaxSeg) s_sg[threadIdx.x] = a.sg[threadIdx.x];
    if (kWrite) {
        // the super tiles' first positions, 8 a thread
        uint32_t t[PER], sum = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = threadIdx.x * PER + i;
            t[i] = c < a.stride ? a.total[c] : 0u;
            sum += t[i];
        }
        uint32_t first = block_prefix(sum, s_part);
        if (threadIdx.x == NB - 1) s_all = add_sat(first, sum);
        uint32_t at = first;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = threadIdx.x * PER + i;
            if (c < a.stride) s_cnt[c] = at + row[c];
            at += t[i];
        }
        __syncthreads();
        if ((int64_t)s_all > a.max_pairs) {  // (the same in every block)
            write_cut(a, s_all, s_cnt, s_sg, s_part);
            return;
        }
        if (b == 0) {
            put_ranges(a, threadIdx.x * PER, t, first, s_part);
            if (threadIdx.x == 0) a.rc->n_pairs = (int32_t)s_all;
        }
        walk<true, false>(a, s_cnt, s_sg, b, nblk, Cut{});
    } else {
        for (int c = threadIdx.x; c < a.stride; c += NB) s_cnt[c] = 0u;
        __syncthreads();
        walk<false, false>(a, s_cnt, s_sg, b, nblk, Cut{});
        uint32_t n[PER];
        list_counts(s_cnt, s_part, a.total_sup, a.stride, threadIdx.x * PER, n);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = threadIdx.x * PER + i;
            if (c < a.stride) row[c] = n[i];
        }
    }
}

// kColTile columns (super tiles): each column's counts become exclusive
// prefixes over the blocks, in place, and its total.  A thread holds kColRows counts of one column, all in flight at once.
__global__ __launch_bounds__(NB) void k_bin_columns(uint32_t* __restrict__ hist, uint32_t* __restrict__ total,
                                                    int nblk, int stride) {
    constexpr int NG = NB / kColTile;
    __shared__ uint32_t s_sum[NG][kColTile];
    const int col = threadIdx.x % kColTile, rg = threadIdx.x / kColTile;
    const int c = blockIdx.x * kColTile + col;
    const int per = (nblk + NG - 1) / NG;  // at most kColRows
    uint32_t* h = hist + c;
    uint32_t v[kColRows], sum = 0;
#pragma unroll
    for (int i = 0; i < kColRows; ++i) {
        const int r = rg * per + i;
        v[i] = i < per && r < nblk ? h[(int64_t)r * stride] : 0u;
        sum += v[i];
    }
    s_sum[rg][col] = sum;
    __syncthreads();
    uint32_t pre = 0, all = 0;
    for (int i = 0; i < NG; ++i) {
        const uint32_t x = s_sum[i][col];
        pre += i < rg ? x : 0u;
        all += x;
    }
#pragma unroll
    for (int i = 0; i < kColRows; ++i) {
        const int r = rg * per + i;
        if (i < per && r < nblk) h[(int64_t)r * stride] = pre;
        pre += v[i];
    }
    if (rg == 0) total[c] = all;
}

// ------------------------------------------------------------------ lists
constexpr int NS = 256;  // threads of a sorting block
static_assert(NS * 8 == kSortCap, "a list is at most 8 items a thread");

__device__ __forceinline__ uint32_t list_word(uint64_t item) {
    const uint32_t low = (uint32_t)item;
    return (low >> 4) | (low << kMaskShift);  // entry | mask << kMaskShift
}
static_assert(kMaskShift == 28, "an item's low word is the list word rotated by the mask's four bits");

// Bucket of a depth key among nb over the keys [lo, lo + span]: every step of
// the mapping is monotone, so the buckets are in depth order.
__device__ __forceinline__ int bucket_of(uint32_t key, uint32_t lo, float scale, int nb) {
    return min((int)((float)(key - lo) * scale), nb - 1);
}
__device__ __forceinline__ float bucket_scale(uint32_t lo, uint32_t hi, int nb) {
    return (float)nb / ((float)(hi - lo) + 1.f);
}

// The same with the buckets of equal share of n items (share = nb / n) whose
// counts up to each of the buckets above are cdf: the distribution function,
// linear within a bucket.  Rounded at every step (an exact f - bk from an
// unrounded product could be negative where f rounds up to bk, and the
// order of the buckets with it).
__device__ __forceinline__ int bucket_by_share(uint32_t key, uint32_t lo, float scale, int nb,
                                               const uint16_t* __restrict__ cdf, float share) {
#pragma clang fp contract(off)
    const float f = (float)(key - lo) * scale;
    const int bk = min((int)f, nb - 1);
    const float c0 = (float)cdf[bk], c1 = (float)cdf[bk + 1];
    const float at = c0 + fminf(f - (float)bk, 1.f) * (c1 - c0);
    return min((int)(at * share), nb - 1);
}

// Smallest and largest of the block's values; s2: 2 x waves words.
template <int kThreads>
__device__ __forceinline__ void block_min_max(uint32_t& lo, uint32_t& hi, uint32_t* s2) {
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
    }
    constexpr int W = kThreads / 64;
    if ((threadIdx.x & 63) == 0) {
        s2[threadIdx.x >> 6] = lo;
        s2[W + (threadIdx.x >> 6)] = hi;
    }
    __syncthreads();
    for (int i = 0; i < W; ++i) {
        lo = min(lo, s2[i]);
        hi = max(hi, s2[W + i]);
    }
    __syncthreads();
}

// Exclusive prefixes of the block's n counts in place (c[n] = the total), and
// the largest count; n is a multiple of the threads, PER = n / threads.
template <int kThreads, int PER>
__device__ __forceinline__ uint32_t block_scan_counts(uint32_t* c, uint32_t* s2) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    constexpr int W = kThreads / 64;
    uint32_t v[PER], sum = 0, big = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        v[i] = c[threadIdx.x * PER + i];
        sum += v[i];
        big = max(big, v[i]);
    }
    uint32_t x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    for (int o = 32; o > 0; o >>= 1) big = max(big, (uint32_t)__shfl_xor((int)big, o, 64));
    if (lane == 63) s2[wv] = x;
    if (lane == 0) s2[W + wv] = big;
    __syncthreads();
    uint32_t first = x - sum;
    for (int i = 0; i < W; ++i) {
        first += i < wv ? s2[i] : 0u;
        big = max(big, s2[W + i]);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        c[threadIdx.x * PER + i] = first;
        first += v[i];
    }
    if (threadIdx.x == kThreads - 1) c[kThreads * PER] = first;
    __syncthreads();
    return big;
}


__device__ __forceinline__ void order_pair(uint64_t& x, uint64_t& y) {
    const uint64_t lo = x < y ? x : y, hi = x < y ? y : x;
    x = lo;
    y = hi;
}

// Batcher's odd-even merge sort of K values in registers.
template <int K>
__device__ __forceinline__ void sort_regs(uint64_t (&v)[K]) {
#pragma unroll
    for (int p = 1; p < K; p <<= 1)
#pragma unroll
        for (int k = p; k >= 1; k >>= 1)
#pragma unroll
            for (int j = k % p; j + k < K; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < K && (i + j) / (2 * p) == (i + j + k) / (2 * p)) order_pair(v[i + j], v[i + j + k]);
}

// Merge sort of n <= NS * 8 items, 8 a thread (item i of thread t: v[j], t * 8
// + j, padded with ~0): in registers, then merges of runs twice as long each,
// every thread finding where its 8 outputs begin in the two runs (a binary
// search along the merge path) and merging from there.  Whatever the keys.
// Runs of one wave's threads need no block barrier.
__device__ __forceinline__ void merge_sort(int n, uint64_t* lds, uint64_t (&v)[8]) {
    constexpr int K = 8;
    const int o = threadIdx.x * K;
    sort_regs<K>(v);
    for (int L = K; L < n; L <<= 1) {
        const bool block = 2 * L > 64 * K;
        // (the runs' readers are done: a wave's own LDS accesses complete in order)
        if (block) __syncthreads();
        else __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < K; ++j) lds[(o + j)] = v[j];
        if (block) __syncthreads();
        else __builtin_amdgcn_wave_barrier();
        const int base = o & ~(2 * L - 1), d = o - base;
        if (base + L >= n) continue;  // the second run is all padding: already in order
        const int A = base, B = base + L;
        int lo = d > L ? d - L : 0, hi = d < L ? d : L;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (lds[(A + mid)] <= lds[(B + d - 1 - mid)]) lo = mid + 1;
            else hi = mid;
        }
        int ia = lo, ib = d - lo;
        uint64_t ka = ia < L ? lds[(A + ia)] : ~0ull, kb = ib < L ? lds[(B + ib)] : ~0ull;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const bool ta = ka <= kb;
            v[j] = ta ? ka : kb;
            ia += ta ? 1 : 0;
            ib += ta ? 0 : 1;
            const int i = ta ? ia : ib;
            const uint64_t nx = i < L ? lds[((ta ? A : B) + i)] : ~0ull;
            ka = ta ? nx : ka;
            kb = ta ? kb : nx;
        }
    }
}

// A long list's pieces and chunks: pos, count, and for a piece (by_index) the
// list's first item.
struct SortPiece {
    int32_t pos, n, list, by_index;
};
static_assert(sizeof(SortPiece) == sizeof(int4), "one 16-byte word");

// Huge lists: chunks of kHugeRun items are sorted one by one, then as many
// chunks as there will be groups are merged to one group each, then the groups:
// an item is placed among 2 sqrt(chunks) others' windows, in place of every
// chunk's.  The chunks lie in the list words' two buffers (low and high words;
// the second is free once the items are written), the groups in the items'
// place.  Whole passes of one 32x32 image, with the radix sorts, with one block
// a list and with this: 500,000 Gaussians 646, 858 and 372 us, at one depth
// 702, 2,490 and 312; 2,000,000 735, 20,695 and 575, at one depth 749, 17,404
// and 470; 5,000,000 1,200, not measured and 1,330.  The line lies at 65,536
// items: 130,000 at one depth take 724 us undivided, 282 so, spread ones 284
// and 276.
constexpr int kHugeRun = 4096;
// (Even: blocks eight apart, which share an L2, then have the same part of
// their groups, and the other groups' windows with it.)
__device__ __forceinline__ int huge_group(int n) {
    const int chunks = (n + kHugeRun - 1) / kHugeRun;
    int g = 2;
    while (g * g < chunks) g += 2;
    return g;
}

// The huge lists' units (count(items) each) dealt to `blocks` blocks in turn:
// f(first item of the list, its items, unit).
template <class Count, class Fn>
__device__ __forceinline__ void huge_units(const int32_t* __restrict__ huge_lists, int lists,
                                           const int32_t* __restrict__ ranges, int block, int blocks, Count&& count, Fn&& f) {
    int next = block;
    for (int h = 0; h < lists; ++h) {
        const int S = huge_lists[h], start = ranges[2 * S], n = ranges[2 * S + 1] - start, units = count(n);
        for (; next < units; next += blocks) f(start, n, next);
        next -= units;
    }
}

// Merge of sorted runs: a block takes the (at most) kMergeRun items from `off`
// on of a list of n items in runs of R, `group` runs to a group; an item's
// place in its group is its index in its run plus the items before it in every
// other run of the group, which are found in that run's window between the
// block's first and last item, through LDS (a window much longer than the
// block's items, where the depths are uneven: item by item).
// s_win: kWindow (twice the block's items: most windows are one step), s_at:
// NM words.
constexpr int kMergeRun = 1024, kWindow = 2 * kMergeRun, NM = 256, kLongWindow = 4 * kWindow;
template <class Load, class Put>
__device__ __forceinline__ void merge_runs(Load&& load, Put&& put, int n, int R, int group, int off, uint64_t* s_win,
                                           int* s_at) {
    constexpr int PER = kMergeRun / NM;
    const int own = off / R, runs = (n + R - 1) / R;
    const int g0 = group < runs ? own / group * group : 0, g1 = group < runs ? min(g0 + group, runs) : runs;
    const int r0 = off - own * R;                       // the block's first item within its run
    const int cnt = min(min(n - own * R, R) - r0, kMergeRun);
    uint64_t v[PER];
    int rank[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = (int)threadIdx.x * PER + j;
        v[j] = i < cnt ? load(off + i) : ~0ull;
        rank[j] = r0 + i;
    }
    const uint64_t first = load(off), last = load(off + cnt - 1);
    auto before = [&](int base, int lo, int hi, uint64_t key) {  // items of [base + lo, base + hi) below key, from base
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (load(base + mid) < key) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    };
    for (int c0 = g0; c0 < g1; c0 += NM / 2) {  // the other runs, NM / 2 windows at a time
        const int gn = min(g1 - c0, NM / 2);
        __syncthreads();
        if ((int)threadIdx.x < 2 * gn) {
            const int q = threadIdx.x >> 1, base = (c0 + q) * R;
            s_at[threadIdx.x] = before(base, 0, min(n - base, R), threadIdx.x & 1 ? last : first);
        }
        __syncthreads();
        for (int q = 0; q < gn; ++q) {
            if (c0 + q == own) continue;
            const int wl = s_at[2 * q], wh = s_at[2 * q + 1], base = (c0 + q) * R;  // (block-uniform)
            if (wh - wl > kLongWindow) {
#pragma unroll
                for (int j = 0; j < PER; ++j) rank[j] += before(base, wl, wh, v[j]);
                continue;
            }
#pragma unroll
            for (int j = 0; j < PER; ++j) rank[j] += wl;
            for (int t0 = wl; t0 < wh; t0 += kWindow) {
                const int tn = min(wh - t0, kWindow);
                uint64_t w[kWindow / NM];  // (all on their way together)
#pragma unroll
                for (int u = 0; u < kWindow / NM; ++u) {
                    const int i = u * NM + (int)threadIdx.x;
                    w[u] = i < tn ? load(base + t0 + i) : 0;
                }
                __syncthreads();
#pragma unroll
                for (int u = 0; u < kWindow / NM; ++u) {
                    const int i = u * NM + (int)threadIdx.x;
                    if (i < tn) s_win[i] = w[u];
                }
                __syncthreads();
                // (a thread's items are neighbours: the first one's place by
                // bisection, the others' from there on in growing steps)
                int lo = 0, hi = tn;
#pragma unroll
                for (int j = 0; j < PER; ++j) {
                    if (j) {
                        int step = 1;
                        hi = lo;
                        while (hi < tn && s_win[hi] < v[j]) {
                            lo = hi + 1;
                            hi += step;
                            step <<= 1;
                        }
                        hi = min(hi, tn);
                    }
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if (s_win[mid] < v[j]) lo = mid + 1;
                        else hi = mid;
                    }
                    rank[j] += lo;
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = (int)threadIdx.x * PER + j;
        if (i < cnt) put(g0 * R + rank[j], v[j]);
    }
    __syncthreads();
}

// Divides the long lists by depth: a block per list counts its items into
// kSplitBuckets buckets between its nearest and farthest, writes the items'
// indices in bucket order to the list's (not yet used) words, and hands the
// buckets out as pieces of up to kSortCap items, kPieceRun on average.  The
// items themselves stay where they are.  A list that this does not divide
// (one bucket holds too much) is sorted in chunks and merged instead.  Bound by the latency of its three
// passes over the list, so the first 4,096 keys, all of most lists, are read
// once, the others' next step is loaded while a step is counted or placed, and
// half as many threads as a block may have let the lists of a frame be in
// flight together: the city's 48 -> 41 us high above it, and 107 -> 88 near
// the ground, where lists have up to 46,000 items (before the loads ahead).
// Steps twice as long, by keys or by threads, take as long or longer (93, 89).
constexpr int NP = 512;
constexpr int kHeld = 8;  // keys of a list a thread keeps in registers
constexpr int kPieceBlocks = 3072;
constexpr int kSplitBuckets = 8192;
constexpr int kPieceRun = kSortCap / 2;
constexpr int kMaxPieces = kHugeList / kPieceRun;
__global__ __launch_bounds__(NP) void k_bin_split(const uint64_t* __restrict__ items, const int32_t* __restrict__ ranges,
                                                  const int32_t* __restrict__ long_lists,
                                                  const int32_t* __restrict__ huge_lists, RasterCounters* rc,
                                                  SortPiece* __restrict__ pieces, uint2* __restrict__ chunks,
                                                  uint32_t* __restrict__ words, uint32_t* __restrict__ high_words) {
    __shared__ __align__(16) uint32_t s_cnt[kSplitBuckets + 1];
    __shared__ uint32_t s_piece[kMaxPieces + 1];
    __shared__ uint32_t s_red[2 * NP / 64];
    static_assert(kHugeRun == NP * 8 && kHugeRun * 2 <= kSplitBuckets, "a chunk is 8 items a thread and fits the counts' place");
    const int nl = rc->n_long, nh = rc->n_huge;  // (one load)
    if (nh)
        huge_units(huge_lists, nh, ranges, blockIdx.x, gridDim.x, [](int n) { return (n + kHugeRun - 1) / kHugeRun; },
                   [&](int start, int n, int unit) {
            const int off = unit * kHugeRun, m = min(n - off, kHugeRun), o = threadIdx.x * 8;
            const uint64_t* src = items + start + off;
            uint64_t v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = o + j < m ? src[o + j] : ~0ull;
            merge_sort(m, reinterpret_cast<uint64_t*>(s_cnt), v);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (o + j < m) {
                    words[start + off + o + j] = (uint32_t)v[j];
                    high_words[start + off + o + j] = (uint32_t)(v[j] >> 32);
                }
            __syncthreads();
        });
    for (int li = blockIdx.x; li < nl; li += gridDim.x) {
        const int S = long_lists[li];
        const int start = ranges[2 * S], n = ranges[2 * S + 1] - start;
        const uint64_t* src = items + start;
        // A step is kHeld keys of every thread.  The first step's stay in
        // registers for the three passes (many long lists have no more); the
        // others' are loaded a step ahead.
        const uint32_t* keys = reinterpret_cast<const uint32_t*>(src) + 1;
        uint32_t held[kHeld], lo = 0xffffffffu, hi = 0u;
        auto load = [&](int base, uint32_t (&k)[kHeld]) {
#pragma unroll
            for (int j = 0; j < kHeld; ++j) {
                const int i = base + j * NP + (int)threadIdx.x;
                k[j] = i < n ? keys[2 * (int64_t)i] : 0u;
            }
        };
        load(0, held);
        auto steps = [&](auto&& f) {
            uint32_t cur[kHeld], next[kHeld] = {};
#pragma unroll
            for (int j = 0; j < kHeld; ++j) cur[j] = held[j];
            for (int base = 0; base < n; base += kHeld * NP) {  // block-uniform
                if (base + kHeld * NP < n) load(base + kHeld * NP, next);
                f(base + (int)threadIdx.x, cur, base + kHeld * NP <= n);
#pragma unroll
                for (int j = 0; j < kHeld; ++j) cur[j] = next[j];
            }
        };
        steps([&](int i, const uint32_t (&k)[kHeld], bool) {
#pragma unroll
            for (int j = 0; j < kHeld; ++j)
                if (i + j * NP < n) {
                    lo = min(lo, k[j]);
                    hi = max(hi, k[j]);
                }
        });
        for (int i = threadIdx.x; i < kSplitBuckets; i += NP) s_cnt[i] = 0u;
        block_min_max<NP>(lo, hi, s_red);
        const float scale = bucket_scale(lo, hi, kSplitBuckets);
        steps([&](int i, const uint32_t (&k)[kHeld], bool) {
#pragma unroll
            for (int j = 0; j < kHeld; ++j)
                if (i + j * NP < n) atomicAdd(&s_cnt[bucket_of(k[j], lo, scale, kSplitBuckets)], 1u);
        });
        __syncthreads();
        const uint32_t big = block_scan_counts<NP, kSplitBuckets / NP>(s_cnt, s_red);
        const int np = (n + kPieceRun - 1) / kPieceRun;
        if (big > (uint32_t)kPieceRun) {  // block-uniform
            if (threadIdx.x == 0) {
                const int m = (n + kSortCap - 1) / kSortCap, at = atomicAdd(&rc->n_chunks, m);
                for (int q = 0; q < m; ++q) chunks[at + q] = make_uint2((uint32_t)S, (uint32_t)q);
            }
            __syncthreads();
            continue;
        }
        // piece p begins at the first bucket that begins at or after p * kPieceRun
        for (int i = threadIdx.x; i <= np; i += NP) s_piece[i] = (uint32_t)n;
        __syncthreads();
        for (int i = threadIdx.x; i < kSplitBuckets; i += NP)
            if (s_cnt[i + 1] > s_cnt[i]) atomicMin(&s_piece[s_cnt[i] / kPieceRun], s_cnt[i]);
        __syncthreads();
        for (int p = threadIdx.x; p < np; p += NP) {
            const uint32_t first = s_piece[p];
            if (first >= (uint32_t)n) continue;  // no bucket begins there
            int q = p + 1;
            while (q < np && s_piece[q] >= (uint32_t)n) ++q;
            const uint32_t end = q < np ? s_piece[q] : (uint32_t)n;
            pieces[atomicAdd(&rc->n_pieces, 1)] = SortPiece{start + (int)first, (int)(end - first), start, 1};
        }
        __syncthreads();  // (the prefixes become cursors)
        steps([&](int i, const uint32_t (&k)[kHeld], bool full) {
            if (full) {  // (the step's places asked for together)
                uint32_t at[kHeld];
#pragma unroll
                for (int j = 0; j < kHeld; ++j) at[j] = atomicAdd(&s_cnt[bucket_of(k[j], lo, scale, kSplitBuckets)], 1u);
#pragma unroll
                for (int j = 0; j < kHeld; ++j) words[start + (int)at[j]] = (uint32_t)(i + j * NP);
            } else {
#pragma unroll
                for (int j = 0; j < kHeld; ++j)
                    if (i + j * NP < n)
                        words[start + (int)atomicAdd(&s_cnt[bucket_of(k[j], lo, scale, kSplitBuckets)], 1u)] =
                            (uint32_t)(i + j * NP);
            }
        });
        __syncthreads();  // before the next list
    }
}

// Blocks up to total_sup: one super tile's list each, if it fits; the blocks
// after them: the long lists' pieces, and the chunks for k_bin_merge (in
// place).
//
// A list is spread over buckets between its nearest and farthest item (four
// items or so each), an item's place among its bucket's is the number of
// smaller ones there: O(n) LDS accesses, where a merge sort's twelve rounds
// of data-dependent reads conflict on the banks at every step.  Where the
// depths crowd (a near footprint among far ones is enough), the counts
// themselves say how: read as a piecewise linear distribution function they
// spread the same keys over buckets of equal share.  What still crowds after
// that (ties, mostly) takes the merge sort.
// Latency again (barriers, LDS round trips): seven blocks a CU, and a block
// per piece up to 3,072 of them (1,024, three pieces one after another, left a
// third of the chip idle at the end): the city's 75 -> 57 us.
constexpr int kBuckets = 1024;
constexpr uint32_t kCrowd = 64;
__global__ __launch_bounds__(NS) __attribute__((amdgpu_waves_per_eu(7))) void k_bin_sort(uint64_t* __restrict__ items, const int32_t* __restrict__ ranges,
                                                 int total_sup, const RasterCounters* rc,
                                                 const SortPiece* __restrict__ pieces,
                                                 const uint2* __restrict__ chunks, uint32_t* __restrict__ words,
                                                 const int32_t* __restrict__ huge_lists,
                                                 const uint32_t* __restrict__ high_words, int32_t* status) {
    if (status && blockIdx.x == 0 && threadIdx.x == 0) *status = rc->overflow;  // (final since k_bin<true>)
    __shared__ uint64_t lds[kSortCap];
    __shared__ uint32_t s_cnt[kBuckets + 1];
    __shared__ uint16_t s_cdf[kBuckets + 2];
    __shared__ uint32_t s_red[2 * NS / 64];
    const bool own = (int)blockIdx.x < total_sup;
    const int np = own ? 1 : rc->n_pieces, total = own ? 1 : np + rc->n_chunks;
    const int step = own ? 1 : (int)gridDim.x - total_sup;
    // Blocks go to the 8 XCDs in turn: an eighth of the pieces in a row to
    // each, so that a list's pieces, which gather its items from all over it,
    // read one L2 (frames near the ground, 8 M items in pieces: 81 -> 62 us).
    const int per = (total + 7) / 8, rounds = own ? 1 : 8 * per;
    for (int b = own ? 0 : (int)blockIdx.x - total_sup; b < rounds; b += step) {  // block-uniform
        const int i = own ? 0 : (b & 7) * per + (b >> 3);
        if (i >= total) continue;
        SortPiece p;
        if (own) {
            p = SortPiece{ranges[2 * blockIdx.x], 0, 0, 0};
            p.n = ranges[2 * blockIdx.x + 1] - p.pos;
            if (p.n <= 0 || p.n > kSortCap) return;
        } else if (i < np) {
            p = pieces[i];
        } else {
            const uint2 ch = chunks[i - np];
            p = SortPiece{ranges[2 * ch.x] + (int)ch.y * kSortCap, 0, 0, 2};
            p.n = min(ranges[2 * ch.x + 1] - p.pos, kSortCap);
        }
        const int n = p.n;
        if (p.by_index < 2) {
            uint64_t v[8];
            uint32_t r[8];
            uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = j * NS + (int)threadIdx.x;
                v[j] = ~0ull;
                if (k < n) {
                    v[j] = p.by_index ? items[p.list + words[p.pos + k]] : items[p.pos + k];
                    lo = min(lo, (uint32_t)(v[j] >> 32));
                    hi = max(hi, (uint32_t)(v[j] >> 32));
                }
            }
            for (int k = threadIdx.x; k < kBuckets; k += NS) s_cnt[k] = 0u;
            block_min_max<NS>(lo, hi, s_red);
            const float scale = bucket_scale(lo, hi, kBuckets);
            bool eq = false;  // equalised buckets
            const float share = (float)kBuckets / (float)n;
            auto bucket = [&](uint64_t x) {
                const uint32_t key = (uint32_t)(x >> 32);
                return eq ? bucket_by_share(key, lo, scale, kBuckets, s_cdf, share) : bucket_of(key, lo, scale, kBuckets);
            };
            auto count = [&]() {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (j * NS + (int)threadIdx.x < n) r[j] = atomicAdd(&s_cnt[bucket(v[j])], 1u);
                __syncthreads();
                return block_scan_counts<NS, kBuckets / NS>(s_cnt, s_red);
            };
            uint32_t big = count();
            if (big > kCrowd) {  // block-uniform
                for (int k = threadIdx.x; k <= kBuckets; k += NS) s_cdf[k] = (uint16_t)s_cnt[k];
                __syncthreads();
                for (int k = threadIdx.x; k < kBuckets; k += NS) s_cnt[k] = 0u;
                eq = true;
                __syncthreads();
                big = count();
            }
            if (big <= kCrowd) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (j * NS + (int)threadIdx.x < n) lds[s_cnt[bucket(v[j])] + r[j]] = v[j];
                __syncthreads();
                for (int k = threadIdx.x; k < n; k += NS) {
                    const uint64_t x = lds[k];
                    const int bk = bucket(x);
                    const int b0 = (int)s_cnt[bk], b1 = (int)s_cnt[bk + 1];
                    int at = b0;
                    for (int q = b0; q < b1; ++q) at += lds[q] < x ? 1 : 0;
                    words[p.pos + at] = list_word(x);
                }
                __syncthreads();  // before the next piece
                continue;
            }
            // crowded: back to 8 consecutive items a thread
#pragma unroll
            for (int j = 0; j < 8; ++j) lds[(j * NS + (int)threadIdx.x)] = v[j];
            __syncthreads();
            const int o = threadIdx.x * 8;
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = lds[(o + j)];
            __syncthreads();
            merge_sort(n, lds, v);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (o + j < n) words[p.pos + o + j] = list_word(v[j]);
        } else {
            uint64_t v[8];
            const int o = threadIdx.x * 8;
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = o + j < n ? items[p.pos + o + j] : ~0ull;
            merge_sort(n, lds, v);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (o + j < n) items[p.pos + o + j] = v[j];
        }
        __syncthreads();
    }
    if (!own && rc->n_huge)
        huge_units(huge_lists, rc->n_huge, ranges, (int)blockIdx.x - total_sup, step,
                   [](int n) { return (n + kMergeRun - 1) / kMergeRun; }, [&](int start, int n, int unit) {
            const uint32_t* low = words + start;
            const uint32_t* high = high_words + start;
            uint64_t* out = items + start;
            merge_runs([&](int i) { return ((uint64_t)high[i] << 32) | low[i]; }, [&](int i, uint64_t v) { out[i] = v; }, n,
                       kHugeRun, huge_group(n), unit * kMergeRun, lds, reinterpret_cast<int*>(s_cnt));
        });
}

// The chunks of the crowded lists, and the groups of the huge ones, merged to
// the lists' words.
__global__ __launch_bounds__(NM) void k_bin_merge(const uint64_t* __restrict__ items,
                                                  const int32_t* __restrict__ ranges, const RasterCounters* rc,
                                                  const uint2* __restrict__ chunks,
                                                  const int32_t* __restrict__ huge_lists, uint32_t* __restrict__ words) {
    constexpr int kUnits = kSortCap / kMergeRun;
    __shared__ uint64_t s_win[kWindow];
    __shared__ int s_at[NM];
    auto merge = [&](int start, int n, int R, int off) {
        const uint64_t* list = items + start;
        uint32_t* out = words + start;
        merge_runs([&](int i) { return list[i]; }, [&](int i, uint64_t v) { out[i] = list_word(v); }, n, R, 1 << 30, off, s_win,
                   s_at);
    };
    const int nu = rc->n_chunks * kUnits;
    for (int u = blockIdx.x; u < nu; u += gridDim.x) {
        const uint2 ch = chunks[u / kUnits];
        const int start = ranges[2 * ch.x], n = ranges[2 * ch.x + 1] - start;
        const int off = (int)ch.y * kSortCap + (u % kUnits) * kMergeRun;
        if (off < n) merge(start, n, kSortCap, off);  // block-uniform
    }
    if (rc->n_huge)
        // (the same part of every group one after another, eight parts side by side, for the L2s)
        huge_units(huge_lists, rc->n_huge, ranges, blockIdx.x, gridDim.x,
                   [](int n) {
                       const int R = kHugeRun * huge_group(n);
                       return (n + R - 1) / R * (R / kMergeRun);
                   },
                   [&](int start, int n, int unit) {
                       const int R = kHugeRun * huge_group(n), runs = (n + R - 1) / R, w = unit >> 3;
                       const int off = w % runs * R + (w / runs * 8 + (unit & 7)) * kMergeRun;
                       if (off < n) merge(start, n, R, off);
                   });
}

}  // namespace

hipError_t bin_items(const SegTable& tab, Raster& r, int32_t* status, hipStream_t st, Marks* mk) {
    BinArgs a;
    for (int q = 0; q < kMaxSeg; ++q)
        a.sg[q] = SupGeo{q < tab.n ? tab.s[q].sup_base : 0, q < tab.n ? tab.s[q].nsx : 0};
    a.rc = r.cnt; a.rec = r.rec; a.brec = r.brec; a.srow = r.srow; a.srow_y = r.srow_y; a.srow_cap = r.srow_cap;
    a.items = r.items; a.ranges = r.ranges; a.n_sort = r.n_sort; a.long_lists = r.long_lists; a.huge_lists = r.huge_lists;
    a.max_pairs = r.max_pairs; a.total_sup = tab.total_sup;
    a.stride = (tab.total_sup + kColTile - 1) / kColTile * kColTile;
    if (a.stride > kBinLists) return hipErrorInvalidValue;
    const int64_t entries = entry_bound(tab, r.max_entries);
    // Blocks: one per run of entries, up to what two blocks on every CU hold
    // (more only lengthen k_bin_columns), within the counts' buffer.  A batch
    // that runs of 1,024 would leave on a few CUs takes shorter ones, with
    // fewer footprints to a wave (k_bin<true> of 60,000 Gaussians 18 -> 13 us,
    // of 2,000 13 -> 9 us).  The counts lie in a buffer of the radix sorts,
    // idle here: the second value buffer, or the digit counts where that is
    // smaller.
    const int64_t digits = 256 * (int64_t)kSortBlocks, hist_cap = r.max_pairs > digits ? r.max_pairs : digits;
    a.run = entries <= 64 * 1024 ? 256 : (entries <= 128 * 1024 ? 512 : 1024);
    int64_t nblk = (entries + a.run - 1) / a.run;
    if (nblk > kMaxBinBlocks) nblk = kMaxBinBlocks;
    if (nblk > hist_cap / a.stride) nblk = hist_cap / a.stride;
    if (nblk < 1) nblk = 1;
    if (nblk >= 8) nblk &= ~(int64_t)7;
    a.hist = r.max_pairs > digits ? r.pval[1] : r.hist;
    a.total = r.sup_total;
    a.kept = r.block_sums;
    mark(mk, 6, st);
    hipLaunchKernelGGL(k_bin<false>, dim3((unsigned)nblk), dim3(NB), 0, st, a);
    hipLaunchKernelGGL(k_bin_columns, dim3((unsigned)(a.stride / kColTile)), dim3(NB), 0, st, a.hist, r.sup_total,
                       (int)nblk, a.stride);
    mark(mk, 7, st);
    hipLaunchKernelGGL(k_bin<true>, dim3((unsigned)nblk), dim3(NB), 0, st, a);
    mark(mk, 8, st);
    mark(mk, 9, st);
    mark(mk, 10, st);
    // a list longer than kSortCap needs as many entries
    const bool longer = entries > kSortCap;
    // (blocks for the pieces, a few entries' worth each: without work they cost
    // a small batch more than they take from a large one)
    const int64_t piece_blocks = !longer ? 0 : (entries < 256 * kPieceBlocks ? (entries + 255) / 256 : kPieceBlocks);
    SortPiece* pieces = reinterpret_cast<SortPiece*>(r.pieces);
    // (a block per long list, of which there are no more than super tiles, or per huge list's chunk)
    const int64_t chunks = entries > kHugeList ? (entries + kHugeRun - 1) / kHugeRun : 0;
    const int64_t split_blocks = chunks > tab.total_sup ? chunks : tab.total_sup;
    if (longer)
        hipLaunchKernelGGL(k_bin_split, grid_fit(k_bin_split, split_blocks * NP, NP), dim3(NP), 0, st, r.items,
                           r.ranges, r.long_lists, r.huge_lists, r.cnt, pieces, r.chunks, r.pval[0], r.pval[1]);
    hipLaunchKernelGGL(k_bin_sort, dim3((unsigned)(tab.total_sup + (unsigned)piece_blocks)), dim3(NS), 0, st, r.items,
                       r.ranges, tab.total_sup, r.cnt, pieces, r.chunks, r.pval[0], r.huge_lists, r.pval[1], status);
    // (two blocks a CU for the crowded lists; as many as fit for huge ones, 2 M
    // items 692 -> 439 us)
    const int64_t merge_units = chunks * (kHugeRun / kMergeRun);
    if (longer)
        hipLaunchKernelGGL(k_bin_merge, grid_fit(k_bin_merge, (merge_units > 512 ? merge_units : 512) * NM, NM), dim3(NM), 0, st,
                           r.items, r.ranges, r.cnt, r.chunks, r.huge_lists, r.pval[0]);
    mark(mk, 11, st);
    r.sorted_buf = 0;
    return hipGetLastError();
}

}  // namespace gsc
