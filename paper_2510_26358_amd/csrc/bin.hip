// Tile binning: per-tile Gaussian lists in depth order, for all views at once.
//
// Order definition: every (view b, Gaussian i, tile) intersection carries the key
// (global tile, float32 depth bits) and the lists are the stable ascending order of those
// keys over emission order (b, i, ty, tx) -- ties resolve by ascending pair id.
//
// Instead of radix-sorting 64-bit keys over all K intersections, the visible pairs are
// depth-sorted once (V << K items, 32-bit keys) and their intersections are emitted in
// that order; a stable sort on the tile id alone then yields exactly the same order
// (LSD radix passes are stable).  Bytes moved: 4 passes x V + ceil(tile_bits / 8) passes
// x K instead of 6 passes x K with 12-byte records.  Launches with few intersections sort
// each tile's list by itself instead (see per_tile_sort): fewer launches, the same lists.
#include "common.h"

namespace ags {

// Emission.  Output slot k belongs to the last pair j (depth order) with emit_off[j] <= k and
// is slot k - emit_off[j] of that pair's tile rectangle (row-major).  A workgroup fills
// kEmitSlots consecutive slots; since every visible pair owns >= 1 slot, they belong to at
// most kEmitSlots consecutive pairs starting at block_first[workgroup].  Their offsets, and
// for each pair the rectangle's first tile, its width, the view and the ellipse (centre,
// conic, level), are staged in LDS (one thread per pair); each pair marks its first slot
// and a prefix maximum over the slots gives every slot its pair.  A slot whose tile the
// alpha >= alpha_min ellipse does not reach (tile_reached) gets the key n_tiles, which the
// tile sort's first pass drops.  Balanced however unequal the footprints are, and the
// writes are coalesced.
//
// RANK (the pairs are in pair order): the kernel also counts each tile's intersections and writes each
// one's rank in that count to tile_rank.  There are kTileCounts counts [kTileCounts][n_tiles], cleared
// before, of which workgroup g uses number g % kTileCounts: consecutive workgroups run on the eight
// XCDs in turn, so a counter's cache line stays in one XCD's L2 instead of moving between them for
// every atomic (one 960 x 600 view over 300k Gaussians, one count: 66 us, eight 29, sixteen 20; without
// counts 8).
constexpr int kEmitThreads = 256;
constexpr int kTileCounts = 16;   // a multiple of the XCDs
constexpr int kEmitTogether = 8;  // lanes of one tile that share an addition

__device__ __forceinline__ uint32_t lanes_before(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

template <bool RANK>
__global__ __launch_bounds__(kEmitThreads) void emit_kernel(ViewTable vt, const float* records,
                                                            const uint32_t* depth_vals, const uint32_t* emit_off,
                                                            const uint32_t* block_first, const uint32_t* counters,
                                                            long long capacity, uint32_t* tile_keys,
                                                            uint32_t* tile_vals, uint32_t* tile_rank,
                                                            uint32_t* tile_count, uint32_t* ranges) {
    constexpr int S = kEmitSlots, PT = S / kEmitThreads;
    __shared__ uint32_t s_off[S];
    __shared__ uint32_t s_own[S];                     // slot -> local pair index
    __shared__ uint32_t s_q[S], s_first[S];           // pair, global id of the rectangle's first tile
    __shared__ uint32_t s_wp[S], s_org[S], s_wh[S];   // width | pitch << 16, tx0 | ty0 << 16, W | H << 16
    __shared__ float4 s_ell[S];                       // u, v, a, b
    __shared__ float2 s_ell2[S];                      // c, level
    __shared__ uint32_t s_wmax[kEmitThreads / 64];
    const long long k0 = (long long)blockIdx.x * S;
    const uint32_t n_tiles = (uint32_t)vt.tile_base[vt.n_views];
    // every tile's range starts empty; ranges_kernel later sets the non-empty ones
    if (!RANK) {
        for (long long e = (long long)blockIdx.x * kEmitThreads + threadIdx.x; e < 2LL * n_tiles;
             e += (long long)gridDim.x * kEmitThreads)
            ranges[e] = 0u;
    }
    long long keff = counters[CNT_KEFF];
    if (keff > capacity) keff = capacity;
    const long long nv = counters[CNT_V];
    if (k0 >= keff || nv == 0) return;  // uniform per workgroup
    const long long j0 = block_first[blockIdx.x];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    // the workgroup's pairs: from the owner of its first slot to the owner of the next
    // workgroup's first slot (or the last pair); pairs starting at or beyond the workgroup's
    // last slot are not needed
    const long long kend = k0 + S < keff ? k0 + S : keff;
    const long long jlast = k0 + S < keff ? (long long)block_first[blockIdx.x + 1] : nv - 1;
#pragma unroll
    for (int c = 0; c < PT; ++c) {
        const int l = c * kEmitThreads + t;
        const long long j = j0 + l;
        const uint32_t off = j <= jlast ? emit_off[j] : 0xFFFFFFFFu;
        s_off[l] = off;
        s_own[l] = 0u;
        if ((long long)off < kend) {
            const uint32_t q = depth_vals[j];
            const int b = view_of_pair(vt, q);
            const float4* rec = reinterpret_cast<const float4*>(records + (long long)q * kRecFloats);
            const float4 r0 = rec[0], r1 = rec[1], r2 = rec[2];
            const int W = vt.width[b], H = vt.height[b];
            int tx0 = 0, ty0 = 0, tx1 = 0, ty1 = 0;
            tile_rect(r0.x, r0.y, r1.w, r2.x, W, H, vt.tile, tx0, ty0, tx1, ty1);
            s_q[l] = q;
            s_first[l] = (uint32_t)(vt.tile_base[b] + ty0 * vt.ntx[b] + tx0);
            s_wp[l] = (uint32_t)(tx1 - tx0 + 1) | ((uint32_t)vt.ntx[b] << 16);
            s_org[l] = (uint32_t)tx0 | ((uint32_t)ty0 << 16);
            s_wh[l] = (uint32_t)W | ((uint32_t)H << 16);
            s_ell[l] = make_float4(r0.x, r0.y, r0.z, r0.w);
            s_ell2[l] = make_float2(r1.x, tile_tau2(r0.z, r0.w, r1.x, r1.w));
        }
    }
    __syncthreads();
    // slot -> pair: each pair after the first marks its first slot, a prefix maximum fills the
    // rest (every visible pair owns at least one slot, so the marks are distinct)
#pragma unroll
    for (int c = 0; c < PT; ++c) {
        const int l = c * kEmitThreads + t;
        const long long off = (long long)s_off[l];
        if (l > 0 && off < kend) s_own[off - k0] = (uint32_t)l;
    }
    __syncthreads();
    {
        uint32_t v[PT], m = 0;
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            v[i] = max(m, s_own[PT * t + i]);
            m = v[i];
        }
        uint32_t incl = m;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)incl, o, 64);
            if (lane >= o) incl = max(incl, y);
        }
        if (lane == 63) s_wmax[wv] = incl;
        uint32_t excl = (uint32_t)__shfl_up((int)incl, 1, 64);
        if (lane == 0) excl = 0;
        __syncthreads();
#pragma unroll
        for (int x = 0; x < kEmitThreads / 64; ++x)
            if (x < wv) excl = max(excl, s_wmax[x]);
#pragma unroll
        for (int i = 0; i < PT; ++i) s_own[PT * t + i] = max(excl, v[i]);
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < PT; ++c) {
        const long long k = k0 + c * kEmitThreads + t;
        if (k >= keff) break;
        const uint32_t lo = s_own[k - k0];
        const uint32_t r = (uint32_t)(k - (long long)s_off[lo]);
        const uint32_t wp = s_wp[lo], org = s_org[lo], wh = s_wh[lo];
        const uint32_t w = wp & 0xFFFFu;
        // r / w through the float reciprocal: the quotient is at most the rectangle's tile rows
        // (views are under 65,536 pixels a side, so under 2^13 rows), which keeps the float
        // estimate within a hundredth of it, so truncation is off by at most one; the two
        // steps below correct that exactly
        uint32_t row = (uint32_t)((float)r * __builtin_amdgcn_rcpf((float)w));
        row -= row * w > r ? 1u : 0u;
        row += (row + 1u) * w <= r ? 1u : 0u;
        const uint32_t col = r - row * w;
        const int tx = (int)(org & 0xFFFFu) + (int)col;
        const int ty = (int)(org >> 16) + (int)row;
        const float4 e = s_ell[lo];
        const float2 e2 = s_ell2[lo];
        const bool hit = tile_reached(e.x, e.y, e.z, e.w, e2.x, e2.y, tx, ty, vt.tile, (int)(wh & 0xFFFFu),
                                      (int)(wh >> 16));
        const uint32_t tile = hit ? s_first[lo] + row * (wp >> 16) + col : n_tiles;
        tile_keys[k] = tile;
        tile_vals[k] = s_q[lo];
        if (RANK && hit) {
            // Lanes of one tile add together where many meet (a far view's Gaussians in a few tiles: 300k in
            // one tile 287 -> 12 us); the wave's additions are still one instruction, with one wait.
            uint32_t* const count = tile_count + (size_t)(blockIdx.x % kTileCounts) * n_tiles;
            const int self = __lane_id();
            int lead = self;
            uint32_t together = 1, before = 0;
            for (unsigned long long left = __builtin_amdgcn_ballot_w64(true); left;) {
                const int l = __builtin_ctzll(left);
                const unsigned long long same =
                    __builtin_amdgcn_ballot_w64(tile == (uint32_t)__builtin_amdgcn_readlane((int)tile, l)) & left;
                if (__popcll(same) < kEmitTogether) break;
                if ((same >> self) & 1ull) {
                    lead = l;
                    together = (uint32_t)__popcll(same);
                    before = lanes_before(same);
                }
                left &= ~same;
            }
            uint32_t rank = 0;
            if (lead == self) rank = atomicAdd(count + tile, together);
            rank = (uint32_t)__shfl((int)rank, lead, 64) + before;
            tile_rank[k] = rank;
        }
    }
}

// Tile ranges of the sorted list: four consecutive entries per thread, each compared with
// its neighbours; only entries that open or close a tile's run write.
constexpr int kRangeItems = 4;
__global__ __launch_bounds__(256) void ranges_kernel(const uint32_t* keys, const uint32_t* counters,
                                                     long long n_max, uint32_t n_tiles, uint32_t* ranges) {
    long long n = counters[CNT_LIVE];
    if (n > n_max) n = n_max;
    const long long k0 = ((long long)blockIdx.x * blockDim.x + threadIdx.x) * kRangeItems;
    if (k0 >= n) return;
    uint32_t v[kRangeItems + 2];
    v[0] = k0 > 0 ? keys[k0 - 1] : 0xFFFFFFFFu;
    if (k0 + kRangeItems <= n) {
        const uint4 x = *reinterpret_cast<const uint4*>(keys + k0);  // k0 is a multiple of 4
        v[1] = x.x; v[2] = x.y; v[3] = x.z; v[4] = x.w;
    } else {
#pragma unroll
        for (int j = 0; j < kRangeItems; ++j) v[1 + j] = k0 + j < n ? keys[k0 + j] : 0xFFFFFFFFu;
    }
    v[kRangeItems + 1] = k0 + kRangeItems < n ? keys[k0 + kRangeItems] : 0xFFFFFFFFu;
#pragma unroll
    for (int j = 0; j < kRangeItems; ++j) {
        const long long k = k0 + j;
        const uint32_t t = v[1 + j];
        if (k >= n || t >= n_tiles) continue;
        if (v[j] != t) ranges[2 * (long long)t] = (uint32_t)k;
        if (v[2 + j] != t) ranges[2 * (long long)t + 1] = (uint32_t)(k + 1);
    }
}

// Raster work order (see kWorkStrip): per XCD, its tiles by descending list length in 64
// buckets of 4 log2(length + 1), so the few heavy tiles start early instead of trailing the
// launch, while neighbouring tiles (which share records) stay on one XCD's L2.  Workgroup x
// builds XCD x's list, the slots 8 k + x: it clears them to kNoTile, counts its tiles per
// bucket in LDS, scans the counts in descending bucket order, and lets each tile claim a
// slot of its bucket (the order inside a bucket is that of the claims; any order gives the
// same image).
constexpr int kWorkThreads = 1024, kWorkBuckets = 64;
template <typename Len>
__device__ __forceinline__ void work_list_of(int x, int n_tiles, int n_slots, uint32_t* work, Len length) {
    __shared__ uint32_t cnt[kWorkBuckets];
    const int t = threadIdx.x;
    const int per = n_slots / 8;  // slots of one XCD list (a whole number of strips)
    if (t < kWorkBuckets) cnt[t] = 0;
    for (int k = t; k < per; k += kWorkThreads) work[8 * k + x] = kNoTile;
    __syncthreads();
    // i-th tile of XCD x: strip x + 8 (i / kWorkStrip), position i % kWorkStrip in it
    auto tile_of = [&](int i) { return (x + 8 * (i / kWorkStrip)) * kWorkStrip + i % kWorkStrip; };
    auto bucket = [&](int tile) {
        const int b = (int)(4.f * log2f((float)length(tile) + 1.f));
        return b < kWorkBuckets - 1 ? b : kWorkBuckets - 1;
    };
    for (int i = t; i < per; i += kWorkThreads) {
        const int tile = tile_of(i);
        if (tile < n_tiles) atomicAdd(&cnt[bucket(tile)], 1u);
    }
    __syncthreads();
    if (t == 0) {  // exclusive ranks, largest bucket first
        uint32_t run = 0;
        for (int b = kWorkBuckets - 1; b >= 0; --b) {
            const uint32_t c = cnt[b];
            cnt[b] = run;
            run += c;
        }
    }
    __syncthreads();
    for (int i = t; i < per; i += kWorkThreads) {
        const int tile = tile_of(i);
        if (tile < n_tiles) work[8 * atomicAdd(&cnt[bucket(tile)], 1u) + x] = (uint32_t)tile;
    }
}

__global__ __launch_bounds__(kWorkThreads) void work_list_kernel(const uint32_t* ranges, int n_tiles, int n_slots,
                                                                 uint32_t* work) {
    work_list_of((int)blockIdx.x, n_tiles, n_slots, work,
                 [&](int tile) { return ranges[2 * tile + 1] - ranges[2 * tile]; });
}

// ------------------------------------------------------------------------- per-tile sort
//
// The other way to the same lists, for launches whose lists are short: the pairs are emitted in pair
// order, each intersection takes its place in its tile by a counter, and each tile's list is sorted by (depth
// bits, pair id).  Six launches instead of 23 (seven where lists may be long), of which none reads more than a few
// megabytes: a launch costs about 4.5 us however little it does, so the two radix sorts cost about
// 170 us of a 300k-Gaussian single view's step and 60 us of one over 4k.
//
// pair_reduce_kernel and pair_apply_kernel compact the visible pairs in pair order and scan their tile
// counts: out[j] = first slot of the j-th visible pair, which[j] = that pair, block_first as for
// emit_apply_kernel, and the counters.  sums: [gridDim][2] (slots, visible pairs) of each block.
constexpr int kPairThreads = 256, kPairItems = 8, kPairBlock = kPairThreads * kPairItems;

__device__ __forceinline__ uint2 wave_inclusive2(uint2 v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = (uint32_t)__shfl_up((int)v.x, o, 64), y = (uint32_t)__shfl_up((int)v.y, o, 64);
        if (lane >= o) {
            v.x += x;
            v.y += y;
        }
    }
    return v;
}

// Inclusive scan over the workgroup; `total` of all threads.
__device__ __forceinline__ uint2 block_inclusive2(uint2 v, uint2* wave_tot, uint2& total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    v = wave_inclusive2(v, lane);
    if (lane == 63) wave_tot[w] = v;
    __syncthreads();
    total = make_uint2(0u, 0u);
#pragma unroll
    for (int x = 0; x < kPairThreads / 64; ++x) {
        const uint2 y = wave_tot[x];
        if (x < w) {
            v.x += y.x;
            v.y += y.y;
        }
        total.x += y.x;
        total.y += y.y;
    }
    __syncthreads();
    return v;
}

// pair_z: null where a pair with a count has a depth (the projection's); given records may hold a NaN whose
// bits are kNoDepth, and such a pair is listed nowhere, as in the depth sort.
__device__ __forceinline__ void load_counts(const uint32_t* pair_count, const uint32_t* pair_z, long long n,
                                            long long i0, uint32_t (&c)[kPairItems]) {
    if (i0 + kPairItems <= n) {  // i0 is a multiple of 8: 16-byte aligned
        const uint4 p = reinterpret_cast<const uint4*>(pair_count + i0)[0];
        const uint4 q = reinterpret_cast<const uint4*>(pair_count + i0)[1];
        c[0] = p.x; c[1] = p.y; c[2] = p.z; c[3] = p.w;
        c[4] = q.x; c[5] = q.y; c[6] = q.z; c[7] = q.w;
    } else {
#pragma unroll
        for (int k = 0; k < kPairItems; ++k) c[k] = i0 + k < n ? pair_count[i0 + k] : 0u;
    }
    if (pair_z) {
#pragma unroll
        for (int k = 0; k < kPairItems; ++k)
            if (i0 + k < n && pair_z[i0 + k] == kNoDepth) c[k] = 0u;
    }
}

// Also clears the tile counts and the number of segments, with workgroups of its own where the tiles outnumber the
// pairs (1000 pairs, 32,400 tiles: all binning 119 -> 67 us).
__global__ __launch_bounds__(kPairThreads) void pair_reduce_kernel(const uint32_t* pair_count, const uint32_t* pair_z,
                                                                   long long n, uint2* sums, uint32_t* tile_count,
                                                                   long long n_counts, uint2* segs) {
    __shared__ uint2 wave_tot[kPairThreads / 64];
    const long long g = (long long)blockIdx.x * kPairThreads + threadIdx.x;
    if (g == 0) segs[0] = make_uint2(0u, 0u);
    for (long long e = g; e < n_counts; e += (long long)gridDim.x * kPairThreads) tile_count[e] = 0u;
    uint32_t c[kPairItems];
    load_counts(pair_count, pair_z, n, g * kPairItems, c);
    uint2 v = make_uint2(0u, 0u), total;
#pragma unroll
    for (int k = 0; k < kPairItems; ++k) {
        v.x += c[k];
        v.y += c[k] ? 1u : 0u;
    }
    block_inclusive2(v, wave_tot, total);
    if (threadIdx.x == 0 && (long long)blockIdx.x * kPairBlock < n) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kPairThreads) void pair_apply_kernel(const uint32_t* pair_count, const uint32_t* pair_z,
                                                                  long long n, const uint2* sums, long long capacity,
                                                                  uint32_t* which, uint32_t* out,
                                                                  uint32_t* block_first, uint32_t* counters) {
    __shared__ uint2 wave_tot[kPairThreads / 64];
    uint2 pre = make_uint2(0u, 0u), before, total;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += kPairThreads) {
        pre.x += sums[b].x;
        pre.y += sums[b].y;
    }
    block_inclusive2(pre, wave_tot, before);
    const long long i0 = ((long long)blockIdx.x * kPairThreads + threadIdx.x) * kPairItems;
    uint32_t c[kPairItems];
    load_counts(pair_count, pair_z, n, i0, c);
    uint2 v = make_uint2(0u, 0u);
#pragma unroll
    for (int k = 0; k < kPairItems; ++k) {
        v.x += c[k];
        v.y += c[k] ? 1u : 0u;
    }
    const uint2 incl = block_inclusive2(v, wave_tot, total);
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        const uint32_t K = before.x + total.x;
        const bool over = (long long)K > capacity;
        counters[CNT_K] = K;
        counters[CNT_V] = before.y + total.y;
        counters[CNT_OVERFLOW] = over ? 1u : 0u;
        counters[CNT_KEFF] = over ? (uint32_t)capacity : K;
    }
    uint32_t run = before.x + incl.x - v.x, j = before.y + incl.y - v.y;
#pragma unroll
    for (int k = 0; k < kPairItems; ++k) {
        if (!c[k]) continue;
        which[j] = (uint32_t)(i0 + k);
        out[j] = run;
        const long long e = (long long)run + c[k];
        for (long long m = ((long long)run + kEmitSlots - 1) / kEmitSlots * kEmitSlots; m < e && m < capacity;
             m += kEmitSlots)
            block_first[m / kEmitSlots] = j;
        run += c[k];
        ++j;
    }
}

constexpr uint32_t kTileSortMost = 2048;  // entries that a workgroup sorts in LDS: 16 KB
constexpr uint32_t kTileSortMerge = kTileSortMost / 2;  // the same by merges, which alternate between two buffers

// A longer list is sorted in segments; one of more than kRunsFrom first in runs of kTileSortMerge.  Entries of a
// segment on average: few enough that hardly one is over kTileSortMost, as an uneven sample makes them, since a
// second reading of the list by one segment is waited for (lists of 300k, read: 232 us by 512, 424 by 1024).
constexpr uint32_t kRunsFrom = 5u << 16;
constexpr uint32_t kSegRead = 512, kSegSearch = 1024;
__device__ __forceinline__ uint32_t tile_segments(uint32_t n) {
    const uint32_t per = n > kRunsFrom ? kSegSearch : kSegRead;
    return (n + per - 1) / per;
}
// Segments that a launch can have: the lists' entries are at most `capacity`, and each list has one more at most.
static long long tile_sort_segments(long long capacity) { return capacity / kSegRead + capacity / kTileSortMost; }
static_assert(kSegSearch == kTileSortMerge, "a run for each segment");

// The tile counts to the tiles' ranges, the first place of each (tile, count) and the list total
// (workgroups 8 and up, 1024 tiles each, adding up the tiles before their own), the segments of the long lists
// (segs, whose count was cleared before), and the raster work order
// (workgroups 0..7, from the counts alone, so that nobody waits).
__global__ __launch_bounds__(kWorkThreads) void tile_scan_kernel(const uint32_t* tile_count, uint32_t* tile_base,
                                                                 uint32_t* ranges, int n_tiles, int n_slots,
                                                                 uint32_t* work, uint2* segs, uint32_t* counters) {
    auto length = [&](int tile) {
        uint32_t n = 0;
#pragma unroll
        for (int x = 0; x < kTileCounts; ++x) n += tile_count[(size_t)x * n_tiles + tile];
        return n;
    };
    if (blockIdx.x < 8) {
        work_list_of((int)blockIdx.x, n_tiles, n_slots, work, length);
        return;
    }
    __shared__ uint32_t wave_tot[2][kWorkThreads / 64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int first = ((int)blockIdx.x - 8) * kWorkThreads, tile = first + t;
    uint32_t before = 0;
    for (int i = t; i < first; i += kWorkThreads) before += length(i);
    uint32_t c[kTileCounts], sum = 0;
#pragma unroll
    for (int x = 0; x < kTileCounts; ++x) {
        c[x] = tile < n_tiles ? tile_count[(size_t)x * n_tiles + tile] : 0u;
        sum += c[x];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)incl, o, 64);
        if (lane >= o) incl += y;
        before += (uint32_t)__shfl_xor((int)before, o, 64);
    }
    if (lane == 63) {
        wave_tot[0][w] = incl;
        wave_tot[1][w] = before;
    }
    __syncthreads();
    uint32_t run = incl - sum, total = 0;
#pragma unroll
    for (int x = 0; x < kWorkThreads / 64; ++x) {
        run += (x < w ? wave_tot[0][x] : 0u) + wave_tot[1][x];
        total += wave_tot[0][x] + wave_tot[1][x];
    }
    if (blockIdx.x == gridDim.x - 1 && t == 0) counters[CNT_LIVE] = total;
    for (unsigned long long left = __builtin_amdgcn_ballot_w64(sum > kTileSortMost); left; left &= left - 1) {
        const int lead = __builtin_ctzll(left);  // the wave writes a long list's segments
        const uint32_t m = tile_segments((uint32_t)__builtin_amdgcn_readlane((int)sum, lead));
        uint32_t at = 0;
        if (lane == lead) at = 1 + atomicAdd(&segs[0].x, m);
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, lead);
        for (uint32_t j = lane; j < m; j += 64) segs[at + j] = make_uint2((uint32_t)(tile - lane + lead), j);
    }
    if (tile >= n_tiles) return;
    reinterpret_cast<uint2*>(ranges)[tile] = sum ? make_uint2(run, run + sum) : make_uint2(0u, 0u);
#pragma unroll
    for (int x = 0; x < kTileCounts; ++x) {
        tile_base[(size_t)x * n_tiles + tile] = run;
        run += c[x];
    }
}

// Each intersection's pair id to its place in its tile.
constexpr int kPlaceItems = kEmitSlots / 256;
__global__ __launch_bounds__(256) void place_kernel(const uint32_t* tile_keys, const uint32_t* tile_vals,
                                                    const uint32_t* tile_rank, const uint32_t* tile_base,
                                                    const uint32_t* counters, long long capacity, uint32_t n_tiles,
                                                    uint32_t* out) {
    long long n = counters[CNT_KEFF];
    if (n > capacity) n = capacity;
    const long long k0 = (long long)blockIdx.x * kEmitSlots + threadIdx.x;  // the slots of one emission workgroup
    const uint32_t* base = tile_base + (size_t)(blockIdx.x % kTileCounts) * n_tiles;
    uint32_t t[kPlaceItems], q[kPlaceItems], r[kPlaceItems];
#pragma unroll
    for (int j = 0; j < kPlaceItems; ++j) {
        const long long k = k0 + 256 * j;
        t[j] = k < n ? tile_keys[k] : n_tiles;
        q[j] = k < n ? tile_vals[k] : 0u;
        r[j] = k < n ? tile_rank[k] : 0u;  // not written where the tile was rejected, and not used
    }
#pragma unroll
    for (int j = 0; j < kPlaceItems; ++j)
        if (t[j] < n_tiles) out[base[t[j]] + r[j]] = q[j];
}

// A tile's list sorted by (depth bits, pair id), a strict order: by one workgroup, or in segments by several.
//
// Up to kTileSortMost entries in LDS: by buckets of the depth bits between the entries' least and greatest,
// then each entry by its rank in its bucket, which holds a few; a chain of some ten dependent LDS accesses, where
// merging takes a hundred for 1000 entries.  Where some bucket holds more than kBucketMost (equal depths, a far
// outlier), kTileSortMerge entries at a time: runs of 64 by each element's rank among its run, then merges in
// which an element's place is its index in its own run plus its rank in the other (a binary search).
// One 960 x 600 view over 300k Gaussians (2280 lists, up to 1286 entries): 30 us by merges alone, 15
// by buckets; three views over 600k 50 and 34.
//
// A longer list is cut into ranges of keys at the quantiles of a sample, which each of the list's workgroups takes
// for itself.  A segment's workgroup picks the entries of its range and counts those before it, which is where
// its own begin, so nobody waits for anybody; a range of more entries than LDS holds is halved and its parts
// done in turn.  Up to kRunsFrom entries the workgroup reads the whole list; of a list beyond, tile_runs_kernel has
// sorted runs, and it searches each of them for the ends of its range.  Reading grows with the square of the list,
// but up to the line it takes about as long as the radix sorts, and a launch without longer lists is not
// delayed by the runs' kernel (4.5 us).  All binning, all Gaussians of a view in one tile, us:
//   Gaussians                     5k   20k   50k  100k  200k  300k  400k  500k     1M
//   one workgroup a list         197   954        6136
//   reading the list              67    73    92   121   171   248   360   670
//   searching runs               106    91    90    98   123   168   184   222    690
//   radix sorts over all         115   120   151   215   220   222   228   232    266
constexpr int kTileSortThreads = 256;
constexpr int kTileSortItems = kTileSortMost / kTileSortThreads;
constexpr int kBuckets = 1024, kBucketMost = 48;
constexpr int kMergeItems = 4;  // searches a thread runs side by side
// The thread's number, opaque to the optimiser: what follows from it is formed where it is used, instead of
// being kept in registers around the loops of tile_sort_kernel.
__device__ __forceinline__ int thread_number() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// A value that all lanes hold, in scalar registers.
__device__ __forceinline__ uint32_t uniform32(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ unsigned long long uniform64(unsigned long long v) {
    return ((unsigned long long)uniform32((uint32_t)(v >> 32)) << 32) | uniform32((uint32_t)v);
}

// Orders the wave's own LDS accesses (which complete in order) for the compiler.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One level of merges of runs of R (a power of two) of n elements: element i to place(i's new place).
template <typename Load, typename Place>
__device__ __forceinline__ void merge_level(uint32_t n, uint32_t R, Load load, Place place) {
#pragma unroll 1
    for (uint32_t i0 = thread_number(); i0 < n; i0 += kMergeItems * kTileSortThreads) {
        unsigned long long key[kMergeItems];
        uint32_t lo[kMergeItems], ps[kMergeItems], pl[kMergeItems];  // the other run: start, length
#pragma unroll
        for (int k = 0; k < kMergeItems; ++k) {
            const uint32_t i = i0 + k * kTileSortThreads;
            const bool in = i < n;
            key[k] = in ? load(i) : 0ull;
            ps[k] = (i ^ R) & ~(R - 1);
            pl[k] = in && ps[k] < n ? (n - ps[k] < R ? n - ps[k] : R) : 0u;
            lo[k] = 0;
        }
#pragma unroll 1
        for (uint32_t step = R; step > 0; step >>= 1) {
#pragma unroll
            for (int k = 0; k < kMergeItems; ++k) {
                const uint32_t m = lo[k] + step;
                if (m <= pl[k] && load(ps[k] + m - 1) < key[k]) lo[k] = m;
            }
        }
#pragma unroll
        for (int k = 0; k < kMergeItems; ++k) {
            const uint32_t i = i0 + k * kTileSortThreads;
            if (i < n) place((i & ~(2 * R - 1)) + (i & (R - 1)) + lo[k], key[k]);
        }
    }
}

// Sorts len <= kTileSortMost entries (of the ids id_of(0 .. len), which may lie in a) into a; false, and a as it was,
// if a bucket is too full.
template <typename Id>
__device__ __forceinline__ bool bucket_sort(Id id_of, const uint32_t* pair_z, int len, unsigned long long* a,
                                            uint32_t (&first)[kBuckets + 1], uint32_t (&part)[3][4]) {
    using u64 = unsigned long long;
    const int t = thread_number(), lane = t & 63, w = t >> 6;
    constexpr int BT = kBuckets / kTileSortThreads;
    uint32_t id[kTileSortItems], z[kTileSortItems], lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int k = 0; k < kTileSortItems; ++k) {
        const int i = t + k * kTileSortThreads;
        if (i < len) id[k] = id_of(i);
    }
#pragma unroll
    for (int k = 0; k < kTileSortItems; ++k) {
        const int i = t + k * kTileSortThreads;
        if (i >= len) continue;
        z[k] = pair_z[id[k]];
        lo = min(lo, z[k]);
        hi = max(hi, z[k]);
    }
#pragma unroll
    for (int k = 0; k < BT; ++k) first[BT * t + k] = 0u;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
    }
    if (lane == 0) {
        part[0][w] = lo;
        part[1][w] = hi;
    }
    __syncthreads();
    lo = min(min(part[0][0], part[0][1]), min(part[0][2], part[0][3]));
    hi = max(max(part[1][0], part[1][1]), max(part[1][2], part[1][3]));
    const int bits = hi > lo ? 32 - __builtin_clz(hi - lo) : 0, shift = bits > 10 ? bits - 10 : 0;
    uint32_t at[kTileSortItems];
#pragma unroll
    for (int k = 0; k < kTileSortItems; ++k)
        if (t + k * kTileSortThreads < len) at[k] = atomicAdd(&first[(z[k] - lo) >> shift], 1u);
    __syncthreads();
    // counts to first places; the fullest bucket
    uint32_t c[BT], sum = 0, most = 0;
#pragma unroll
    for (int k = 0; k < BT; ++k) {
        c[k] = first[BT * t + k];
        sum += c[k];
        most = max(most, c[k]);
    }
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)incl, o, 64);
        if (lane >= o) incl += y;
        most = max(most, (uint32_t)__shfl_xor((int)most, o, 64));
    }
    if (lane == 63) {
        part[2][w] = incl;
        part[0][w] = most;
    }
    __syncthreads();
    most = max(max(part[0][0], part[0][1]), max(part[0][2], part[0][3]));
    if (most > (uint32_t)kBucketMost) {  // uniform over the workgroup
        __syncthreads();                 // before `part` is written again
        return false;
    }
    uint32_t run = incl - sum;
#pragma unroll
    for (int x = 0; x < 3; ++x) run += x < w ? part[2][x] : 0u;
#pragma unroll
    for (int k = 0; k < BT; ++k) {
        first[BT * t + k] = run;
        run += c[k];
    }
    if (t == kTileSortThreads - 1) first[kBuckets] = run;
    __syncthreads();
    uint32_t from[kTileSortItems], to[kTileSortItems];
#pragma unroll
    for (int k = 0; k < kTileSortItems; ++k) {
        from[k] = to[k] = 0u;
        if (t + k * kTileSortThreads >= len) continue;
        const uint32_t b = (z[k] - lo) >> shift;
        from[k] = first[b];
        to[k] = first[b + 1];
        a[from[k] + at[k]] = ((u64)z[k] << 32) | id[k];
        at[k] = 0u;
    }
    __syncthreads();
#pragma unroll 1
    for (uint32_t j = 0; j < most; ++j)
#pragma unroll
        for (int k = 0; k < kTileSortItems; ++k)
            if (from[k] + j < to[k]) at[k] += a[from[k] + j] < (((u64)z[k] << 32) | id[k]) ? 1u : 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTileSortItems; ++k)
        if (t + k * kTileSortThreads < len) a[from[k] + at[k]] = ((u64)z[k] << 32) | id[k];
    __syncthreads();
    return true;
}

// Sorts len <= kTileSortMerge entries (of the ids id_of(0 .. len), which may lie in the upper half of buf) into
// one of the halves of buf, and returns where that begins.
template <typename Id>
__device__ __forceinline__ uint32_t merge_sort(Id id_of, const uint32_t* pair_z, uint32_t len,
                                               unsigned long long* buf) {
    using u64 = unsigned long long;
    const int t = thread_number(), lane = t & 63;
    for (uint32_t i = t; i - lane < len; i += kTileSortThreads) {  // wave-uniform
        // the last run's fillers are distinct and above every key, whose id is below 2^31
        const uint32_t q = i < len ? id_of(i) : 0xFFFFFFC0u + (uint32_t)lane;
        const uint32_t z = i < len ? pair_z[q] : 0xFFFFFFFFu;
        const u64 key = ((u64)z << 32) | q;
        // ranks by the depth bits alone, four to an LDS read; lanes of equal depth find another's
        // entry in their place, and then the run is ranked by (depth, id)
        u64* const run = buf + (i - lane);
        uint32_t* const rz = reinterpret_cast<uint32_t*>(run);
        rz[lane] = z;
        wave_sync();
        int rank = 0;
#pragma unroll 4
        for (int j = 0; j < 16; ++j) {
            const uint4 v = reinterpret_cast<const uint4*>(rz)[j];
            rank += (v.x < z ? 1 : 0) + (v.y < z ? 1 : 0) + (v.z < z ? 1 : 0) + (v.w < z ? 1 : 0);
        }
        if (i >= len) rank = lane;
        wave_sync();
        run[rank] = key;
        wave_sync();
        if (__builtin_amdgcn_ballot_w64(run[rank] != key) != 0ull) {
            wave_sync();
            run[lane] = key;
            wave_sync();
            rank = 0;
#pragma unroll 4
            for (int j = 0; j < 64; ++j) rank += run[j] < key ? 1 : 0;
            wave_sync();
            run[rank] = key;
        }
    }
    __syncthreads();
    uint32_t from = 0;
#pragma unroll 1
    for (uint32_t R = 64; R < len; R <<= 1, from ^= kTileSortMerge) {
        const u64* const in = buf + from;
        u64* const out = buf + (from ^ kTileSortMerge);
        merge_level((len + 63) & ~63u, R, [&](uint32_t i) { return in[i]; },
                    [&](uint32_t p, u64 key) { out[p] = key; });
        __syncthreads();
    }
    return from;
}

// Minimum, maximum and sum over the workgroup.
__device__ __forceinline__ void block_range(unsigned long long& least, unsigned long long& most, uint32_t& sum,
                                            unsigned long long (&part)[3][4]) {
    using u64 = unsigned long long;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const u64 x = __shfl_xor(least, o, 64), y = __shfl_xor(most, o, 64);
        least = x < least ? x : least;
        most = y > most ? y : most;
        sum += (uint32_t)__shfl_xor((int)sum, o, 64);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        part[0][w] = least;
        part[1][w] = most;
        part[2][w] = sum;
    }
    __syncthreads();
    sum = 0;
#pragma unroll
    for (int x = 0; x < kTileSortThreads / 64; ++x) {
        least = part[0][x] < least ? part[0][x] : least;
        most = part[1][x] > most ? part[1][x] : most;
        sum += (uint32_t)part[2][x];
    }
}

// The lists of more than kRunsFrom entries in sorted runs of kTileSortMerge, to the same places of `runs`.
__global__ __launch_bounds__(kTileSortThreads) void tile_runs_kernel(const uint32_t* pair_z, const uint32_t* ranges,
                                                                     const uint2* segs, const uint32_t* list,
                                                                     uint32_t* runs) {
    __shared__ __align__(16) unsigned long long buf[kTileSortMost];
    __shared__ uint32_t first[kBuckets + 1], part[3][4];
    for (uint32_t x = blockIdx.x; x < segs[0].x; x += gridDim.x) {
        const uint2 job = segs[1 + x];
        const uint2 se = reinterpret_cast<const uint2*>(ranges)[job.x];
        const uint32_t n = se.y - se.x, at = job.y * kTileSortMerge;  // as many runs as segments
        if (n <= kRunsFrom) continue;
        const uint32_t len = min(n - at, kTileSortMerge);
        const uint32_t* const q = list + se.x + at;
        auto id_of = [&](uint32_t i) { return q[i]; };
        uint32_t from = 0;
        if (!bucket_sort(id_of, pair_z, (int)len, buf, first, part)) from = merge_sort(id_of, pair_z, len, buf);
        for (uint32_t i = threadIdx.x; i < len; i += kTileSortThreads) runs[se.x + at + i] = (uint32_t)buf[from + i];
        __syncthreads();
    }
}

// Workgroups 0 .. n_work - 1: the lists of up to kTileSortMost entries, in the raster work order, the longest
// first; the others, last because most launches have none of them: the segments in segs (their number in
// segs[0].x, then (tile, segment)).  A tile's ids in `list` go to qb in order, the tile's id to tiles; runs: null
// where no list can be longer than kRunsFrom.  The LDS lets seven waves a SIMD run, and the registers have to:
// with 96 all lists of a 300k view took 4 us longer, with a spill the launch itself started 1.5 us later.
// Hence the loops of the segments are not unrolled, and a thread's number is formed anew in each of their parts.
__global__ __launch_bounds__(kTileSortThreads, 7) void tile_sort_kernel(
    const uint32_t* pair_z, const uint32_t* ranges, const uint32_t* work, const uint2* segs, uint32_t n_work,
    const uint32_t* list, const uint32_t* runs, uint32_t* tiles, uint32_t* qb) {
    using u64 = unsigned long long;
    __shared__ __align__(16) u64 buf[kTileSortMost];
    __shared__ uint32_t first[kBuckets + 1], part[3][4];
    const bool segment = blockIdx.x >= n_work;
    uint2 job = make_uint2(0u, 0u);
    if (segment) {
        if (blockIdx.x - n_work >= segs[0].x) return;
        job = segs[1 + blockIdx.x - n_work];
    } else {
        job.x = work[blockIdx.x];
        if (job.x == kNoTile) return;
    }
    const uint32_t tile = job.x;
    const uint2 se = reinterpret_cast<const uint2*>(ranges)[tile];
    const uint32_t n = se.y - se.x, s = se.x;
    if (n == 0u || (!segment && n > kTileSortMost)) return;
    const uint32_t* const q = list + s;
    if (!segment && bucket_sort([&](int i) { return q[i]; }, pair_z, (int)n, buf, first, part)) {
        for (uint32_t i = threadIdx.x; i < n; i += kTileSortThreads) {
            tiles[s + i] = tile;
            qb[s + i] = (uint32_t)buf[i];
        }
        return;
    }
    // A sample of the list gives a segment its keys [lo, end); then the entries from lo up to hi, which is end
    // unless they are too many, are picked and sorted, until they are done up to the end.
    __shared__ u64 range_part[3][4];
    __shared__ uint32_t n_in;
    auto key_of = [&](uint32_t id) { return ((u64)pair_z[id] << 32) | id; };
    uint32_t* const picked = reinterpret_cast<uint32_t*>(buf + kTileSortMerge);  // up to kTileSortMost ids
    u64 lo = 0ull, end = ~0ull, hi = end;
    uint32_t limit = segment ? kTileSortMost : kTileSortMerge;
    bool sampled = !segment;
    for (;;) {
        __syncthreads();
        uint32_t c = limit, below = 0u;
        if (!sampled) {
#pragma unroll 1
            for (uint32_t i = thread_number(); i < c; i += kTileSortThreads)
                picked[i] = q[(uint32_t)((u64)i * n / c)];
            __syncthreads();
        } else {
            const int t = thread_number();
            if (t == 0) n_in = 0u;
            __syncthreads();
            u64 least = ~0ull, most = 0ull;
            if (runs && n > kRunsFrom) {
                // each run's entries of [lo, hi) lie together: two binary searches a run, side by side
                const uint32_t* const r = runs + s;
                const uint32_t n_runs = (n + kTileSortMerge - 1) / kTileSortMerge;
#pragma unroll 1
                for (uint32_t i0 = t; i0 < n_runs; i0 += kMergeItems * kTileSortThreads) {
                    uint32_t from[kMergeItems], first_in[kMergeItems], first_out[kMergeItems], len[kMergeItems];
#pragma unroll
                    for (int k = 0; k < kMergeItems; ++k) {
                        const uint32_t i = i0 + k * kTileSortThreads;
                        from[k] = i * kTileSortMerge;
                        len[k] = i < n_runs ? (n - from[k] < kTileSortMerge ? n - from[k] : kTileSortMerge) : 0u;
                        first_in[k] = first_out[k] = 0u;
                    }
#pragma unroll 1
                    for (uint32_t step = kTileSortMerge; step > 0; step >>= 1) {
#pragma unroll
                        for (int k = 0; k < kMergeItems; ++k) {
                            const uint32_t x = first_in[k] + step, y = first_out[k] + step;
                            if (x <= len[k] && key_of(r[from[k] + x - 1]) < lo) first_in[k] = x;
                            if (y <= len[k] && key_of(r[from[k] + y - 1]) < hi) first_out[k] = y;
                        }
                    }
#pragma unroll
                    for (int k = 0; k < kMergeItems; ++k) {
                        below += first_in[k];
                        if (first_in[k] == first_out[k]) continue;
                        const u64 x = key_of(r[from[k] + first_in[k]]), y = key_of(r[from[k] + first_out[k] - 1]);
                        least = x < least ? x : least;
                        most = y > most ? y : most;
                        const uint32_t k_in = first_out[k] - first_in[k], p = atomicAdd(&n_in, k_in);
#pragma unroll 1
                        for (uint32_t e = 0; e < k_in && p + e < limit; ++e)
                            picked[p + e] = r[from[k] + first_in[k] + e];
                    }
                }
            } else {
                // most entries are told by their depth bits alone; the next ids are asked for behind the depths
                const uint32_t z_lo = (uint32_t)(lo >> 32), z_hi = (uint32_t)((hi - 1) >> 32);
                constexpr int U = 8;
                uint32_t id[U];
                auto load = [&](uint32_t i0) {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const uint32_t i = i0 + u * kTileSortThreads;
                        id[u] = i < n ? q[i] : 0xFFFFFFFFu;
                    }
                };
                load(t);
#pragma unroll 1
                for (uint32_t i0 = t; i0 - t < n; i0 += U * kTileSortThreads) {
                    uint32_t z[U], now[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        now[u] = id[u];
                        z[u] = pair_z[now[u] == 0xFFFFFFFFu ? 0u : now[u]];
                    }
                    load(i0 + U * kTileSortThreads);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (now[u] == 0xFFFFFFFFu) z[u] = 0xFFFFFFFFu;  // past the list: not below any end
                        below += z[u] < z_lo ? 1u : 0u;
                        const bool near = z[u] >= z_lo && z[u] <= z_hi;
                        if (__builtin_amdgcn_ballot_w64(near) == 0ull) continue;
                        const u64 key = ((u64)z[u] << 32) | now[u];
                        if (near && key < lo) ++below;
                        if (near && key >= lo && key < hi) {
                            least = key < least ? key : least;
                            most = key > most ? key : most;
                            const uint32_t p = atomicAdd(&n_in, 1u);
                            if (p < limit) picked[p] = now[u];
                        }
                    }
                }
            }
            block_range(least, most, below, range_part);
            least = uniform64(least);
            most = uniform64(most);
            below = uniform32(below);
            c = uniform32(n_in);
            if (c > limit) {
                if (least == most) return;  // a tile lists a pair once, so keys are distinct: buffers in use twice
                hi = least + (most - least) / 2 + 1;
                continue;
            }
        }
        auto id_of = [&](uint32_t i) { return picked[i]; };
        uint32_t from = 0;
        if (limit == kTileSortMost) {
            if (!bucket_sort(id_of, pair_z, (int)c, buf, first, part)) {
                limit = kTileSortMerge;
                continue;
            }
        } else {
            from = merge_sort(id_of, pair_z, c, buf);
        }
        if (!sampled) {
            const uint32_t m = tile_segments(n);
            if (job.y > 0) lo = uniform64(buf[from + job.y * c / m]);
            if (job.y + 1 < m) end = uniform64(buf[from + (job.y + 1) * c / m]);
            hi = end;
            sampled = true;
            continue;
        }
#pragma unroll 1
        for (uint32_t i = thread_number(); i < c; i += kTileSortThreads) {
            tiles[s + below + i] = tile;
            qb[s + below + i] = (uint32_t)buf[from + i];
        }
        if (hi == end) return;
        lo = hi;
        hi = end;
    }
}

// Stage entry from externally supplied records: counts and depth bits per pair.
__global__ void count_from_records_kernel(ViewTable vt, const float* records, const uint8_t* valid,
                                          long long n_pairs, uint32_t* pair_count, uint32_t* pair_z) {
    long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n_pairs) return;
    uint32_t cnt = 0;
    if (valid[q]) {
        const int b = view_of_pair(vt, q);
        const float4* rec = reinterpret_cast<const float4*>(records + q * kRecFloats);
        const float4 r0 = rec[0], r1 = rec[1], r2 = rec[2];
        int tx0, ty0, tx1, ty1;
        if (tile_rect(r0.x, r0.y, r1.w, r2.x, vt.width[b], vt.height[b], vt.tile, tx0, ty0, tx1, ty1))
            cnt = (uint32_t)((tx1 - tx0 + 1) * (ty1 - ty0 + 1));
    }
    pair_count[q] = cnt;
    pair_z[q] = cnt ? __float_as_uint(reinterpret_cast<const float4*>(records + q * kRecFloats)[1].z) : kNoDepth;
}

void launch_count_from_records(const ViewTable& vt, const float* records, const uint8_t* valid,
                               long long n_pairs, uint32_t* pair_count, uint32_t* pair_z,
                               hipStream_t s) {
    if (n_pairs <= 0) return;
    hipLaunchKernelGGL(count_from_records_kernel, dim3((unsigned)((n_pairs + 255) / 256)), dim3(256),
                       0, s, vt, records, valid, n_pairs, pair_count, pair_z);
}

// Which way a launch takes: the lists sorted tile by tile, or two radix sorts over all.  Tile by tile
// is six or seven launches (about 4.5 us each however little they do) against 23, but its atomics, scattered
// places and sorts cost more per intersection.  Binning of one 300k-Gaussian view (0.5M
// intersections) 190 us by radix sorts, 51 tile by tile; three views over 600k (2.4M) 208 and 158; four
// over 1M (7.5M) 304 and 361.  Long lists cost it the most (see the table at bucket_sort): lists are at most 4096
// entries long because no view has more Gaussians, or the capacity leaves 512 a tile on average, which bounds
// no single list, and no view has more than 2^20 Gaussians.  If those all lie in one tile it is as fast as the
// radix sorts up to 500k, at 1M 690 us and 266.  Its scans, of 2048 pairs or 1024 tiles a workgroup, each of
// which adds up the sums of those before it, grow with the square of their number: per tile and by radix sorts,
// 30k Gaussians in 32,400 tiles 109 and 124 us, 65,536 tiles 151 and 143, 129,600 tiles 233 and 161 (200k: 138 and
// 222, 213 and 240, 369 and 251); 4.2M pairs of which 400k are visible 234 and 252, 8.4M 395 and 371, 34M
// 1514 and 1099.
constexpr long long kTileSortCapacity = 1ll << 22, kTileSortShort = 4096, kTileSortMean = 512;
constexpr long long kTileSortLongest = 1ll << 20, kTileSortTiles = 1ll << 16, kTileSortPairs = 1ll << 23;
// No list is longer than its view's Gaussian range, or than the capacity.
static long long longest_list(const ViewTable& vt, long long capacity) {
    long long n = 0;
    for (int b = 0; b < vt.n_views; ++b) n = max(n, (long long)vt.g_end[b] - vt.g_begin[b]);
    return min(n, capacity);
}

static bool per_tile_sort(const ViewTable& vt, long long n_pairs, long long capacity) {
    const long long n_tiles = vt.tile_base[vt.n_views];
    if (n_pairs <= 0 || n_pairs > kTileSortPairs || n_tiles <= 0 || n_tiles > kTileSortTiles) return false;
    if (capacity <= 0 || capacity > kTileSortCapacity) return false;
    const long long longest = longest_list(vt, capacity);
    return longest <= kTileSortShort || (longest <= kTileSortLongest && capacity <= kTileSortMean * n_tiles);
}

// Two sets of counts, then the segments.  Reserved for every launch, whichever way it takes: the workspace of a
// larger capacity, view or map has room for a smaller one.
size_t tile_sort_bytes(long long n_tiles, long long capacity) {
    const size_t tiles = (size_t)min(n_tiles, kTileSortTiles), cap = (size_t)min(capacity, kTileSortCapacity);
    return 2 * kTileCounts * tiles * sizeof(uint32_t) + (1 + (size_t)tile_sort_segments(cap)) * sizeof(uint2);
}

static int launch_binning_per_tile(BinArgs& a, hipStream_t s) {
    const int n_tiles = a.vt.tile_base[a.vt.n_views];
    const unsigned pgrid = (unsigned)((a.n_pairs + kPairBlock - 1) / kPairBlock);
    uint2* sums = reinterpret_cast<uint2*>(a.depth_keys[0]);
    const uint32_t* const z = a.given_depths ? a.pair_z : nullptr;
    uint32_t* const count = a.tile_count;
    uint32_t* const base = a.tile_count + (size_t)kTileCounts * n_tiles;
    uint2* const segs = reinterpret_cast<uint2*>(base + (size_t)kTileCounts * n_tiles);
    const long long n_counts = (long long)kTileCounts * n_tiles;
    const unsigned clear_grid = (unsigned)((n_counts + 16 * kPairThreads - 1) / (16 * kPairThreads));
    hipLaunchKernelGGL(pair_reduce_kernel, dim3(max(pgrid, clear_grid)), dim3(kPairThreads), 0, s, a.pair_count, z,
                       a.n_pairs, sums, count, n_counts, segs);
    hipLaunchKernelGGL(pair_apply_kernel, dim3(pgrid), dim3(kPairThreads), 0, s, a.pair_count, z, a.n_pairs, sums,
                       a.capacity, a.depth_vals[0], a.emit_off, a.block_first, a.counters);
    const unsigned egrid = (unsigned)((a.capacity + kEmitSlots - 1) / kEmitSlots);
    uint32_t* const tk = a.tile_keys[0];
    uint32_t* const tr = a.tile_keys[1];
    uint32_t* const tv = a.final_vals;
    uint32_t* const list = a.final_vals == a.tile_vals[0] ? a.tile_vals[1] : a.tile_vals[0];
    hipLaunchKernelGGL(emit_kernel<true>, dim3(egrid), dim3(kEmitThreads), 0, s, a.vt, a.records, a.depth_vals[0],
                       a.emit_off, a.block_first, a.counters, a.capacity, tk, tv, tr, count, a.ranges);
    const unsigned tgrid = 8 + (unsigned)((n_tiles + kWorkThreads - 1) / kWorkThreads);
    hipLaunchKernelGGL(tile_scan_kernel, dim3(tgrid), dim3(kWorkThreads), 0, s, count, base, a.ranges, n_tiles,
                       raster_blocks(a.vt), a.work, segs, a.counters);
    hipLaunchKernelGGL(place_kernel, dim3(egrid), dim3(256), 0, s, tk, tv, tr, base, a.counters, a.capacity,
                       (uint32_t)n_tiles, list);
    const uint32_t seg_grid = (uint32_t)tile_sort_segments(a.capacity);
    uint32_t* const runs = longest_list(a.vt, a.capacity) > kRunsFrom ? tr : nullptr;
    if (runs)
        hipLaunchKernelGGL(tile_runs_kernel, dim3(min(seg_grid, 1024u)), dim3(kTileSortThreads), 0, s, a.pair_z,
                           a.ranges, segs, list, runs);
    const uint32_t n_work = (uint32_t)raster_blocks(a.vt);
    hipLaunchKernelGGL(tile_sort_kernel, dim3(n_work + seg_grid), dim3(kTileSortThreads), 0, s, a.pair_z, a.ranges,
                       a.work, segs, n_work, list, runs, tk, tv);
    return (int)hipGetLastError();
}

int launch_binning(BinArgs& a, hipStream_t s) {
    if (per_tile_sort(a.vt, a.n_pairs, a.capacity)) return launch_binning_per_tile(a, s);
    const long long Q = a.n_pairs;
    // 1-2. stable depth sort of the visible pairs: the first pass reads every pair's depth
    //    key (pair_z; kNoDepth for a pair no view keeps) with the pair id as value, drops the
    //    invisible ones and counts the visible ones into CNT_V; its last pass also lays out
    //    the pairs' tile counts in depth order, in emit_off
    int r = launch_radix_sort(a.depth_keys, a.depth_vals, Q, nullptr, 32, a.depth_grid, a.sort_tmp, s,
                              a.pair_count, a.emit_off, a.counters + CNT_V, kNoDepth, a.pair_z);
    const uint32_t* dvals = a.depth_vals[r];
    // 3. intersection offsets in depth order (in place), total K, overflow flag, first pair
    //    of each emission workgroup
    launch_emit_scan(a.emit_off, nullptr, a.emit_off, Q, a.counters + CNT_V, a.counters, a.capacity,
                     a.block_first, a.scan_tmp, s);
    // 4. emit (tile id, pair id) in depth order into the buffer from which an even/odd
    //    number of tile-sort passes ends in final_vals
    const int tp = sort_passes(a.tile_bits);
    const int first = (a.final_vals == a.tile_vals[0]) ? (tp % 2) : 1 - (tp % 2);
    const unsigned egrid = (unsigned)((a.capacity + kEmitSlots - 1) / kEmitSlots > 0
                                          ? (a.capacity + kEmitSlots - 1) / kEmitSlots
                                          : 1);
    hipLaunchKernelGGL(emit_kernel<false>, dim3(egrid), dim3(kEmitThreads), 0, s, a.vt, a.records, dvals, a.emit_off,
                       a.block_first, a.counters, a.capacity, a.tile_keys[first], a.tile_vals[first], nullptr,
                       nullptr, a.ranges);
    // 5. stable sort by tile id
    uint32_t* tk[2] = {a.tile_keys[first], a.tile_keys[1 - first]};
    uint32_t* tv[2] = {a.tile_vals[first], a.tile_vals[1 - first]};
    //    (its first pass drops the intersections the ellipse test rejected, key n_tiles)
    const long long n_tiles_all = a.vt.tile_base[a.vt.n_views];
    int rt = launch_radix_sort(tk, tv, a.capacity, a.counters + CNT_KEFF, a.tile_bits, a.tile_grid, a.sort_tmp,
                               s, nullptr, nullptr, a.counters + CNT_LIVE, (uint32_t)n_tiles_all);
    // 6. per-tile ranges
    const long long n_tiles = a.vt.tile_base[a.vt.n_views];
    const unsigned rgrid = (unsigned)((a.capacity + 256 * kRangeItems - 1) / (256 * kRangeItems) > 0
                                          ? (a.capacity + 256 * kRangeItems - 1) / (256 * kRangeItems)
                                          : 1);
    hipLaunchKernelGGL(ranges_kernel, dim3(rgrid), dim3(256), 0, s, tk[rt], a.counters, a.capacity,
                       (uint32_t)n_tiles, a.ranges);
    // 7. raster work order
    if (n_tiles > 0)
        hipLaunchKernelGGL(work_list_kernel, dim3(8), dim3(kWorkThreads), 0, s, a.ranges, (int)n_tiles,
                           raster_blocks(a.vt), a.work);
    (void)tv;
    return (int)hipGetLastError();
}

}  // namespace ags
