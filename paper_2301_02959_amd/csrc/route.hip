// fs_route_bucketize: jagged ids -> (tier, owner) -> stable bucketize by owner.
//
// A stable counting sort of the n lookups by destination bucket, in three steps
// that touch each lookup twice:
//   route_remap     one tile of 2048 lookups (small batches: 512 or 1024) per block: table of each lookup, global
//                   row g, placement entry, destination; per-tile bucket
//                   histogram (the own bucket and one other by ballots, the rest by LDS adds) plus the tile's three tier
//                   counts; dest (u16) and g (u32) go to the workspace; each block also
//                   validates its share of the offsets
//   route_scan      one block per bucket (and per tier): exclusive scan of its per-tile
//                   counts over the tiles, and its total (skipped when the counts are few
//                   enough for every scatter block to sum them itself)
//   route_scatter   same tiles: each wave ranks its consecutive lookups by
//                   ballot matching against a wave-private running histogram in
//                   LDS, adds the tile's and the bucket's base, writes
//                   out_rows / out_pos
//                   (its first block also writes bucket_offsets and tier_counts)
//   route_prepare / route_finalize   only for an empty batch: the offsets check and the
//                   zero outputs
// No spin-waits anywhere: the only cross-block communication is between launches.
#include <atomic>

#include "fs_common.h"

namespace fs {

constexpr int kRouteItems = 8;                        // lookups per thread
constexpr int kRouteStripe = 32;                      // tiles per XCD stripe in the scatter
// Up to this many tile counts (tiles x (buckets + 3)) every scatter block sums them itself, the threads of a block
// sharing a bucket's tiles, and route_scan is not launched: 8192 lookups over 8 buckets take 5.5 us of GPU time
// after the remap instead of 9, 80 k over 64 (2747 counts) 6 instead of 8, and the host saves a launch (2.3 us).
// At 6499 counts the two are even on the GPU, at 14 k the sums are 12 us slower.
constexpr int64_t kRouteSumMax = 6144;
// Small batches take tiles of 512 and 1024 lookups instead of 2048, whose counts every scatter block sums too: a block's
// time is its chain of rounds, its share of random placement reads and the memory's latency.  Both kernels, 2048 / 1024 / 512
// lookups to a tile, us: 8192 lookups over 8 buckets 11.9 / 10.0 / 9.9, 50 k over 64 13.1 / 10.1 / 9.4, 83 k (10.9 k counts of
// 512) 13.2 / 10.8 / 10.2, 130 k (17 k) 13.1 / 10.8 / 11.1, 260 k over 8 (5.6 k) 13.7 / 10.7 / 10.4, 520 k (11.2 k) 15.6 / 13.1 /
// 14.2; 260 k over 64 (17 k counts of 1024) 16.9 / 12.7, over 128 (33 k) 17.2 / 15.2, 520 k over 64 (34 k) 18.1 / 18.2.  Around the
// first line (11 k counts of 512), 1024 / 512, in a graph: 24 buckets 12 k 11.0 / 11.7, 13 k 11.1 / 12.0; 64 buckets 12 k
// 10.5 / 9.9, 13 k 10.3 / 10.4, 17 k 10.7 / 10.8; 128 buckets 12 k 10.5 / 9.6, 15 k 10.5 / 10.1, 19 k 11.0 / 10.9.  Up to 128
// buckets: there the threads that share a bucket bring its counts in one round.
constexpr int64_t kRouteSmallCounts[2] = {11000, 33500};         // of tiles of 512 and 1024 lookups
constexpr int64_t kRouteSmallTiles = 512;
constexpr int kRouteSmallBuckets = 128;
// Beyond one tile for every CU the remap counts the first foreign bucket by ballots too (LEAD).  16 M lookups, every row
// on one other GPU: 76 us with a full match of the buckets, 83 with plain adds, 73 so; rows dealt over 8 buckets 82, 73.5,
// 73.5.  2.4 M: plain 20.7 and 16.4, so 16.9 and 16.8.  Up to one tile the waves' own chains are the time, and the ballots
// cost 0.4 us of 8.6 where the adds that meet cost 0.2.
constexpr int64_t kRouteLeadTiles = 256;
// From this many bits of the bucket number (more than 2048 buckets) a scatter thread owns up to 16 buckets, and has the
// loads of all of them in flight: 20 M lookups over 4096 buckets 523 us bucket by bucket, 412 so, 72 M over 16 tables 1457,
// 1379.  With fewer the blocks then come to their stores at other times and write 3 % more: 72 M over 2048 buckets 923,
// 953, over 128 359, 380.
constexpr int kRouteBasesBits = 12;

__global__ __launch_bounds__(kBlock) void route_prepare_kernel(
    const int64_t* __restrict__ offsets, int64_t S, int64_t n, int32_t* status)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = false;
    for (int64_t s = tid; s < S; s += stride) bad |= offsets[s] > offsets[s + 1];
    if (tid == 0) bad |= offsets[0] != 0 || offsets[S] != n;
    if (ballot(bad) != 0 && lane_id() == 0) report(status, FS_DEV_BAD_OFFSETS);
}

// A tile's tables and their rows, staged in LDS when there are at most this many of them.
constexpr int kRouteTileTables = 64;

// What the remap and the scatter are given, as one argument: the runtime spends 0.5 us more on a launch of 16.
struct RouteArgs {
    const int64_t* ids;
    const int64_t* offsets;
    const int64_t* row_base;
    const uint32_t* placement;
    int64_t B, n, tiles;
    uint16_t* dest;                  // [n] a lookup's bucket,
    uint32_t* g;                     // its row,
    int32_t* slot;                   // and its replica slot (or null), from one to the other
    uint32_t* tile_hist;             // buckets, then the three tiers: [tiles][U + 3] if by_tile, else [U + 3][tiles]
    const uint32_t* totals;
    int64_t* out_rows;
    int32_t* out_pos;
    int32_t* out_slots;
    int64_t* bucket_offsets;
    int64_t* tier_counts;
    int32_t* status;
    int T, U, W, self, by_tile;
};

template <bool LEAD, int ITEMS>
__global__ __launch_bounds__(kBlock) void route_remap_kernel(const RouteArgs a)
{
    const int64_t* const ids = a.ids;
    const int64_t* const offsets = a.offsets;
    const int64_t* const row_base = a.row_base;
    const uint32_t* const placement = a.placement;
    const int64_t B = a.B, n = a.n, tiles = a.tiles;
    const int T = a.T, U = a.U, W = a.W, self = a.self;
    uint16_t* const dest_out = a.dest;
    uint32_t* const g_out = a.g;
    int32_t* const slot_out = a.slot;
    constexpr int kTile = kBlock * ITEMS;
    extern __shared__ uint32_t lds_hist[];            // [U]
    __shared__ int tile_tables[2];
    __shared__ int64_t table_end[kRouteTileTables];   // tables t_lo .. t_hi of the tile: first lookup after table t,
    __shared__ int64_t table_first[kRouteTileTables]; // its first row,
    __shared__ int64_t table_rows[kRouteTileTables];  // and how many it has
    __shared__ unsigned int wave_counts[kWavesPerBlock][3];   // tiers 1 and 2, lookups of the own bucket
    const int64_t tile = blockIdx.x;
    const int64_t base = tile * kTile;
    const int w = wave_id();

    // Every load that waits for nothing goes out first: the ids, this block's share of the offsets (checked at
    // the very end), the table bounds: of all tables if they fit, so that no load waits for the search of the tile's.
    int64_t id[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = base + (int64_t)it * kBlock + threadIdx.x;
        id[it] = load_stream(ids + (i < n ? i : n - 1));             // past the end: the last id again, unused
    }
    const int64_t S = (int64_t)T * B;                                // S segments over `tiles` blocks
    const int64_t per = (S + tiles - 1) / tiles;
    const int64_t s_lo = (int64_t)blockIdx.x * per;
    const int64_t s_hi = s_lo + per < S ? s_lo + per : S;
    const bool has_segment = s_lo + threadIdx.x < s_hi;
    int64_t seg0 = 0, seg1 = 0;
    if (has_segment) { seg0 = offsets[s_lo + threadIdx.x]; seg1 = offsets[s_lo + threadIdx.x + 1]; }
    const int64_t last = (base + kTile < n ? base + kTile : n) - 1;
    const int64_t R_all = row_base[T];                // rows of all tables; g must stay below it (and below 2^32 - 1)
    const bool all_staged = T <= kRouteTileTables;    // uniform
    int t_lo, t_hi;
    int staged_from;                                  // the table that table_end[0] is of
    bool staged = true;                               // block-uniform
    if (all_staged) {
        // every wave finds the tile's first and last table itself: a lane for each
        const int k = lane_id() < T ? lane_id() : T - 1;
        const int64_t starts = offsets[(int64_t)k * B];
        t_lo = __popcll(ballot(lane_id() > 0 && lane_id() < T && starts <= base));
        t_hi = __popcll(ballot(lane_id() > 0 && lane_id() < T && starts <= last));
        staged_from = 0;
        if (w == 0 && lane_id() < T) {
            const int64_t first = row_base[k];
            table_end[k] = offsets[(int64_t)(k + 1) * B];
            table_first[k] = first;
            table_rows[k] = row_base[k + 1] - first;
        }
        for (int b = threadIdx.x; b < U; b += kBlock) lds_hist[b] = 0;
        __syncthreads();
    } else {
        for (int b = threadIdx.x; b < U; b += kBlock) lds_hist[b] = 0;
        if (w < 2) {                                                 // two waves find the tile's first and last table
            const int t = wave_table_of(offsets, T, B, w == 0 ? base : last);
            if (lane_id() == 0) tile_tables[w] = t;
        }
        __syncthreads();
        t_lo = tile_tables[0];
        t_hi = tile_tables[1];
        staged_from = t_lo;
        staged = t_hi - t_lo < kRouteTileTables;
        if (staged) {
            const int k = threadIdx.x;
            if (k <= t_hi - t_lo) {
                table_end[k] = offsets[(int64_t)(t_lo + k + 1) * B];
                table_first[k] = row_base[t_lo + k];
                table_rows[k] = row_base[t_lo + k + 1] - row_base[t_lo + k];
            }
            __syncthreads();
        }
    }
    t_lo = __builtin_amdgcn_readfirstlane(t_lo);
    t_hi = __builtin_amdgcn_readfirstlane(t_hi);
    const int group_base = (self / W) * W;
    const bool rows_ok = R_all >= 1 && R_all < 4294967295LL;
    int32_t faults = rows_ok ? 0 : FS_DEV_BAD_ID;

    const int64_t first_lo = staged ? table_first[t_lo - staged_from] : row_base[t_lo];
    const int64_t rows_lo = staged ? table_rows[t_lo - staged_from] : row_base[t_lo + 1] - first_lo;
    int64_t g[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = base + (int64_t)it * kBlock + threadIdx.x;
        int64_t first = first_lo, rows_t = rows_lo;
        if (t_lo != t_hi) {                                          // block-uniform
            if (staged) {
                int k = t_lo - staged_from;
                while (k < t_hi - staged_from && table_end[k] <= i) ++k;
                first = table_first[k];
                rows_t = table_rows[k];
            } else {
                int t = t_lo;
                while (t < t_hi && offsets[(int64_t)(t + 1) * B] <= i) ++t;
                first = row_base[t];
                rows_t = row_base[t + 1] - first;
            }
        }
        int64_t x = id[it];
        const bool valid = i < n;
        if (x < 0 || x >= rows_t) { if (valid) faults |= FS_DEV_BAD_ID; x = 0; }
        int64_t row = first + x;
        if ((uint64_t)row >= (uint64_t)R_all) { if (valid) faults |= FS_DEV_BAD_ID; row = 0; }   // row_base not ascending
        g[it] = row;
    }
    uint32_t e[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) e[it] = rows_ok ? placement[g[it]] : 0u;
    // Counts of the wave: the tiers and the own bucket with one ballot each, and (LEAD) one more for the bucket of the
    // wave's first lookup that goes elsewhere: a bucket that most of the rest go to (few buckets, whole tables or a hot row
    // on one other GPU) is nearly always that one.  What is left are plain LDS adds, of which few meet in one word.
    uint32_t in_tier1 = 0, in_tier2 = 0, own = 0;                    // tier 0: the tile's other lookups
    uint32_t led = 0, in_led = 0;                                    // led: any bucket if the first item has none
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = base + (int64_t)it * kBlock + threadIdx.x;
        const bool valid = i < n;
        const uint32_t tier = e[it] >> FS_TIER_SHIFT;
        const uint32_t owner = e[it] & FS_OWNER_MASK;
        uint32_t dest = (uint32_t)self;                              // tier 0, and every fault
        if (tier == FS_TIER_GROUP) { if (owner < (uint32_t)W) dest = (uint32_t)group_base + owner; else if (valid) faults |= FS_DEV_BAD_PLACEMENT; }
        if (tier == FS_TIER_SHARDED) { if (owner < (uint32_t)U) dest = owner; else if (valid) faults |= FS_DEV_BAD_PLACEMENT; }
        if (tier > FS_TIER_SHARDED && valid) faults |= FS_DEV_BAD_PLACEMENT;
        if (valid) {
            dest_out[i] = (uint16_t)dest;
            g_out[i] = (uint32_t)g[it];
            // a replicated row's entry names no owner: its owner bits carry the row's replica slot, if it has one
            if (slot_out != nullptr)
                slot_out[i] = (tier == FS_TIER_GLOBAL && owner != FS_OWNER_MASK) ? (int32_t)owner : -1;
        }
        const bool foreign = valid && dest != (uint32_t)self;
        if constexpr (LEAD) {
            if (it == 0) led = (uint32_t)__builtin_amdgcn_readlane((int)dest, __builtin_ctzll(ballot(foreign) | (1ull << 63)));
            const bool same = foreign && dest == led;
            in_led += (uint32_t)__popcll(ballot(same));
            if (foreign && !same) atomicAdd(&lds_hist[dest], 1u);
        } else if (foreign) {
            atomicAdd(&lds_hist[dest], 1u);
        }
        in_tier1 += (uint32_t)__popcll(ballot(valid && tier == FS_TIER_GROUP));
        in_tier2 += (uint32_t)__popcll(ballot(valid && tier == FS_TIER_SHARDED));
        own += (uint32_t)__popcll(ballot(valid && dest == (uint32_t)self));
    }
    if (lane_id() == 0) {
        wave_counts[w][0] = in_tier1; wave_counts[w][1] = in_tier2; wave_counts[w][2] = own;
        if (LEAD && in_led != 0) atomicAdd(&lds_hist[led], in_led);
    }
    __syncthreads();
    auto waves_sum = [&](int k) {
        uint32_t v = 0;
        for (int q = 0; q < kWavesPerBlock; ++q) v += wave_counts[q][k];
        return v;
    };
    uint32_t* my_hist = a.by_tile ? a.tile_hist + tile * (U + 3) : a.tile_hist + tile;
    const int64_t step = a.by_tile ? 1 : tiles;
    for (int b = threadIdx.x; b < U; b += kBlock) my_hist[b * step] = b == self ? waves_sum(2) : lds_hist[b];
    // tier counts travel as three more histogram rows (no global atomics: 3 hot addresses
    // shared by every wave of the grid serialise in L2)
    if (threadIdx.x < 3) {
        const uint32_t in_tile = (uint32_t)(n - base < kTile ? n - base : kTile);
        const uint32_t in_tier = threadIdx.x == 0 ? in_tile - waves_sum(0) - waves_sum(1) : waves_sum(threadIdx.x - 1);
        my_hist[(U + threadIdx.x) * step] = in_tier;
    }

    bool bad = has_segment && seg0 > seg1;
    for (int64_t sg = s_lo + threadIdx.x + kBlock; sg < s_hi; sg += kBlock) bad |= offsets[sg] > offsets[sg + 1];
    if (blockIdx.x == 0 && threadIdx.x == 0) bad |= offsets[0] != 0 || offsets[S] != n;
    if (bad) faults |= FS_DEV_BAD_OFFSETS;
    if (ballot(faults != 0) != 0) {
        for (int off = 32; off > 0; off >>= 1) faults |= __shfl_down(faults, off);
        if (lane_id() == 0) report(a.status, faults);
    }
}

// One block per bucket b: tile_hist[b][0..tiles) -> exclusive prefix in place, total[b].
constexpr int kRouteScanBlock = 1024;                 // U + 3 blocks only: as many threads each as a block can have

__global__ __launch_bounds__(kRouteScanBlock) void route_scan_kernel(uint32_t* __restrict__ tile_hist, int64_t tiles,
                                                                     uint32_t* __restrict__ totals)
{
    __shared__ uint32_t wave_sums[16];
    uint32_t* h = tile_hist + (int64_t)blockIdx.x * tiles;
    const int64_t per = (tiles + kRouteScanBlock - 1) / kRouteScanBlock;
    const int64_t lo = (int64_t)threadIdx.x * per < tiles ? (int64_t)threadIdx.x * per : tiles;
    const int64_t hi = lo + per < tiles ? lo + per : tiles;
    uint32_t sum = 0;
    for (int64_t k = lo; k < hi; ++k) sum += h[k];
    uint32_t total;
    uint32_t run = block_exclusive_scan(sum, wave_sums, &total);
    if (threadIdx.x == 0) totals[blockIdx.x] = total;
    for (int64_t k = lo; k < hi; ++k) { const uint32_t v = h[k]; h[k] = run; run += v; }
}

// SUM: the counts are few, route_scan has not run: tile_hist holds plain counts and every block adds up what it needs.
template <int NBITS, bool SUM, int ITEMS>
__global__ __launch_bounds__(kBlock) void route_scatter_kernel(const RouteArgs a)
{
    const int64_t n = a.n, tiles = a.tiles;
    const int U = a.U;
    const uint32_t* const tile_hist = a.tile_hist;                      // scanned, unless SUM
    const uint32_t* const totals = a.totals;
    const int32_t* const slot_in = a.slot;
    int64_t* const bucket_offsets = a.bucket_offsets;
    int64_t* const tier_counts = a.tier_counts;
    extern __shared__ uint32_t lds[];
    uint32_t* bucket_base = lds;                                        // [U] first output index of the tile in bucket b
    uint16_t* wave_hist = reinterpret_cast<uint16_t*>(lds + U);         // [waves][U]
    __shared__ uint32_t wave_sums[16];
    constexpr int kBins = 1 << NBITS;                                   // U <= kBins
    constexpr int kParts = SUM && kBins < kBlock ? kBlock / kBins : 1;
    __shared__ uint32_t part_all[kParts > 1 ? kBlock : 1];
    __shared__ uint32_t part_before[kParts > 1 ? kBlock : 1];
    // tiles in stripes per XCD: consecutive tiles write neighbouring pieces of every bucket's range,
    // which one XCD's L2 merges into whole lines (0.082 -> 0.073 ms on 15.7 M lookups)
    const int64_t tile = SUM ? (int64_t)blockIdx.x : xcd_striped_tile(blockIdx.x, kRouteStripe);
    if (tile >= tiles) return;                                          // block-uniform, before any barrier
    const int64_t base = tile * (kBlock * ITEMS);
    const int w = wave_id();
    const int lane = lane_id();

    uint32_t dest[ITEMS];
    uint32_t rank[ITEMS];
    uint32_t g[ITEMS];
    int32_t slot[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = base + (int64_t)w * (kWave * ITEMS) + it * kWave + lane;
        const bool valid = i < n;
        dest[it] = valid ? a.dest[i] : 0;
        g[it] = valid ? a.g[i] : 0;
        slot[it] = (valid && slot_in != nullptr) ? slot_in[i] : -1;
    }

    // the tile's first index in every bucket: exclusive scan of the bucket totals (every block repeats it: U is
    // small) plus the lookups of the tiles before
    {
        const int stride = U + 3;                                       // SUM: tile_hist is [tiles][U + 3]
        const int per = (U + kBlock - 1) / kBlock;
        const int lo = threadIdx.x * per < U ? threadIdx.x * per : U;
        const int hi = lo + per < U ? lo + per : U;
        const bool writes_offsets = blockIdx.x == 0;                    // tile 0 exists whenever this kernel runs
        if constexpr (kParts > 1) {
            // fewer buckets than threads: kParts threads share a bucket, each sums every kParts-th tile
            const int b = threadIdx.x & (kBins - 1);
            const int part = threadIdx.x >> NBITS;
            uint32_t all = 0, before = 0;
            const int bc = b < U ? b : 0;
            constexpr int kAhead = 16;                                  // loads in flight, none behind a predicate
            for (int k0 = part; k0 < (int)tiles; k0 += kAhead * kParts) {
                uint32_t v[kAhead];
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    const int k = k0 + q * kParts;
                    v[q] = tile_hist[(k < (int)tiles ? k : (int)tiles - 1) * stride + bc];
                }
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    const int k = k0 + q * kParts;
                    all += k < (int)tiles ? v[q] : 0u;
                    before += k < (int)tile ? v[q] : 0u;
                }
            }
            part_all[threadIdx.x] = all;
            part_before[threadIdx.x] = before;
            __syncthreads();
        }
        uint32_t unused;
        if constexpr (SUM || NBITS < kRouteBasesBits) {
            uint32_t sum = 0;
            for (int b = lo; b < hi; ++b) {
                uint32_t all = 0, before = 0;
                if constexpr (kParts > 1) {
                    for (int q = 0; q < kParts && q < (int)tiles; ++q) { all += part_all[q * kBins + b]; before += part_before[q * kBins + b]; }
                } else if constexpr (SUM) {
#pragma unroll 8
                    for (int k = 0; k < (int)tiles; ++k) {
                        const uint32_t v = tile_hist[k * stride + b];
                        all += v;
                        before += k < (int)tile ? v : 0u;
                    }
                } else {
                    all = totals[b];
                    before = tile_hist[(int64_t)b * tiles + tile];
                }
                bucket_base[b] = sum + before;
                if (writes_offsets) bucket_offsets[b] = (int64_t)sum;   // both completed below
                sum += all;
            }
            const uint32_t run = block_exclusive_scan(sum, wave_sums, &unused);
            for (int b = lo; b < hi; ++b) {
                bucket_base[b] += run;
                if (writes_offsets) bucket_offsets[b] += (int64_t)run;
            }
        } else {
            constexpr int kPer = kBins / kBlock;                        // per <= kPer: a thread's loads all in flight
            uint32_t all[kPer], before[kPer];
            uint32_t sum = 0;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int b = lo + q < hi ? lo + q : U - 1;             // past its buckets: the last one again, unused
                all[q] = totals[b];
                before[q] = tile_hist[(int64_t)b * tiles + tile];
            }
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                if (lo + q >= hi) all[q] = 0;
                sum += all[q];
            }
            uint32_t run = block_exclusive_scan(sum, wave_sums, &unused);
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                if (lo + q < hi) {
                    bucket_base[lo + q] = run + before[q];
                    if (writes_offsets) bucket_offsets[lo + q] = (int64_t)run;
                    run += all[q];
                }
            }
        }
        if (writes_offsets) {
            if (threadIdx.x == 0) bucket_offsets[U] = n;                // every lookup has a bucket
            if (tier_counts != nullptr && w < 3) {                      // wave w adds up tier w
                uint32_t v = 0;
                if constexpr (SUM) {
                    for (int k = lane; k < (int)tiles; k += kWave) v += tile_hist[k * stride + U + w];
                    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
                } else {
                    v = totals[U + w];
                }
                if (lane == 0) tier_counts[w] = (int64_t)v;
            }
        }
    }
    for (int b = threadIdx.x; b < kWavesPerBlock * U; b += kBlock) wave_hist[b] = 0;
    __syncthreads();

    uint16_t* my_hist = wave_hist + w * U;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = base + (int64_t)w * (kWave * ITEMS) + it * kWave + lane;
        const bool valid = i < n;
        const uint64_t same = match_bits_n<NBITS>(dest[it], valid);
        const uint32_t before = popc_below(same);
        uint32_t seen = 0;
        if (valid) seen = my_hist[dest[it]];
        __builtin_amdgcn_wave_barrier();
        rank[it] = seen + before;
        if (valid && before == 0) my_hist[dest[it]] = (uint16_t)(seen + __popcll(same));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // per bucket: turn the waves' counts into the waves' first output index
    for (int b = threadIdx.x; b < U; b += kBlock) {
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < kWavesPerBlock; ++k) {
            const uint32_t v = wave_hist[k * U + b];
            wave_hist[k * U + b] = (uint16_t)run;
            run += v;
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = base + (int64_t)w * (kWave * ITEMS) + it * kWave + lane;
        if (i < n) {
            const uint32_t j = bucket_base[dest[it]] + my_hist[dest[it]] + rank[it];
            a.out_rows[j] = (int64_t)g[it];
            a.out_pos[j] = (int32_t)i;
            if (slot_in != nullptr) a.out_slots[j] = slot[it];
        }
    }
}

__global__ __launch_bounds__(kBlock) void route_finalize_kernel(
    int U, int64_t* __restrict__ bucket_offsets, int64_t* __restrict__ tier_counts)
{
    for (int b = threadIdx.x; b <= U; b += kBlock) bucket_offsets[b] = 0;
    if (tier_counts != nullptr && threadIdx.x < 3) tier_counts[threadIdx.x] = 0;
}

static int64_t route_tiles(int64_t n, int items) { return (n + kBlock * items - 1) / (kBlock * items); }

static int route_items(int64_t n, int64_t U)
{
    for (int k = 0; k < 2 && U <= kRouteSmallBuckets; ++k) {
        const int items = 2 << k;
        const int64_t tiles = route_tiles(n, items);
        if (tiles <= kRouteSmallTiles && tiles * (U + 3) <= kRouteSmallCounts[k]) return items;
    }
    return kRouteItems;
}

// Room for the tile counts, never less than a smaller batch or fewer buckets ask for: a workspace sized for a caller's
// largest batch serves the smaller ones.
static int64_t route_counts(int64_t n, int64_t U)
{
    int64_t counts = route_tiles(n, kRouteItems) * (U + 3);
    const int64_t small_buckets = U < kRouteSmallBuckets ? U : kRouteSmallBuckets;
    for (int k = 0; k < 2; ++k) {
        const int64_t tiles = route_tiles(n, 2 << k);
        int64_t small = (tiles < kRouteSmallTiles ? tiles : kRouteSmallTiles) * (small_buckets + 3);
        if (small > kRouteSmallCounts[k]) small = kRouteSmallCounts[k];
        if (counts < small) counts = small;
    }
    return counts;
}

// All three entry points: host checks, workspace carving, and the launches (remap, scan unless the counts are few, scatter).
static fs_status route_run(
    const int64_t* ids, const int64_t* offsets, int32_t T, int32_t B,
    const int64_t* row_base, const uint32_t* placement,
    int64_t n, int32_t U, int32_t W, int32_t self,
    int64_t* bucket_offsets, int64_t* out_rows, int32_t* out_pos,
    int64_t* tier_counts,
    void* workspace, size_t* workspace_bytes, void* stream, int32_t* dev_status,
    bool with_slots = false, int32_t* out_slots = nullptr)
{
    if (!workspace_bytes) return FS_ERR_NULL;
    if (n < 0 || n >= (1LL << 31) || T < 1 || B < 1 || (int64_t)T * B >= (1LL << 31)) return FS_ERR_SIZE;
    if (U < 1 || U > FS_MAX_BUCKETS || W < 1 || U % W != 0 || self < 0 || self >= U) return FS_ERR_CONFIG;

    const int items = route_items(n, U);
    const int64_t tiles = route_tiles(n, items);
    Carver ws(workspace);
    uint32_t* totals = ws.take<uint32_t>((size_t)U + 3);
    uint32_t* tile_hist = ws.take<uint32_t>((size_t)route_counts(n, U));
    uint32_t* g_tmp = ws.take<uint32_t>((size_t)n);
    uint16_t* dest_tmp = ws.take<uint16_t>((size_t)n);
    int32_t* slot_tmp = with_slots ? ws.take<int32_t>((size_t)n) : nullptr;
    if (!workspace) { *workspace_bytes = ws.used; return FS_OK; }
    if (*workspace_bytes < ws.used || (reinterpret_cast<uintptr_t>(workspace) & 255)) return FS_ERR_WORKSPACE;
    if (!offsets || !row_base || !placement || !bucket_offsets) return FS_ERR_NULL;
    if (n > 0 && (!ids || !out_rows || !out_pos || (with_slots && !out_slots))) return FS_ERR_NULL;

    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t S = (int64_t)T * B;
    const int dest_bits = bits_for((uint64_t)(U - 1));
    if (n == 0) {
        const unsigned prep_grid = (unsigned)((S + kBlock - 1) / kBlock < 1024 ? (S + kBlock - 1) / kBlock : 1024);
        FS_LAUNCH("route_prepare", route_prepare_kernel, dim3(prep_grid), dim3(kBlock), s,
                  offsets, S, n, dev_status);
        FS_LAUNCH("route_finalize", route_finalize_kernel, dim3(1), dim3(kBlock), s,
                  (int)U, bucket_offsets, tier_counts);
        return FS_OK;
    }
    {
        const bool sum = items < kRouteItems || tiles * ((int64_t)U + 3) <= kRouteSumMax;
        RouteArgs a;
        a.ids = ids; a.offsets = offsets; a.row_base = row_base; a.placement = placement;
        a.B = (int64_t)B; a.n = n; a.tiles = tiles;
        a.dest = dest_tmp; a.g = g_tmp; a.slot = slot_tmp; a.tile_hist = tile_hist; a.totals = totals;
        a.out_rows = out_rows; a.out_pos = out_pos; a.out_slots = out_slots;
        a.bucket_offsets = bucket_offsets; a.tier_counts = tier_counts; a.status = dev_status;
        a.T = (int)T; a.U = (int)U; a.W = (int)W; a.self = (int)self; a.by_tile = sum ? 1 : 0;
#define FS_REMAP(LEAD, ITEMS)                                                                                      \
    FS_LAUNCH_SMEM("route_remap", (route_remap_kernel<LEAD, ITEMS>), dim3((unsigned)tiles), dim3(kBlock), (size_t)U * sizeof(uint32_t), s, a)
        if (items == 2) FS_REMAP(false, 2);
        else if (items == 4) FS_REMAP(false, 4);
        else if (tiles > kRouteLeadTiles && U > 1) FS_REMAP(true, kRouteItems);
        else FS_REMAP(false, kRouteItems);
#undef FS_REMAP
        if (!sum)
            FS_LAUNCH("route_scan", route_scan_kernel, dim3((unsigned)U + 3), dim3(kRouteScanBlock), s, tile_hist, tiles, totals);
        const unsigned scatter_grid = (unsigned)(sum ? tiles : xcd_striped_grid(tiles, kRouteStripe));
        const size_t scatter_lds = (size_t)U * sizeof(uint32_t) + (size_t)kWavesPerBlock * U * sizeof(uint16_t);
#define FS_SCATTER_AS(NB, SUM, ITEMS)                                                                              \
    FS_LAUNCH_SMEM("route_scatter", (route_scatter_kernel<NB, SUM, ITEMS>), dim3(scatter_grid), dim3(kBlock), scatter_lds, s, a)
#define FS_SCATTER(NB)                                                                                             \
    if (sum) FS_SCATTER_AS(NB, true, kRouteItems);                                                                 \
    else FS_SCATTER_AS(NB, false, kRouteItems)
#define FS_SCATTER_SMALL(NB)                                                                                       \
    if (items == 2) FS_SCATTER_AS(NB, true, 2);                                                                    \
    else if (items == 4) FS_SCATTER_AS(NB, true, 4);                                                               \
    else FS_SCATTER(NB)
        switch (dest_bits) {                            // U <= FS_MAX_BUCKETS = 2^12
            case 1: FS_SCATTER_SMALL(1); break;  case 2: FS_SCATTER_SMALL(2); break;  case 3: FS_SCATTER_SMALL(3); break;
            case 4: FS_SCATTER_SMALL(4); break;  case 5: FS_SCATTER_SMALL(5); break;  case 6: FS_SCATTER_SMALL(6); break;
            case 7: FS_SCATTER_SMALL(7); break;  case 8: FS_SCATTER(8); break;  case 9: FS_SCATTER(9); break;
            case 10: FS_SCATTER(10); break;  case 11: FS_SCATTER(11); break;
            default: FS_SCATTER(12); break;
        }
#undef FS_SCATTER_SMALL
#undef FS_SCATTER
#undef FS_SCATTER_AS
    }
    return FS_OK;
}

// ---- the variant that allocates nothing ----------------------------------------
// Its workspace is this array: one copy per GPU, held until the process ends.  The name below is a
// host-side stand-in; the device address of each GPU's copy comes from hipGetSymbolAddress and is
// what every launch receives.
static __device__ __align__(256) unsigned char scratch[FS_ROUTE_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

static fs_status scratch_of_current_device(void** ptr)
{
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) return FS_ERR_DEVICE;
    void* p = g_scratch_ptr[device].load(std::memory_order_acquire);
    if (p == nullptr) {                                   // first call on this GPU (two racing threads find the same address)
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return FS_ERR_DEVICE;
        g_scratch_ptr[device].store(p, std::memory_order_release);
    }
    *ptr = p;
    return FS_OK;
}

}  // namespace fs

extern "C" fs_status fs_route_bucketize(
    const int64_t* ids, const int64_t* offsets, int32_t T, int32_t B,
    const int64_t* row_base, const uint32_t* placement,
    int64_t n, int32_t U, int32_t W, int32_t self,
    int64_t* bucket_offsets, int64_t* out_rows, int32_t* out_pos,
    int64_t* tier_counts,
    void* workspace, size_t* workspace_bytes, void* stream, int32_t* dev_status)
{
    return fs::route_run(ids, offsets, T, B, row_base, placement, n, U, W, self, bucket_offsets, out_rows, out_pos,
                         tier_counts, workspace, workspace_bytes, stream, dev_status);
}

extern "C" fs_status fs_route_bucketize_slots(
    const int64_t* ids, const int64_t* offsets, int32_t T, int32_t B,
    const int64_t* row_base, const uint32_t* placement,
    int64_t n, int32_t U, int32_t W, int32_t self,
    int64_t* bucket_offsets, int64_t* out_rows, int32_t* out_pos, int32_t* out_slots,
    int64_t* tier_counts,
    void* workspace, size_t* workspace_bytes, void* stream, int32_t* dev_status)
{
    return fs::route_run(ids, offsets, T, B, row_base, placement, n, U, W, self, bucket_offsets, out_rows, out_pos,
                         tier_counts, workspace, workspace_bytes, stream, dev_status, true, out_slots);
}

extern "C" fs_status fs_route_bucketize_noalloc(
    const int64_t* ids, const int64_t* offsets, int32_t T, int32_t B,
    const int64_t* row_base, const uint32_t* placement,
    int64_t n, int32_t U, int32_t W, int32_t self,
    int64_t* bucket_offsets, int64_t* out_rows, int32_t* out_pos,
    int64_t* tier_counts, void* stream, int32_t* dev_status)
{
    using namespace fs;
    size_t need = 0;                                      // size query: host checks only, nothing launched
    fs_status rc = route_run(ids, offsets, T, B, row_base, placement, n, U, W, self, bucket_offsets, out_rows, out_pos,
                             tier_counts, nullptr, &need, stream, dev_status);
    if (rc != FS_OK) return rc;
    if (need > (size_t)FS_ROUTE_NOALLOC_SCRATCH_BYTES) return FS_ERR_WORKSPACE;
    void* ws = nullptr;
    rc = scratch_of_current_device(&ws);
    if (rc != FS_OK) return rc;
    size_t have = (size_t)FS_ROUTE_NOALLOC_SCRATCH_BYTES;
    return route_run(ids, offsets, T, B, row_base, placement, n, U, W, self, bucket_offsets, out_rows, out_pos,
                     tier_counts, ws, &have, stream, dev_status);
}
