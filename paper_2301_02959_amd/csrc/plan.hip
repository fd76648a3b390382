// fs_plan_replication: row-frequency histogram and top-k rows under a byte budget.
//
// ACCUMULATE  plan_histogram: each block counts a span of the sampled ids (2048 to 2 M of them, see hist_span).  Zipf
//             samples hit a few rows most of the time, so a block counts in a table of 2^14 entries in LDS, two slots
//             to choose from for a row (the first row to claim a slot keeps it); only rows that find both taken and
//             the final flush reach the global counters, as saturating 32-bit atomic adds.  The offsets are checked by
//             the same blocks, or by plan_check_offsets before them where there are many.
// SELECT      plan_mark / plan_move: stable compaction of the candidate rows (count > 0, or all) in ascending row order into
//             (key = ~count, value = row), reading counts once (plan_scan between them where the tiles are many);
//             a stable radix sort by key then yields (count desc, row asc); plan_emit writes the
//             first k = min(budget / bytes_per_row, #candidates) rows, k, and the tier-0 tags.
// The candidate count lives in device memory; the sort kernels read it there.
//
// fs_plan_tiers (further down) reuses the compaction and the sort and cuts the sorted rows into
// tiers at the breakpoints of the per-row cost model.
#include "fs_common.h"
#include "radix_sort.h"

namespace fs {

constexpr int kSelTile = kBlock * 32;     // rows per block in the compaction (fewer, larger tiles: the one-block
                                          // scan of the tile counts is what they cost)

// Bad offsets count nothing, so all of them are checked before the first count.  Few segments and blocks: every
// block of the histogram checks them all itself (SELF).  Otherwise the blocks of this kernel check a share each and leave
// their verdicts, which every block of the histogram reads: no flag to set beforehand.
constexpr int kCheckBlocksMax = 256;          // one verdict per thread of a histogram block at most
constexpr int kCheckPerThread = 4;
constexpr int64_t kCheckSelfSegments = 8192;  // 8 segments to a thread of a histogram block
constexpr int64_t kCheckSelfBlocks = 256;     // at most 16 MB read out of the L2s in all; a launch costs 4 to 5 us

__global__ __launch_bounds__(kBlock) void plan_check_offsets_kernel(
    const int64_t* __restrict__ offsets, int64_t S, int64_t n, int32_t* __restrict__ verdicts, int32_t* status)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool bad = false;
    for (int64_t s = tid; s < S; s += stride) bad |= offsets[s] > offsets[s + 1];
    if (tid == 0) bad |= offsets[0] != 0 || offsets[S] != n;
    const int any = __syncthreads_or(bad);
    if (threadIdx.x == 0) {
        verdicts[blockIdx.x] = any ? 1 : 0;
        if (any) report(status, FS_DEV_BAD_OFFSETS);
    }
}

constexpr int kHistSlotBits = 14;
// Spans of up to 2048 ids (half as many as the slots) take 2^12 entries: a quarter of the slots to clear and to look through
// at the end.  8192 ids 7.3 -> 5.0 us (Zipf(1.3)), 7.6 -> 6.6 (Zipf(1.05)), 300 k 10.5 -> 8.4 and 14.6 -> 13.3.
constexpr int kHistSmallSlotBits = 12;
constexpr uint32_t kHistMul1 = 2654435761u, kHistMul1Inv = 0x0e8b2f51u;    // odd multipliers: bijections of 32-bit words,
constexpr uint32_t kHistMul2 = 2246822519u, kHistMul2Inv = 0xb6c92f47u;    // undone by their inverses mod 2^32
constexpr int kHistBlock = 1024;          // 16 waves per span: a span per 256 threads leaves the chip idle

// One block counts the ids of [blockIdx.x * span, + span) into an LDS table of 2^14 (short spans: 2^12) entries of 32 bits
// (64 KB: two blocks per CU, so that one block's flush, a stretch of nothing but global adds, runs beside
// the other's counting).  A row takes the first of its two slots (two hashes of the row) that is free or
// already its own; a row that finds both taken by other rows is added to the global counter at once.  An
// entry does not hold the row: the slot is the top 14 (12) bits of a hash that is a bijection of 32-bit words,
// so the other 18 (20) bits (plus one, so that a used entry is never zero, and one bit for which hash it was)
// name the row, and the 12 (10) bits above them count it; a count that wraps sends its 4096 (1024) to the global
// counter at once.  At the end the table is flushed with one saturating add per used slot.  The first row
// to claim a slot keeps it, so the counts stay exact.
// What the kernel costs is its global adds: the chip retires about 27 G of them a second wherever they land
// (one table of 64 KB or 1 GB of counters, one XCD's or all, returning or not), and a span cannot need fewer
// than it has distinct rows.  Measured: (row, count) pairs of 64 bits, half as many entries in the same LDS:
// 7 % slower on 10^9 ids of Zipf(1.3), 6 to 8 % on batches of 16 M and 72 M ids, 7 % FASTER on 67 M ids of
// Zipf(1.3) in one round of 512 blocks (fewer entries to flush when all blocks flush together); a quarter
// as many entries 3 to 13 % slower again; 2^14 pairs and one block per CU 0.49 ms instead of 0.39 ms on
// those 67 M ids; counting the most popular rows in registers changed nothing (the LDS is not the limit).
typedef int64_t Id2 __attribute__((ext_vector_type(2)));

template <bool SELF, int SLOT_BITS>
__global__ __launch_bounds__(kHistBlock) void plan_histogram_kernel(
    const int64_t* __restrict__ ids, const int64_t* __restrict__ offsets, int T, int64_t B,
    const int64_t* __restrict__ row_base, int64_t n, int64_t R, int64_t span, uint32_t* __restrict__ counts,
    const int32_t* __restrict__ verdicts, int num_verdicts, int32_t* status)
{
    constexpr int kSlots = 1 << SLOT_BITS;
    constexpr int kRestBits = 32 - SLOT_BITS;                   // bits of a row's hash that its slot does not give
    constexpr int kCountShift = kRestBits + 2;                      // entry: [count | which hash | rest + 1]
    constexpr uint32_t kTagMask = (1u << kCountShift) - 1u;
    constexpr uint32_t kCountMax = (1u << (32 - kCountShift)) - 1u;
    __shared__ uint32_t table[kSlots];         // 0 = free
    __shared__ int span_tables[2];
    bool bad = false;
    if constexpr (SELF) {
        const int S = (int)(T * B);            // at most kCheckSelfSegments
        for (int sg = threadIdx.x; sg < S; sg += kHistBlock) bad |= offsets[sg] > offsets[sg + 1];
        if (threadIdx.x == 0) bad |= offsets[0] != 0 || offsets[S] != n;
    } else {
        bad = (int)threadIdx.x < num_verdicts && verdicts[threadIdx.x] != 0;
    }
    const int64_t base = (int64_t)blockIdx.x * span;
    const int64_t end = base + span < n ? base + span : n;
    if (base >= end) return;
    for (int s = threadIdx.x; s < kSlots; s += kHistBlock) table[s] = 0;
    if (threadIdx.x < 2 * kWave) {              // a wave each for the first and the last id's table
        const int t = wave_table_of(offsets, T, B, threadIdx.x < kWave ? base : end - 1);
        if (lane_id() == 0) span_tables[wave_id()] = t;
    }
    if (__syncthreads_or(bad)) {               // bad offsets (they keep the search above in range): count nothing
        if (SELF && blockIdx.x == 0 && threadIdx.x == 0) report(status, FS_DEV_BAD_OFFSETS);
        return;
    }
    const int t_lo = __builtin_amdgcn_readfirstlane(span_tables[0]);
    const int t_hi = __builtin_amdgcn_readfirstlane(span_tables[1]);
    int32_t faults = 0;
    // Counts one row in the LDS table.  At most one global add comes of it: of 1 for a row that finds both
    // its slots taken, of a full count field for a row whose count in the table has just wrapped to zero.  The
    // add is issued here and its old value handed back (`*went` = the row + 1, `*amount`), so that the caller
    // can look at the answers of a whole batch of ids at once instead of waiting for each on its own.
    auto count_row = [&](uint32_t g, uint32_t* went, uint32_t* amount, uint32_t* old) {
        const uint32_t h1 = g * kHistMul1;
        const uint32_t s1 = h1 >> kRestBits;
        const uint32_t tag1 = (h1 & ((1u << kRestBits) - 1u)) + 1u;
        uint32_t e = table[s1];
        if (e == 0) e = atomicCAS(&table[s1], 0u, tag1);
        uint32_t* mine = nullptr;
        if (e == 0 || (e & kTagMask) == tag1) mine = &table[s1];
        else {
            const uint32_t h2 = (g ^ (g >> 15)) * kHistMul2;
            const uint32_t s2 = h2 >> kRestBits;
            const uint32_t tag2 = ((h2 & ((1u << kRestBits) - 1u)) + 1u) | (1u << (kRestBits + 1));
            e = table[s2];
            if (e == 0) e = atomicCAS(&table[s2], 0u, tag2);
            if (e == 0 || (e & kTagMask) == tag2) mine = &table[s2];
        }
        if (mine != nullptr) {
            // the count is the entry's top field: a carry out of it is lost, the tag below it stays whole
            const uint32_t before = atomicAdd(mine, 1u << kCountShift);
            if ((before >> kCountShift) != kCountMax) return;
            *amount = kCountMax + 1u;                               // wrapped to zero: that many counts go to memory now
        }
        *went = g + 1u;
        *old = atomicAdd(counts + g, *amount);
    };
    auto settle = [&](uint32_t went, uint32_t amount, uint32_t old) {   // the add wrapped: pin the counter at the maximum
        if (went != 0 && old > 0xFFFFFFFFu - amount) {
            atomicExch(counts + (went - 1u), 0xFFFFFFFFu);
            faults |= FS_DEV_COUNT_OVERFLOW;
        }
    };
    // The span table by table (nearly always one): the table's first row and size are the same for all of
    // its ids, so the loop over the ids loads nothing but the ids, two to a lane (16 bytes) where the
    // address allows it.
    // Where the rows change to another table's late in a span they find the slots taken by rows that don't come any more, the
    // new table's most popular ones too, and a quarter of the block's remaining ids go one by one to one global counter.  So
    // the slots are emptied first where that saves more than it costs, up to an add for every slot: from as many ids on as
    // there are slots with an eighth as many still to come, and from half as many on with twice as many still to come.
    // Never / from as many on, however few come / so, Zipf(1.2), 40 M rows in all, us: 34 M ids of 8 tables 363, 275 and 279,
    // 40 M 454, 459 and 307, 50 M 474, 361 and 361, 40 M of 26 382, 300 and 291, 60 M of 200 654, 526 and 350, 20 M of 1000
    // 250, 215 and 215, 72 M of 16, Zipf(1.1), 893, 815 and 817, 10^9 of 4, Zipf(1.3), 3.82, 3.19 and 3.19 ms; with only twice as
    // many still to come, however many came, 40 M of 26 364.  Up to 8 M ids, where every block is on the chip at once, the
    // block that empties its slots late is the last: 6 M of 16 67.6, 70.4 and 69.6, 7 M 76, 80 and 79, but 7 M of 1000 120,
    // 101 and 100.
    int64_t held = 0;                                                // ids counted since the slots were last empty
    for (int t = t_lo;; ++t) {
        const bool done = t > t_hi;
        int64_t lo = 0, hi = 0;
        if (!done) {
            lo = offsets[(int64_t)t * B];
            hi = offsets[(int64_t)(t + 1) * B];
            lo = lo > base ? lo : base;
            hi = hi < end ? hi : end;
            if (lo >= hi) continue;
        }
        const bool empty = held >= kSlots / 2 && end - lo >= (held >= kSlots ? kSlots / 8 : 2 * kSlots);
        if (done || empty) {                                         // block-uniform
            __syncthreads();
            // The flush: one saturating add per used slot.  A thread's adds are all issued before the first old
            // value is looked at: one after the other, each waiting for its answer, they are the longest stretch
            // of a span (nothing else runs on the CU beside the block that holds its LDS).
            constexpr int kPerThread = kSlots / kHistBlock;
            constexpr int kBatch = kPerThread < 8 ? kPerThread : 8;
#pragma unroll 1
            for (int s0 = 0; s0 < kPerThread; s0 += kBatch) {
                uint32_t tag[kBatch], add[kBatch], old[kBatch];
#pragma unroll
                for (int q = 0; q < kBatch; ++q) {
                    const int s = (s0 + q) * kHistBlock + threadIdx.x;
                    const uint32_t e = table[s];
                    table[s] = 0;
                    add[q] = e >> kCountShift;
                    // the row back from its slot and the rest of its hash: both hashes are bijections of 32-bit words
                    const uint32_t h = ((uint32_t)s << kRestBits) | ((e & ((1u << (kRestBits + 1)) - 1u)) - 1u);
                    uint32_t g;
                    if ((e >> (kRestBits + 1)) & 1u) {
                        const uint32_t y = h * kHistMul2Inv;
                        g = y ^ (y >> 15) ^ (y >> 30);
                    } else {
                        g = h * kHistMul1Inv;
                    }
                    tag[q] = e != 0 ? g + 1u : 0u;
                }
#pragma unroll
                for (int q = 0; q < kBatch; ++q)
                    old[q] = (tag[q] != 0 && add[q] != 0) ? atomicAdd(counts + (tag[q] - 1u), add[q]) : 0u;
#pragma unroll
                for (int q = 0; q < kBatch; ++q) {
                    if (tag[q] != 0 && add[q] != 0 && old[q] > 0xFFFFFFFFu - add[q]) {     // wrapped: pin the counter at the maximum
                        atomicExch(counts + (tag[q] - 1u), 0xFFFFFFFFu);
                        faults |= FS_DEV_COUNT_OVERFLOW;
                    }
                }
            }
            if (done) break;
            __syncthreads();
            held = 0;
        }
        held += hi - lo;
        const int64_t first = row_base[t];
        const int64_t rows_t = row_base[t + 1] - first;
        auto count_one = [&](int64_t id, uint32_t* went, uint32_t* amount, uint32_t* old) {
            *went = 0;
            *amount = 1u;
            *old = 0;
            if (id < 0 || id >= rows_t) { faults |= FS_DEV_BAD_ID; id = 0; }
            if ((uint64_t)(first + id) >= (uint64_t)R) { faults |= FS_DEV_BAD_ID; return; }   // row_base does not fit R
            count_row((uint32_t)(first + id), went, amount, old);
        };
        if ((reinterpret_cast<uintptr_t>(ids + lo) & 15) != 0) {         // an odd first id: on its own
            if (threadIdx.x == 0) {
                uint32_t went, amount, old;
                count_one(load_stream(ids + lo), &went, &amount, &old);
                settle(went, amount, old);
            }
            ++lo;
        }
        const Id2* pairs = reinterpret_cast<const Id2*>(ids + lo);
        const int64_t num_pairs = (hi - lo) >> 1;
        constexpr int kAhead = 4;                                // pairs of ids in flight per thread
        int64_t p = threadIdx.x;
        for (; p + (int64_t)(kAhead - 1) * kHistBlock < num_pairs; p += (int64_t)kAhead * kHistBlock) {
            Id2 id[kAhead];
            uint32_t went[2 * kAhead], amount[2 * kAhead], old[2 * kAhead];
#pragma unroll
            for (int q = 0; q < kAhead; ++q) id[q] = load_stream(pairs + p + (int64_t)q * kHistBlock);
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                count_one(id[q].x, &went[2 * q], &amount[2 * q], &old[2 * q]);
                count_one(id[q].y, &went[2 * q + 1], &amount[2 * q + 1], &old[2 * q + 1]);
            }
#pragma unroll
            for (int q = 0; q < 2 * kAhead; ++q) settle(went[q], amount[q], old[q]);
        }
        for (; p < num_pairs; p += kHistBlock) {
            const Id2 id = load_stream(pairs + p);
            uint32_t went[2], amount[2], old[2];
            count_one(id.x, &went[0], &amount[0], &old[0]);
            count_one(id.y, &went[1], &amount[1], &old[1]);
            settle(went[0], amount[0], old[0]);
            settle(went[1], amount[1], old[1]);
        }
        if (((hi - lo) & 1) != 0 && threadIdx.x == kHistBlock - 1) {     // an odd last id
            uint32_t went, amount, old;
            count_one(load_stream(ids + hi - 1), &went, &amount, &old);
            settle(went, amount, old);
        }
    }
    if (ballot(faults != 0) != 0) {
        for (int off = 32; off > 0; off >>= 1) faults |= __shfl_down(faults, off);
        if (lane_id() == 0) report(status, faults);
    }
}

// Span length for n ids: 2048 ids up to 256 spans, then 129 to 256 spans of whole rounds of 2048 ids, up to 32 k each (one
// block of 8192 ids spends its time on its 16 k slots and a chain of rounds: 14.9 us, four blocks of 2048 with the offsets
// checked inside 8.6; 4.2 M ids 105 us at 16 k as at 32 k), then 32 k spans.  Shorter spans are never more than 256, so that
// the blocks check the offsets themselves (257 and a launch for the check: 7 us more); rounds broken up for a span on every
// CU gain nothing (540 k ids in 235 spans of 2304 23.6 us, in 132 of 4096 22.5).  From one 64 k span for each of the two
// blocks a CU holds, spans of up to 128 k ids, shortened so that their number is a multiple of the CU count
// where that is possible.  A popular row is flushed once per span, so a planning pass over very many ids
// (from 2^27) takes spans of up to 2 M ids, all of one length and a whole number of rounds over the chip's
// 512 resident blocks: 10^9 ids of Zipf(1.3) over 4 tables 3.47 ms with spans of up to 512 k, 3.15 with 1 M, 2.89 with 2 M, 400 M
// 1.52 and 1.32, 600 M of Zipf(1.05) 8.73 and 8.72.  A training batch of a flatter law (72 M ids of Zipf(1.1) over 16 tables)
// did better with the shorter spans (1.13 ms at 96 k, 1.25 ms at 144 k): the first rows to arrive keep the slots, and a fresh
// table serves the rows that repeat within a stretch.
constexpr int64_t kHistSpanSmall = 32768;
constexpr int64_t kHistSpanLarge = 131072;
constexpr int64_t kHistSpanHuge = 2097152;
constexpr int64_t kHistHugeFrom = (int64_t)1 << 27;
constexpr int64_t kHistCus = 256;

static int64_t hist_span(int64_t n)
{
    if (n < 2 * kHistCus * (kHistSpanLarge / 2)) {                // under one 64 k span for every CU, twice over
        const int64_t share = ((n + kHistCus - 1) / kHistCus + 2047) / 2048 * 2048;
        return share < kHistSpanSmall ? (share > 2048 ? share : 2048) : kHistSpanSmall;
    }
    const int64_t longest = n >= kHistHugeFrom ? kHistSpanHuge : kHistSpanLarge;
    const int64_t per_round = n >= kHistHugeFrom ? 2 * kHistCus : kHistCus;
    const int64_t rounds = (n + per_round * longest - 1) / (per_round * longest);
    int64_t s = (n + per_round * rounds - 1) / (per_round * rounds);
    s = (s + 8191) / 8192 * 8192;                                // whole rounds of 8 ids per thread
    return s < longest ? s : longest;
}

// ---- selection --------------------------------------------------------------
// Reads counts once: each wave packs the candidates of its 2048 rows, in row order, at their own place in a staging
// buffer, four waves to a tile of 8192 rows, whose candidates are counted.
// VEC: a lane loads four consecutive counters at once (counts 16-byte aligned); the packed order is the same.
// Bound by the stream of the counters: 80 M of them, 1.6 M
// candidates, 62 us (5.1 TB/s), 200 M 181.  With the positions of all 32 rows of a lane held until the block's waves had met,
// 66 and 195 (three times the registers, twice the vector instructions).
constexpr int kMarkSpan = kSelTile / kWavesPerBlock;      // consecutive rows per wave

// The number of candidates of each wave's share, 16 bits each, first wave lowest.
typedef uint64_t WaveCounts;

template <bool VEC, bool ZERO>
__global__ __launch_bounds__(kBlock) void plan_mark_kernel(
    const uint32_t* __restrict__ counts, int64_t R, uint32_t* __restrict__ tile_count, WaveCounts* __restrict__ tile_waves,
    uint32_t* __restrict__ tile_bits, SortPair* __restrict__ stage)
{
    __shared__ uint32_t wave_sum[kWavesPerBlock];
    __shared__ uint32_t wave_bits[kWavesPerBlock];
    constexpr int kItems = kMarkSpan / kWave;
    constexpr int kStep = VEC ? 4 : 1;                    // consecutive rows per lane and load
    const int w = wave_id();
    const int lane = lane_id();
    const int64_t base = (int64_t)blockIdx.x * kSelTile + (int64_t)w * kMarkSpan;
    const uint32_t rows = (uint32_t)(R - base < kMarkSpan ? (R - base < 0 ? 0 : R - base) : kMarkSpan);      // the wave's
    const bool whole = rows == kMarkSpan;
    // item `it` of a lane is row base + row_of(it): with VEC, load it / 4 brings rows 4 * lane .. 4 * lane + 3 of a
    // stretch of 256
    auto row_of = [&](int it) -> uint32_t { return VEC ? (it / 4) * (kWave * 4) + lane * 4 + (it & 3) : it * kWave + lane; };
    uint32_t cnt[kItems];
    const uint32_t* mine = counts + base;
    if (whole) {
        if constexpr (VEC) {
#pragma unroll
            for (int v = 0; v < kItems / 4; ++v) {
                const u32x4 c = reinterpret_cast<const u32x4*>(mine)[v * kWave + lane];
                cnt[4 * v] = c[0]; cnt[4 * v + 1] = c[1]; cnt[4 * v + 2] = c[2]; cnt[4 * v + 3] = c[3];
            }
        } else {
#pragma unroll
            for (int it = 0; it < kItems; ++it) cnt[it] = mine[row_of(it)];
        }
    } else {
#pragma unroll
        for (int it = 0; it < kItems; ++it) cnt[it] = row_of(it) < rows ? mine[row_of(it)] : 0u;
    }
    SortPair* const to = stage + base;
    const uint32_t first = (uint32_t)base;                // rows are below 2^32
    uint32_t total = 0, bits = 0;                         // bits: the counts or-ed together: how many bits the sort has to look at
    // Position of a candidate among the wave's: those of earlier stretches, those of lower lanes in its stretch
    // (one ballot per item position), and the lane's own earlier items of the stretch.
#pragma unroll
    for (int it0 = 0; it0 < kItems; it0 += kStep) {
        uint64_t cand[kStep];
        uint32_t at = total;
#pragma unroll
        for (int e = 0; e < kStep; ++e) {
            cand[e] = ballot(ZERO ? (whole || row_of(it0 + e) < rows) : cnt[it0 + e] != 0u);
            at = __builtin_amdgcn_mbcnt_hi((uint32_t)(cand[e] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)cand[e], at));
            total += (uint32_t)__popcll(cand[e]);
            bits |= cnt[it0 + e];
        }
#pragma unroll
        for (int e = 0; e < kStep; ++e) {
            if (ZERO ? (whole || row_of(it0 + e) < rows) : cnt[it0 + e] != 0u) {
                to[at] = SortPair{~cnt[it0 + e], first + row_of(it0 + e)};
                ++at;
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) bits |= __shfl_xor(bits, o);
    if (lane == 0) { wave_sum[w] = total; wave_bits[w] = bits; }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t all = 0;
        WaveCounts each = 0;
        bits = 0;
        for (int k = 0; k < kWavesPerBlock; ++k) {
            all += wave_sum[k];
            each |= (WaveCounts)wave_sum[k] << (16 * k);
            bits |= wave_bits[k];
        }
        tile_count[blockIdx.x] = all;
        tile_waves[blockIdx.x] = each;
        tile_bits[blockIdx.x] = bits;
    }
}

static fs_status launch_mark(const uint32_t* counts, int64_t R, int allow_zero, int64_t sel_tiles, uint32_t* tile_count,
                             WaveCounts* tile_waves, uint32_t* tile_bits, SortPair* stage, hipStream_t s)
{
#define FS_MARK(VEC, ZERO)                                                                                          \
    FS_LAUNCH("plan_mark", (plan_mark_kernel<VEC, ZERO>), dim3((unsigned)sel_tiles), dim3(kBlock), s,                \
              counts, R, tile_count, tile_waves, tile_bits, stage)
    const bool vec = (reinterpret_cast<uintptr_t>(counts) & 15) == 0;
    if (vec && !allow_zero) FS_MARK(true, false);
    else if (vec) FS_MARK(true, true);
    else if (!allow_zero) FS_MARK(false, false);
    else FS_MARK(false, true);
#undef FS_MARK
    return FS_OK;
}

constexpr int kScanBlock = 1024;

// `v` or-ed over the threads of the block, in every thread.  `waves` is LDS scratch of 16 words.
__device__ __forceinline__ uint32_t block_or(uint32_t v, uint32_t* waves)
{
    for (int off = 32; off > 0; off >>= 1) v |= __shfl_xor(v, off);
    if (lane_id() == 0) waves[wave_id()] = v;
    __syncthreads();
    v = 0;
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) v |= waves[k];
    return v;
}

constexpr int64_t kScanLdsTiles = 15 * kScanBlock;               // 126 M rows: 60 KB of LDS

__host__ __device__ inline int scan_run(int64_t tiles) { return (int)((tiles + kScanBlock - 1) / kScanBlock) | 1; }

__global__ __launch_bounds__(kScanBlock) void plan_scan_kernel(uint32_t* __restrict__ tile_count, int64_t tiles,
                                                               const uint32_t* __restrict__ tile_bits,
                                                               int64_t* __restrict__ num_candidates,
                                                               uint32_t* __restrict__ count_bits)
{
    __shared__ uint32_t wave_bits[16];
    __shared__ uint32_t wave_sums[16];
    extern __shared__ uint32_t s_count[];                        // [kScanBlock * per] where the tiles fit
    if (tiles <= kScanLdsTiles) {
        // The counts to LDS, every load in flight at once; a thread sums a run of consecutive tiles there (an odd number
        // of them: no two lanes' runs start in one bank), ONE scan over the block's 1024 sums, the thread then leaves its
        // run's prefixes in place.  9.8 k tiles 6.8 us; each thread summing its run from memory 12.
        const int per = scan_run(tiles);
        const int lo = threadIdx.x * per;
        uint32_t bits = 0;
        constexpr int kRound = 16;
        for (int q0 = 0; q0 < per; q0 += kRound) {
            uint32_t v[kRound], b[kRound];
#pragma unroll
            for (int q = 0; q < kRound; ++q) {
                const int k = (q0 + q) * kScanBlock + (int)threadIdx.x;
                v[q] = tile_count[k < tiles ? k : tiles - 1];
                b[q] = tile_bits[k < tiles ? k : tiles - 1];
            }
#pragma unroll
            for (int q = 0; q < kRound; ++q) {
                const int k = (q0 + q) * kScanBlock + (int)threadIdx.x;
                if (q0 + q < per) s_count[k] = k < tiles ? v[q] : 0u;
                bits |= b[q];                                    // past the end: the last tile's again
            }
        }
        __syncthreads();
        uint32_t sum = 0;
        for (int k = lo; k < lo + per; ++k) sum += s_count[k];
        uint32_t total;
        uint32_t run = block_exclusive_scan(sum, wave_sums, &total);
        for (int k = lo; k < lo + per; ++k) { const uint32_t v = s_count[k]; s_count[k] = run; run += v; }
        __syncthreads();
        for (int k = threadIdx.x; k < tiles; k += kScanBlock) tile_count[k] = s_count[k];
        bits = block_or(bits, wave_bits);
        if (threadIdx.x == 0) { *num_candidates = (int64_t)total; *count_bits = bits; }
        return;
    }
    uint32_t bits = 0;
    uint32_t carry = 0;                                          // coalesced rounds of 1024 tiles, 8 rounds of loads in flight
    for (int64_t base = 0; base < tiles; base += 8 * kScanBlock) {
        uint32_t v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t k = base + (int64_t)q * kScanBlock + threadIdx.x;
            v[q] = k < tiles ? tile_count[k] : 0u;
            bits |= k < tiles ? tile_bits[k] : 0u;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t k = base + (int64_t)q * kScanBlock + threadIdx.x;
            uint32_t total;
            const uint32_t before = block_exclusive_scan(v[q], wave_sums, &total);
            if (k < tiles) tile_count[k] = carry + before;
            carry += total;
        }
    }
    bits = block_or(bits, wave_bits);
    if (threadIdx.x == 0) { *num_candidates = (int64_t)carry; *count_bits = bits; }
}

// Moves each tile's packed candidates to their final place (tile_base = scanned tile counts).
// SUM: few tiles, plan_scan has not run: tile_base holds plain counts, every block sums those before its own, and the
// first one writes the number of candidates and the bits of their counts.
template <bool SUM>
__global__ __launch_bounds__(kBlock) void plan_move_kernel(
    const uint32_t* __restrict__ tile_base, const WaveCounts* __restrict__ tile_waves, int64_t tiles,
    const uint32_t* __restrict__ tile_bits, int64_t* __restrict__ num_candidates, uint32_t* __restrict__ count_bits,
    const SortPair* __restrict__ stage, SortPair* __restrict__ pairs)
{
    const int64_t tile = blockIdx.x;
    const WaveCounts each = tile_waves[tile];
    uint32_t first;
    if constexpr (SUM) {
        __shared__ uint32_t wave_sums[16];
        __shared__ uint32_t wave_bits[16];
        uint32_t before = 0, bits = 0;
        const int64_t last = tile == 0 ? tiles : tile;           // the first block adds up all of them
        for (int64_t k = threadIdx.x; k < last; k += kBlock) {
            before += tile_base[k];
            if (tile == 0) bits |= tile_bits[k];
        }
        uint32_t sum;
        block_exclusive_scan(before, wave_sums, &sum);
        first = tile == 0 ? 0u : sum;
        if (tile == 0) {                                         // block-uniform
            bits = block_or(bits, wave_bits);
            if (threadIdx.x == 0) { *num_candidates = (int64_t)sum; *count_bits = bits; }
        }
    } else {
        first = tile_base[tile];
    }
    // a wave moves the candidates of the wave that packed them
    const int w = wave_id();
    for (int k = 0; k < w; ++k) first += (uint32_t)(each >> (16 * k)) & 0xFFFFu;
    const uint32_t n = (uint32_t)(each >> (16 * w)) & 0xFFFFu;
    const SortPair* from = stage + tile * kSelTile + w * kMarkSpan;
    for (uint32_t i = lane_id(); i < n; i += kWave) pairs[first + i] = from[i];
}

// Compaction and sort of the candidates, shared by the two planners: rows in (count desc, row asc) order behind their
// keys ~count, in pairs_a or pairs_b as sort_result_in_b(*count_bits, first_bits) says.
// Up to 1024 tiles (8 M rows) the moving blocks sum the tile counts themselves, at most four loads to a thread, and
// the scan is no launch of its own; beyond, what each of the blocks would read again is more than the scan costs.
constexpr int64_t kMoveSumTiles = 1024;

struct PlanScratch {
    int64_t* num_cand;
    uint32_t* count_bits;
    uint32_t* tile_count;
    uint32_t* tile_bits;
    WaveCounts* tile_waves;
    SortPair* pairs_a;
    SortPair* pairs_b;
    char* sort_scratch;
    int first_bits;
};

// Digits of the selection's sort: 10, 10, 6, 6 bits up to 2^26 rows, 8, 8, 8, 8 beyond; as many passes run as the
// largest count needs.  Over few candidates a pass costs its launches, and counts below 1024 (small batches) or of 17 to 20
// bits (profiles) take a pass less with the wide digits; a wide pass over many candidates costs up to two narrow ones, and
// the more rows, the more of them a profile touches.  Sort in us, wide : narrow, for largest counts of 9 / 15 / 20 / 23 / 27
// bits: 4 M rows, 160 k candidates 81 : 85, 91 : 86, 92 : 93, 99 : 93, 105 : 100; 32 M, 1.3 M 87 : 94, 103 : 94, 104 : 106,
// 116 : 108, 127 : 117; 80 M, 16 M 195 : 225, 317 : 225, 319 : 300, 386 : 303, 464 : 378.  Digits of
// 10, 10, 10, 2 bits cost 124 on 32 M rows and 23 bits, and 1221 : 1010 on 200 M rows, 50 M candidates and 27 bits.
constexpr int64_t kSelectionWideRows = (int64_t)1 << 26;

static int selection_first_bits(int64_t R) { return R <= kSelectionWideRows ? 10 : 8; }

static PlanScratch take_plan_scratch(Carver& ws, int64_t R)
{
    PlanScratch p;
    const size_t tiles = (size_t)((R + kSelTile - 1) / kSelTile);
    p.num_cand = ws.take<int64_t>(1);
    p.count_bits = ws.take<uint32_t>(1);
    p.tile_count = ws.take<uint32_t>(tiles);
    p.tile_bits = ws.take<uint32_t>(tiles);
    p.tile_waves = ws.take<WaveCounts>(tiles);
    p.pairs_a = ws.take<SortPair>((size_t)R);
    p.pairs_b = ws.take<SortPair>((size_t)R);
    p.sort_scratch = ws.take<char>(R > 0 ? radix_sort_scratch_bytes(R) : 0);
    p.first_bits = selection_first_bits(R);
    return p;
}

static fs_status sort_candidates(const uint32_t* counts, int64_t R, int allow_zero, const PlanScratch& p, hipStream_t s)
{
    const int64_t tiles = (R + kSelTile - 1) / kSelTile;
    if (fs_status rc = launch_mark(counts, R, allow_zero, tiles, p.tile_count, p.tile_waves, p.tile_bits, p.pairs_b, s); rc != FS_OK) return rc;
    if (tiles <= kMoveSumTiles) {
        FS_LAUNCH("plan_move", plan_move_kernel<true>, dim3((unsigned)tiles), dim3(kBlock), s, p.tile_count, p.tile_waves, tiles,
                  p.tile_bits, p.num_cand, p.count_bits, p.pairs_b, p.pairs_a);
    } else {
        const size_t lds = tiles <= kScanLdsTiles ? (size_t)kScanBlock * (size_t)scan_run(tiles) * sizeof(uint32_t) : 0;
        FS_LAUNCH_SMEM("plan_scan", plan_scan_kernel, dim3(1), dim3(kScanBlock), lds, s, p.tile_count, tiles, p.tile_bits, p.num_cand,
                       p.count_bits);
        FS_LAUNCH("plan_move", plan_move_kernel<false>, dim3((unsigned)tiles), dim3(kBlock), s, p.tile_count, p.tile_waves, tiles,
                  p.tile_bits, p.num_cand, p.count_bits, p.pairs_b, p.pairs_a);
    }
    SortJob job;
    job.pairs_a = p.pairs_a; job.pairs_b = p.pairs_b;
    job.m_max = R; job.m_dev = p.num_cand;
    job.varying = p.count_bits; job.first_bits = p.first_bits;
    job.scratch = p.sort_scratch; job.stream = s;
    return radix_sort(job);
}

__global__ __launch_bounds__(kBlock) void plan_emit_kernel(
    const SortPair* __restrict__ pairs_a, const SortPair* __restrict__ pairs_b, const uint32_t* __restrict__ count_bits, int first_bits, const int64_t* __restrict__ num_candidates, int64_t cap,
    int64_t* __restrict__ sel_rows, int64_t* __restrict__ num_selected, uint32_t* __restrict__ placement)
{
    const SortPair* pairs = sort_result_in_b(*count_bits, first_bits) ? pairs_b : pairs_a;
    const int64_t nc = *num_candidates;
    const int64_t k = cap < nc ? cap : nc;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < k; i += stride) {
        const uint32_t g = pairs[i][1];
        sel_rows[i] = (int64_t)g;
        if (placement != nullptr) placement[g] &= FS_OWNER_MASK;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *num_selected = k;
}

// ---- tier planner -----------------------------------------------------------
// After the same compaction and sort, rows stand in descending frequency order with
// key = ~count.  The breakpoints are thresholds on the count (found on the host from the
// parameters), so points A, C and the Flex breakpoint are partition points of the sorted keys;
// point B and the Flex budget need sums of counts over prefixes, which come from one pass of
// per-tile sums plus a scan of those.  One block then finds every cut, a wave to each 64-way search.
constexpr int kSumTile = 4096;                // sorted counts per tile sum

typedef unsigned __int128 u128;
typedef __int128 i128;

struct TierConsts {
    uint64_t thr_a, thr_c, thr_f;             // smallest count at or above the breakpoint (2^63: none)
    int64_t static_term;                      // (dp U - 1) S
    int64_t dyn_factor;                       // U B
    int64_t flex_cost;                        // (dp U / W - 1) S
    int32_t granule, W, tiers;
};

__global__ __launch_bounds__(kBlock) void tiers_tile_sums_kernel(
    const SortPair* __restrict__ pairs_a, const SortPair* __restrict__ pairs_b, const uint32_t* __restrict__ count_bits, int first_bits,
    const int64_t* __restrict__ num_candidates, uint64_t* __restrict__ tile_sum)
{
    const SortPair* pairs = sort_result_in_b(*count_bits, first_bits) ? pairs_b : pairs_a;
    __shared__ uint64_t part[kWavesPerBlock];
    const int64_t K = *num_candidates;
    // candidates are usually a few per cent of the rows: the blocks walk the tiles that hold any (a block for every
    // 4096 rows: 13 us for 40 M rows, now 6.5, and the scan of the sums 16, now 4.4)
    for (int64_t tile = blockIdx.x; tile * kSumTile < K; tile += gridDim.x) {
        const int64_t base = tile * kSumTile;
        uint64_t sum = 0;
#pragma unroll
        for (int i = 0; i < kSumTile / kBlock; ++i) {
            const int64_t k = base + i * kBlock + threadIdx.x;
            sum += k < K ? (uint32_t)~pairs[k][0] : 0u;
        }
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off);
        if (lane_id() == 0) part[wave_id()] = sum;
        __syncthreads();
        if (threadIdx.x == 0) tile_sum[tile] = part[0] + part[1] + part[2] + part[3];
        __syncthreads();
    }
}

// tile_sum[t] -> sum of the tiles before t, for the tiles that hold candidates, and the grand total behind them.  One block.
__global__ __launch_bounds__(kScanBlock) void tiers_scan_sums_kernel(uint64_t* __restrict__ tile_sum,
                                                                     const int64_t* __restrict__ num_candidates)
{
    const int64_t tiles = (*num_candidates + kSumTile - 1) / kSumTile;
    __shared__ uint64_t wave_tot[kScanBlock / kWave];
    const int lane = lane_id();
    const int w = wave_id();
    uint64_t carry = 0;
    for (int64_t base = 0; base < tiles; base += kScanBlock) {
        const int64_t k = base + threadIdx.x;
        const uint64_t v = k < tiles ? tile_sum[k] : 0;
        uint64_t incl = v;
        for (int off = 1; off < kWave; off <<= 1) {
            const uint64_t up = __shfl_up(incl, off);
            if (lane >= off) incl += up;
        }
        __syncthreads();                       // wave_tot of the previous round has been read
        if (lane == kWave - 1) wave_tot[w] = incl;
        __syncthreads();
        uint64_t before = 0, all = 0;
        for (int q = 0; q < kScanBlock / kWave; ++q) {
            const uint64_t t = wave_tot[q];
            if (q < w) before += t;
            all += t;
        }
        if (k < tiles) tile_sum[k] = carry + before + incl - v;
        carry += all;
    }
    if (threadIdx.x == 0) tile_sum[tiles] = carry;
}

// First index in [lo, hi) at which pred turns false (pred holds on a prefix of the range); hi if it
// never does.  Every lane of the wave calls it with the same bounds; 64 probes per round.
template <typename Pred>
__device__ __forceinline__ int64_t wave_partition_point(int64_t lo, int64_t hi, Pred pred)
{
    const int lane = lane_id();
    while (lo < hi) {
        const int64_t step = (hi - lo + kWave - 1) / kWave;
        const int64_t probe = lo + (int64_t)(lane + 1) * step - 1;      // last index of this lane's piece
        const bool holds = probe < hi ? pred(probe) : false;
        int pieces = __popcll(ballot(holds));                            // whole pieces on which pred holds
        // The count is the same in every lane, and left to itself the compiler does the two bound updates
        // below in scalar registers, where (hipcc of ROCm 7.2, gfx950) the second of two back-to-back
        // 64-bit compare-and-selects reuses the first one's condition bit: lo then takes hi's branch
        // whenever the probe past new_lo lies outside the range.  Held in a vector register the count
        // makes them vector selects.
        asm volatile("" : "+v"(pieces));
        const int64_t new_lo = lo + (int64_t)pieces * step;
        const int64_t first_false_probe = new_lo + step - 1;
        hi = first_false_probe < hi ? first_false_probe : hi;
        lo = new_lo < hi ? new_lo : hi;
    }
    return lo;
}

// Sum of the first k sorted counts: the scanned tile sums plus a partial tile, summed by the block with every load in flight
// at once.  `waves` is LDS scratch; every thread of the block must call it.
__device__ __forceinline__ uint64_t prefix_count(const SortPair* __restrict__ pairs, const uint64_t* __restrict__ tile_sum,
                                                 int64_t k, uint64_t* waves)
{
    const int64_t t = k / kSumTile;
    const int rest = (int)(k - t * kSumTile);
    constexpr int kPer = kSumTile / kBlock;
    const uint64_t before = tile_sum[t];
    uint32_t v[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = j * kBlock + (int)threadIdx.x;
        v[j] = ~pairs[i < rest ? t * kSumTile + i : 0][0];
    }
    uint64_t part = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) part += j * kBlock + (int)threadIdx.x < rest ? v[j] : 0u;
    for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
    __syncthreads();                                                 // `waves` may still be read from a previous call
    if (lane_id() == 0) waves[wave_id()] = part;
    __syncthreads();
    uint64_t sum = before;
    for (int q = 0; q < kWavesPerBlock; ++q) sum += waves[q];
    return sum;
}

// Summed DP memory terms of the first k rows, times U * S:  k (dp U - 1) S - U B P(k).
__device__ __forceinline__ i128 cum_memory(const TierConsts& c, int64_t k, uint64_t prefix)
{
    return (i128)k * (i128)c.static_term - (i128)c.dyn_factor * (i128)prefix;
}

// The searches are chains of dependent loads, so each has a wave of its own: breakpoints A, C and FLEX and point B.
// The budget and the sums of the two tiers follow, the sums' partial tiles read by the whole block at once.  1.5 M candidates:
// one wave doing all of it, and every row of point B's tile tested on its own, 39 us; the sums by the first wave, 16 loads
// in flight, the first tier's three times over, 29; so 12.
__global__ __launch_bounds__(kBlock) void tiers_cuts_kernel(
    const SortPair* __restrict__ pairs_a, const SortPair* __restrict__ pairs_b, const uint32_t* __restrict__ count_bits, int first_bits,
    const int64_t* __restrict__ num_candidates,
    const uint64_t* __restrict__ tile_sum, const TierConsts c, int64_t* __restrict__ cuts)
{
    const SortPair* pairs = sort_result_in_b(*count_bits, first_bits) ? pairs_b : pairs_a;
    const int lane = lane_id();
    const int64_t K = *num_candidates;
    const int64_t tiles = (K + kSumTile - 1) / kSumTile;
    auto at_least = [&](uint64_t thr) {
        return wave_partition_point(0, K, [&](int64_t i) { return (uint64_t)(uint32_t)~pairs[i][0] >= thr; });
    };
    __shared__ int64_t found[kWavesPerBlock];
    const int w = __builtin_amdgcn_readfirstlane(wave_id());
    if (w < 3) {
        const int64_t at = at_least(w == 0 ? c.thr_a : w == 1 ? c.thr_c : c.thr_f);
        if (lane == 0) found[w] = at;
    }
    if (w == 3) {
        // point B: the summed terms are <= 0 on a prefix of k = 0 .. K.  Tile boundaries first
        // (k_t = min(t * tile, K), P(k_t) = tile_sum[t]), then pieces of 64 rows of the one tile that holds it,
        // then the rows of the one piece.
        const int64_t t_false = wave_partition_point(0, tiles + 1, [&](int64_t t) {
            const int64_t k = t * kSumTile < K ? t * kSumTile : K;
            return cum_memory(c, k, tile_sum[t]) <= 0;
        });
        int64_t kB = K;
        if (t_false <= tiles) {
            const int64_t t0 = t_false - 1;                              // boundary t0 holds, t0 + 1 does not
            const int64_t first = t0 * kSumTile;
            constexpr int kPer = kSumTile / kWave;                       // consecutive rows per lane: a piece
            static_assert(kPer == kWave, "a piece has a row for every lane");
            auto wave_inclusive = [&](uint64_t v) {
                for (int off = 1; off < kWave; off <<= 1) {
                    const uint64_t up = __shfl_up(v, off);
                    if (lane >= off) v += up;
                }
                return v;
            };
            uint64_t mine = 0;
            uint32_t v[kPer];
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int64_t i = first + (int64_t)lane * kPer + q;
                v[q] = ~pairs[i < K ? i : K - 1][0];
            }
#pragma unroll
            for (int q = 0; q < kPer; ++q) mine += first + (int64_t)lane * kPer + q < K ? v[q] : 0u;
            const uint64_t upto = tile_sum[t0] + wave_inclusive(mine);
            const int64_t piece_end = first + (int64_t)(lane + 1) * kPer;
            const int whole = __popcll(ballot(cum_memory(c, piece_end < K ? piece_end : K, upto) <= 0));   // < 64
            const uint64_t before = whole == 0 ? tile_sum[t0] : __shfl(upto, whole - 1);
            const int64_t i = first + (int64_t)whole * kPer + lane;
            const uint64_t run = before + wave_inclusive(i < K ? (uint32_t)~pairs[i][0] : 0u);
            kB = first + (int64_t)whole * kPer + __popcll(ballot(i < K && cum_memory(c, i + 1, run) <= 0));
        }
        if (lane == 0) found[3] = kB;
    }
    __syncthreads();
    const int64_t kA = found[0], kC = found[1], kF = found[2], kB = found[3];

    const int64_t gran = c.granule;
    __shared__ uint64_t wave_part[kWavesPerBlock];
    const int64_t n_dp = (c.tiers == 2 ? kB : kA) / gran * gran;
    int64_t n_flex = 0;
    const uint64_t sum_dp = prefix_count(pairs, tile_sum, n_dp, wave_part);
    if (c.tiers != 2) {
        const i128 saved = -cum_memory(c, n_dp, sum_dp);                 // >= 0
        int64_t room = K - n_dp;
        if (kF - n_dp < room) room = kF > n_dp ? kF - n_dp : 0;
        int64_t lo = 0, hi = room;                                       // most rows j with j * flex_cost <= saved
        if (c.flex_cost > 0) {
            while (lo < hi) {
                const int64_t mid = lo + (hi - lo + 1) / 2;
                if ((i128)mid * (i128)c.flex_cost <= saved) lo = mid; else hi = mid - 1;
            }
        } else {
            lo = room;
        }
        n_flex = lo / gran * gran;
    }
    const uint64_t sum_both = n_flex == 0 ? sum_dp : prefix_count(pairs, tile_sum, n_dp + n_flex, wave_part);      // block-uniform
    if (threadIdx.x == 0) {
        cuts[0] = K; cuts[1] = kA; cuts[2] = kB; cuts[3] = kC; cuts[4] = kF;
        cuts[5] = n_dp; cuts[6] = n_flex;
        cuts[7] = (int64_t)tile_sum[tiles]; cuts[8] = (int64_t)sum_dp; cuts[9] = (int64_t)(sum_both - sum_dp);
    }
}

__global__ __launch_bounds__(kBlock) void tiers_emit_kernel(
    const SortPair* __restrict__ pairs_a, const SortPair* __restrict__ pairs_b, const uint32_t* __restrict__ count_bits, int first_bits,
    const int64_t* __restrict__ cuts, int64_t cap, int W,
    int64_t* __restrict__ sorted_rows, uint32_t* __restrict__ placement)
{
    const SortPair* pairs = sort_result_in_b(*count_bits, first_bits) ? pairs_b : pairs_a;
    const int64_t n_dp = cuts[5];
    const int64_t n_both = n_dp + cuts[6];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    // four rows to a thread in flight: each is a load of the row and, for a replicated one, a load of its entry
    constexpr int kAhead = 4;
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < n_both; i0 += kAhead * stride) {
        uint32_t g[kAhead], tag[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) g[q] = i0 + q * stride < n_both ? pairs[i0 + q * stride][1] : 0u;
        if (placement != nullptr) {
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                const int64_t i = i0 + q * stride;
                tag[q] = i < n_dp ? placement[g[q]] & FS_OWNER_MASK : (1u << FS_TIER_SHIFT) | ((uint32_t)(i - n_dp) % (uint32_t)W);
            }
        }
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const int64_t i = i0 + q * stride;
            if (i >= n_both) break;
            if (i < cap) sorted_rows[i] = (int64_t)g[q];
            if (placement != nullptr) placement[g[q]] = tag[q];
        }
    }
}

}  // namespace fs

extern "C" fs_status fs_plan_replication(
    const int64_t* ids, const int64_t* offsets, int32_t T, int32_t B,
    const int64_t* row_base, int64_t n, int64_t R,
    uint32_t* counts, int32_t flags,
    int64_t budget_bytes, int64_t bytes_per_row,
    int64_t* sel_rows, int64_t* num_selected,
    uint32_t* placement,
    void* workspace, size_t* workspace_bytes, void* stream, int32_t* dev_status)
{
    using namespace fs;
    if (!workspace_bytes) return FS_ERR_NULL;
    if (flags & ~(FS_PLAN_ACCUMULATE | FS_PLAN_SELECT | FS_PLAN_TAG | FS_PLAN_ALLOW_ZERO)) return FS_ERR_CONFIG;
    if ((flags & FS_PLAN_TAG) && !(flags & FS_PLAN_SELECT)) return FS_ERR_CONFIG;
    if (R < 1 || R >= 4294967295LL) return FS_ERR_SIZE;
    const bool acc = flags & FS_PLAN_ACCUMULATE;
    const bool sel = flags & FS_PLAN_SELECT;
    if (acc && (n < 0 || n >= (1LL << 31) || T < 1 || B < 1 || (int64_t)T * B >= (1LL << 31))) return FS_ERR_SIZE;
    if (sel && (budget_bytes < 0 || bytes_per_row < 1)) return FS_ERR_SIZE;

    Carver ws(workspace);
    int32_t* verdicts = ws.take<int32_t>(kCheckBlocksMax);
    const PlanScratch p = take_plan_scratch(ws, sel ? R : 0);
    if (!workspace) { *workspace_bytes = ws.used; return FS_OK; }
    if (*workspace_bytes < ws.used || (reinterpret_cast<uintptr_t>(workspace) & 255)) return FS_ERR_WORKSPACE;
    if (!counts) return FS_ERR_NULL;
    if (acc && (!offsets || !row_base || (n > 0 && !ids))) return FS_ERR_NULL;
    if (acc && ((reinterpret_cast<uintptr_t>(ids) & 7) || (reinterpret_cast<uintptr_t>(counts) & 3))) return FS_ERR_ALIGN;   // natural alignment: ids are read two at a time
    if (sel && !num_selected) return FS_ERR_NULL;
    if ((flags & FS_PLAN_TAG) && !placement) return FS_ERR_NULL;
    const int64_t cap = sel ? budget_bytes / bytes_per_row : 0;
    if (sel && cap > 0 && !sel_rows) return FS_ERR_NULL;

    hipStream_t s = static_cast<hipStream_t>(stream);
    if (acc) {
        const int64_t S = (int64_t)T * B;
        const int64_t span = hist_span(n);
        const int64_t blocks = (n + span - 1) / span;
#define FS_HISTOGRAM(SELF, BITS, VERDICTS)                                                                           \
    FS_LAUNCH("plan_histogram", (plan_histogram_kernel<SELF, BITS>), dim3((unsigned)blocks), dim3(kHistBlock), s,     \
              ids, offsets, (int)T, (int64_t)B, row_base, n, R, span, counts, verdicts, VERDICTS, dev_status)
        const bool small = span <= (1 << (kHistSmallSlotBits - 1));
        if (n > 0 && S <= kCheckSelfSegments && blocks <= kCheckSelfBlocks) {
            if (small) FS_HISTOGRAM(true, kHistSmallSlotBits, 0);
            else FS_HISTOGRAM(true, kHistSlotBits, 0);
        } else {
            const int64_t wanted = (S + kBlock * kCheckPerThread - 1) / (kBlock * kCheckPerThread);
            const int grid = (int)(wanted < kCheckBlocksMax ? wanted : kCheckBlocksMax);
            FS_LAUNCH("plan_check_offsets", plan_check_offsets_kernel, dim3((unsigned)grid), dim3(kBlock), s,
                      offsets, S, n, verdicts, dev_status);
            if (n > 0) {
                if (small) FS_HISTOGRAM(false, kHistSmallSlotBits, grid);
                else FS_HISTOGRAM(false, kHistSlotBits, grid);
            }
        }
#undef FS_HISTOGRAM
    }
    if (sel) {
        const int allow_zero = (flags & FS_PLAN_ALLOW_ZERO) ? 1 : 0;
        if (fs_status rc = sort_candidates(counts, R, allow_zero, p, s); rc != FS_OK) return rc;
        FS_LAUNCH("plan_emit", plan_emit_kernel, dim3(1024), dim3(kBlock), s,
                  p.pairs_a, p.pairs_b, p.count_bits, p.first_bits, p.num_cand, cap, sel_rows, num_selected, (flags & FS_PLAN_TAG) ? placement : nullptr);
    }
    return FS_OK;
}

extern "C" fs_status fs_plan_tiers(
    const uint32_t* counts, int64_t R, const fs_tier_params* params, int32_t tiers,
    int64_t* sorted_rows, int64_t cap, int64_t* cuts, uint32_t* placement,
    void* workspace, size_t* workspace_bytes, void* stream, int32_t* dev_status)
{
    using namespace fs;
    (void)dev_status;
    if (!workspace_bytes || !params) return FS_ERR_NULL;
    if (R < 1 || R >= 4294967295LL || cap < 0) return FS_ERR_SIZE;
    if (tiers != 2 && tiers != 3) return FS_ERR_CONFIG;
    const fs_tier_params& p = *params;
    if (p.num_samples < 1 || p.num_samples >= (1LL << 40) || p.B < 1 || p.B >= (1LL << 31)) return FS_ERR_CONFIG;
    if (p.U < 1 || p.U > FS_MAX_BUCKETS || p.W < 1 || p.U % p.W != 0) return FS_ERR_CONFIG;
    if (p.dp_multiplier < 1 || p.dp_multiplier > 1024 || p.granule < 1 || p.granule > (1 << 20)) return FS_ERR_CONFIG;
    const int64_t bw_max = 1LL << 20;
    if (p.a2a_global < 1 || p.a2a_global >= bw_max || p.a2a_intra < 1 || p.a2a_intra >= bw_max ||
        p.ar_global < 1 || p.ar_global >= bw_max || p.ar_cross < 1 || p.ar_cross >= bw_max)
        return FS_ERR_CONFIG;

    const int64_t sum_tiles = (R + kSumTile - 1) / kSumTile;
    Carver ws(workspace);
    uint64_t* tile_sum = ws.take<uint64_t>((size_t)sum_tiles + 1);
    const PlanScratch q = take_plan_scratch(ws, R);
    if (!workspace) { *workspace_bytes = ws.used; return FS_OK; }
    if (*workspace_bytes < ws.used || (reinterpret_cast<uintptr_t>(workspace) & 255)) return FS_ERR_WORKSPACE;
    if (!counts || !cuts) return FS_ERR_NULL;
    if (cap > 0 && !sorted_rows) return FS_ERR_NULL;

    // Breakpoints as thresholds on the count, exact: the smallest count c with
    //   A:    U B c >= (dp U - 1) S                      (DP memory term <= 0)
    //   C:    2 B ar_global c >= a2a_global S            (DP traffic term <= 0)
    //   FLEX: 2 B (a2a_intra - a2a_global) W ar_cross c >= S a2a_global a2a_intra
    auto ceil_div = [](u128 num, u128 den) -> uint64_t {
        const u128 q = (num + den - 1) / den;
        return q > (u128)1 << 62 ? (uint64_t)1 << 62 : (uint64_t)q;
    };
    TierConsts c;
    c.static_term = ((int64_t)p.dp_multiplier * p.U - 1) * p.num_samples;
    c.dyn_factor = (int64_t)p.U * p.B;
    c.flex_cost = ((int64_t)p.dp_multiplier * (p.U / p.W) - 1) * p.num_samples;
    c.granule = p.granule;
    c.W = p.W;
    c.tiers = tiers;
    c.thr_a = ceil_div((u128)c.static_term, (u128)c.dyn_factor);
    c.thr_c = ceil_div((u128)p.a2a_global * (u128)p.num_samples, (u128)2 * p.B * p.ar_global);
    c.thr_f = p.a2a_intra > p.a2a_global
                  ? ceil_div((u128)p.num_samples * p.a2a_global * p.a2a_intra,
                             (u128)2 * p.B * (p.a2a_intra - p.a2a_global) * p.W * p.ar_cross)
                  : (uint64_t)1 << 62;

    hipStream_t s = static_cast<hipStream_t>(stream);
    if (fs_status rc = sort_candidates(counts, R, 0, q, s); rc != FS_OK) return rc;
    const unsigned sum_grid = sum_tiles < 2048 ? (unsigned)sum_tiles : 2048u;        // 8 blocks per CU
    FS_LAUNCH("tiers_tile_sums", tiers_tile_sums_kernel, dim3(sum_grid), dim3(kBlock), s,
              q.pairs_a, q.pairs_b, q.count_bits, q.first_bits, q.num_cand, tile_sum);
    FS_LAUNCH("tiers_scan_sums", tiers_scan_sums_kernel, dim3(1), dim3(kScanBlock), s, tile_sum, q.num_cand);
    FS_LAUNCH("tiers_cuts", tiers_cuts_kernel, dim3(1), dim3(kBlock), s, q.pairs_a, q.pairs_b, q.count_bits, q.first_bits, q.num_cand,
              tile_sum, c, cuts);
    FS_LAUNCH("tiers_emit", tiers_emit_kernel, dim3(1024), dim3(kBlock), s, q.pairs_a, q.pairs_b, q.count_bits, q.first_bits, cuts, cap, (int)p.W,
              sorted_rows, placement);
    return FS_OK;
}
