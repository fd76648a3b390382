// Stable LSD radix sort of (key, value) pairs, up to 10 bits per pass (27-bit row ids: 3 passes).
//
// Per pass, three launches over tiles of 4096 pairs (sorts of few pairs take smaller tiles and may do without the
// second, see sort_shape):
//   sort_count    digit histogram of every tile.  A block takes a group of consecutive tiles, so that there are at most
//                 1024 groups: its histogram runs on over them, what stands in it before a tile is the tile's prefix
//                 inside the group, what stands in it at the end the group's row of sums
//   sort_scan     exclusive scan of every digit's sums over the groups, and the digits' totals
//   sort_scatter  each wave ranks its consecutive pairs against a wave-private running histogram in LDS (ballot
//                 matching keeps equal digits in order); the tile is put in digit order in LDS, then written out so
//                 that consecutive lanes write consecutive addresses of one digit's run
// Stability comes from wave -> tile -> digit prefix order; no block ever waits for another.
// The first pass can read (int64 row, int32 position) directly, validating them on the way.  Between passes key and
// value lie side by side (apart in very large sorts); the last pass can write them apart.
#include "radix_sort.h"

namespace fs {

constexpr int kSortMaxBins = 1 << kSortMaxDigitBits;
constexpr int kLargeBlock = 512, kLargeItems = 8;

__device__ __forceinline__ int64_t sort_count_of(const int64_t* m_dev, int64_t m_max)
{
    if (m_dev == nullptr) return m_max;
    const int64_t m = *m_dev;
    return m < 0 ? 0 : (m < m_max ? m : m_max);
}

struct PairReader {                           // pairs of an earlier pass
    const SortPair* pairs;
    __device__ __forceinline__ PairReader from(int64_t base) const { return {pairs + base}; }
    __device__ __forceinline__ uint32_t key(uint32_t i) const { return pairs[i][0]; }
    __device__ __forceinline__ void pair(uint32_t i, uint32_t* k, uint32_t* v, int32_t*) const
    {
        const SortPair p = pairs[i];
        *k = p[0];
        *v = p[1];
    }
};

struct SplitReader {                          // keys and values of an earlier pass, apart
    const uint32_t* keys;
    const uint32_t* vals;
    __device__ __forceinline__ SplitReader from(int64_t base) const { return {keys + base, vals + base}; }
    __device__ __forceinline__ uint32_t key(uint32_t i) const { return keys[i]; }
    __device__ __forceinline__ void pair(uint32_t i, uint32_t* k, uint32_t* v, int32_t*) const
    {
        *k = keys[i];
        *v = vals[i];
    }
};

struct RowPosReader {                         // pairs are (rows[i], pos[i]), validated
    const int64_t* rows;
    const int32_t* pos;
    int64_t R;
    int64_t n;
    __device__ __forceinline__ RowPosReader from(int64_t base) const { return {rows + base, pos + base, R, n}; }
    // one unsigned compare each also catches the negative values (R < 2^32, n < 2^31)
    __device__ __forceinline__ uint32_t key(uint32_t i) const
    {
        const uint64_t r = (uint64_t)load_stream(rows + i);
        return r >= (uint64_t)R ? 0u : (uint32_t)r;
    }
    __device__ __forceinline__ void pair(uint32_t i, uint32_t* k, uint32_t* v, int32_t* faults) const
    {
        uint64_t r = (uint64_t)load_stream(rows + i);
        uint32_t p = (uint32_t)load_stream(pos + i);
        if (r >= (uint64_t)R) { r = 0; *faults |= FS_DEV_BAD_ID; }
        if (p >= (uint32_t)n) { p = 0; *faults |= FS_DEV_BAD_ID; }
        *k = (uint32_t)r;
        *v = p;
    }
};

// A pass whose digit is the same in all keys would copy the pairs: every kernel of it returns at once.  `varying`
// (or null) has, at least, every bit set in which two keys differ.  The first pass always runs (it moves the pairs
// out of their source).
__device__ __forceinline__ bool sort_pass_idle(const uint32_t* varying, int shift)
{
    return varying != nullptr && shift > 0 && (*varying >> shift) == 0;
}

// What the kernels of a pass are given, as one argument: the runtime spends 0.5 us more on a launch of 16.
struct SortArgs {
    int64_t m_max;
    const int64_t* m_dev;
    const uint32_t* varying;
    uint32_t* tile_hist;             // [tiles][bins], if a group has several
    uint32_t* group_sums;            // [groups][bins], rows of kSortMaxBins without a scan; the scan's prefixes after it
    uint32_t* later_sums;            // without a scan: the later passes' tables, [passes][tiles][kSortMaxBins]; else null
    int64_t later_tiles;
    const uint32_t* totals;
    SortPair* pairs_out;             // or null
    uint32_t* keys_out;
    uint32_t* vals_out;
    int32_t* status;
    int shift, later, next_bits;     // later: passes after this one; the next one's digit
};

// The tiles are dealt to at most this many groups, consecutive ones to a group.
constexpr int kSortMaxGroups = 1024;

__host__ __device__ __forceinline__ int64_t sort_group_tiles(int64_t used) { return (used + kSortMaxGroups - 1) / kSortMaxGroups; }

// Plain LDS adds, with two guards against popular digits: a wave's keys that share the digit of its first one, a popular
// row's, go with one add, and the histogram has four copies, a lane's by its number, so that where a second digit is
// popular its adds meet in four words instead of in one.  15.7 M keys of 9 bits, all different / in row order after one
// pass / two digits in turn: adds alone 16, 49, 53 us, the first digit apart 12, 15, 31, four copies alone 12, 16, 17, one add
// per distinct digit by ballot matching 28 whatever they are: with these guards memory is what bounds it (5 TB/s).  Small
// tiles: the adds alone, the rest costs more than it saves.
template <typename Reader, int NBITS, int BLOCK, int ITEMS>
__global__ __launch_bounds__(BLOCK) void sort_count_kernel(const Reader in, const SortArgs a)
{
    const int shift = a.shift;
    constexpr int bins = 1 << NBITS;
    constexpr int kTile = BLOCK * ITEMS;
    constexpr int kCopies = ITEMS > 4 ? 4 : 1;         // small tiles: clearing and adding up four cost more than they save
    typedef uint32_t Copies __attribute__((ext_vector_type(kCopies)));
    __shared__ __attribute__((aligned(16))) uint32_t hist[bins * kCopies];
    if (sort_pass_idle(a.varying, shift)) return;
    const int64_t m = sort_count_of(a.m_dev, a.m_max);
    const int64_t used = (m + kTile - 1) / kTile;      // tiles that hold pairs (m may live on the device)
    const int64_t per = sort_group_tiles(used);
    const int64_t t0 = (int64_t)blockIdx.x * per;
    if (t0 >= used) return;                            // block-uniform
    const int64_t t1 = t0 + per < used ? t0 + per : used;
    constexpr uint32_t mask = (uint32_t)bins - 1u;
    uint32_t key[ITEMS];
    auto load = [&](int64_t tile) {
        const int64_t base = tile * kTile;
        const uint32_t left = (uint32_t)(m - base < kTile ? m - base : kTile);
        const Reader r = in.from(base);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const uint32_t i = it * BLOCK + threadIdx.x;
            key[it] = r.key(i < left ? i : left - 1u);           // past the end: the last one again, not counted
        }
    };
    load(t0);
    for (int b = threadIdx.x; b < bins * kCopies; b += BLOCK) hist[b] = 0;
    __syncthreads();
    auto copies_sum = [&](int b) {
        const Copies v = reinterpret_cast<const Copies*>(hist)[b];
        uint32_t sum = 0;
#pragma unroll
        for (int c = 0; c < kCopies; ++c) sum += v[c];
        return sum;
    };
    for (int64_t t = t0; t < t1; ++t) {
        uint32_t digit[ITEMS];
        const uint32_t left = (uint32_t)(m - t * kTile < kTile ? m - t * kTile : kTile);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) digit[it] = (key[it] >> shift) & mask;
        if (t + 1 < t1) load(t + 1);
        if (per > 1) {                                           // block-uniform
            for (int b = threadIdx.x; b < bins; b += BLOCK) a.tile_hist[t * bins + b] = copies_sum(b);
            __syncthreads();
        }
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const bool valid = it * BLOCK + threadIdx.x < left;
            if constexpr (kCopies == 1) {
                if (valid) atomicAdd(&hist[digit[it]], 1u);
                continue;
            }
            const bool same = valid && digit[it] == (uint32_t)__builtin_amdgcn_readfirstlane((int)digit[it]);
            const uint64_t all = ballot(same);
            const bool leads = same && popc_below(all) == 0;
            if (valid && (!same || leads))
                atomicAdd(&hist[digit[it] * kCopies + threadIdx.x % kCopies], leads ? (uint32_t)__popcll(all) : 1u);
        }
        __syncthreads();
    }
    const int64_t stride = a.later_sums != nullptr ? kSortMaxBins : bins;
    for (int b = threadIdx.x; b < bins; b += BLOCK) a.group_sums[(int64_t)blockIdx.x * stride + b] = copies_sum(b);
    if (a.later_sums == nullptr) return;
    // the later passes' counts of this tile, which the scatters add to, start at zero
    for (int k = 0; k < a.later; ++k) {
        u32x4* row = reinterpret_cast<u32x4*>(a.later_sums + ((int64_t)k * a.later_tiles + blockIdx.x) * kSortMaxBins);
        for (int q = threadIdx.x; q < kSortMaxBins / 4; q += BLOCK) row[q] = u32x4{0u, 0u, 0u, 0u};
    }
}

// group_sums[group][digit] -> exclusive prefix over the groups, in place, and totals[digit].  A block takes 32 digits, its
// 32 rows of threads a slice of the groups each, with all their loads in flight at once: one round of memory latency
// whatever the number of groups.
constexpr int kScanBins = 32;
constexpr int kScanSlices = 32;
static_assert(kScanSlices * 32 == kSortMaxGroups, "at most 32 groups to a thread");

__global__ __launch_bounds__(kScanBins * kScanSlices) void sort_scan_kernel(
    uint32_t* __restrict__ group_sums, int bins, int tile_pairs, int64_t m_max, const int64_t* __restrict__ m_dev,
    const uint32_t* __restrict__ varying, int shift, uint32_t* __restrict__ totals)
{
    __shared__ uint32_t part[kScanSlices][kScanBins];
    if (sort_pass_idle(varying, shift)) return;
    const int64_t m = sort_count_of(m_dev, m_max);
    const int64_t used = (m + tile_pairs - 1) / tile_pairs;
    if (used == 0) return;
    const int64_t per_group = sort_group_tiles(used);
    const int groups = (int)((used + per_group - 1) / per_group);
    const int per = (groups + kScanSlices - 1) / kScanSlices;
    const int slice = threadIdx.x / kScanBins;
    const int b = blockIdx.x * kScanBins + threadIdx.x % kScanBins;
    const int bc = b < bins ? b : bins - 1;
    const int lo = slice * per;
    auto scan = [&](auto most) {                                 // per <= most
        constexpr int kMost = decltype(most)::value;
        uint32_t v[kMost];
        uint32_t sum = 0;
#pragma unroll
        for (int q = 0; q < kMost; ++q) {
            const int g = lo + q < groups ? lo + q : groups - 1;
            v[q] = group_sums[(int64_t)g * bins + bc];
        }
#pragma unroll
        for (int q = 0; q < kMost; ++q) {
            if (q >= per || lo + q >= groups) v[q] = 0;
            sum += v[q];
        }
        part[slice][threadIdx.x % kScanBins] = sum;
        __syncthreads();
        uint32_t run = 0;
#pragma unroll
        for (int s = 0; s < kScanSlices; ++s) {
            const uint32_t p = part[s][threadIdx.x % kScanBins];
            run += s < slice ? p : 0u;
        }
        if (b < bins) {
            if (slice == kScanSlices - 1) totals[b] = run + sum;
#pragma unroll
            for (int q = 0; q < kMost; ++q) {
                if (q < per && lo + q < groups) group_sums[(int64_t)(lo + q) * bins + b] = run;
                run += v[q];
            }
        }
    };
    if (per <= 4) scan(std::integral_constant<int, 4>());        // block-uniform
    else if (per <= 12) scan(std::integral_constant<int, 12>());
    else scan(std::integral_constant<int, 32>());
}

// SUM: few groups (of one tile each); no scan has run, group_sums holds plain counts, and every block adds up the
// digits' totals and what stands before its tile itself, one vector load per group and thread, 16 in flight, while its
// pairs are on the way.  It also counts the next pass's digits, by the tile that its pairs go to, with an add to memory for
// every stretch of neighbours with one counter: only the first pass has a count launch.
template <typename Reader, int NBITS, int BLOCK, int ITEMS, int STRIPE, bool SUM>
__global__ __launch_bounds__(BLOCK) void sort_scatter_kernel(const Reader in, const SortArgs a)
{
    const int shift = a.shift;
    const uint32_t* const group_sums = a.group_sums;             // scanned, unless SUM
    constexpr int bins = 1 << NBITS;
    constexpr int kTile = BLOCK * ITEMS;
    constexpr int kWaves = BLOCK / kWave;
    constexpr int kWaveSpan = kWave * ITEMS;
    constexpr int kBinsPerThread = (bins + BLOCK - 1) / BLOCK;
    __shared__ uint32_t out_base[bins];                         // global index of the tile's first pair of a digit,
                                                                // minus the digit's first index inside the tile
    __shared__ uint16_t wave_hist[kWaves][bins];
    __shared__ SortPair s_pair[kTile];
    __shared__ uint32_t wave_sums[16];
    if (sort_pass_idle(a.varying, shift)) return;
    const int64_t m = sort_count_of(a.m_dev, a.m_max);
    const int64_t used = (m + kTile - 1) / kTile;
    const int64_t per_group = sort_group_tiles(used);
    constexpr uint32_t mask = (uint32_t)bins - 1u;
    const int w = wave_id();
    const int lane = lane_id();
    int32_t faults = 0;

    // Tiles in stripes per XCD (the grid is a multiple of 8, so a block stays on its XCD over the
    // grid stride): consecutive tiles write neighbouring runs of every digit's region, a few tens of
    // bytes each, and one XCD's L2 then merges what four XCDs would write into one 128-byte line
    // piece by piece (scatter 0.343 -> 0.327 ms per step on 15.7 M pairs).
    const int64_t padded = STRIPE == 1 ? used : xcd_striped_grid_dev(used, STRIPE);
    for (int64_t v = blockIdx.x; v < padded; v += gridDim.x) {
        const int64_t tile = STRIPE == 1 ? v : xcd_striped_tile((unsigned)v, STRIPE);
        if (tile >= used) continue;                              // block-uniform
        const int64_t base = tile * kTile;
        const uint32_t left = (uint32_t)(m - base < kTile ? m - base : kTile);
        const uint32_t first = w * kWaveSpan + lane;             // the thread's items: first + it * kWave
        uint32_t key[ITEMS];
        uint32_t val[ITEMS];
        uint32_t rank[ITEMS];
        const Reader r = in.from(base);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const uint32_t i = first + it * kWave;
            r.pair(i < left ? i : left - 1u, &key[it], &val[it], &faults);   // past the end: the last one again, not ranked
        }
        uint32_t tot[kBinsPerThread];                            // the digits' totals
        uint32_t before_tile[kBinsPerThread];                    // and their pairs in the tiles before this one
        typedef uint32_t Bins __attribute__((ext_vector_type(kBinsPerThread)));    // 1, 2 or 4: aligned (256-byte tables)
        const bool has_bins = threadIdx.x * kBinsPerThread < bins;
        const uint32_t my_bins = has_bins ? threadIdx.x : 0u;
        if constexpr (SUM) {
#pragma unroll
            for (int q = 0; q < kBinsPerThread; ++q) { tot[q] = 0; before_tile[q] = 0; }
            const Bins* mine = reinterpret_cast<const Bins*>(group_sums) + my_bins;
            constexpr int kAhead = 16;
            for (int t0 = 0; t0 < (int)used; t0 += kAhead) {
                Bins x[kAhead];
#pragma unroll
                for (int e = 0; e < kAhead; ++e) x[e] = mine[(t0 + e < (int)used ? t0 + e : (int)used - 1) * (kSortMaxBins / kBinsPerThread)];
#pragma unroll
                for (int e = 0; e < kAhead; ++e) {
#pragma unroll
                    for (int q = 0; q < kBinsPerThread; ++q) {
                        tot[q] += t0 + e < (int)used ? x[e][q] : 0u;
                        before_tile[q] += t0 + e < (int)tile ? x[e][q] : 0u;
                    }
                }
            }
        }
        for (int b = lane; b < bins; b += kWave) wave_hist[w][b] = 0;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // the zeroing above, seen by the wave's other lanes
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const bool valid = first + it * kWave < left;
            const uint32_t digit = (key[it] >> shift) & mask;
            const uint64_t same = match_bits_n<NBITS>(digit, valid);
            const uint32_t before = popc_below(same);
            const uint32_t seen = wave_hist[w][digit];
            __builtin_amdgcn_wave_barrier();
            rank[it] = seen + before;
            if (valid && before == 0) wave_hist[w][digit] = (uint16_t)(seen + __popcll(same));
            __builtin_amdgcn_wave_barrier();
        }
        if constexpr (!SUM) {
            const uint32_t group = (uint32_t)tile / (uint32_t)per_group;        // tiles < 2^31
            const Bins t = reinterpret_cast<const Bins*>(a.totals)[my_bins];
            Bins g = reinterpret_cast<const Bins*>(group_sums + (int64_t)group * bins)[my_bins];
            if (per_group > 1) g += reinterpret_cast<const Bins*>(a.tile_hist + tile * bins)[my_bins];
#pragma unroll
            for (int q = 0; q < kBinsPerThread; ++q) { tot[q] = t[q]; before_tile[q] = g[q]; }
        }
        __syncthreads();

        // per digit: waves' counts -> waves' offsets inside the digit; the tile's count of the digit
        uint32_t count[kBinsPerThread];
        uint32_t sum = 0, tsum = 0;
#pragma unroll
        for (int q = 0; q < kBinsPerThread; ++q) {
            const int b = threadIdx.x * kBinsPerThread + q;
            uint32_t run = 0;
            if (has_bins) {
#pragma unroll
                for (int k = 0; k < kWaves; ++k) {
                    const uint32_t x = wave_hist[k][b];
                    wave_hist[k][b] = (uint16_t)run;
                    run += x;
                }
            }
            count[q] = run;
            sum += run;
            tsum += has_bins ? tot[q] : 0u;
        }
        // exclusive scans over the digits: inside the tile (sum) and over the whole input (totals)
        uint32_t unused;
        uint32_t in_tile = block_exclusive_scan(sum, wave_sums, &unused);
        uint32_t in_all = block_exclusive_scan(tsum, wave_sums, &unused);
#pragma unroll
        for (int q = 0; q < kBinsPerThread; ++q) {
            const int b = threadIdx.x * kBinsPerThread + q;
            if (has_bins) {
                out_base[b] = in_all + before_tile[q] - in_tile;
#pragma unroll
                for (int k = 0; k < kWaves; ++k) wave_hist[k][b] = (uint16_t)(wave_hist[k][b] + in_tile);
            }
            in_tile += count[q];
            in_all += tot[q];
        }
        __syncthreads();
        // the tile in digit order, in LDS
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            if (first + it * kWave < left) {
                const uint32_t digit = (key[it] >> shift) & mask;
                s_pair[(uint32_t)wave_hist[w][digit] + rank[it]] = SortPair{key[it], val[it]};
            }
        }
        __syncthreads();
        if constexpr (SUM) {
            uint32_t* const next_sums = a.later != 0 ? a.later_sums : nullptr;
            if (next_sums != nullptr && !sort_pass_idle(a.varying, shift + NBITS)) {          // block-uniform
                const uint32_t next_mask = (1u << a.next_bits) - 1u;
#pragma unroll
                for (int it = 0; it < ITEMS; ++it) {
                    const uint32_t at = it * BLOCK + threadIdx.x;
                    const uint32_t k = s_pair[at < left ? at : left - 1u][0];
                    const uint32_t j = out_base[(k >> shift) & mask] + at;
                    const uint32_t counter = (j / kTile) * (uint32_t)kSortMaxBins + ((k >> (shift + NBITS)) & next_mask);
                    // a popular row's pairs stand side by side: one add for a stretch of lanes with one counter
                    const uint32_t below = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)counter, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
                    const bool starts = at < left && counter != below;               // lane 0: -1 is no counter
                    const uint64_t later_starts = ballot(starts) >> lane >> 1;
                    const uint32_t valid_lanes = (uint32_t)__popcll(ballot(at < left));
                    if (starts)
                        atomicAdd(next_sums + counter, later_starts != 0 ? (uint32_t)__builtin_ctzll(later_starts) + 1u : valid_lanes - (uint32_t)lane);
                }
            }
        }
        if (a.pairs_out != nullptr) {                              // block-uniform
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) {
                const uint32_t at = it * BLOCK + threadIdx.x;
                if (at < left) {
                    const SortPair p = s_pair[at];
                    a.pairs_out[out_base[(p[0] >> shift) & mask] + at] = p;
                }
            }
        } else {
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) {
                const uint32_t at = it * BLOCK + threadIdx.x;
                if (at < left) {
                    const SortPair p = s_pair[at];
                    const uint32_t j = out_base[(p[0] >> shift) & mask] + at;
                    a.keys_out[j] = p[0];
                    a.vals_out[j] = p[1];
                }
            }
        }
        __syncthreads();
    }
    if (ballot(faults != 0) != 0) {
        for (int off = 32; off > 0; off >>= 1) faults |= __shfl_down(faults, off);
        if (lane == 0) report(a.status, faults);
    }
}

// Large sorts: 8 waves to a tile of 4096 pairs, 8 ranking rounds each, two tiles to a CU by their registers (held to 80 of
// them, three: the L2s then merge fewer of the runs' pieces, 15.7 M pairs 279 -> 289 us, 72 M uniform ones 1469 -> 1646).  What
// bounds them is the memory's rate for a stream that reads and writes at once (a 4-bit scatter of 15.7 M pairs, nearly a copy, takes 49 us, this one
// with 9 bits 59; 4 waves of 16 rounds 62 to 72, tiles of 8192 61, 16 waves 80).  Small ones, up to 256 tiles of 1024
// pairs: a block's time is its chain of ranking rounds and of the memory's latency, and the smaller tiles have four
// rounds.  Up to 64 of them (128 where the count is on the device: the plan's candidates, usually a few per cent of the
// rows that the buffers are sized for) there is no scan launch.
// fs_sort_lookups as a whole against 4 waves of 16 rounds, keys and values apart, two scan launches and a count by
// ballots, Zipf(1.1) over 80 M rows, us: 8192 pairs 27 -> 20.5, 65 k 52 -> 31.5, 262 k 51 -> 39.5, 1 M 67 -> 52.5, 4.2 M 146 ->
// 115, 15.7 M 308 -> 280, 72 M 1391 -> 1288.
constexpr int kSmallBlock = 256, kSmallItems = 4;
constexpr int kSortStripe = 16;              // tiles per XCD stripe in the scatter
constexpr int64_t kSortSmallTiles = 256;
constexpr int64_t kSortSumTiles = 64;
constexpr int kSortMaxPasses = 4;
static_assert(kSortMaxPasses * 2 * kSortSumTiles >= kSortSmallTiles);
// Blocks of the scatter at most; they walk the tiles with a grid stride.  Where the count is on the device it is usually a
// few per cent of what the buffers hold, and a pass may be idle: fewer blocks, six rounds of the 512 that the chip holds.
constexpr int64_t kSortScatterGrid = 8192;
constexpr int64_t kSortScatterGridDev = 3072;

struct SortShape {
    bool small;
    bool sum;                                // no scan launch
    int64_t tiles;
    int tile_pairs;
};

static SortShape sort_shape(int64_t m_max, bool device_count)
{
    const int small_tile = kSmallBlock * kSmallItems;
    const int64_t small_tiles = (m_max + small_tile - 1) / small_tile;
    if (small_tiles <= kSortSmallTiles)
        return {true, small_tiles <= (device_count ? 2 : 1) * kSortSumTiles, small_tiles, small_tile};
    const int large_tile = kLargeBlock * kLargeItems;
    return {false, false, (m_max + large_tile - 1) / large_tile, large_tile};
}

struct SortTables {
    uint32_t* totals;
    uint32_t* group_sums;
    uint32_t* tile_hist;
};

static SortTables take_tables(Carver& c, int64_t m_max)
{
    const int64_t large_tile = kLargeBlock * kLargeItems;
    const int64_t tiles = (m_max + large_tile - 1) / large_tile;
    // never less than a smaller m_max asks for: a workspace sized for a caller's largest batch serves the smaller ones
    const int64_t small = (m_max + kSmallBlock * kSmallItems - 1) / (kSmallBlock * kSmallItems);
    int64_t groups = tiles < kSortMaxGroups ? tiles : kSortMaxGroups;
    const int64_t small_rows = kSortMaxPasses * (small < 2 * kSortSumTiles ? small : 2 * kSortSumTiles);     // a table for every pass
    if (groups < small_rows) groups = small_rows;
    SortTables t;
    t.totals = c.take<uint32_t>((size_t)kSortMaxBins);
    t.group_sums = c.take<uint32_t>((size_t)kSortMaxBins * (size_t)groups);
    t.tile_hist = c.take<uint32_t>(tiles > kSortMaxGroups ? (size_t)kSortMaxBins * (size_t)tiles : 0);
    return t;
}

size_t radix_sort_scratch_bytes(int64_t m_max)
{
    Carver c(nullptr);
    take_tables(c, m_max);
    return c.used;
}

struct SortPass {
    SortShape shape;
    SortTables t;
    int64_t m_max;
    const int64_t* m_dev;
    const uint32_t* varying;
    int shift;
    SortPlace to;
    int number, passes;                      // this pass's number
    int next_bits;                           // the next one's digit, if there is one
    int32_t* status;
    hipStream_t stream;
};

template <int NBITS, typename Reader>
static fs_status launch_sort_pass(const Reader& in, const SortPass& p)
{
    constexpr int bins = 1 << NBITS;
    const int64_t groups = p.shape.tiles < kSortMaxGroups ? p.shape.tiles : kSortMaxGroups;
    // without a scan every pass has a table of its own
    const int64_t table = p.shape.tiles * kSortMaxBins;
    SortArgs a;
    a.m_max = p.m_max; a.m_dev = p.m_dev; a.varying = p.varying;
    a.tile_hist = p.t.tile_hist;
    a.group_sums = p.shape.sum ? p.t.group_sums + p.number * table : p.t.group_sums;
    a.later_sums = p.shape.sum ? a.group_sums + table : nullptr;
    a.later_tiles = p.shape.tiles;
    a.totals = p.t.totals;
    a.pairs_out = p.to.pairs; a.keys_out = p.to.keys; a.vals_out = p.to.vals; a.status = p.status;
    a.shift = p.shift; a.later = p.passes - 1 - p.number; a.next_bits = p.next_bits;
#define FS_COUNT(BLOCK, ITEMS)                                                                                        \
    FS_LAUNCH("sort_count", (sort_count_kernel<Reader, NBITS, BLOCK, ITEMS>), dim3((unsigned)groups), dim3(BLOCK), p.stream, in, a)
#define FS_SCATTER(BLOCK, ITEMS, STRIPE, SUM, GRID)                                                                   \
    FS_LAUNCH("sort_scatter", (sort_scatter_kernel<Reader, NBITS, BLOCK, ITEMS, STRIPE, SUM>), dim3((unsigned)(GRID)), dim3(BLOCK), \
              p.stream, in, a)
    if (p.shape.small && (p.number == 0 || !p.shape.sum)) FS_COUNT(kSmallBlock, kSmallItems);
    if (!p.shape.small) FS_COUNT(kLargeBlock, kLargeItems);
    if (!p.shape.sum)
        FS_LAUNCH("sort_scan", sort_scan_kernel, dim3((bins + kScanBins - 1) / kScanBins), dim3(kScanBins * kScanSlices), p.stream,
                  p.t.group_sums, bins, p.shape.tile_pairs, p.m_max, p.m_dev, p.varying, p.shift, p.t.totals);
    if (p.shape.small && p.shape.sum) FS_SCATTER(kSmallBlock, kSmallItems, 1, true, p.shape.tiles);
    if (p.shape.small && !p.shape.sum) FS_SCATTER(kSmallBlock, kSmallItems, 1, false, p.shape.tiles);
    if (!p.shape.small) {
        const int64_t padded = xcd_striped_grid(p.shape.tiles, kSortStripe);       // a multiple of 8, as the largest grid is
        const int64_t most = p.m_dev != nullptr ? kSortScatterGridDev : kSortScatterGrid;
        FS_SCATTER(kLargeBlock, kLargeItems, kSortStripe, false, padded < most ? padded : most);
    }
#undef FS_COUNT
#undef FS_SCATTER
    return FS_OK;
}

fs_status radix_sort(const SortJob& job)
{
    if (job.m_max <= 0) return FS_OK;
    const int least = job.rows != nullptr ? 1 : kSortPairsBits;
    const int key_bits = job.key_bits < least ? least : job.key_bits > 32 ? 32 : job.key_bits;
    SortPass p;
    p.shape = sort_shape(job.m_max, job.m_dev != nullptr);
    if (p.shape.tiles > 0x7FFFFFFF) return FS_ERR_SIZE;
    Carver c(job.scratch);
    p.t = take_tables(c, job.m_max);
    p.m_max = job.m_max; p.m_dev = job.m_dev; p.varying = job.varying; p.stream = job.stream;
    p.shift = 0;
    const int passes = job.varying == nullptr ? radix_sort_passes(key_bits) : 4;          // with `varying`: 32 bits
    p.passes = passes;
    for (int k = 0; k < passes; ++k) {
        const int nbits = sort_digit_bits(job, key_bits, passes, k, p.shift);
        p.number = k;
        p.next_bits = k + 1 < passes ? sort_digit_bits(job, key_bits, passes, k + 1, p.shift + nbits) : 0;
        const SortPlace from = sort_place_after(job, passes, k - 1);
        p.to = sort_place_after(job, passes, k);
        fs_status rc = FS_OK;
        if (k == 0 && job.rows != nullptr) {
            const RowPosReader in{job.rows, job.pos, job.R, job.n};
            p.status = job.status;
#define FS_SORT_ROWS(NB) rc = launch_sort_pass<NB>(in, p)
            FS_DISPATCH_BITS(nbits, FS_SORT_ROWS)
#undef FS_SORT_ROWS
        } else if (from.pairs == nullptr) {
            const SplitReader in{from.keys, from.vals};
            p.status = nullptr;
#define FS_SORT_SPLIT(NB) rc = launch_sort_pass<NB>(in, p)
            FS_DISPATCH_BITS_FROM_5(nbits, FS_SORT_SPLIT)
#undef FS_SORT_SPLIT
        } else {
            const PairReader in{from.pairs};
            p.status = nullptr;
#define FS_SORT_PAIRS(NB) rc = launch_sort_pass<NB>(in, p)
            FS_DISPATCH_BITS_FROM_5(nbits, FS_SORT_PAIRS)
#undef FS_SORT_PAIRS
        }
        if (rc != FS_OK) return rc;
        p.shift += nbits;
    }
    return FS_OK;
}

}  // namespace fs
