// fs_seq_grad_bwd: row_grads[u(r), :] = sum of f32(grad_out[pos[j], :]) over the lookups of row r.
//
// Sort-by-row segmented reduction:
//   radix sort        stable by row, the first pass reading and validating (row, pos) itself; lookups of one row keep their j order, which is
//                     ascending pos for any fs_route_bucketize output
//   bwd_count_heads   per 256-lookup chunk of the sorted order: number of runs that
//                     start in it, with a block-local exclusive prefix
//   bwd_scan_blocks   exclusive scan of the per-block sums -> index of every run,
//                     *num_unique (few blocks: no launch, every wave adds up their sums itself)
//   bwd_segreduce     a wave walks one chunk left to right, the rows' addresses in scalar registers and
//                     8 rows in flight; a run that starts in the chunk goes to row_grads, the piece that
//                     continues a run from the previous chunk goes to carry[chunk]
//   bwd_singletons    runs of one lookup (most runs: the cold tail) are skipped by the walk and
//                     converted here, fully parallel
//   bwd_chunk_sums    in place of these two for few chunks: a block brings one chunk's rows to LDS, every
//                     load in flight at once, and sums the run pieces out of LDS side by side
//   bwd_fold          for every run that spills over a chunk end: row_grads += carry of
//                     the following chunks, left to right
// which is exactly the summation order stated in flexshard.h (chunk = FS_BWD_TILE).
// variant 1 replaces carry + fold by fp32 atomic adds into pre-zeroed rows.
// HBM-bound: grad_out is read once (random 16*units-byte rows), row_grads written once.
// (fs_seq_grad_bwd's variant 1 still reads and writes row_grads with atomics in L2.)
#include "fs_common.h"
#include "radix_sort.h"
#include "run_end.h"
#include "update_rules.h"

namespace fs {

constexpr int kChunk = FS_BWD_TILE;
constexpr int kChunksPerBlock = 64;          // bwd_count_heads: chunks per block
constexpr int kSinglesSplit = 4;             // bwd_singletons: waves per chunk (divides kChunk / 64)
constexpr int kWalkAhead = 8;                // rows per batch of a walking wave, the next batch in flight beside it

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

// Block b covers chunks [64 b, 64 b + 64): 16 waves, each walks 4 of them (with 4 waves of 16 chunks
// each the kernel's time was the chain of 16 dependent rounds of loads per wave).  chunk_local[c] = runs
// that start in the block's chunks before c; block_sum[b] = runs that start in the block.  A wave's 16 rounds of
// loads are all issued at once, two each (with four, a round at a time: 8192 lookups 9.9 us, now 4.6 with the scan over
// the blocks inside; 4.2 M 18, now 11).
constexpr int kHeadsBlock = 1024;

// `v` of the lane below; lane 0 gets `first`.
__device__ __forceinline__ uint32_t from_lane_below(uint32_t v, uint32_t first)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
}

// `v` of the lane above; lane 63 gets `last`.
__device__ __forceinline__ uint32_t from_lane_above(uint32_t v, uint32_t last)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)v, 0x130 /* wave_shl:1 */, 0xf, 0xf, false);
}

// TOTAL: one block is all there is, and it writes the number of runs.
template <bool TOTAL>
__global__ __launch_bounds__(kHeadsBlock) void bwd_count_heads_kernel(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, int64_t m, int64_t chunks,
    uint32_t n, uint32_t R,
    uint32_t* __restrict__ chunk_local, uint32_t* __restrict__ block_sum, int64_t cap,
    int64_t* __restrict__ num_unique, uint32_t* __restrict__ num_long /* or null */, int32_t* status)
{
    __shared__ uint32_t heads[kChunksPerBlock];
    const int w = wave_id();
    const int lane = lane_id();
    if (num_long != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *num_long = 0;       // bwd_fold counts here
    constexpr int kPerWave = kChunksPerBlock / (kHeadsBlock / kWave);
    bool disorder = false, bad = false, unsorted = false;
    // The wave's chunks follow one another, so its rounds of 64 lookups do: all rounds are loaded before the first is
    // looked at, and a lookup's predecessor is the lane's below (for lane 0 the previous round's last).
    constexpr int kPerChunk = kChunk / kWave;
    constexpr int kRounds = kPerWave * kPerChunk;
    const int64_t wave_first = ((int64_t)blockIdx.x * kChunksPerBlock + w * kPerWave) * kChunk;
    uint32_t key[kRounds], val[kRounds];
    uint32_t last_key = 0, last_val = 0;
    if (wave_first > 0 && wave_first < m) { last_key = keys[wave_first - 1]; last_val = vals[wave_first - 1]; }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t k = wave_first + r * kWave + lane;
        key[r] = k < m ? keys[k] : 0u;
        val[r] = k < m ? vals[k] : 0u;
    }
#pragma unroll
    for (int q = 0; q < kPerWave; ++q) {
        uint32_t count = 0;
#pragma unroll
        for (int s = 0; s < kPerChunk; ++s) {
            const int r = q * kPerChunk + s;
            const int64_t k = wave_first + r * kWave + lane;
            const uint32_t prev = from_lane_below(key[r], last_key);
            const uint32_t pval = from_lane_below(val[r], last_val);
            bool head = false;
            if (k < m) {
                head = k == 0 || key[r] != prev;
                if (!head && val[r] < pval) disorder = true;
                // pairs a caller sorted (the library's own sort has validated its input): the kernels
                // below clamp a position outside the batch, here it is reported
                if (key[r] >= R || val[r] >= n) bad = true;
                if (k > 0 && key[r] < prev) unsorted = true;
            }
            count += (uint32_t)__popcll(ballot(head));
            last_key = (uint32_t)__builtin_amdgcn_readlane((int)key[r], kWave - 1);
            last_val = (uint32_t)__builtin_amdgcn_readlane((int)val[r], kWave - 1);
        }
        if (lane == 0) heads[w * kPerWave + q] = count;
    }
    if (ballot(disorder) != 0 && lane == 0) report(status, FS_DEV_POS_ORDER);
    if (ballot(bad) != 0 && lane == 0) report(status, FS_DEV_BAD_ID);
    if (ballot(unsorted) != 0 && lane == 0) report(status, FS_DEV_NOT_SORTED);
    __syncthreads();
    if (w == 0) {
        const uint32_t mine = heads[lane];
        uint32_t incl = mine;
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t up = __shfl_up(incl, off);
            if (lane >= off) incl += up;
        }
        const int64_t chunk = (int64_t)blockIdx.x * kChunksPerBlock + lane;
        if (chunk < chunks) chunk_local[chunk] = incl - mine;
        if (lane == kWave - 1) {
            if constexpr (TOTAL) {
                block_sum[0] = incl;
                *num_unique = (int64_t)incl;
                if ((int64_t)incl > cap) report(status, FS_DEV_UNIQUE_OVERFLOW);
            } else {
                block_sum[blockIdx.x] = incl;
            }
        }
    }
}

// One block: block_sum[0..blocks) -> exclusive prefix in place, block_sum[blocks] = total.
constexpr int kScanBlock = 1024;

__global__ __launch_bounds__(kScanBlock) void bwd_scan_blocks_kernel(
    uint32_t* __restrict__ block_sum, int64_t blocks, int64_t cap, int64_t* __restrict__ num_unique,
    int32_t* status)
{
    __shared__ uint32_t wave_sums[16];
    uint32_t carry = 0;                                          // coalesced rounds of 1024 entries
    for (int64_t base = 0; base < blocks; base += kScanBlock) {
        const int64_t k = base + threadIdx.x;
        const uint32_t v = k < blocks ? block_sum[k] : 0u;
        uint32_t total;
        const uint32_t before = block_exclusive_scan(v, wave_sums, &total);
        if (k < blocks) block_sum[k] = carry + before;
        carry += total;
    }
    if (threadIdx.x == 0) {
        block_sum[blocks] = carry;
        *num_unique = (int64_t)carry;
        if ((int64_t)carry > cap) report(status, FS_DEV_UNIQUE_OVERFLOW);
    }
}

// Up to this many blocks of the counting kernel (524 k lookups) their sums are added up where they are needed, by every
// wave with one load and six adds, in place of a scan launch.  The backward without and with that launch, us: 50 k lookups
// 24.4 : 26.6, 300 k 59.9 : 61.8, with the optimizer step 36.6 : 39.7 and (260 k) 63.9 : 64.7, 500 k 82.9 : 82.0, 1 M 140 : 138; 4.2 M
// of 128 columns 283 : 280.
constexpr int64_t kSumBlocks = 32;

__host__ __device__ __forceinline__ int64_t heads_blocks(int64_t chunks) { return (chunks + kChunksPerBlock - 1) / kChunksPerBlock; }

// `v` added up over the wave's lanes up to each, itself included.
__device__ __forceinline__ uint32_t wave_sums_upto(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111 /* row_shr:1 */, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112 /* row_shr:2 */, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114 /* row_shr:4 */, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118 /* row_shr:8 */, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142 /* row_bcast:15 */, 0xa, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143 /* row_bcast:31 */, 0xc, 0xf, false);
    return v;
}

// `v` added up over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_sums_upto(v), kWave - 1);
}

// Runs that start in the chunks before `chunk` (at most `chunks`); the same in every lane of the wave, all of which call it.
__device__ __forceinline__ uint32_t runs_before(const uint32_t* __restrict__ block_base,
                                                const uint32_t* __restrict__ chunk_local, int64_t chunk, int64_t chunks)
{
    const int64_t blocks = heads_blocks(chunks);
    const bool past = chunk >= chunks;
    const int64_t before = past ? blocks : chunk / kChunksPerBlock;
    uint32_t base;
    if (blocks == 1) {
        base = past ? block_base[0] : 0u;
    } else if (blocks <= kSumBlocks) {                       // uniform: block_base holds plain sums
        static_assert(kSumBlocks <= kWave);
        const int k = lane_id() < (int)blocks ? lane_id() : 0;
        const uint32_t v = block_base[k];
        base = wave_sum(lane_id() < (int)before ? v : 0u);
    } else {
        base = block_base[before];
    }
    return past ? base : base + chunk_local[chunk];
}

// The first block's first wave reports the number of runs where no kernel before it did.
__device__ __forceinline__ void report_runs(const uint32_t* __restrict__ block_base, const uint32_t* __restrict__ chunk_local,
                                            int64_t chunks, int64_t cap, int64_t* __restrict__ num_unique, int32_t* status)
{
    const int64_t blocks = heads_blocks(chunks);
    if (blocks == 1 || blocks > kSumBlocks) return;
    const uint32_t runs = runs_before(block_base, chunk_local, chunks, chunks);
    if (lane_id() == 0) {
        *num_unique = (int64_t)runs;
        if ((int64_t)runs > cap) report(status, FS_DEV_UNIQUE_OVERFLOW);
    }
}

template <int DT>
struct Vec;
template <>
struct Vec<FS_F32> {
    static constexpr int N = 4;
    static __device__ __forceinline__ void load(const u32x4& x, float* f)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(x[i]);   // (a bit_cast of a vector element miscompiles)
    }
};
template <>
struct Vec<FS_F16> {
    static constexpr int N = 8;
    static __device__ __forceinline__ void load(const u32x4& x, float* f)
    {
        const f16x8 h = __builtin_bit_cast(f16x8, x);
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = (float)h[i];
    }
};
template <>
struct Vec<FS_BF16> {
    static constexpr int N = 8;
    static __device__ __forceinline__ void load(const u32x4& x, float* f)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(x[i] << 16);
            f[2 * i + 1] = __uint_as_float(x[i] & 0xFFFF0000u);
        }
    }
};

constexpr uint32_t kEndBit = 0x80000000u;        // of a listed position (positions are < 2^31): the run's piece ends here

// The segmented sum for few chunks, where a walk of the chunk leaves the chip idle and costs its serial chain of
// loads whatever the batch (54 us for 8192 lookups of 256-byte rows).  One block takes one chunk, one slab of up
// to 16 pieces of its rows: the lookups it sums are listed in LDS, their rows follow with every load in flight at
// once (64 KB), and the chunk's run pieces are then summed out of LDS side by side, four columns to a lane, each
// piece left to right as the walk does it.  Bound by two rounds of memory latency and the longest run's chain in
// LDS: 9.0 us for those 8192 lookups, 14 us (was 63) for 50 k of 144-byte rows.  It sums runs of one
// lookup too, unless the optimizer's kernel takes them.  512 and 1024 threads per block measure the same, slabs of
// 8 and 4 pieces are no faster anywhere and 4 are slower from 1 M lookups on.
constexpr int kSlabPieces = 16;                  // 16-byte pieces of a row per slab
constexpr int kChunkLoads = 16;                  // loads a thread keeps in flight
// Up to this many chunks.  5 k / 40 k / 300 k / 3 M lookups, the whole backward, this kernel against the walk:
// 48-byte rows 70 : 81, 103 : 115, 134 : 139, 262 : 280 us; 208-byte 73 : 84, 104 : 116, 154 : 154, 431 : 385;
// 1 KB 68 : 85, 107 : 121, 206 : 205, 966 : 819.
constexpr int64_t kSumsMaxChunks = 1024;

template <int P_, int DT>                        // P_: pieces per slab, 0: `pieces`
__global__ __launch_bounds__(kBlock) void bwd_chunk_sums_kernel(
    const u32x4* __restrict__ grad, int units, int D, int pieces, int slabs,
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, int64_t m, int64_t chunks, uint32_t n,
    const uint32_t* __restrict__ block_base, const uint32_t* __restrict__ chunk_local,
    int64_t* __restrict__ uniq_rows, float* __restrict__ row_grads, int64_t cap,
    float* __restrict__ carry, int atomic, uint8_t* __restrict__ applied,
    int64_t* __restrict__ num_unique, int32_t* status)
{
    static_assert(kChunk == kBlock, "a thread per lookup of the chunk");
    constexpr int N = Vec<DT>::N;
    const int P = P_ != 0 ? P_ : pieces;
    extern __shared__ __attribute__((aligned(16))) u32x4 s_rows[];   // [kChunk][P]
    __shared__ uint32_t s_pos[kChunk];
    __shared__ uint32_t s_start[kChunk + 1];     // a run piece's first row in s_rows
    __shared__ uint32_t s_run[kChunk];           // its run index
    __shared__ uint32_t wave_n[kWavesPerBlock][3];
    const int t = threadIdx.x;
    const int w = wave_id();
    if (blockIdx.x == 0 && w == 0) report_runs(block_base, chunk_local, chunks, cap, num_unique, status);
    const int64_t chunk = blockIdx.x / slabs;
    const int slab = (int)(blockIdx.x - chunk * slabs);
    const int64_t k0 = chunk * kChunk;
    const int64_t k1 = k0 + kChunk < m ? k0 + kChunk : m;
    const int64_t k = k0 + t;
    const bool valid = k < k1;
    const int64_t ks = valid ? k : k1 - 1;       // no load behind a predicate
    const uint32_t key = keys[ks];
    const uint32_t prev_key = keys[ks > 0 ? ks - 1 : 0];
    const uint32_t next_key = keys[ks + 1 < m ? ks + 1 : ks];
    uint32_t pos = vals[ks];
    const uint32_t first_run = runs_before(block_base, chunk_local, chunk, chunks);
    pos = pos < n ? pos : 0u;                    // a position outside the batch reads row 0
    const bool head = valid && (k == 0 || key != prev_key);          // a run starts here
    const bool last = k + 1 >= m || key != next_key;                 // it ends here
    const bool keep = valid && !(applied != nullptr && head && last);// a row looked up once is the update kernel's
    const bool start = keep && (head || t == 0);                     // a piece of a run starts here
    const uint64_t hb = ballot(head), kb = ballot(keep), sb = ballot(start);
    if (lane_id() == 0) {
        wave_n[w][0] = (uint32_t)__popcll(hb); wave_n[w][1] = (uint32_t)__popcll(kb); wave_n[w][2] = (uint32_t)__popcll(sb);
    }
    __syncthreads();
    uint32_t heads = (uint32_t)popc_below(hb) + (head ? 1u : 0u), at = (uint32_t)popc_below(kb), piece = (uint32_t)popc_below(sb);
    uint32_t rows = 0, num_pieces = 0;
#pragma unroll
    for (int q = 0; q < kWavesPerBlock; ++q) {
        if (q < w) { heads += wave_n[q][0]; at += wave_n[q][1]; piece += wave_n[q][2]; }
        rows += wave_n[q][1];
        num_pieces += wave_n[q][2];
    }
    if (rows == 0) return;                                           // block-uniform
    const int64_t run = (int64_t)first_run + heads - 1;
    if (keep) s_pos[at] = pos;
    if (start) { s_start[piece] = at; s_run[piece] = (uint32_t)run; }
    if (t == 0) s_start[num_pieces] = rows;
    if (slab == 0 && keep && head && run < cap) {
        uniq_rows[run] = (int64_t)key;
        if (applied != nullptr) applied[run] = 0;                    // this row's gradient is in row_grads
    }
    const bool cont = k0 > 0 && keys[k0 - 1] == keys[k0];            // the first piece continues the previous chunk's run
    const bool goes_on = k1 < m && keys[k1] == keys[k1 - 1];         // the last run goes on in the next chunk
    __syncthreads();

    const uint32_t total = rows * (uint32_t)P;
    const uint32_t inv = (65536u + (uint32_t)P - 1u) / (uint32_t)P;  // e / P = e * inv >> 16 for e < 4096, P <= 16
    const int piece0 = slab * P;
    for (uint32_t e0 = 0; e0 < total; e0 += kBlock * kChunkLoads) {
        u32x4 x[kChunkLoads];
#pragma unroll
        for (int j = 0; j < kChunkLoads; ++j) {
            uint32_t e = e0 + j * kBlock + t;
            e = e < total ? e : total - 1;
            const uint32_t r = P_ != 0 ? e / (uint32_t)P : (e * inv) >> 16;
            const int c = piece0 + (int)(e - r * (uint32_t)P);
            x[j] = load_stream(grad + (int64_t)s_pos[r] * units + (c < units ? c : units - 1));
        }
#pragma unroll
        for (int j = 0; j < kChunkLoads; ++j) {
            const uint32_t e = e0 + j * kBlock + t;
            if (e < total) s_rows[e] = x[j];
        }
    }
    __syncthreads();

    // A lane sums four columns of a run's piece, or one where the chunk has no more pieces than then fit side by side: the
    // long runs of a popular row leave the other lanes idle, and their chain is the block's time.  262 k lookups of 1 KB
    // rows, Zipf(1.3) 141 -> 128 us (the walk before this kernel: 141), all of one row 199 -> 182 (181); of f32
    // 111 -> 102 (116) and 143 -> 131 (122).
    if (num_pieces <= (uint32_t)(kBlock / (P * N))) {
        auto value = [&](uint32_t r, int c) -> float {
            if constexpr (DT == FS_F32) return __uint_as_float(reinterpret_cast<const uint32_t*>(s_rows)[r * (P * N) + c]);
            const uint16_t v = reinterpret_cast<const uint16_t*>(s_rows)[r * (P * N) + c];
            if constexpr (DT == FS_F16) return (float)__builtin_bit_cast(_Float16, v);
            return __uint_as_float((uint32_t)v << 16);
        };
        const uint32_t p = t / (P * N);
        const int c = t - (int)p * (P * N);
        const int col = slab * P * N + c;
        if (p >= num_pieces || col >= D) return;                     // no barrier below
        uint32_t r = s_start[p];
        const uint32_t end = s_start[p + 1];
        const int64_t u = s_run[p];
        float acc = value(r++, c);
        for (; r + 8 <= end; r += 8) {
            float f[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = value(r + j, c);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc = acc + f[j];
        }
        for (; r < end; ++r) acc = acc + value(r, c);
        const bool continues = cont && p == 0;
        float* dst;
        if (continues && !atomic) dst = carry + chunk * D + col;
        else if (u < cap) dst = row_grads + u * D + col;
        else return;
        if (atomic && (continues || (goes_on && p == num_pieces - 1))) unsafeAtomicAdd(dst, acc);
        else store_stream(dst, acc);
        return;
    }
    const int quads = P * (N / 4);
    const int slots = kBlock / quads;
    const int slot = t / quads;
    const int quad = t - slot * quads;
    const int col = slab * P * N + quad * 4;
    if (slot >= slots || col >= D) return;                           // no barrier below
    auto load_quad = [&](uint32_t r) -> f32x4 {
        if constexpr (N == 4) {
            const u32x4 v = s_rows[r * P + quad];
            return f32x4{__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3])};
        } else {
            const u32x2 v = reinterpret_cast<const u32x2*>(s_rows)[r * (2 * P) + quad];
            if constexpr (DT == FS_F16) {
                const f16x4 h = __builtin_bit_cast(f16x4, v);
                return f32x4{(float)h[0], (float)h[1], (float)h[2], (float)h[3]};
            } else {
                return f32x4{__uint_as_float(v[0] << 16), __uint_as_float(v[0] & 0xFFFF0000u),
                             __uint_as_float(v[1] << 16), __uint_as_float(v[1] & 0xFFFF0000u)};
            }
        }
    };
    for (uint32_t p = slot; p < num_pieces; p += slots) {
        uint32_t r = s_start[p];
        const uint32_t end = s_start[p + 1];
        const int64_t u = s_run[p];
        f32x4 acc = load_quad(r++);
        for (; r + 8 <= end; r += 8) {
            f32x4 f[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = load_quad(r + j);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc = acc + f[j];
        }
        for (; r < end; ++r) acc = acc + load_quad(r);
        const bool continues = cont && p == 0;
        float* dst;
        if (continues && !atomic) dst = carry + chunk * D + col;
        else if (u < cap) dst = row_grads + u * D + col;
        else continue;
        if (atomic && (continues || (goes_on && p == num_pieces - 1))) {
#pragma unroll
            for (int q = 0; q < 4; ++q) unsafeAtomicAdd(dst + q, acc[q]);
        } else {
            store_stream(reinterpret_cast<f32x4*>(dst), acc);
        }
    }
}

// VB bytes of a row as a lane holds them, and their elements as floats.
template <int VB>
struct Bytes;
template <>
struct Bytes<4> {
    typedef uint32_t type;
    template <int DT>
    static __device__ __forceinline__ void load(uint32_t x, float* f)
    {
        if constexpr (DT == FS_F32) {
            f[0] = __uint_as_float(x);
        } else if constexpr (DT == FS_F16) {
            const f16x2 h = __builtin_bit_cast(f16x2, x);
            f[0] = (float)h[0]; f[1] = (float)h[1];
        } else {
            f[0] = __uint_as_float(x << 16); f[1] = __uint_as_float(x & 0xFFFF0000u);
        }
    }
};
template <>
struct Bytes<8> {
    typedef u32x2 type;
    template <int DT>
    static __device__ __forceinline__ void load(const u32x2& x, float* f)
    {
        constexpr int H = DT == FS_F32 ? 1 : 2;
        Bytes<4>::load<DT>(x[0], f);
        Bytes<4>::load<DT>(x[1], f + H);
    }
};
// The segmented sum.  A wave walks one chunk left to right (one slab of 64 * VB bytes of its rows, VB bytes to a
// lane).  The lookups of repeated rows are listed in LDS, position and run index; the walk reads a batch of 8 of
// them with one LDS load, hands the positions to scalar registers, and has the next batch's rows in flight while it
// sums this one's.  A run's end is a bit of a scalar mask, so nothing in the walk diverges and a finished piece
// leaves as one coalesced store.  Bound by the mix of the gradient stream with the stores' (the whole chip's reads
// and writes, 5.2 TB/s on 512-byte rows), below some 8 k chunks by the walk's serial chain.
// 4 bytes to a lane for rows of up to 256 bytes: a chunk per wave instead of four of them in 16-lane groups with 16
// bytes to a lane gives four times the waves and no divergent flushes: 1.05 M lookups of 256-byte rows 74 -> 58 us,
// 4.2 M 244 -> 206, 8.4 M (a table's head row is a quarter of them) 438 -> 408.  8 bytes for longer rows, where both
// measure the same within the runs' spread (15.7 M lookups of 512-byte rows 1528 us, 72 M 5.9 to 7.0 ms where the bare
// stream of the same mix takes 6.4 to 7.6; 4 bytes on 72 M 1 % more): the chip's rate is what bounds them.  On 256-byte
// rows 8 would leave half the lanes idle (937 us).  16 rows to a batch instead of 8 measure the same.
template <int VB, int DT>
__global__ __launch_bounds__(kBlock) void bwd_segreduce_kernel(
    const unsigned char* __restrict__ grad, int row_bytes, int D,
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, int64_t m, int64_t chunks, uint32_t n,
    const uint32_t* __restrict__ block_base, const uint32_t* __restrict__ chunk_local,
    int64_t* __restrict__ uniq_rows, float* __restrict__ row_grads, int64_t cap,
    float* __restrict__ carry, int atomic, uint8_t* __restrict__ applied,
    int64_t* __restrict__ num_unique, int32_t* status)
{
    constexpr int U = kWalkAhead;
    constexpr int ES = DT == FS_F32 ? 4 : 2;
    constexpr int N = VB / ES;                                       // elements per lane
    typedef typename Bytes<VB>::type part_t;
    __shared__ uint32_t s_pos[kWavesPerBlock][kChunk + kWave];
    __shared__ uint32_t s_run[kWavesPerBlock][kChunk + kWave];
    const int w = wave_id();
    const int lane = lane_id();
    if (blockIdx.x == 0 && blockIdx.y == 0 && w == 0) report_runs(block_base, chunk_local, chunks, cap, num_unique, status);
    const int64_t chunk = (int64_t)blockIdx.x * kWavesPerBlock + w;
    if (chunk >= chunks) return;                                     // wave-uniform; no block barrier below
    const int64_t k0 = chunk * kChunk;
    const int64_t k1 = k0 + kChunk < m ? k0 + kChunk : m;
    uint32_t* pos_of = s_pos[w];
    uint32_t* run_of = s_run[w];
    constexpr int Q = kChunk / kWave;
    uint32_t key[Q], prev[Q], next[Q], pos[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {                                    // all loads in one round, none behind a predicate
        const int64_t k = k0 + q * kWave + lane;
        const int64_t ks = k < k1 ? k : k1 - 1;
        key[q] = keys[ks];
        prev[q] = keys[ks > 0 ? ks - 1 : 0];
        next[q] = keys[ks + 1 < m ? ks + 1 : ks];
        pos[q] = vals[ks];
    }
    uint32_t runs = runs_before(block_base, chunk_local, chunk, chunks);
    uint32_t listed = 0;
    bool cont = false;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t k = k0 + q * kWave + lane;
        const bool valid = k < k1;
        const bool head = valid && (k == 0 || key[q] != prev[q]);
        const bool last = k + 1 >= m || key[q] != next[q];
        const bool keep = valid && !(head && last);                  // runs of one lookup are another kernel's
        const bool end = last || k + 1 == k1;
        const uint64_t hb = ballot(head), kb = ballot(keep);
        const uint32_t at = listed + (uint32_t)popc_below(kb);
        const uint32_t run = runs + (uint32_t)popc_below(hb) + (head ? 1u : 0u) - 1u;
        if (keep) {
            pos_of[at] = (pos[q] < n ? pos[q] : 0u) | (end ? kEndBit : 0u);   // a position outside the batch reads row 0
            run_of[at] = run;
        }
        if (keep && head && blockIdx.y == 0 && (int64_t)run < cap) {
            uniq_rows[run] = (int64_t)key[q];
            if (applied != nullptr) applied[run] = 0;                // this row's gradient is in row_grads
        }
        if (q == 0) cont = k0 > 0 && (hb & 1) == 0;                  // the first piece continues the previous chunk's run
        runs += (uint32_t)__popcll(hb);
        listed += (uint32_t)__popcll(kb);
    }
    const int cnt = (int)listed;
    if (cnt == 0) return;
    static_assert(3 * U <= kWave);
    pos_of[cnt + lane] = 0u;                                         // batches issued past the end (up to 3 U - 1 lookups) read row 0, unused
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const bool goes_on = k1 < m && keys[k1] == keys[k1 - 1];         // the chunk's last run goes on in the next
    const int byte = (blockIdx.y * kWave + lane) * VB;
    const bool lane_on = byte < row_bytes;
    const unsigned char* my_grad = grad + (lane_on ? byte : 0);
    const int col = byte / ES;
    float acc[N];
    bool fresh = true;

    auto issue = [&](part_t* x, uint32_t* ends, uint32_t& run, int e0) {
        const uint32_t p = pos_of[e0 + lane % U];
        run = run_of[e0 + lane % U];
        *ends = (uint32_t)ballot((p & kEndBit) != 0);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const uint32_t pj = (uint32_t)__builtin_amdgcn_readlane((int)p, j) & ~kEndBit;
            x[j] = load_stream(reinterpret_cast<const part_t*>(my_grad + (int64_t)pj * row_bytes));
        }
    };
    auto consume = [&](const part_t* x, uint32_t ends, uint32_t run, int e0) {
#pragma unroll
        for (int j = 0; j < U; ++j) {
            if (e0 + j < cnt) {
                float f[N];
                Bytes<VB>::template load<DT>(x[j], f);
                if (fresh) {
#pragma unroll
                    for (int q = 0; q < N; ++q) acc[q] = f[q];
                } else {
#pragma unroll
                    for (int q = 0; q < N; ++q) acc[q] = acc[q] + f[q];
                }
                fresh = false;
                if ((ends >> j) & 1u) {
                    const int64_t u = (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)run, j);
                    float* dst = nullptr;
                    if (cont && !atomic) dst = carry + chunk * D;
                    else if (u < cap) dst = row_grads + u * D;
                    if (dst != nullptr && lane_on) {
                        if (atomic && (cont || (goes_on && e0 + j == cnt - 1))) {
#pragma unroll
                            for (int q = 0; q < N; ++q) unsafeAtomicAdd(dst + col + q, acc[q]);
                        } else {
                            typedef float out_t __attribute__((ext_vector_type(N)));
                            out_t o;
#pragma unroll
                            for (int q = 0; q < N; ++q) o[q] = acc[q];
                            store_stream(reinterpret_cast<out_t*>(dst + col), o);
                        }
                    }
                    fresh = true;
                    cont = false;
                }
            }
        }
    };
    part_t xa[U], xb[U];
    uint32_t ea, eb, ra, rb;
    issue(xa, &ea, ra, 0);
#pragma unroll 1
    for (int e0 = 0; e0 < cnt; e0 += 2 * U) {
        issue(xb, &eb, rb, e0 + U);
        consume(xa, ea, ra, e0);
        issue(xa, &ea, ra, e0 + 2 * U);
        consume(xb, eb, rb, e0 + U);
    }
}

// Moves CNT * 64/LG listed singletons: the rows' loads first, then conversion and stores.  An index
// past the list repeats the last entry (same bytes to the same place), so nothing is predicated.
template <int CNT, int LG, int DT, bool EXACT>
__device__ __forceinline__ void singles_batch(
    const u32x4* __restrict__ grad, int units, int D, const uint32_t* s_pos, const uint32_t* s_run,
    const uint32_t* s_key, float* stage, uint32_t s, uint32_t singles, int c, bool all_fit, int64_t cap,
    int64_t* __restrict__ uniq_rows, float* __restrict__ row_grads)
{
    constexpr int N = Vec<DT>::N;
    constexpr int RPI = kWave / LG;
    const int g = lane_id() / LG;
    const bool lane_on = c < units;
    const int cc = lane_on ? c : 0;
    u32x4 x[CNT];
    uint32_t run[CNT];
    uint32_t at[CNT];
#pragma unroll
    for (int j = 0; j < CNT; ++j) {
        const uint32_t want = s + j * RPI + g;
        at[j] = want < singles ? want : singles - 1;
        run[j] = s_run[at[j]];
        x[j] = load_stream(grad + (int64_t)s_pos[at[j]] * (EXACT ? LG : units) + cc);
    }
    const int lig = lane_id() % LG;
#pragma unroll
    for (int j = 0; j < CNT; ++j) {
        const bool fits = all_fit || (int64_t)run[j] < cap;          // the same for the whole group
        float f[N];
        Vec<DT>::load(x[j], f);
        float* row = row_grads + (int64_t)run[j] * D;
        if constexpr (N == 4) {
            if (lane_on && fits) store_stream(reinterpret_cast<f32x4*>(row + cc * 4), f32x4{f[0], f[1], f[2], f[3]});
        } else {
            // 8 floats per lane: stored as they are, each 16-byte store would cover half of every
            // 32 bytes.  Through the wave's LDS slab lane i takes floats [4i, 4i+4) of each half of
            // the group's columns instead, and both stores are fully coalesced.
            float* gs = stage + g * LG * 8;
            *reinterpret_cast<f32x4*>(gs + lig * 8) = f32x4{f[0], f[1], f[2], f[3]};
            *reinterpret_cast<f32x4*>(gs + lig * 8 + 4) = f32x4{f[4], f[5], f[6], f[7]};
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const f32x4 lo = *reinterpret_cast<const f32x4*>(gs + lig * 4);
            const f32x4 hi = *reinterpret_cast<const f32x4*>(gs + LG * 4 + lig * 4);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int slab = (c - lig) * 8;                          // first column of the group's slab
            const int col_lo = slab + lig * 4;
            const int col_hi = slab + LG * 4 + lig * 4;
            if (fits && col_lo < D) store_stream(reinterpret_cast<f32x4*>(row + col_lo), lo);
            if (fits && col_hi < D) store_stream(reinterpret_cast<f32x4*>(row + col_hi), hi);
        }
        if (fits && c == 0) uniq_rows[run[j]] = (int64_t)s_key[at[j]];
    }
}

// The singletons of a wave's share of one chunk, listed in LDS (position, run index, row), in order.
// kSinglesSplit waves share a chunk: each reads all of its keys (run indices need the heads before
// it) but lists only the singletons of its own quarter.  Shorter-lived waves with less to move each
// are faster here, as for a plain copy: 1, 2, 4, 8 waves per chunk take 0.366, 0.340, 0.340, 0.389 ms
// on 15.7 M lookups and 2.63, 2.54, 2.50, 2.72 ms on 72 M.  Returns false (wave-uniform) if the wave
// has nothing to do; *runs_end = index after the last run that starts in the part of the chunk read so far.
__device__ __forceinline__ bool list_singletons(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, int64_t m, int64_t chunks, uint32_t n,
    const uint32_t* __restrict__ block_base, const uint32_t* __restrict__ chunk_local,
    uint32_t* s_pos, uint32_t* s_run, uint32_t* s_key, uint32_t* singles_out, uint32_t* runs_end, int spread = 0)
{
    const int lane = lane_id();
    const int64_t wave_global = (int64_t)blockIdx.x * kWavesPerBlock + wave_id();
    const int64_t part_global = wave_global >> spread;
    const int64_t chunk = part_global / kSinglesSplit;
    const int part = (int)(part_global % kSinglesSplit);
    const bool mine = (lane >> (6 - spread)) == (int)(wave_global & ((1 << spread) - 1));
    if (chunk >= chunks) return false;
    const int64_t k0 = chunk * kChunk;
    const int64_t k1 = k0 + kChunk < m ? k0 + kChunk : m;
    // One round of loads, none behind a predicate: the chunk's keys, the ones before and after it, the positions of the
    // part.  A lookup's neighbours are its lane's; the ends of the list are known by index (no key can stand for "none",
    // a caller's list may hold any 32-bit word).
    constexpr int Q = kChunk / kWave;
    static_assert(kSinglesSplit == Q, "a part is one round of 64 lookups");
    uint32_t key[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t k = k0 + q * kWave + lane;
        key[q] = keys[k < k1 ? k : k1 - 1];
    }
    const uint32_t before = keys[k0 > 0 ? k0 - 1 : 0];
    const uint32_t after = keys[k1 < m ? k1 : k1 - 1];
    const int64_t my_k = k0 + part * kWave + lane;
    const uint32_t my_pos = vals[my_k < k1 ? my_k : k1 - 1];
    const uint32_t first_run = runs_before(block_base, chunk_local, chunk, chunks);

    uint32_t heads_before = 0, singles = 0, last = before;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t k = k0 + q * kWave + lane;
        const bool valid = k < k1;
        const uint32_t prev = from_lane_below(key[q], last);
        const uint32_t next = from_lane_above(key[q], q + 1 < Q ? (uint32_t)__builtin_amdgcn_readlane((int)key[q + 1 < Q ? q + 1 : q], 0) : after);
        const bool head = valid && (k == 0 || key[q] != prev);
        const uint64_t hb = ballot(head);
        if (q == part) {                                         // wave-uniform
            const bool single = mine && head && (k + 1 >= m || key[q] != (k + 1 < k1 ? next : after));
            const uint64_t sb = ballot(single);
            if (single) {
                const uint32_t at = (uint32_t)popc_below(sb);
                s_pos[at] = my_pos < n ? my_pos : 0u;            // a position outside the batch reads row 0
                s_run[at] = first_run + heads_before + (uint32_t)popc_below(hb);
                s_key[at] = key[q];
            }
            singles = (uint32_t)__popcll(sb);
        }
        heads_before += (uint32_t)__popcll(hb);
        last = (uint32_t)__builtin_amdgcn_readlane((int)key[q], kWave - 1);
    }
    *singles_out = singles;
    *runs_end = first_run + heads_before;
    if (singles == 0) return false;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    return true;
}

// The backward that applies the optimizer step itself, for rows looked up once: their gradient is the
// one converted row, so instead of writing it to row_grads (and an optimizer step reading it back) the
// wave updates the table row in place: gradient row in, table row in and out, 1.5 KB of traffic per
// 512-byte row where gradient-out-and-back-in costs 3.5 KB.  The arithmetic and the lane layout are those
// of fs_sparse_update's kernel (RowUpdate: lane i of a group holds quads i and LG + i of the row), which
// the gradient reaches through the same LDS transposition that the plain kernel uses for its stores; the
// new rows are therefore bit for bit what fs_seq_grad_bwd followed by fs_sparse_update writes.
// applied[u] = 1 tells the optimizer step that follows (for the rows summed from several lookups) to
// leave entry u alone.  Rows of up to 64 pieces.
template <int CNT, int LG, int DT, int OPT, bool EXACT>
__device__ __forceinline__ void singles_update_batch(
    const u32x4* __restrict__ grad, const UpdateArgs& a, const uint32_t* s_pos, const uint32_t* s_run,
    const uint32_t* s_key, float* stage, uint32_t s, uint32_t singles, int64_t cap,
    int64_t* __restrict__ uniq_rows, uint8_t* __restrict__ applied)
{
    constexpr int N = Vec<DT>::N;
    constexpr int P = N / 4;
    constexpr int RPI = kWave / LG;
    typedef typename Quad<DT>::type quad_t;
    const int g = lane_id() / LG;
    const int lig = lane_id() % LG;
    const int units = EXACT ? LG : a.units;
    const int64_t D = EXACT ? LG * N : a.D;
    const bool piece_on = lig < units;                               // the lane's 16-byte piece of the gradient row exists
    int col[P];
    bool on[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int c = (p * LG + lig) * 4;
        on[p] = c < D;
        col[p] = on[p] ? c : 0;
    }
    const quad_t* wq = reinterpret_cast<const quad_t*>(a.weights);
    quad_t* wq_out = reinterpret_cast<quad_t*>(a.weights);
    quad_t* store_out = reinterpret_cast<quad_t*>(a.store);

    u32x4 x[CNT];
    quad_t wx[CNT][P];
    f32x4 sx[CNT][P];
    float srow[CNT];
    int64_t row[CNT];
    uint32_t run[CNT];
    bool ok[CNT];
    int slot[CNT];
#pragma unroll
    for (int j = 0; j < CNT; ++j) {
        const uint32_t want = s + j * RPI + g;
        const uint32_t at = want < singles ? want : singles - 1;     // past the list: the last entry again, not stored
        run[j] = s_run[at];
        const uint32_t key = s_key[at];
        ok[j] = want < singles && (int64_t)run[j] < cap && (int64_t)key < a.R;
        row[j] = (int64_t)key < a.R ? (int64_t)key : 0;
        x[j] = load_stream(grad + (int64_t)s_pos[at] * units + (piece_on ? lig : 0));
#pragma unroll
        for (int p = 0; p < P; ++p) {
            wx[j][p] = load_stream(wq + ((row[j] * D + col[p]) >> 2));
            if constexpr (OPT == FS_OPT_ADAGRAD)
                sx[j][p] = load_stream(reinterpret_cast<const f32x4*>(a.state + row[j] * D + col[p]));
        }
        if constexpr (OPT == FS_OPT_ADAGRAD_ROWWISE) srow[j] = a.state[row[j]];
        slot[j] = -1;
        if (a.store != nullptr) slot[j] = a.slot_of_row[row[j]];     // (wave-uniform branch: the load itself is not predicated)
    }
#pragma unroll
    for (int j = 0; j < CNT; ++j) {
        if (!ok[j]) slot[j] = -1;
        if (slot[j] >= a.k) { if (lig == 0) report(a.status, FS_DEV_BAD_ID); slot[j] = -1; }
    }
#pragma unroll
    for (int j = 0; j < CNT; ++j) {
        float f[N];
        Vec<DT>::load(x[j], f);
        f32x4 gx[P];
        if constexpr (N == 4) {
            gx[0] = f32x4{f[0], f[1], f[2], f[3]};                   // lane i holds quad i already
        } else {
            // 8 consecutive floats per lane -> quads i and LG + i, through the wave's LDS slab
            float* gs = stage + g * LG * 8;
            *reinterpret_cast<f32x4*>(gs + lig * 8) = f32x4{f[0], f[1], f[2], f[3]};
            *reinterpret_cast<f32x4*>(gs + lig * 8 + 4) = f32x4{f[4], f[5], f[6], f[7]};
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            gx[0] = *reinterpret_cast<const f32x4*>(gs + lig * 4);
            gx[1] = *reinterpret_cast<const f32x4*>(gs + LG * 4 + lig * 4);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        RowUpdate<LG, DT, OPT>::apply(wx[j], gx, sx[j], srow[j], on, col, row[j], D, lig, ok[j], slot[j], a.lr, a.eps,
                                      wq_out, store_out, a.state);
        const uint32_t want = s + j * RPI + g;
        if (want < singles && (int64_t)run[j] < cap && lig == 0) {
            uniq_rows[run[j]] = (int64_t)s_key[want];
            applied[run[j]] = 1;
        }
    }
}

// 2^spread waves share a part where there are few chunks: a wave's time is its chain of rows, each with a division and a
// square root to an element, and 640 waves leave most SIMDs idle.  The backward with the step, spread 0 / 1 / 2 / 3, us
// (with 16 entries to a wave of the step that follows): 10 k lookups of 512-byte rows 59 / 50 / 43 / 39 (36), of f16 rows with
// element-wise state 43 / 38 / 35 / 34 (33); 50 k 74 / 64 / 56 / 52 (49) and 54 / 51 / 47 / 46 (43); 260 k 111 / 105 / 100 / 101
// and 84 / 78 / 76 / 76; 1 M 228 / 221 / 221 / 234 and 180 / 176 / 174 / 188; 2 M of 256-byte rows 205 / 207 / 220 / 247.
static int update_spread(int64_t chunks) { return chunks <= 256 ? 3 : chunks <= 2048 ? 2 : chunks <= 4608 ? 1 : 0; }

template <int LG, int DT, int OPT, bool EXACT>
__global__ __launch_bounds__(kBlock) void bwd_singletons_update_kernel(
    const u32x4* __restrict__ grad, const UpdateArgs a,
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, int64_t m, int64_t chunks, uint32_t n,
    const uint32_t* __restrict__ block_base, const uint32_t* __restrict__ chunk_local,
    int64_t* __restrict__ uniq_rows, int64_t cap, uint8_t* __restrict__ applied, int spread)
{
    constexpr int RPI = kWave / LG;
    constexpr int CNT = 2;                                           // rows a group keeps in flight (each brings a gradient row, a table
                                                                     // row and its state): 1 and 2 measure the same, 4 is 5 % and 8 is
                                                                     // 25 % slower on 15.7 M lookups of 512-byte rows
    __shared__ uint32_t s_pos[kWavesPerBlock][kChunk / kSinglesSplit];
    __shared__ uint32_t s_run[kWavesPerBlock][kChunk / kSinglesSplit];
    __shared__ uint32_t s_key[kWavesPerBlock][kChunk / kSinglesSplit];
    __shared__ __attribute__((aligned(16))) float s_stage[kWavesPerBlock][kWave * 8];
    const int w = wave_id();
    uint32_t singles, runs_end;
    if (!list_singletons(keys, vals, m, chunks, n, block_base, chunk_local, s_pos[w], s_run[w], s_key[w], &singles,
                         &runs_end, spread))
        return;                                                      // wave-uniform; no block barrier below
    for (uint32_t s = 0; s < singles; s += CNT * RPI)
        singles_update_batch<CNT, LG, DT, OPT, EXACT>(grad, a, s_pos[w], s_run[w], s_key[w], s_stage[w], s, singles, cap,
                                                       uniq_rows, applied);
}

// Runs of one lookup need no sum: row_grads[u] = f32(grad_out[pos]).  They are most of the runs
// (the cold tail of the popularity distribution) and a store in the sequential walk above stalls
// the wave's later loads (loads and stores share one in-order counter), so this kernel converts
// them instead, fully parallel: a wave takes a quarter of a chunk, finds its singletons and their
// run indices with ballots, lists them in LDS and moves 64/LG rows per instruction, 8 in flight.
template <int LG, int DT, bool EXACT>
__global__ __launch_bounds__(kBlock) void bwd_singletons_kernel(
    const u32x4* __restrict__ grad, int units, int D,
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, int64_t m, int64_t chunks, uint32_t n,
    const uint32_t* __restrict__ block_base, const uint32_t* __restrict__ chunk_local,
    int64_t* __restrict__ uniq_rows, float* __restrict__ row_grads, int64_t cap)
{
    constexpr int RPI = kWave / LG;
    constexpr int UNR = 8;
    __shared__ uint32_t s_pos[kWavesPerBlock][kChunk / kSinglesSplit];
    __shared__ uint32_t s_run[kWavesPerBlock][kChunk / kSinglesSplit];
    __shared__ uint32_t s_key[kWavesPerBlock][kChunk / kSinglesSplit];
    __shared__ __attribute__((aligned(16))) float s_stage[kWavesPerBlock][kWave * 8];   // store transposition, per wave
    const int w = wave_id();
    const int lane = lane_id();
    uint32_t singles, runs_end;
    if (!list_singletons(keys, vals, m, chunks, n, block_base, chunk_local, s_pos[w], s_run[w], s_key[w], &singles,
                         &runs_end))
        return;                                                  // wave-uniform; no block barrier below
    const int c = blockIdx.y * LG + lane % LG;
    const bool all_fit = (int64_t)runs_end <= cap;
    // Full batches of UNR instructions, then ONE batch of exactly as many instructions as the rest
    // needs: padding the last batch with repeats of the last row would write that row again and
    // again, and with ~18 singletons per chunk that is a third of the kernel's traffic.
    uint32_t s = 0;
    for (; s + UNR * RPI <= singles; s += UNR * RPI)
        singles_batch<UNR, LG, DT, EXACT>(grad, units, D, s_pos[w], s_run[w], s_key[w], s_stage[w], s, singles, c, all_fit,
                                          cap, uniq_rows, row_grads);
    if (s < singles) {
#define FS_TAIL(CNT) case CNT: singles_batch<CNT, LG, DT, EXACT>(grad, units, D, s_pos[w], s_run[w], s_key[w],    \
                                                                 s_stage[w], s, singles, c, all_fit, cap, uniq_rows, \
                                                                 row_grads); break
        switch ((singles - s + RPI - 1) / RPI) {
            FS_TAIL(1); FS_TAIL(2); FS_TAIL(3); FS_TAIL(4); FS_TAIL(5); FS_TAIL(6); FS_TAIL(7);
            default: singles_batch<UNR, LG, DT, EXACT>(grad, units, D, s_pos[w], s_run[w], s_key[w], s_stage[w], s,
                                                       singles, c, all_fit, cap, uniq_rows, row_grads);
        }
#undef FS_TAIL
    }
}

// A run that goes on over many chunks, left to bwd_fold_long: row_grads[run] += carry[first .. last], left to right.
struct LongRun {
    uint32_t run;
    uint32_t first, last;                        // chunks
};
// Runs with more carries than this are left to it, where the batch is large enough (chunks times columns) for the launch
// to be worth its 3 to 5 us.  The backward without and with it, Zipf(1.3) and Zipf(1.05) over 50 M rows: 300 k lookups (1172
// chunks) of 128 columns 52 : 54 and 62 : 66 us, of 256 80 : 75 and 93 : 96, 1 M (4102) of 64 93 : 97 and 107 : 107, of 128
// 111 : 105 and 125 : 125 (Zipf(1.1) over 8 tables: the folds alone 8 : 12), of 256 197 : 167 and 224 : 219, 4.2 M of 64
// 293 : 287 and 313 : 314, of 256 657 : 519 and 729 : 691.
constexpr int64_t kFoldLong = 64;
constexpr int64_t kFoldLongWork = 1000000;

// One wave per chunk; a wave whose chunk starts a spilling run (one that goes on into the next
// chunk) adds the carries of the chunks the run goes on into, left to right.
// VL: consecutive columns per lane.  Rows of up to 64 or 128 columns take 1 or 2, so that all lanes of the wave carry a
// share and the same registers hold four times or twice as many carries in flight.
template <int VL>
__global__ __launch_bounds__(kBlock) void bwd_fold_kernel(
    const uint32_t* __restrict__ keys, int64_t m, int64_t chunks,
    const uint32_t* __restrict__ block_base, const uint32_t* __restrict__ chunk_local,
    float* __restrict__ row_grads, int D, int64_t cap, const float* __restrict__ carry,
    LongRun* __restrict__ long_runs /* or null */, uint32_t* __restrict__ num_long)
{
    const int64_t chunk = (int64_t)blockIdx.x * kWavesPerBlock + wave_id();
    const int64_t k0 = chunk * kChunk;
    const int64_t k1 = k0 + kChunk;
    if (k1 >= m) return;                                             // nothing follows this chunk
    // Every index the decision needs, loaded in one round: a wave's time here is a chain of
    // dependent loads, and there are as many waves as chunks.
    const uint32_t key = keys[k1 - 1];
    const uint32_t next = keys[k1];
    const uint32_t head = keys[k0];
    const uint32_t before = keys[k0 > 0 ? k0 - 1 : 0];
    const bool has_far = chunk + 2 < chunks;                         // then (chunk + 2) * kChunk < m
    const uint32_t far = keys[has_far ? k1 + kChunk : k1];
    // Runs before a chunk from what stands in chunk_local for it.  Few blocks: their sums added up once, a lane for each.
    const int64_t blocks = heads_blocks(chunks);
    uint32_t upto = 0;
    if (blocks > 1 && blocks <= kSumBlocks) upto = wave_sums_upto(lane_id() < (int)blocks ? block_base[lane_id()] : 0u);
    auto runs_at = [&](int64_t c, uint32_t local) {                  // c < chunks, the same in the whole wave
        const int block = __builtin_amdgcn_readfirstlane((int)(c / kChunksPerBlock));
        if (blocks > kSumBlocks) return block_base[block] + local;
        return (block == 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)upto, block - 1)) + local;
    };
    const uint32_t local_here = chunk_local[chunk], local_next = chunk_local[chunk + 1];
    const uint32_t local_far = chunk_local[has_far ? chunk + 2 : chunk];
    const uint32_t runs = runs_at(chunk + 1, local_next);
    const int64_t u = (int64_t)runs - 1;
    if (next != key) return;                                         // the chunk's last run ends with it
    // The run goes on into a chunk that starts with its row and has no other run before it.  In an ascending list the row
    // alone says so; in a list that a caller brings in another order a row may come again in a later run, and the count keeps
    // any two runs from going on into one chunk.
    auto goes_on_into = [&](int64_t c, uint32_t first, uint32_t local) { return (first == key) & (runs_at(c, local) == runs); };
    if (k0 > 0 && before == key && goes_on_into(chunk, head, local_here)) return;          // it started in an earlier chunk
    if (u >= cap) return;
    const int64_t last_chunk = last_chunk_of_run(chunk, chunks, has_far && goes_on_into(chunk + 2, far, local_far),
                                                 [&](int64_t c) { return goes_on_into(c, keys[c * kChunk], chunk_local[c]); });
    if (long_runs != nullptr && last_chunk - chunk > kFoldLong) {
        if (lane_id() == 0) long_runs[atomicAdd(num_long, 1u)] = {(uint32_t)u, (uint32_t)(chunk + 1), (uint32_t)last_chunk};
        return;
    }
    typedef float Cols __attribute__((ext_vector_type(VL)));
    constexpr int kAhead = 128 / VL;             // carries in flight: the longest run's chain is latency-bound
    constexpr int kRest = 8;
    for (int col = lane_id() * VL; col < D; col += kWave * VL) {
        Cols acc = *reinterpret_cast<const Cols*>(row_grads + u * D + col);
        int64_t cc = chunk + 1;
        for (; cc + kAhead <= last_chunk + 1; cc += kAhead) {
            Cols part[kAhead];
#pragma unroll
            for (int j = 0; j < kAhead; ++j)
                part[j] = *reinterpret_cast<const Cols*>(carry + (cc + j) * D + col);
#pragma unroll
            for (int j = 0; j < kAhead; ++j) acc = acc + part[j];
        }
        for (; cc + 1 <= last_chunk; cc += kRest) {              // the rest, eight at a time, the last of them repeated
            Cols part[kRest];
#pragma unroll
            for (int j = 0; j < kRest; ++j) {
                const int64_t at = cc + j < last_chunk ? cc + j : last_chunk;
                part[j] = *reinterpret_cast<const Cols*>(carry + at * D + col);
            }
#pragma unroll
            for (int j = 0; j < kRest; ++j)
                if (cc + j <= last_chunk) acc = acc + part[j];
        }
        if (cc == last_chunk) acc = acc + *reinterpret_cast<const Cols*>(carry + cc * D + col);   // most runs: one carry
        *reinterpret_cast<Cols*>(row_grads + u * D + col) = acc;
    }
}

// The long runs, a block to 32 columns of one.  Four waves bring the carries to LDS, 256 at a time in two buffers, the
// next 256 in flight; the first wave adds them up, a column to a lane.  In LDS a column's carries lie one after the other,
// so that one read brings a lane four of them.  Bound by that chain of reads and adds, 15
// clocks a carry: 8.4 M lookups of 128 columns over one table, whose head row spans 8900 chunks, 55 us (all waves loading and
// then waiting for the adds 80 to 110); over four tables, 2100 chunks, both folds 35, the wave per chunk alone 65.
constexpr int kLongCols = 32;
constexpr int kLongLoads = 8;                                        // 16-byte loads a thread has in flight
constexpr int kLongRows = kLongLoads * kBlock * 4 / kLongCols;       // carries in a buffer
constexpr int kLongBlock = kWave + kBlock;
constexpr unsigned kLongGrid = 512;                                  // two blocks a CU, by their LDS

__global__ __launch_bounds__(kLongBlock) void bwd_fold_long_kernel(
    float* __restrict__ row_grads, int D, const float* __restrict__ carry, const LongRun* __restrict__ long_runs,
    const uint32_t* __restrict__ num_long)
{
    __shared__ __attribute__((aligned(16))) float cols[2][kLongCols][kLongRows + 4];      // 4 apart: the columns' banks, in reads and in writes
    const int slabs = (D + kLongCols - 1) / kLongCols;
    const int64_t items = (int64_t)*num_long * slabs;
    constexpr int kQuads = kLongCols / 4;                            // threads to a row
    constexpr int kPerLoad = kBlock / kQuads;                        // rows to a load of the four waves
    const bool loads = threadIdx.x >= kWave;                         // wave-uniform
    const int quad = threadIdx.x % kQuads;
    const int row0 = ((int)threadIdx.x - kWave) / kQuads;
    for (int64_t item = blockIdx.x; item < items; item += gridDim.x) {
        const LongRun r = long_runs[item / slabs];
        const int col0 = (int)(item % slabs) * kLongCols;
        const int count = (int)(r.last - r.first) + 1;
        const int my_col = col0 + quad * 4 < D ? col0 + quad * 4 : D - 4;        // D is a multiple of 4
        const float* const first = carry + (int64_t)r.first * D + my_col;
        f32x4 x[kLongLoads];
        auto load = [&](int from) {
#pragma unroll
            for (int j = 0; j < kLongLoads; ++j) {
                const int c = from + j * kPerLoad + row0;
                x[j] = load_stream(reinterpret_cast<const f32x4*>(first + (int64_t)(c < count ? c : count - 1) * D));
            }
        };
        auto store = [&](int buffer) {
#pragma unroll
            for (int j = 0; j < kLongLoads; ++j) {
#pragma unroll
                for (int i = 0; i < 4; ++i) cols[buffer][quad * 4 + i][j * kPerLoad + row0] = x[j][i];
            }
        };
        const int col = col0 + (int)threadIdx.x;
        const bool adds = threadIdx.x < kLongCols && col < D;
        float* const dst = row_grads + (int64_t)r.run * D + (adds ? col : 0);
        float acc = adds ? *dst : 0.0f;
        if (loads) {
            load(0);
            store(0);
            if (kLongRows < count) load(kLongRows);
        }
        __syncthreads();
        int buffer = 0;
        for (int from = 0; from < count; from += kLongRows, buffer ^= 1) {
            if (loads) {
                if (from + kLongRows < count) store(buffer ^ 1);
                if (from + 2 * kLongRows < count) load(from + 2 * kLongRows);
            } else if (adds) {
                // 32 at a time, the next 32 on their way while these are added (the scheduler would put the reads off)
                constexpr int kBatch = 32;
                static_assert(kLongRows % (2 * kBatch) == 0);
                const int n = count - from < kLongRows ? count - from : kLongRows;
                const f32x4* mine = reinterpret_cast<const f32x4*>(cols[buffer][threadIdx.x]);
                f32x4 f[2][kBatch / 4];
                auto read = [&](f32x4* to, int k) {
#pragma unroll
                    for (int j = 0; j < kBatch / 4; ++j) to[j] = mine[(k < kLongRows ? k : 0) / 4 + j];
                    __builtin_amdgcn_sched_barrier(0);
                };
                auto add = [&](const f32x4* these, int k) {
                    if (k + kBatch <= n) {                           // uniform
#pragma unroll
                        for (int j = 0; j < kBatch; ++j) acc = acc + these[j / 4][j % 4];
                    } else {
#pragma unroll
                        for (int j = 0; j < kBatch; ++j)
                            if (k + j < n) acc = acc + these[j / 4][j % 4];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                read(f[0], 0);
                for (int k = 0; k < n; k += 2 * kBatch) {
                    read(f[1], k + kBatch);
                    add(f[0], k);
                    read(f[0], k + 2 * kBatch);
                    add(f[1], k + kBatch);
                }
            }
            __syncthreads();
        }
        if (adds) *dst = acc;
    }
}

// variant 1: rows that receive atomic adds start at zero.
__global__ __launch_bounds__(kBlock) void bwd_zero_spilled_kernel(
    const uint32_t* __restrict__ keys, int64_t m, int64_t chunks,
    const uint32_t* __restrict__ block_base, const uint32_t* __restrict__ chunk_local,
    float* __restrict__ row_grads, int D, int64_t cap)
{
    const int64_t chunk = (int64_t)blockIdx.x * kWavesPerBlock + wave_id();
    if (chunk >= chunks || chunk == 0) return;
    const int64_t k0 = chunk * kChunk;
    if (keys[k0 - 1] != keys[k0]) return;
    const int64_t u = (int64_t)runs_before(block_base, chunk_local, chunk, chunks) - 1;
    if (u >= cap) return;
    for (int col = lane_id() * 4; col < D; col += kWave * 4)
        *reinterpret_cast<f32x4*>(row_grads + u * D + col) = f32x4{0.f, 0.f, 0.f, 0.f};
}

__global__ void bwd_empty_kernel(int64_t* num_unique) { *num_unique = 0; }

template <int LG>
static fs_status launch_singletons(fs_dtype dtype, const void* grad, int units, int D, const uint32_t* keys,
                                   const uint32_t* vals, int64_t m, int64_t chunks, uint32_t n, const uint32_t* block_base,
                                   const uint32_t* chunk_local, int64_t* uniq_rows, float* row_grads, int64_t cap,
                                   hipStream_t stream)
{
    const int64_t waves = chunks * kSinglesSplit;
    if ((waves + kWavesPerBlock - 1) / kWavesPerBlock > 0x7FFFFFFF) return FS_ERR_SIZE;
    const dim3 grid((unsigned)((waves + kWavesPerBlock - 1) / kWavesPerBlock), (unsigned)((units + LG - 1) / LG));
    const u32x4* g = static_cast<const u32x4*>(grad);
#define FS_SINGLE_LAUNCH(DT, EX)                                                                                   \
    FS_LAUNCH("bwd_singletons", (bwd_singletons_kernel<LG, DT, EX>), grid, dim3(kBlock), stream, g, units, D, keys,     \
              vals, m, chunks, n, block_base, chunk_local, uniq_rows, row_grads, cap)
    const bool exact = units == LG && LG >= 16;
    if (dtype == FS_F32) { if (exact) FS_SINGLE_LAUNCH(FS_F32, (LG >= 16)); else FS_SINGLE_LAUNCH(FS_F32, false); }
    else if (dtype == FS_F16) { if (exact) FS_SINGLE_LAUNCH(FS_F16, (LG >= 16)); else FS_SINGLE_LAUNCH(FS_F16, false); }
    else { if (exact) FS_SINGLE_LAUNCH(FS_BF16, (LG >= 16)); else FS_SINGLE_LAUNCH(FS_BF16, false); }
#undef FS_SINGLE_LAUNCH
    return FS_OK;
}

static fs_status launch_chunk_sums(fs_dtype dtype, const void* grad, int units, int D, const uint32_t* keys,
                                   const uint32_t* vals, int64_t m, int64_t chunks, uint32_t n, const uint32_t* block_base,
                                   const uint32_t* chunk_local, int64_t* uniq_rows, float* row_grads, int64_t cap,
                                   float* carry, int atomic, uint8_t* applied, int64_t* num_unique, int32_t* status, hipStream_t stream)
{
    const int slabs = (units + kSlabPieces - 1) / kSlabPieces;
    const int pieces = (units + slabs - 1) / slabs;
    if (chunks * slabs > 0x7FFFFFFF) return FS_ERR_SIZE;
    const dim3 grid((unsigned)(chunks * slabs));
    const size_t lds = (size_t)kChunk * pieces * 16;
    const u32x4* g = static_cast<const u32x4*>(grad);
#define FS_SUMS_LAUNCH(P, DT)                                                                                      \
    FS_LAUNCH_SMEM("bwd_chunk_sums", (bwd_chunk_sums_kernel<P, DT>), grid, dim3(kBlock), lds, stream, g, units, D, pieces, \
                   slabs, keys, vals, m, chunks, n, block_base, chunk_local, uniq_rows, row_grads, cap, carry, atomic, applied, \
                   num_unique, status)
#define FS_SUMS(DT)                                                                                                \
    if (pieces == kSlabPieces) FS_SUMS_LAUNCH(kSlabPieces, DT);                                                    \
    else FS_SUMS_LAUNCH(0, DT)
    if (dtype == FS_F32) { FS_SUMS(FS_F32); }
    else if (dtype == FS_F16) { FS_SUMS(FS_F16); }
    else { FS_SUMS(FS_BF16); }
#undef FS_SUMS
#undef FS_SUMS_LAUNCH
    return FS_OK;
}

template <int VB>
static fs_status launch_segreduce(fs_dtype dtype, const void* grad, int units, int D, const uint32_t* keys,
                             const uint32_t* vals, int64_t m, int64_t chunks, uint32_t n, const uint32_t* block_base,
                             const uint32_t* chunk_local, int64_t* uniq_rows, float* row_grads, int64_t cap,
                             float* carry, int atomic, uint8_t* applied, int64_t* num_unique, int32_t* status, hipStream_t stream)
{
    const dim3 grid((unsigned)((chunks + kWavesPerBlock - 1) / kWavesPerBlock), (unsigned)((units * 16 + kWave * VB - 1) / (kWave * VB)));
    const unsigned char* g = static_cast<const unsigned char*>(grad);
#define FS_SEG_LAUNCH(DT)                                                                                         \
    FS_LAUNCH("bwd_segreduce", (bwd_segreduce_kernel<VB, DT>), grid, dim3(kBlock), stream, g, units * 16, D, keys, vals, m,    \
              chunks, n, block_base, chunk_local, uniq_rows, row_grads, cap, carry, atomic, applied, num_unique, status)
    if (dtype == FS_F32) FS_SEG_LAUNCH(FS_F32);
    else if (dtype == FS_F16) FS_SEG_LAUNCH(FS_F16);
    else FS_SEG_LAUNCH(FS_BF16);
#undef FS_SEG_LAUNCH
    return FS_OK;
}

// fs_seq_grad_bwd_update's kernel for the rows looked up once (rows of up to 64 pieces).
template <int LG, int DT>
static fs_status launch_singletons_update_opt(int optimizer, const void* grad, const UpdateArgs& a, const uint32_t* keys,
                                              const uint32_t* vals, int64_t m, int64_t chunks, uint32_t n,
                                              const uint32_t* block_base, const uint32_t* chunk_local, int64_t* uniq_rows,
                                              int64_t cap, uint8_t* applied, hipStream_t stream)
{
    const int spread = update_spread(chunks);
    const int64_t waves = (chunks * kSinglesSplit) << spread;
    if ((waves + kWavesPerBlock - 1) / kWavesPerBlock > 0x7FFFFFFF) return FS_ERR_SIZE;
    const dim3 grid((unsigned)((waves + kWavesPerBlock - 1) / kWavesPerBlock));
    const u32x4* g = static_cast<const u32x4*>(grad);
#define FS_SU_LAUNCH(OPT, EX)                                                                                      \
    FS_LAUNCH("bwd_singletons_update", (bwd_singletons_update_kernel<LG, DT, OPT, EX>), grid, dim3(kBlock), stream, g, a, \
              keys, vals, m, chunks, n, block_base, chunk_local, uniq_rows, cap, applied, spread)
    const bool exact = a.units == LG;
    if (optimizer == FS_OPT_SGD) { if (exact) FS_SU_LAUNCH(FS_OPT_SGD, true); else FS_SU_LAUNCH(FS_OPT_SGD, false); }
    else if (optimizer == FS_OPT_ADAGRAD) { if (exact) FS_SU_LAUNCH(FS_OPT_ADAGRAD, true); else FS_SU_LAUNCH(FS_OPT_ADAGRAD, false); }
    else { if (exact) FS_SU_LAUNCH(FS_OPT_ADAGRAD_ROWWISE, true); else FS_SU_LAUNCH(FS_OPT_ADAGRAD_ROWWISE, false); }
#undef FS_SU_LAUNCH
    return FS_OK;
}

template <int LG>
static fs_status launch_singletons_update(fs_dtype dtype, int optimizer, const void* grad, const UpdateArgs& a,
                                          const uint32_t* keys, const uint32_t* vals, int64_t m, int64_t chunks, uint32_t n,
                                          const uint32_t* block_base, const uint32_t* chunk_local, int64_t* uniq_rows,
                                          int64_t cap, uint8_t* applied, hipStream_t stream)
{
    if (dtype == FS_F32)
        return launch_singletons_update_opt<LG, FS_F32>(optimizer, grad, a, keys, vals, m, chunks, n, block_base, chunk_local,
                                                        uniq_rows, cap, applied, stream);
    if (dtype == FS_F16)
        return launch_singletons_update_opt<LG, FS_F16>(optimizer, grad, a, keys, vals, m, chunks, n, block_base, chunk_local,
                                                        uniq_rows, cap, applied, stream);
    return launch_singletons_update_opt<LG, FS_BF16>(optimizer, grad, a, keys, vals, m, chunks, n, block_base, chunk_local,
                                                     uniq_rows, cap, applied, stream);
}

// Everything after the sort: (keys, vals) are the lookups in (row, position) order.
struct BwdScratch {
    uint32_t* chunk_local;
    uint32_t* block_base;
    float* carry;
    LongRun* long_runs;                          // null: no run can be long enough
    uint32_t* num_long;
};

static fs_status launch_fold(const uint32_t* keys, int64_t m, int64_t chunks, const BwdScratch& w, float* row_grads, int D,
                             int64_t cap, hipStream_t s)
{
    const dim3 grid((unsigned)((chunks + kWavesPerBlock - 1) / kWavesPerBlock));
#define FS_FOLD(VL)                                                                                                      \
    FS_LAUNCH("bwd_fold", bwd_fold_kernel<VL>, grid, dim3(kBlock), s, keys, m, chunks, w.block_base, w.chunk_local, row_grads, \
              D, cap, w.carry, w.long_runs, w.num_long)
    if (D <= kWave) FS_FOLD(1);
    else if (D <= 2 * kWave) FS_FOLD(2);                  // D is a multiple of 4: rows are whole 16-byte pieces
    else FS_FOLD(4);
#undef FS_FOLD
    if (w.long_runs != nullptr)
        FS_LAUNCH("bwd_fold_long", bwd_fold_long_kernel, dim3(kLongGrid), dim3(kLongBlock), s, row_grads, D, w.carry, w.long_runs, w.num_long);
    return FS_OK;
}

static fs_status bwd_after_sort(const void* grad_out, int64_t n, int D, fs_dtype dtype, int units,
                                const uint32_t* keys, const uint32_t* vals, int64_t m, int64_t R, int variant,
                                int64_t* uniq_rows, float* row_grads, int64_t cap_unique, int64_t* num_unique,
                                const BwdScratch& w, hipStream_t s, int32_t* dev_status,
                                const UpdateArgs* update = nullptr, int optimizer = 0, uint8_t* applied = nullptr)
{
    const int64_t chunks = (m + kChunk - 1) / kChunk;
    const int64_t blocks = heads_blocks(chunks);
    if (blocks == 1) {
        FS_LAUNCH("bwd_count_heads", bwd_count_heads_kernel<true>, dim3(1), dim3(kHeadsBlock), s, keys, vals, m, chunks,
                  (uint32_t)n, (uint32_t)R, w.chunk_local, w.block_base, cap_unique, num_unique, w.num_long, dev_status);
    } else {
        FS_LAUNCH("bwd_count_heads", bwd_count_heads_kernel<false>, dim3((unsigned)blocks), dim3(kHeadsBlock), s, keys, vals, m,
                  chunks, (uint32_t)n, (uint32_t)R, w.chunk_local, w.block_base, cap_unique, num_unique, w.num_long, dev_status);
        if (blocks > kSumBlocks)
            FS_LAUNCH("bwd_scan_blocks", bwd_scan_blocks_kernel, dim3(1), dim3(kScanBlock), s,
                  w.block_base, blocks, cap_unique, num_unique, dev_status);
    }
    const unsigned wave_grid = (unsigned)((chunks + kWavesPerBlock - 1) / kWavesPerBlock);
    if (variant == 1)
        FS_LAUNCH("bwd_zero_spilled", bwd_zero_spilled_kernel, dim3(wave_grid), dim3(kBlock), s,
                  keys, m, chunks, w.block_base, w.chunk_local, row_grads, D, cap_unique);
    fs_status rc;
    const bool few = chunks <= kSumsMaxChunks;
    if (few)
        rc = launch_chunk_sums(dtype, grad_out, units, D, keys, vals, m, chunks, (uint32_t)n, w.block_base, w.chunk_local,
                               uniq_rows, row_grads, cap_unique, w.carry, variant, applied, num_unique, dev_status, s);
    else if (units <= 16)
        rc = launch_segreduce<4>(dtype, grad_out, units, D, keys, vals, m, chunks, (uint32_t)n, w.block_base, w.chunk_local,
                            uniq_rows, row_grads, cap_unique, w.carry, variant, applied, num_unique, dev_status, s);
    else
        rc = launch_segreduce<8>(dtype, grad_out, units, D, keys, vals, m, chunks, (uint32_t)n, w.block_base, w.chunk_local,
                            uniq_rows, row_grads, cap_unique, w.carry, variant, applied, num_unique, dev_status, s);
    if (rc != FS_OK) return rc;
    if (update != nullptr) {                     // rows looked up once are updated in place, the others flagged for the step below
#define FS_SINGLE_UPDATE(LG)                                                                                    \
    rc = launch_singletons_update<LG>(dtype, optimizer, grad_out, *update, keys, vals, m, chunks, (uint32_t)n,    \
                                      w.block_base, w.chunk_local, uniq_rows, cap_unique, applied, s)
        if (units <= 1) FS_SINGLE_UPDATE(1);         // the group sizes of fs_sparse_update: the row-wise rule's sum of
        else if (units <= 2) FS_SINGLE_UPDATE(2);    // squares is taken over the group, and both must round alike
        else if (units <= 4) FS_SINGLE_UPDATE(4);
        else if (units <= 8) FS_SINGLE_UPDATE(8);
        else if (units <= 16) FS_SINGLE_UPDATE(16);
        else if (units <= 32) FS_SINGLE_UPDATE(32);
        else FS_SINGLE_UPDATE(64);
#undef FS_SINGLE_UPDATE
        if (rc != FS_OK) return rc;
        rc = launch_fold(keys, m, chunks, w, row_grads, D, cap_unique, s);
        if (rc != FS_OK) return rc;
        UpdateArgs rest = *update;               // the optimizer step on the rows whose gradient is in row_grads
        rest.uniq_rows = uniq_rows; rest.row_grads = row_grads; rest.cap = cap_unique; rest.num_unique = num_unique;
        rest.skip = applied;
        return sparse_update_launch(rest, dtype, optimizer, s);
    }
    if (!few) {
#define FS_SINGLE(LG)                                                                                           \
    rc = launch_singletons<LG>(dtype, grad_out, units, D, keys, vals, m, chunks, (uint32_t)n, w.block_base,       \
                               w.chunk_local, uniq_rows, row_grads, cap_unique, s)
        if (units <= 1) FS_SINGLE(1);
        else if (units <= 2) FS_SINGLE(2);
        else if (units <= 4) FS_SINGLE(4);
        else if (units <= 8) FS_SINGLE(8);
        else if (units <= 16) FS_SINGLE(16);
        else if (units <= 32) FS_SINGLE(32);
        else FS_SINGLE(64);
#undef FS_SINGLE
        if (rc != FS_OK) return rc;
    }
    if (variant == 0) return launch_fold(keys, m, chunks, w, row_grads, D, cap_unique, s);
    return FS_OK;
}

static BwdScratch take_bwd_scratch(Carver& ws, int64_t m, int D, int variant)
{
    const int64_t chunks = (m + kChunk - 1) / kChunk;
    const int64_t blocks = (chunks + kChunksPerBlock - 1) / kChunksPerBlock;
    BwdScratch w;
    w.chunk_local = ws.take<uint32_t>((size_t)chunks);
    w.block_base = ws.take<uint32_t>((size_t)blocks + 1);
    w.carry = ws.take<float>(variant == 0 ? (size_t)chunks * (size_t)D : 0);
    const bool may_long = variant == 0 && chunks * D > kFoldLongWork;
    w.long_runs = ws.take<LongRun>(may_long ? (size_t)(chunks / kFoldLong) + 1 : 0);      // each goes on into more than kFoldLong chunks, no two into one
    w.num_long = ws.take<uint32_t>(may_long ? 1 : 0);
    if (!may_long) { w.long_runs = nullptr; w.num_long = nullptr; }
    return w;
}

}  // namespace fs

extern "C" fs_status fs_seq_grad_bwd(
    const void* grad_out, int64_t n, int32_t D, fs_dtype dtype,
    const int64_t* rows, const int32_t* pos, int64_t j0, int64_t j1, int64_t R,
    int32_t variant,
    int64_t* uniq_rows, float* row_grads, int64_t cap_unique, int64_t* num_unique,
    void* workspace, size_t* workspace_bytes, void* stream, int32_t* dev_status)
{
    using namespace fs;
    if (!workspace_bytes) return FS_ERR_NULL;
    const int es = dtype_bytes(dtype);
    if (es == 0) return FS_ERR_DTYPE;
    if (R < 1 || R >= 4294967295LL || n < 0 || n >= (1LL << 31) || D < 1 || j0 < 0 || j0 > j1 || cap_unique < 0)
        return FS_ERR_SIZE;
    if (variant != 0 && variant != 1) return FS_ERR_CONFIG;
    const int64_t row_bytes = (int64_t)D * es;
    if (row_bytes % 16 != 0) return FS_ERR_ALIGN;
    const int64_t m = j1 - j0;
    if (m >= (1LL << 31)) return FS_ERR_SIZE;
    const int units = (int)(row_bytes / 16);

    Carver ws(workspace);
    SortPair* pairs_a = ws.take<SortPair>((size_t)m);
    SortPair* pairs_b = ws.take<SortPair>((size_t)m);
    char* sort_scratch = ws.take<char>(radix_sort_scratch_bytes(m));
    const BwdScratch scratch = take_bwd_scratch(ws, m, (int)D, (int)variant);
    if (!workspace) { *workspace_bytes = ws.used; return FS_OK; }
    if (*workspace_bytes < ws.used || (reinterpret_cast<uintptr_t>(workspace) & 255)) return FS_ERR_WORKSPACE;
    if (!num_unique) return FS_ERR_NULL;

    hipStream_t s = static_cast<hipStream_t>(stream);
    if (m == 0) {
        FS_LAUNCH("bwd_empty", bwd_empty_kernel, dim3(1), dim3(1), s, num_unique);
        return FS_OK;
    }
    if (!grad_out || !rows || !pos) return FS_ERR_NULL;
    if (cap_unique > 0 && (!uniq_rows || !row_grads)) return FS_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(grad_out) | reinterpret_cast<uintptr_t>(row_grads)) & 15) return FS_ERR_ALIGN;

    SortJob job;                                 // the sort's first pass reads (row, pos) itself
    job.rows = rows + j0; job.pos = pos + j0; job.R = R; job.n = n; job.status = dev_status;
    job.pairs_a = pairs_a; job.pairs_b = pairs_b;
    job.m_max = m; job.key_bits = bits_for((uint64_t)(R - 1));
    job.scratch = sort_scratch; job.stream = s;
    // rows and positions apart in the buffer that the last pass does not read
    uint32_t* keys = reinterpret_cast<uint32_t*>((radix_sort_passes(job.key_bits) & 1) ? pairs_a : pairs_b);
    uint32_t* vals = keys + m;
    job.keys_out = keys; job.vals_out = vals;
    fs_status rc = radix_sort(job);
    if (rc != FS_OK) return rc;
    return bwd_after_sort(grad_out, n, (int)D, dtype, units, keys, vals, m, R, (int)variant, uniq_rows, row_grads,
                          cap_unique, num_unique, scratch, s, dev_status);
}

extern "C" fs_status fs_sort_lookups(
    const int64_t* rows, const int32_t* pos, int64_t j0, int64_t j1, int64_t R, int64_t n,
    uint32_t* sorted_rows, uint32_t* sorted_pos,
    void* workspace, size_t* workspace_bytes, void* stream, int32_t* dev_status)
{
    using namespace fs;
    if (!workspace_bytes) return FS_ERR_NULL;
    if (R < 1 || R >= 4294967295LL || n < 0 || n >= (1LL << 31) || j0 < 0 || j0 > j1) return FS_ERR_SIZE;
    const int64_t m = j1 - j0;
    if (m >= (1LL << 31)) return FS_ERR_SIZE;
    const int key_bits = bits_for((uint64_t)(R - 1));
    // What is needed for any R is one buffer and the tables: the caller's arrays can be the other buffer.  A second one is
    // asked for where a middle pass is faster with it, and used if it is there (three passes, us, without : with: 262 k
    // pairs 36.9 : 35.8, 1 M 54.4 : 50.7, 4.2 M 105.8 : 102.5, 15.7 M 279.4 : 279.4; where pairs lie apart anyway no gain).
    Carver ws(workspace);
    SortPair* pairs_a = ws.take<SortPair>((size_t)m);
    char* sort_scratch = ws.take<char>(radix_sort_scratch_bytes(m));
    const size_t needed = ws.used;
    SortPair* pairs_b = nullptr;
    if (radix_sort_passes(key_bits) > 2 && m < kSortSplitFrom) pairs_b = ws.take<SortPair>((size_t)m);
    if (!workspace) { *workspace_bytes = ws.used; return FS_OK; }
    if (*workspace_bytes < needed || (reinterpret_cast<uintptr_t>(workspace) & 255)) return FS_ERR_WORKSPACE;
    if (*workspace_bytes < ws.used) pairs_b = nullptr;
    if (m == 0) return FS_OK;
    if (!rows || !pos || !sorted_rows || !sorted_pos) return FS_ERR_NULL;
    SortJob job;
    job.rows = rows + j0; job.pos = pos + j0; job.R = R; job.n = n; job.status = dev_status;
    job.pairs_a = pairs_a; job.pairs_b = pairs_b;
    job.keys_out = sorted_rows; job.vals_out = sorted_pos;
    job.m_max = m; job.key_bits = key_bits;
    job.scratch = sort_scratch; job.stream = static_cast<hipStream_t>(stream);
    return radix_sort(job);
}

extern "C" fs_status fs_seq_grad_bwd_sorted(
    const void* grad_out, int64_t n, int32_t D, fs_dtype dtype,
    const uint32_t* sorted_rows, const uint32_t* sorted_pos, int64_t m, int64_t R,
    int32_t variant,
    int64_t* uniq_rows, float* row_grads, int64_t cap_unique, int64_t* num_unique,
    void* workspace, size_t* workspace_bytes, void* stream, int32_t* dev_status)
{
    using namespace fs;
    if (!workspace_bytes) return FS_ERR_NULL;
    const int es = dtype_bytes(dtype);
    if (es == 0) return FS_ERR_DTYPE;
    if (R < 1 || R >= 4294967295LL || n < 0 || n >= (1LL << 31) || D < 1 || m < 0 || m >= (1LL << 31) || cap_unique < 0)
        return FS_ERR_SIZE;
    if (variant != 0 && variant != 1) return FS_ERR_CONFIG;
    const int64_t row_bytes = (int64_t)D * es;
    if (row_bytes % 16 != 0) return FS_ERR_ALIGN;
    const int units = (int)(row_bytes / 16);
    Carver ws(workspace);
    const BwdScratch scratch = take_bwd_scratch(ws, m, (int)D, (int)variant);
    if (!workspace) { *workspace_bytes = ws.used; return FS_OK; }
    if (*workspace_bytes < ws.used || (reinterpret_cast<uintptr_t>(workspace) & 255)) return FS_ERR_WORKSPACE;
    if (!num_unique) return FS_ERR_NULL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (m == 0) {
        FS_LAUNCH("bwd_empty", bwd_empty_kernel, dim3(1), dim3(1), s, num_unique);
        return FS_OK;
    }
    if (!grad_out || !sorted_rows || !sorted_pos) return FS_ERR_NULL;
    if (cap_unique > 0 && (!uniq_rows || !row_grads)) return FS_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(grad_out) | reinterpret_cast<uintptr_t>(row_grads)) & 15) return FS_ERR_ALIGN;
    return bwd_after_sort(grad_out, n, (int)D, dtype, units, sorted_rows, sorted_pos, m, R, (int)variant, uniq_rows,
                          row_grads, cap_unique, num_unique, scratch, s, dev_status);
}

extern "C" fs_status fs_seq_grad_bwd_update(
    const void* grad_out, int64_t n, int32_t D, fs_dtype dtype,
    const uint32_t* sorted_rows, const uint32_t* sorted_pos, int64_t m, int64_t R,
    void* weights, int32_t optimizer, float lr, float eps, float* state,
    void* store, const int32_t* slot_of_row, int64_t k,
    int64_t* uniq_rows, float* row_grads, int64_t cap_unique, int64_t* num_unique,
    void* workspace, size_t* workspace_bytes, void* stream, int32_t* dev_status)
{
    using namespace fs;
    if (!workspace_bytes) return FS_ERR_NULL;
    const int es = dtype_bytes(dtype);
    if (es == 0) return FS_ERR_DTYPE;
    if (R < 1 || R >= 4294967295LL || n < 0 || n >= (1LL << 31) || D < 1 || m < 0 || m >= (1LL << 31) || cap_unique < 0 ||
        k < 0 || k >= (1LL << 31))
        return FS_ERR_SIZE;
    if (optimizer != FS_OPT_SGD && optimizer != FS_OPT_ADAGRAD && optimizer != FS_OPT_ADAGRAD_ROWWISE) return FS_ERR_CONFIG;
    const int64_t row_bytes = (int64_t)D * es;
    if (row_bytes % 16 != 0) return FS_ERR_ALIGN;
    const int units = (int)(row_bytes / 16);
    Carver ws(workspace);
    const BwdScratch scratch = take_bwd_scratch(ws, m, (int)D, 0);
    uint8_t* applied = ws.take<uint8_t>((size_t)cap_unique);
    if (!workspace) { *workspace_bytes = ws.used; return FS_OK; }
    if (*workspace_bytes < ws.used || (reinterpret_cast<uintptr_t>(workspace) & 255)) return FS_ERR_WORKSPACE;
    if (!num_unique || !weights) return FS_ERR_NULL;
    if (optimizer != FS_OPT_SGD && !state) return FS_ERR_NULL;
    if ((store != nullptr) != (slot_of_row != nullptr)) return FS_ERR_NULL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (m == 0) {
        FS_LAUNCH("bwd_empty", bwd_empty_kernel, dim3(1), dim3(1), s, num_unique);
        return FS_OK;
    }
    if (!grad_out || !sorted_rows || !sorted_pos) return FS_ERR_NULL;
    if (cap_unique > 0 && (!uniq_rows || !row_grads)) return FS_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(grad_out) | reinterpret_cast<uintptr_t>(row_grads) | reinterpret_cast<uintptr_t>(weights) |
         reinterpret_cast<uintptr_t>(store) | reinterpret_cast<uintptr_t>(state)) & 15)
        return FS_ERR_ALIGN;
    UpdateArgs a;
    a.weights = static_cast<u32x4*>(weights); a.R = R; a.units = units; a.D = D;
    a.uniq_rows = uniq_rows; a.row_grads = row_grads; a.cap = cap_unique; a.num_unique = num_unique;
    a.lr = lr; a.eps = eps; a.state = state;
    a.store = static_cast<u32x4*>(store); a.slot_of_row = slot_of_row; a.k = k; a.status = dev_status;
    a.skip = nullptr;
    if (units > kWave || cap_unique == 0) {
        // rows of more than 64 pieces (or no room for any row): the two steps one after the other
        const fs_status rc = bwd_after_sort(grad_out, n, (int)D, dtype, units, sorted_rows, sorted_pos, m, R, 0, uniq_rows,
                                            row_grads, cap_unique, num_unique, scratch, s, dev_status);
        if (rc != FS_OK || cap_unique == 0) return rc;
        return sparse_update_launch(a, dtype, optimizer, s);
    }
    return bwd_after_sort(grad_out, n, (int)D, dtype, units, sorted_rows, sorted_pos, m, R, 0, uniq_rows, row_grads,
                          cap_unique, num_unique, scratch, s, dev_status, &a, optimizer, applied);
}
