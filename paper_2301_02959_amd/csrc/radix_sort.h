// Stable LSD radix sort of (uint32 key, uint32 value) pairs, used by the backward
// (key = row, value = position) and by the replication plan (key = inverted count,
// value = row).  Hand-written for 64-lane waves: see radix_sort.hip.
#pragma once

#include "fs_common.h"

namespace fs {

constexpr int kSortMaxDigitBits = 10;
constexpr int kSortPairsBits = 5;            // the shortest digit by which pairs are sorted
static_assert(kSortPairsBits <= (kSortMaxDigitBits + 1) / 2);

// A pair between two passes: [0] the key, [1] the value.  Side by side they leave the scatter as one store and a
// digit's run is twice as long as in an array of its own (very large sorts from `rows` keep them apart, in the same buffers).
typedef u32x2 SortPair;

struct SortJob {
    // Where the first pass reads its pairs.
    //   rows == nullptr: pairs_a holds them.
    //   rows != nullptr: pair q is (uint32) rows[q], (uint32) pos[q], validated on the fly
    //                    (row outside [0, R) -> 0, pos outside [0, n) -> 0, FS_DEV_BAD_ID into *status).
    const int64_t* rows = nullptr;
    const int32_t* pos = nullptr;
    int64_t R = 0;
    int64_t n = 0;
    int32_t* status = nullptr;
    // Buffers of m_max pairs; the passes go from one to the other, the first pass of `rows` into pairs_a.  Without pairs_b
    // (sorts of `rows` only) keys_out and vals_out serve as the other one, from the first pass on if their number is odd.
    SortPair* pairs_a = nullptr;
    SortPair* pairs_b = nullptr;
    // Where the last pass writes keys and values apart; null: as pairs, into the buffer whose turn it is.  They may
    // lie in the buffer that the last pass does not read: pairs_a after an odd number of passes from `rows`, else pairs_b.
    uint32_t* keys_out = nullptr;
    uint32_t* vals_out = nullptr;
    // Number of pairs: *m_dev if m_dev != nullptr (device memory, read by the kernels; at most m_max) else m_max.
    int64_t m_max = 0;
    const int64_t* m_dev = nullptr;
    int key_bits = 32;               // the sort is by the low key_bits bits of the key; of pairs, by at least kSortPairsBits
    // A device word with every bit set in which two keys differ (or null).  Passes above its highest set bit copy
    // nothing and return at once; the result is then where the last pass that ran left it, which only the device knows:
    // sort_result_in_b below.  For 32-bit keys that came in pairs_a; keys_out must be null.
    const uint32_t* varying = nullptr;
    // With `varying`, the bits of the first two passes; two more share the rest.  Without it the bits are spread evenly
    // over as few passes as possible.
    int first_bits = kSortMaxDigitBits;
    void* scratch = nullptr;         // radix_sort_scratch_bytes(m_max) bytes
    hipStream_t stream = nullptr;
};

// From this many pairs on they lie apart between passes too.  Side by side the scatter's stores are half as many and its
// runs twice as long, but the count reads 8 bytes for a key of 4, which costs more where a pass no longer fits the 256 MB
// memory-side cache.  Side by side : apart, us, rows of 27 bits: 8.4 M 170 : 175, 15.7 M 278 : 286, 30 M 534 : 532,
// 72 M 1367 : 1310; of 29 bits 182 : 190, 300 : 317, 572 : 587, 1464 : 1443; of 22 bits 162 : 161, 261 : 263, 494 : 480, 1236 : 1137.
constexpr int64_t kSortSplitFrom = (int64_t)1 << 25;

// Where pairs lie before or after a pass: side by side, or (pairs == nullptr) apart.
struct SortPlace {
    SortPair* pairs;
    uint32_t* keys;
    uint32_t* vals;
};

// Where pass k (of `passes`) leaves its pairs; k = -1: where those lie that do not come from `rows`.
inline SortPlace sort_place_after(const SortJob& job, int passes, int k)
{
    if (k < 0) return {job.pairs_a, nullptr, nullptr};
    const bool out = k == passes - 1 || (job.pairs_b == nullptr && (passes - 1 - k) % 2 == 0);
    if (out && job.keys_out != nullptr) return {nullptr, job.keys_out, job.vals_out};
    SortPair* const buffer = job.pairs_b == nullptr || (k % 2 == 0) == (job.rows != nullptr) ? job.pairs_a : job.pairs_b;
    if (job.m_dev != nullptr || job.m_max < kSortSplitFrom) return {buffer, nullptr, nullptr};
    uint32_t* const words = reinterpret_cast<uint32_t*>(buffer);
    return {nullptr, words, words + job.m_max};
}

// Number of passes over keys of key_bits bits.
inline int radix_sort_passes(int key_bits)
{
    if (key_bits < 1) key_bits = 1;
    if (key_bits > 32) key_bits = 32;
    return (key_bits + kSortMaxDigitBits - 1) / kSortMaxDigitBits;
}

// Bits of pass k's digit, the bits below `shift` done.  They are spread evenly over the passes: 27 bits -> 9, 9, 9; where
// passes can turn out idle the digits are fixed: 32 bits -> 10, 10, 6, 6 or 8, 8, 8, 8.  A pass after the first has at least
// kSortPairsBits (11 bits -> 6, 5).
inline int sort_digit_bits(const SortJob& job, int key_bits, int passes, int k, int shift)
{
    const int even = (key_bits - shift + (passes - k) - 1) / (passes - k);
    return job.varying != nullptr && k < 2 ? job.first_bits : even;
}

// Scratch the sort needs for up to m_max pairs (beyond the two buffers).
size_t radix_sort_scratch_bytes(int64_t m_max);

fs_status radix_sort(const SortJob& job);

#ifdef __HIPCC__
// Whether a sort with `varying` and `first_bits` left its result in pairs_b.
__device__ __forceinline__ bool sort_result_in_b(uint32_t varying, int first_bits)
{
    const int bits = varying == 0 ? 1 : 32 - __builtin_clz(varying);
    const int passes = bits <= first_bits ? 1 : bits <= 2 * first_bits ? 2 : bits <= 16 + first_bits ? 3 : 4;
    return passes & 1;
}
#endif

}  // namespace fs
