// Stable sort of up to 2^19 small keys by node: the contributors of a
// gradient, or the deliveries of an iteration, by the node they go to.
//
// Two counting passes over half of the key's bits each (LSD), in three
// launches after the caller's own key kernel, which counts the first digit of
// its tile (sort_keys_tile): scatter, count, scatter.  A scatter workgroup
// adds up the tiles' counts itself instead of waiting for a scan's launch.
// (Counting the second digit in the first scatter, with atomics at the places
// it writes to, saved a launch and cost 20 us.)  The library sort this
// replaces took nine launches of 6 us at 132,000 keys of 15 bits and eight of
// 5 us at 20,000.  Up to the limit this sort is the faster one (a training step
// with it / with the library's, 64 slots: 58,500 keys 322 / 337 us, 136,500
// 356 / 385, 253,500 454 / 516, 507,000 660 / 742); past it the counts that
// each scatter workgroup adds up, tiles times bins, would grow with the square
// of the keys, and the library's takes over, as for keys of more than 20 bits.
#pragma once

#include <algorithm>

#include "common.h"

namespace tgm {

constexpr int kSortTile = 2048;          // keys of a workgroup (256 threads)
constexpr int kSortMax = 1 << 19;        // keys at most (256 tiles)
constexpr int kSortDigit = 10;           // bits of a digit at most

struct SortBuffers {
    int64_t capacity = 0;                // keys
    int bits = 0;                        // of the largest key
    uint32_t *keys[2] = {nullptr, nullptr};
    int32_t *vals[2] = {nullptr, nullptr};
    uint32_t *out_keys = nullptr;
    int32_t *out_vals = nullptr;
    int32_t *hist[2] = {nullptr, nullptr};   // [tiles][bins of the digit]
    char *tmp = nullptr;                 // the library sort's
    size_t tmp_bytes = 0;
};

// The digits of a sort of n keys below 2^bits
struct SortPlan {
    int64_t n;
    int bits0, bits1, tiles;
    uint32_t *keys[2], *out_keys;
    int32_t *vals[2], *out_vals, *hist[2];
};

// Bits that hold the keys 0 .. last
inline int key_bits(int64_t last)
{
    int bits = 1;
    while (bits < 31 && (int64_t(1) << bits) <= last)
        ++bits;
    return bits;
}

// Bytes of the library sort's work space for up to `capacity` keys of `bits`
// bits (0: never taken)
tgm_status_t sort_tmp_bytes(SortBuffers *b);
// Space for sorts of up to `capacity` keys 0 .. last, through the caller's
// alloc(T **, count) -> bool (a create call's)
template <class A>
tgm_status_t sort_create(SortBuffers *b, int64_t capacity, int64_t last, A alloc)
{
    b->capacity = std::max<int64_t>(capacity, 1);
    b->bits = key_bits(last);
    const int64_t n = b->capacity, tiles = cdiv(std::min<int64_t>(n, kSortMax), kSortTile);
    bool ok = alloc(&b->out_keys, n) && alloc(&b->out_vals, n);
    for (int k = 0; k < 2; ++k)
        ok = ok && alloc(&b->keys[k], n) && alloc(&b->vals[k], n) &&
             alloc(&b->hist[k], tiles << kSortDigit);
    if (!ok)
        return TGM_ENOMEM;
    const tgm_status_t st = sort_tmp_bytes(b);
    if (st != TGM_OK)
        return st;
    return b->tmp_bytes == 0 || alloc(&b->tmp, (int64_t)b->tmp_bytes) ? TGM_OK : TGM_ENOMEM;
}
void sort_destroy(SortBuffers *b);
// keys[0][i] (and, where sort_plan's tiles is positive, hist[0]) must be
// written by sort_keys_tile on sort_tiles(n) workgroups of 256 threads before
// sort_launch; value i is i.  Sorted: out_keys, out_vals.
SortPlan sort_plan(const SortBuffers &b, int64_t n);
inline int64_t sort_tiles(int64_t n) { return cdiv(n, kSortTile); }
tgm_status_t sort_launch(const SortBuffers &b, const SortPlan &p, hipStream_t s);

// One workgroup's tile of keys: key(i) for i < n, their first digit counted.
// count: 2^kSortDigit ints of LDS.
template <class F>
__device__ __forceinline__ void sort_keys_tile(const SortPlan &p, int tile, int32_t *count,
                                               F key)
{
    const int bins0 = 1 << p.bits0, tid = threadIdx.x;
    if (p.tiles > 0) {
        for (int d = tid; d < bins0; d += 256)
            count[d] = 0;
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < kSortTile / 256; ++u) {
        const int64_t i = (int64_t)tile * kSortTile + u * 256 + tid;
        if (i < p.n) {
            const uint32_t k = key(i);
            p.keys[0][i] = k;
            if (p.tiles > 0)
                atomicAdd(&count[k & (bins0 - 1)], 1);
            else
                p.vals[0][i] = (int32_t)i;
        }
    }
    if (p.tiles > 0) {
        __syncthreads();
        for (int d = tid; d < bins0; d += 256)
            p.hist[0][(int64_t)tile * bins0 + d] = count[d];
    }
}

}  // namespace tgm
