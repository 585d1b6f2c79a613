#include <hip/hip_runtime.h>

#include <hipcub/hipcub.hpp>

#include <algorithm>

#include "sort.h"

using namespace tgm;

namespace {

// Scatter of one digit, one tile of keys per workgroup, stable.  base[w][d]
// is the place of wavefront w's first key with digit d: the keys of smaller
// digits anywhere, then those of digit d in earlier tiles and in earlier
// wavefronts of this one.  A wavefront takes its 512 keys 64 at a time; equal
// digits among the 64 find their order with one ballot per digit bit.  Bound
// by latency (the counts of all tiles, then eight rounds of ballots and LDS).
template <int PASS>
__global__ __launch_bounds__(256) void k_sort_scatter(SortPlan p)
{
    constexpr int kBins = 1 << kSortDigit;
    __shared__ int32_t base[4][kBins];
    __shared__ int32_t scan[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tile = blockIdx.x;
    const int bits = PASS ? p.bits1 : p.bits0, shift = PASS ? p.bits0 : 0;
    const int bins = 1 << bits, per = (bins + 255) / 256;
    const int32_t *hist = p.hist[PASS];
    for (int d = tid; d < 4 * bins; d += 256)
        base[d / bins][d % bins] = 0;
    __syncthreads();
    // this tile's keys, and their counts by wavefront
    const int64_t i0 = (int64_t)tile * kSortTile + wave * (kSortTile / 4);
    uint32_t key[kSortTile / 256];
    int32_t val[kSortTile / 256];
#pragma unroll
    for (int u = 0; u < kSortTile / 256; ++u) {
        const int64_t i = i0 + u * kWave + lane, at = min(i, p.n - 1);
        key[u] = PASS ? p.keys[1][at] : p.keys[0][at];
        val[u] = PASS ? p.vals[1][at] : (int32_t)i;
    }
#pragma unroll
    for (int u = 0; u < kSortTile / 256; ++u)
        if (i0 + u * kWave + lane < p.n)
            atomicAdd(&base[wave][(key[u] >> shift) & (bins - 1)], 1);
    // thread t's digits are t per .. t per + per - 1: keys of each anywhere
    // and in earlier tiles
    int32_t all[kBins / 256], before[kBins / 256], mine = 0;
#pragma unroll
    for (int e = 0; e < kBins / 256; ++e) {
        all[e] = before[e] = 0;
        const int d = tid * per + e;
        if (e < per && d < bins) {
            // (loads in flight together: one after the other they took most
            // of the launch)
            constexpr int kAhead = 16;
            for (int t = 0; t < p.tiles; t += kAhead) {
                int32_t x[kAhead];
#pragma unroll
                for (int v = 0; v < kAhead; ++v)
                    x[v] = hist[(int64_t)min(t + v, p.tiles - 1) * bins + d];
#pragma unroll
                for (int v = 0; v < kAhead; ++v) {
                    all[e] += t + v < p.tiles ? x[v] : 0;
                    before[e] += t + v < tile ? x[v] : 0;
                }
            }
            mine += all[e];
        }
    }
    int32_t run = mine;   // inclusive scan over the threads, wavefront by wavefront
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t x = __shfl_up(run, o, kWave);
        run += lane >= o ? x : 0;
    }
    if (lane == 63)
        scan[wave] = run;
    __syncthreads();
    run -= mine;
    for (int w = 0; w < wave; ++w)
        run += scan[w];
#pragma unroll
    for (int e = 0; e < kBins / 256; ++e) {
        const int d = tid * per + e;
        if (e < per && d < bins) {
            int32_t at = run + before[e];
            run += all[e];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int32_t c = base[w][d];
                base[w][d] = at;
                at += c;
            }
        }
    }
    __syncthreads();
    const uint64_t below = (uint64_t(1) << lane) - 1;
#pragma unroll
    for (int u = 0; u < kSortTile / 256; ++u) {
        const bool on = i0 + u * kWave + lane < p.n;
        const uint32_t d = (key[u] >> shift) & (bins - 1);
        uint64_t same = __ballot(on);
        for (int b = 0; b < bits; ++b) {
            const uint64_t set = __ballot((d >> b) & 1);
            same &= (d >> b) & 1 ? set : ~set;
        }
        // every lane reads its digit's place before the first of a group
        // moves it on (one wavefront: its LDS accesses stay in order)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int32_t first = base[wave][d];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (on) {
            const int32_t at = first + __popcll(same & below);
            if ((same & below) == 0)
                base[wave][d] = first + __popcll(same);
            if (PASS) {
                p.out_keys[at] = key[u];
                p.out_vals[at] = val[u];
            } else {
                p.keys[1][at] = key[u];
                p.vals[1][at] = val[u];
            }
        }
    }
}

// The second digit's counts of each tile
__global__ __launch_bounds__(256) void k_sort_count(SortPlan p)
{
    __shared__ int32_t count[1 << kSortDigit];
    const int tid = threadIdx.x, bins = 1 << p.bits1;
    const int64_t i0 = (int64_t)blockIdx.x * kSortTile + tid;
    uint32_t key[kSortTile / 256];
#pragma unroll
    for (int u = 0; u < kSortTile / 256; ++u)
        key[u] = p.keys[1][min(i0 + u * 256, p.n - 1)];
    for (int d = tid; d < bins; d += 256)
        count[d] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSortTile / 256; ++u)
        if (i0 + u * 256 < p.n)
            atomicAdd(&count[(key[u] >> p.bits0) & (bins - 1)], 1);
    __syncthreads();
    for (int d = tid; d < bins; d += 256)
        p.hist[1][(int64_t)blockIdx.x * bins + d] = count[d];
}

}  // namespace

SortPlan tgm::sort_plan(const SortBuffers &b, int64_t n)
{
    SortPlan p;
    p.n = n;
    p.bits0 = (b.bits + 1) / 2;
    p.bits1 = std::max(1, b.bits - p.bits0);
    p.tiles = n <= kSortMax && b.bits <= 2 * kSortDigit ? (int)sort_tiles(n) : 0;
    for (int k = 0; k < 2; ++k) {
        p.keys[k] = b.keys[k];
        p.vals[k] = b.vals[k];
        p.hist[k] = b.hist[k];
    }
    p.out_keys = b.out_keys;
    p.out_vals = b.out_vals;
    return p;
}

tgm_status_t tgm::sort_tmp_bytes(SortBuffers *b)
{
    b->tmp_bytes = 0;
    if (b->capacity <= kSortMax && b->bits <= 2 * kSortDigit)
        return TGM_OK;
    // the library sort picks its method by size: room for each size it may get
    const int64_t least = b->bits > 2 * kSortDigit ? 1 : kSortMax;
    for (int64_t n = b->capacity; n >= least; n /= 2) {
        size_t bytes = 0;
        if (hipcub::DeviceRadixSort::SortPairs(nullptr, bytes, b->keys[0], b->out_keys,
                                               b->vals[0], b->out_vals, (int)n, 0,
                                               b->bits) != hipSuccess)
            return TGM_EDEVICE;
        b->tmp_bytes = std::max(b->tmp_bytes, std::max<size_t>(bytes, 1));
    }
    return TGM_OK;
}

void tgm::sort_destroy(SortBuffers *b)
{
    for (int k = 0; k < 2; ++k) {
        (void)hipFree(b->keys[k]);
        (void)hipFree(b->vals[k]);
        (void)hipFree(b->hist[k]);
    }
    (void)hipFree(b->out_keys);
    (void)hipFree(b->out_vals);
    (void)hipFree(b->tmp);
}

tgm_status_t tgm::sort_launch(const SortBuffers &b, const SortPlan &p, hipStream_t s)
{
    if (p.n <= 0)
        return TGM_OK;
    if (p.n > b.capacity)
        return TGM_ESIZE;
    if (p.tiles == 0) {
        size_t bytes = b.tmp_bytes;
        TGM_HIP(hipcub::DeviceRadixSort::SortPairs(b.tmp, bytes, b.keys[0], b.out_keys, b.vals[0],
                                                   b.out_vals, (int)p.n, 0, b.bits, s));
        return TGM_OK;
    }
    TGM_LAUNCH((k_sort_scatter<0>), dim3((unsigned)p.tiles), dim3(256), 0, s, p);
    TGM_LAUNCH(k_sort_count, dim3((unsigned)p.tiles), dim3(256), 0, s, p);
    TGM_LAUNCH((k_sort_scatter<1>), dim3((unsigned)p.tiles), dim3(256), 0, s, p);
    return TGM_OK;
}
