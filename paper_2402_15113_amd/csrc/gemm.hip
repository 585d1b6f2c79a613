// Grouped fp32 GEMM on the matrix cores: one launch computes several
// independent products C = op(A) op(B), so that the many small products of a
// training step or of APAN's update share a grid (a launch costs 2.5 us and
// most of these products have fewer tiles than the chip has CUs).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"

using namespace tgm;

namespace {

// A workgroup of 4 wavefronts takes a tile of 64 rows and 16 NB columns, NB =
// 7 or 4; wavefront w holds rows 16 w .. 16 w + 15 of it in NB accumulators.
// 112 columns because most outputs here are M = 100 (or 2M = 200) wide, which
// 64-wide tiles would pad to 128 (or 256); the launcher takes the width with
// less padding.  The k range goes in steps of 32 through two LDS buffers,
// one barrier per step, loads two steps ahead.  Operands load 16 bytes at a time along their
// contiguous direction (the hardware takes them at any 4-byte alignment, so
// odd leading dimensions need no other path) from a scalar base and a
// fixed per-thread offset, so a step's 56 MFMAs per wavefront come with few vector
// instructions: with 4-byte loads and recomputed addresses the address
// arithmetic took longer than the products.
//
// Precision.  With a transposed A (the weight gradients, whose reductions run
// over thousands of rows that nearly cancel) the accumulators are added to a
// second set every 128 k: a chain of fp32 additions loses accuracy in
// proportion to its length, and 512-long ones doubled the error of a training
// step's gradient (2.0e-6 relative, against 0.9e-6 with 240-long ones).
//
// Edges.  Rows past m and columns past n of a tile are never stored: a
// k-contiguous operand clamps its row, and an operand contiguous along the
// tile's columns moves its last vector back to end at the edge and stores it
// at the column it came from.  Only the reduction's tail needs zeros, and
// only its last step (or a tile narrower than one vector) loads by elements.
constexpr int kTK = 32, kLdK = kTK + 4;
constexpr int kTiles16 = 64, kTiles32 = 160;   // 64-row tiles up to which 16 or 32 rows are taken
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

struct GemmGroup {
    int n;
    GemmProb p[kGemmGroup];
};

// One operand's tile: COLS rows (of A) or columns (of B) by kTK of k.
// KC: contiguous along k (element (c, k) at X[c ld + k]), else along c
// (X[k ld + c]).  LDS layout [c][k] for KC, [k][c] otherwise.  TH threads
// take NV vectors each, PU rows (KC: of the tile, else of k) apart; a load's
// address is a scalar base that advances by steps plus a fixed 32-bit offset.
template <bool KC, int COLS>
struct Operand {
    static constexpr int PER = KC ? kTK / 4 : COLS / 4;   // vectors per row
    static constexpr int TH = COLS == 112 ? 224 : COLS == 16 ? 128 : 256;
    static constexpr int PU = TH / PER;
    static constexpr int NV = (KC ? COLS : kTK) / PU;
    static constexpr int kLd = KC ? kLdK : COLS + 4;
    static constexpr int kFloats = (KC ? COLS : kTK) * kLd;
    static_assert(TH % PER == 0 && PU * NV == (KC ? COLS : kTK), "");
    const float *base;
    int64_t step;
    uint32_t off[NV];
    int at;
    bool on, narrow;
    f4 v[2][NV];

    __device__ __forceinline__ void init(const float *X, int ld, int c0, int n, int k0, int tid)
    {
        narrow = !KC && n - c0 < 4;
        on = tid < TH;
        const int t = min(tid, TH - 1), r = t / PER, c = 4 * (t % PER);
        if (KC) {
            base = X + (int64_t)c0 * ld + k0;
            step = kTK;
            at = r * kLd + c;
#pragma unroll
            for (int u = 0; u < NV; ++u)
                off[u] = 4u * (uint32_t)(min(r + PU * u, n - 1 - c0) * ld + c);
        } else {
            const int m = narrow ? c : min(c, n - 4 - c0);   // moved back to end at the edge
            base = X + (int64_t)k0 * ld + c0;
            step = (int64_t)kTK * ld;
            at = r * kLd + m;
#pragma unroll
            for (int u = 0; u < NV; ++u)
                off[u] = 4u * (uint32_t)((r + PU * u) * ld + m);
        }
    }
    // a whole step of kTK into register set S (not for a narrow operand)
    template <int S>
    __device__ __forceinline__ void load()
    {
#pragma unroll
        for (int u = 0; u < NV; ++u)
            v[S][u] = *reinterpret_cast<const f4u *>(reinterpret_cast<const char *>(base) +
                                                     off[u]);
    }
    // the step at `base` by elements into set 0, `left` <= kTK of it in range:
    // zeros past that
    __device__ __forceinline__ void load_tail(int left, int ld, int c0, int n, int tid)
    {
        const int t = min(tid, TH - 1), r = t / PER, c = 4 * (t % PER);
#pragma unroll
        for (int u = 0; u < NV; ++u)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                if (KC) {
                    const int k = c + x;
                    const float y = base[min(r + PU * u, n - 1 - c0) * ld + min(k, left - 1)];
                    v[0][u][x] = k < left ? y : 0.f;
                } else {
                    const int k = r + PU * u, m = narrow ? c : min(c, n - 4 - c0);
                    const float y = base[(int64_t)min(k, left - 1) * ld + min(m + x, n - 1 - c0)];
                    v[0][u][x] = k < left ? y : 0.f;
                }
            }
    }
    template <int S>
    __device__ __forceinline__ void store(float *lds) const
    {
        if (TH == 256 || on)
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                if (KC) {
                    *reinterpret_cast<f4 *>(lds + at + u * PU * kLd) = v[S][u];
                } else {   // a moved vector need not be 16-byte aligned in LDS
                    *reinterpret_cast<f4u *>(lds + at + u * PU * kLd) = v[S][u];
                }
            }
    }
    // the last step, whose first `skip` elements of k the step before had:
    // zeros there (in both operands: zero times an infinity is no zero)
    template <int S>
    __device__ __forceinline__ void skip_first(int skip, int tid)
    {
        const int t = min(tid, TH - 1), r = t / PER, c = 4 * (t % PER);
        if ((KC ? c : r) < skip)
#pragma unroll
            for (int u = 0; u < NV; ++u)
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    v[S][u][x] = (KC ? c + x : r + PU * u) < skip ? 0.f : v[S][u][x];
    }
    // E consecutive k from `k` on of row or column c
    template <int E>
    static __device__ __forceinline__ f4 frag(const float *lds, int c, int k)
    {
        f4 r = {0.f, 0.f, 0.f, 0.f};
        if (KC && E == 4) {
            r = *reinterpret_cast<const f4 *>(lds + c * kLdK + k);
        } else if (KC) {
            const f2 y = *reinterpret_cast<const f2 *>(lds + c * kLdK + k);
            r.x = y.x;
            r.y = y.y;
        } else {
#pragma unroll
            for (int x = 0; x < E; ++x)
                r[x] = lds[(k + x) * kLd + c];
        }
        return r;
    }
};

template <bool TA, bool TB, int NB, int ROWS>
__device__ __forceinline__ void gemm_tile(const GemmProb &p, int m0, int n0, int bz, int z,
                                          float *lds)
{
    typedef Operand<!TA, ROWS> OA;
    typedef Operand<TB, 16 * NB> OB;
    constexpr int kBuf = OA::kFloats + OB::kFloats;
    // ROWS / 16 wavefronts side by side; the rest split each step's k range
    constexpr int RG = ROWS / 16, KW = kTK * RG / 4, E = KW >= 16 ? 4 : 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int q = lane >> 4, rl = lane & 15, wr = 16 * (wave % RG), ks = wave / RG;
    const int live = p.live ? *p.live : INT32_MAX;
    int k_lo = 0, k_hi = p.k;
    if (TA) {
        k_hi = min(p.k, live);
        const int chunk = ((k_hi + p.splits - 1) / p.splits + kTK - 1) / kTK * kTK;
        k_lo = z * chunk;
        k_hi = min(k_hi, k_lo + chunk);
    } else if (m0 >= live) {
        return;   // the whole tile is past the live rows
    }
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 acc[NB], one = zero, sum[NB], sum_one = zero;   // sum: TA only
#pragma unroll
    for (int j = 0; j < NB; ++j)
        acc[j] = sum[j] = zero;
    auto fold = [&]() {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            sum[j] += acc[j];
            acc[j] = zero;
        }
        sum_one += one;
        one = zero;
    };
    const bool sums = TA && p.colsum && n0 == 0;
    if (k_lo < k_hi) {
        OA a;
        OB b;
        a.init(p.A + bz * p.sA, p.lda, m0, p.m, k_lo, tid);
        b.init(p.B + bz * p.sB, p.ldb, n0, p.n, k_lo, tid);
        // While step i multiplies from one LDS buffer, step i + 1 (loaded
        // during step i - 1) is on its way to the other, and step i + 2
        // loads.  The loads have no condition around them (the compiler waits
        // for such loads where the paths join): past the last step they read
        // that step again.  The last step ends at the reduction's end and
        // overlaps the step before, with zeros where it does.  The barrier
        // orders LDS only, so the loads stay in flight across it.
        const int len = k_hi - k_lo, steps = (len + kTK - 1) / kTK;
        auto compute = [&](int i, const float *la) {
            const float *lb = la + OA::kFloats;
#pragma unroll
            for (int h = 0; h < (KW + 15) / 16; ++h) {
                const int k = KW * ks + 16 * h + E * q;
                const f4 av = OA::template frag<E>(la, wr + rl, k);
                f4 bv[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    bv[j] = OB::template frag<E>(lb, 16 * j + rl, k);
                // column blocks innermost: consecutive MFMAs are independent
#pragma unroll
                for (int x = 0; x < E; ++x) {
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        acc[j] = mfma_16x16x4(av[x], bv[j][x], acc[j]);
                    if (TA && sums)
                        one = mfma_16x16x4(av[x], 1.f, one);
                }
            }
            if (TA && (i & 3) == 3)
                fold();
        };
        const float *const a0 = a.base, *const b0 = b.base;
        if (len >= kTK && !a.narrow && !b.narrow) {
            const int skip = steps * kTK - len;
            auto seek = [&](int i) {
                const int64_t k = min(i * kTK, len - kTK);
                a.base = a0 + k * (a.step / kTK);
                b.base = b0 + k * (b.step / kTK);
            };
            a.template load<0>();
            b.template load<0>();
            seek(1);
            a.template load<1>();
            b.template load<1>();
            issue_fence();
            a.template store<0>(lds);
            b.template store<0>(lds + OA::kFloats);
            lds_barrier();
            for (int i = 0;; i += 2) {
                seek(i + 2);
                a.template load<0>();
                b.template load<0>();
                issue_fence();
                compute(i, lds);
                if (i + 1 >= steps)
                    break;
                if (skip > 0 && i + 2 == steps) {
                    a.template skip_first<1>(skip, tid);
                    b.template skip_first<1>(skip, tid);
                }
                a.template store<1>(lds + kBuf);
                b.template store<1>(lds + kBuf + OA::kFloats);
                lds_barrier();
                seek(i + 3);
                a.template load<1>();
                b.template load<1>();
                issue_fence();
                compute(i + 1, lds + kBuf);
                if (i + 2 >= steps)
                    break;
                if (skip > 0 && i + 3 == steps) {
                    a.template skip_first<0>(skip, tid);
                    b.template skip_first<0>(skip, tid);
                }
                a.template store<0>(lds);
                b.template store<0>(lds + OA::kFloats);
                lds_barrier();
            }
        } else {   // shorter than a step, or narrow: by elements
            for (int i = 0; i < steps; ++i) {
                a.base = a0 + i * a.step;
                b.base = b0 + i * b.step;
                const int left = min(kTK, len - i * kTK);
                a.load_tail(left, p.lda, m0, p.m, tid);
                b.load_tail(left, p.ldb, n0, p.n, tid);
                lds_barrier();   // every wave is done with the step before
                a.template store<0>(lds);
                b.template store<0>(lds + OA::kFloats);
                lds_barrier();
                compute(i, lds);
            }
        }
    }
    if (RG < 4) {   // the wavefronts' parts of the reduction, in pairs
        lds_barrier();
        f4 *part = reinterpret_cast<f4 *>(lds) + (wave % RG) * NB * kWave + lane;
        if (ks > 0)
#pragma unroll
            for (int j = 0; j < NB; ++j)
                part[((ks - 1) * RG * NB + j) * kWave] = acc[j];
        lds_barrier();
        if (ks > 0)
            return;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            acc[j] += part[j * kWave];
            if (RG == 1)
                acc[j] += part[(NB + j) * kWave] + part[(2 * NB + j) * kWave];
        }
    }
    if (TA)
        fold();
    // The epilogue's loads go out together, at clamped places: one behind the
    // other, each behind its element's condition, they took longer than the
    // products of a small output (about 20 of 28 us at 1,800 x 100).
    float *C = p.C + bz * p.sC + (TA ? z * p.split_stride : 0);
    f4 (&x)[NB] = TA ? sum : acc;
    int rows[4], cols[NB];
#pragma unroll
    for (int v = 0; v < 4; ++v)
        rows[v] = min(m0 + wr + 4 * q + v, p.m - 1);
#pragma unroll
    for (int j = 0; j < NB; ++j)
        cols[j] = min(n0 + 16 * j + rl, p.n - 1);
    if (p.bias) {
        const float *bias = p.bias + bz * p.sBias;
        float y[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j)
            y[j] = bias[cols[j]];
#pragma unroll
        for (int j = 0; j < NB; ++j)
            x[j] += f4{y[j], y[j], y[j], y[j]};
    }
    if (p.gate) {
        f4 y[NB];
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < NB; ++j)
                y[j][v] = p.gate[(int64_t)rows[v] * p.ldg + cols[j]];
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[j][v] = y[j][v] > 0.f ? x[j][v] : 0.f;
    }
    if (p.row_on) {
        int on[4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
            on[v] = p.row_on[rows[v]];
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[j][v] = on[v] <= 0 && cols[j] < p.zero_cols ? 0.f : x[j][v];
    }
    if (p.accumulate) {
        f4 y[NB];
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < NB; ++j)
                y[j][v] = C[(int64_t)rows[v] * p.ldc + cols[j]];
#pragma unroll
        for (int j = 0; j < NB; ++j)
            x[j] += y[j];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (m0 + wr + 4 * q + v >= p.m)
            continue;
        float *c = C + (int64_t)rows[v] * p.ldc;
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (n0 + 16 * j + rl < p.n)
                c[cols[j]] = x[j][v];
        if (sums && rl == 0)
            p.colsum[z * p.colsum_stride + bz * p.sColsum + rows[v]] = sum_one[v];
    }
}

template <bool TA, bool TB, int ROWS>
__global__ __launch_bounds__(256, TB ? 3 : 2) void k_gemm(GemmGroup g)
{
    constexpr int kA = Operand<!TA, ROWS>::kFloats, kB = Operand<TB, 112>::kFloats;
    __shared__ __align__(16) float lds[2 * (kA + kB)];
    const int t = blockIdx.x;
    int i = 0;
    while (i + 1 < g.n && t >= g.p[i + 1].tile0)
        ++i;
    const GemmProb &p = g.p[i];
    int r = t - p.tile0;
    const int tn = r % p.tiles_n;
    r /= p.tiles_n;
    const int tm = r % p.tiles_m;
    r /= p.tiles_m;
    const int bz = r % p.batch, z = r / p.batch;
    if (p.wide)
        gemm_tile<TA, TB, 7, ROWS>(p, tm * ROWS, tn * 112, bz, z, lds);
    else
        gemm_tile<TA, TB, 4, ROWS>(p, tm * ROWS, tn * 64, bz, z, lds);
}

}  // namespace

tgm_status_t tgm::gemm_launch(bool ta, bool tb, const GemmProb *probs, int n, hipStream_t s)
{
    // Rows of a tile: 64 where that gives the chip work enough, else 32 or
    // 16, whose wavefronts share a step's reduction, so that a tile with few
    // others on the chip is done sooner (1,800 x 100 by 200: 13 us with 64
    // rows, 29 workgroups).  Smaller tiles read B more often.
    auto wide = [](const GemmProb &p) { return cdiv(p.n, 112) * 112 <= cdiv(p.n, 64) * 64; };
    auto count = [&](const GemmProb &p, int rows) {
        return cdiv(p.n, wide(p) ? 112 : 64) * cdiv(p.m, rows) * p.batch *
               (ta ? std::max(p.splits, 1) : 1);
    };
    int64_t t64 = 0;
    for (int i = 0; i < n; ++i)
        if (probs[i].m > 0 && probs[i].n > 0 && probs[i].batch > 0)
            t64 += count(probs[i], 64);
    const int rows = ta || t64 > kTiles32 ? 64 : t64 > kTiles16 ? 32 : 16;
    GemmGroup g;
    g.n = 0;
    int64_t tiles = 0;
    for (int i = 0; i < n; ++i) {
        GemmProb p = probs[i];
        if (p.m <= 0 || p.n <= 0 || p.batch <= 0)
            continue;
        if (g.n == kGemmGroup)
            return TGM_EINVAL;
        if (!ta || p.splits < 1)
            p.splits = 1;
        p.wide = wide(p);
        p.tiles_n = (int)cdiv(p.n, p.wide ? 112 : 64);
        p.tiles_m = (int)cdiv(p.m, rows);
        p.tile0 = (int)tiles;
        tiles += count(p, rows);
        if (tiles > INT32_MAX)
            return TGM_EINVAL;
        g.p[g.n++] = p;
    }
    if (g.n == 0)
        return TGM_OK;
    const dim3 grid((unsigned)tiles);
    if (ta && tb)
        return TGM_EINVAL;   // no product here has both operands transposed
    if (ta)
        TGM_LAUNCH((k_gemm<true, false, 64>), grid, dim3(256), 0, s, g);
    else if (tb && rows == 64)
        TGM_LAUNCH((k_gemm<false, true, 64>), grid, dim3(256), 0, s, g);
    else if (tb && rows == 32)
        TGM_LAUNCH((k_gemm<false, true, 32>), grid, dim3(256), 0, s, g);
    else if (tb)
        TGM_LAUNCH((k_gemm<false, true, 16>), grid, dim3(256), 0, s, g);
    else if (rows == 64)
        TGM_LAUNCH((k_gemm<false, false, 64>), grid, dim3(256), 0, s, g);
    else if (rows == 32)
        TGM_LAUNCH((k_gemm<false, false, 32>), grid, dim3(256), 0, s, g);
    else
        TGM_LAUNCH((k_gemm<false, false, 16>), grid, dim3(256), 0, s, g);
    return TGM_OK;
}
