// Training step after the stage: the link-prediction loss of the batch, its
// gradient with respect to every weight of the model and of the predictor,
// the optimizer step, and the repack of the model's operands (Sec. 5,
// training settings: link prediction on equal numbers of positive and
// negative pairs; App. C.2: the loss and backward steps of the training
// stage).
//
// Every reduction has a fixed order, so results are bit-reproducible: the
// weight gradients are MFMA GEMMs whose long reduction dimension (roots,
// nodes) is split over workgroups into partial sums that the optimizer's
// launch adds in split order; the gradient of each node's updated memory
// gathers its contributions (the roots and neighbour slots that read it)
// after a stable radix sort by node.
//
// The attention's backward works on aggregates, as its forward does: with
// a_s = [s'_u || efeat || phi] the row of slot s, q the root's query and per
// head u = W_k^t q, the scores are a_s . u (b_k shifts every score of a head
// alike, and a softmax ignores that), o = W_v abar + b_v with abar = sum_s
// alpha_s a_s, and so
//   dabar = W_v^t do, dalpha_s = a_s . dabar (b_v shifts them alike too),
//   dscore_s = alpha_s (dalpha_s - sum alpha dalpha) / sqrt(d_h),
//   du = sum_s dscore_s a_s, dq = W_k du, dW_k = sum q (x) du,
//   dW_v = sum do (x) abar, ds'_u = dscore_s u + alpha_s dabar (memory part).
// Every product then runs over (root, head) rows instead of slots: at a
// batch of 4,000 (12,000 roots, 10 slots each, M = 100, 386-wide rows) 5.6
// GFLOP instead of 46, and neither the slot rows (185 MB) nor their keys and
// values are stored.  Two iterations of the training loop at that size took
// 5.35 ms with products over slots and a launch (or two) per product, and
// 1.71 ms with these, grouped eight launches to a step; one step at a batch
// of 600: 966 and 218 us.
// Rows too wide for a wavefront's registers, and many heads, take the products
// over slots (slot_form).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <utility>

#include "common.h"
#include "sort.h"

using namespace tgm;

namespace {

// ------------------------------------------------------------- predictor
// One wavefront per event e < b (lanes over the hidden units j < M <= 128):
// z+ = Zs[e] + Zd[e] + b_p, z- = Zs[e] + Zd[b + e] + b_p, the two scores, the
// event's loss, and the gradients of the scores (dsc) and pre-activations.
struct PredArgs {
    int b, M;
    const float *Zs, *Zd;        // [b x M], [2b x M]
    const float *b_p, *w_out, *b_out;
    float *dZsrc, *dZdst, *act;  // [b x M], [2b x M], [2b x M]
    float *dsc, *lossv;          // [2b], [b]
};

__device__ __forceinline__ float softplusf(float x)
{
    return x > 0.f ? x + log1pf(expf(-x)) : log1pf(expf(x));
}
__device__ __forceinline__ float sigmoidf(float x) { return 1.f / (1.f + expf(-x)); }

__global__ __launch_bounds__(256) void k_pred(PredArgs a)
{
    const int e = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (e >= a.b)
        return;
    const int M = a.M, b = a.b;
    float zp[2], zn[2], sp = 0.f, sn = 0.f;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int j = lane + 64 * u;
        zp[u] = zn[u] = 0.f;
        if (j < M) {
            const float zs = a.Zs[(int64_t)e * M + j] + a.b_p[j];
            zp[u] = zs + a.Zd[(int64_t)e * M + j];
            zn[u] = zs + a.Zd[(int64_t)(b + e) * M + j];
            sp += a.w_out[j] * fmaxf(zp[u], 0.f);
            sn += a.w_out[j] * fmaxf(zn[u], 0.f);
        }
    }
    sp = wave_sum(sp) + a.b_out[0];
    sn = wave_sum(sn) + a.b_out[0];
    const float dsp = (sigmoidf(sp) - 1.f) / (float)b, dsn = sigmoidf(sn) / (float)b;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int j = lane + 64 * u;
        if (j >= M)
            continue;
        const float dzp = zp[u] > 0.f ? dsp * a.w_out[j] : 0.f;
        const float dzn = zn[u] > 0.f ? dsn * a.w_out[j] : 0.f;
        a.dZsrc[(int64_t)e * M + j] = dzp + dzn;
        a.dZdst[(int64_t)e * M + j] = dzp;
        a.dZdst[(int64_t)(b + e) * M + j] = dzn;
        a.act[(int64_t)e * M + j] = fmaxf(zp[u], 0.f);
        a.act[(int64_t)(b + e) * M + j] = fmaxf(zn[u], 0.f);
    }
    if (lane == 0) {
        a.dsc[e] = dsp;
        a.dsc[b + e] = dsn;
        a.lossv[e] = softplusf(-sp) + softplusf(sn);
    }
}

// ------------------------------------------------------------- attention
// What the step needs besides its products' outputs, one launch (the keys'
// workgroups, which take longest, first):
//   root rows   Xo[r][M .. 2M) = s'_v (the query's and the output
//               projection's input), one wavefront per root;
//   node rows   X[p] = [mail || phi(mail_ts - mem_ts)] and Hm[p] = mem[p] of
//               the node set's nodes with mail, zeros without, one wavefront
//               per node;
//   sort keys   contributor r < R is root r (it reads s' of node
//               root_pos[r]), R + sl is slot sl (node nbr_pos[sl]); empty
//               slots get the key cap, past every node;
//   c_q         W_q phi(0) + b_q, one wavefront per unit.
struct RowArgs {
    int R, nb, M, D_m, D_t, cap, ldx;
    int n_root, n_node, n_key;   // workgroups of the first three parts
    const int32_t *root_pos, *nbr_pos, *cnt, *n_nodes, *ver;
    const double *mem_ts, *mail_ts, *omega, *beta;
    const float *s_new, *mem, *mail, *W_q, *b_q;
    float *Xo, *X, *Hm, *cq;
    SortPlan sort;
};

__global__ __launch_bounds__(256) void k_train_rows(RowArgs a)
{
    __shared__ int32_t count[1 << kSortDigit];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int M = a.M, D_m = a.D_m, D_t = a.D_t;
    int blk = blockIdx.x;
    if (blk < a.n_key) {
        sort_keys_tile(a.sort, blk, count, [&](int64_t t) {
            uint32_t key;
            if (t < a.R) {
                key = (uint32_t)a.root_pos[t];
            } else {
                const int64_t sl = t - a.R;
                const int r = (int)(sl / a.nb), j = (int)(sl % a.nb);
                key = j < a.cnt[r] ? (uint32_t)a.nbr_pos[sl] : (uint32_t)a.cap;
            }
            return min(key, (uint32_t)a.cap);
        });
        return;
    }
    blk -= a.n_key;
    if (blk < a.n_root) {
        const int r = blk * 4 + wave;
        if (r < a.R)
            wave_copy_row(a.Xo + (int64_t)r * 2 * M + M, a.s_new + (int64_t)a.root_pos[r] * M, M,
                          lane);
        return;
    }
    blk -= a.n_root;
    if (blk < a.n_node) {
        const int p = blk * 4 + wave;
        if (p >= min(*a.n_nodes, a.cap))
            return;
        float *x = a.X + (int64_t)p * a.ldx, *hm = a.Hm + (int64_t)p * M;
        if (a.ver[p] < 0) {
            for (int k = lane; k < D_m + D_t; k += kWave)
                x[k] = 0.f;
            for (int k = lane; k < M; k += kWave)
                hm[k] = 0.f;
            return;
        }
        const double dt = a.mail_ts[p] - a.mem_ts[p];
        wave_copy_2rows(hm, a.mem + (int64_t)p * M, M, x, a.mail + (int64_t)p * D_m, D_m, lane);
        for (int d = lane; d < D_t; d += kWave)
            x[D_m + d] = time_enc(a.omega[d], a.beta[d], dt);
        return;
    }
    blk -= a.n_node;
    const int k = blk * 4 + wave;
    if (k >= M)
        return;
    float acc = 0.f;
    for (int d = lane; d < D_t; d += kWave)
        acc += a.W_q[(int64_t)k * (M + D_t) + M + d] * time_enc(a.omega[d], a.beta[d], 0.0);
    acc = wave_sum(acc);
    if (lane == 0)
        a.cq[k] = acc + a.b_q[k];
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}

struct AttArgs {
    int R, nb, M, D_e, D_t, H, ldu;
    float scale;
    const int32_t *cnt, *root_pos, *nbr_pos, *eid;
    const double *root_ts, *nts, *omega, *beta;
    const float *s_new, *efeat, *U;   // U [R x H x ldu]
    float *alpha;                     // [R x H x nb]
    float *abar;                      // forward: sum_s alpha_s a_s [R x H x ldu]
    float *dbar;                      // backward: dabar in, du out [R x H x ldu]
    float *dKm;                       // backward: [R nb x M], filled slots only
};

// A row [s' || efeat || phi] in a wavefront's registers: lane l holds columns
// l + 64 i of each part, zero past the part's width (CE, CT: 64-wide groups
// of the edge features and time codes; M <= 128).
template <int CE, int CT>
struct Row {
    float m[2], e[CE], t[CT];

    __device__ __forceinline__ void load_cols(const float *x, const AttArgs &a, int lane)
    {
        const int M = a.M, D_e = a.D_e, D_t = a.D_t;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            m[i] = x[min(lane + kWave * i, M - 1)];
#pragma unroll
        for (int i = 0; i < CE; ++i)
            e[i] = D_e > 0 ? x[M + min(lane + kWave * i, D_e - 1)] : 0.f;
#pragma unroll
        for (int i = 0; i < CT; ++i)
            t[i] = D_t > 0 ? x[M + D_e + min(lane + kWave * i, D_t - 1)] : 0.f;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            m[i] = lane + kWave * i < M ? m[i] : 0.f;
#pragma unroll
        for (int i = 0; i < CE; ++i)
            e[i] = lane + kWave * i < D_e ? e[i] : 0.f;
#pragma unroll
        for (int i = 0; i < CT; ++i)
            t[i] = lane + kWave * i < D_t ? t[i] : 0.f;
    }
    __device__ __forceinline__ void store_cols(float *x, const AttArgs &a, int lane) const
    {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (lane + kWave * i < a.M)
                x[lane + kWave * i] = m[i];
#pragma unroll
        for (int i = 0; i < CE; ++i)
            if (lane + kWave * i < a.D_e)
                x[a.M + lane + kWave * i] = e[i];
#pragma unroll
        for (int i = 0; i < CT; ++i)
            if (lane + kWave * i < a.D_t)
                x[a.M + a.D_e + lane + kWave * i] = t[i];
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            m[i] = 0.f;
#pragma unroll
        for (int i = 0; i < CE; ++i)
            e[i] = 0.f;
#pragma unroll
        for (int i = 0; i < CT; ++i)
            t[i] = 0.f;
    }
    __device__ __forceinline__ float dot(const Row &o) const   // this lane's part
    {
        float p = 0.f;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            p = fmaf(m[i], o.m[i], p);
#pragma unroll
        for (int i = 0; i < CE; ++i)
            p = fmaf(e[i], o.e[i], p);
#pragma unroll
        for (int i = 0; i < CT; ++i)
            p = fmaf(t[i], o.t[i], p);
        return p;
    }
    __device__ __forceinline__ void axpy(float w, const Row &o)
    {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            m[i] = fmaf(w, o.m[i], m[i]);
#pragma unroll
        for (int i = 0; i < CE; ++i)
            e[i] = fmaf(w, o.e[i], e[i]);
#pragma unroll
        for (int i = 0; i < CT; ++i)
            t[i] = fmaf(w, o.t[i], t[i]);
    }
};

// The rows of up to NC slots of a root, every load issued before the time
// codes are computed.
template <int CE, int CT, int NC>
struct SlotRows {
    Row<CE, CT> x[NC];

    __device__ __forceinline__ void load(const AttArgs &a, int r, int j0, int nj, int lane)
    {
        const int64_t sl = (int64_t)r * a.nb + j0 + min(lane, nj - 1);
        const int32_t pos = a.nbr_pos[sl], ev = a.eid[sl];
        const double dt = a.root_ts[r] - a.nts[sl];
        const int M = a.M, D_e = a.D_e, D_t = a.D_t;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int jj = min(j, nj - 1);
            const float *s = a.s_new + (int64_t)__builtin_amdgcn_readlane(pos, jj) * M;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                x[j].m[i] = s[min(lane + kWave * i, M - 1)];
            if (D_e > 0) {
                const float *f = a.efeat + (int64_t)__builtin_amdgcn_readlane(ev, jj) * D_e;
#pragma unroll
                for (int i = 0; i < CE; ++i)
                    x[j].e[i] = f[min(lane + kWave * i, D_e - 1)];
            } else {
#pragma unroll
                for (int i = 0; i < CE; ++i)
                    x[j].e[i] = 0.f;
            }
        }
        const long long dti = __double_as_longlong(dt);
        const int lo = (int)dti, hi = (int)(dti >> 32);
#pragma unroll
        for (int i = 0; i < CT; ++i) {
            if (kWave * i >= D_t) {
#pragma unroll
                for (int j = 0; j < NC; ++j)
                    x[j].t[i] = 0.f;
                continue;
            }
            const int d = min(lane + kWave * i, D_t - 1);
            const double om = a.omega[d], be = a.beta[d];
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const int jj = min(j, nj - 1);
                const unsigned l = (unsigned)__builtin_amdgcn_readlane(lo, jj);
                const long long h = __builtin_amdgcn_readlane(hi, jj);
                x[j].t[i] = time_enc(om, be, __longlong_as_double((h << 32) | l));
            }
        }
    }
};

// Forward values again, one wavefront per root: per head the scores of the
// root's slots, their softmax alpha and abar = sum_s alpha_s a_s.  Roots with
// up to NC slots keep their rows in registers for every head and both passes;
// longer ones read them again.  Bound by the vector ALUs: the time codes, the
// two dot products and the weighted sums of every slot.
template <int CE, int CT, int NC>
__global__ __launch_bounds__(256) void k_att_fwd(AttArgs a)
{
    const int r = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= a.R)
        return;
    const int cr = __builtin_amdgcn_readfirstlane(a.cnt[r]);
    SlotRows<CE, CT, NC> rows;
    if (cr > 0 && cr <= NC)
        rows.load(a, r, 0, cr, lane);
    for (int eta = 0; eta < a.H; ++eta) {
        const int64_t o = ((int64_t)r * a.H + eta) * a.ldu;
        Row<CE, CT> acc;
        acc.clear();
        if (cr > 0) {
            Row<CE, CT> u;
            u.load_cols(a.U + o, a, lane);
            float mine = -INFINITY;   // lane j < cr: the score of slot j
            for (int j0 = 0; j0 < cr; j0 += NC) {
                const int nj = min(NC, cr - j0);
                if (cr > NC)
                    rows.load(a, r, j0, nj, lane);
#pragma unroll
                for (int j = 0; j < NC; ++j)
                    if (j < nj) {
                        const float sc = wave_total(rows.x[j].dot(u)) * a.scale;
                        mine = lane == j0 + j ? sc : mine;
                    }
            }
            const float mx = wave_max(mine);
            const float ex = lane < cr ? expf(mine - mx) : 0.f;
            const float al = ex / wave_total(ex);
            if (lane < cr)
                a.alpha[((int64_t)r * a.H + eta) * a.nb + lane] = al;
            for (int j0 = 0; j0 < cr; j0 += NC) {
                const int nj = min(NC, cr - j0);
                if (cr > NC)
                    rows.load(a, r, j0, nj, lane);
#pragma unroll
                for (int j = 0; j < NC; ++j)
                    if (j < nj)
                        acc.axpy(lane_value(al, j0 + j), rows.x[j]);
            }
        }
        acc.store_cols(a.abar + o, a, lane);
    }
}

// Backward, one wavefront per root and the same layout: per head dalpha_s =
// a_s . dabar, the scores' gradients, du = sum_s dscore_s a_s (in place of
// dabar) and each slot's gradient of s'_u, summed over the heads.
template <int CE, int CT, int NC>
__global__ __launch_bounds__(256) void k_att_bwd(AttArgs a)
{
    const int r = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= a.R)
        return;
    const int cr = __builtin_amdgcn_readfirstlane(a.cnt[r]), M = a.M;
    SlotRows<CE, CT, NC> rows;
    if (cr > 0 && cr <= NC)
        rows.load(a, r, 0, cr, lane);
    float dk[NC][2];
#pragma unroll
    for (int j = 0; j < NC; ++j)
        dk[j][0] = dk[j][1] = 0.f;
    for (int eta = 0; eta < a.H; ++eta) {
        const int64_t o = ((int64_t)r * a.H + eta) * a.ldu;
        Row<CE, CT> acc;
        acc.clear();
        if (cr > 0) {
            Row<CE, CT> db;
            db.load_cols(a.dbar + o, a, lane);
            float um[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                um[i] = a.U[o + min(lane + kWave * i, M - 1)];
            const float al = lane < cr ? a.alpha[((int64_t)r * a.H + eta) * a.nb + lane] : 0.f;
            float da = 0.f;   // lane j < cr: dalpha of slot j
            for (int j0 = 0; j0 < cr; j0 += NC) {
                const int nj = min(NC, cr - j0);
                if (cr > NC)
                    rows.load(a, r, j0, nj, lane);
#pragma unroll
                for (int j = 0; j < NC; ++j)
                    if (j < nj) {
                        const float d = wave_total(rows.x[j].dot(db));
                        da = lane == j0 + j ? d : da;
                    }
            }
            const float dsc = al * (da - wave_total(al * da)) * a.scale;
            for (int j0 = 0; j0 < cr; j0 += NC) {
                const int nj = min(NC, cr - j0);
                if (cr > NC)
                    rows.load(a, r, j0, nj, lane);
#pragma unroll
                for (int j = 0; j < NC; ++j)
                    if (j < nj) {
                        const float w = lane_value(dsc, j0 + j), aj = lane_value(al, j0 + j);
                        acc.axpy(w, rows.x[j]);
                        float g[2];
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            g[i] = w * um[i] + aj * db.m[i];
                        if (cr <= NC) {
                            dk[j][0] += g[0];
                            dk[j][1] += g[1];
                        } else {   // the heads' sum in memory
                            float *x = a.dKm + ((int64_t)r * a.nb + j0 + j) * M;
#pragma unroll
                            for (int i = 0; i < 2; ++i)
                                if (lane + kWave * i < M)
                                    x[lane + kWave * i] =
                                        g[i] + (eta > 0 ? x[lane + kWave * i] : 0.f);
                        }
                    }
            }
        }
        acc.store_cols(a.dbar + o, a, lane);
    }
    if (cr <= NC)
#pragma unroll
        for (int j = 0; j < NC; ++j)
            if (j < cr)
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (lane + kWave * i < M)
                        a.dKm[((int64_t)r * a.nb + j) * M + lane + kWave * i] = dk[j][i];
}

// The same attention by slots, for the trainers that slot_form names: every
// slot's row [s'_u || efeat || phi], its key and value are stored, and the
// products run over slots instead of (root, head) rows.  Rows of any width,
// and a cost and work space that do not grow with the heads.
struct SlotArgs {
    int R, nb, M, D_e, D_t, H;
    float scale;
    const int32_t *cnt, *nbr_pos, *eid;
    const double *root_ts, *nts, *omega, *beta;
    const float *s_new, *efeat, *Q, *dXo;   // Q [R x M], dXo [R x 2M]
    float *rows;                            // [R nb x Dkv], zero past the count
    float *KV, *dKV;                        // [R nb x 2M]
    float *alpha, *Xo, *dQ;                 // [R x H x nb], [R x 2M], [R x M]
};

// One wavefront per slot: its row
__global__ __launch_bounds__(256) void k_slot_rows(SlotArgs a)
{
    const int64_t sl = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63, M = a.M, D_e = a.D_e, D_t = a.D_t;
    if (sl >= (int64_t)a.R * a.nb)
        return;
    const int r = (int)(sl / a.nb), j = (int)(sl % a.nb), Dkv = M + D_e + D_t;
    float *x = a.rows + sl * Dkv;
    if (j >= a.cnt[r]) {
        for (int k = lane; k < Dkv; k += kWave)
            x[k] = 0.f;
        return;
    }
    wave_copy_row(x, a.s_new + (int64_t)a.nbr_pos[sl] * M, M, lane);
    if (D_e > 0)
        wave_copy_row(x + M, a.efeat + (int64_t)a.eid[sl] * D_e, D_e, lane);
    const double dt = a.root_ts[r] - a.nts[sl];
    for (int d = lane; d < D_t; d += kWave)
        x[M + D_e + d] = time_enc(a.omega[d], a.beta[d], dt);
}

// One wavefront per root, lanes over the outputs k = lane, lane + 64: per head
// the scores q . K of its slots, their softmax alpha and o = sum_s alpha_s V_s.
__global__ __launch_bounds__(256) void k_slot_fwd(SlotArgs a)
{
    const int r = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= a.R)
        return;
    const int M = a.M, H = a.H, nb = a.nb, dh = M / H;
    const int cr = __builtin_amdgcn_readfirstlane(a.cnt[r]);
    const float *kv = a.KV + (int64_t)r * nb * 2 * M;
    float q[2], o[2] = {0.f, 0.f};
    int head[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = lane + kWave * i;
        q[i] = k < M ? a.Q[(int64_t)r * M + k] : 0.f;
        head[i] = k < M ? k / dh : -1;
    }
    for (int eta = 0; eta < H && cr > 0; ++eta) {
        float mine = -INFINITY;   // lane j < cr: the score of slot j
        for (int j = 0; j < cr; ++j) {
            float p = 0.f;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (head[i] == eta)
                    p = fmaf(q[i], kv[(int64_t)j * 2 * M + lane + kWave * i], p);
            const float sc = wave_total(p) * a.scale;
            mine = lane == j ? sc : mine;
        }
        const float mx = wave_max(mine);
        const float ex = lane < cr ? expf(mine - mx) : 0.f;
        const float al = ex / wave_total(ex);
        if (lane < cr)
            a.alpha[((int64_t)r * H + eta) * nb + lane] = al;
        for (int j = 0; j < cr; ++j) {
            const float aj = lane_value(al, j);
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (head[i] == eta)
                    o[i] = fmaf(aj, kv[(int64_t)j * 2 * M + M + lane + kWave * i], o[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (lane + kWave * i < M)
            a.Xo[(int64_t)r * 2 * M + lane + kWave * i] = o[i];
}

// Backward, the same layout: dalpha_s = do . V_s, the scores' gradients, dV_s
// = alpha_s do, dK_s = dscore_s q, dq = sum_s dscore_s K_s; zero rows past the
// count.
__global__ __launch_bounds__(256) void k_slot_bwd(SlotArgs a)
{
    const int r = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (r >= a.R)
        return;
    const int M = a.M, H = a.H, nb = a.nb, dh = M / H;
    const int cr = __builtin_amdgcn_readfirstlane(a.cnt[r]);
    const float *kv = a.KV + (int64_t)r * nb * 2 * M;
    float *dkv = a.dKV + (int64_t)r * nb * 2 * M;
    float q[2], g[2], dq[2] = {0.f, 0.f};
    int head[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = lane + kWave * i;
        q[i] = k < M ? a.Q[(int64_t)r * M + k] : 0.f;
        g[i] = k < M ? a.dXo[(int64_t)r * 2 * M + k] : 0.f;
        head[i] = k < M ? k / dh : -1;
    }
    for (int eta = 0; eta < H && cr > 0; ++eta) {
        const float al = lane < cr ? a.alpha[((int64_t)r * H + eta) * nb + lane] : 0.f;
        float da = 0.f;   // lane j < cr: dalpha of slot j
        for (int j = 0; j < cr; ++j) {
            float p = 0.f;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (head[i] == eta)
                    p = fmaf(g[i], kv[(int64_t)j * 2 * M + M + lane + kWave * i], p);
            const float d = wave_total(p);
            da = lane == j ? d : da;
        }
        const float dsc = al * (da - wave_total(al * da)) * a.scale;
        for (int j = 0; j < cr; ++j) {
            const float w = lane_value(dsc, j), aj = lane_value(al, j);
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (head[i] == eta) {
                    const int64_t k = (int64_t)j * 2 * M + lane + kWave * i;
                    dq[i] = fmaf(w, kv[k], dq[i]);
                    dkv[k] = w * q[i];
                    dkv[k + M] = aj * g[i];
                }
        }
    }
    for (int k = max(cr, 0) * 2 * M + lane; k < nb * 2 * M; k += kWave)
        dkv[k] = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (lane + kWave * i < M)
            a.dQ[(int64_t)r * M + lane + kWave * i] = dq[i];
}

// ------------------------------------------- gradient of the new memories
// The contributors sorted by node (a stable sort, so in contributor order
// within a node) are summed in blocks of 64 sorted positions, one wavefront
// each: a node's run that lies inside a block is finished there; the part of
// a run that began in an earlier block goes to head[block], and the start of
// a run that goes on past the block to tail[block].  k_ds_join then adds the
// open runs, block by block, so a hub's thousands of contributors spread over
// many wavefronts.  ds[p] is the sum of dXo[r][M .. 2M) over its roots and of
// dKm[sl] over its slots; every node of the node set has a contributor.
constexpr int kDsBatch = 8;   // rows in flight

__global__ __launch_bounds__(256) void k_ds_block(int64_t n_items, int32_t cap, int M, int R,
                                                  const uint32_t *__restrict__ keys,
                                                  const int32_t *__restrict__ vals,
                                                  const float *__restrict__ dXo,
                                                  const float *__restrict__ dKm,
                                                  float *__restrict__ ds,
                                                  float *__restrict__ head,
                                                  float *__restrict__ tail)
{
    const int64_t blk = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t i0 = blk * kWave;
    if (i0 >= n_items)
        return;
    const int64_t i = min(i0 + lane, n_items - 1);
    const bool in = i0 + lane < n_items;
    const uint32_t key = in ? keys[i] : (uint32_t)cap;
    const int32_t val = vals[i];
    const uint32_t before = i0 > 0 ? keys[i0 - 1] : ~0u;
    const uint32_t after = i0 + kWave < n_items ? keys[i0 + kWave] : ~0u;
    const uint32_t up = (uint32_t)__shfl_up((int)key, 1, kWave);   // every lane active
    const uint32_t down = (uint32_t)__shfl_down((int)key, 1, kWave);
    const uint32_t prev = lane > 0 ? up : before, next = lane < 63 ? down : after;
    const uint64_t live = __ballot(key < (uint32_t)cap);
    if (live == 0)
        return;
    const int n = 64 - __clzll(live);   // the empty slots sort last
    const uint64_t starts = __ballot(key != prev), ends = __ballot(key != next);
    const int c0 = min(lane, M - 1), c1 = min(lane + kWave, M - 1);
    float a0 = 0.f, a1 = 0.f;
    bool open = true;   // the run began before this block
    for (int b = 0; b < n; b += kDsBatch) {
        float x[kDsBatch][2];
#pragma unroll
        for (int u = 0; u < kDsBatch; ++u) {
            const int c = __builtin_amdgcn_readlane(val, min(b + u, n - 1));
            const float *row = c < R ? dXo + (int64_t)c * 2 * M + M
                                     : dKm + (int64_t)(c - R) * M;
            x[u][0] = row[c0];
            x[u][1] = row[c1];
        }
#pragma unroll
        for (int u = 0; u < kDsBatch; ++u) {
            const int k = b + u;
            if (k >= n)
                break;
            if ((starts >> k) & 1) {
                a0 = a1 = 0.f;
                open = false;
            }
            a0 += x[u][0];
            a1 += x[u][1];
            const bool end = (ends >> k) & 1;
            if (end || k == 63) {
                float *o = open ? head + blk * M
                                : end ? ds + (int64_t)__builtin_amdgcn_readlane((int)key, k) * M
                                      : tail + blk * M;
                if (lane < M)
                    o[lane] = a0;
                if (lane + kWave < M)
                    o[lane + kWave] = a1;
            }
        }
    }
}

// One wavefront per block whose last run goes on: tail[block], then the heads
// of the blocks the run reaches, in order.
__global__ __launch_bounds__(256) void k_ds_join(int64_t n_items, int32_t cap, int M,
                                                 const uint32_t *__restrict__ keys,
                                                 const float *__restrict__ head,
                                                 const float *__restrict__ tail,
                                                 float *__restrict__ ds)
{
    const int64_t blk = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t last = blk * kWave + kWave - 1;
    if (last + 1 >= n_items)
        return;
    const uint32_t p = keys[last];
    if (p >= (uint32_t)cap || keys[last + 1] != p ||
        (keys[blk * kWave] == p && blk > 0 && keys[blk * kWave - 1] == p))
        return;   // no run goes on, or it began in an earlier block
    const int c0 = min(lane, M - 1), c1 = min(lane + kWave, M - 1);
    float a0 = tail[blk * M + c0], a1 = tail[blk * M + c1];
    // how many blocks follow: their first keys, 64 at a time
    for (int64_t f = blk + 1;; f += kWave) {
        const int64_t at = (f + lane) * kWave;
        const uint64_t same = __ballot(at < n_items && keys[min(at, n_items - 1)] == p);
        const int n = ~same == 0 ? 64 : __ffsll((long long)~same) - 1;
        for (int b = 0; b < n; b += kDsBatch) {
            float x[kDsBatch][2];
#pragma unroll
            for (int u = 0; u < kDsBatch; ++u) {
                const float *row = head + (f + min(b + u, n - 1)) * M;
                x[u][0] = row[c0];
                x[u][1] = row[c1];
            }
#pragma unroll
            for (int u = 0; u < kDsBatch; ++u)
                if (b + u < n) {
                    a0 += x[u][0];
                    a1 += x[u][1];
                }
        }
        if (n < kWave)
            break;
    }
    if (lane < M)
        ds[(int64_t)p * M + lane] = a0;
    if (lane + kWave < M)
        ds[(int64_t)p * M + lane + kWave] = a1;
}

// ------------------------------------------------------------------- GRU
// One thread per (node, hidden unit): the gates again from Gx = X W_ih^t +
// b_ih and Gh = Hm W_hh^t + b_hh, then the gradients of the gate
// pre-activations: dGx = [da_r | da_z | da_n], dGh = [da_r | da_z | da_n r].
__global__ __launch_bounds__(256) void k_gru_bwd(const int32_t *__restrict__ n_nodes, int cap,
                                                 int M, const int32_t *__restrict__ ver,
                                                 const float *__restrict__ Gx,
                                                 const float *__restrict__ Gh,
                                                 const float *__restrict__ Hm,
                                                 const float *__restrict__ ds,
                                                 float *__restrict__ dGx, float *__restrict__ dGh)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= (int64_t)cap * M)
        return;
    const int p = (int)(t / M), j = (int)(t % M);
    if (p >= min(*n_nodes, cap))   // the weight gradients' sums end at the node set
        return;
    const int64_t o = (int64_t)p * 3 * M;
    if (ver[p] < 0) {
        dGx[o + j] = dGx[o + M + j] = dGx[o + 2 * M + j] = 0.f;
        dGh[o + j] = dGh[o + M + j] = dGh[o + 2 * M + j] = 0.f;
        return;
    }
    const float r = sigmoidf(Gx[o + j] + Gh[o + j]);
    const float z = sigmoidf(Gx[o + M + j] + Gh[o + M + j]);
    const float hn = Gh[o + 2 * M + j];
    const float n = tanhf(Gx[o + 2 * M + j] + r * hn);
    const float d = ds[(int64_t)p * M + j];
    const float dn = d * (1.f - z), dz = d * (Hm[(int64_t)p * M + j] - n);
    const float dan = dn * (1.f - n * n);
    const float dar = dan * hn * r * (1.f - r), daz = dz * z * (1.f - z);
    dGx[o + j] = dar;
    dGx[o + M + j] = daz;
    dGx[o + 2 * M + j] = dan;
    dGh[o + j] = dar;
    dGh[o + M + j] = daz;
    dGh[o + 2 * M + j] = dan * r;
}

// ------------------------------------------------------------- optimizer
// The end of a step, one thread per parameter: its gradient from the split
// products (added in split order), then the optimizer.  Tensor k's element
// (row, col) is sum_z part[z stride + row ld + col]; columns at or past ld
// (the query's time columns, whose input is phi(0) for every root) are the
// row's sum times phi(0).  b_k has no part: its gradient is zero, since it
// shifts all the scores of a head alike.  One more workgroup sums the loss
// and b_out's gradient in a fixed order, the latter pair by pair: the positive
// and the negative scores' gradients nearly cancel.
struct GradSeg {
    int64_t off;           // first parameter
    int cols, ld, splits;
    const float *part;     // null: zero
    int64_t stride;
    const float *rows;     // row sums [splits][rows_stride] for the columns past ld
    int64_t rows_stride;
};

struct FinishArgs {
    GradSeg seg[17];
    int64_t n;
    float *theta, *grad, *m1, *m2;
    const double *omega, *beta;
    int adam;
    float lr, b1, b2, eps, c1, c2;   // c1 = 1 - b1^t, c2 = 1 - b2^t
    const float *lossv, *dsc;
    int b;
    float *loss, *loss_out;
};

__device__ __forceinline__ void optimize(const FinishArgs &f, int64_t t, float g)
{
    f.grad[t] = g;
    if (!f.adam) {
        f.theta[t] -= f.lr * g;
        return;
    }
    const float a = f.b1 * f.m1[t] + (1.f - f.b1) * g;
    const float v = f.b2 * f.m2[t] + (1.f - f.b2) * g * g;
    f.m1[t] = a;
    f.m2[t] = v;
    f.theta[t] -= f.lr * (a / f.c1) / (sqrtf(v / f.c2) + f.eps);
}

__global__ __launch_bounds__(256) void k_grad_finish(FinishArgs f)
{
    if (blockIdx.x == gridDim.x - 1) {   // loss = (1/b) sum of the events' losses; b_out
        __shared__ float sum[2][256];
        float x = 0.f, y = 0.f;
        for (int e = threadIdx.x; e < f.b; e += 256) {
            x += f.lossv[e];
            y += f.dsc[e] + f.dsc[f.b + e];
        }
        sum[0][threadIdx.x] = x;
        sum[1][threadIdx.x] = y;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if ((int)threadIdx.x < w) {
                sum[0][threadIdx.x] += sum[0][threadIdx.x + w];
                sum[1][threadIdx.x] += sum[1][threadIdx.x + w];
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            const float l = sum[0][0] / (float)f.b;
            *f.loss = l;
            if (f.loss_out)
                *f.loss_out = l;
            optimize(f, f.n - 1, sum[1][0]);
        }
        return;
    }
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= f.n - 1)
        return;
    int k = 0;
    while (k < 16 && t >= f.seg[k + 1].off)
        ++k;
    const GradSeg &s = f.seg[k];
    const int i = (int)(t - s.off), row = i / s.cols, col = i - row * s.cols;
    float g = 0.f;
    if (s.part) {
        const bool past = col >= s.ld;
        const float *p = past ? s.rows + row : s.part + (int64_t)row * s.ld + col;
        const int64_t stride = past ? s.rows_stride : s.stride;
        int z = 0;
        for (; z + 4 <= s.splits; z += 4) {
            const float x0 = p[z * stride], x1 = p[(z + 1) * stride], x2 = p[(z + 2) * stride],
                        x3 = p[(z + 3) * stride];
            g = (((g + x0) + x1) + x2) + x3;
        }
        for (; z < s.splits; ++z)
            g += p[z * stride];
        if (past)
            g *= time_enc(f.omega[col - s.ld], f.beta[col - s.ld], 0.0);
    }
    optimize(f, t, g);
}

constexpr int kNParams = 17;

}  // namespace

struct tgm_trainer {
    tgm_model_t model = nullptr;
    int32_t M = 0, D_e = 0, D_t = 0, H = 0, nb = 0, D_m = 0, D_x = 0, Dq = 0, Dkv = 0;
    int32_t max_roots = 0, max_b = 0, max_nodes = 0;
    int32_t opt = TGM_OPT_ADAM;
    float lr = 1e-4f, beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f;
    int64_t steps = 0;
    int64_t n_params = 0;
    int64_t off[kNParams + 1] = {};
    float *theta = nullptr, *grad = nullptr, *m1 = nullptr, *m2 = nullptr;
    int32_t ldu = 0, ldx = 0;   // row strides of the (root, head) rows and of X
    // work space
    float *part = nullptr;      // split weight gradients, see train_grads
    float *Zs = nullptr, *Zd = nullptr, *dZsrc = nullptr, *dZdst = nullptr, *act = nullptr;
    float *dsc = nullptr, *lossv = nullptr, *loss = nullptr, *cq = nullptr;
    float *Q = nullptr, *Xo = nullptr, *dO = nullptr, *dXo = nullptr,
          *dQ = nullptr;
    float *U = nullptr, *abar = nullptr, *dbar = nullptr;   // [R x H x ldu]; dbar: dabar, then du
    bool slots = false;   // attention by slots (slot_form): the next three instead of U, abar, dbar
    float *rows = nullptr, *KV = nullptr, *dKV = nullptr;
    float *alpha = nullptr, *dKm = nullptr, *ds = nullptr;
    float *X = nullptr, *Hm = nullptr, *Gx = nullptr, *Gh = nullptr, *dGx = nullptr,
          *dGh = nullptr;
    SortBuffers sort;   // contributors by node-set position
    float *ds_head = nullptr, *ds_tail = nullptr;       // [sorted blocks x M] open runs
    float *p(int k) const { return theta + off[k]; }
    float *gr(int k) const { return grad + off[k]; }
};

namespace {

// Parts a weight gradient's reduction is cut into at most, and at least the
// length of a part.
constexpr int kMaxSplits = 32, kMinSplit = 256, kGradBlocks = 2048;

// out = x op(w): the products of the forward pass and of the gradients that
// go back through it.  x [m x k] (leading dimension ldx).
GemmProb mul(int m, int n, int k, const float *x, int ldx, const float *w, int ldw, float *out,
             int ldo, const float *bias = nullptr)
{
    GemmProb p;
    p.m = m;
    p.n = n;
    p.k = k;
    p.A = x;
    p.lda = ldx;
    p.B = w;
    p.ldb = ldw;
    p.C = out;
    p.ldc = ldo;
    p.bias = bias;
    return p;
}

// The same once per head, with the strides of one head in x, w and out
GemmProb heads(GemmProb p, int H, int64_t sx, int64_t sw, int64_t so, int64_t sbias = 0)
{
    p.batch = H;
    p.sA = sx;
    p.sB = sw;
    p.sC = so;
    p.sBias = sbias;
    return p;
}

// A weight gradient dw [m x n] = g^t x over at most `rows` rows, about
// `expect` of them, cut into parts of about `len` rows at *at (advanced),
// with g's row sums behind them.
GemmProb grad_of(int m, int n, int rows, int expect, int len, const float *g, int ldg,
                 const float *x, int ldx, float **at, int heads_ = 1)
{
    GemmProb p = mul(m, n, rows, g, ldg, x, ldx, *at, n);
    p.splits = std::max(1, std::min(kMaxSplits, expect / len));
    p.batch = heads_;
    p.split_stride = (int64_t)heads_ * m * n;
    p.sC = (int64_t)m * n;
    p.colsum = *at + p.splits * p.split_stride;
    p.colsum_stride = (int64_t)heads_ * m;
    p.sColsum = m;
    *at = p.colsum + p.splits * p.colsum_stride;
    return p;
}

template <int CE, int CT, int NC>
tgm_status_t att_launch(bool bwd, const AttArgs &a, hipStream_t s)
{
    const dim3 grid((unsigned)cdiv((int64_t)a.R * kWave, 256));
    if (bwd)
        TGM_LAUNCH((k_att_bwd<CE, CT, NC>), grid, dim3(256), 0, s, a);
    else
        TGM_LAUNCH((k_att_fwd<CE, CT, NC>), grid, dim3(256), 0, s, a);
    return TGM_OK;
}

// Rows of up to 192 edge features and 128 time codes keep 10 slots (70
// registers); wider ones take the larger row, 5 slots at a time.
constexpr int kAttTimeCodes = 6 * kWave;   // at most

bool att_narrow(int D_e, int D_t) { return D_e <= 3 * kWave && D_t <= 2 * kWave; }
int att_slots(int D_e, int D_t) { return att_narrow(D_e, D_t) ? 10 : 5; }

tgm_status_t att_dispatch(bool bwd, const AttArgs &a, hipStream_t s)
{
    if (att_narrow(a.D_e, a.D_t))
        return att_launch<3, 2, 10>(bwd, a, s);
    return att_launch<4, 6, 5>(bwd, a, s);
}

// Whether a trainer's attention runs by slots: rows wider than a wavefront's
// registers hold (D_e <= 256 always), and many heads.  Over (root, head) rows
// both the cost and the work space grow with the heads, by slots hardly
// (three arrays of R H ldu floats against R nb (Dkv + 4 M)), and rows that
// stay in the registers for all heads grow less than those loaded again for
// each.  A step in us, (root, head) rows / slots, M = 100, 172 or 186 edge
// features, 100 time codes:
//   10 slots (in registers)  600 events, 10 heads 340 / 417, 20: 462 / 486,
//     25: 520 / 523, 50: 881 / 709;  2,400 events, 10: 794 / 886, 20:
//     1,227 / 1,031, 50: 2,763 / 1,491
//   20 slots (loaded again)  600 events, 5: 478 / 570, 10: 741 / 667, 20:
//     1,243 / 835;  2,400 events, 5: 1,138 / 1,387, 10: 1,951 / 1,551, 20:
//     3,555 / 1,849
// At M = 8, 32 and 128, 8 heads and 20 slots: 334 / 266, 371 / 319 and 560 /
// 583 (600 events); at 64 slots 10 heads lie just past the line (1,789 /
// 1,996), 20 well past it (3,295 / 2,687).
constexpr int kSlotHeads = 32, kSlotHeadsAgain = 8;   // from so many heads on

bool slot_form(const tgm_model *m)
{
    return m->D_t > kAttTimeCodes ||
           m->H >= (m->nb > att_slots(m->D_e, m->D_t) ? kSlotHeadsAgain : kSlotHeads);
}

}  // namespace

// ======================================================================== API

extern "C" tgm_status_t tgm_trainer_destroy(tgm_trainer_t tr)
{
    if (!tr)
        return TGM_EINVAL;
    void *bufs[] = {tr->theta, tr->grad, tr->m1, tr->m2, tr->part, tr->Zs, tr->Zd, tr->dZsrc,
                    tr->dZdst, tr->act, tr->dsc, tr->lossv, tr->loss, tr->cq, tr->Q,
                    tr->Xo, tr->dO, tr->dXo, tr->dQ, tr->U, tr->abar, tr->dbar, tr->alpha,
                    tr->rows, tr->KV, tr->dKV, tr->dKm, tr->ds, tr->X, tr->Hm, tr->Gx, tr->Gh, tr->dGx, tr->dGh,
                    tr->ds_head, tr->ds_tail};
    for (void *b : bufs)
        (void)hipFree(b);
    sort_destroy(&tr->sort);
    delete tr;
    return TGM_OK;
}

extern "C" tgm_status_t tgm_trainer_create(tgm_model_t m, const tgm_weights *w,
                                           const tgm_predictor *pred, const tgm_optimizer *opt,
                                           void *stream, tgm_trainer_t *out)
{
    if (!out)
        return TGM_EINVAL;
    *out = nullptr;
    if (!m || !w || !pred || !opt || m->kind != TGM_MODEL_TGN)
        return TGM_EINVAL;
    if (!w->W_ih || !w->W_hh || !w->b_ih || !w->b_hh || !w->W_q || !w->b_q || !w->W_k ||
        !w->b_k || !w->W_v || !w->b_v || !w->W_o || !w->b_o || !pred->W_src || !pred->W_dst ||
        !pred->b_p || !pred->w_out)
        return TGM_EINVAL;
    if ((opt->kind != TGM_OPT_SGD && opt->kind != TGM_OPT_ADAM) || !(opt->lr >= 0.f) ||
        (opt->kind == TGM_OPT_ADAM &&
         (!(opt->beta1 >= 0.f && opt->beta1 < 1.f) || !(opt->beta2 >= 0.f && opt->beta2 < 1.f) ||
          !(opt->eps > 0.f))))
        return TGM_EINVAL;
    if (m->M > 128 || m->max_roots % 3 != 0)
        return TGM_EINVAL;
    tgm_trainer *tr = new tgm_trainer();
    tr->model = m;
    const int M = m->M, D_e = m->D_e, D_t = m->D_t, nb = m->nb;
    tr->M = M;
    tr->D_e = D_e;
    tr->D_t = D_t;
    tr->H = m->H;
    tr->nb = nb;
    tr->D_m = m->D_m;
    tr->D_x = m->D_x;
    tr->Dq = M + D_t;
    tr->Dkv = M + D_e + D_t;
    tr->max_roots = m->max_roots;
    tr->max_b = m->max_roots / 3;
    tr->max_nodes = m->max_nodes;
    tr->opt = opt->kind;
    tr->lr = opt->lr;
    tr->beta1 = opt->beta1;
    tr->beta2 = opt->beta2;
    tr->eps = opt->eps;
    const int64_t D_x = tr->D_x, Dq = tr->Dq, Dkv = tr->Dkv;
    const int64_t sizes[kNParams] = {3 * M * D_x, 3 * (int64_t)M * M, 3 * M, 3 * M, M * Dq, M,
                                     M * Dkv, M, M * Dkv, M, 2 * (int64_t)M * M, M,
                                     (int64_t)M * M, (int64_t)M * M, M, M, 1};
    for (int k = 0; k < kNParams; ++k)
        tr->off[k + 1] = tr->off[k] + sizes[k];
    tr->n_params = tr->off[kNParams];
    const int64_t R = tr->max_roots, B = tr->max_b, S = R * nb, C = tr->max_nodes;
    const int64_t n_items = R + S, H = tr->H, blocks = cdiv(n_items, kWave);
    tr->slots = slot_form(m);
    tr->ldu = round_up((int32_t)Dkv, 4);
    tr->ldx = round_up((int32_t)D_x, 4);
    int64_t part = 0;   // every split product and its row sums at kMaxSplits
    for (const auto &mn : {std::pair<int64_t, int64_t>{3 * M, D_x}, {3 * M, M}, {M, M}, {M, Dkv},
                           {M, Dkv}, {M, 2 * M}, {M, M}, {M, M}, {1, M}})
        part += kMaxSplits * mn.first * (mn.second + 1);
    tgm_status_t st = TGM_OK;
    auto alloc = [&](auto **ptr, int64_t count) {
        if (st == TGM_OK &&
            dev_malloc(ptr, sizeof(**ptr) * (size_t)std::max<int64_t>(count, 1)) != hipSuccess)
            st = TGM_ENOMEM;
    };
    alloc(&tr->theta, tr->n_params);
    alloc(&tr->grad, tr->n_params);
    alloc(&tr->m1, tr->n_params);
    alloc(&tr->m2, tr->n_params);
    alloc(&tr->part, part);
    alloc(&tr->Zs, B * M);
    alloc(&tr->Zd, 2 * B * M);
    alloc(&tr->dZsrc, B * M);
    alloc(&tr->dZdst, 2 * B * M);
    alloc(&tr->act, 2 * B * M);
    alloc(&tr->dsc, 2 * B);
    alloc(&tr->lossv, B);
    alloc(&tr->loss, 1);
    alloc(&tr->cq, M);
    alloc(&tr->Q, R * M);
    alloc(&tr->Xo, R * 2 * M);
    alloc(&tr->dO, R * M);
    alloc(&tr->dXo, R * 2 * M);
    alloc(&tr->dQ, R * M);
    if (tr->slots) {
        alloc(&tr->rows, S * Dkv);
        alloc(&tr->KV, S * 2 * M);
        alloc(&tr->dKV, S * 2 * M);
    } else {
        alloc(&tr->U, R * H * tr->ldu);
        alloc(&tr->abar, R * H * tr->ldu);
        alloc(&tr->dbar, R * H * tr->ldu);
    }
    alloc(&tr->alpha, R * H * nb);
    alloc(&tr->dKm, S * M);
    alloc(&tr->ds, C * M);
    alloc(&tr->X, C * tr->ldx);
    alloc(&tr->Hm, C * M);
    alloc(&tr->Gx, C * 3 * M);
    alloc(&tr->Gh, C * 3 * M);
    alloc(&tr->dGx, C * 3 * M);
    alloc(&tr->dGh, C * 3 * M);
    alloc(&tr->ds_head, blocks * M);
    alloc(&tr->ds_tail, blocks * M);
    if (st == TGM_OK)
        st = sort_create(&tr->sort, n_items, C, [&](auto **ptr, int64_t n) {
            alloc(ptr, n);
            return st == TGM_OK;
        });
    if (st != TGM_OK) {
        tgm_trainer_destroy(tr);
        return st;
    }
    // the parameter vector: the model's weights and the predictor's
    hipStream_t s = as_stream(stream);
    const float *src[kNParams] = {w->W_ih, w->W_hh, w->b_ih, w->b_hh, w->W_q, w->b_q,
                                  w->W_k, w->b_k, w->W_v, w->b_v, w->W_o, w->b_o,
                                  pred->W_src, pred->W_dst, pred->b_p, pred->w_out, nullptr};
    for (int k = 0; k < kNParams && st == TGM_OK; ++k)
        if (src[k])
            st = upload(tr->p(k), src[k], sizeof(float) * (size_t)sizes[k]);
    if (st == TGM_OK)
        st = upload(tr->p(16), &pred->b_out, sizeof(float));
    if (st == TGM_OK &&
        (hipMemsetAsync(tr->m1, 0, sizeof(float) * tr->n_params, s) != hipSuccess ||
         hipMemsetAsync(tr->m2, 0, sizeof(float) * tr->n_params, s) != hipSuccess ||
         hipMemsetAsync(tr->grad, 0, sizeof(float) * tr->n_params, s) != hipSuccess ||
         hipMemsetAsync(tr->loss, 0, sizeof(float), s) != hipSuccess ||
         hipStreamSynchronize(s) != hipSuccess))
        st = TGM_EDEVICE;
    if (st != TGM_OK) {
        tgm_trainer_destroy(tr);
        return st;
    }
    *out = tr;
    return TGM_OK;
}

extern "C" tgm_status_t tgm_trainer_info(tgm_trainer_t tr, int64_t *n_params, int64_t *sizes,
                                         int64_t *steps)
{
    if (!tr)
        return TGM_EINVAL;
    if (n_params)
        *n_params = tr->n_params;
    if (sizes)
        for (int k = 0; k < kNParams; ++k)
            sizes[k] = tr->off[k + 1] - tr->off[k];
    if (steps)
        *steps = tr->steps;
    return TGM_OK;
}

extern "C" tgm_status_t tgm_trainer_read(tgm_trainer_t tr, float *params, float *grad,
                                         float *loss, void *stream)
{
    if (!tr)
        return TGM_EINVAL;
    hipStream_t s = as_stream(stream);
    const size_t bytes = sizeof(float) * (size_t)tr->n_params;
    if (params)
        TGM_HIP(hipMemcpyAsync(params, tr->theta, bytes, hipMemcpyDeviceToDevice, s));
    if (grad)
        TGM_HIP(hipMemcpyAsync(grad, tr->grad, bytes, hipMemcpyDeviceToDevice, s));
    if (loss)
        TGM_HIP(hipMemcpyAsync(loss, tr->loss, sizeof(float), hipMemcpyDeviceToDevice, s));
    return TGM_OK;
}

tgm_status_t tgm::train_step_launch(tgm_trainer_t tr, tgm_model_t m, tgm_graph_t g, int32_t b,
                                    const tgm_sample_buffers &sb, const tgm_fetch_buffers &fb,
                                    const float *mem_new, const float *h, int32_t cap,
                                    float *loss_out, hipStream_t s)
{
    if (!tr || !m || !g || tr->model != m || b < 0 || cap < 0 || !mem_new || !h)
        return TGM_EINVAL;
    if (b == 0)
        return TGM_OK;
    if (3 * b > tr->max_roots || cap > tr->max_nodes)
        return TGM_ESIZE;
    if (!sb.root_pos || !sb.root_ts || !sb.nbr_pos || !sb.eid || !sb.nts || !sb.cnt ||
        !sb.n_nodes || !fb.mem || !fb.mem_ts || !fb.mail || !fb.mail_ts || !fb.ver)
        return TGM_EINVAL;
    if (g->D_e != tr->D_e || (tr->D_e > 0 && !g->efeat))
        return TGM_EINVAL;
    const int M = tr->M, nb = tr->nb, R = 3 * b, H = tr->H, dh = M / H;
    const int Dq = tr->Dq, Dkv = tr->Dkv, D_x = tr->D_x, ldu = tr->ldu, ldx = tr->ldx;
    const int64_t S = (int64_t)R * nb, n_items = R + S;
    const float *W_ih = tr->p(0), *W_hh = tr->p(1), *b_ih = tr->p(2), *b_hh = tr->p(3);
    const float *W_q = tr->p(4), *b_q = tr->p(5), *W_k = tr->p(6), *b_k = tr->p(7);
    const float *W_v = tr->p(8), *b_v = tr->p(9), *W_o = tr->p(10), *b_o = tr->p(11);
    const float *W_src = tr->p(12), *W_dst = tr->p(13);
    const float *h_rest = h + (int64_t)b * M;
    float *s_v = tr->Xo + M;   // the roots' new memories, rows of 2M

    RowArgs ra{R, nb, M, tr->D_m, tr->D_t, cap, ldx, (int)cdiv(R, 4), (int)cdiv(cap, 4),
               (int)sort_tiles(n_items), sb.root_pos, sb.nbr_pos, sb.cnt, sb.n_nodes, fb.ver,
               fb.mem_ts, fb.mail_ts, m->omega, m->beta, mem_new, fb.mem, fb.mail, W_q, b_q,
               tr->Xo, tr->X, tr->Hm, tr->cq, sort_plan(tr->sort, n_items)};
    TGM_LAUNCH(k_train_rows,
               dim3((unsigned)(ra.n_root + ra.n_node + ra.n_key + cdiv(M, 4))), dim3(256), 0, s,
               ra);
    const SlotArgs sl{R, nb, M, tr->D_e, tr->D_t, H, 1.f / sqrtf((float)dh), sb.cnt, sb.nbr_pos,
                      sb.eid, sb.root_ts, sb.nts, m->omega, m->beta, mem_new, g->efeat, tr->Q,
                      tr->dXo, tr->rows, tr->KV, tr->dKV, tr->alpha, tr->Xo, tr->dQ};
    const dim3 per_root((unsigned)cdiv((int64_t)R * kWave, 256));
    if (tr->slots)
        TGM_LAUNCH(k_slot_rows, dim3((unsigned)cdiv(S, 4)), dim3(256), 0, s, sl);
    // the predictor's layers, the queries and the GRU's gates (by slots: the
    // keys and values too)
    {
        GemmProb g[7] = {mul(b, M, M, h, M, W_src, M, tr->Zs, M),
                         mul(2 * b, M, M, h_rest, M, W_dst, M, tr->Zd, M),
                         mul(R, M, M, s_v, 2 * M, W_q, Dq, tr->Q, M, tr->cq),
                         mul(cap, 3 * M, D_x, tr->X, ldx, W_ih, D_x, tr->Gx, 3 * M, b_ih),
                         mul(cap, 3 * M, M, tr->Hm, M, W_hh, M, tr->Gh, 3 * M, b_hh)};
        g[3].live = g[4].live = sb.n_nodes;
        if (tr->slots) {
            g[5] = mul((int)S, M, Dkv, tr->rows, Dkv, W_k, Dkv, tr->KV, 2 * M, b_k);
            g[6] = mul((int)S, M, Dkv, tr->rows, Dkv, W_v, Dkv, tr->KV + M, 2 * M, b_v);
        }
        TGM_TRY_STATUS(gemm_launch(false, true, g, tr->slots ? 7 : 5, s));
    }
    PredArgs pa{b, M, tr->Zs, tr->Zd, tr->p(14), tr->p(15), tr->p(16), tr->dZsrc, tr->dZdst,
                tr->act, tr->dsc, tr->lossv};
    TGM_LAUNCH(k_pred, dim3((unsigned)cdiv((int64_t)b * kWave, 256)), dim3(256), 0, s, pa);
    // u = W_k^t q per head; the gradient of the output projection, h's where
    // its ReLU let the value through
    {
        GemmProb g[3] = {
            heads(mul(R, Dkv, dh, tr->Q, M, W_k, Dkv, tr->U, H * ldu), H, dh, (int64_t)dh * Dkv,
                  ldu),
            mul(b, M, M, tr->dZsrc, M, W_src, M, tr->dO, M),
            mul(2 * b, M, M, tr->dZdst, M, W_dst, M, tr->dO + (int64_t)b * M, M)};
        g[1].gate = h;
        g[2].gate = h_rest;
        g[1].ldg = g[2].ldg = M;
        const int u = tr->slots ? 1 : 0;   // (no u by slots)
        TGM_TRY_STATUS(gemm_launch(false, false, g + u, 3 - u, s));
    }
    AttArgs aa{R, nb, M, tr->D_e, tr->D_t, H, ldu, 1.f / sqrtf((float)dh), sb.cnt, sb.root_pos,
               sb.nbr_pos, sb.eid, sb.root_ts, sb.nts, m->omega, m->beta, mem_new, g->efeat,
               tr->U, tr->alpha, tr->abar, tr->dbar, tr->dKm};
    if (tr->slots) {
        TGM_LAUNCH(k_slot_fwd, per_root, dim3(256), 0, s, sl);
    } else {   // o = W_v abar + b_v per head (zero without neighbours)
        TGM_TRY_STATUS(att_dispatch(false, aa, s));
        GemmProb p = heads(mul(R, dh, Dkv, tr->abar, H * ldu, W_v, Dkv, tr->Xo, 2 * M, b_v), H,
                           ldu, (int64_t)dh * Dkv, dh, dh);
        p.row_on = sb.cnt;
        p.zero_cols = dh;
        TGM_TRY_STATUS(gemm_launch(false, true, &p, 1, s));
    }
    {   // gradient of [o || s'_v]; o is no output of a root without neighbours
        GemmProb p = mul(R, 2 * M, M, tr->dO, M, W_o, 2 * M, tr->dXo, 2 * M);
        p.row_on = sb.cnt;
        p.zero_cols = M;
        TGM_TRY_STATUS(gemm_launch(false, false, &p, 1, s));
    }
    GemmProb v = mul(R, M, M, tr->dQ, M, W_q, Dq, tr->dXo + M, 2 * M);   // the query's part
    v.accumulate = 1;
    if (tr->slots) {   // dq, dK and dV; then the slots' gradient of s'_u and the roots' of s'_v
        TGM_LAUNCH(k_slot_bwd, per_root, dim3(256), 0, s, sl);
        const GemmProb k = mul((int)S, M, M, tr->dKV, 2 * M, W_k, Dkv, tr->dKm, M);
        TGM_TRY_STATUS(gemm_launch(false, false, &k, 1, s));
        GemmProb p[2] = {mul((int)S, M, M, tr->dKV + M, 2 * M, W_v, Dkv, tr->dKm, M), v};
        p[0].accumulate = 1;
        TGM_TRY_STATUS(gemm_launch(false, false, p, 2, s));
    } else {   // dabar = W_v^t do per head
        const GemmProb p = heads(mul(R, Dkv, dh, tr->dXo, 2 * M, W_v, Dkv, tr->dbar, H * ldu), H,
                                 dh, (int64_t)dh * Dkv, ldu);
        TGM_TRY_STATUS(gemm_launch(false, false, &p, 1, s));
        TGM_TRY_STATUS(att_dispatch(true, aa, s));
        // dq = W_k du per head, then its part of the roots' gradient of s'_v
        const GemmProb q = heads(mul(R, dh, Dkv, tr->dbar, H * ldu, W_k, Dkv, tr->dQ, M), H, ldu,
                                 (int64_t)dh * Dkv, dh);
        TGM_TRY_STATUS(gemm_launch(false, true, &q, 1, s));
        TGM_TRY_STATUS(gemm_launch(false, false, &v, 1, s));
    }
    // each node's gradient: its contributors' rows, sorted by node
    TGM_TRY_STATUS(sort_launch(tr->sort, ra.sort, s));
    TGM_LAUNCH(k_ds_block, dim3((unsigned)cdiv(n_items, 256)), dim3(256), 0, s, n_items, cap, M,
               R, tr->sort.out_keys, tr->sort.out_vals, tr->dXo, tr->dKm, tr->ds, tr->ds_head,
               tr->ds_tail);
    TGM_LAUNCH(k_ds_join, dim3((unsigned)cdiv(n_items, 256)), dim3(256), 0, s, n_items, cap, M,
               tr->sort.out_keys, tr->ds_head, tr->ds_tail, tr->ds);
    // memory updater (GRU) backward
    TGM_LAUNCH(k_gru_bwd, dim3((unsigned)cdiv((int64_t)cap * M, 256)), dim3(256), 0, s,
               sb.n_nodes, cap, M, fb.ver, tr->Gx, tr->Gh, tr->Hm, tr->ds, tr->dGx, tr->dGh);
    // every weight gradient, then the optimizer
    // (a batch's node set has about as many nodes as roots: hubs recur)
    const int nodes = std::min(cap, R + R / 2);
    float *at = tr->part;
    const int64_t kv_rows = tr->slots ? cdiv(M, 64) * S : H * cdiv(dh, 64) * R;
    const int64_t tiles = cdiv(3 * M, 64) * (cdiv(D_x, 64) + cdiv(M, 112)) * nodes +
                          2 * cdiv(Dkv, 112) * kv_rows + 3 * cdiv(M, 64) * R;
    const int len = (int)std::max<int64_t>(kMinSplit, tiles / kGradBlocks);
    GemmProb w[9] = {
        grad_of(3 * M, D_x, cap, nodes, len, tr->dGx, 3 * M, tr->X, ldx, &at),
        grad_of(3 * M, M, cap, nodes, len, tr->dGh, 3 * M, tr->Hm, M, &at),
        grad_of(M, M, R, R, len, tr->dQ, M, s_v, 2 * M, &at),
        tr->slots ? grad_of(M, Dkv, (int)S, (int)S, len, tr->dKV, 2 * M, tr->rows, Dkv, &at)
                  : grad_of(dh, Dkv, R, R, len, tr->Q, M, tr->dbar, H * ldu, &at, H),
        tr->slots ? grad_of(M, Dkv, (int)S, (int)S, len, tr->dKV + M, 2 * M, tr->rows, Dkv, &at)
                  : grad_of(dh, Dkv, R, R, len, tr->dXo, 2 * M, tr->abar, H * ldu, &at, H),
        grad_of(M, 2 * M, R, R, len, tr->dO, M, tr->Xo, 2 * M, &at),
        grad_of(M, M, b, b, len, tr->dZsrc, M, h, M, &at),
        grad_of(M, M, 2 * b, 2 * b, len, tr->dZdst, M, h_rest, M, &at),
        grad_of(1, M, 2 * b, 2 * b, len, tr->dsc, 1, tr->act, M, &at)};
    w[0].live = w[1].live = sb.n_nodes;
    if (!tr->slots) {
        w[3].sA = w[4].sA = dh;
        w[3].sB = w[4].sB = ldu;
    }
    TGM_TRY_STATUS(gemm_launch(true, false, w, 9, s));
    tr->steps++;
    FinishArgs f{};
    // the tensors in vector order: the product that gives them, whether its
    // row sums do, and the tensor's row length
    const struct {
        int prob, sums, cols;
    } src[kNParams] = {{0, 0, D_x}, {1, 0, M}, {0, 1, 1}, {1, 1, 1}, {2, 0, Dq},   {2, 1, 1},
                       {3, 0, Dkv}, {-1, 0, 1}, {4, 0, Dkv}, {4, 1, 1}, {5, 0, 2 * M}, {5, 1, 1},
                       {6, 0, M},   {7, 0, M},  {6, 1, 1},   {8, 0, M}, {-1, 0, 1}};
    for (int k = 0; k < kNParams; ++k) {
        GradSeg &d = f.seg[k];
        d.off = tr->off[k];
        d.cols = d.ld = src[k].cols;
        if (src[k].prob < 0)
            continue;
        const GemmProb &p = w[src[k].prob];
        d.splits = p.splits;
        d.part = src[k].sums ? p.colsum : p.C;
        d.stride = src[k].sums ? p.colsum_stride : p.split_stride;
        d.rows = p.colsum;
        d.rows_stride = p.colsum_stride;
        if (k == 4)
            d.ld = M;
    }
    f.n = tr->n_params;
    f.theta = tr->theta;
    f.grad = tr->grad;
    f.m1 = tr->m1;
    f.m2 = tr->m2;
    f.omega = m->omega;
    f.beta = m->beta;
    f.adam = tr->opt == TGM_OPT_ADAM;
    f.lr = tr->lr;
    f.b1 = tr->beta1;
    f.b2 = tr->beta2;
    f.eps = tr->eps;
    f.c1 = (float)(1.0 - std::pow((double)tr->beta1, (double)tr->steps));
    f.c2 = (float)(1.0 - std::pow((double)tr->beta2, (double)tr->steps));
    f.lossv = tr->lossv;
    f.dsc = tr->dsc;
    f.b = b;
    f.loss = tr->loss;
    f.loss_out = loss_out;
    TGM_LAUNCH(k_grad_finish, dim3((unsigned)cdiv(f.n, 256) + 1), dim3(256), 0, s, f);
    ModelParams mp{W_ih, W_hh, b_ih, b_hh, W_q, b_q, W_k, b_k, W_v, b_v, W_o, b_o};
    return model_repack(m, mp, s);
}

extern "C" tgm_status_t tgm_train_step(tgm_trainer_t tr, tgm_model_t m, tgm_graph_t g, int32_t b,
                                       const tgm_sample_buffers *sb, const tgm_fetch_buffers *fb,
                                       const float *mem_new, const float *h, int32_t cap,
                                       float *loss, void *stream)
{
    if (!sb || !fb)
        return TGM_EINVAL;
    return tgm::train_step_launch(tr, m, g, b, *sb, *fb, mem_new, h, cap, loss,
                                  as_stream(stream));
}

extern "C" tgm_status_t tgm_state_set_training(tgm_state_t st, tgm_trainer_t tr, float *loss_log,
                                               int64_t log_len)
{
    if (!st || (tr && loss_log && log_len < 1))
        return TGM_EINVAL;
    st->trainer = tr;
    st->loss_log = tr ? loss_log : nullptr;
    st->loss_log_len = tr && loss_log ? log_len : 0;
    return TGM_OK;
}
