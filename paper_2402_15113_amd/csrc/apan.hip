// APAN, the third model family of the paper's experiments (Sec. 5; App. B:
// an RNN memory updater with an attention mechanism and asynchronous
// propagation).  Per node a mailbox of the K latest mails (a ring of K rows
// and times, its head and count); the mails an event generates for its two
// endpoints go to the endpoints and to their sampled neighbours; a node's
// memory update attends over its mailbox and feeds the aggregate to a GRU;
// the embedding is the updated memory.  Mail deliveries and memory writes of
// iteration i form its write set, committed before the fetch of iteration
// i + s + 1 (Eq. 2), as for the other families.
//
// One call per iteration (tgm_apan_step): commit the due write sets, gather
// the node set's memories and mailboxes, the attention and the GRU, the
// embeddings, and the staging of the iteration's write set.  The deliveries
// of an iteration are stably sorted by node; the delivery index is
// monotone in (t, e, role, slot), so each node's segment is in mail order and
// its last K entries are the ones its mailbox keeps.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "common.h"
#include "sort.h"

using namespace tgm;

namespace {

constexpr int kApanMaxK = 16;

struct ApanRows {   // the node set's rows
    const int32_t *nodes, *n_nodes;
    int cap, M, D_m, D_t, K;
    const float *mem, *mb;          // tables [N x M], [N x K x D_m]
    const double *mem_ts, *mb_ts;   // [N], [N x K]
    const int32_t *ver, *mb_head, *mb_cnt;
    float *f_mem, *f_mb;            // fetched [cap x M], [cap x K x D_m] (oldest first)
    double *f_mem_ts, *f_mb_ts;     // [cap], [cap x K]
    int32_t *f_ver, *f_cnt;         // [cap]
    int32_t *flag;                  // staging flags of the iteration's slot [n_flag]
    int n_flag, n_gather;           // workgroups of the gather
    // attention
    const float *u;                 // [cap x D_x]
    const double *omega, *beta;
    float scale;
    float *X;                       // [cap x D_x]
    double *t_new, *new_ts;         // [cap]; new_ts may be null
};

// Gather of the node set's memory rows, times, versions and mail counts, one
// wavefront per node; the workgroups past n_gather clear the staging flags.
__global__ __launch_bounds__(256) void k_apan_gather(ApanRows a)
{
    if ((int)blockIdx.x >= a.n_gather) {
        const int i = ((int)blockIdx.x - a.n_gather) * 256 + threadIdx.x;
        if (i < a.n_flag)
            a.flag[i] = 0;
        return;
    }
    const int p = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (p >= min(*a.n_nodes, a.cap))
        return;
    const int v = a.nodes[p], M = a.M;
    wave_copy_row(a.f_mem + (int64_t)p * M, a.mem + (int64_t)v * M, M, lane);
    if (lane == 0) {
        a.f_mem_ts[p] = a.mem_ts[v];
        a.f_ver[p] = a.ver[v];
        a.f_cnt[p] = a.mb_cnt[v];
    }
}

// The fetch of the mailboxes and the attention over them, one wavefront per
// node.  u = W_k^t q has been formed for the node, so the score of mail j is
// u . [mail_j || phi(t_newest - t_j)] / sqrt(M); q . b_k shifts all of a
// node's scores alike, which the softmax ignores.  Writes the mails oldest
// first (f_mb, f_mb_ts), t_newest and the GRU's input row X[p] = [sum_j
// alpha_j mail_j || phi(t_newest - mem_ts)]; a node without mail gets no row
// (the GRU keeps its memory).
//
// A node's mails stay in the wavefront's registers (lane l holds columns l +
// 64 i of each) from their one load to their copy and their weighted sum.  As
// a copy to f_mb and an attention that read f_mb twice the two launches took
// 65 us at a batch of 1,000 (2,800 nodes, 32 MB of mails); this one 16 us.
template <int NC, int CD>   // K <= NC, D_m <= 64 CD
__global__ __launch_bounds__(256) void k_apan_attn(ApanRows a)
{
    const int p = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (p >= a.cap)
        return;
    const int D_m = a.D_m, D_t = a.D_t, D_x = D_m + D_t, K = a.K;
    const bool in = p < min(*a.n_nodes, a.cap);
    const int v = in ? a.nodes[p] : 0;
    const int cnt = in ? __builtin_amdgcn_readfirstlane(a.mb_cnt[v]) : 0;
    if (cnt == 0) {
        if (lane == 0) {
            const double t = in ? a.mem_ts[v] : 0.0;
            a.t_new[p] = t;
            if (a.new_ts)
                a.new_ts[p] = t;
        }
        return;
    }
    const int first = ((__builtin_amdgcn_readfirstlane(a.mb_head[v]) - cnt) % K + K) % K;
    auto slot = [&](int j) { return first + j < K ? first + j : first + j - K; };
    const float *box = a.mb + (int64_t)v * K * D_m;
    float x[NC][CD], u[CD];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const float *row = box + (int64_t)slot(min(j, cnt - 1)) * D_m;
#pragma unroll
        for (int i = 0; i < CD; ++i)
            x[j][i] = row[min(lane + kWave * i, D_m - 1)];
    }
    const double tj = a.mb_ts[(int64_t)v * K + slot(min(lane, cnt - 1))];
    const float *up = a.u + (int64_t)p * D_x;
#pragma unroll
    for (int i = 0; i < CD; ++i)
        u[i] = up[min(lane + kWave * i, D_m - 1)];
    const double mts = a.mem_ts[v];
    issue_fence();
    if (lane < cnt)
        a.f_mb_ts[(int64_t)p * K + lane] = tj;
    const long long tb = __double_as_longlong(tj);
    const int tlo = (int)tb, thi = (int)(tb >> 32);
    auto time_of = [&](int j) {
        const unsigned l = (unsigned)__builtin_amdgcn_readlane(tlo, j);
        const long long h = __builtin_amdgcn_readlane(thi, j);
        return __longlong_as_double((h << 32) | l);
    };
    const double tref = time_of(cnt - 1);
    float part[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j)
        part[j] = 0.f;
    for (int d = lane; d < D_t; d += kWave) {   // while the rows are on their way
        const float ud = up[D_m + d];
        const double om = a.omega[d], be = a.beta[d];
        a.X[(int64_t)p * D_x + D_m + d] = time_enc(om, be, tref - mts);
#pragma unroll
        for (int j = 0; j < NC; ++j)
            if (j < cnt)
                part[j] = fmaf(ud, time_enc(om, be, tref - time_of(j)), part[j]);
    }
#pragma unroll
    for (int i = 0; i < CD; ++i)
        u[i] = lane + kWave * i < D_m ? u[i] : 0.f;
    float mine = -INFINITY;   // lane j < cnt: the score of mail j
#pragma unroll
    for (int j = 0; j < NC; ++j)
        if (j < cnt) {
            float *row = a.f_mb + ((int64_t)p * K + j) * D_m;
#pragma unroll
            for (int i = 0; i < CD; ++i) {
                part[j] = fmaf(u[i], x[j][i], part[j]);
                if (lane + kWave * i < D_m)
                    row[lane + kWave * i] = x[j][i];
            }
            const float sc = wave_total(part[j]) * a.scale;
            mine = lane == j ? sc : mine;
        }
    float mx = mine;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        mx = fmaxf(mx, __shfl_xor(mx, o, kWave));
    const float ex = lane < cnt ? expf(mine - mx) : 0.f;
    const float al = ex / wave_total(ex);
    float acc[CD];
#pragma unroll
    for (int i = 0; i < CD; ++i)
        acc[i] = 0.f;
#pragma unroll
    for (int j = 0; j < NC; ++j)
        if (j < cnt) {
            const float w = lane_value(al, j);
#pragma unroll
            for (int i = 0; i < CD; ++i)
                acc[i] = fmaf(w, x[j][i], acc[i]);
        }
#pragma unroll
    for (int i = 0; i < CD; ++i)
        if (lane + kWave * i < D_m)
            a.X[(int64_t)p * D_x + lane + kWave * i] = acc[i];
    if (lane == 0) {
        a.t_new[p] = tref;
        if (a.new_ts)
            a.new_ts[p] = tref;
    }
}

// The query projection's constant part W_q phi(0) + b_q, one wavefront per unit
__global__ __launch_bounds__(256) void k_apan_cq(int M, int D_t, const float *__restrict__ W_q,
                                                 const float *__restrict__ b_q,
                                                 const double *__restrict__ beta,
                                                 double *__restrict__ cq)
{
    const int d = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6), lane = threadIdx.x & 63;
    if (d >= M)
        return;
    double acc = 0.0;
    for (int t = lane; t < D_t; t += kWave)
        acc += (double)W_q[(int64_t)d * (M + D_t) + M + t] * cos(beta[t]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        acc += __shfl_xor(acc, o, kWave);
    if (lane == 0)
        cq[d] = acc + (double)b_q[d];
}

// The key projection with the query's folded in, in fp64 at creation:
// u = W_k^t (W_q [s || phi(0)] + b_q) = Wqk^t s + c_u, Wqk [M x D_x].
__global__ __launch_bounds__(256) void k_apan_fold(int M, int D_x, int D_t,
                                                   const float *__restrict__ W_q,
                                                   const double *__restrict__ cq,
                                                   const float *__restrict__ W_k,
                                                   float *__restrict__ Wqk,
                                                   float *__restrict__ c_u)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x, m = blockIdx.y;
    if (x >= D_x)
        return;
    double acc = 0.0;
    for (int d = 0; d < M; ++d)
        acc += (m < M ? (double)W_q[(int64_t)d * (M + D_t) + m] : cq[d]) *
               (double)W_k[(int64_t)d * D_x + x];
    if (m < M)
        Wqk[(int64_t)m * D_x + x] = (float)acc;
    else
        c_u[x] = (float)acc;
}

// The GRU cell from the gate pre-activations Gx = X W_ih^t + b_ih and
// Gh = mem W_hh^t + b_hh, one thread per (node, unit); nodes without mail
// keep their memory.
__global__ __launch_bounds__(256) void k_apan_gru(const int32_t *__restrict__ n_nodes, int cap,
                                                  int M, const int32_t *__restrict__ f_cnt,
                                                  const float *__restrict__ Gx,
                                                  const float *__restrict__ Gh,
                                                  const float *__restrict__ f_mem,
                                                  float *__restrict__ s_new)
{
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= (int64_t)cap * M)
        return;
    const int p = (int)(t / M), j = (int)(t % M);
    if (p >= min(*n_nodes, cap))
        return;
    const float h = f_mem[(int64_t)p * M + j];
    if (f_cnt[p] == 0) {
        s_new[(int64_t)p * M + j] = h;
        return;
    }
    const int64_t o = (int64_t)p * 3 * M;
    const float r = 1.f / (1.f + expf(-(Gx[o + j] + Gh[o + j])));
    const float z = 1.f / (1.f + expf(-(Gx[o + M + j] + Gh[o + M + j])));
    const float n = tanhf(Gx[o + 2 * M + j] + r * Gh[o + 2 * M + j]);
    s_new[(int64_t)p * M + j] = (1.f - z) * n + z * h;
}

// What follows the new memories, one launch: the sort keys of the deliveries
// (first, they take longest), the embeddings h[r] = s_new[root_pos[r]], and
// the staged memory rows of the batch's endpoints.
//   Delivery d = ((k 2 + role)(nb + 1) + slot) of batch event k: the mail of
// endpoint v (role 0: src, 1: dst) to v (slot 0) or to its neighbour in
// sampled slot (slot - 1) of root role b + k.  Sort key: the node, or N (past
// every node) for empty and unused deliveries.
//   Memory rows by node-set position: flag[p] = 1 and the new memory for every
// position that is a source or destination, one wavefront per endpoint
// occurrence (all occurrences of a node write the same values).
struct AfterArgs {
    int32_t b, nb, propagate, N, M;
    int n_keys, n_embed;   // workgroups of the first two parts
    const int32_t *root, *nbr, *cnt, *root_pos, *nodes;
    const float *s_new;
    const double *t_new;
    float *h;
    int32_t *flag, *node;
    float *r_mem;
    double *r_ts;
    SortPlan sort;
};

__global__ __launch_bounds__(256) void k_apan_after(AfterArgs a)
{
    __shared__ int32_t count[1 << kSortDigit];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, M = a.M;
    int blk = blockIdx.x;
    if (blk < a.n_keys) {
        const int per = a.nb + 1;
        sort_keys_tile(a.sort, blk, count, [&](int64_t d) {
            const int slot = (int)(d % per), kr = (int)(d / per), role = kr & 1, k = kr >> 1;
            const int r = role * a.b + k;
            int32_t w = a.N;
            if (slot == 0)
                w = a.root[r];
            else if (a.propagate && slot - 1 < a.cnt[r])
                w = a.nbr[(int64_t)r * a.nb + slot - 1];
            return min((uint32_t)w, (uint32_t)a.N);
        });
        return;
    }
    blk -= a.n_keys;
    if (blk < a.n_embed) {
        const int r = blk * 4 + wave;
        if (r < 3 * a.b)
            wave_copy_row(a.h + (int64_t)r * M, a.s_new + (int64_t)a.root_pos[r] * M, M, lane);
        return;
    }
    const int e = (blk - a.n_embed) * 4 + wave;
    if (e >= 2 * a.b)
        return;
    const int p = a.root_pos[e];
    wave_copy_row(a.r_mem + (int64_t)p * M, a.s_new + (int64_t)p * M, M, lane);
    if (lane == 0) {
        a.flag[p] = 1;
        a.node[p] = a.nodes[p];
        a.r_ts[p] = a.t_new[p];
    }
}

struct StageArgs2 {
    int32_t b, nb, M, D_e, D_m, K, N;
    int64_t first;
    const uint32_t *keys;       // sorted
    const int32_t *dels;        // their deliveries
    const int32_t *root_pos;    // [3b]
    const float *s_new, *efeat;
    const double *t;
    // the slot's delivery rows, indexed by sorted position
    int32_t *d_node, *d_rank, *d_keep;   // d_keep: count kept for the node, 0 = dropped
    float *d_mail;
    double *d_t;
};

// One wavefront per sorted delivery: rows that the node's mailbox keeps (the
// last K of its segment) are written with their rank among the kept ones.
// Lane l looks at the key K - l places before (l <= K) or l - K after, which
// is as far as a kept row's segment matters (K <= 16).
__global__ __launch_bounds__(256) void k_apan_stage_mail(StageArgs2 a, int64_t n)
{
    const int64_t i = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63, K = a.K;
    if (i >= n)
        return;
    const uint32_t w = a.keys[i];
    const int64_t at = i - K + lane;
    const bool same = lane <= 2 * K && at >= 0 && at < n &&
                      a.keys[min(max(at, (int64_t)0), n - 1)] == w;
    // the segment is contiguous: its rows before and after this one, up to K
    const uint64_t near = __ballot(same);
    const int before = __popcll(near & ((uint64_t(1) << K) - 1));
    const int after = __popcll(near >> (K + 1));
    if (w >= (uint32_t)a.N || after >= K) {
        if (lane == 0)
            a.d_keep[i] = 0;
        return;
    }
    const int keep = min(before + 1 + after, K), rank = keep - 1 - after;
    const int d = a.dels[i];
    const int per = a.nb + 1;
    const int kr = d / per, role = kr & 1, k = kr >> 1;
    const int pv = a.root_pos[role * a.b + k], po = a.root_pos[(1 - role) * a.b + k];
    const int M = a.M, D_e = a.D_e;
    float *row = a.d_mail + i * a.D_m;
    wave_copy_row(row, a.s_new + (int64_t)pv * M, M, lane);
    wave_copy_row(row + M, a.s_new + (int64_t)po * M, M, lane);
    if (D_e > 0)
        wave_copy_row(row + 2 * M, a.efeat + (a.first + k) * D_e, D_e, lane);
    if (lane == 0) {
        a.d_node[i] = (int32_t)w;
        a.d_rank[i] = rank;
        a.d_keep[i] = keep;
        a.d_t[i] = a.t[a.first + k];
    }
}

__global__ __launch_bounds__(256) void k_apan_clear_flags(int32_t *__restrict__ flag, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        flag[i] = 0;
}

// ------------------------------------------------------------- commit
// One write set's memory rows (by node-set position, one wavefront each), and
// its kept mails into the ring at head + rank (heads are updated after)
struct CommitArgs {
    int cap, n_mem, M, D_m, K;   // n_mem: workgroups of the memory rows
    int64_t iter, n_del;
    const int32_t *flag, *node, *d_node, *d_rank, *d_keep, *head;
    const float *r_mem, *d_mail;
    const double *r_ts, *d_t;
    float *mem, *mb;
    double *mem_ts, *mb_ts;
    int32_t *ver;
};

__global__ __launch_bounds__(256) void k_apan_commit(CommitArgs a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((int)blockIdx.x < a.n_mem) {
        const int p = (int)blockIdx.x * 4 + wave;
        if (p >= a.cap || !a.flag[p])
            return;
        const int v = a.node[p];
        wave_copy_row(a.mem + (int64_t)v * a.M, a.r_mem + (int64_t)p * a.M, a.M, lane);
        if (lane == 0) {
            a.mem_ts[v] = a.r_ts[p];
            a.ver[v] = (int32_t)a.iter;
        }
        return;
    }
    const int64_t i = ((int64_t)blockIdx.x - a.n_mem) * 4 + wave;
    if (i >= a.n_del || a.d_keep[i] == 0)
        return;
    const int v = a.d_node[i];
    const int slot = (a.head[v] + a.d_rank[i]) % a.K;
    wave_copy_row(a.mb + ((int64_t)v * a.K + slot) * a.D_m, a.d_mail + i * a.D_m, a.D_m, lane);
    if (lane == 0)
        a.mb_ts[(int64_t)v * a.K + slot] = a.d_t[i];
}

__global__ __launch_bounds__(256) void k_apan_commit_heads(int64_t n, int K,
                                                           const int32_t *__restrict__ d_node,
                                                           const int32_t *__restrict__ d_rank,
                                                           const int32_t *__restrict__ d_keep,
                                                           int32_t *__restrict__ head,
                                                           int32_t *__restrict__ cnt)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n || d_keep[i] == 0 || d_rank[i] != d_keep[i] - 1)
        return;
    const int v = d_node[i], k = d_keep[i];
    head[v] = (head[v] + k) % K;
    cnt[v] = min(K, cnt[v] + k);
}

// The committed mailboxes oldest first, one wavefront per node; rows past the
// count are zero.
__global__ __launch_bounds__(256) void k_apan_read_mb(int32_t N, int K, int D_m,
                                                      const float *__restrict__ mb,
                                                      const double *__restrict__ mb_ts,
                                                      const int32_t *__restrict__ head,
                                                      const int32_t *__restrict__ cnt,
                                                      float *__restrict__ out,
                                                      double *__restrict__ out_ts)
{
    const int v = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (v >= N)
        return;
    const int c = cnt[v], hd = head[v];
    for (int j = 0; j < K; ++j) {
        float *dst = out + ((int64_t)v * K + j) * D_m;
        if (j < c) {
            const int slot = ((hd - c + j) % K + K) % K;
            wave_copy_row(dst, mb + ((int64_t)v * K + slot) * D_m, D_m, lane);
            if (lane == 0)
                out_ts[(int64_t)v * K + j] = mb_ts[(int64_t)v * K + slot];
        } else {
            for (int k = lane; k < D_m; k += kWave)
                dst[k] = 0.f;
            if (lane == 0)
                out_ts[(int64_t)v * K + j] = 0.0;
        }
    }
}

// Mailboxes given oldest first with their counts into the rings: mail j at
// slot j, head = count mod K; counts are clamped to [0, K].
__global__ __launch_bounds__(256) void k_apan_load_mb(int32_t N, int K, int D_m,
                                                      const float *__restrict__ in,
                                                      const double *__restrict__ in_ts,
                                                      const int32_t *__restrict__ in_cnt,
                                                      float *__restrict__ mb,
                                                      double *__restrict__ mb_ts,
                                                      int32_t *__restrict__ head,
                                                      int32_t *__restrict__ cnt)
{
    const int v = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (v >= N)
        return;
    const int c = min(max(in_cnt[v], 0), K);
    for (int j = 0; j < c; ++j) {
        wave_copy_row(mb + ((int64_t)v * K + j) * D_m, in + ((int64_t)v * K + j) * D_m, D_m,
                      lane);
        if (lane == 0)
            mb_ts[(int64_t)v * K + j] = in_ts[(int64_t)v * K + j];
    }
    if (lane == 0) {
        head[v] = c % K;
        cnt[v] = c;
    }
}

__global__ void k_apan_init(int32_t N, int M, int K, int D_m, float *__restrict__ mem,
                            double *__restrict__ mem_ts, int32_t *__restrict__ ver,
                            float *__restrict__ mb, double *__restrict__ mb_ts,
                            int32_t *__restrict__ head, int32_t *__restrict__ cnt)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t k = t0; k < (int64_t)N * M; k += stride)
        mem[k] = 0.f;
    for (int64_t k = t0; k < (int64_t)N * K * D_m; k += stride)
        mb[k] = 0.f;
    for (int64_t k = t0; k < (int64_t)N * K; k += stride)
        mb_ts[k] = 0.0;
    for (int64_t k = t0; k < N; k += stride) {
        mem_ts[k] = 0.0;
        ver[k] = -1;
        head[k] = 0;
        cnt[k] = 0;
    }
}

}  // namespace

struct tgm_apan {
    int32_t N = 0, M = 0, D_e = 0, D_t = 0, D_m = 0, D_x = 0, nb = 0, K = 0, s = 0;
    int32_t max_batch = 0, max_nodes = 0, propagate = 1;
    // weights (plain, device)
    float *W_ih = nullptr, *W_hh = nullptr, *b_ih = nullptr, *b_hh = nullptr;
    double *omega = nullptr, *beta = nullptr;
    // committed tables
    float *mem = nullptr, *mb = nullptr;
    double *mem_ts = nullptr, *mb_ts = nullptr;
    int32_t *ver = nullptr, *head = nullptr, *cnt = nullptr;
    // fetched rows of the last step and the updater's work space
    float *Wqk = nullptr, *c_u = nullptr;   // the key projection with the query's folded in
    // what they are folded from, freed by the end of creation; cq: W_q phi(0) + b_q
    float *W_q = nullptr, *b_q = nullptr, *W_k = nullptr;
    double *cq = nullptr;
    float *f_mem = nullptr, *f_mb = nullptr, *U = nullptr, *X = nullptr, *Gx = nullptr,
          *Gh = nullptr;
    double *f_mem_ts = nullptr, *f_mb_ts = nullptr, *t_new = nullptr;
    int32_t *f_ver = nullptr, *f_cnt = nullptr;
    // staging
    SortBuffers sort;   // deliveries by node
    // ring of s + 1 write sets: memory rows by node-set position, mail rows
    // by sorted delivery position
    struct Slot {
        int64_t iter = -1;
        int64_t n_del = 0;
        bool staged = false;
    };
    std::vector<Slot> ring;
    int32_t *r_flag = nullptr, *r_node = nullptr;
    float *r_mem = nullptr;
    double *r_ts = nullptr;
    int32_t *d_node = nullptr, *d_rank = nullptr, *d_keep = nullptr;
    float *d_mail = nullptr;
    double *d_t = nullptr;
    int64_t committed_through = -1, staged_through = -1;
    int64_t max_del() const { return 2 * (int64_t)max_batch * (nb + 1); }
};

namespace {

tgm_status_t apan_commit_through(tgm_apan *a, int64_t target, hipStream_t s)
{
    const int slots = a->s + 1;
    for (int64_t j = a->committed_through + 1; j <= target; ++j) {
        tgm_apan::Slot &sl = a->ring[j % slots];
        if (!sl.staged || sl.iter != j)
            return TGM_EORDER;
        const int64_t r = j % slots;
        const int64_t cap = a->max_nodes, md = a->max_del();
        CommitArgs ca{(int)cap, (int)cdiv(cap, 4), a->M, a->D_m, a->K, j, sl.n_del,
                      a->r_flag + r * cap, a->r_node + r * cap, a->d_node + r * md,
                      a->d_rank + r * md, a->d_keep + r * md, a->head, a->r_mem + r * cap * a->M,
                      a->d_mail + r * md * a->D_m, a->r_ts + r * cap, a->d_t + r * md, a->mem,
                      a->mb, a->mem_ts, a->mb_ts, a->ver};
        TGM_LAUNCH(k_apan_commit, dim3((unsigned)(ca.n_mem + cdiv(sl.n_del, 4))), dim3(256), 0, s,
                   ca);
        if (sl.n_del > 0)
            TGM_LAUNCH(k_apan_commit_heads, dim3((unsigned)cdiv(sl.n_del, 256)), dim3(256), 0,
                       s, sl.n_del, a->K, a->d_node + r * md, a->d_rank + r * md,
                       a->d_keep + r * md, a->head, a->cnt);
        sl.staged = false;
        a->committed_through = j;
    }
    return TGM_OK;
}

}  // namespace

// ======================================================================== API

extern "C" tgm_status_t tgm_apan_destroy(tgm_apan_t a)
{
    if (!a)
        return TGM_EINVAL;
    void *bufs[] = {a->W_ih, a->W_hh, a->b_ih, a->b_hh, a->W_q, a->b_q, a->W_k, a->omega,
                    a->beta, a->mem, a->mb, a->mem_ts, a->mb_ts, a->ver, a->head, a->cnt,
                    a->Wqk, a->c_u, a->cq, a->f_mem, a->f_mb, a->U, a->X, a->Gx, a->Gh,
                    a->f_mem_ts, a->f_mb_ts, a->t_new, a->f_ver, a->f_cnt, a->r_flag, a->r_node,
                    a->r_mem, a->r_ts, a->d_node, a->d_rank, a->d_keep, a->d_mail, a->d_t};
    for (void *b : bufs)
        (void)hipFree(b);
    sort_destroy(&a->sort);
    delete a;
    return TGM_OK;
}

extern "C" tgm_status_t tgm_apan_create(const tgm_apan_desc *d, const tgm_weights *w,
                                        void *stream, tgm_apan_t *out)
{
    if (!out)
        return TGM_EINVAL;
    *out = nullptr;
    if (!d || !w || d->N <= 0 || d->M <= 0 || d->M > 128 || d->D_e < 0 || d->D_e > 256 ||
        d->D_t < 0 || d->nb < 1 || d->nb > 64 || d->K_mb < 1 || d->K_mb > kApanMaxK ||
        d->s < 0 || d->max_batch <= 0 || d->max_nodes <= 0)
        return TGM_EINVAL;
    if (!w->W_ih || !w->W_hh || !w->b_ih || !w->b_hh || !w->W_q || !w->b_q || !w->W_k ||
        !w->b_k || (d->D_t > 0 && (!w->omega || !w->beta)))
        return TGM_EINVAL;
    tgm_apan *a = new tgm_apan();
    a->N = d->N;
    a->M = d->M;
    a->D_e = d->D_e;
    a->D_t = d->D_t;
    a->D_m = 2 * d->M + d->D_e;
    a->D_x = a->D_m + d->D_t;
    a->nb = d->nb;
    a->K = d->K_mb;
    a->s = d->s;
    a->max_batch = d->max_batch;
    a->max_nodes = d->max_nodes;
    a->propagate = d->propagate != 0;
    a->ring.resize(d->s + 1);
    const int64_t N = a->N, M = a->M, K = a->K, D_m = a->D_m, D_x = a->D_x, D_t = a->D_t;
    const int64_t C = a->max_nodes, MD = a->max_del(), slots = d->s + 1;
    tgm_status_t st = TGM_OK;
    auto alloc = [&](auto **ptr, int64_t count) {
        if (st == TGM_OK &&
            dev_malloc(ptr, sizeof(**ptr) * (size_t)std::max<int64_t>(count, 1)) != hipSuccess)
            st = TGM_ENOMEM;
    };
    alloc(&a->W_ih, 3 * M * D_x);
    alloc(&a->W_hh, 3 * M * M);
    alloc(&a->b_ih, 3 * M);
    alloc(&a->b_hh, 3 * M);
    alloc(&a->W_q, M * (M + D_t));
    alloc(&a->b_q, M);
    alloc(&a->W_k, M * D_x);
    alloc(&a->omega, D_t);
    alloc(&a->beta, D_t);
    alloc(&a->mem, N * M);
    alloc(&a->mb, N * K * D_m);
    alloc(&a->mem_ts, N);
    alloc(&a->mb_ts, N * K);
    alloc(&a->ver, N);
    alloc(&a->head, N);
    alloc(&a->cnt, N);
    alloc(&a->f_mem, C * M);
    alloc(&a->f_mb, C * K * D_m);
    alloc(&a->Wqk, M * D_x);
    alloc(&a->c_u, D_x);
    alloc(&a->cq, M);
    alloc(&a->U, C * D_x);
    alloc(&a->X, C * D_x);
    alloc(&a->Gx, C * 3 * M);
    alloc(&a->Gh, C * 3 * M);
    alloc(&a->f_mem_ts, C);
    alloc(&a->f_mb_ts, C * K);
    alloc(&a->t_new, C);
    alloc(&a->f_ver, C);
    alloc(&a->f_cnt, C);
    alloc(&a->r_flag, slots * C);
    alloc(&a->r_node, slots * C);
    alloc(&a->r_mem, slots * C * M);
    alloc(&a->r_ts, slots * C);
    alloc(&a->d_node, slots * MD);
    alloc(&a->d_rank, slots * MD);
    alloc(&a->d_keep, slots * MD);
    alloc(&a->d_mail, slots * MD * D_m);
    alloc(&a->d_t, slots * MD);
    if (st == TGM_OK)
        st = sort_create(&a->sort, MD, N, [&](auto **ptr, int64_t n) {
            alloc(ptr, n);
            return st == TGM_OK;
        });
    hipStream_t s = as_stream(stream);
    if (st == TGM_OK) {
        const struct {
            void *dst;
            const void *src;
            size_t bytes;
        } up[] = {{a->W_ih, w->W_ih, 4 * (size_t)(3 * M * D_x)}, {a->W_hh, w->W_hh, 4 * (size_t)(3 * M * M)},
                  {a->b_ih, w->b_ih, 4 * (size_t)(3 * M)}, {a->b_hh, w->b_hh, 4 * (size_t)(3 * M)},
                  {a->W_q, w->W_q, 4 * (size_t)(M * (M + D_t))}, {a->b_q, w->b_q, 4 * (size_t)M},
                  {a->W_k, w->W_k, 4 * (size_t)(M * D_x)}, {a->omega, w->omega, 8 * (size_t)D_t},
                  {a->beta, w->beta, 8 * (size_t)D_t}};
        for (const auto &u : up)
            if (st == TGM_OK && u.bytes > 0)
                st = upload(u.dst, u.src, u.bytes);
    }
    if (st == TGM_OK) {
        hipLaunchKernelGGL(k_apan_init, dim3(1024), dim3(256), 0, s, a->N, a->M, a->K, a->D_m,
                           a->mem, a->mem_ts, a->ver, a->mb, a->mb_ts, a->head, a->cnt);
        hipLaunchKernelGGL(k_apan_clear_flags, dim3((unsigned)cdiv(slots * C, 256)), dim3(256), 0,
                           s, a->r_flag, (int)(slots * C));
        hipLaunchKernelGGL(k_apan_cq, dim3((unsigned)cdiv(M, 4)), dim3(256), 0, s, a->M, a->D_t,
                           a->W_q, a->b_q, a->beta, a->cq);
        hipLaunchKernelGGL(k_apan_fold, dim3((unsigned)cdiv(D_x, 256), (unsigned)M + 1), dim3(256),
                           0, s, a->M, a->D_x, a->D_t, a->W_q, a->cq, a->W_k, a->Wqk, a->c_u);
        if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
            st = TGM_EDEVICE;
    }
    // (b_k, which shifts all of a node's scores alike, is not needed at all)
    (void)hipFree(a->W_q);
    (void)hipFree(a->b_q);
    (void)hipFree(a->W_k);
    (void)hipFree(a->cq);
    a->W_q = a->b_q = a->W_k = nullptr;
    a->cq = nullptr;
    if (st != TGM_OK) {
        tgm_apan_destroy(a);
        return st;
    }
    *out = a;
    return TGM_OK;
}

extern "C" tgm_status_t tgm_apan_step(tgm_apan_t a, tgm_graph_t g, int64_t iter,
                                      const tgm_sample_buffers *sb, int32_t cap, float *mem_new,
                                      double *new_mem_ts, float *h, void *stream)
{
    if (!a || !g || !sb || !mem_new || !h || cap < 0)
        return TGM_EINVAL;
    if (!sb->root || !sb->root_pos || !sb->nbr || !sb->cnt || !sb->nodes || !sb->n_nodes)
        return TGM_EINVAL;
    if (g->N != a->N || g->D_e != a->D_e || (a->D_e > 0 && !g->efeat))
        return TGM_EINVAL;
    if (cap > a->max_nodes)
        return TGM_ESIZE;
    if (iter != a->staged_through + 1)
        return TGM_EORDER;
    const int64_t lo = iter * (int64_t)a->max_batch;
    if (lo >= g->E || iter < 0)
        return TGM_ERANGE;
    const int32_t b = (int32_t)std::min<int64_t>(a->max_batch, g->E - lo);
    const int M = a->M, D_m = a->D_m, D_t = a->D_t, D_x = a->D_x, K = a->K, nb = a->nb;
    const int R = 3 * b;
    hipStream_t s = as_stream(stream);
    // the write sets a fetch at iter sees: <= iter - 1 - s (Eq. 2)
    TGM_TRY_STATUS(apan_commit_through(a, iter - 1 - a->s, s));
    const int slots = a->s + 1;
    tgm_apan::Slot &sl = a->ring[iter % slots];
    if (sl.staged)
        return TGM_EORDER;   // cannot happen: commits run ahead of the ring
    const int64_t r = iter % slots, C = a->max_nodes, MD = a->max_del();
    ApanRows ar{sb->nodes, sb->n_nodes, cap, M, D_m, D_t, K, a->mem, a->mb, a->mem_ts,
                a->mb_ts, a->ver, a->head, a->cnt, a->f_mem, a->f_mb, a->f_mem_ts,
                a->f_mb_ts, a->f_ver, a->f_cnt, a->r_flag + r * C, (int)C, (int)cdiv(cap, 4),
                a->U, a->omega, a->beta, 1.f / sqrtf((float)M), a->X, a->t_new, new_mem_ts};
    TGM_LAUNCH(k_apan_gather, dim3((unsigned)(ar.n_gather + cdiv(C, 256))), dim3(256), 0, s, ar);
    if (cap > 0) {
        auto mul = [&](int n, int k, const float *x, const float *w, int ldw, float *out,
                       const float *bias) {   // rows of the node set only
            GemmProb p;
            p.m = cap;
            p.n = n;
            p.k = k;
            p.A = x;
            p.lda = k;
            p.B = w;
            p.ldb = ldw;
            p.C = out;
            p.ldc = n;
            p.bias = bias;
            p.live = sb->n_nodes;
            return p;
        };
        // the mailbox attention: u per node, then scores and the aggregate
        const GemmProb u = mul(D_x, M, a->f_mem, a->Wqk, D_x, a->U, a->c_u);
        TGM_TRY_STATUS(gemm_launch(false, false, &u, 1, s));
        const dim3 grid((unsigned)cdiv((int64_t)cap * kWave, 256));
        if (K <= 10 && D_m <= 6 * kWave)   // 60 registers of mails, else 128
            TGM_LAUNCH((k_apan_attn<10, 6>), grid, dim3(256), 0, s, ar);
        else
            TGM_LAUNCH((k_apan_attn<kApanMaxK, 8>), grid, dim3(256), 0, s, ar);
        // the GRU on [aggregate || phi(t_newest - mem_ts)]
        const GemmProb g[2] = {mul(3 * M, D_x, a->X, a->W_ih, D_x, a->Gx, a->b_ih),
                               mul(3 * M, M, a->f_mem, a->W_hh, M, a->Gh, a->b_hh)};
        TGM_TRY_STATUS(gemm_launch(false, true, g, 2, s));
        TGM_LAUNCH(k_apan_gru, dim3((unsigned)cdiv((int64_t)cap * M, 256)), dim3(256), 0, s,
                   sb->n_nodes, cap, M, a->f_cnt, a->Gx, a->Gh, a->f_mem, mem_new);
    }
    // the embeddings and the write set of iter: memory rows of the endpoints,
    // mail deliveries
    const int64_t n_del = (int64_t)2 * b * (nb + 1);
    if (b > 0) {
        const SortPlan plan = sort_plan(a->sort, n_del);
        AfterArgs fa{b, nb, a->propagate, a->N, M, (int)sort_tiles(n_del), (int)cdiv(R, 4),
                     sb->root, sb->nbr, sb->cnt, sb->root_pos, sb->nodes, mem_new, a->t_new, h,
                     a->r_flag + r * C, a->r_node + r * C, a->r_mem + r * C * M, a->r_ts + r * C,
                     plan};
        TGM_LAUNCH(k_apan_after, dim3((unsigned)(fa.n_keys + fa.n_embed + cdiv(2 * b, 4))),
                   dim3(256), 0, s, fa);
        TGM_TRY_STATUS(sort_launch(a->sort, plan, s));
        StageArgs2 sa{b, nb, M, a->D_e, D_m, K, a->N, lo, a->sort.out_keys, a->sort.out_vals,
                      sb->root_pos, mem_new, g->efeat, g->t, a->d_node + r * MD,
                      a->d_rank + r * MD, a->d_keep + r * MD, a->d_mail + r * MD * D_m,
                      a->d_t + r * MD};
        TGM_LAUNCH(k_apan_stage_mail, dim3((unsigned)cdiv(n_del * kWave, 256)), dim3(256), 0, s,
                   sa, n_del);
    }
    sl.iter = iter;
    sl.n_del = n_del;
    sl.staged = true;
    a->staged_through = iter;
    return TGM_OK;
}

namespace {

void apan_restart(tgm_apan *a, int64_t iter)
{
    for (tgm_apan::Slot &sl : a->ring)
        sl = tgm_apan::Slot{};
    a->committed_through = iter - 1;
    a->staged_through = iter - 1;
}

}  // namespace

extern "C" tgm_status_t tgm_apan_reset(tgm_apan_t a, void *stream)
{
    if (!a)
        return TGM_EINVAL;
    hipStream_t s = as_stream(stream);
    TGM_LAUNCH(k_apan_init, dim3(1024), dim3(256), 0, s, a->N, a->M, a->K, a->D_m, a->mem,
               a->mem_ts, a->ver, a->mb, a->mb_ts, a->head, a->cnt);
    apan_restart(a, 0);
    return TGM_OK;
}

extern "C" tgm_status_t tgm_apan_load(tgm_apan_t a, int64_t iter, const float *mem,
                                      const double *mem_ts, const int32_t *ver, const float *mb,
                                      const double *mb_ts, const int32_t *mb_cnt, void *stream)
{
    if (!a || iter < 0 || !mem || !mem_ts || !ver || !mb || !mb_ts || !mb_cnt)
        return TGM_EINVAL;
    hipStream_t s = as_stream(stream);
    const size_t N = a->N, M = a->M;
    TGM_HIP(hipMemcpyAsync(a->mem, mem, 4 * N * M, hipMemcpyDeviceToDevice, s));
    TGM_HIP(hipMemcpyAsync(a->mem_ts, mem_ts, 8 * N, hipMemcpyDeviceToDevice, s));
    TGM_HIP(hipMemcpyAsync(a->ver, ver, 4 * N, hipMemcpyDeviceToDevice, s));
    TGM_LAUNCH(k_apan_load_mb, dim3((unsigned)cdiv((int64_t)N * kWave, 256)), dim3(256), 0, s,
               a->N, a->K, a->D_m, mb, mb_ts, mb_cnt, a->mb, a->mb_ts, a->head, a->cnt);
    apan_restart(a, iter);
    return TGM_OK;
}

extern "C" tgm_status_t tgm_apan_flush(tgm_apan_t a, void *stream)
{
    if (!a)
        return TGM_EINVAL;
    return apan_commit_through(a, a->staged_through, as_stream(stream));
}

extern "C" tgm_status_t tgm_apan_read(tgm_apan_t a, float *mem, double *mem_ts, int32_t *ver,
                                      float *mb, double *mb_ts, int32_t *mb_cnt, void *stream)
{
    if (!a || (!mb) != (!mb_ts))
        return TGM_EINVAL;
    hipStream_t s = as_stream(stream);
    const size_t N = a->N, M = a->M;
    if (mem)
        TGM_HIP(hipMemcpyAsync(mem, a->mem, 4 * N * M, hipMemcpyDeviceToDevice, s));
    if (mem_ts)
        TGM_HIP(hipMemcpyAsync(mem_ts, a->mem_ts, 8 * N, hipMemcpyDeviceToDevice, s));
    if (ver)
        TGM_HIP(hipMemcpyAsync(ver, a->ver, 4 * N, hipMemcpyDeviceToDevice, s));
    if (mb_cnt)
        TGM_HIP(hipMemcpyAsync(mb_cnt, a->cnt, 4 * N, hipMemcpyDeviceToDevice, s));
    if (mb)
        TGM_LAUNCH(k_apan_read_mb, dim3((unsigned)cdiv((int64_t)N * kWave, 256)), dim3(256), 0,
                   s, a->N, a->K, a->D_m, a->mb, a->mb_ts, a->head, a->cnt, mb, mb_ts);
    return TGM_OK;
}

extern "C" tgm_status_t tgm_apan_fetched(tgm_apan_t a, float *mem, double *mem_ts, int32_t *ver,
                                         float *mb, double *mb_ts, int32_t *mb_cnt, void *stream)
{
    if (!a)
        return TGM_EINVAL;
    hipStream_t s = as_stream(stream);
    const size_t C = a->max_nodes, M = a->M, K = a->K, D_m = a->D_m;
    if (mem)
        TGM_HIP(hipMemcpyAsync(mem, a->f_mem, 4 * C * M, hipMemcpyDeviceToDevice, s));
    if (mem_ts)
        TGM_HIP(hipMemcpyAsync(mem_ts, a->f_mem_ts, 8 * C, hipMemcpyDeviceToDevice, s));
    if (ver)
        TGM_HIP(hipMemcpyAsync(ver, a->f_ver, 4 * C, hipMemcpyDeviceToDevice, s));
    if (mb)
        TGM_HIP(hipMemcpyAsync(mb, a->f_mb, 4 * C * K * D_m, hipMemcpyDeviceToDevice, s));
    if (mb_ts)
        TGM_HIP(hipMemcpyAsync(mb_ts, a->f_mb_ts, 8 * C * K, hipMemcpyDeviceToDevice, s));
    if (mb_cnt)
        TGM_HIP(hipMemcpyAsync(mb_cnt, a->f_cnt, 4 * C, hipMemcpyDeviceToDevice, s));
    return TGM_OK;
}
