// lif_readout.hip -- the paper's readout and loss (Sec. 3.3, App. C): a
// weighted leaky integrator (LI) per class, with the LIF neuron's V/I
// dynamics and no spikes, fed by the last hidden layer's merged spike queue;
// its logit is the integral of e^{-t/tau_LI} V(t) over [0, tau_max] (Eq.
// weighted_leaky_integrator_full), scaled by a fixed temperature multiplier
// before the softmax cross-entropy.  Also the scatter of queue-time
// gradients back to the spikes that formed the queue (the inverse of the
// layer merge).
//
// The LI state is linear in its inputs and never resets, so the logit is a
// superposition over the queue's events: z_c = sum_e W[src_e, c] G(t_e),
// where G(t0) is the weighted integral of one unit event at t0,
//   G(t0) = kappa e^{-t0/tau_LI} [T_m (1 - e^{-r/T_m}) - T_s (1 - e^{-r/T_s})],
//   r = tau_max - t0, T_x = tau_LI tau_x / (tau_LI + tau_x),
// which is the interval-by-interval closed form of the paper summed over
// intervals.  Every factor is at most 1, so no exponent overflows (the
// product e^{t_i/tau_m} e^{-t_i/T_m} of the printed form is e^{-t_i/tau_LI}).
//
// Passes (no atomics on floating-point values; every sum has a fixed order):
//   k_li_events   per (sample, kLiChunk events): G and dG/dt0 of every event,
//                 the chunk's part of the logits, and H[b][src] += G (64-bit
//                 fixed-point integer atomics, exact and order-free).
//   k_li_ce       per sample: the logits (chunks in order); softmax of beta z,
//                 the sample's loss and dL/dz = beta (p - onehot) / B.
//   k_li_grads    dL/dW[c][k] = sum_b H[b][c] dL/dz[b][k], dL/dt_e =
//                 dG(t_e) sum_k W[src_e][k] dL/dz[b][k], and the batch mean of
//                 the loss, by ranges of workgroups.
#include "lif_common.hpp"
#include "lif_host.hpp"

namespace lif {

constexpr int kLiThreads = 256;
constexpr double kHistScale = 1099511627776.0;     // 2^40: fixed-point step of H

struct LiModel {
    double kappa, inv_li, Tm, Ts, tau_max, beta;
};

static LiModel make_li(const lif_li_params& q)
{
    LiModel m;
    m.kappa = q.tau_syn / (q.tau_mem - q.tau_syn);
    const bool unweighted = isinf(q.tau_li);
    m.inv_li = unweighted ? 0.0 : 1.0 / q.tau_li;
    m.Tm = unweighted ? q.tau_mem : q.tau_li * q.tau_mem / (q.tau_li + q.tau_mem);
    m.Ts = unweighted ? q.tau_syn : q.tau_li * q.tau_syn / (q.tau_li + q.tau_syn);
    m.tau_max = q.tau_max;
    m.beta = q.beta;
    return m;
}

// G(t0) and dG/dt0 of one unit event (zero at or after tau_max).
__device__ __forceinline__ double2 event_kernel(const LiModel& m, double t0)
{
    if (!(t0 < m.tau_max)) return make_double2(0.0, 0.0);
    const double w0 = exp(-t0 * m.inv_li);
    const double r = m.tau_max - t0;
    const double am = exp(-r / m.Tm), as = exp(-r / m.Ts);
    // T (1 - e^{-r/T}) = -T expm1(-r/T), accurate for small r
    const double G = m.kappa * w0 * (-m.Tm * expm1(-r / m.Tm) + m.Ts * expm1(-r / m.Ts));
    const double dG = -G * m.inv_li + m.kappa * w0 * (as - am);
    return make_double2(G, dG);
}

// One workgroup per (sample, chunk of kLiChunk events), a quarter of it per
// wave.  The logits: a wave holds its classes in the low lanes of one or more
// lane groups of `group` lanes (the power of two holding ncls), each group taking
// every (64 / group)-th event, kU events in flight; groups, then waves are added
// in order.  A workgroup per sample left half the chip idle and a chain of
// loads per wave (494 us at 512 -> 20, B = 128, ~7 k events, and 44 us for G, dG
// and H in passes of their own; 45 us for all of it here, bound by the latency
// of the row gathers: 64 us with chunks of 512 events, 52 us with 16 in flight).
constexpr int kLiChunk = 256;

__global__ __launch_bounds__(kLiThreads) void k_li_events(const float* __restrict__ ev_t,
                                                          const int32_t* __restrict__ ev_src,
                                                          const int32_t* __restrict__ ev_n, int E_max, int chunks,
                                                          LiModel m, const float* __restrict__ WT, int C_in, int ncls,
                                                          int group, double2* __restrict__ gk,
                                                          unsigned long long* __restrict__ H,
                                                          double* __restrict__ zpart)
{
    constexpr int nw = kLiThreads / kWave, kPerWave = kLiChunk / nw;
    __shared__ double s_g[kLiChunk];
    __shared__ int s_row[kLiChunk];
    __shared__ double part[nw][kWave];
    const int b = blockIdx.y, ch = blockIdx.x;
    const int wave = (int)threadIdx.x / kWave, lane = (int)threadIdx.x % kWave;
    const int nb = clamp_count(ev_n[b], E_max);
    const int k0 = ch * kLiChunk, cnt = min(kLiChunk, nb - k0);
    if (cnt <= 0) return;
    // the wave's events: kernel values, source rows, histogram
    const int w0 = wave * kPerWave;
    for (int i = w0 + lane; i < w0 + kPerWave; i += kWave) {
        double2 g = make_double2(0.0, 0.0);
        int src = 0;
        if (i < cnt) {
            const size_t at = (size_t)b * E_max + k0 + i;
            g = event_kernel(m, (double)ev_t[at]);
            src = clamp_src(ev_src[at], C_in);
            gk[at] = g;
            if (H && g.x != 0.0)
                atomicAdd(&H[(size_t)b * C_in + src], (unsigned long long)llrint(g.x * kHistScale));
        }
        s_g[i] = g.x;
        s_row[i] = src * ncls;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int c = lane & (group - 1), g0 = lane / group, ng = kWave / group;
    const bool live = c < ncls;
    double acc = 0.0;
    constexpr int kU = 8;
    const int wend = min(w0 + kPerWave, cnt);
    for (int e = w0 + g0; e < wend; e += kU * ng) {
        float w[kU];
        double G[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int x = e + u * ng, xx = x < wend ? x : e;
            w[u] = live ? WT[(size_t)s_row[xx] + c] : 0.0f;
            G[u] = x < wend ? s_g[xx] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) acc = fma(G[u], (double)w[u], acc);
    }
    part[wave][lane] = acc;
    __syncthreads();
    if ((int)threadIdx.x < ncls) {
        double z = 0.0;
        for (int q = 0; q < nw; ++q)
            for (int u = 0; u < ng; ++u) z += part[q][u * group + (int)threadIdx.x];
        zpart[((size_t)b * chunks + ch) * ncls + threadIdx.x] = z;
    }
}

// One wave per sample (lanes are classes, ncls <= 64): the logits; with labels
// the sample's loss and dL/dz.
__global__ __launch_bounds__(kWave) void k_li_ce(const double* __restrict__ zpart, const int32_t* __restrict__ ev_n,
                                                 int E_max, int chunks, int B, int ncls,
                                                 const int32_t* __restrict__ labels, double beta,
                                                 float* __restrict__ logits, double* __restrict__ dz,
                                                 double* __restrict__ loss_b)
{
    const int b = blockIdx.x, c = threadIdx.x;
    const bool live = c < ncls;
    const int used = (clamp_count(ev_n[b], E_max) + kLiChunk - 1) / kLiChunk;
    double z = 0.0;
    const double* zp = zpart + (size_t)b * chunks * ncls + (live ? c : 0);
    for (int q0 = 0; q0 < used; q0 += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = zp[(size_t)min(q0 + u, used - 1) * ncls];
#pragma unroll
        for (int u = 0; u < 8; ++u) z += q0 + u < used ? v[u] : 0.0;
    }
    if (live && logits) logits[(size_t)b * ncls + c] = (float)z;
    if (!labels) return;
    const double y = live ? beta * z : -INFINITY;
    double mx = y;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, kWave));
    const double ex = live ? exp(y - mx) : 0.0;
    double sum = ex;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
    const int lab = min(max(labels[b], 0), ncls - 1);
    const double p = ex / sum;
    if (live) dz[(size_t)b * ncls + c] = beta * (p - (c == lab ? 1.0 : 0.0)) / (double)B;
    const double y_lab = __shfl(y, lab, kWave);
    if (c == 0) loss_b[b] = log(sum) - (y_lab - mx);
}

__global__ void k_li_loss(const double* __restrict__ loss_b, int B, float* __restrict__ loss)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double s = 0.0;
    for (int b = 0; b < B; ++b) s += loss_b[b];
    loss[0] = (float)(s / (double)B);
}

__global__ __launch_bounds__(kLiThreads) void k_fill_u64(unsigned long long* __restrict__ p, size_t n)
{
    const size_t i = (size_t)blockIdx.x * kLiThreads + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// dL/dW: kGwLanes threads per element, each summing every kGwLanes-th sample in
// order, their sums added in order (fixed whatever the launch).
constexpr int kGwLanes = 8;

__device__ __forceinline__ void li_grad_w(int block, const unsigned long long* __restrict__ H, int B, int C_in,
                                          int ncls, const double* __restrict__ dz, float* __restrict__ grad_WT)
{
    const size_t t = (size_t)block * kLiThreads + threadIdx.x;
    const size_t i = t / kGwLanes;
    const int part = (int)(t % kGwLanes);
    const bool live = i < (size_t)C_in * ncls;
    const int c = live ? (int)(i / ncls) : 0, k = live ? (int)(i % ncls) : 0;
    double s = 0.0;
    for (int b0 = part; b0 < B; b0 += 4 * kGwLanes) {
        long long h[4];
        double d[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = min(b0 + u * kGwLanes, B - 1);
            h[u] = (long long)H[(size_t)b * C_in + c];
            d[u] = dz[(size_t)b * ncls + k];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (b0 + u * kGwLanes < B && h[u]) s = fma((double)h[u] / kHistScale, d[u], s);
    }
#pragma unroll
    for (int off = 1; off < kGwLanes; off <<= 1) s += __shfl_xor(s, off, kWave);
    if (live && part == 0) grad_WT[i] = (float)s;
}

__device__ __forceinline__ void li_grad_t(int block, int bpe, const int32_t* __restrict__ ev_src,
                                          const int32_t* __restrict__ ev_n, int E_max, const float* __restrict__ WT,
                                          int C_in, int ncls, const double2* __restrict__ gk,
                                          const double* __restrict__ dz, float* __restrict__ grad_t)
{
    __shared__ double s_dz[kWave];
    const int b = block / bpe;
    if (threadIdx.x < kWave) s_dz[threadIdx.x] = (int)threadIdx.x < ncls ? dz[(size_t)b * ncls + threadIdx.x] : 0.0;
    __syncthreads();
    const int e = (block % bpe) * kLiThreads + (int)threadIdx.x;
    if (e >= E_max) return;
    const size_t at = (size_t)b * E_max + e;
    if (e >= clamp_count(ev_n[b], E_max)) {
        grad_t[at] = 0.0f;
        return;
    }
    const double dG = gk[at].y;
    double s = 0.0;
    if (dG != 0.0) {
        const float* row = WT + (size_t)clamp_src(ev_src[at], C_in) * ncls;
#pragma unroll 4
        for (int k = 0; k < ncls; ++k) s = fma((double)row[k], s_dz[k], s);
    }
    grad_t[at] = (float)(dG * s);
}

// The batch mean of the loss, one wave: lane l the samples l, l + 64, ...
__device__ __forceinline__ void li_loss(const double* __restrict__ loss_b, int B, float* __restrict__ loss)
{
    if (threadIdx.x >= kWave) return;
    double s = 0.0;
    for (int b = (int)threadIdx.x; b < B; b += kWave) s += loss_b[b];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, kWave);
    if (threadIdx.x == 0) loss[0] = (float)(s / (double)B);
}

// What the labels ask for, by ranges of workgroups: wblocks of dL/dW, tblocks
// (bpe per sample) of dL/dt, then one of the loss.
__global__ __launch_bounds__(kLiThreads) void k_li_grads(int wblocks, int tblocks, int bpe,
                                                         const int32_t* __restrict__ ev_src,
                                                         const int32_t* __restrict__ ev_n, int B, int E_max,
                                                         const float* __restrict__ WT, int C_in, int ncls,
                                                         const double2* __restrict__ gk,
                                                         const unsigned long long* __restrict__ H,
                                                         const double* __restrict__ dz,
                                                         const double* __restrict__ loss_b,
                                                         float* __restrict__ grad_WT, float* __restrict__ grad_t,
                                                         float* __restrict__ loss)
{
    const int k = (int)blockIdx.x;
    if (k < wblocks) li_grad_w(k, H, B, C_in, ncls, dz, grad_WT);
    else if (k < wblocks + tblocks) li_grad_t(k - wblocks, bpe, ev_src, ev_n, E_max, WT, C_in, ncls, gk, dz, grad_t);
    else if (loss) li_loss(loss_b, B, loss);
}

// grad_out_t[b][perm[b][j]] = grad_ev_t2[b][j] for the queue's events, 0 for
// every other spike slot.
__global__ __launch_bounds__(kLiThreads) void k_fill_f32(float* __restrict__ p, size_t n)
{
    const size_t i = (size_t)blockIdx.x * kLiThreads + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

__global__ __launch_bounds__(kLiThreads) void k_merge_grad(const float* __restrict__ g2,
                                                           const int32_t* __restrict__ perm,
                                                           const int32_t* __restrict__ ev_n2, int E2_max,
                                                           size_t per_sample, float* __restrict__ grad_out_t)
{
    const int b = blockIdx.y;
    const int j = blockIdx.x * kLiThreads + threadIdx.x;
    if (j >= clamp_count(ev_n2[b], E2_max)) return;
    const int p = perm[(size_t)b * E2_max + j];
    if (p >= 0 && (size_t)p < per_sample) grad_out_t[(size_t)b * per_sample + p] = g2[(size_t)b * E2_max + j];
}

struct LiLayout {
    size_t gk, zpart, dz, loss_b, H, total;
};

static int li_chunks(int E_max) { return E_max > 0 ? (E_max + kLiChunk - 1) / kLiChunk : 1; }

static LiLayout li_layout(int B, int E_max, int C_in, int ncls)
{
    LiLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    L.gk = take((size_t)B * E_max * sizeof(double2));
    L.zpart = take((size_t)B * li_chunks(E_max) * ncls * sizeof(double));
    L.dz = take((size_t)B * ncls * sizeof(double));
    L.loss_b = take((size_t)B * sizeof(double));
    L.H = take((size_t)B * C_in * sizeof(unsigned long long));
    L.total = off + 256;
    return L;
}

static int check_li(const lif_li_params* q)
{
    if (!q) return LIF_ERR_ARG;
    if (!(q->tau_syn > 0.0) || !(q->tau_mem > q->tau_syn) || !isfinite(q->tau_mem)) return LIF_ERR_TAU;
    if (!(q->tau_li > 0.0)) return LIF_ERR_TAU;                     // +inf allowed: unweighted
    if (!(q->tau_max > 0.0) || !isfinite(q->tau_max) || !isfinite(q->beta)) return LIF_ERR_ARG;
    return LIF_OK;
}

}  // namespace lif

extern "C" size_t lif_li_readout_workspace_size(int B, int E_max, int C_in, int N_cls)
{
    if (B < 0 || E_max < 0 || C_in < 1 || N_cls < 1) return 0;
    return lif::li_layout(B, E_max, C_in, N_cls).total;
}

extern "C" int lif_li_readout(const float* ev_t, const int32_t* ev_src, const int32_t* ev_n, int B, int E_max,
                              const float* WT, int C_in, int N_cls, const lif_li_params* q,
                              const int32_t* labels, float* logits, float* loss, float* grad_WT,
                              float* grad_ev_t, void* ws, size_t ws_bytes, lif_stream_t stream_)
{
    using namespace lif;
    int rc = check_li(q);
    if (rc) return rc;
    if (B < 0 || E_max < 0 || C_in < 1 || N_cls < 1) return LIF_ERR_ARG;
    if (N_cls > LIF_LI_MAX_CLASSES) return LIF_ERR_SIZE;
    if ((size_t)C_in * (size_t)N_cls >= ((size_t)1 << 31) || (size_t)B * (size_t)E_max >= ((size_t)1 << 40))
        return LIF_ERR_SIZE;
    if (!WT || !ws || (B > 0 && !ev_n) || ((size_t)B * E_max > 0 && (!ev_t || !ev_src))) return LIF_ERR_ARG;
    if (!labels && (loss || grad_WT || grad_ev_t)) return LIF_ERR_ARG;
    const LiLayout L = li_layout(B, E_max, C_in, N_cls);
    if (ws_bytes < L.total) return LIF_ERR_WORKSPACE;
    hipStream_t stream = (hipStream_t)stream_;
    char* base = (char*)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    double2* gk = (double2*)(base + L.gk);
    double* zpart = (double*)(base + L.zpart);
    double* dz = (double*)(base + L.dz);
    double* loss_b = (double*)(base + L.loss_b);
    unsigned long long* H = (unsigned long long*)(base + L.H);
    const LiModel m = make_li(*q);
    if (B == 0) {
        if (loss) TIMED_LAUNCH("li_loss", k_li_loss, dim3(1), dim3(1), 0, stream, loss_b, 0, loss);
        if (grad_WT) {
            const size_t n = (size_t)C_in * N_cls;
            TIMED_LAUNCH("li_fill", k_fill_f32, dim3((unsigned)((n + kLiThreads - 1) / kLiThreads)),
                         dim3(kLiThreads), 0, stream, grad_WT, n);
        }
        return check_launch();
    }
    const int chunks = li_chunks(E_max);
    const int bpe = (E_max + kLiThreads - 1) / kLiThreads;
    const size_t nw = (size_t)C_in * N_cls;
    const size_t wblocks = grad_WT ? (nw * kGwLanes + kLiThreads - 1) / kLiThreads : 0;
    const size_t tblocks = grad_ev_t ? (size_t)B * bpe : 0;
    if (wblocks + tblocks >= 0x7fffffff) return LIF_ERR_SIZE;
    if (grad_WT) {
        const size_t nh = (size_t)B * C_in;
        TIMED_LAUNCH("li_fill", k_fill_u64, dim3((unsigned)((nh + kLiThreads - 1) / kLiThreads)), dim3(kLiThreads),
                     0, stream, H, nh);
    }
    int group = 1;
    while (group < N_cls) group <<= 1;
    if (E_max > 0)
        TIMED_LAUNCH("li_events", k_li_events, dim3((unsigned)chunks, (unsigned)B), dim3(kLiThreads), 0, stream, ev_t,
                     ev_src, ev_n, E_max, chunks, m, WT, C_in, N_cls, group, gk, grad_WT ? H : nullptr, zpart);
    TIMED_LAUNCH("li_ce", k_li_ce, dim3((unsigned)B), dim3(kWave), 0, stream, zpart, ev_n, E_max, chunks, B, N_cls,
                 labels, m.beta, logits, dz, loss_b);
    if (loss || grad_WT || tblocks)
        TIMED_LAUNCH("li_grads", k_li_grads, dim3((unsigned)(wblocks + tblocks + 1)), dim3(kLiThreads), 0, stream,
                     (int)wblocks, (int)tblocks, bpe, ev_src, ev_n, B, E_max, WT, C_in, N_cls, gk, H, dz, loss_b,
                     grad_WT, grad_ev_t, loss);
    return check_launch();
}

extern "C" int lif_merge_grad(const float* grad_ev_t2, const int32_t* perm, const int32_t* ev_n2, int B, int E2_max,
                              int N, int s_max, float* grad_out_t, lif_stream_t stream_)
{
    using namespace lif;
    if (B < 0 || E2_max < 0 || N < 1 || s_max < 1) return LIF_ERR_ARG;
    if (!grad_out_t || (B > 0 && !ev_n2) || ((size_t)B * E2_max > 0 && (!grad_ev_t2 || !perm))) return LIF_ERR_ARG;
    hipStream_t stream = (hipStream_t)stream_;
    const size_t per = (size_t)N * (size_t)s_max, n = (size_t)B * per;
    if (n)
        TIMED_LAUNCH("merge_grad_fill", k_fill_f32, dim3((unsigned)((n + kLiThreads - 1) / kLiThreads)),
                     dim3(kLiThreads), 0, stream, grad_out_t, n);
    if (B > 0 && E2_max > 0)
        TIMED_LAUNCH("merge_grad", k_merge_grad, dim3((unsigned)((E2_max + kLiThreads - 1) / kLiThreads), (unsigned)B),
                     dim3(kLiThreads), 0, stream, grad_ev_t2, perm, ev_n2, E2_max, per, grad_out_t);
    return check_launch();
}
