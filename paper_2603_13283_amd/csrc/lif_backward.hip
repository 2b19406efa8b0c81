// lif_backward.hip -- exact gradients of the LIF layer's spike times
// (Appendix D.3, Eq. ift_vjp, chained through the hard resets).
//
// Writing each reset as the subtraction of (V_th - V_reset) e^{-(t - t_s)/tm}
// (exact, because V is continuous at input events and equals V_th at t_s),
// spike s of a neuron is the root of
//   F_s = sum_{k: t_k < t_s} w_k K(t_s - t_k)
//         - (V_th - V_reset) sum_{s' < s} e^{-(t_s - t_s')/tm} - V_th,
// K(u) = kappa (e^{-u/tm} - e^{-u/ts}).  The implicit function theorem gives
// dt_s = -(dF_s/dt_s)^{-1} dF_s with dF_s/dt_s = dV/dt at the spike
// = (I(t_s) - V_th)/tm (Eq. mem_dyn), floored by the solver regularisation.
// With mu_s the adjoint of constraint F_s,
//   lambda_s = g_s - ((V_th - V_reset)/tm) sum_{s'' > s} mu_s'' e^{-(t_s'' - t_s)/tm}
//   mu_s     = -lambda_s / max(dV/dt(t_s), reg)                  (k_spike_adjoint)
// and every input event k collects, with P^m_k = sum over the spikes s
// that come after event k of mu_s e^{-(t_s - t_k)/tm} and P^s_k the same
// with ts,
//   dL/dw_{i, src_k} += kappa (P^m_k - P^s_k)
//   dL/dt_k          += w_{i, src_k} kappa (P^m_k / tm - P^s_k / ts).
// Spike s comes after event k iff k < out_k[s], the forward pass's own count
// of the events consumed before the spike (not a comparison of float32
// times, which can round a spike onto the time of the event before it; the
// offset t_s - t_k is then taken as 0).
// With the suffix sums Q_s = sum_{s' >= s} mu_s' e^{-(t_s' - t_s)/t.} over a
// neuron's spikes, P_k = Q_s e^{-(t_s - t_k)/t.} for the first spike s after
// event k: between two spikes of the neuron P is a per-neuron constant times a
// per-event exponential that all neurons share.  With times referred to a
// multiple ref of kRefTs tau_s (so that no exponential leaves the float64 range)
//   P_k = R_s H_k,  R_s = Q_s e^{-(t_s - ref)/t.},  H_k = e^{(t_k - ref)/t.},
// R tabulated per spike and H per event before the walk: passing a spike is a
// switch to the next R, and the walk evaluates no exponential.
//
// dL/dW sums one term per (event, neuron) into element (source, neuron).  As
// global atomics these adds bound the walk (184 G adds/s on this card wherever
// the rows lie, against 4100 G adds/s into LDS), so a workgroup keeps
// the dL/dW block of 64 neurons and a range of at most kAdjRows channels in
// LDS and walks, for those neurons, only the events of that range: the events
// of each (sample, channel range) are listed in time order first
// (k_bwd_setup counts, k_bwd_plan scans, k_bwd_scatter places them), every
// (event, neuron) pair is still walked once.  One range's list holds all events.
// Where few neurons have adjoints (a layer that fires little, or an upstream
// gradient on few spikes), or the call is small, only those neurons are walked
// (listed per sample, 64 of them to a wave) and their terms go to global atomics;
// which of the two is decided on the device (k_bwd_plan).
//
// Both gradients are bitwise reproducible.  dL/dW sums contributions from
// every sample that sees the same (channel, neuron): they are
// added as 64-bit fixed-point integers (integer addition is exact and order
// free) with a power-of-two scale chosen per call so that no sum can
// overflow (k_bwd_plan); dL/dt of an event sums over the neuron tiles,
// whose partial sums are stored per tile and added in tile order (of the few
// neurons: per chunk of a sample's list, in chunk order).
#include <type_traits>

#include "lif_common.hpp"
#include "lif_host.hpp"
#include "lif_scan.hpp"
#include "lif_walk.hpp"

namespace lif {

constexpr int kAdjThreads = 768;                 // threads of an adjoint workgroup
constexpr int kAdjWaves = kAdjThreads / kWave;
constexpr int kAdjRows = 318;                    // channels of a dL/dW block: 159 KB of LDS
constexpr int kAdjMaxRanges = 1024;              // channel ranges that the event lists take
constexpr int kListChunk = 1024;                 // events one wave counts or places
constexpr int kCus = 256;
constexpr int kPlanThreads = 1024;
constexpr long long kFewUnits = 4096;            // units of a kWayFew walk (3072 waves are resident)
// (event, neuron) pairs of a call up to which it takes kWayFew without the lists and
// blocks of the other: five short kernels against six.  700 -> 256, B = 8, 2000
// events (4.1 M pairs, half of the neurons firing): 46 against 81 us; 700 -> 512,
// B = 16 (16 M): 133 against 94 us.
constexpr double kFewPairs = 8388608.0;

// How a call is split; a function of the sizes alone.
struct BwdPlan {
    int tiles;        // 64-neuron tiles
    int nr, rows;     // channel ranges of `rows` channels
    bool lds;         // dL/dW blocks in LDS (else global atomics)
    int nch;          // list chunks per sample
    int Q;            // parts of a (sample, range) list
    int S;            // workgroups per (tile, range), which add to the same block
};

static BwdPlan bwd_plan(int B, int E_max, int C_in, int N)
{
    BwdPlan P{};
    P.tiles = (N + kWave - 1) / kWave;
    P.nr = (C_in + kAdjRows - 1) / kAdjRows;
    // past kAdjMaxRanges ranges (325 632 channels) a range's list is a
    // small part of the stream and the wave counters of the list build no
    // longer fit: one range, dL/dW by global atomics
    // (and calls of few pairs: kFewPairs)
    P.lds = P.nr <= kAdjMaxRanges && (double)B * (double)E_max * (double)N > kFewPairs;
    if (!P.lds) P.nr = 1;
    P.rows = (C_in + P.nr - 1) / P.nr;
    // (at least one chunk: the plan pass then writes every list's start, also of
    // queues without room for an event, whose lists are empty)
    P.nch = E_max > 0 ? (E_max + kListChunk - 1) / kListChunk : 1;
    // parts: enough (sample, part) units for four per wave of a full chip,
    // none longer than 1024 events and none much shorter than 128 (a unit
    // starts with a search in every neuron's spikes)
    const long long len = E_max / P.nr > 0 ? E_max / P.nr : 1;
    const long long groups = (long long)P.tiles * P.nr;
    const long long have = groups * (B > 0 ? B : 1);
    long long Q = (4ll * kCus * kAdjWaves + have - 1) / have;
    // three units for each wave of a workgroup
    const long long three = (3ll * kAdjWaves + (B > 0 ? B : 1) - 1) / (B > 0 ? B : 1);
    Q = Q > three ? Q : three;
    Q = Q > (len + 1023) / 1024 ? Q : (len + 1023) / 1024;
    Q = Q < (len + 127) / 128 ? Q : (len + 127) / 128;
    P.Q = (int)(Q < 1 ? 1 : Q);
    P.S = 1;
    if (!P.lds) return P;
    // workgroups per block: the split that leaves the fewest compute units
    // idle in the last round (one workgroup per compute unit at a time),
    // a little against splitting, since split blocks are added by atomics
    const long long units = (long long)(B > 0 ? B : 1) * P.Q;
    const long long most = (units + kAdjWaves - 1) / kAdjWaves;
    double best = 0.0;
    for (int S = 1; S <= 64 && S <= most; ++S) {
        const long long rounds = (groups * S + kCus - 1) / kCus;
        const double cost = (double)rounds * (1.0 / S + 0.01);
        if (S == 1 || cost < best) {
            best = cost;
            P.S = S;
        }
    }
    return P;
}

// Reference of a time: the multiple of len = kRefTs tau_s at or before it, as an
// index.  (Past 2e9 of them float32 times that differ are thousands of tau_s
// apart; the index saturates there and the offset is bounded.)
constexpr double kRefTs = 100.0;

__device__ __forceinline__ int ref_index(double t, double inv_len) { return (int)fmin(fmax(t * inv_len, 0.0), 2.0e9); }

__device__ __forceinline__ double ref_offset(double t, int idx, double len)
{
    return fmin(fma(-(double)idx, len, t), 4.0 * len);
}

// f^d (d >= 0) or g^-d, g = 1 / f.
__device__ __forceinline__ double ref_pow(double f, double g, int d)
{
    double x = d < 0 ? g : f, r = 1.0;
    for (unsigned e = (unsigned)(d < 0 ? -d : d); e; e >>= 1) {
        if (e & 1u) r *= x;
        x *= x;
    }
    return r;
}

// An event of a list: its time, source, place in the sample, reference, and
// H = (e^{(t - ref)/tm}, e^{(t - ref)/ts}).
struct alignas(32) ListEvent {
    double Hm, Hs;
    float t;
    int src, k, ref;
};

__device__ __forceinline__ ListEvent list_event(double len, double inv_len, double inv_tm, double inv_ts, float t,
                                                int src, int k)
{
    ListEvent e;
    e.t = t;
    e.src = src;
    e.k = k;
    e.ref = ref_index((double)t, inv_len);
    const double dr = ref_offset((double)t, e.ref, len);
    e.Hm = exp(dr * inv_tm);
    e.Hs = exp(dr * inv_ts);
    return e;
}

__device__ __forceinline__ ListEvent list_event(const Model& m, float t, int src, int k)
{
    const double len = kRefTs * m.ts;
    return list_event(len, 1.0 / len, m.inv_tm, m.inv_ts, t, src, k);
}

// What a setup workgroup found: the largest finite sum_s |mu_s| of its neurons, and
// whether one was not finite.
struct BwdPart {
    double mx;
    long long spikes;     // of the neurons with adjoints
    int bad, live;        // live: neurons with adjoints
};

// What a call turned out to be: the fixed-point scale of dL/dW (wide: its terms
// take the full conversion, fx_term) and the way it is walked (k_bwd_plan).
enum BwdWay { kWayBlocks = 0, kWayFew = 1, kWayNone = 2 };
struct BwdCall {
    double scale;
    int wide, way;
};

struct BwdLayout {
    BwdPlan P;
    size_t q, ns, part, call, live, nlive, pairs, cnt, start, list, gw, gt, total;
};

constexpr int kSetupBlocks = 2048;

static BwdLayout bwd_layout(int B, int E_max, int C_in, int N, int s_max)
{
    BwdLayout L{};
    L.P = bwd_plan(B, E_max, C_in, N);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    L.q = take((size_t)B * N * s_max * sizeof(double2));
    L.ns = take((size_t)B * N * sizeof(int32_t));
    L.part = take(kSetupBlocks * sizeof(BwdPart));
    L.call = take(sizeof(BwdCall));
    L.live = take((size_t)B * N * sizeof(int32_t));
    L.nlive = take((size_t)B * sizeof(int32_t));
    L.pairs = take(((size_t)B * L.P.tiles + 1) * sizeof(int32_t));      // the first word counts them
    const bool lists = L.P.nr > 1;
    L.cnt = take(lists ? (size_t)B * L.P.nr * L.P.nch * sizeof(int32_t) : 0);
    L.start = take(lists ? (size_t)B * (L.P.nr + 1) * sizeof(int32_t) : 0);
    L.list = take(L.P.lds ? (size_t)B * E_max * sizeof(ListEvent) : 0);
    L.gw = take((size_t)C_in * N * sizeof(long long));
    L.gt = take((size_t)L.P.tiles * B * E_max * sizeof(double));
    L.total = off + 256;
    return L;
}

// Suffix sums of one neuron's spike adjoints, last spike first (lambda_s and
// mu_s as in spike_adjoints): ro[s] = (R^m_s, R^s_s), the sums over s' >= s of
// mu_s' e^{-(t_s' - ref)/tm} and with ts, ref the spike's own reference.  Spikes are read kSufBatch at a time
// (the recurrence waits for loads once per batch).  Returns sum_s |mu_s|; early is
// set when a (handed-over) spike time lies before the event before it, et[k - 1].
constexpr int kSufBatch = 4;

__device__ __forceinline__ double spike_suffix_sums(const Model& m, int ns, const float* __restrict__ ts,
                                                    const float* __restrict__ is, const float* __restrict__ g,
                                                    double2* __restrict__ ro, const int32_t* __restrict__ ks,
                                                    const float* __restrict__ et, int nb, bool& early)
{
    const double len = kRefTs * m.ts;
    const double jump = (m.th - m.vr) * m.inv_tm;
    double Qm = 0.0, Qs = 0.0, tn = 0.0, asum = 0.0;
    for (int s1 = ns - 1; s1 >= 0; s1 -= kSufBatch) {
        float tb[kSufBatch], ib[kSufBatch], gb[kSufBatch], eb[kSufBatch];
        int kb[kSufBatch];
#pragma unroll
        for (int u = 0; u < kSufBatch; ++u) {
            const int s = max(s1 - u, 0);
            kb[u] = ks[s];
            tb[u] = ts[s];
            ib[u] = is[s];
            gb[u] = g[s];
        }
#pragma unroll
        for (int u = 0; u < kSufBatch; ++u) eb[u] = nb > 0 ? et[min(max(kb[u], 1), nb) - 1] : 0.0f;
#pragma unroll
        for (int u = 0; u < kSufBatch; ++u) {
            const int s = s1 - u;
            if (s < 0) break;
            if (s + 1 < ns) {
                const double dt = tn - (double)tb[u];
                Qm *= exp(-dt * m.inv_tm);
                Qs *= exp(-dt * m.inv_ts);
            }
            const double lam = (double)gb[u] - jump * Qm;
            const double vp = fmax(((double)ib[u] - m.th) * m.inv_tm, m.reg);
            const double mu = vp > 0.0 ? -lam / vp : 0.0;
            Qm += mu;
            Qs += mu;
            tn = (double)tb[u];
            asum += fabs(mu);
            const double dr = ref_offset(tn, ref_index(tn, 1.0 / len), len);
            ro[s] = make_double2(Qm * exp(-dr * m.inv_tm), Qs * exp(-dr * m.inv_ts));
            early = early || (kb[u] > 0 && tb[u] < eb[u]);
        }
    }
    return asum;
}

// Backward setup in one pass (grid-stride over every thread): the
// fixed-point accumulators of dL/dW (where blocks are split) set to zero;
// the suffix sums of every (sample, neuron)'s spike adjoints with its spike
// count (0 when all its adjoints are exactly 0: such a neuron adds exactly 0
// everywhere and is not walked; a NaN sum keeps it; the complement of the count
// when a spike time of its lies before an event that the spike follows); per workgroup its BwdPart; and
// with one channel range the list of every sample's events, else the events of each (sample, chunk) counted per
// channel range, cnt[b][r][chunk], one wave per chunk.
constexpr int kSetupThreads = 256;

__global__ __launch_bounds__(kSetupThreads) void k_bwd_setup(
    const float* __restrict__ ev_t, const int32_t* __restrict__ ev_src, const int32_t* __restrict__ ev_n, int B,
    int E_max, int C_in, int N, Model m, long long* __restrict__ gw, size_t nW, const float* __restrict__ out_t,
    const int32_t* __restrict__ out_n,
    const float* __restrict__ out_i, const int32_t* __restrict__ out_k, const float* __restrict__ grad_out_t,
    double2* __restrict__ rtab, int32_t* __restrict__ ns_eff, BwdPart* __restrict__ part, int32_t* __restrict__ pairs,
    int nr, int rows, int nch,
    int32_t* __restrict__ cnt, ListEvent* __restrict__ list)
{
    __shared__ BwdPart s_p[kSetupThreads / kWave];
    __shared__ int32_t s_cnt[kSetupThreads / kWave][kAdjMaxRanges];
    const size_t gtid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t gs = (size_t)gridDim.x * blockDim.x;
    const int lane = (int)threadIdx.x % kWave, wv = (int)threadIdx.x / kWave;
    if (gw)
        for (size_t i = gtid; i < nW; i += gs) gw[i] = 0;
    const size_t nn = (size_t)B * (size_t)N;
    if (gtid == 0) pairs[0] = 0;
    BwdPart pt{0.0, 0, 0, 0};
    for (size_t idx = gtid; idx < nn; idx += gs) {
        const int ns = max(min(out_n[idx], m.s_max), 0);
        const size_t o = idx * (size_t)m.s_max;
        const int b = (int)(idx / (size_t)N);
        bool early = false;
        const double ms = spike_suffix_sums(m, ns, out_t + o, out_i + o, grad_out_t + o, rtab + o, out_k + o,
                                            ev_t + (size_t)b * E_max, clamp_count(ev_n[b], E_max), early);
        ns_eff[idx] = ms != 0.0 ? (early ? ~ns : ns) : 0;
        if (isfinite(ms)) pt.mx = fmax(pt.mx, ms);
        else pt.bad = 1;
        if (ms != 0.0) {
            ++pt.live;
            pt.spikes += ns;
        }
    }
    auto join = [](BwdPart& x, const BwdPart& y) {
        x.mx = fmax(x.mx, y.mx);
        x.spikes += y.spikes;
        x.bad |= y.bad;
        x.live += y.live;
    };
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1)
        join(pt, BwdPart{__shfl_xor(pt.mx, off, kWave), __shfl_xor(pt.spikes, off, kWave),
                         __shfl_xor(pt.bad, off, kWave), __shfl_xor(pt.live, off, kWave)});
    if (lane == 0) s_p[wv] = pt;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < kSetupThreads / kWave; ++q) join(pt, s_p[q]);
        part[blockIdx.x] = pt;
    }
    if (nr == 1) {
        for (size_t i = gtid; list && i < (size_t)B * E_max; i += gs) {
            const int b = (int)(i / (size_t)E_max), k = (int)(i % (size_t)E_max);
            if (k < clamp_count(ev_n[b], E_max)) list[i] = list_event(m, ev_t[i], clamp_src(ev_src[i], C_in), k);
        }
        return;
    }
    const size_t nwv = gs / kWave;
    for (size_t w = gtid / kWave; w < (size_t)B * nch; w += nwv) {
        const int b = (int)(w / (size_t)nch), ch = (int)(w % (size_t)nch);
        const int nb = clamp_count(ev_n[b], E_max);
        for (int r = lane; r < nr; r += kWave) s_cnt[wv][r] = 0;
        wave_lds_sync();
        const int k1 = min((ch + 1) * kListChunk, nb);
        for (int k = ch * kListChunk + lane; k < k1; k += kWave)
            atomicAdd(&s_cnt[wv][clamp_src(ev_src[(size_t)b * E_max + k], C_in) / rows], 1);
        wave_lds_sync();
        for (int r = lane; r < nr; r += kWave) cnt[((size_t)b * nr + r) * nch + ch] = s_cnt[wv][r];
        wave_lds_sync();
    }
}

// Workgroup 0: the fixed-point scale of the dL/dW sums and the way of the walk.
// Every contribution
// kappa (P^m - P^s) of a neuron is at most 2 kappa sum_s |mu_s| in size and a
// sum takes at most one contribution per event of the batch, so with
// bound = 2 kappa max_neuron(sum_s |mu_s|) (events in the batch) the scale
// 2^(62 - ceil(log2 bound)) keeps every sum below 2^62 (neurons whose sum is not
// finite left out: their own columns have no value, the others keep theirs).  A
// contribution is
// then below 2^62 / events; wide marks a call where that may reach
// 2^51, or where a sum is not finite.
// The way: kWayBlocks walks every (event, neuron) pair into LDS blocks (k_adjoint),
// kWayFew the neurons that have adjoints (few_way), kWayNone nothing.
// Workgroup 1 + b: the list of sample b's neurons that have adjoints, in neuron
// order, its chunks of 64 appended to pairs; and the exclusive prefix sum of the
// sample's event counts in (range, chunk) order, and where each range's list starts.
// Whether the neurons with adjoints alone are walked, their terms added by global
// atomics (scattered columns: 40 to 120 G adds/s) instead of every pair into LDS
// blocks (550 to 750 G pairs/s): by the pairs of the neurons with adjoints, on
// average over the samples, against all of them.  Measured, few against blocks:
// 700 -> 512, B = 128, 10 k events: 852 against 924 us at 7.0 %, 1050 against 928 at
// 8.8 %; 32768 -> 2048, B = 16, 100 k events (sums of 512 MB, past the 256 MB that the
// last-level cache holds): 3.08 against 4.01 ms at 3.6 %, 4.04 against 4.20 at 5.4 %,
// 6.7 against 4.4 at 12 %.  The blocks' clearing and adding is worth another 2^21
// pairs (2000 -> 1024, B = 2, 5000 events, 27 %: 46 against 58 us of walk).  Lists so
// sparse that their events are outnumbered by the spikes passed between them make
// the blocks' walk take event by event (32768 -> 2048, 500 events/s over 40 s, 8
// spikes a neuron: 3.9 against 4.8 ms).
__device__ __forceinline__ bool few_way(double live, double spikes, double ev, double B, double C_in, double N, int nr,
                                        bool lds)
{
    if (!lds) return true;
    const double share = C_in * N * sizeof(long long) > 0x1p28 ? 18.0 : 13.0;
    if (live * ev <= B * ev * N / share + 0x1p21 * B) return true;
    return nr >= 8 && spikes * kWave * nr >= 1.5 * ev * N;
}

__global__ __launch_bounds__(kPlanThreads) void k_bwd_plan(const BwdPart* __restrict__ part, int nparts,
                                                   const int32_t* __restrict__ ev_n, int B, int E_max, int C_in,
                                                   int N, double kappa, bool lds, const int32_t* __restrict__ ns_eff,
                                                   BwdCall* __restrict__ call, int32_t* __restrict__ live,
                                                   int32_t* __restrict__ nlive, int32_t* __restrict__ pairs,
                                                   int nr, int nch, int32_t* __restrict__ cnt,
                                                   int32_t* __restrict__ start)
{
    const int tid = (int)threadIdx.x, lane = tid % kWave, wv = tid / kWave;
    if (blockIdx.x == 0) {
        __shared__ double s_v[4][kPlanThreads / kWave];
        double mx = 0.0, ev = 0.0, nl = 0.0, sp = 0.0;
        bool bad = false;
        for (int i = tid; i < nparts; i += kPlanThreads) {
            const BwdPart q = part[i];
            bad |= q.bad != 0;
            mx = fmax(mx, q.mx);
            nl += (double)q.live;
            sp += (double)q.spikes;
        }
        for (int b = tid; b < B; b += kPlanThreads) ev += (double)clamp_count(ev_n[b], E_max);
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) {
            mx = fmax(mx, __shfl_xor(mx, off, kWave));
            ev += __shfl_xor(ev, off, kWave);
            nl += __shfl_xor(nl, off, kWave);
            sp += __shfl_xor(sp, off, kWave);
        }
        if (lane == 0) {
            s_v[0][wv] = mx;
            s_v[1][wv] = ev;
            s_v[2][wv] = nl;
            s_v[3][wv] = sp;
        }
        bad = __syncthreads_or(bad);
        if (tid == 0) {
            for (int q = 1; q < kPlanThreads / kWave; ++q) {
                mx = fmax(mx, s_v[0][q]);
                ev += s_v[1][q];
                nl += s_v[2][q];
                sp += s_v[3][q];
            }
            const double bound = 2.0 * kappa * mx * fmax(ev, 1.0);
            int ex = 0;
            if (bound > 0.0 && isfinite(bound)) frexp(bound, &ex);    // bound < 2^ex
            BwdCall c;
            c.scale = ldexp(1.0, 62 - ex);
            c.wide = bad || !(ev >= 4096.0) || !isfinite(bound) ? 1 : 0;
            c.way = kWayNone;
            if (nl > 0.0) c.way = few_way(nl, sp, ev, (double)B, (double)C_in, (double)N, nr, lds) ? kWayFew : kWayBlocks;
            *call = c;
        }
        return;
    }
    const int b = (int)blockIdx.x - 1;
    __shared__ int s_w[kPlanThreads / kWave];
    __shared__ int s_at;
    int nl = 0;
    for (int i0 = 0; i0 < N; i0 += kPlanThreads) {
        const int i = i0 + tid;
        const bool f = i < N && ns_eff[(size_t)b * N + i] != 0;
        const unsigned long long bal = __ballot(f);
        if (lane == 0) s_w[wv] = __popcll(bal);
        __syncthreads();
        int before = nl;
        for (int q = 0; q < kPlanThreads / kWave; ++q) {
            before += q < wv ? s_w[q] : 0;
            nl += s_w[q];
        }
        if (f) live[(size_t)b * N + before + __popcll(bal & ((1ull << lane) - 1ull))] = i;
        __syncthreads();
    }
    const int nc = (nl + kWave - 1) / kWave;
    if (tid == 0) {
        nlive[b] = nl;
        s_at = nc ? atomicAdd(pairs, nc) : 0;
    }
    __syncthreads();
    for (int q = tid; q < nc; q += kPlanThreads) pairs[1 + s_at + q] = b * ((N + kWave - 1) / kWave) + q;
    if (nr == 1) return;
    int32_t* c = cnt + (size_t)b * nr * nch;
    const int n = nr * nch;
    int base = 0;
    for (int i0 = 0; i0 < n; i0 += kPlanThreads) {
        const int i = i0 + tid;
        const int v = i < n ? c[i] : 0;
        int incl = v;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int x = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += x;
        }
        if (lane == kWave - 1) s_w[wv] = incl;
        __syncthreads();
        int before = base, tot = 0;
        for (int q = 0; q < kPlanThreads / kWave; ++q) {
            if (q < wv) before += s_w[q];
            tot += s_w[q];
        }
        const int ex = before + incl - v;
        if (i < n) {
            c[i] = ex;
            if (i % nch == 0) start[(size_t)b * (nr + 1) + i / nch] = ex;
        }
        base += tot;
        __syncthreads();
    }
    if (tid == 0) start[(size_t)b * (nr + 1) + nr] = base;
}

// The lists of several ranges: every event at its range's next place, in time
// order (one wave per (sample, chunk); equal ranges among
// 64 events ranked by ballots over the bits of the range).  kWayFew: no list; the
// fixed-point sums set to zero instead (gw, unless the setup pass has).
__global__ __launch_bounds__(kSetupThreads) void k_bwd_scatter(const float* __restrict__ ev_t,
                                                               const int32_t* __restrict__ ev_src,
                                                               const int32_t* __restrict__ ev_n, int B, int E_max,
                                                               int C_in, Model m, int nr, int rows, int nch,
                                                               const int32_t* __restrict__ cnt,
                                                               ListEvent* __restrict__ list,
                                                               const BwdCall* __restrict__ call,
                                                               long long* __restrict__ gw, size_t nW)
{
    const int way = call->way;
    if (way == kWayNone) return;
    if (way == kWayFew) {
        const size_t gtid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, gs = (size_t)gridDim.x * blockDim.x;
        if (gw)
            for (size_t i = gtid; i < nW; i += gs) gw[i] = 0;
        return;
    }
    __shared__ int32_t s_at[kSetupThreads / kWave][kAdjMaxRanges];
    const int lane = (int)threadIdx.x % kWave, wv = (int)threadIdx.x / kWave;
    const size_t w = (size_t)blockIdx.x * (kSetupThreads / kWave) + wv;
    if (w >= (size_t)B * nch) return;
    const int b = (int)(w / (size_t)nch), ch = (int)(w % (size_t)nch);
    const int nb = clamp_count(ev_n[b], E_max);
    const int k0 = ch * kListChunk, k1 = min(k0 + kListChunk, nb);
    if (k0 >= k1) return;
    int32_t* at = s_at[wv];
    for (int r = lane; r < nr; r += kWave) at[r] = cnt[((size_t)b * nr + r) * nch + ch];
    wave_lds_sync();
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int k = k0 + lane; k - lane < k1; k += kWave) {
        const bool ok = k < k1;
        const size_t o = (size_t)b * E_max + (ok ? k : k0);
        const int src = clamp_src(ev_src[o], C_in);
        const float t = ev_t[o];
        const int r = ok ? src / rows : 0;
        unsigned long long same = __ballot(ok);
        for (int bit = 1; bit < nr; bit <<= 1) {
            const unsigned long long m = __ballot((r & bit) != 0);
            same &= (r & bit) ? m : ~m;
        }
        const int pos = at[r] + __popcll(same & below);
        wave_lds_sync();
        if (ok) {
            list[(size_t)b * E_max + pos] = list_event(m, t, src, k);
            if ((same & below) == 0ull) at[r] = pos + __popcll(same);
        }
        wave_lds_sync();
    }
}

// Accumulators -> float32 outputs: dL/dW from fixed point (where blocks are
// split or neurons few; else the walk has written it), dL/dt as the sum of the
// tiles' (kWayFew: the chunks') partial sums in order (0 on padding).
__global__ __launch_bounds__(256) void k_bwd_convert(const long long* __restrict__ gw, bool split,
                                                     const BwdCall* __restrict__ call,
                                                     float* __restrict__ grad_WT, size_t nW,
                                                     const double* __restrict__ gt, int tiles,
                                                     const int32_t* __restrict__ nlive,
                                                     const int32_t* __restrict__ ev_n, int E_max,
                                                     float* __restrict__ grad_ev_t, size_t nT)
{
    const size_t gtid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t gs = (size_t)gridDim.x * blockDim.x;
    const int way = call->way;
    if (way == kWayNone) {
        for (size_t i = gtid; i < nW; i += gs) grad_WT[i] = 0.0f;
    } else if (split || way == kWayFew) {
        const double inv = 1.0 / call->scale;
        for (size_t i = gtid; i < nW; i += gs) grad_WT[i] = (float)((double)gw[i] * inv);
    }
    if (gt)
        for (size_t i = gtid; i < nT; i += gs) {
            const int b = (int)(i / (size_t)E_max), k = (int)(i % (size_t)E_max);
            double s = 0.0;
            if (way != kWayNone && k < clamp_count(ev_n[b], E_max)) {
                const int nq = way == kWayFew ? (nlive[b] + kWave - 1) / kWave : tiles;
                for (int q = 0; q < nq; ++q) s += gt[(size_t)q * nT + i];
            }
            grad_ev_t[i] = (float)s;
        }
}

// A term v ks as a 64-bit integer, rounded to nearest even.  When it is below
// 2^51 in size (not kWide), the integer is in the low bits of the sum with
// 1.5 2^52, whose own bits are 0x43380000 in the high word: three instructions
// against eleven.
template <bool kWide>
__device__ __forceinline__ unsigned long long fx_term(double v, double ks)
{
    if constexpr (kWide) return (unsigned long long)llrint(v * ks);
    return (unsigned long long)__double_as_longlong(fma(v, ks, 0x1.8p52)) - 0x4338000000000000ull;
}

struct AdjArgs {
    const float* ev_t;
    const int32_t *ev_src, *ev_n;
    const float* WT;
    const float* out_t;
    const int32_t *out_k, *ns;
    const double2* r;
    const BwdCall* call;
    const int32_t *live, *nlive, *pairs;
    const int32_t* start;
    const ListEvent* list;
    long long* gw;
    float* grad_WT;
    double* gt;
    size_t nT;
    double kappa, inv_tm, inv_ts, len, inv_len;            // len: kRefTs tau_s
    double fm, fs, gm, gs;                                 // e^{-len/tm}, e^{-len/ts} and their reciprocals
    int B, E_max, C_in, N, s_max, tiles, nr, rows, Q, S;
};

// P at time tk from the R of a neuron's spikes s .. ns - 1 (its first spike is
// entry so), exponentials and all: the general form of P = R H.  A spike whose
// float32 time lies before tk counts with offset 0.  (len and inv_len are the
// numbers that the table was built with: a spike time on a multiple of len may
// fall on either side of it under any others.  A call: inlined, the
// constants of its exponentials would hold registers all through the walk.)
__device__ __noinline__ double2 p_at(const float* ts, const double2* rr, int s, int ns, double tk, double len,
                                     double inv_len, double inv_tm, double inv_ts)
{
    double am = 0.0, as = 0.0;
    double2 q1 = make_double2(0.0, 0.0);
    for (;; ++s) {
        const double t1 = (double)ts[s], dr = ref_offset(t1, ref_index(t1, inv_len), len);
        q1 = make_double2(rr[s].x * exp(dr * inv_tm), rr[s].y * exp(dr * inv_ts));       // Q_s
        const double du = t1 - tk;
        if (!(du < 0.0)) return make_double2(fma(q1.x, exp(-du * inv_tm), am), fma(q1.y, exp(-du * inv_ts), as));
        if (s + 1 >= ns) return make_double2(am + q1.x, as + q1.y);
        const double t2 = (double)ts[s + 1], d2 = ref_offset(t2, ref_index(t2, inv_len), len), dt = t2 - t1;
        am += q1.x - rr[s + 1].x * exp((d2 - dt) * inv_tm);                              // mu_s
        as += q1.y - rr[s + 1].y * exp((d2 - dt) * inv_ts);
    }
}

// One workgroup per (64 neurons, channel range, slice of the (sample, part)
// units); lanes are neurons and a wave takes one unit at a time (a counter in
// LDS), walking its listed events backwards: at event k, with P = R H, dL/dw
// += kappa (P^m - P^s) into the block in LDS and the tile's part of dL/dt_k,
// the sum over lanes of w kappa (P^m/tm - P^s/ts), is stored; then a lane with
// spikes between the listed event before it and event k switches its R.  The
// spikes that a group of kGrp events passes are looked up before the group, all
// lanes together (at most two per lane); a group where a lane passes more takes its
// last event by itself until they fit.  Units with spike times before events that
// the spikes follow take the walk without a reference, with P from p_at there (setup
// looks for these spikes; a check in every group of the common walk cost it 4 %).
// kLds = false: the listed neurons, dL/dW by global atomics; kTime: dL/dt wanted
// (else no weight is read).
// Bound by VALU issue (78 % busy at the first shape below, 74 % at the second):
// about 30 instructions per (event, 64 neurons), float64 four cycles each.  H
// and the rows come by lane reads: as LDS broadcasts they shared the pipe
// with the adds and bounded the walk (1.44 against 0.97 ms).  Twelve waves of up
// to 168 registers against sixteen of 128 with spills: 5.9 against 7.0 ms at the
// second shape with three units per wave, when it took that long.  With dL/dt,
// 700 -> 512, B = 128, 10 k events, 70 % firing: 0.99 ms; 32768 -> 2048, B = 16,
// 100 k events: 5.4 ms (one wave per 64 events with global atomics: 3.69 and 22.4
// ms).
template <bool kLds, bool kTime>
__device__ __forceinline__ void adjoint_units(const AdjArgs& a, unsigned long long* s_acc, int& s_next)
{
    const int lane = (int)threadIdx.x % kWave;
    // kLds: the workgroup's tile of 64 neurons and channel range; else a unit
    // brings its own 64 neurons, a chunk of its sample's list
    int tile = (int)(blockIdx.x % (unsigned)a.tiles);
    const int r = kLds ? (int)((blockIdx.x / (unsigned)a.tiles) % (unsigned)a.nr) : 0;
    const int slice = kLds ? (int)(blockIdx.x / ((unsigned)a.tiles * (unsigned)a.nr)) : (int)blockIdx.x;
    const int S = kLds ? a.S : (int)gridDim.x;
    const int c0 = r * a.rows, rows = kLds ? min(a.rows, a.C_in - c0) : 0;
    int n = tile * kWave + lane;
    bool live = n < a.N;
    int nc = live ? n : 0;
    // parts of a sample's list: of whole blocks of 64 events, for kFewUnits units
    // in all, none longer than 1024 events
    int Q = a.Q;
    if constexpr (!kLds) {
        const int blocks = (a.E_max + kWave - 1) / kWave;
        const int per = (int)min(max((long long)a.pairs[0] * blocks / kFewUnits, 1ll), 16ll);
        Q = (blocks + per - 1) / per;
    }
    if (kLds)
        for (int i = (int)threadIdx.x; i < rows * kWave; i += (int)blockDim.x) s_acc[i] = 0ull;
    if (threadIdx.x == 0) s_next = 0;
    __syncthreads();
    const double scale = a.call->scale, ks = a.kappa * scale;
    const bool wide = __builtin_amdgcn_readfirstlane(a.call->wide) != 0;
    const double ktm = a.kappa * a.inv_tm, kts = -a.kappa * a.inv_ts;
    const bool lists = kLds && a.nr > 1;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)a.WT, (short)0, (int)((uint32_t)a.C_in * (uint32_t)a.N * 4u), kRsrcWord3);
    const long long units = (long long)(kLds ? a.B : a.pairs[0]) * Q;
    for (;;) {
        int u = 0;
        if (lane == 0) u = atomicAdd(&s_next, 1);
        u = __builtin_amdgcn_readfirstlane(u);
        const long long id = slice + (long long)u * S;
        if (id >= units) break;
        int b = (int)(id / Q);
        const int q = (int)(id % Q);
        if constexpr (!kLds) {
            const int pair = __builtin_amdgcn_readfirstlane(a.pairs[1 + b]);
            b = pair / a.tiles;
            tile = pair % a.tiles;
            live = tile * kWave + lane < a.nlive[b];
            n = nc = live ? a.live[(size_t)b * a.N + tile * kWave + lane] : 0;
        }
        const int nb = clamp_count(a.ev_n[b], a.E_max);
        const int L0 = lists ? a.start[(size_t)b * (a.nr + 1) + r] : 0;
        const int L1 = lists ? a.start[(size_t)b * (a.nr + 1) + r + 1] : nb;
        const int per = ((L1 - L0 + Q - 1) / Q + kWave - 1) / kWave * kWave;
        const int l0 = L0 + q * per, l1 = min(l0 + per, L1);
        if (l0 >= l1) continue;
        const ListEvent* ll = a.list + (size_t)b * a.E_max;
        // a block of 64 listed events at l (lane i: event l + i, the last one
        // again past l1)
        // (kWayFew: the sample's own events in order, no list)
        const float* et = a.ev_t + (size_t)b * a.E_max;
        auto load = [&](int l) {
            const int x = min(l + lane, l1 - 1);
            if constexpr (kLds) return ll[x];
            else
                return list_event(a.len, a.inv_len, a.inv_tm, a.inv_ts, et[x],
                                  clamp_src(a.ev_src[(size_t)b * a.E_max + x], a.C_in), x);
        };
        auto rl_f = [](float v, int l) {
            return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
        };
        const size_t bn = (size_t)b * a.N + nc;
        int ns = live ? a.ns[bn] : 0;
        const bool early = __ballot(ns < 0) != 0ull;
        ns = ns < 0 ? ~ns : ns;
        const size_t so = bn * (size_t)a.s_max;            // the neuron's spikes
        double* gt = kTime ? a.gt + (size_t)tile * a.nT + (size_t)b * a.E_max : nullptr;
        int lb = l0 + ((l1 - l0 - 1) / kWave) * kWave;     // the topmost block
        ListEvent cur = load(lb);
        const int kfirst = kLds ? __builtin_amdgcn_readfirstlane(ll[l0].k) : l0;
        if (__ballot(ns > 0 && a.out_k[so + max(ns - 1, 0)] > kfirst) == 0ull) {
            // no neuron fires after the unit's first event
            if (kTime)
                for (int l = l0 + lane; l < l1; l += kWave) gt[kLds ? ll[l].k : l] = 0.0;
            continue;
        }
        int cnt = l1 - lb;                                 // events of the block
        int sp;                                            // first spike with out_k > k of the walk's event
        {
            const int kt = __builtin_amdgcn_readlane(cur.k, cnt - 1);
            int lo = 0, hi = ns;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (a.out_k[so + mid] > kt) hi = mid; else lo = mid + 1;
            }
            sp = lo;
        }
        // the next spike the walk meets, sp - 1 (when sp >= 1), and k of the one
        // after it.  Loaded under the lanes' condition and nothing else, straight
        // into place: selects on the loaded values wait for the loads (5 % of the
        // walk at the second shape).
        int k1 = 0, k2 = 0;
        float t1 = 0.0f;
        double2 R1 = make_double2(0.0, 0.0);
        auto refill = [&]() {
            const size_t i1 = so + max(sp - 1, 0), i2 = so + max(sp - 2, 0);
            k1 = a.out_k[i1];
            t1 = a.out_t[i1];
            R1 = a.r[i1];
            k2 = a.out_k[i2];
        };
        if (ns > 0) refill();
        // The unit's reference is its first event's.  A unit over more than 3 len
        // (sparse streams, lists of few channels) has none: there the walk
        // carries P itself instead of R, with the decays from event to event;
        // that walk also looks out for spike times before events that the spikes
        // follow (offsets of 0: p_at).
        const int ref = __builtin_amdgcn_readfirstlane(kLds ? ll[l0].ref : ref_index((double)et[l0], a.inv_len));
        const bool other = early || __builtin_amdgcn_readlane(cur.ref, cnt - 1) - ref > 3;
        // R of a spike at time t referred to reference r
        auto refer = [&](double2 v, float t, int r) {
            const int d = ref_index((double)t, a.inv_len) - r;
            if (__builtin_expect(d != 0, 0)) {
                v.x *= ref_pow(a.fm, a.gm, d);
                v.y *= ref_pow(a.fs, a.gs, d);
            }
            return v;
        };
        auto load_w = [&](int woff, int g, float (&w)[kGrp]) {
            if constexpr (kTime) {
#pragma unroll
                for (int j = 0; j < kGrp; ++j)
                    w[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                         rsrc, (uint32_t)nc * 4u,
                                                         __builtin_amdgcn_readlane(woff, g * kGrp + j), 0));
            }
        };
        // the walk: kWide as in fx_term, kRef with a reference
        auto walk = [&](auto wide_tag, auto ref_tag) {
            constexpr bool kWide = decltype(wide_tag)::value, kRef = decltype(ref_tag)::value;
            auto add_w = [&](unsigned long long x, int ro) {
                if constexpr (kLds) atomicAdd(&s_acc[ro + lane], x);
                else if (x != 0ull) atomicAdd((unsigned long long*)&a.gw[(size_t)ro + n], x);
            };
            const int rmul = kLds ? kWave : a.N;
            double Rm = 0.0, Rs = 0.0;
            float w[kGrp], wn[kGrp];
            int woff = cur.src * a.N * 4;
            load_w(woff, (cnt - 1) / kGrp, w);
            // R of spike sp, or its P at event e of the block; then 1 when a
            // lane's spike lies before that event
            auto take = [&](int e) {
                Rm = Rs = 0.0;
                bool early = false;
                if (sp < ns) {
                    const float t = a.out_t[so + sp];
                    const double2 v = refer(a.r[so + sp], t, kRef ? ref : __builtin_amdgcn_readlane(cur.ref, e));
                    Rm = kRef ? v.x : v.x * read_lane_double(cur.Hm, e);
                    Rs = kRef ? v.y : v.y * read_lane_double(cur.Hs, e);
                    early = t < rl_f(cur.t, e);
                    // (waited for here: a load into Rm or Rs still in flight on
                    // some path has every group wait for its newest loads)
                    asm volatile("" : "+v"(Rm), "+v"(Rs));
                }
                return __ballot(early) != 0ull ? 1 : 0;
            };
            int late = take(cnt - 1), again = 0;           // the last take's; R to be taken at the next block
            for (;;) {
                const bool more = lb > l0;
                ListEvent nxt = cur;
                if (more) nxt = load(lb - kWave);
                // factors of the block's events: H referred to the unit's
                // reference, or the decays to the listed event below
                double hm = cur.Hm, hs = cur.Hs;
                if constexpr (kRef) {
                    if (__ballot(cur.ref != ref)) {
                        asm volatile("");
                        const int d = min(max(cur.ref - ref, 0), 3);
                        hm *= ref_pow(a.gm, a.fm, d);
                        hs *= ref_pow(a.gs, a.fs, d);
                    }
                } else {
                    float tb = __shfl_up(cur.t, 1, kWave);
                    if (lane == 0) tb = rl_f(more ? nxt.t : cur.t, more ? kWave - 1 : 0);
                    const double dt = fmax((double)cur.t - (double)tb, 0.0);
                    hm = exp(-dt * a.inv_tm);
                    hs = exp(-dt * a.inv_ts);
                }
                const int row = (cur.src - c0) * rmul;
                const int woff_n = nxt.src * a.N * 4;
                // k and time of the event below the block (past the unit's
                // first event spikes do not matter)
                const int kbelow = __builtin_amdgcn_readlane(more ? nxt.k : cur.k, more ? kWave - 1 : 0);
                float tbelow = 0.0f;
                if constexpr (!kRef) tbelow = rl_f(more ? nxt.t : cur.t, more ? kWave - 1 : 0);
                for (int g = (cnt - 1) / kGrp; g >= 0; --g) {
                    const int klo = g > 0 ? __builtin_amdgcn_readlane(cur.k, g > 0 ? g * kGrp - 1 : 0) : kbelow;
                    int ne = min(kGrp, cnt - g * kGrp);
                    bool any = false, any2 = false;
                    int x1 = -1, x2 = -1;                  // R switched after event x of the group
                    double2 X1 = make_double2(0.0, 0.0), X2 = X1;
                    // the spikes that the group passes; while a lane passes too
                    // many of them (or, late, spikes come before their events)
                    // the group's last event is taken by itself
                    for (;;) {
                        const bool pass = sp >= 1 && k1 > klo;
                        any = __ballot(pass) != 0ull;
                        any2 = false;
                        // (scalars: the branches below and the flags set under them are uniform)
                        bool slow = false;
                        if constexpr (!kRef) slow = __builtin_amdgcn_readfirstlane(late) != 0;
                        if (any && (kRef || !slow)) {
                            const bool pass2 = pass && sp >= 2 && k2 > klo;
                            any2 = __ballot(pass2) != 0ull;
                            int y1 = 0;
#pragma unroll
                            for (int j = 0; j < kGrp; ++j)
                                y1 += __builtin_amdgcn_readlane(cur.k, g * kGrp + j) < k1 ? 1 : 0;
                            // what R is referred to below event e + 1: the unit's
                            // reference, or (P) the time of the listed event e
                            auto below = [&](double2 v, float t, int e) {
                                if constexpr (kRef) return refer(v, t, ref);
                                const int l = max(e, 0);
                                int rb = __shfl(cur.ref, l, kWave);
                                double Hm = __shfl(cur.Hm, l, kWave), Hs = __shfl(cur.Hs, l, kWave);
                                if (e < 0) {
                                    rb = __builtin_amdgcn_readlane(nxt.ref, kWave - 1);
                                    Hm = read_lane_double(nxt.Hm, kWave - 1);
                                    Hs = read_lane_double(nxt.Hs, kWave - 1);
                                }
                                v = refer(v, t, rb);
                                return make_double2(v.x * Hm, v.y * Hs);
                            };
                            // the listed event below, event y1 - 1
                            const int el = g * kGrp + min(y1, kGrp - 1) - 1;
                            bool bad = false;
                            if constexpr (!kRef) {
                                const float te = __shfl(cur.t, max(el, 0), kWave);
                                bad = pass && t1 < (el < 0 ? tbelow : te);
                            }
                            float t2 = 0.0f;
                            int el2 = -1;
                            if (__builtin_expect(any2, 0)) {
                                int y2 = 0;
                                if (pass2) t2 = a.out_t[so + sp - 2];
#pragma unroll
                                for (int j = 0; j < kGrp; ++j)
                                    y2 += __builtin_amdgcn_readlane(cur.k, g * kGrp + j) < k2 ? 1 : 0;
                                el2 = g * kGrp + min(y2, kGrp - 1) - 1;
                                bad = bad || (pass2 && sp >= 3 && a.out_k[so + max(sp - 3, 0)] > klo);
                                if constexpr (!kRef) {
                                    const float te2 = __shfl(cur.t, max(el2, 0), kWave);
                                    bad = bad || (pass2 && t2 < (el2 < 0 ? tbelow : te2));
                                }
                                x2 = pass2 ? y2 : -1;
                            }
                            slow = __ballot(bad) != 0ull;
                            if (!slow) {
                                if constexpr (!kRef) {         // (all lanes: the shuffles)
                                    X1 = below(R1, t1, el);
                                    if (any2) X2 = below(pass2 ? a.r[so + sp - 2] : X2, t2, el2);
                                }
                                if (pass) {
                                    x1 = y1;
                                    if constexpr (kRef) {
                                        // (a copy: the next R1 then loads into R1's registers)
                                        double2 q = R1;
                                        asm volatile("" : "+v"(q.x), "+v"(q.y));
                                        X1 = below(q, t1, el);
                                    }
                                    --sp;
                                    if (pass2) {
                                        if constexpr (kRef) X2 = below(a.r[so + sp - 1], t2, el2);
                                        --sp;
                                    }
                                    refill();
                                }
                            }
                        }
                        if (__builtin_expect(!slow, 1)) break;
                        {
                            const int e = g * kGrp + ne - 1;
                            const double fm = read_lane_double(hm, e), fs = read_lane_double(hs, e);
                            double2 P = kRef ? make_double2(Rm * fm, Rs * fs) : make_double2(Rm, Rs);
                            if constexpr (!kRef) {
                                if (late) {
                                    P = make_double2(0.0, 0.0);
                                    if (sp < ns)
                                        P = p_at(a.out_t + so, a.r + so, sp, ns, (double)rl_f(cur.t, e), a.len,
                                                 a.inv_len, a.inv_tm, a.inv_ts);
                                }
                                Rm *= fm;
                                Rs *= fs;
                            }
                            add_w(fx_term<kWide>(P.x - P.y, ks), __builtin_amdgcn_readlane(row, e));
                            if constexpr (kTime) {
                                float we = w[0];
#pragma unroll
                                for (int j = 1; j < kGrp; ++j) we = ne - 1 == j ? w[j] : we;
                                double s = (double)we * fma(ktm, P.x, kts * P.y);
#pragma unroll
                                for (int off = kWave / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, kWave);
                                if (lane == 0) gt[__builtin_amdgcn_readlane(cur.k, e)] = s;
                            }
                            const int kp = ne > 1 ? __builtin_amdgcn_readlane(cur.k, max(e - 1, 0)) : klo;
                            const int sp0 = sp;
                            while (sp > 0 && ns > 0 && a.out_k[so + sp - 1] > kp) --sp;
                            if (late || __ballot(sp < sp0)) {
                                // R at the listed event below (below the block: there)
                                if (kRef || e > 0) late = take(max(e - 1, 0));
                                else again = 1;
                                if (ns > 0) refill();
                            }
                        }
                        if (--ne == 0) break;
                    }
                    // (one set of loads for the group below in this block or the
                    // next: in two branches the compiler copies the loaded
                    // values, and waits for them, right away)
                    load_w(g > 0 ? woff : woff_n, g > 0 ? g - 1 : (more ? kWave / kGrp - 1 : 0), wn);
                    if (__builtin_expect(ne > 0, 1)) {
                        double ca[kGrp / 2], c4[kGrp / 2];
                        auto events = [&](auto full_tag) {
                            constexpr bool kFull = decltype(full_tag)::value;
#pragma unroll
                            for (int jj = kGrp - 1; jj >= 0; --jj) {
                                double cj = 0.0;
                                if (kFull || jj < ne) {
                                    const int e = g * kGrp + jj;
                                    const double fm = read_lane_double(hm, e), fs = read_lane_double(hs, e);
                                    const double Pm = kRef ? Rm * fm : Rm, Ps = kRef ? Rs * fs : Rs;
                                    add_w(fx_term<kWide>(Pm - Ps, ks), __builtin_amdgcn_readlane(row, e));
                                    if constexpr (kTime) cj = (double)w[jj] * fma(ktm, Pm, kts * Ps);
                                    if constexpr (!kRef) {
                                        Rm *= fm;
                                        Rs *= fs;
                                    }
                                    if (any && __ballot(x1 == jj)) {
                                        asm volatile("");          // a branch, not eight selects per event
                                        if (x1 == jj) {
                                            Rm = X1.x;
                                            Rs = X1.y;
                                        }
                                    }
                                    if (any2 && __ballot(x2 == jj)) {
                                        asm volatile("");
                                        if (x2 == jj) {
                                            Rm = X2.x;
                                            Rs = X2.y;
                                        }
                                    }
                                }
                                // (the first exchange of group_sum8 as soon as
                                // both of its values are there)
                                if constexpr (kTime) {
                                    if (jj >= kGrp / 2) ca[jj - kGrp / 2] = cj;
                                    else c4[jj] = swap_sum32(cj, ca[jj]);
                                }
                            }
                        };
                        if (ne == kGrp) events(std::true_type{});
                        else events(std::false_type{});
                        if constexpr (kTime) {
                            const double s = group_sum4(c4, lane);
                            const int j = ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
                            const int k = __shfl(cur.k, g * kGrp + j, kWave);
                            if ((lane & 7) == 0 && j < ne) gt[k] = s;
                        }
                    }
                    if constexpr (kTime) {
#pragma unroll
                        for (int j = 0; j < kGrp; ++j) {
                            asm volatile("" : "+v"(wn[j]));    // the wait for the loads here, not among the events
                            w[j] = wn[j];
                        }
                    }
                }
                if (!more) break;
                cur = nxt;
                woff = woff_n;
                lb -= kWave;
                cnt = kWave;
                if (!kRef && again) {
                    late = take(cnt - 1);
                    again = 0;
                }
            }
        };
        if (__builtin_expect(other, 0)) walk(std::true_type{}, std::false_type{});
        else if (__builtin_expect(wide, 0)) walk(std::true_type{}, std::true_type{});
        else walk(std::false_type{}, std::true_type{});
    }
    if constexpr (kLds) {
        __syncthreads();
        const double inv = 1.0 / scale;
        for (int i = (int)threadIdx.x; i < rows * kWave; i += (int)blockDim.x) {
            const int nn = tile * kWave + i % kWave;
            if (nn >= a.N) continue;
            const size_t at = (size_t)(c0 + i / kWave) * a.N + nn;
            const long long v = (long long)s_acc[i];
            if (a.S == 1) a.grad_WT[at] = (float)((double)v * inv);
            else if (v) atomicAdd((unsigned long long*)&a.gw[at], (unsigned long long)v);
        }
    }
}

template <bool kTime>
__global__ __launch_bounds__(kAdjThreads) void k_adjoint(const AdjArgs a)
{
    extern __shared__ unsigned long long s_acc[];          // kWayBlocks: [rows][64] sums
    __shared__ int s_next;
    const int way = __builtin_amdgcn_readfirstlane(a.call->way);
    if (way == kWayBlocks) adjoint_units<true, kTime>(a, s_acc, s_next);
    else if (way == kWayFew) adjoint_units<false, kTime>(a, s_acc, s_next);
}

int backward_impl(const float* ev_t, const int32_t* ev_src, const int32_t* ev_n, int B, int E_max, const float* WT,
                  int C_in, int N, const lif_params* p, const float* out_t, const int32_t* out_n,
                  const float* out_i, const int32_t* out_k, const float* grad_out_t, float* grad_WT,
                  float* grad_ev_t, void* ws, size_t ws_bytes, hipStream_t stream)
{
    int rc = check_params(p);
    if (rc) return rc;
    if (B < 0 || E_max < 0 || C_in < 1 || N < 1) return LIF_ERR_ARG;
    if (!WT || !out_t || !out_n || !out_i || !out_k || !grad_out_t || !grad_WT || !ws) return LIF_ERR_ARG;
    if (B > 0 && !ev_n) return LIF_ERR_ARG;
    if ((size_t)B * (size_t)E_max > 0 && (!ev_t || !ev_src)) return LIF_ERR_ARG;
    if ((size_t)C_in * (size_t)N >= ((size_t)1 << 29)) return LIF_ERR_SIZE;   // 32-bit W^T byte offsets
    BwdLayout L = bwd_layout(B, E_max, C_in, N, p->s_max);
    if (ws_bytes < L.total) return LIF_ERR_WORKSPACE;
    const BwdPlan& P = L.P;
    // kWayFew alone: at most 256 workgroups, of as few waves as hold its units
    const size_t fewu = (size_t)B * P.tiles * ((E_max + kWave - 1) / kWave);      // at most
    const size_t few_waves = fewu < (size_t)kCus * kAdjWaves ? (fewu + kCus - 1) / kCus : kAdjWaves;
    const size_t few_wgs = few_waves ? (fewu + few_waves - 1) / few_waves : 1;
    const size_t wgs = P.lds ? (size_t)P.tiles * P.nr * P.S : (few_wgs < (size_t)kCus ? few_wgs : kCus);
    if ((size_t)B * ((E_max + kSeg - 1) / kSeg) * P.tiles > 0x7fffffff || wgs > 0x7fffffff ||
        (size_t)B * P.Q > 0x3fffffff)
        return LIF_ERR_SIZE;
    Model m = make_model(*p);
    char* base = (char*)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    double2* q = (double2*)(base + L.q);
    int32_t* ns = (int32_t*)(base + L.ns);
    BwdPart* part = (BwdPart*)(base + L.part);
    BwdCall* call = (BwdCall*)(base + L.call);
    int32_t* live = (int32_t*)(base + L.live);
    int32_t* nlive = (int32_t*)(base + L.nlive);
    int32_t* pairs = (int32_t*)(base + L.pairs);
    const bool lists = P.nr > 1;
    int32_t* cnt = lists ? (int32_t*)(base + L.cnt) : nullptr;
    int32_t* start = lists ? (int32_t*)(base + L.start) : nullptr;
    ListEvent* list = P.lds ? (ListEvent*)(base + L.list) : nullptr;
    const size_t nW = (size_t)C_in * N, nT = (size_t)B * E_max, nn = (size_t)B * N;
    const bool split = P.S > 1;                            // blocks of several workgroups (else the walk writes dL/dW)
    long long* gw = (long long*)(base + L.gw);
    // the sums are set to zero by the setup pass where they are used for certain or
    // are small, else by k_bwd_scatter if they turn out to be used
    const bool zero = split || !lists || nW <= ((size_t)1 << 19);
    double* gt = grad_ev_t ? (double*)(base + L.gt) : nullptr;
    const size_t chunks = (size_t)B * P.nch;
    size_t work = nn;
    if (zero && nW > work) work = nW;
    if (lists && chunks * kWave > work) work = chunks * kWave;
    if (!lists && list && nT > work) work = nT;
    size_t blocks = (work + kSetupThreads - 1) / kSetupThreads;
    blocks = blocks < 1 ? 1 : (blocks > kSetupBlocks ? kSetupBlocks : blocks);
    TIMED_LAUNCH("bwd_setup", k_bwd_setup, dim3((unsigned)blocks), dim3(kSetupThreads), 0, stream, ev_t, ev_src,
                 ev_n, B, E_max, C_in, N, m, zero ? gw : nullptr, nW, out_t, out_n, out_i, out_k, grad_out_t, q, ns,
                 part, pairs, P.nr, P.rows, P.nch, cnt, list);
    TIMED_LAUNCH("bwd_plan", k_bwd_plan, dim3((unsigned)(1 + B)), dim3(kPlanThreads), 0, stream, part, (int)blocks,
                 ev_n, B, E_max, C_in, N, m.kappa, P.lds, ns, call, live, nlive, pairs, P.nr, P.nch, cnt, start);
    if (lists && chunks) {
        size_t sblocks = (chunks + kSetupThreads / kWave - 1) / (kSetupThreads / kWave);
        const size_t zblocks = zero ? 0 : (nW / 8 + kSetupThreads - 1) / kSetupThreads;   // (eight words a thread)
        const size_t cap = sblocks > kSetupBlocks ? sblocks : kSetupBlocks;
        if (zblocks > sblocks) sblocks = zblocks < cap ? zblocks : cap;
        TIMED_LAUNCH("bwd_scatter", k_bwd_scatter, dim3((unsigned)sblocks), dim3(kSetupThreads), 0, stream, ev_t, ev_src,
                     ev_n, B, E_max, C_in, m, P.nr, P.rows, P.nch, cnt, list, call, zero ? nullptr : gw, nW);
    }
    size_t most = ((size_t)B * P.Q + P.S - 1) / P.S;          // units of a workgroup
    if (P.lds && (fewu + wgs - 1) / wgs > most) most = (fewu + wgs - 1) / wgs;
    if (!P.lds) most = few_waves;
    const int waves = (int)(most < 1 ? 1 : (most > kAdjWaves ? kAdjWaves : most));
    const size_t lds = P.lds ? (size_t)P.rows * kWave * sizeof(long long) : 0;
    const double len = kRefTs * m.ts;
    const AdjArgs a{ev_t, ev_src, ev_n, WT, out_t, out_k, ns, q, call, live, nlive, pairs, start, list, gw, grad_WT, gt,
                    nT, m.kappa, m.inv_tm, m.inv_ts, len, 1.0 / len, exp(-len * m.inv_tm), exp(-len * m.inv_ts),
                    exp(len * m.inv_tm), exp(len * m.inv_ts), B, E_max, C_in, N, m.s_max, P.tiles, P.nr, P.rows, P.Q,
                    P.S};
    auto adjoint = [&](auto kern) -> int {
        // the block exceeds the default dynamic-LDS limit; the attribute is
        // set on every call (for the current device; no state kept here)
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)(kAdjRows * kWave * sizeof(long long))) != hipSuccess)
            return LIF_ERR_HIP;
        TIMED_LAUNCH("event_adjoint", kern, dim3((unsigned)wgs), dim3(kWave * waves), lds, stream, a);
        return LIF_OK;
    };
    rc = gt ? adjoint(k_adjoint<true>) : adjoint(k_adjoint<false>);
    if (rc) return rc;
    work = nW;
    if (gt && nT > work) work = nT;
    blocks = (work + 255) / 256;
    blocks = blocks < 1 ? 1 : (blocks > 2048 ? 2048 : blocks);
    TIMED_LAUNCH("bwd_convert", k_bwd_convert, dim3((unsigned)blocks), dim3(256), 0, stream, gw, split, call, grad_WT,
                 nW, gt, P.tiles, nlive, ev_n, E_max, grad_ev_t, nT);
    return check_launch();
}

}  // namespace lif

extern "C" size_t lif_layer_backward_workspace_size(int B, int E_max, int C_in, int N_out, const lif_params* p)
{
    if (B < 0 || E_max < 0 || C_in < 1 || N_out < 1 || !p || p->s_max < 1) return 0;
    return lif::bwd_layout(B, E_max, C_in, N_out, p->s_max).total;
}

extern "C" int lif_layer_backward(const float* ev_t, const int32_t* ev_src, const int32_t* ev_n, int B, int E_max,
                                  const float* WT, int C_in, int N_out, const lif_params* p, const float* out_t,
                                  const int32_t* out_n, const float* out_i, const int32_t* out_k,
                                  const float* grad_out_t, float* grad_WT, float* grad_ev_t, void* ws,
                                  size_t ws_bytes, lif_stream_t stream)
{
    return lif::backward_impl(ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, p, out_t, out_n, out_i, out_k,
                              grad_out_t, grad_WT, grad_ev_t, ws, ws_bytes, (hipStream_t)stream);
}
