// lif_forward.hip -- forward pass of the event-driven LIF layer on gfx950.
//
// Pipeline for one call (a sample is one sorted event queue, shared by the
// N neurons of the layer):
//   k_aggregate  per (sample, segment, tile of 64 NPL neurons): the affine
//                map M(dt) of Eq. affine depends only on the gap to the
//                previous event, so the segment's maps are computed once per
//                sample (the first tile's wave stores them, and the composed
//                map of the segment: the maps form a semigroup,
//                M(a) M(b) = M(a + b)) and shared by every neuron.  One wave walks
//                the segment from the zero state in the eigen-coordinates
//                (U, J) of the maps (two FMAs per neuron-event, the decays as
//                scalar operands).  Lane l holds NPL adjacent neurons and
//                reads their weights of an event with one vector load from
//                the event's W^T row.  The result is the b-part of the
//                Combine of the segment's maps.
//   k_carry      per (sample, 64 neurons): exclusive Combine scan over the
//                segments (diagonal maps in (U, J)), giving the no-reset
//                state entering every segment; it overwrites the aggregates.
//   k_check      per (sample, segment, tile): re-walk from the carried state
//                with a no-crossing screen per inter-event interval
//                (screen_value).  Resets only lower V, so a sub-block of kSub
//                events whose no-reset trajectory passes every screen holds
//                no spike whatever happened before it; a flagged sub-block
//                reserves a pool entry and stores its entering state there.
//   k_resolve    per (sample, neuron) with flagged sub-blocks, one wave: walks
//                only those, in time order, passing over every sub-block whose
//                key bound (stored by the check pass) lies below the key of
//                the current reset deficit.  The wave rebuilds the no-reset
//                state at every interval start of four sub-blocks at a time
//                and computes each interval's crossing key.  Spikes found so
//                far lower V by a known decaying amount (the reset deficit),
//                which corrects the no-reset states exactly; an interval
//                crosses iff its key is at least the deficit's current key
//                (the interval rule of Sec. 3.2.2, one compare per interval).
//                The spike time is solved by bracketed Newton (Appendix D.1),
//                V is hard-reset and the same interval is tested again from
//                the spike (Appendix E.2).
// The sequential baseline k_sequential (Appendix E.3) runs the same interval
// rule and root solve one event at a time per (sample, neuron).
#include "lif_common.hpp"
#include "lif_host.hpp"
#include "lif_walk.hpp"
#include "lif_reg.hpp"
#include <type_traits>

namespace lif {

// Pool of entering states: one entry (the no-reset (U, J) entering the
// sub-block) per flagged (sub-block, neuron), in per-sample slices.  The
// check pass reserves the entries (one atomic per wave) and writes them; the
// resolve pass rebuilds the sub-block's interval states from them.
constexpr uint32_t kNoSlot = 0xffffffffu;

// Mask word of a (sample, segment, neuron): the flagged sub-blocks in bits
// 0..3, the pool offset of the pair's first entry in bits 4..31.
constexpr int kMaskBits = 4;
static_assert(kSubPerSeg <= kMaskBits, "mask word layout");

// Search key of an interval whose crossing test is "reset deficit at its
// start <= crit" (crossing_data).  The deficit of the spikes so far is
// D(t) = dref e^{-(t - tref)/tm}, so at an interval that starts at t0 the
// test reads ln(crit) + t0/tm >= ln(dref) + tref/tm.  crit < 0 (never
// crosses) gives NaN, for which every comparison is false; crit = 0 gives
// -inf, which only the deficit of no spike at all (ln 0) reaches.
__device__ __forceinline__ double crossing_key(const Model& m, double crit, double t0)
{
    if (!(crit >= 0.0)) return __builtin_nan("");
    if (crit == 0.0) return -INFINITY;
    return log(crit) + t0 * m.inv_tm;
}

// The hardware logarithm ln x of a double x, and how far it may be from it: the
// rounding to float (2^-24), v_log_f32 (an ulp of log2 x), ln 2 as a float and the
// product (half an ulp each), under 1.2e-5 at the ends of the float range and
// under 1e-5 + |ln x| 2^-21 everywhere.  Past the float range it is the end of it.
__device__ __forceinline__ double log_coarse(double x) { return (double)__logf(fminf((float)x, 3.0e38f)); }
__device__ __forceinline__ double log_margin(double l) { return fma(fabs(l), 0x1p-21, 1e-5); }

// Upper bound, as a float, of the crossing keys of a sub-block's intervals from
// the largest value z of its screens (V / kappa; screen_value) and its last
// event's time: an interval's crit is at most V_lin's tangent bound minus th, so
// key <= ln(kappa z - th) + t_last / tm.  The margins cover the hardware
// logarithm, the rounding to float and the rounding of the interval states
// (the 1e-9 of th_lo).  Below the deficit's key, none of the intervals crosses.
__device__ __forceinline__ float key_bound(const Model& m, double z, double t_last)
{
    const double x = fmax(fma(m.kappa, z, -m.th), 0.0) + 1e-9 * fmax(1.0, m.th);
    if (!(x < 3.0e38)) return INFINITY;
    const double l = log_coarse(x);
    const float f = (float)(l + log_margin(l) + t_last * m.inv_tm);
    return f + fabsf(f) * 0x1p-22f;
}

// Per-sample counters (pool use, work-list length) each take their
// own 128-byte line: many waves update them with atomics, and atomics on one
// line are serialised.  The resolve pass's list counter is word kTaken of the first
// line, whose own word is only read by then.
constexpr int kCtr = 32;
constexpr int kTaken = 16;

// ---------------------------------------------------------------------------
// k_prep
// ---------------------------------------------------------------------------
// Decay record of event k (gap to the previous event, or to t = 0).
__device__ __forceinline__ Decay make_decay(const Model& m, const float* __restrict__ t, int k)
{
    double dt = (double)t[k] - (k > 0 ? (double)t[k - 1] : 0.0);
    Decay d;
    d.A = exp(-dt * m.inv_tm);
    d.D = exp(-dt * m.inv_ts);
    d.C = unit_kernel(m, dt, d.A);
    d.lk = dt * m.inv_ktm;
    return d;
}

// Decays dec[B][E_pad] (identity maps past each sample's last event, so
// that the walks run whole sub-blocks), the composed maps (A, D) of every
// segment, and the reset of status words, counters and outputs (out_t is
// filled with +inf when given: the resolve pass writes only neurons that
// fire).
__global__ __launch_bounds__(256) void k_prep(const float* __restrict__ ev_t, const int32_t* __restrict__ ev_n,
                                              int B, int E_max, int E_pad, int S, Model m, Decay* __restrict__ dec,
                                              double2* __restrict__ segm, int32_t* __restrict__ status,
                                              uint32_t* __restrict__ counters, size_t n_counters,
                                              int32_t* __restrict__ out_n, uint32_t* __restrict__ listed, size_t nn,
                                              float* __restrict__ out_t, float* __restrict__ out_i,
                                              int32_t* __restrict__ out_k, size_t n_out)
{
    const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    if (tid < LIF_STATUS_WORDS) status[tid] = 0;
    for (size_t i = tid; i < n_counters; i += stride) counters[i] = 0u;
    for (size_t i = tid; i < nn; i += stride) {
        out_n[i] = 0;
        if (listed) listed[i] = 0u;
    }
    if (out_t) {
        for (size_t i = tid; i < n_out; i += stride) {
            out_t[i] = INFINITY;
            if (out_i) out_i[i] = 0.0f;
            if (out_k) out_k[i] = 0;
        }
    }
    const size_t nev = (size_t)B * (size_t)E_pad;
    for (size_t idx = tid; idx < nev; idx += stride) {
        const int b = (int)(idx / (size_t)E_pad), k = (int)(idx % (size_t)E_pad);
        Decay d{1.0, 1.0, 0.0, 0.0};
        if (k < clamp_count(ev_n[b], E_max)) d = make_decay(m, ev_t + (size_t)b * E_max, k);
        dec[idx] = d;
    }
    if (segm) {
        for (size_t idx = tid; idx < (size_t)B * S; idx += stride) {
            const int b = (int)(idx / (size_t)S), j = (int)(idx % (size_t)S);
            const int nb = clamp_count(ev_n[b], E_max), k0 = j * kSeg;
            double2 r = make_double2(1.0, 1.0);
            if (k0 < nb) {
                const float* tt = ev_t + (size_t)b * E_max;
                const double T = (double)tt[min(k0 + kSeg, nb) - 1] - (k0 > 0 ? (double)tt[k0 - 1] : 0.0);
                r = make_double2(exp(-T * m.inv_tm), exp(-T * m.inv_ts));
            }
            segm[idx] = r;
        }
    }
}

// Optional input validation (LIF_VALIDATE).
__global__ __launch_bounds__(256) void k_validate(const float* __restrict__ ev_t, const int32_t* __restrict__ ev_src,
                                                  const int32_t* __restrict__ ev_n, int B, int E_max, int C_in,
                                                  int32_t* __restrict__ status)
{
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (size_t)B * (size_t)E_max) return;
    int b = (int)(idx / (size_t)E_max), k = (int)(idx % (size_t)E_max);
    if (k == 0 && (ev_n[b] < 0 || ev_n[b] > E_max)) atomicOr(&status[LIF_ST_FLAGS], LIF_WARN_BAD_COUNT);
    if (k >= clamp_count(ev_n[b], E_max)) return;
    float t = ev_t[idx];
    int f = 0;
    if (!isfinite(t) || t < 0.0f) f |= LIF_WARN_NONFINITE;
    if (k > 0 && !(ev_t[idx - 1] <= t)) f |= LIF_WARN_UNSORTED;
    int s = ev_src[idx];
    if (s < 0 || s >= C_in) f |= LIF_WARN_BAD_SOURCE;
    if (f) atomicOr(&status[LIF_ST_FLAGS], f);
}

// One event in eigen-coordinates: decay over the gap, then the jump.
template <int NPL>
__device__ __forceinline__ void step(double A, double D, const float (&w)[NPL], double (&U)[NPL], double (&J)[NPL])
{
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
        const double x = (double)w[i];
        U[i] = fma(A, U[i], x);
        J[i] = fma(D, J[i], x);
    }
}

// One event in eigen-coordinates: decay over the gap, then the jump.
__device__ __forceinline__ void step1(double2 ad, float w, double& U, double& J)
{
    const double x = (double)w;
    U = fma(ad.x, U, x);
    J = fma(ad.y, J, x);
}

// Walk the n events of a group starting at e0 (n = kGrp on every group but
// a sample's last).
template <int NPL>
__device__ __forceinline__ void walk_grp(const double2* __restrict__ lad, int e0, int n, const float (&w)[kGrp][NPL],
                                         double (&U)[NPL], double (&J)[NPL])
{
    if (n >= kGrp) {
#pragma unroll
        for (int j = 0; j < kGrp; ++j) {
            const double2 ad = lad[e0 + j];
            step<NPL>(ad.x, ad.y, w[j], U, J);
        }
    } else {
#pragma unroll
        for (int j = 0; j < kGrp; ++j)
            if (j < n) {
                const double2 ad = lad[e0 + j];
                step<NPL>(ad.x, ad.y, w[j], U, J);
            }
    }
}

template <int NPL>
__global__ __launch_bounds__(kWave * kWalkWaves) void k_aggregate(
    const float* __restrict__ ev_t, const int32_t* __restrict__ ev_src, const int32_t* __restrict__ ev_n, int E_max,
    int E_pad, const float* __restrict__ WT, int C_in, int N, int tiles, int S, int items, Model m,
    Decay* __restrict__ dec, double2* __restrict__ segm, double2* __restrict__ agg, int32_t* __restrict__ status,
    uint32_t* __restrict__ counters, size_t n_counters, uint32_t* __restrict__ listed, size_t nn,
    int32_t* __restrict__ out_n, float* __restrict__ out_t, float* __restrict__ out_i, int32_t* __restrict__ out_k,
    size_t n_out, int tmB)
{
    {
        // resets for the later passes: status words, per-sample counters,
        // listed flags, and the outputs (the resolve pass writes only the
        // neurons that fire: counts 0, times +inf, currents and event
        // counts 0), grid-stride over every thread
        const size_t gt = (size_t)blockIdx.x * blockDim.x + threadIdx.x, gs = (size_t)gridDim.x * blockDim.x;
        if (gt < LIF_STATUS_WORDS) status[gt] = 0;
        for (size_t i = gt; i < n_counters; i += gs) counters[i] = 0u;
        for (size_t i = gt; i < nn; i += gs) {
            listed[i] = 0u;
            if (out_n) out_n[i] = 0;
        }
        if (out_t)
            for (size_t i = gt; i < n_out; i += gs) {
                out_t[i] = INFINITY;
                if (out_i) out_i[i] = 0.0f;
                if (out_k) out_k[i] = 0;
            }
    }
    __shared__ double2 s_ad[kWalkWaves][kSeg];
    WalkCoords c;
    if (!walk_coords<NPL>(items, tiles, S, ev_n, E_max, N, c, tmB)) return;
    double2* lad = s_ad[threadIdx.x / kWave];
    // the decays of the segment's events (identity past the sample's last
    // event); the first tile's wave stores them, and the segment's composed
    // map, for the later passes
    {
        const float* tt = ev_t + (size_t)c.b * E_max;
        Decay* dd = dec + (size_t)c.b * E_pad + c.k0;
#pragma unroll
        for (int h = 0; h < kSrcRegs; ++h) {
            const int e = h * kWave + c.lane;
            Decay dk{1.0, 1.0, 0.0, 0.0};
            if (c.k0 + e < c.nb) dk = make_decay(m, tt, c.k0 + e);
            lad[e] = make_double2(dk.A, dk.D);
            if (c.tile == 0) dd[e] = dk;
        }
        if (c.tile == 0 && c.lane == 0) {
            const double T = (double)tt[c.k0 + c.cnt - 1] - (c.k0 > 0 ? (double)tt[c.k0 - 1] : 0.0);
            segm[(size_t)c.b * S + c.seg] = make_double2(exp(-T * m.inv_tm), exp(-T * m.inv_ts));
        }
    }
    const Stage st = stage_segment(c, ev_src + (size_t)c.b * E_max + c.k0, nullptr, WT, C_in, N, lad, nullptr);
    double U[NPL], J[NPL];
#pragma unroll
    for (int i = 0; i < NPL; ++i) U[i] = J[i] = 0.0;
    // Two weight buffers in alternation (no register copies): wa holds the
    // even and wb the odd groups.
    float wa[kGrp][NPL], wb[kGrp][NPL];
    load_grp<NPL>(st, 0, wa);
    for (int e0 = 0; e0 < c.cnt; e0 += 2 * kGrp) {
        load_grp<NPL>(st, e0 + kGrp, wb);
        walk_grp<NPL>(lad, e0, c.cnt - e0, wa, U, J);
        if (e0 + kGrp >= c.cnt) break;
        load_grp<NPL>(st, e0 + 2 * kGrp, wa);
        walk_grp<NPL>(lad, e0 + kGrp, c.cnt - e0 - kGrp, wb, U, J);
    }
    if (c.live) {
        const size_t row = ((size_t)c.b * S + c.seg) * N + c.n0;
#pragma unroll
        for (int i = 0; i < NPL; ++i) agg[row + i] = make_double2(U[i], J[i]);
    }
}

// Exclusive scan over segments of the Combine of Eq. affine in (U, J):
// s_in(j + 1) = M(T_j) s_in(j) + agg_j, s_in(0) = 0, where M(T_j) =
// diag(A_j, D_j) (segm).  A workgroup of kCarryWaves waves takes one
// (sample, 64-neuron tile); lanes are neurons and wave w the w-th contiguous
// range of at most kCarryBatch segments per round.  Each wave folds its range
// from the zero state (its aggregates loaded at once and kept), the range
// totals are combined across waves in LDS, and each wave walks its range
// again from its incoming state, writing the carries over the aggregates
// (each element is read before it is written, by the same wave).
constexpr int kCarryWaves = 8;
constexpr int kCarryBatch = 16;

__global__ __launch_bounds__(kWave * kCarryWaves) void k_carry(
    const int32_t* __restrict__ ev_n, int B, int E_max, int N, int tiles, int S, const double2* __restrict__ segm,
    const double2* agg, double2* carry)
{
    __shared__ double2 tot[kCarryWaves][kWave];      // range map b-part
    __shared__ double2 dec_tot[kCarryWaves];         // range map diagonal
    const int b = blockIdx.x / tiles, tile = blockIdx.x % tiles;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int n = tile * kWave + lane;
    const bool live = n < N;
    const int nc = live ? n : N - 1;
    const int nb = clamp_count(ev_n[b], E_max);
    const int Sb = (nb + kSeg - 1) / kSeg;
    double U = 0.0, J = 0.0;                         // state entering the current round
    for (int r0 = 0; r0 < Sb; r0 += kCarryWaves * kCarryBatch) {
        const int per = min(kCarryBatch, (Sb - r0 + kCarryWaves - 1) / kCarryWaves);
        const int j_lo = min(r0 + wave * per, Sb), j_hi = min(j_lo + per, Sb);
        double2 a[kCarryBatch], M[kCarryBatch];
#pragma unroll
        for (int j = 0; j < kCarryBatch; ++j) {
            const int jj = min(j_lo + j, Sb - 1);
            a[j] = agg[((size_t)b * S + jj) * N + nc];
            M[j] = segm[(size_t)b * S + jj];
        }
        // fold the range from zero
        double fU = 0.0, fJ = 0.0, pA = 1.0, pD = 1.0;
#pragma unroll
        for (int j = 0; j < kCarryBatch; ++j) {
            if (j_lo + j < j_hi) {
                fU = fma(M[j].x, fU, a[j].x);
                fJ = fma(M[j].y, fJ, a[j].y);
                pA *= M[j].x;
                pD *= M[j].y;
            }
        }
        tot[wave][lane] = make_double2(fU, fJ);
        if (lane == 0) dec_tot[wave] = make_double2(pA, pD);
        __syncthreads();
        // incoming state of this wave's range: the earlier ranges applied in order
        double iU = U, iJ = J;
        for (int w = 0; w < wave; ++w) {
            const double2 g = tot[w][lane], gd = dec_tot[w];
            iU = fma(gd.x, iU, g.x);
            iJ = fma(gd.y, iJ, g.y);
        }
        // state after the whole round (for the next round)
        for (int w = 0; w < kCarryWaves; ++w) {
            const double2 g = tot[w][lane], gd = dec_tot[w];
            U = fma(gd.x, U, g.x);
            J = fma(gd.y, J, g.y);
        }
        __syncthreads();
        // walk the range again, writing the carry entering each segment
#pragma unroll
        for (int j = 0; j < kCarryBatch; ++j) {
            if (j_lo + j < j_hi) {
                if (live) carry[((size_t)b * S + j_lo + j) * N + n] = make_double2(iU, iJ);
                iU = fma(M[j].x, iU, a[j].x);
                iJ = fma(M[j].y, iJ, a[j].y);
            }
        }
    }
}

// Screen of one group of intervals on the walk itself: z takes the largest
// screen_value.  (A coarse bound per group first, with a second walk of the
// groups that pass it, costs 6 instead of 8 float64 operations per
// neuron-event, but of a layer that fires nearly every group passes for some
// lane: VALU-bound at 21 instructions, 2.44 ms at 32768 -> 2048, B = 16, 100 k
// events.)
template <int NPL>
__device__ __forceinline__ void screen_grp(const Model& m, const double2* __restrict__ lad,
                                           const double* __restrict__ llk, int e0, int n,
                                           const float (&w)[kGrp][NPL], double (&U)[NPL], double (&J)[NPL],
                                           double (&z)[NPL])
{
    auto take = [&](int j) {
        const double lk = llk[e0 + j];
        const double2 ad = lad[e0 + j];
#pragma unroll
        for (int i = 0; i < NPL; ++i) z[i] = fmax(z[i], screen_value(m, U[i], J[i], lk));
        step<NPL>(ad.x, ad.y, w[j], U, J);
    };
    if (n >= kGrp) {
#pragma unroll
        for (int j = 0; j < kGrp; ++j) take(j);
    } else {
#pragma unroll
        for (int j = 0; j < kGrp; ++j)
            if (j < n) take(j);
    }
}

// Re-walk from the carried no-reset state with the no-crossing screen on
// every interval: the interval before each event of the sub-block and, in
// the sub-block holding the sample's last event, the open interval after it
// (up to t_end).  A flagged (sub-block, neuron) sets a bit in the neuron's
// sub-block mask of the segment; the entering state (U, J) of every
// sub-block is kept in LDS until the pool entries are reserved.  At the end
// of the item the wave reserves entries for all its flagged sub-blocks with
// one atomic on the sample's pool counter, in lane order, so that the
// entries of one (segment, neuron) are consecutive: the mask word of the pair
// holds the sub-block bits and the pool offset of its first entry, and the
// entry of a flagged sub-block is that offset plus the number of flagged
// sub-blocks before it (none past the pool capacity: the resolve pass then
// rebuilds that sub-block's entering state from the segment's carried
// state).  The wave writes the entering states; the first segment to flag a
// neuron appends it to the sample's work list.
template <bool kBounds>
__global__ __launch_bounds__(kWave * kWalkWaves) void k_check(
    const float* __restrict__ ev_t, const int32_t* __restrict__ ev_src, const int32_t* __restrict__ ev_n, int E_max,
    int E_pad, const float* __restrict__ WT, int C_in, int N, int tiles, int S, int items, Model m,
    const Decay* __restrict__ dec, double2* carry, uint32_t* __restrict__ mask, double2* __restrict__ pool,
    uint32_t* __restrict__ pool_count, uint32_t pool_cap, uint32_t* __restrict__ listed,
    uint32_t* __restrict__ work, uint32_t* __restrict__ nwork)
// kBounds: key bounds are stored for k_resolve.  carry: a pair whose flagged
// sub-blocks all have pool entries no longer needs its carried state (only its
// own wave reads it before), and the four sub-blocks' bounds (key_bound; -inf
// when not flagged) take its place.
// work: per-sample lists of the neurons with flagged sub-blocks (capacity N
// each); nwork: per-sample list lengths.
{
    constexpr int NPL = 1;                  // one neuron per lane (occupancy)
    __shared__ double2 s_ad[kWalkWaves][kSeg];
    __shared__ double s_lk[kWalkWaves][kSeg];
    __shared__ double2 s_ent[kWalkWaves][kSubPerSeg][kWave];   // entering state of each sub-block
    __shared__ float s_kb[kBounds ? kWalkWaves : 1][kSubPerSeg][kWave];   // and its key bound
    WalkCoords c;
    if (!walk_coords<NPL>(items, tiles, S, ev_n, E_max, N, c)) return;
    const int lane = c.lane;
    const int wv = threadIdx.x / kWave;
    double2* lad = s_ad[wv];
    double* llk = s_lk[wv];
    const Stage st = stage_segment(c, ev_src + (size_t)c.b * E_max + c.k0, dec + (size_t)c.b * E_pad + c.k0, WT,
                                   C_in, N, lad, llk);
    const size_t row = ((size_t)c.b * S + c.seg) * N + c.n0;
    const unsigned long long below = (1ull << lane) - 1ull;
    double U[NPL], J[NPL];
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
        const double2 s0 = carry[row + i];
        U[i] = s0.x;
        J[i] = s0.y;
    }
    uint32_t msk[NPL];
#pragma unroll
    for (int i = 0; i < NPL; ++i) msk[i] = 0u;
    // The open interval after the sample's last event, up to t_end.
    const bool last_seg = c.k0 + c.cnt == c.nb;
    const double open_lk = last_seg ? (m.t_end - (double)ev_t[(size_t)c.b * E_max + c.nb - 1]) * m.inv_ktm : 0.0;
    // Two weight buffers in alternation: wa holds the first and wb the second
    // group of each sub-block.
    float wa[kGrp][NPL], wb[kGrp][NPL];
    load_grp<NPL>(st, 0, wa);
    for (int q = 0; q < kSubPerSeg; ++q) {
        const int q0 = q * kSub;
        if constexpr (kBounds) s_kb[wv][q][lane] = -INFINITY;
        if (q0 >= c.cnt) {
            if constexpr (kBounds) continue;
            break;
        }
        double U0[NPL], J0[NPL], z[NPL];
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            U0[i] = U[i];
            J0[i] = J[i];
            z[i] = -INFINITY;
        }
        load_grp<NPL>(st, q0 + kGrp, wb);
        screen_grp<NPL>(m, lad, llk, q0, c.cnt - q0, wa, U, J, z);
        if (q0 + kGrp < c.cnt) {
            load_grp<NPL>(st, q0 + kSub, wa);
            screen_grp<NPL>(m, lad, llk, q0 + kGrp, c.cnt - q0 - kGrp, wb, U, J, z);
        }
        if (last_seg && q0 + kSub >= c.cnt && open_lk > 0.0) {
#pragma unroll
            for (int i = 0; i < NPL; ++i)
                z[i] = fmax(z[i], J[i] > m.th ? fma(J[i] - m.th, open_lk, U[i] - J[i]) : U[i] - J[i]);
        }
        s_ent[wv][q][lane] = make_double2(U0[0], J0[0]);
        const bool flag = c.live && z[0] >= m.thk_lo;
        if (flag) msk[0] |= 1u << q;
        if constexpr (kBounds) {
            if (__ballot(flag)) {
                const double tl = (double)ev_t[(size_t)c.b * E_max + c.k0 + min(q0 + kSub, c.cnt) - 1];
                if (flag) s_kb[wv][q][lane] = key_bound(m, z[0], tl);
            }
        }
    }
    // Pool entries of the wave's flagged sub-blocks: one reservation, slots
    // in lane order (exclusive prefix sum of the per-lane counts).
    {
        uint32_t mine = 0;
#pragma unroll
        for (int i = 0; i < NPL; ++i) mine += (uint32_t)__popc(msk[i]);
        uint32_t ex = mine;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t v = (uint32_t)__shfl_up((int)ex, off, kWave);
            if (lane >= off) ex += v;
        }
        const uint32_t total = (uint32_t)__shfl((int)ex, kWave - 1, kWave);
        ex -= mine;
        uint32_t base = 0;
        if (total) {
            if (lane == 0) base = atomicAdd(&pool_count[(size_t)c.b * kCtr], total);
            base = (uint32_t)__shfl((int)base, 0, kWave) + ex;
        }
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            if (c.live) mask[row + i] = msk[i] | (base << kMaskBits);
            if constexpr (kBounds) {
                if (c.live && msk[i] && base + (uint32_t)__popc(msk[i]) <= pool_cap)
                    *reinterpret_cast<float4*>(&carry[row + i]) =
                        make_float4(s_kb[wv][0][lane], s_kb[wv][1][lane], s_kb[wv][2][lane], s_kb[wv][3][lane]);
            }
            for (uint32_t mm = msk[i]; mm; mm &= mm - 1u) {
                if (base < pool_cap) pool[(size_t)c.b * pool_cap + base] = s_ent[wv][__builtin_ctz(mm)][lane];
                ++base;
            }
        }
    }
    // Work list of the sample: the first segment to flag a neuron appends it
    // (one OR per flagged neuron, one counter update per wave).
    bool want[NPL], first[NPL];
    unsigned long long wm = 0ull;
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
        want[i] = c.live && msk[i] != 0u;
        wm |= __ballot(want[i]);
    }
    if (wm) {
        unsigned long long fmk[NPL];
        uint32_t tot = 0;
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            first[i] = false;
            if (want[i]) first[i] = atomicOr(&listed[(size_t)c.b * N + c.n0 + i], 1u) == 0u;
            fmk[i] = __ballot(first[i]);
            tot += (uint32_t)__popcll(fmk[i]);
        }
        if (tot) {
            uint32_t wbase = 0;
            if (lane == 0) wbase = atomicAdd(&nwork[(size_t)c.b * kCtr], tot);
            wbase = (uint32_t)__shfl((int)wbase, 0, kWave);
            uint32_t before = 0;
#pragma unroll
            for (int i = 0; i < NPL; ++i) {
                if (first[i])
                    work[(size_t)c.b * N + wbase + before + (uint32_t)__popcll(fmk[i] & below)] =
                        (uint32_t)((size_t)c.b * N + c.n0 + i);
                before += (uint32_t)__popcll(fmk[i]);
            }
        }
    }
}
// Crossing data of one interval of length L that starts in the no-reset
// state (V0, I0) and ends with V1 (A, D: its decays): the interval reaches
// the threshold iff the reset deficit at its start is <= crit (crit < 0:
// never), by interval_max's test D a <= g; the spike then lies in
// (lo, hi] with F(hi) = fhi - deficit.  Zero-length intervals never cross.
// Floating-point contraction is off here and in interval_max, so every
// inlined copy performs the same IEEE operations.
__device__ __forceinline__ void crossing_data(const Model& m, double V0, double I0, double V1, double L, double A,
                                              double D, double& crit, double& hi, double& fhi)
{
#pragma clang fp contract(off)
    crit = -1.0;
    hi = 0.0;
    fhi = -INFINITY;
    if (!(L > 0.0)) return;
    const IntervalMax im = interval_max(m, V0, I0, V1, L, A, D);
    if (im.g >= 0.0) crit = im.a > 0.0 ? im.g / im.a : INFINITY;
    hi = im.hi;
    fhi = im.Fhi;
}

// Crossing data of the open interval (t_last, t_end] after a sample's last
// event, from the state (V, I) right after it.
__device__ __forceinline__ void open_interval_data(const Model& m, double V, double I, double L, double& crit,
                                                   double& hi, double& fhi)
{
    double A = 0.0, D = 0.0, V1 = 0.0;
    if (!isinf(L)) {
        A = exp(-L * m.inv_tm);
        D = exp(-L * m.inv_ts);
        V1 = V * A + unit_kernel(m, L, A) * I;
    }
    crossing_data(m, V, I, V1, L, A, D, crit, hi, fhi);
}

__device__ __forceinline__ int rl_int(int v, int l) { return __builtin_amdgcn_readlane(v, l); }

__device__ __forceinline__ double rl_double(double v, int l)
{
    unsigned long long u = (unsigned long long)__double_as_longlong(v);
    unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, l);
    unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Flagged sub-blocks of the whole call, by every wave.
__device__ __forceinline__ unsigned long long flagged_total(const uint32_t* __restrict__ pool_count, int B)
{
    unsigned long long f = 0;
    for (int b = (int)threadIdx.x % kWave; b < B; b += kWave) f += pool_count[(size_t)b * kCtr];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) f += __shfl_xor(f, off, kWave);
    return f;
}

// Status words fixed once the check pass has run, by the grid's last wave (the
// only writer of these words in the call): events consumed, flagged sub-blocks,
// sub-blocks past the pool's capacity.
__device__ __forceinline__ void resolve_status(const int32_t* __restrict__ ev_n, int B, int E_max,
                                               const uint32_t* __restrict__ pool_count, uint32_t pool_cap,
                                               int32_t* __restrict__ status)
{
    const int lane = (int)threadIdx.x % kWave;
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x >= blockDim.x - kWave) {
        unsigned long long ev = 0, fl = 0, fb = 0;
        for (int bb = lane; bb < B; bb += kWave) {
            ev += (unsigned long long)clamp_count(ev_n[bb], E_max);
            const uint32_t pc = pool_count[(size_t)bb * kCtr];
            fl += pc;
            fb += pc > pool_cap ? pc - pool_cap : 0u;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            ev += __shfl_xor(ev, off, kWave);
            fl += __shfl_xor(fl, off, kWave);
            fb += __shfl_xor(fb, off, kWave);
        }
        if (lane == 0) {
            auto sat = [](unsigned long long x) { return (int32_t)(x > 0x7fffffffull ? 0x7fffffffull : x); };
            status[LIF_ST_EVENTS] = sat(ev);
            status[LIF_ST_CAND_BLOCKS] = sat(fl);
            status[LIF_ST_WALKED_BLOCKS] = sat(fl);
            status[LIF_ST_POOL_FALLBACK] = sat(fb);
        }
    }
}

// ---------------------------------------------------------------------------
// Resolve pass: one wave per neuron that has flagged sub-blocks (the work lists
// of the check pass).  Intervals outside flagged sub-blocks provably hold no
// spike.  The flagged sub-blocks are taken in time order:
//   * Candidate list: per chunk of kChunkEv events, the sub-block masks (two
//     segments per lane) are compacted into a time-ordered list in LDS with
//     one wave prefix sum, with the pool slot and key bound of every
//     candidate; candidates whose bound lies below the key K of the current
//     reset deficit cannot hold a crossing and are left out.
//   * Windows: the next kWinCand candidates whose bound still reaches K (one
//     ballot per 64), one interval per lane.  The loads of the window after
//     the one at work are in flight.
//   * Interval i crosses iff key_i >= K (crossing_key), so one ballot finds
//     the window's earliest crossing.  Its spike time is solved wave-uniform,
//     the deficit and K are raised, and the search resumes at the same
//     interval (a second spike in it, App. E.2 restart).
//   * The open interval after the sample's last event follows the window
//     that holds the sample's last sub-block.
//   * Spikes are buffered in LDS and written out kWave at a time.
// Most flagged sub-blocks lie in the wake of a spike, where the no-reset V is
// above threshold but the true one is not: the key bounds leave a few windows
// per spike of them.
// ---------------------------------------------------------------------------
constexpr int kChunkEv = 8192;                   // events per chunk of the candidate list
constexpr int kChunkSeg = kChunkEv / kSeg;       // segments per chunk
constexpr int kSegPerLane = kChunkSeg / kWave;   // mask words per lane
static_assert(kChunkSeg % kWave == 0 && kSubPerSeg <= 8, "chunk layout; 3-bit sub-block field of a candidate");
constexpr int kCandCap = kChunkSeg * kSubPerSeg; // candidates of one chunk
constexpr int kWinCand = kWave / kSub;           // candidates per window (one interval per lane)
constexpr int kResolveWaves = 4;                 // independent waves of a workgroup

// The line between the two passes (see where they are launched).
constexpr unsigned long long kRingMost = 65536;  // flagged sub-blocks of a call
constexpr size_t kRingDense = (size_t)1 << 22;   // sub-blocks of a call, flagged or not

struct ResolveLds {
    uint32_t cand[kCandCap];                     // (segment in chunk << 3) | sub-block
    uint32_t slot[kCandCap];                     // pool slot of each candidate (kNoSlot: none)
    float kub[kCandCap];                         // key bound
    double sp_t0[kWave], sp_y[kWave];            // spike buffer: interval start, e^{-u/tm},
    float si[kWave];                             // I at the spike,
    int32_t sk[kWave];                           // events consumed before the spike
};

// Entering no-reset state of sub-block kq0 (of the segment whose first
// event is k0) from the segment's carried state (U, J), for a sub-block past
// the pool's capacity, by the whole wave: lane e loads event k0 + e's weight
// and decays, and every lane follows the same serial walk over events k0 ..
// kq0 - 1 with those values broadcast (the check pass's operations, so the
// state has the bits a pool entry would hold).  Wave-uniform result.
__device__ double2 rebuild_entry(double U, double J, int k0, int kq0, int n, int N, int C_in,
                                 const int32_t* __restrict__ src, const Decay* __restrict__ d,
                                 const float* __restrict__ WT)
{
    const int lane = (int)threadIdx.x % kWave;
    const int ne = kq0 - k0;
    float we = 0.0f;
    double A = 1.0, D = 1.0;
    if (lane < ne) {
        we = WT[(size_t)clamp_src(src[k0 + lane], C_in) * (size_t)N + n];
        const Decay dk = d[k0 + lane];
        A = dk.A;
        D = dk.D;
    }
    for (int e = 0; e < ne; ++e) {
        const float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, we), e));
        step1(make_double2(rl_double(A, e), rl_double(D, e)), w, U, J);
    }
    return make_double2(U, J);
}

// Lane E's value of the calling lane's row of 16 lanes (DPP row broadcast).
template <int E>
__device__ __forceinline__ int row_bcast(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x150 + E, 0xf, 0xf, false);
}

template <int E>
__device__ __forceinline__ double row_bcast(double v)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)row_bcast<E>((int)(unsigned)u), hi = (unsigned)row_bcast<E>((int)(unsigned)(u >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The value of lane j - Dist of the calling lane's row of 16 lanes (DPP
// row shift); lanes j < Dist get fill.
template <int Dist>
__device__ __forceinline__ double row_shr(double v, double fill)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const unsigned long long f = (unsigned long long)__double_as_longlong(fill);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)f, (int)(unsigned)u, 0x110 + Dist, 0xf,
                                                              0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)(f >> 32), (int)(unsigned)(u >> 32),
                                                              0x110 + Dist, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// One step of the row's inclusive scan of event maps in (U, J): lane j's map
// (a, b) (x -> a x + b) composed after the map of lane j - Dist.
template <int Dist>
__device__ __forceinline__ void scan_step(double& aU, double& bU, double& aJ, double& bJ)
{
    const double paU = row_shr<Dist>(aU, 1.0), pbU = row_shr<Dist>(bU, 0.0);
    const double paJ = row_shr<Dist>(aJ, 1.0), pbJ = row_shr<Dist>(bJ, 0.0);
    bU = fma(aU, pbU, bU);
    aU *= paU;
    bJ = fma(aJ, pbJ, bJ);
    aJ *= paJ;
}

// The no-reset states of a sub-block's intervals from its entering state u0
// (one row of 16 lanes, lane j holding event j of the sub-block with decays
// (A, D) and weight w): the maps of events 0 .. j composed by a log-depth
// scan within the row (App. B: the maps form a semigroup), so lane j gets
// the state at the start of its interval (after event j - 1) and after its
// event.
__device__ __forceinline__ void row_states(double2 u0, double A, double D, float w, double& U0, double& J0,
                                           double& U1, double& J1)
{
    double aU = A, bU = (double)w, aJ = D, bJ = (double)w;
    scan_step<1>(aU, bU, aJ, bJ);
    scan_step<2>(aU, bU, aJ, bJ);
    scan_step<4>(aU, bU, aJ, bJ);
    scan_step<8>(aU, bU, aJ, bJ);
    U1 = fma(aU, u0.x, bU);
    J1 = fma(aJ, u0.y, bJ);
    U0 = fma(row_shr<1>(aU, 1.0), u0.x, row_shr<1>(bU, 0.0));
    J0 = fma(row_shr<1>(aJ, 1.0), u0.y, row_shr<1>(bJ, 0.0));
}

// A value <= e^x for the staging screen: the float exponential (relative
// error below 2^-16 for |x| <= 88, argument rounding included) scaled by
// 1 - 2^-10; 0 below the float range and at most FLT_MAX above it (beyond
// it the deficit exceeds any state the screen could pass).
__device__ __forceinline__ double exp_lower(double x)
{
    return (1.0 - 0x1p-10) * (double)fminf(__expf((float)x), 3.0e38f);
}

// A window's loads: lane l takes interval j = l % kSub of candidate c (of lanes
// l / kSub; none when c < 0): its closing event's source, decays and times and the
// candidate's entering state.
struct WinIn {
    int k, sc;
    bool ok;
    uint32_t cw, slot;
    double A, D;
    float ta, tb;
    double2 u0;
};

__device__ __forceinline__ WinIn win_load(const ResolveLds& sh, int c, int seg0, int nb, const float* __restrict__ tt,
                                          const int32_t* __restrict__ src, const Decay* __restrict__ d,
                                          const double2* __restrict__ pool)
{
    const int j = (int)threadIdx.x % kSub, cc = max(c, 0);
    WinIn in;
    in.cw = sh.cand[cc];
    in.slot = sh.slot[cc];
    const int k = (seg0 + (int)(in.cw >> 3)) * kSeg + (int)(in.cw & 7u) * kSub + j;
    in.ok = c >= 0 && k < nb;
    in.k = min(k, nb - 1);
    in.sc = src[in.k];
    const double2 ad = *reinterpret_cast<const double2*>(&d[in.k]);       // (A, D)
    in.A = ad.x;
    in.D = ad.y;
    in.ta = tt[max(in.k - 1, 0)];
    in.tb = tt[in.k];
    in.u0 = pool[in.slot != kNoSlot ? in.slot : 0u];    // the pool holds at least one entry
    return in;
}

// Wave-uniform resolve state of one neuron: the reset deficit of the spikes
// so far is D(t) = dref e^{-(t - tref)/tm} for t after the latest spike (dref =
// 0: none yet), and K <= ln(dref) + tref/tm its key (a lower bound, two log_margin
// from it at most while dref is a float, for the candidates' key bounds).
struct Chain {
    int ns;              // spikes so far
    double dref, tref, K;
};

// Spikes [from, to) from the LDS buffer to the outputs (coalesced); the
// spike times t0 - tm ln y are taken here, 64 at a time, off the chain.
__device__ __forceinline__ void flush_spikes(ResolveLds& sh, const Model& m, int from, int to, float* __restrict__ st,
                                             float* __restrict__ si, int32_t* __restrict__ sk)
{
    const int lane = (int)threadIdx.x % kWave;
    wave_lds_sync();
    if (from + lane < to) {
        const int q = (from + lane) % kWave;
        st[from + lane] = (float)(sh.sp_t0[q] - m.tm * log(sh.sp_y[q]));
        if (si) si[from + lane] = sh.si[q];
        if (sk) sk[from + lane] = sh.sk[q];
    }
    wave_lds_sync();
}

// Offset u of the spike in an interval of length L from the no-reset state
// (V0, I0) with deficit Dk at its start, after y = ylo when the latest spike
// lies in it too (V1, A, D: its end state and decays); all wave-uniform.
// Returns y = e^{-u/tm} and e^{-u r} (polynomial solve when tau_m / tau_s is an
// integer plus one, else bracketed Newton on the interval's closed-form
// maximum).
template <int PI>
__device__ __forceinline__ double spike_y(const Model& m, double V0, double I0, double V1, double L, double A, double D,
                                          double Dk, double ylo, double& E2)
{
    const double kI = m.kappa * I0, c0v = V0 - Dk + kI;
    double y = 0.0;
    if constexpr (PI > 0) {
        if (root_poly<PI>(m, c0v, kI, ylo, y)) {
            E2 = ipow<PI>(y);
            return y;
        }
    }
    const IntervalMax im = interval_max(m, V0, I0, V1, L, A, D);
    double E1;
    root_h(m, c0v, kI, 0.0, V0 - m.th - Dk, im.hi, im.Fhi - Dk, &E1, &E2, nullptr);
    return rcp_refined(E1);
}

// One neuron by one wave; returns its spike count.
template <int PI>
__device__ int resolve_neuron(ResolveLds& sh, int b, int n, const float* __restrict__ ev_t,
                              const int32_t* __restrict__ ev_src, const int32_t* __restrict__ ev_n, int E_max,
                              const float* __restrict__ WT, int C_in, int N, int E_pad, int S, const Model& m,
                              const Decay* __restrict__ dec, const double2* __restrict__ carry,
                              const uint32_t* __restrict__ mask, uint32_t pool_cap, const double2* __restrict__ pool,
                              float* __restrict__ out_t, int32_t* __restrict__ out_n, float* __restrict__ out_i,
                              int32_t* __restrict__ out_k)
{
    const int lane = (int)threadIdx.x % kWave;
    const size_t row0 = (size_t)b * S * N + n;            // mask and carry of segment j: row0 + j N
    // a chunk's mask words (lane l: segments kSegPerLane l + h of it) are loaded
    // two chunks ahead and its key bounds one chunk ahead; words past the
    // sample's segments are dropped when used
    const int nb = __builtin_amdgcn_readfirstlane(clamp_count(ev_n[b], E_max));
    const int Sb = (nb + kSeg - 1) / kSeg;
    uint32_t mw[kSegPerLane], m1[kSegPerLane];
    float4 kb[kSegPerLane];
    auto load_mask = [&](int seg0, uint32_t (&w)[kSegPerLane]) {
#pragma unroll
        for (int h = 0; h < kSegPerLane; ++h) {
            const int sj = seg0 + lane * kSegPerLane + h;
            w[h] = sj < S ? mask[row0 + (size_t)sj * N] : 0u;
        }
    };
    auto flagged = [&](int seg0, uint32_t w, int h) {
        return seg0 + lane * kSegPerLane + h < Sb ? w & ((1u << kSubPerSeg) - 1u) : 0u;
    };
    // (+inf where a pair's sub-blocks do not all have pool entries)
    auto load_bounds = [&](int seg0, const uint32_t (&w)[kSegPerLane]) {
#pragma unroll
        for (int h = 0; h < kSegPerLane; ++h) {
            const uint32_t mv = flagged(seg0, w[h], h);
            kb[h] = make_float4(INFINITY, INFINITY, INFINITY, INFINITY);
            if (mv && (w[h] >> kMaskBits) + (uint32_t)__popc(mv) <= pool_cap)
                kb[h] = *reinterpret_cast<const float4*>(
                    &carry[row0 + (size_t)(seg0 + lane * kSegPerLane + h) * N]);
        }
    };
    load_mask(0, mw);
    load_mask(kChunkSeg, m1);
    load_bounds(0, mw);
    const float* tt = ev_t + (size_t)b * E_max;
    const int32_t* src = ev_src + (size_t)b * E_max;
    const Decay* d = dec + (size_t)b * E_pad;
    const size_t idx = (size_t)b * N + n;
    float* st = out_t + idx * (size_t)m.s_max;
    float* si = out_i ? out_i + idx * (size_t)m.s_max : nullptr;
    int32_t* sk = out_k ? out_k + idx * (size_t)m.s_max : nullptr;
    Chain ch{0, 0.0, 0.0, -INFINITY};
    bool more = true;                                     // false at s_max
    for (int seg0 = 0; seg0 < Sb && more; seg0 += kChunkSeg) {
        // ---- this chunk's flagged sub-blocks as a time-ordered list.  Before
        // the first spike every one of them is a candidate, and neither the
        // list nor its first window waits for the bounds.
        const bool all = ch.ns == 0;
        uint32_t keep[kSegPerLane];
        int pc = 0;
#pragma unroll
        for (int h = 0; h < kSegPerLane; ++h) {
            keep[h] = flagged(seg0, mw[h], h);
            if (!all) {
                const float k4[4] = {kb[h].x, kb[h].y, kb[h].z, kb[h].w};
#pragma unroll
                for (int q = 0; q < kSubPerSeg; ++q)
                    if (!((double)k4[q] >= ch.K)) keep[h] &= ~(1u << q);
            }
            pc += __popc(keep[h]);
        }
        int ex = pc;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int v = __shfl_up(ex, off, kWave);
            if (lane >= off) ex += v;
        }
        const int tot = rl_int(ex, kWave - 1);
        const int o0 = ex - pc;
        {
            int o = o0;
#pragma unroll
            for (int h = 0; h < kSegPerLane; ++h) {
                const uint32_t mv = flagged(seg0, mw[h], h), rel = mw[h] >> kMaskBits;
#pragma unroll
                for (int q = 0; q < kSubPerSeg; ++q) {
                    if (keep[h] & (1u << q)) {
                        const uint32_t r = rel + (uint32_t)__popc(mv & ((1u << q) - 1u));
                        sh.cand[o] = ((uint32_t)(lane * kSegPerLane + h) << 3) | (uint32_t)q;
                        sh.slot[o] = r < pool_cap ? (uint32_t)b * pool_cap + r : kNoSlot;
                        ++o;
                    }
                }
            }
        }
        wave_lds_sync();
        // the lane's candidate of the next window at or after `from` whose
        // bound reaches K (-1: none), the window's size in wn; moves `from`
        // past it
        int from = 0, wn = 0;
        auto select = [&](double K) {
            int mine = -1;
            wn = 0;
            while (from < tot && wn < kWinCand) {
                const int i = from + lane;
                unsigned long long hit = __ballot(i < tot && (double)sh.kub[min(i, tot - 1)] >= K);
                int last = from + kWave;
                while (hit && wn < kWinCand) {
                    const int f = __builtin_ctzll(hit);
                    if (lane / kSub == wn) mine = from + f;
                    ++wn;
                    hit &= hit - 1ull;
                    if (wn == kWinCand) last = from + f + 1;
                }
                from = last;
            }
            return mine;
        };
        auto load_wt = [&](const WinIn& in) { return WT[(size_t)clamp_src(in.sc, C_in) * (size_t)N + n]; };
        // the first window: the first kWinCand candidates (all of the list
        // reach K)
        wn = min(tot, kWinCand);
        from = wn;
        int c = lane / kSub < wn ? lane / kSub : -1;
        WinIn in{};
        float wv = 0.0f;
        if (wn > 0) in = win_load(sh, c, seg0, nb, tt, src, d, pool);
        {
            int o = o0;
#pragma unroll
            for (int h = 0; h < kSegPerLane; ++h) {
                const float k4[4] = {kb[h].x, kb[h].y, kb[h].z, kb[h].w};
#pragma unroll
                for (int q = 0; q < kSubPerSeg; ++q)
                    if (keep[h] & (1u << q)) sh.kub[o++] = k4[q];
            }
        }
        wave_lds_sync();
        if (wn > 0) wv = load_wt(in);
        uint32_t m2[kSegPerLane];
        load_mask(seg0 + 2 * kChunkSeg, m2);
        load_bounds(seg0 + kChunkSeg, m1);
        while (wn > 0) {
            // the next window, loaded while this one is at work, on the
            // expectation of a spike in this one: at its first interval's
            // start or later, so the deficit's key will be at least Kp
            const int from_c = from, ns_c = ch.ns;
            const double tf = (double)__builtin_bit_cast(
                float, rl_int(__builtin_bit_cast(int, in.k > 0 ? in.ta : 0.0f), 0));
            const double Dp = fma(ch.dref, exp_lower(-(tf - ch.tref) * m.inv_tm), m.dth);
            const double lp = log_coarse(Dp), Kp = fmax(ch.K, lp - log_margin(lp) + tf * m.inv_tm);
            int c_n = select(Kp);
            WinIn nx = in;
            float wvn = 0.0f;
            if (wn > 0) nx = win_load(sh, c_n, seg0, nb, tt, src, d, pool);
            // ---- the window: interval states, keys, crossings
            if (__ballot(c >= 0 && (double)sh.kub[max(c, 0)] >= ch.K)) {
                double2 u0 = in.u0;
                unsigned long long lost = __ballot(c >= 0 && in.slot == kNoSlot);
                while (lost) {
                    const int l = __builtin_ctzll(lost);
                    const uint32_t cx = (uint32_t)rl_int((int)in.cw, l);
                    const int seg = seg0 + (int)(cx >> 3);
                    const double2 cs = carry[row0 + (size_t)seg * N];
                    const double2 e = rebuild_entry(cs.x, cs.y, seg * kSeg, seg * kSeg + (int)(cx & 7u) * kSub, n, N,
                                                    C_in, src, d, WT);
                    if (lane / kSub == l / kSub) u0 = e;
                    lost &= ~(0xffffull << (l / kSub * kSub));
                }
                double U0, J0, U, J;
                row_states(u0, in.A, in.D, wv, U0, J0, U, J);
                double V0 = v_of(m, U0, J0), I0 = J0, V1 = v_of(m, U, J), A = in.A, D = in.D;
                float t0f = in.k > 0 ? in.ta : 0.0f;
                double L = (double)in.tb - (double)t0f;
                bool ok = in.ok && L > 0.0;
                int kev = in.k;
                const unsigned long long end = __ballot(in.ok && in.k == nb - 1);
                if (wn > 0) wvn = load_wt(nx);
                // the window's intervals, then (after the sample's last
                // event) the open interval, on lane 0
#pragma unroll 1
                for (int open = 0; open < 2; ++open) {
                    if (open) {
                        if (!end || !more) break;
                        const int l = __builtin_ctzll(end);
                        V0 = rl_double(V1, l);
                        I0 = rl_double(J, l);
                        t0f = __builtin_bit_cast(float, rl_int(__builtin_bit_cast(int, in.tb), l));
                        L = m.t_end - (double)t0f;
                        A = D = V1 = 0.0;
                        if (!isinf(L)) {
                            A = exp(-L * m.inv_tm);
                            D = exp(-L * m.inv_ts);
                            V1 = V0 * A + unit_kernel(m, L, A) * I0;
                        }
                        ok = lane == 0 && L > 0.0;
                        kev = nb;
                    }
                    // the deficit at the interval's start, and the no-crossing
                    // screen of the true state
                    const double t0 = (double)t0f;
                    double x = exp(-(t0 - ch.tref) * m.inv_tm), Dl = ch.dref * x;
                    ok = ok && (V0 - Dl) + (I0 > m.th ? (I0 - m.th) * (L * m.inv_tm) : 0.0) >= m.th_lo;
                    if (__ballot(ok) == 0ull) continue;
                    // crossing iff Dl a <= g (interval_max)
                    double g = V1 - m.th, a = A;
                    const bool inner = I0 > m.th && I0 * D < m.th;
                    if (__ballot(ok && inner)) {
                        const double gi = V0 + m.kappa * I0 - m.th_1k * exp(m.ts_tm * log(I0 * m.inv_th));
                        g = inner ? gi : g;
                        a = inner ? 1.0 : a;
                    }
                    int at = 0;
                    double ylo = 1.0;
                    for (;;) {
                        const unsigned long long cm = __ballot(lane >= at && ok && Dl * a <= g);
                        if (cm == 0ull) break;
                        const int f = __builtin_ctzll(cm);
                        if (f != at) ylo = 1.0;
                        at = f;
                        const double Is = rl_double(I0, at), ts0 = (double)__builtin_bit_cast(
                                                                 float, rl_int(__builtin_bit_cast(int, t0f), at));
                        const double Dk = rl_double(Dl, at);
                        double E2;
                        const double y = spike_y<PI>(m, rl_double(V0, at), Is, rl_double(V1, at), rl_double(L, at),
                                                     rl_double(A, at), rl_double(D, at), Dk, ylo, E2);
                        if (lane == 0) {
                            const int q = ch.ns % kWave;
                            sh.sp_t0[q] = ts0;
                            sh.sp_y[q] = y;
                            sh.si[q] = (float)(Is * (E2 * y));
                            sh.sk[q] = rl_int(kev, at);
                        }
                        // the deficit raised by dth e^{u/tm} in the interval's
                        // frame
                        const double xa = rl_double(x, at);
                        if (ch.ns > 0 && xa > 1e-30) {
                            ch.dref = fma(m.dth, rcp_refined(y * xa), ch.dref);
                        } else {
                            ch.dref = fma(m.dth, rcp_refined(y), Dk);
                            ch.tref = ts0;
                            x = exp(-(t0 - ts0) * m.inv_tm);
                        }
                        Dl = ch.dref * x;
                        ylo = y;
                        ++ch.ns;
                        if (ch.ns % kWave == 0) flush_spikes(sh, m, ch.ns - kWave, ch.ns, st, si, sk);
                        more = ch.ns < m.s_max;
                        if (!more) break;
                    }
                    const double lk = log_coarse(ch.dref);
                    ch.K = ch.ns > 0 ? lk - log_margin(lk) + ch.tref * m.inv_tm : -INFINITY;
                    if (!more) break;
                }
                if (!more) break;
            }
            if (ch.ns == ns_c) {                          // no spike: the next window by the K there is
                from = from_c;
                c_n = select(ch.K);
                if (wn > 0) {
                    nx = win_load(sh, c_n, seg0, nb, tt, src, d, pool);
                    wvn = load_wt(nx);
                }
            }
            c = c_n;
            in = nx;
            wv = wvn;
        }
        wave_lds_sync();                                  // the list is rewritten by the next chunk
#pragma unroll
        for (int h = 0; h < kSegPerLane; ++h) {
            mw[h] = m1[h];
            m1[h] = m2[h];
        }
    }
    flush_spikes(sh, m, ch.ns - ch.ns % kWave, ch.ns, st, si, sk);
    if (lane == 0) out_n[idx] = ch.ns;
    return ch.ns;
}

// Work-list driven: the per-sample lists of neurons built by the check pass
// are taken as one concatenated list.  Wave w of the grid (the workgroups' first
// waves first) takes entry w, then, when the list is longer than the grid, the
// next one that no wave has taken (a counter, read an entry ahead; on a shorter
// list thousands of waves would wait 15 us in line for it).  Status counts are
// added once per workgroup.
template <int PI>
__global__ __launch_bounds__(kWave * kResolveWaves) void k_resolve(
    const float* __restrict__ ev_t, const int32_t* __restrict__ ev_src, const int32_t* __restrict__ ev_n, int B,
    int E_max, const float* __restrict__ WT, int C_in, int N, int E_pad, int S, Model m,
    const Decay* __restrict__ dec, const double2* __restrict__ carry, const uint32_t* __restrict__ mask,
    uint32_t pool_cap, const double2* __restrict__ pool, const uint32_t* __restrict__ pool_count,
    const uint32_t* __restrict__ work, const uint32_t* __restrict__ nwork, uint32_t* __restrict__ taken,
    unsigned long long most, float* __restrict__ out_t, int32_t* __restrict__ out_n, float* __restrict__ out_i, int32_t* __restrict__ out_k,
    int32_t* __restrict__ status)
{
    __shared__ ResolveLds s_lds[kResolveWaves];
    const int lane = (int)threadIdx.x % kWave, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    ResolveLds& sh = s_lds[wv];
    const uint32_t nwaves = gridDim.x * kResolveWaves;
    resolve_status(ev_n, B, E_max, pool_count, pool_cap, status);
    if (flagged_total(pool_count, B) <= most) return;                    // k_resolve_ring's
    // spikes and capped neurons of this workgroup's neurons, added to the
    // status words once at its end
    __shared__ unsigned long long s_spikes;
    __shared__ uint32_t s_capped;
    if (threadIdx.x == 0) {
        s_spikes = 0ull;
        s_capped = 0u;
    }
    __syncthreads();
    unsigned long long spikes = 0;
    uint32_t capped = 0;
    // Running sum of the list lengths over groups of 64 samples (one load per
    // lane, a wave prefix sum): entry w of the concatenated lists belongs to
    // the first sample whose running sum exceeds w.
    int b0 = 0;               // first sample of the current group
    uint32_t base = 0;        // entries of the samples before the group
    uint32_t incl = 0;        // running sum up to and including sample b0 + lane
    auto load_group = [&]() {
        uint32_t c = b0 + lane < B ? nwork[(size_t)(b0 + lane) * kCtr] : 0u;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const uint32_t v = (uint32_t)__shfl_up((int)c, off, kWave);
            if (lane >= off) c += v;
        }
        incl = base + c;
    };
    load_group();
    uint32_t total = (uint32_t)rl_int((int)incl, kWave - 1);
    for (int bb = kWave; bb < B; bb += kWave) {
        uint32_t c = bb + lane < B ? nwork[(size_t)(bb + lane) * kCtr] : 0u;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) c += (uint32_t)__shfl_xor((int)c, off, kWave);
        total += c;
    }
    uint32_t next = 0;
    for (uint32_t w = wv * gridDim.x + blockIdx.x; w < total;
         w = total > nwaves ? nwaves + (uint32_t)__builtin_amdgcn_readfirstlane((int)next) : total) {
        unsigned long long past = __ballot(b0 + lane < B && incl <= w);
        while (past == ~0ull) {              // w lies beyond the whole group
            base = (uint32_t)__shfl((int)incl, kWave - 1, kWave);
            b0 += kWave;
            if (b0 >= B) break;
            load_group();
            past = __ballot(b0 + lane < B && incl <= w);
        }
        const int l = __popcll(past);        // samples of the group whose entries end at or before w
        const int b = b0 + l;
        if (b0 >= B || l >= kWave || b >= B) break;
        const uint32_t before = l > 0 ? (uint32_t)__shfl((int)incl, l - 1, kWave) : base;
        if (lane == 0 && total > nwaves) next = atomicAdd(taken, 1u);
        const uint32_t bn = (uint32_t)__builtin_amdgcn_readfirstlane((int)work[(size_t)b * N + (w - before)]);
        const int ns = resolve_neuron<PI>(sh, (int)(bn / (uint32_t)N), (int)(bn % (uint32_t)N), ev_t, ev_src, ev_n,
                                      E_max, WT, C_in, N, E_pad, S, m, dec, carry, mask, pool_cap, pool, out_t, out_n,
                                      out_i, out_k);
        spikes += (unsigned long long)ns;
        capped += ns >= m.s_max ? 1u : 0u;
    }
    if (lane == 0 && spikes) {
        atomicAdd(&s_spikes, spikes);
        atomicAdd(&s_capped, capped);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_spikes) {
        const int32_t sp = (int32_t)(s_spikes > 0x7fffffffull ? 0x7fffffffull : s_spikes);
        atomicAdd(&status[LIF_ST_SPIKES], sp);
        atomicAdd(&status[LIF_ST_ROOT_SOLVES], sp);
        if (s_capped) {
            atomicAdd(&status[LIF_ST_CAPPED], (int32_t)s_capped);
            atomicOr(&status[LIF_ST_FLAGS], LIF_WARN_SPIKE_CAP);
        }
    }
}

}  // namespace lif

#include "lif_ring.hpp"

namespace lif {

// Status words of a sequential forward call, from what the pass wrote:
// spikes and capped neurons from the counts, events from the queue lengths.
// Each workgroup adds its sums with one atomic per word (one workgroup per
// kStatusPer counts); the status words start at zero (reset by k_prep).  The
// parallel path fills the same words inside its resolve pass.
constexpr int kStatusThreads = 1024;
constexpr int kStatusBatch = 8;
constexpr int kStatusPer = kStatusThreads * kStatusBatch;

__global__ __launch_bounds__(kStatusThreads) void k_status(const int32_t* __restrict__ ev_n, int B, int E_max, int N,
                                                           int s_max, const int32_t* __restrict__ out_n,
                                                           int32_t* __restrict__ status)
{
    __shared__ unsigned long long part[kStatusThreads / kWave][3];
    unsigned long long spikes = 0, capped = 0, events = 0;
    const size_t nn = (size_t)B * (size_t)N;
    for (size_t i0 = (size_t)blockIdx.x * kStatusPer + threadIdx.x; i0 < nn; i0 += (size_t)gridDim.x * kStatusPer) {
        int c[kStatusBatch];
#pragma unroll
        for (int u = 0; u < kStatusBatch; ++u) {
            const size_t i = i0 + (size_t)u * kStatusThreads;
            c[u] = i < nn ? out_n[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < kStatusBatch; ++u) {
            spikes += (unsigned long long)c[u];
            capped += c[u] >= s_max ? 1u : 0u;
        }
    }
    if (blockIdx.x == 0) {
        for (int b = threadIdx.x; b < B; b += kStatusThreads)
            events += (unsigned long long)clamp_count(ev_n[b], E_max);
    }
    unsigned long long v[3] = {spikes, capped, events};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[q] += __shfl_xor(v[q], off, kWave);
    }
    const int wave = (int)threadIdx.x / kWave;
    if (threadIdx.x % kWave == 0) {
#pragma unroll
        for (int q = 0; q < 3; ++q) part[wave][q] = v[q];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t[3] = {0, 0, 0};
        for (int w = 0; w < kStatusThreads / kWave; ++w)
            for (int q = 0; q < 3; ++q) t[q] += part[w][q];
        auto sat = [](unsigned long long x) { return (int32_t)(x > 0x7fffffffull ? 0x7fffffffull : x); };
        if (t[0]) {
            atomicAdd(&status[LIF_ST_SPIKES], sat(t[0]));
            atomicAdd(&status[LIF_ST_ROOT_SOLVES], sat(t[0]));
        }
        if (t[1]) {
            atomicAdd(&status[LIF_ST_CAPPED], sat(t[1]));
            atomicOr(&status[LIF_ST_FLAGS], LIF_WARN_SPIKE_CAP);
        }
        if (t[2]) atomicAdd(&status[LIF_ST_EVENTS], sat(t[2]));
    }
}

static unsigned status_blocks(int B, int N)
{
    const size_t nn = (size_t)B * (size_t)N;
    const size_t g = (nn + kStatusPer - 1) / kStatusPer;
    return (unsigned)(g < 1 ? 1 : (g > 64 ? 64 : g));
}

// Sequential baseline (Appendix E.3): one thread per (sample, neuron)
// consumes every event in order with the same interval test and root solve.
// The state (V, I) is the true one, so each interval starts with deficit 0;
// spikes inside it raise the deficit and the rest of the interval is
// re-tested.
// QUEUE: every neuron has its own queue (a layer with synaptic delays):
// ev_t holds the arrival times [B][N][E_max], q_k the sample's event index of
// each entry, and each thread computes its own decays (no shared table).
template <bool QUEUE>
__global__ __launch_bounds__(64) void k_sequential(const float* __restrict__ ev_t, const int32_t* __restrict__ ev_src,
                                                   const int32_t* __restrict__ ev_n, const int32_t* __restrict__ q_k,
                                                   int B, int E_max, const float* __restrict__ WT, int C_in, int N,
                                                   Model m, int E_pad, const Decay* __restrict__ dec,
                                                   float* __restrict__ out_t, int32_t* __restrict__ out_n,
                                                   float* __restrict__ out_i, int32_t* __restrict__ out_k)
{
    const size_t idx_raw = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = idx_raw < (size_t)B * (size_t)N;
    const size_t idx = live ? idx_raw : 0;            // lanes past the end run neuron 0 and write nothing
    int b = (int)(idx / (size_t)N), n = (int)(idx % (size_t)N);
    int nb = clamp_count(ev_n[b], E_max);
    const float* tt = ev_t + (QUEUE ? idx : (size_t)b) * (size_t)E_max;
    const int32_t* src = ev_src + (size_t)b * E_max;
    const int32_t* qk = QUEUE ? q_k + idx * (size_t)E_max : nullptr;
    const Decay* d = QUEUE ? nullptr : dec + (size_t)b * E_pad;
    float* st = out_t + idx * (size_t)m.s_max;
    float* si = out_i ? out_i + idx * (size_t)m.s_max : nullptr;
    int32_t* sk = out_k ? out_k + idx * (size_t)m.s_max : nullptr;
    int ns = 0;
    bool capped = false;
    double V = 0.0, I = 0.0, t_prev = 0.0;
    for (int k = 0; k <= nb && !capped; ++k) {
        double L, A, C, Dd;
        if (k < nb) {
            const Decay e = QUEUE ? make_decay(m, tt, k) : d[k];
            A = e.A; C = e.C; Dd = e.D;
            L = (double)tt[k] - t_prev;
        } else {
            L = m.t_end - t_prev;                      // open interval after the last event
            if (!(L > 0.0)) break;
            if (isinf(L)) {
                A = 0.0; C = 0.0; Dd = 0.0;
            } else {
                A = exp(-L * m.inv_tm);
                Dd = exp(-L * m.inv_ts);
                C = unit_kernel(m, L, A);
            }
        }
        double V1 = A * V + C * I;
        // no-crossing screen V0 + max(I0 - th, 0) L / tm >= th_lo (screen_value)
        if (L > 0.0 && V + (I > m.th ? (I - m.th) * (L * m.inv_tm) : 0.0) >= m.th_lo) {
            IntervalMax im = interval_max(m, V, I, V1, L, A, Dd);
            double Dk = 0.0, lo = 0.0, ylo = 1.0, Flo = V - m.th;
            const double kI = m.kappa * I;
            while (Dk * im.a <= im.g) {
                const SpikeY sp = solve_spike_y(m, V - Dk + kI, kI, lo, ylo, Flo, im.hi, im.Fhi - Dk);
                const double u = -m.tm * log(sp.y);
                if (live) {
                    st[ns] = (float)(t_prev + u);
                    if (si) si[ns] = (float)(I * (sp.E2 * sp.y));
                    if (sk) sk[ns] = k;
                }
                ++ns;
                Dk += m.dth * sp.E1;
                lo = u;
                ylo = sp.y;
                Flo = -m.dth * sp.E1;
                if (ns >= m.s_max) { capped = true; break; }
            }
            V1 -= Dk * A;                               // true V at the end of the interval
        }
        V = V1;
        if (k < nb) {
            const int se = QUEUE ? min(max(qk[k], 0), nb - 1) : k;
            I = Dd * I + (double)WT[(size_t)clamp_src(src[se], C_in) * (size_t)N + n];
            t_prev = (double)tt[k];
        }
    }
    if (live) {
        out_n[idx] = ns;
        for (int s = ns; s < m.s_max; ++s) {
            st[s] = INFINITY;
            if (si) si[s] = 0.0f;
            if (sk) sk[s] = 0;
        }
    }
}

__global__ void k_status_zero(int32_t* __restrict__ status)
{
    if (threadIdx.x < LIF_STATUS_WORDS) status[threadIdx.x] = 0;
}

int launch_sequential_queue(const float* q_t, const int32_t* q_k, const int32_t* ev_src, const int32_t* ev_n, int B,
                            int E_max, const float* WT, int C_in, int N, const Model& m, float* out_t, int32_t* out_n,
                            float* out_i, int32_t* out_k, int32_t* status, hipStream_t stream)
{
    const size_t nn = (size_t)B * N;
    TIMED_LAUNCH("status_zero", k_status_zero, dim3(1), dim3(kWave), 0, stream, status);
    if (nn)
        TIMED_LAUNCH("sequential", k_sequential<true>, dim3((unsigned)((nn + 63) / 64)), dim3(64), 0, stream, q_t,
                     ev_src, ev_n, q_k, B, E_max, WT, C_in, N, m, 0, nullptr, out_t, out_n, out_i, out_k);
    TIMED_LAUNCH("status", k_status, dim3(status_blocks(B, N)), dim3(kStatusThreads), 0, stream, ev_n, B, E_max, N,
                 m.s_max, out_n, status);
    return check_launch();
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
FwdLayout fwd_layout(int B, int E_max, int N, int pool_cap)
{
    FwdLayout L{};
    L.S = (E_max + kSeg - 1) / kSeg;
    L.E_pad = L.S * kSeg;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    const size_t BS = (size_t)B * L.S;
    L.dec = take((size_t)B * L.E_pad * sizeof(Decay));
    L.segm = take(BS * sizeof(double2));
    // segment aggregates, overwritten in place by the carried states
    L.carry = take(BS * N * sizeof(double2));
    L.mask = take(BS * N * sizeof(uint32_t));
    // per sample: pool use, work-list length
    L.n_counters = 2 * (size_t)B * kCtr;
    L.counters = take(L.n_counters * sizeof(uint32_t));
    L.listed = take((size_t)B * N * sizeof(uint32_t));
    L.work = take((size_t)B * N * sizeof(uint32_t));
    // Pool of entering states: one 16-byte entry per flagged (sub-block,
    // neuron), in per-sample slices sized at a quarter of the dense bound
    // (every sub-block of every neuron flagged), at least 4096 entries (the
    // dense bound when smaller), and at most 1 GiB in all unless that leaves
    // fewer than 4096 per sample.  A full slice only sends the excess
    // sub-blocks through a slower rebuild from the segment's carried state,
    // with identical results.  lif_params.pool_cap >= 0 sets the slice size.
    const size_t dense = (size_t)L.S * kSubPerSeg * N;
    size_t cap = dense / 4 > 4096 ? dense / 4 : (dense < 4096 ? dense : 4096);
    const size_t budget = (size_t)1 << 30;
    if (B > 0 && (size_t)B * cap * sizeof(double2) > budget) {
        const size_t fit = budget / ((size_t)B * sizeof(double2));
        const size_t floor_ = dense < 4096 ? dense : 4096;
        cap = fit > floor_ ? fit : floor_;
    }
    if (pool_cap >= 0) cap = (size_t)pool_cap;
    if (B > 0 && (size_t)B * cap > 0xfffffff0ull) cap = 0xfffffff0ull / (size_t)B;   // slot indices are 32-bit
    L.pool_cap = cap;
    const size_t recs = (size_t)B * cap;
    L.pool = take((recs > 0 ? recs : 1) * sizeof(double2));   // at least one entry (a safe load address)
    L.total = off + 256;
    return L;
}

// Neurons per lane of the segment walks: NPL-wide weight loads need W^T rows
// of a multiple of NPL floats and an aligned base.
static int pick_npl(const float* WT, int N)
{
    const uintptr_t a = (uintptr_t)WT;
    if (N % 4 == 0 && a % 16 == 0) return 4;
    if (N % 2 == 0 && a % 8 == 0) return 2;
    return 1;
}

struct FwdPtrs {
    Decay* dec;
    double2 *segm, *carry;
    uint32_t* mask;
    uint32_t *counters, *pool_count, *nwork, *listed, *work;
    double2* pool;
};

// W^T past this size (half an XCD's L2): the aggregate pass goes tile by tile of
// 256 neurons, so that an XCD gathers from few columns at a time (32768 -> 2048,
// B = 16, 100 k events: 2.07 -> 1.59 ms; 2312 -> 1024, B = 64: 318 -> 303 us).  The
// check pass, whose tiles are 64 neurons and which reads the carried states and
// writes masks, stays sample-major (2.28 ms against 2.73 ms by tiles and 2.37 ms
// by groups of four).
constexpr size_t kTileMajorW = (size_t)2 << 20;

template <int NPL>
static void launch_walks(const FwdLayout& L, const FwdPtrs& P, const float* ev_t, const int32_t* ev_src,
                         const int32_t* ev_n, int B, int E_max, const float* WT, int C_in, int N, const Model& m,
                         int32_t* status, bool validate, int32_t* out_n, float* out_t, float* out_i, int32_t* out_k,
                         hipStream_t stream, bool check = true, bool bounds = false)
{
    const int tiles = (N + kWave * NPL - 1) / (kWave * NPL);
    const size_t items = (size_t)B * L.S * tiles;
    const unsigned blocks = (unsigned)((items + kWalkWaves - 1) / kWalkWaves);
    const int tmB = NPL == 4 && (size_t)C_in * N * sizeof(float) > kTileMajorW ? B : 0;
    // the aggregate pass also computes the decays and resets the counters and
    // status words (validation flags are ORed in after it)
    TIMED_LAUNCH("aggregate", k_aggregate<NPL>, dim3(blocks), dim3(kWave * kWalkWaves), 0, stream,
                 ev_t, ev_src, ev_n, E_max, L.E_pad, WT, C_in, N, tiles, L.S, (int)items, m, P.dec, P.segm,
                 P.carry, status, P.counters, L.n_counters, P.listed, (size_t)B * N, out_n, out_t, out_i, out_k,
                 out_t ? (size_t)B * N * (size_t)m.s_max : (size_t)0, tmB);
    if (validate)
        TIMED_LAUNCH("validate", k_validate, dim3((unsigned)(((size_t)B * E_max + 255) / 256)), dim3(256), 0,
                     stream, ev_t, ev_src, ev_n, B, E_max, C_in, status);
    const int ctiles = (N + kWave - 1) / kWave;
    TIMED_LAUNCH("carry", k_carry, dim3((unsigned)((size_t)B * ctiles)), dim3(kWave * kCarryWaves), 0, stream,
                 ev_n, B, E_max, N, ctiles, L.S, P.segm, P.carry, P.carry);
    if (!check) return;
    // The check pass takes one neuron per lane whatever NPL the aggregate
    // uses: its screen and pool state make wider lanes cost occupancy
    // (about 200 VGPRs at four neurons per lane against under 80 at one).
    const int ctl = (N + kWave - 1) / kWave;
    const size_t citems = (size_t)B * L.S * ctl;
    const unsigned cblocks = (unsigned)((citems + kWalkWaves - 1) / kWalkWaves);
    auto run = [&](auto kern) {
        TIMED_LAUNCH("check", kern, dim3(cblocks), dim3(kWave * kWalkWaves), 0, stream,
                     ev_t, ev_src, ev_n, E_max, L.E_pad, WT, C_in, N, ctl, L.S, (int)citems, m, P.dec, P.carry, P.mask,
                     P.pool, P.pool_count, (uint32_t)L.pool_cap, P.listed, P.work, P.nwork);
    };
    if (bounds) run(k_check<true>);
    else run(k_check<false>);
}

int forward_impl(bool sequential, const float* ev_t, const int32_t* ev_src, const int32_t* ev_n, int B, int E_max,
                 const float* WT, int C_in, int N, const lif_params* p, float* out_t, int32_t* out_n,
                 float* out_i, int32_t* out_k, int32_t* status, void* ws, size_t ws_bytes, hipStream_t stream)
{
    int rc = validate_forward_args(ev_t, ev_src, ev_n, B, E_max, WT, C_in, N, p, out_t, out_n, status);
    if (rc) return rc;
    if (!ws) return LIF_ERR_ARG;
    FwdLayout L = fwd_layout(B, E_max, N, p->pool_cap);
    if (ws_bytes < L.total) return LIF_ERR_WORKSPACE;
    Model m = make_model(*p);
    char* base = (char*)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    FwdPtrs P;
    P.dec = (Decay*)(base + L.dec);
    P.segm = (double2*)(base + L.segm);
    P.carry = (double2*)(base + L.carry);
    P.mask = (uint32_t*)(base + L.mask);
    P.counters = (uint32_t*)(base + L.counters);
    P.pool_count = P.counters;
    P.nwork = P.counters + (size_t)B * kCtr;
    P.listed = (uint32_t*)(base + L.listed);
    P.work = (uint32_t*)(base + L.work);
    P.pool = (double2*)(base + L.pool);

    const size_t nev = (size_t)B * L.E_pad;
    const size_t nn = (size_t)B * N;
    const size_t items_max = (size_t)B * L.S * ((N + kWave - 1) / kWave);
    if (items_max > 0x7fffffff || nn > 0xffffffffull) return LIF_ERR_SIZE;
    // mask words hold a per-sample pool offset in 28 bits
    if ((size_t)L.S * kSubPerSeg * N >= ((size_t)1 << (32 - kMaskBits))) return LIF_ERR_SIZE;
    const size_t n_out = nn * (size_t)p->s_max;
    const bool validate = (p->flags & LIF_VALIDATE) && (size_t)B * E_max;
    if (sequential || items_max == 0) {
        // decays and resets in their own pass (the parallel path folds them
        // into the aggregate and carry passes)
        size_t work_items = nev > n_out ? nev : n_out;
        size_t blocks = (work_items + 255) / 256;
        if (blocks > 2048) blocks = 2048;
        if (blocks < 1) blocks = 1;
        TIMED_LAUNCH("prep", k_prep, dim3((unsigned)blocks), dim3(256), 0, stream,
                     ev_t, ev_n, B, E_max, L.E_pad, L.S, m, P.dec, sequential ? nullptr : P.segm, status, P.counters,
                     L.n_counters, out_n, sequential ? nullptr : P.listed, nn, sequential ? nullptr : out_t, out_i,
                     out_k, n_out);
        if (validate)
            TIMED_LAUNCH("validate", k_validate, dim3((unsigned)(((size_t)B * E_max + 255) / 256)), dim3(256), 0,
                         stream, ev_t, ev_src, ev_n, B, E_max, C_in, status);
    }
    if (sequential) {
        if (nn)
            TIMED_LAUNCH("sequential", k_sequential<false>, dim3((unsigned)((nn + 63) / 64)), dim3(64), 0, stream,
                         ev_t, ev_src, ev_n, nullptr, B, E_max, WT, C_in, N, m, L.E_pad, P.dec, out_t, out_n, out_i,
                         out_k);
        TIMED_LAUNCH("status", k_status, dim3(status_blocks(B, N)), dim3(kStatusThreads), 0, stream, ev_n, B, E_max, N, m.s_max, out_n,
                     status);
        return check_launch();
    }
    if (items_max == 0) return check_launch();
    const bool bounds = (size_t)L.S * kSubPerSeg * nn > kRingDense;
    switch (pick_npl(WT, N)) {
    case 4: launch_walks<4>(L, P, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N, m, status, validate, out_n, out_t, out_i,
                            out_k, stream, true, bounds); break;
    case 2: launch_walks<2>(L, P, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N, m, status, validate, out_n, out_t, out_i,
                            out_k, stream, true, bounds); break;
    default: launch_walks<1>(L, P, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N, m, status, validate, out_n, out_t,
                             out_i, out_k, stream, true, bounds); break;
    }
    // Which resolve pass: the ring pass prepares every flagged sub-block and
    // follows each chain with the least latency (700 -> 256, B = 32, 6 k flagged:
    // 33 us against 50 us); the wave-per-neuron pass skips by key bounds
    // (2312 -> 1024 in bursts, B = 64, 11 M flagged: 3.9 against 0.63 ms; 32768 ->
    // 2048, B = 16, 18 M: 9.7 against 1.23 ms).  The ring pass costs 0.3 to 0.4 ns
    // a flagged sub-block beyond its chains (whole forwards of 700 -> 512, B = 128:
    // 782 against 713 us at 225 k), so the line lies where that reaches a chain's
    // length (kRingMost).  The count is known on the device only: calls that could
    // flag many launch both, and one of them leaves at once.  That second launch costs
    // a short call 3 to 6 us (700 -> 256, B = 32: 60 against 66 us), and the bounds
    // gain where a large share of the sub-blocks is flagged (there, of 2.6 M: 217
    // against 213 us at 115 k, 419 against 323 us at 350 k), so calls below
    // kRingDense sub-blocks in all, whose layers fire at a few percent of that,
    // launch the ring alone.
    const unsigned rgrid = (unsigned)(nn < 1024 ? nn : 1024);
    const bool both = bounds;
    const size_t rwg = (nn + kResolveWaves - 1) / kResolveWaves;
    const unsigned wgrid = (unsigned)(rwg < 1024 ? rwg : 1024);
    auto resolve = [&](auto wave, auto ring) {
        if (both)
            TIMED_LAUNCH("resolve", wave, dim3(wgrid), dim3(kWave * kResolveWaves), 0, stream, ev_t, ev_src, ev_n, B,
                         E_max, WT, C_in, N, L.E_pad, L.S, m, P.dec, P.carry, P.mask, (uint32_t)L.pool_cap, P.pool,
                         P.pool_count, P.work, P.nwork, P.counters + kTaken, kRingMost, out_t, out_n,
                         out_i, out_k, status);
        TIMED_LAUNCH("resolve", ring, dim3(rgrid), dim3(kWave * kRingWaves), 0, stream, ev_t, ev_src, ev_n, B,
                     E_max, WT, C_in, N, L.E_pad, L.S, m, P.dec, P.carry, P.mask, (uint32_t)L.pool_cap, P.pool,
                     P.pool_count, P.work, P.nwork, both ? kRingMost : ~0ull, out_t, out_n, out_i, out_k, status);
    };
    switch (m.p_int) {
    case 1: resolve(k_resolve<1>, k_resolve_ring<1>); break;
    case 2: resolve(k_resolve<2>, k_resolve_ring<2>); break;
    case 3: resolve(k_resolve<3>, k_resolve_ring<3>); break;
    case 4: resolve(k_resolve<4>, k_resolve_ring<4>); break;
    default: resolve(k_resolve<0>, k_resolve_ring<0>); break;
    }
    return check_launch();
}

}  // namespace lif

extern "C" size_t lif_layer_forward_workspace_size(int B, int E_max, int C_in, int N_out, const lif_params* p)
{
    (void)C_in;
    if (B < 0 || E_max < 0 || N_out < 1 || !p) return 0;
    return lif::fwd_layout(B, E_max, N_out, p->pool_cap).total;
}

extern "C" int lif_layer_forward(const float* ev_t, const int32_t* ev_src, const int32_t* ev_n, int B, int E_max,
                                 const float* WT, int C_in, int N_out, const lif_params* p, float* out_t,
                                 int32_t* out_n, float* out_i, int32_t* out_k, int32_t* status, void* ws,
                                 size_t ws_bytes, lif_stream_t stream)
{
    return lif::forward_impl(false, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, p, out_t, out_n, out_i, out_k,
                             status, ws, ws_bytes, (hipStream_t)stream);
}

extern "C" int lif_layer_forward_sequential(const float* ev_t, const int32_t* ev_src, const int32_t* ev_n, int B,
                                            int E_max, const float* WT, int C_in, int N_out, const lif_params* p,
                                            float* out_t, int32_t* out_n, float* out_i, int32_t* out_k,
                                            int32_t* status, void* ws, size_t ws_bytes, lif_stream_t stream)
{
    return lif::forward_impl(true, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, p, out_t, out_n, out_i, out_k,
                             status, ws, ws_bytes, (hipStream_t)stream);
}

namespace lif {

// ---------------------------------------------------------------------------
// Spike-count regularisers (App. E.1, Eq. loss): for every (sample, neuron)
// and every input interval j (between events j - 1 and j, and the open one
// after the last event up to t_end), the largest V of the interval's
// trajectory from its true start state (resets of earlier intervals
// applied, none inside it), split into the intervals that hold a spike
// (out_k = j) and the silent ones.  The no-reset state comes from the
// forward's segment scan (k_aggregate, k_carry); the resets enter as the
// decaying deficit (V_th - V_reset) e^{-(t - t_s)/tm} of each earlier spike.
// ---------------------------------------------------------------------------


// Per (sample, segment, 64 neurons): the segment's intervals (and the open
// one in the sample's last segment); per lane the sums of the hinge terms
// and the interval counts, part = (sum under, silent count, sum over,
// spiking count); with rec, the per-interval records and, per (sample,
// segment, neuron), the sums over the segment's active intervals of the
// decays from the segment's start (the input event before it) to the
// interval's argmax, local = (under: e^{-./tm}, e^{-./ts}; over: the same).
// kRec: records and local sums for the gradient; kSlope: with end-point slopes
// (dL/dt wanted).  Nearly every interval of a wave is without a spike on all of
// its lanes and takes the straight path, and the lookup of the lane's next spike
// stays in a register.  Bound by VALU issue (73 % busy) and the records' stores:
// 700 -> 512, B = 128, 10 k events, 5.2 GB of records: 3.45 -> 1.89 ms (the
// quotient, logarithm and spike lookups of every interval: 141 VALU, 92 scalar
// instructions and 19 branches per event before, 73, 28 and 7 now).
template <bool kRec, bool kSlope>
__global__ __launch_bounds__(kWave * kWalkWaves) void k_reg_walk(
    const float* __restrict__ ev_t, const int32_t* __restrict__ ev_src, const int32_t* __restrict__ ev_n, int E_max,
    int E_pad, const float* __restrict__ WT, int C_in, int N, int tiles, int S, int items, Model m,
    const Decay* __restrict__ dec, const double2* __restrict__ carry, const float* __restrict__ out_t,
    const int32_t* __restrict__ out_n, const int32_t* __restrict__ out_k, double4* __restrict__ part,
    float2* __restrict__ rec, double4* __restrict__ local)
{
    __shared__ double2 s_ad[kWalkWaves][kSeg];
    __shared__ double s_c[kWalkWaves][kSeg];
    __shared__ float s_t[kWalkWaves][kSeg + 1];
    WalkCoords c;
    if (!walk_coords<1>(items, tiles, S, ev_n, E_max, N, c)) return;
    const int lane = c.lane, wv = (int)threadIdx.x / kWave;
    const int n = c.n0;
    double2* lad = s_ad[wv];
    double* lc = s_c[wv];
    float* lt = s_t[wv];
    const float* tt = ev_t + (size_t)c.b * E_max;
    const Decay* dd = dec + (size_t)c.b * E_pad + c.k0;
    // lt[e] = start of interval k0 + e (the time of event k0 + e - 1, or 0)
#pragma unroll
    for (int h = 0; h < kSrcRegs; ++h) {
        const int e = h * kWave + lane;
        lc[e] = dd[e].C;
        if (e < c.cnt) lt[e + 1] = tt[c.k0 + e];
    }
    if (lane == 0) lt[0] = c.k0 > 0 ? tt[c.k0 - 1] : 0.0f;
    const Stage st = stage_segment(c, ev_src + (size_t)c.b * E_max + c.k0, dd, WT, C_in, N, lad, nullptr);
    const double2 cs = carry[((size_t)c.b * S + c.seg) * N + n];
    double U = cs.x, J = cs.y;
    // the neuron's spikes: the deficit at the segment's start from those of
    // earlier intervals, then the ones inside taken in order
    const size_t base = ((size_t)c.b * N + n) * (size_t)m.s_max;
    const float* ts = out_t + base;
    const int32_t* ks = out_k + base;
    const int ns = c.live ? min(out_n[(size_t)c.b * N + n], m.s_max) : 0;
    const double t_start = (double)lt[0];
    double Dft = 0.0;
    int sp = 0, knext = ns > 0 ? ks[0] : -1;             // the next spike's interval (-1: none)
    auto advance = [&]() {
        ++sp;
        knext = sp < ns ? ks[sp] : -1;
    };
    while (knext >= 0 && knext < c.k0) {
        Dft += m.dth * exp(-(t_start - (double)ts[sp]) * m.inv_tm);
        advance();
    }
    double su = 0.0, so = 0.0;
    int nspk = 0, nint = c.cnt;
    float2* rb = kRec ? rec + (size_t)c.b * (E_max + 1) * N + n : nullptr;
    double cdm = 1.0, cds = 1.0;                 // decays from the segment's start to the interval's start
    double4 loc = make_double4(0.0, 0.0, 0.0, 0.0);
    auto take = [&](int j, const RegArg& ra, double V0, double I1, double A, double Dd, double t1, bool input_end) {
        const double h = m.th - ra.vmax;
        float sgn = h > 0.0 ? 1.0f : 0.0f;
        double under = fmax(h, 0.0);
        const bool spk = knext == j;
        const bool any = __ballot(spk) != 0ull;
        if (any) {
            asm volatile("");
            if (spk) {
                so += fmax(-h, 0.0);
                ++nspk;
                under = 0.0;
                sgn = h < 0.0 ? -1.0f : 0.0f;
            }
        }
        su += under;
        if constexpr (kRec) {
            const bool end = ra.at_end && input_end;      // (the open interval's end t_end is no input time)
            const float code = ra.at_start ? kRecStartCode : (end ? kRecEndCode : (float)ra.em);
            float y = (float)ra.es;
            if constexpr (kSlope) {
                const double v = ra.at_start ? (j > 0 ? J - V0 : 0.0) : I1 - ra.vmax;
                y = ra.at_start || end ? (float)(v * m.inv_tm) : y;
            }
            if (c.live) rb[(size_t)j * N] = make_float2(sgn * code, sgn == 0.0f ? 0.0f : y);
            const double pm = sgn > 0.0f ? cdm : 0.0, ps = sgn > 0.0f ? cds : 0.0;
            loc.x = fma(pm, ra.em, loc.x);
            loc.y = fma(ps, ra.es, loc.y);
            if (any && sgn < 0.0f) {
                loc.z = fma(cdm, ra.em, loc.z);
                loc.w = fma(cds, ra.es, loc.w);
            }
            cdm *= A;
            cds *= Dd;
        }
        // the deficit at the interval's end, with the spikes inside it
        Dft *= A;
        if (any) {
            while (knext == j) {
                Dft += m.dth * exp(-(t1 - (double)ts[sp]) * m.inv_tm);
                advance();
            }
        }
    };
    const int ng = (c.cnt + kGrp - 1) / kGrp;
    float wa[kGrp][1], wb[kGrp][1];
    load_grp<1>(st, 0, wa);
    auto group = [&](int g, const float (&w)[kGrp][1]) {
#pragma unroll
        for (int jj = 0; jj < kGrp; ++jj) {
            const int e = g * kGrp + jj;
            if (e >= c.cnt) break;
            const double2 ad = lad[e];
            const double V0 = fma(m.kappa, U - J, -Dft), V1 = fma(V0, ad.x, lc[e] * J), I1 = J * ad.y;
            take(c.k0 + e, reg_vmax_in(m, V0, J, ad.x, ad.y, V1, I1), V0, I1, ad.x, ad.y, (double)lt[e + 1], true);
            step1(ad, w[jj][0], U, J);
        }
    };
    for (int g = 0; g < ng; g += 2) {
        if (g + 1 < ng) load_grp<1>(st, (g + 1) * kGrp, wb);
        group(g, wa);
        if (g + 1 >= ng) break;
        if (g + 2 < ng) load_grp<1>(st, (g + 2) * kGrp, wa);
        group(g + 1, wb);
    }
    if (c.k0 + c.cnt == c.nb) {
        // the open interval after the sample's last event, up to t_end
        const double t0 = (double)lt[c.cnt];
        const double L = m.t_end - t0;
        const double A = isinf(L) ? 0.0 : exp(-L * m.inv_tm), Dd = isinf(L) ? 0.0 : exp(-L * m.inv_ts);
        const double V0 = v_of(m, U, J) - Dft;
        take(c.nb, reg_vmax_arg(m, V0, J, L, A, Dd), V0, J * Dd, A, Dd, m.t_end, false);
        ++nint;
    }
    if (c.live) part[((size_t)c.b * S + c.seg) * N + n] = make_double4(su, (double)(nint - nspk), so, (double)nspk);
    if (kRec && c.live) local[((size_t)c.b * S + c.seg) * N + n] = loc;
}

// Per (sample, neuron): the sums over the segments in order, then the means
// over the silent and the spiking intervals (0 for an empty set).
__global__ __launch_bounds__(256) void k_reg_reduce(const double4* __restrict__ part, const int32_t* __restrict__ ev_n,
                                                    int B, int E_max, int N, int S, double th, double* __restrict__ ub,
                                                    double* __restrict__ ob, float* __restrict__ under,
                                                    float* __restrict__ over, double2* __restrict__ counts)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)B * N) return;
    const int b = (int)(i / (size_t)N), n = (int)(i % (size_t)N);
    const int nb = clamp_count(ev_n[b], E_max);
    const int Sb = (nb + kSeg - 1) / kSeg;
    double su = 0.0, nsil = 0.0, so = 0.0, nspk = 0.0;
#pragma unroll 8                   // (eight loads in flight: the sums alone are a chain of latencies)
    for (int s = 0; s < Sb; ++s) {
        const double4 p = part[((size_t)b * S + s) * N + n];
        su += p.x;
        nsil += p.y;
        so += p.z;
        nspk += p.w;
    }
    if (Sb == 0) {             // no event: the one interval [0, t_end) at rest (V_max = 0)
        su = th;
        nsil = 1.0;
    }
    const double u = nsil > 0.0 ? su / nsil : 0.0;
    const double o = nspk > 0.0 ? so / nspk : 0.0;
    ub[i] = u;
    ob[i] = o;
    if (under) under[i] = (float)u;
    if (over) over[i] = (float)o;
    if (counts) counts[i] = make_double2(nsil, nspk);
}

// The two loss terms.  Per neuron (a workgroup takes tiles of kMeanN of them, its
// rows of threads every kMeanB-th sample) the batch means and the gates of the mean
// spike count against the target; a neuron's two terms replace its first
// sample's ub and ob, which only its own threads have read.  The means over the
// neurons follow in k_reg_loss, or (one workgroup, loss given) at once.  Every sum is
// in a fixed order.  One workgroup walked the whole batch before: 112 -> 8 us at
// B = 128, N = 512; with up to kMeanOne tiles and kMeanB samples one still does, the
// second launch being the larger part there (delayed regularisers of 64 -> 64, B = 2:
// 56.9 us with two launches, 54.1 us with one; of 64 -> 60, B = 40: 59 against 62 us).
constexpr int kRegThreads = 256, kMeanN = 16, kMeanB = kRegThreads / kMeanN, kMeanOne = 4;

__device__ __forceinline__ void reg_loss_means(const double* ub, const double* ob, int N, float* __restrict__ loss)
{
    __shared__ double s_reg[kRegThreads], s_over[kRegThreads];
    double lr = 0.0, lo = 0.0;
    for (int n = threadIdx.x; n < N; n += kRegThreads) {
        lr += ub[n];
        lo += ob[n];
    }
    s_reg[threadIdx.x] = lr;
    s_over[threadIdx.x] = lo;
    __syncthreads();
    for (int off = kRegThreads / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) {
            s_reg[threadIdx.x] += s_reg[threadIdx.x + off];
            s_over[threadIdx.x] += s_over[threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        loss[0] = (float)(s_reg[0] / (double)N);
        loss[1] = (float)(s_over[0] / (double)N);
    }
}

__global__ __launch_bounds__(kRegThreads) void k_reg_mean(double* ub, double* ob, const int32_t* __restrict__ out_n,
                                                          int B, int N, int s_max, double c_target,
                                                          double2* __restrict__ gates, float* __restrict__ loss)
{
    __shared__ double4 s_p[kMeanB][kMeanN];
    const int nl = (int)threadIdx.x % kMeanN, bl = (int)threadIdx.x / kMeanN;
    for (int n0 = (int)blockIdx.x * kMeanN; n0 < N; n0 += (int)gridDim.x * kMeanN) {
        const int n = n0 + nl;
        double4 p = make_double4(0.0, 0.0, 0.0, 0.0);
        if (n < N) {
#pragma unroll 4
            for (int b = bl; b < B; b += kMeanB) {
                const size_t i = (size_t)b * N + n;
                const double cnt = (double)min(out_n[i], s_max);
                p.x += cnt;
                p.y += ub[i];
                p.z += ob[i];
                p.w += fmax(cnt / c_target - 1.0, 0.0) * ob[i];
            }
        }
        s_p[bl][nl] = p;
        __syncthreads();
        if (bl == 0 && n < N) {
            for (int q = 1; q < kMeanB; ++q) {
                const double4 o = s_p[q][nl];
                p.x += o.x;
                p.y += o.y;
                p.z += o.z;
                p.w += o.w;
            }
            const double cb = p.x / (double)B;
            const double gu = fmax(1.0 - cb / c_target, 0.0), go = fmax(cb / c_target - 1.0, 0.0);
            ub[n] = gu * (p.y / (double)B) + go * (p.z / (double)B);
            ob[n] = p.w;
            if (gates) gates[n] = make_double2(gu, go);
        }
        __syncthreads();
    }
    if (loss) reg_loss_means(ub, ob, N, loss);
}

__global__ __launch_bounds__(kRegThreads) void k_reg_loss(const double* __restrict__ ub, const double* __restrict__ ob,
                                                          int N, float* __restrict__ loss)
{
    reg_loss_means(ub, ob, N, loss);
}

void launch_reg_loss(double* ub, double* ob, const int32_t* out_n, int B, int N, int s_max, double c_target,
                     float* loss, double2* gates, hipStream_t stream)
{
    const int tiles = (N + kMeanN - 1) / kMeanN;
    const bool one = loss && tiles <= kMeanOne && B <= kMeanB;
    TIMED_LAUNCH("reg_mean", k_reg_mean, dim3(one ? 1u : (unsigned)tiles), dim3(kRegThreads), 0, stream, ub, ob, out_n,
                 B, N, s_max, c_target, gates, one ? loss : nullptr);
    if (loss && !one) TIMED_LAUNCH("reg_loss", k_reg_loss, dim3(1), dim3(kRegThreads), 0, stream, ub, ob, N, loss);
}

struct RegLayout {
    FwdLayout f;
    size_t part, ub, ob, status, total;
};

static RegLayout reg_layout(int B, int E_max, int N)
{
    RegLayout R;
    R.f = fwd_layout(B, E_max, N, 0);
    size_t off = R.f.total;
    auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    R.part = take((size_t)B * R.f.S * N * sizeof(double4));
    R.ub = take((size_t)B * N * sizeof(double));
    R.ob = take((size_t)B * N * sizeof(double));
    R.status = take(LIF_STATUS_WORDS * sizeof(int32_t));
    R.total = off + 256;
    return R;
}

}  // namespace lif

extern "C" size_t lif_spike_count_reg_workspace_size(int B, int E_max, int C_in, int N_out)
{
    (void)C_in;
    if (B < 0 || E_max < 0 || N_out < 1) return 0;
    return lif::reg_layout(B, E_max, N_out).total;
}

extern "C" int lif_spike_count_reg(const float* ev_t, const int32_t* ev_src, const int32_t* ev_n, int B, int E_max,
                                   const float* WT, int C_in, int N_out, const lif_params* p, const float* out_t,
                                   const int32_t* out_n, const int32_t* out_k, double c_target, float* loss,
                                   float* under, float* over, void* ws, size_t ws_bytes, lif_stream_t stream_)
{
    using namespace lif;
    int rc = validate_forward_args(ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, p, out_t, out_n, out_n);
    if (rc) return rc;
    if (!out_k || !loss || !ws || !(c_target > 0.0) || !isfinite(c_target)) return LIF_ERR_ARG;
    const RegLayout R = reg_layout(B, E_max, N_out);
    if (ws_bytes < R.total) return LIF_ERR_WORKSPACE;
    const size_t items_max = (size_t)B * R.f.S * ((N_out + kWave - 1) / kWave);
    if (items_max > 0x7fffffff) return LIF_ERR_SIZE;
    hipStream_t stream = (hipStream_t)stream_;
    const Model m = make_model(*p);
    char* base = (char*)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    FwdPtrs P{};
    P.dec = (Decay*)(base + R.f.dec);
    P.segm = (double2*)(base + R.f.segm);
    P.carry = (double2*)(base + R.f.carry);
    P.mask = (uint32_t*)(base + R.f.mask);
    P.counters = (uint32_t*)(base + R.f.counters);
    P.pool_count = P.counters;
    P.nwork = P.counters + (size_t)B * kCtr;
    P.listed = (uint32_t*)(base + R.f.listed);
    P.work = (uint32_t*)(base + R.f.work);
    P.pool = (double2*)(base + R.f.pool);
    double4* part = (double4*)(base + R.part);
    double* ub = (double*)(base + R.ub);
    double* ob = (double*)(base + R.ob);
    int32_t* st = (int32_t*)(base + R.status);
    const size_t nn = (size_t)B * N_out;
    if (items_max > 0) {
        // the no-reset state entering every segment (the forward's scan)
        switch (pick_npl(WT, N_out)) {
        case 4: launch_walks<4>(R.f, P, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, m, st, false, nullptr, nullptr,
                                nullptr, nullptr, stream, false); break;
        case 2: launch_walks<2>(R.f, P, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, m, st, false, nullptr, nullptr,
                                nullptr, nullptr, stream, false); break;
        default: launch_walks<1>(R.f, P, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, m, st, false, nullptr,
                                 nullptr, nullptr, nullptr, stream, false); break;
        }
        const int tl = (N_out + kWave - 1) / kWave;
        const size_t it = (size_t)B * R.f.S * tl;
        TIMED_LAUNCH("reg_walk", (k_reg_walk<false, false>), dim3((unsigned)((it + kWalkWaves - 1) / kWalkWaves)),
                     dim3(kWave * kWalkWaves), 0, stream, ev_t, ev_src, ev_n, E_max, R.f.E_pad, WT, C_in, N_out, tl,
                     R.f.S, (int)it, m, P.dec, P.carry, out_t, out_n, out_k, part, nullptr, nullptr);
    }
    if (nn)
        TIMED_LAUNCH("reg_reduce", k_reg_reduce, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, stream, part, ev_n,
                     B, E_max, N_out, R.f.S, m.th, ub, ob, under, over, nullptr);
    if (B > 0)
        launch_reg_loss(ub, ob, out_n, B, N_out, m.s_max, c_target, loss, nullptr, stream);
    return check_launch();
}

// ---------------------------------------------------------------------------
// Gradient of lam_reg L_reg + lam_over L_over (App. E.1, Eq. loss), the gates
// held constant (functions of the spike counts).  Each V_max is the value of
// its interval's trajectory at the argmax tau_j = t_{j-1} + u_j:
//   V(tau) = sum_{k < j} w_k K(tau - t_k) - (V_th - V_reset) sum_{s: out_k < j} e^{-(tau - t_s)/tm},
// so with mu_j = dL/dV_max of interval j (G_u for an active under-firing
// interval, G_o for an active over-firing one, 0 otherwise) and
//   P_k = sum_{j > k} mu_j e^{-(tau_j - t_k)/tm}    (Q_k the same with ts)
// every input event k collects
//   dL/dw_{i, src_k} += kappa (P_k - Q_k),   dL/dt_k += w kappa (P_k/tm - Q_k/ts)
// (the adjoint sums of the layer's backward pass with a pseudo-spike at
// each interval's argmax), an argmax at an interval end that is an input
// time adds mu_j V'(tau_j) to that time's gradient, and spike s collects the
// upstream spike-time gradient -((V_th - V_reset)/tm) P_{out_k} e^{-(t_{out_k} - t_s)/tm},
// which the layer's backward pass carries to W and the input times.
// P obeys P_{k-1} = A_k P_k + mu_k e^{-u_k/tm} (A_k the decay into event k),
// a reverse affine scan: per segment the sums over its own intervals (taken
// by k_reg_walk on its forward walk, split by hinge so that the multipliers,
// known only once the whole batch is walked, enter later), a reverse carry
// over segments (k_regg_carry), and the walk back with the carry
// (k_regg_tile, k_regg_walk).  dL/dW is added as 64-bit fixed-point integers (order
// free); dL/dt per neuron tile, the tiles added in order.
// ---------------------------------------------------------------------------
namespace lif {


// Per (sample, neuron): G_u = -lam_reg gu / (N B nsil), G_o = (lam_reg go /
// (N B) + lam_over gi / N) / nspk with gi = ReLU(c / c_target - 1) of its
// spike count c, and |G_u| nsil + |G_o| nspk, a bound of its sums P and Q.
__global__ __launch_bounds__(256) void k_regg_coef(const double2* __restrict__ counts,
                                                   const double2* __restrict__ gates,
                                                   const int32_t* __restrict__ out_n, int B, int N, int s_max,
                                                   double c_target, double lam_reg, double lam_over,
                                                   double2* __restrict__ coef, double* __restrict__ musum,
                                                   long long* __restrict__ gw, size_t nW)
{
    const size_t gtid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, gs = (size_t)gridDim.x * blockDim.x;
    for (size_t x = gtid; x < nW; x += gs) gw[x] = 0;
    const size_t nn = (size_t)B * N;
    for (size_t i = gtid; i < nn; i += gs) {
        const int n = (int)(i % (size_t)N);
        const double2 cnt = counts[i], g = gates[n];
        const double c = (double)min(out_n[i], s_max);
        const double gi = fmax(c / c_target - 1.0, 0.0);
        const double Gu = cnt.x > 0.0 ? -lam_reg * g.x / ((double)N * B) / cnt.x : 0.0;
        const double Go = cnt.y > 0.0 ? (lam_reg * g.y / ((double)N * B) + lam_over * gi / (double)N) / cnt.y : 0.0;
        coef[i] = make_double2(Gu, Go);
        musum[i] = fabs(Gu) * cnt.x + fabs(Go) * cnt.y;
    }
}

void launch_regg_coef(const double2* counts, const double2* gates, const int32_t* out_n, int B, int N, int s_max,
                      double c_target, double lam_reg, double lam_over, double2* coef, double* musum,
                      hipStream_t stream)
{
    const size_t nn = (size_t)B * N;
    size_t blocks = (nn + 255) / 256;
    blocks = blocks < 1 ? 1 : (blocks > 2048 ? 2048 : blocks);
    TIMED_LAUNCH("regg_coef", k_regg_coef, dim3((unsigned)blocks), dim3(256), 0, stream, counts, gates, out_n, B, N,
                 s_max, c_target, lam_reg, lam_over, coef, musum, (long long*)nullptr, (size_t)0);
}

// Fixed-point scale of dL/dW (one workgroup): a contribution is at most
// 2 kappa M (M = the largest bound of k_regg_coef; the float32 decays of the
// records add far less than the bit of headroom), an element sums at most
// one per event of the batch: scale = 2^(61 - ceil(log2(2 kappa M events))).
// A chain of load latencies: 1024 threads with eight loads in flight, 64 -> 10 us
// for 65536 bounds.
constexpr int kScaleThreads = 1024;

__global__ __launch_bounds__(kScaleThreads) void k_regg_scale(const double* __restrict__ musum, size_t nn,
                                                            const int32_t* __restrict__ ev_n, int B, int E_max,
                                                            double kappa, double* __restrict__ scale)
{
    __shared__ double s_max[kScaleThreads], s_ev[kScaleThreads];
    double mx = 0.0, ev = 0.0;
#pragma unroll 8
    for (size_t i = threadIdx.x; i < nn; i += kScaleThreads) mx = fmax(mx, musum[i]);
    for (int b = threadIdx.x; b < B; b += kScaleThreads) ev += (double)clamp_count(ev_n[b], E_max);
    s_max[threadIdx.x] = mx;
    s_ev[threadIdx.x] = ev;
    __syncthreads();
    for (int off = kScaleThreads / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) {
            s_max[threadIdx.x] = fmax(s_max[threadIdx.x], s_max[threadIdx.x + off]);
            s_ev[threadIdx.x] += s_ev[threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double bound = 2.0 * kappa * s_max[0] * fmax(s_ev[0], 1.0);
        int ex = 0;
        if (bound > 0.0 && isfinite(bound)) frexp(bound, &ex);
        scale[0] = ldexp(1.0, 61 - ex);
    }
}

// Per (sample, 64 neurons): the reverse carry over segments.  F(seg) =
// (P, Q) at the input event before segment seg = its own part (local with the
// neuron's G) plus the later segments' F decayed over the segment (its
// composed decays segm); cin[seg] = F(seg + 1) = (P, Q) at the segment's last
// event, 0 for the last segment (its walk adds the open interval itself).
__global__ __launch_bounds__(kWave) void k_regg_carry(const int32_t* __restrict__ ev_n, int E_max, int N, int S,
                                                      const double2* __restrict__ segm,
                                                      const double4* __restrict__ local,
                                                      const double2* __restrict__ coef, double2* __restrict__ cin)
{
    const int b = blockIdx.y, n = blockIdx.x * kWave + (int)threadIdx.x;
    if (n >= N) return;
    const int nb = clamp_count(ev_n[b], E_max);
    const int Sb = (nb + kSeg - 1) / kSeg;
    const double2 G = coef[(size_t)b * N + n];
    double Fm = 0.0, Fs = 0.0;
#pragma unroll 8
    for (int seg = Sb - 1; seg >= 0; --seg) {
        const size_t at = ((size_t)b * S + seg) * N + n;
        const double4 L = local[at];
        const double2 f = segm[(size_t)b * S + seg];
        cin[at] = make_double2(Fm, Fs);
        Fm = fma(f.x, Fm, fma(G.x, L.x, G.y * L.z));
        Fs = fma(f.y, Fs, fma(G.x, L.y, G.y * L.w));
    }
}

// Per (sample, segment, 64 neurons): (P_k, Q_k) from the segment's last
// event down to its first, each event's contributions, and the upstream
// gradient of the lane's spikes inside the segment.  The segment is staged
// as in the forward walks (sources in registers, decays and times in LDS);
// groups of kGrp events are walked from the last backwards with the next
// group's weights and records in flight, the dL/dW terms of a group added
// after its walk and its dL/dt terms summed over the lanes together
// (group_sum8).
constexpr int kRegPre = 4;

__global__ __launch_bounds__(kWave * kWalkWaves) void k_regg_walk(
    const float* __restrict__ ev_t, const int32_t* __restrict__ ev_src, const int32_t* __restrict__ ev_n, int B,
    int E_max, int E_pad, const float* __restrict__ WT, int C_in, int N, int tiles, int S, int items, Model m,
    const Decay* __restrict__ dec, const float2* __restrict__ rec, const double2* __restrict__ coef,
    const double2* __restrict__ cin, const float* __restrict__ out_t, const int32_t* __restrict__ out_n,
    const int32_t* __restrict__ out_k, const double* __restrict__ scale, long long* __restrict__ gw,
    double* __restrict__ gtp, float* __restrict__ grad_spike)
{
    __shared__ double2 s_ad[kWalkWaves][kSeg];
    __shared__ float s_t[kWalkWaves][kSeg];
    WalkCoords c;
    if (!walk_coords<1>(items, tiles, S, ev_n, E_max, N, c)) return;
    const int n = c.n0, lane = c.lane, wv = (int)threadIdx.x / kWave;
    double2* lad = s_ad[wv];
    float* lt = s_t[wv];
    const Decay* d = dec + (size_t)c.b * E_pad;
    const float2* rb = rec + (size_t)c.b * (E_max + 1) * N + n;
    const float* tt = ev_t + (size_t)c.b * E_max;
    const Stage st = stage_segment(c, ev_src + (size_t)c.b * E_max + c.k0, d + c.k0, WT, C_in, N, lad, nullptr);
#pragma unroll
    for (int h = 0; h < kSrcRegs; ++h) {
        const int e = h * kWave + lane;
        if (e < c.cnt) lt[e] = tt[c.k0 + e];
    }
    wave_lds_sync();
    const size_t bn = (size_t)c.b * N + n;
    const double2 G = c.live ? coef[bn] : make_double2(0.0, 0.0);
    const double sc = scale[0];
    const int k1 = c.k0 + c.cnt - 1;
    // (P, Q) at event k1: the later segments' part, and in the last segment
    // the open interval after the sample's last event
    const double2 ci = cin[((size_t)c.b * S + c.seg) * N + n];
    double Pm = ci.x, Ps = ci.y;
    const bool last = k1 + 1 == c.nb;
    const Decay en = last ? Decay{0.0, 0.0, 0.0, 0.0} : d[k1 + 1];
    RecTerm tn = rec_term(rb[(size_t)(k1 + 1) * N], G, en.A, en.D);     // the interval after event k1
    if (last) {
        Pm = fma(tn.mu, tn.em, Pm);
        Ps = fma(tn.mu, tn.es, Ps);
    }
    // the lane's spikes in this segment (out_k in [k0, k1]), last first; the
    // first kRegPre of them and their upstream gradients are held in
    // registers and written back after the walk, so that the walk itself
    // loads nothing but the next group's weights and records.  A wave where
    // some lane has more spikes in the segment (a burst) reads and updates
    // them in the walk instead.
    const float* ts = out_t + bn * (size_t)m.s_max;
    const int32_t* ks = out_k + bn * (size_t)m.s_max;
    float* gsp = grad_spike + bn * (size_t)m.s_max;
    int sp = 0;                                   // spikes with out_k <= k1 (out_k is non-decreasing)
    {
        int hi = c.live ? min(out_n[bn], m.s_max) : 0;
        while (sp < hi) {
            const int mid = (sp + hi) >> 1;
            if (ks[mid] <= k1) sp = mid + 1; else hi = mid;
        }
    }
    int pk[kRegPre];
    float pt[kRegPre], pg[kRegPre];
#pragma unroll
    for (int u = 0; u < kRegPre; ++u) {
        const int q = sp - 1 - u;
        const int kq = q >= 0 ? ks[q] : -1;
        const bool in = kq >= c.k0;
        pk[u] = in ? kq : -1;
        pt[u] = in ? ts[q] : 0.0f;
        pg[u] = in ? gsp[q] : 0.0f;
    }
    const int qx = sp - 1 - kRegPre;
    const bool burst = __ballot(qx >= 0 && ks[max(qx, 0)] >= c.k0) != 0ull;
    double* gt = gtp + ((size_t)c.tile * B + c.b) * E_max + c.k0;
    const double kap = m.kappa, sk = -(m.dth * m.inv_tm);
    auto load_rec = [&](int g, float2 (&r)[kGrp]) {
#pragma unroll
        for (int jj = 0; jj < kGrp; ++jj) r[jj] = rb[(size_t)(c.k0 + min(g * kGrp + jj, c.cnt - 1)) * N];
    };
    auto walk = [&](auto burst_tag) {
        constexpr bool kBurst = decltype(burst_tag)::value;
        int knext = kBurst && sp > 0 ? ks[sp - 1] : -1;
        // the walk of group g (its dL/dt terms ca and fixed-point dL/dW terms ga)
        auto group = [&](int g, const float (&w)[kGrp][1], const float2 (&r)[kGrp], double (&ca)[kGrp],
                         long long (&ga)[kGrp]) {
#pragma unroll
            for (int jj = kGrp - 1; jj >= 0; --jj) {
                const int e = g * kGrp + jj;
                ca[jj] = 0.0;
                ga[jj] = 0;
                if (e >= c.cnt) continue;
                const int k = c.k0 + e;
                const double2 ad = lad[e];
                const RecTerm t = rec_term(r[jj], G, ad.x, ad.y);        // the interval that event e closes
                double gk = (double)w[jj][0] * kap * (Pm * m.inv_tm - Ps * m.inv_ts);
                gk = fma(tn.mu, tn.vs, gk);              // adds 0 unless the argmax is that end
                gk = fma(t.mu, t.ve, gk);
                const long long gq = llrint(kap * (Pm - Ps) * sc);
                ca[jj] = c.live ? gk : 0.0;
                ga[jj] = c.live ? gq : 0ll;
                // spikes between events k - 1 and k: their upstream gradient
                // from P at event k
                if constexpr (kBurst) {
                    if (c.live && knext == k) {
                        const double tk = (double)lt[e];
                        while (sp > 0 && ks[sp - 1] == k) {
                            --sp;
                            gsp[sp] += (float)(sk * Pm * exp(-(tk - (double)ts[sp]) * m.inv_tm));
                        }
                        knext = sp > 0 ? ks[sp - 1] : -1;
                    }
                } else {
                    bool hit = false;
#pragma unroll
                    for (int u = 0; u < kRegPre; ++u) hit |= pk[u] == k;
                    if (__ballot(hit)) {
                        const double tk = (double)lt[e];
#pragma unroll
                        for (int u = 0; u < kRegPre; ++u)
                            if (pk[u] == k) pg[u] += (float)(sk * Pm * exp(-(tk - (double)pt[u]) * m.inv_tm));
                    }
                }
                if (e > 0) {
                    Pm = fma(t.mu, t.em, Pm * ad.x);
                    Ps = fma(t.mu, t.es, Ps * ad.y);
                }
                tn = t;
            }
        };
        // group g's dL/dW terms (zero terms included, so that every group
        // issues the same memory operations) and its dL/dt sums
        auto flush = [&](int g, const double (&ca)[kGrp], const long long (&ga)[kGrp]) {
            const int oreg = g * kGrp < kWave ? st.off[0] : st.off[kSrcRegs - 1];
#pragma unroll
            for (int jj = 0; jj < kGrp; ++jj) {
                const int roff = __builtin_amdgcn_readlane(oreg, (g * kGrp + jj) & (kWave - 1));
                atomicAdd((unsigned long long*)&gw[(size_t)(roff >> 2) + (size_t)n], (unsigned long long)ga[jj]);
            }
            const double sum = group_sum8(ca, lane);
            const int j = ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
            if ((lane & 7) == 0 && g * kGrp + j < c.cnt) gt[g * kGrp + j] = sum;
        };
        // Groups from the last backwards with two groups' weights and records
        // in flight; a group's loads are issued before the atomics of the
        // group walked just before, so that no wait for loads waits for
        // atomics (the memory counter is in order).  Loads past the first
        // group re-read it.
        const int ng = (c.cnt + kGrp - 1) / kGrp;
        float wa[kGrp][1], wb[kGrp][1];
        float2 ra[kGrp], rbuf[kGrp];
        double ca[kGrp];
        long long ga[kGrp];
        load_grp<1>(st, (ng - 1) * kGrp, wa);
        load_rec(ng - 1, ra);
        load_grp<1>(st, max(ng - 2, 0) * kGrp, wb);
        load_rec(max(ng - 2, 0), rbuf);
        for (int g = ng - 1; g >= 0; g -= 2) {
            group(g, wa, ra, ca, ga);
            load_grp<1>(st, max(g - 2, 0) * kGrp, wa);
            load_rec(max(g - 2, 0), ra);
            flush(g, ca, ga);
            if (g < 1) break;
            group(g - 1, wb, rbuf, ca, ga);
            load_grp<1>(st, max(g - 3, 0) * kGrp, wb);
            load_rec(max(g - 3, 0), rbuf);
            flush(g - 1, ca, ga);
        }
    };
    if (burst) {
        walk(std::true_type{});
    } else {
        walk(std::false_type{});
#pragma unroll
        for (int u = 0; u < kRegPre; ++u)
            if (pk[u] >= 0) gsp[sp - 1 - u] = pg[u];
    }
}

// The same walk with dL/dW in LDS: a workgroup takes 16 neurons of all C_in
// channels (kTileRow bytes of LDS per channel) and every slices-th quadruple of
// (segment, sample) items, one item per row of 16 lanes, and adds its sums to
// gw once at the end.  Lane i of a row holds the decays and offsets of event i
// of the current 16 (counted from the segment's last event backwards) and sends
// them to its row by DPP.  Without the LDS the walk waits for its global 64-bit
// atomics, 184 G/s on the whole chip however they are spread (about 20 times
// that in LDS): 700 -> 512, B = 128, 10 k events, 4.05 -> 2.33 ms, now bound by
// VALU issue (64 % busy, two waves per SIMD; three spill: 5.87 ms).
constexpr int kTileN = 16, kTileRow = kTileN * (int)sizeof(long long), kTileWaves = 8;

template <bool kTime>
__global__ __launch_bounds__(kWave * kTileWaves) void k_regg_tile(
    const float* __restrict__ ev_t, const int32_t* __restrict__ ev_src, const int32_t* __restrict__ ev_n, int B,
    int E_max, int E_pad, const float* __restrict__ WT, int C_in, int N, int S, Model m,
    const Decay* __restrict__ dec, const float2* __restrict__ rec, const double2* __restrict__ coef,
    const double2* __restrict__ cin, const float* __restrict__ out_t, const int32_t* __restrict__ out_n,
    const int32_t* __restrict__ out_k, const double* __restrict__ scale, long long* __restrict__ gw,
    double* __restrict__ gtp, float* __restrict__ grad_spike)
{
    extern __shared__ unsigned long long s_gw[];
    const int lane = (int)threadIdx.x % kWave, wv = (int)threadIdx.x / kWave;
    const int rl = lane % kTileN;
    const int nt = (int)blockIdx.x * kTileN + rl;
    const bool in_n = nt < N;
    const int n = in_n ? nt : N - 1;
    for (int x = (int)threadIdx.x; x < C_in * kTileN; x += kWave * kTileWaves) s_gw[x] = 0ull;
    __syncthreads();
    const double sc = scale[0], kap = m.kappa, sk = -(m.dth * m.inv_tm);
    const size_t rstep = (size_t)N * sizeof(float2);
    const int quads = (int)(((long long)B * S + 3) / 4);
    const __amdgpu_buffer_rsrc_t wrs =
        __builtin_amdgcn_make_buffer_rsrc((void*)WT, (short)0, (int)((uint32_t)C_in * (uint32_t)N * 4u), kRsrcWord3);
    for (int q = (int)blockIdx.y * kTileWaves + wv; q < quads; q += (int)gridDim.y * kTileWaves) {
        // a row's item: segment-major, so that the four rows are four samples at
        // the same segment, of equal length but for the samples' last segments
        const long long item = (long long)q * 4 + lane / kTileN;
        const int seg = (int)(item / B), b = (int)(item % B);
        const int nb = item < (long long)B * S ? clamp_count(ev_n[b], E_max) : 0;
        const int k0 = nb > seg * kSeg ? seg * kSeg : 0;
        const int cnt = nb > seg * kSeg ? min(kSeg, nb - k0) : 0;
        if (!__ballot(cnt > 0)) continue;
        const bool live = in_n && cnt > 0;
        const int k1 = k0 + max(cnt - 1, 0);
        const Decay* d = dec + (size_t)b * E_pad;
        const int32_t* ss = ev_src + (size_t)b * E_max;
        const float2* rb = rec + (size_t)b * (E_max + 1) * N + n;
        const size_t bn = (size_t)b * N + n;
        double2 G = coef[bn];
        if (!live) G = make_double2(0.0, 0.0);
        // (P, Q) at event k1, as in k_regg_walk
        const double2 ci = cin[((size_t)b * S + min(seg, S - 1)) * N + n];
        double Pm = ci.x, Ps = ci.y;
        const bool last = k1 + 1 >= nb;
        Decay en{0.0, 0.0, 0.0, 0.0};
        if (!last) en = d[k1 + 1];
        RecTerm tn = rec_term(rb[(size_t)(k1 + 1) * N], G, en.A, en.D);
        if (last) {
            Pm = fma(tn.mu, tn.em, Pm);
            Ps = fma(tn.mu, tn.es, Ps);
        }
        // the lane's spikes of the segment, last first, by their event's place i
        // counted back from k1 (-1: none); bursts read them in the walk
        const float* ts = out_t + bn * (size_t)m.s_max;
        const int32_t* ks = out_k + bn * (size_t)m.s_max;
        float* gsp = grad_spike + bn * (size_t)m.s_max;
        int sp = 0;
        {
            int hi = live ? min(out_n[bn], m.s_max) : 0;
            while (sp < hi) {
                const int mid = (sp + hi) >> 1;
                if (ks[mid] <= k1) sp = mid + 1; else hi = mid;
            }
        }
        int pk[kRegPre];
        float pt[kRegPre], pg[kRegPre];
#pragma unroll
        for (int u = 0; u < kRegPre; ++u) {
            const int x = sp - 1 - u;
            const int kq = x >= 0 ? ks[x] : -1;
            const bool in = kq >= k0;
            pk[u] = in ? k1 - kq : -1;
            pt[u] = in ? ts[x] : 0.0f;
            pg[u] = in ? gsp[x] : 0.0f;
        }
        const int qx = sp - 1 - kRegPre;
        const bool burst = __ballot(qx >= 0 && ks[max(qx, 0)] >= k0) != 0ull;
        double* gt = nullptr;
        if constexpr (kTime) gt = gtp + ((size_t)blockIdx.x * B + b) * E_max + k1;
        const float* te = ev_t + (size_t)b * E_max;
        struct Meta {
            double A, D;
            int wo, lo;
        };
        // event 16 ch + rl of the row (past its first event that one again)
        auto load_meta = [&](int ch) {
            const int k = k0 + max(cnt - 1 - ch * kTileN - rl, 0);
            const double2 ad = *reinterpret_cast<const double2*>(&d[k]);
            const int src = clamp_src(ss[k], C_in);
            return Meta{ad.x, ad.y, src * N * 4, src * kTileN};
        };
        const char* rp = reinterpret_cast<const char*>(rb + (size_t)k1 * N);
        int left = cnt - 1;                       // records after the one at rp
        auto load_half = [&](const Meta& me, auto half, float (&w)[kGrp], float2 (&r)[kGrp]) {
            auto one = [&](auto jj) {
                constexpr int J = decltype(jj)::value;
                const int off = row_bcast<decltype(half)::value * kGrp + J>(me.wo) + n * 4;
                w[J] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wrs, off, 0, 0));
                r[J] = *reinterpret_cast<const float2*>(rp);
                rp -= left > 0 ? rstep : 0;
                --left;
            };
            one(std::integral_constant<int, 0>{}); one(std::integral_constant<int, 1>{});
            one(std::integral_constant<int, 2>{}); one(std::integral_constant<int, 3>{});
            one(std::integral_constant<int, 4>{}); one(std::integral_constant<int, 5>{});
            one(std::integral_constant<int, 6>{}); one(std::integral_constant<int, 7>{});
        };
        int inext = pk[0];                        // the place of the lane's next spike, -1: none
        auto half_walk = [&](int i0, const Meta& me, auto half, const float (&w)[kGrp], const float2 (&r)[kGrp]) {
            double ca[kGrp];
            auto one = [&](auto jj) {
                constexpr int J = decltype(jj)::value, L = decltype(half)::value * kGrp + J;
                const int i = i0 + J;
                const double A = row_bcast<L>(me.A), D = row_bcast<L>(me.D);
                const bool valid = live && i < cnt;
                const RecTerm t = rec_term(r[J], G, A, D);
                if constexpr (kTime) {
                    double gk = (double)w[J] * kap * (Pm * m.inv_tm - Ps * m.inv_ts);
                    gk = fma(tn.mu, tn.vs, gk);
                    gk = fma(t.mu, t.ve, gk);
                    ca[J] = valid ? gk : 0.0;
                }
                const long long gq = llrint(kap * (Pm - Ps) * sc);
                const int at = row_bcast<L>(me.lo) + rl;
                if (valid) atomicAdd(&s_gw[at], (unsigned long long)gq);
                if (__ballot(inext == i)) {       // spikes between events i + 1 and i
                    asm volatile("");
                    if (inext == i) {
                        const double tk = (double)te[k1 - i];
                        if (burst) {
                            while (sp > 0 && ks[sp - 1] == k1 - i) {
                                --sp;
                                gsp[sp] += (float)(sk * Pm * exp(-(tk - (double)ts[sp]) * m.inv_tm));
                            }
                            inext = sp > 0 && ks[sp - 1] >= k0 ? k1 - ks[sp - 1] : -1;
                        } else {
                            int nx = 0x7fffffff;
#pragma unroll
                            for (int u = 0; u < kRegPre; ++u) {
                                if (pk[u] == i) pg[u] += (float)(sk * Pm * exp(-(tk - (double)pt[u]) * m.inv_tm));
                                else if (pk[u] > i) nx = min(nx, pk[u]);
                            }
                            inext = nx;
                        }
                    }
                }
                Pm = fma(t.mu, t.em, Pm * A);
                Ps = fma(t.mu, t.es, Ps * D);
                tn = t;
            };
            one(std::integral_constant<int, 0>{}); one(std::integral_constant<int, 1>{});
            one(std::integral_constant<int, 2>{}); one(std::integral_constant<int, 3>{});
            one(std::integral_constant<int, 4>{}); one(std::integral_constant<int, 5>{});
            one(std::integral_constant<int, 6>{}); one(std::integral_constant<int, 7>{});
            if constexpr (kTime) {
                const double sum = row_sum8(ca, lane);
                const int i = i0 + rl / 2;
                if ((rl & 1) == 0 && i < cnt) gt[-i] = sum;
            }
        };
        // 16 events at a time; the next eight's weights and records, and the
        // next 16's decays and sources, are in flight
        using H0 = std::integral_constant<int, 0>;
        using H1 = std::integral_constant<int, 1>;
        int most = cnt;
        most = max(most, __shfl_xor(most, 16, kWave));
        most = max(most, __shfl_xor(most, 32, kWave));
        most = __builtin_amdgcn_readfirstlane(most);
        Meta m0 = load_meta(0), m1 = load_meta(1);
        float wa[kGrp], wb[kGrp];
        float2 ra[kGrp], rbuf[kGrp];
        load_half(m0, H0{}, wa, ra);
        for (int i0 = 0; i0 < most; i0 += kTileN) {
            const Meta m2 = load_meta(i0 / kTileN + 2);
            load_half(m0, H1{}, wb, rbuf);
            half_walk(i0, m0, H0{}, wa, ra);
            load_half(m1, H0{}, wa, ra);
            half_walk(i0 + kGrp, m0, H1{}, wb, rbuf);
            m0 = m1;
            m1 = m2;
        }
        if (!burst) {
#pragma unroll
            for (int u = 0; u < kRegPre; ++u)
                if (pk[u] >= 0) gsp[sp - 1 - u] = pg[u];
        }
    }
    __syncthreads();
    for (int x = (int)threadIdx.x; x < C_in * kTileN; x += kWave * kTileWaves) {
        const int c = x / kTileN, nn = (int)blockIdx.x * kTileN + x % kTileN;
        const unsigned long long v = s_gw[x];
        if (v != 0ull && nn < N) atomicAdd((unsigned long long*)&gw[(size_t)c * N + nn], v);
    }
}

// Whether a call's dL/dW is summed in LDS (k_regg_tile): the block fits, and the
// walk is long enough to pay for clearing and adding the blocks (C_in x N elements
// per slice).  Whole calls, global atomics against LDS: 1.0 M terms (B = 4,
// 1000 events, N = 256) 81 against 93 us, 2.5 M 103 against 119 us, 8.2 M
// (B = 8, 2000 events, N = 512) 131 against 122 us, 41 M 434 against 345 us.
constexpr size_t kLdsMax = (size_t)160 << 10;        // LDS per CU
constexpr int kCUs = 256;

static bool reg_tiled(int B, int E_max, int C_in, int N)
{
    return (size_t)C_in * kTileRow <= kLdsMax && (size_t)B * E_max * N >= ((size_t)1 << 22);
}

// Fixed point -> float32 dL/dW; dL/dt summed over the tiles in order (0 past
// each sample's last event).
__global__ __launch_bounds__(256) void k_regg_convert(const long long* __restrict__ gw,
                                                     const double* __restrict__ scale, size_t nW,
                                                     float* __restrict__ grad_WT, const double* __restrict__ gtp,
                                                     const int32_t* __restrict__ ev_n, int B, int E_max, int tiles,
                                                     float* __restrict__ grad_ev_t)
{
    const size_t gtid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, gs = (size_t)gridDim.x * blockDim.x;
    const double inv = 1.0 / scale[0];
    for (size_t x = gtid; x < nW; x += gs) grad_WT[x] = (float)((double)gw[x] * inv);
    if (!grad_ev_t) return;
    const size_t nT = (size_t)B * E_max;
    for (size_t x = gtid; x < nT; x += gs) {
        const int b = (int)(x / (size_t)E_max), k = (int)(x % (size_t)E_max);
        double g = 0.0;
        if (k < clamp_count(ev_n[b], E_max))
            for (int t = 0; t < tiles; ++t) g += gtp[(size_t)t * nT + x];
        grad_ev_t[x] = (float)g;
    }
}

struct RegGradLayout {
    RegLayout r;
    size_t rec, counts, gates, coef, musum, scale, local, cin, gw, gtp, total;
};

static RegGradLayout reg_grad_layout(int B, int E_max, int C_in, int N)
{
    RegGradLayout G;
    G.r = reg_layout(B, E_max, N);
    size_t off = G.r.total;
    auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    const size_t BS = (size_t)B * G.r.f.S;
    const int tn = reg_tiled(B, E_max, C_in, N) ? kTileN : kWave, tiles = (N + tn - 1) / tn;
    G.rec = take((size_t)B * ((size_t)E_max + 1) * N * sizeof(float2));
    G.counts = take((size_t)B * N * sizeof(double2));
    G.gates = take((size_t)N * sizeof(double2));
    G.coef = take((size_t)B * N * sizeof(double2));
    G.musum = take((size_t)B * N * sizeof(double));
    G.scale = take(sizeof(double));
    G.local = take(BS * N * sizeof(double4));
    G.cin = take(BS * N * sizeof(double2));
    G.gw = take((size_t)C_in * N * sizeof(long long));
    G.gtp = take((size_t)tiles * B * E_max * sizeof(double));
    G.total = off + 256;
    return G;
}

}  // namespace lif

extern "C" size_t lif_spike_count_reg_backward_workspace_size(int B, int E_max, int C_in, int N_out)
{
    if (B < 0 || E_max < 0 || C_in < 1 || N_out < 1) return 0;
    return lif::reg_grad_layout(B, E_max, C_in, N_out).total;
}

extern "C" int lif_spike_count_reg_backward(const float* ev_t, const int32_t* ev_src, const int32_t* ev_n, int B,
                                            int E_max, const float* WT, int C_in, int N_out, const lif_params* p,
                                            const float* out_t, const int32_t* out_n, const int32_t* out_k,
                                            double c_target, double lam_reg, double lam_over, float* loss,
                                            float* grad_spike, float* grad_WT, float* grad_ev_t, void* ws,
                                            size_t ws_bytes, lif_stream_t stream_)
{
    using namespace lif;
    int rc = validate_forward_args(ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, p, out_t, out_n, out_n);
    if (rc) return rc;
    if (!out_k || !grad_spike || !grad_WT || !ws || !(c_target > 0.0) || !isfinite(c_target) ||
        !isfinite(lam_reg) || !isfinite(lam_over))
        return LIF_ERR_ARG;
    const RegGradLayout G = reg_grad_layout(B, E_max, C_in, N_out);
    if (ws_bytes < G.total) return LIF_ERR_WORKSPACE;
    const int tl = (N_out + kWave - 1) / kWave;
    const size_t items_max = (size_t)B * G.r.f.S * tl;
    if (items_max > 0x7fffffff || B > 65535) return LIF_ERR_SIZE;
    hipStream_t stream = (hipStream_t)stream_;
    const Model m = make_model(*p);
    char* base = (char*)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
    const RegLayout& R = G.r;
    FwdPtrs P{};
    P.dec = (Decay*)(base + R.f.dec);
    P.segm = (double2*)(base + R.f.segm);
    P.carry = (double2*)(base + R.f.carry);
    P.mask = (uint32_t*)(base + R.f.mask);
    P.counters = (uint32_t*)(base + R.f.counters);
    P.pool_count = P.counters;
    P.nwork = P.counters + (size_t)B * kCtr;
    P.listed = (uint32_t*)(base + R.f.listed);
    P.work = (uint32_t*)(base + R.f.work);
    P.pool = (double2*)(base + R.f.pool);
    double4* part = (double4*)(base + R.part);
    double* ub = (double*)(base + R.ub);
    double* ob = (double*)(base + R.ob);
    int32_t* st = (int32_t*)(base + R.status);
    const bool tiled = reg_tiled(B, E_max, C_in, N_out);
    const int gtn = tiled ? kTileN : kWave, gtiles = (N_out + gtn - 1) / gtn;   // of the walk back
    float2* rec = (float2*)(base + G.rec);
    double2* counts = (double2*)(base + G.counts);
    double2* gates = (double2*)(base + G.gates);
    double2* coef = (double2*)(base + G.coef);
    double* musum = (double*)(base + G.musum);
    double* scale = (double*)(base + G.scale);
    double4* local = (double4*)(base + G.local);
    double2* cin = (double2*)(base + G.cin);
    long long* gw = (long long*)(base + G.gw);
    double* gtp = (double*)(base + G.gtp);
    const size_t nn = (size_t)B * N_out, nW = (size_t)C_in * N_out;
    const unsigned wblocks = (unsigned)((items_max + kWalkWaves - 1) / kWalkWaves);
    if (items_max > 0) {
        switch (pick_npl(WT, N_out)) {
        case 4: launch_walks<4>(R.f, P, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, m, st, false, nullptr, nullptr,
                                nullptr, nullptr, stream, false); break;
        case 2: launch_walks<2>(R.f, P, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, m, st, false, nullptr, nullptr,
                                nullptr, nullptr, stream, false); break;
        default: launch_walks<1>(R.f, P, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, m, st, false, nullptr,
                                 nullptr, nullptr, nullptr, stream, false); break;
        }
        auto walk = [&](auto kern) {
            TIMED_LAUNCH("reg_walk", kern, dim3(wblocks), dim3(kWave * kWalkWaves), 0, stream, ev_t, ev_src, ev_n,
                         E_max, R.f.E_pad, WT, C_in, N_out, tl, R.f.S, (int)items_max, m, P.dec, P.carry, out_t, out_n,
                         out_k, part, rec, local);
        };
        if (grad_ev_t) walk(k_reg_walk<true, true>);
        else walk(k_reg_walk<true, false>);
    }
    if (nn)
        TIMED_LAUNCH("reg_reduce", k_reg_reduce, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, stream, part, ev_n,
                     B, E_max, N_out, R.f.S, m.th, ub, ob, nullptr, nullptr, counts);
    if (B > 0)
        launch_reg_loss(ub, ob, out_n, B, N_out, m.s_max, c_target, loss, gates, stream);
    size_t work = nW > nn ? nW : nn;
    size_t blocks = (work + 255) / 256;
    blocks = blocks < 1 ? 1 : (blocks > 2048 ? 2048 : blocks);
    TIMED_LAUNCH("regg_coef", k_regg_coef, dim3((unsigned)blocks), dim3(256), 0, stream, counts, gates, out_n, B,
                 N_out, m.s_max, c_target, lam_reg, lam_over, coef, musum, gw, nW);
    TIMED_LAUNCH("regg_scale", k_regg_scale, dim3(1), dim3(kScaleThreads), 0, stream, musum, nn, ev_n, B, E_max,
                 m.kappa, scale);
    if (items_max > 0) {
        TIMED_LAUNCH("regg_carry", k_regg_carry, dim3((unsigned)tl, (unsigned)B), dim3(kWave), 0, stream, ev_n, E_max,
                     N_out, R.f.S, P.segm, local, coef, cin);
        if (tiled) {
            const size_t lds = (size_t)C_in * kTileRow;
            const long long quads = ((long long)B * R.f.S + 3) / 4;
            const int per = (int)((quads + kTileWaves - 1) / kTileWaves);
            // slices of the items per tile: the fewest rounds of one workgroup per CU
            // in units of a slice (a workgroup's sums cost C_in x 16 atomics, so
            // no more than four rounds, and every wave has an item)
            int slices = 1;
            for (int q = 2; q <= per && (long long)q * gtiles <= 4 * kCUs; ++q)
                if ((long long)((gtiles * q + kCUs - 1) / kCUs) * slices < (long long)((gtiles * slices + kCUs - 1) / kCUs) * q)
                    slices = q;
            auto walk = [&](auto kern) {
                // the attribute belongs to the kernel, not to the call: always the
                // same value, so that calls of other threads do not lower it
                if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax) !=
                    hipSuccess)
                    return false;
                TIMED_LAUNCH("regg_walk", kern, dim3((unsigned)gtiles, (unsigned)slices), dim3(kWave * kTileWaves), lds,
                             stream, ev_t, ev_src, ev_n, B, E_max, R.f.E_pad, WT, C_in, N_out, R.f.S, m, P.dec, rec,
                             coef, cin, out_t, out_n, out_k, scale, gw, gtp, grad_spike);
                return true;
            };
            if (!(grad_ev_t ? walk(k_regg_tile<true>) : walk(k_regg_tile<false>))) return LIF_ERR_HIP;
        } else {
            TIMED_LAUNCH("regg_walk", k_regg_walk, dim3(wblocks), dim3(kWave * kWalkWaves), 0, stream, ev_t, ev_src, ev_n,
                         B, E_max, R.f.E_pad, WT, C_in, N_out, tl, R.f.S, (int)items_max, m, P.dec, rec, coef, cin, out_t,
                         out_n, out_k, scale, gw, gtp, grad_spike);
        }
    }
    work = nW > (size_t)B * E_max ? nW : (size_t)B * E_max;
    blocks = (work + 255) / 256;
    blocks = blocks < 1 ? 1 : (blocks > 2048 ? 2048 : blocks);
    TIMED_LAUNCH("regg_convert", k_regg_convert, dim3((unsigned)blocks), dim3(256), 0, stream, gw, scale, nW, grad_WT,
                 gtp, ev_n, B, E_max, gtiles, grad_ev_t);
    return check_launch();
}

// ---------------------------------------------------------------------------
// Forward pass without a caller workspace: the workspace is a fixed array in
// device memory, one per GPU, held from the library's load until the process
// ends.  Its device address is looked up once per device (with that device
// current) and kept; host code passes only that address to kernels.
// ---------------------------------------------------------------------------
#include <mutex>

namespace lif {

constexpr size_t kScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices];

// The current device's address of the scratch array.
static int scratch_address(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LIF_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LIF_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return LIF_OK;
}

}  // namespace lif

extern "C" size_t lif_layer_forward_noalloc_max_bytes(void) { return lif::kScratchBytes; }

extern "C" int lif_layer_forward_noalloc(const float* ev_t, const int32_t* ev_src, const int32_t* ev_n, int B,
                                         int E_max, const float* WT, int C_in, int N_out, const lif_params* p,
                                         float* out_t, int32_t* out_n, float* out_i, int32_t* out_k,
                                         int32_t* status, lif_stream_t stream)
{
    using namespace lif;
    int rc = validate_forward_args(ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, p, out_t, out_n, status);
    if (rc) return rc;
    lif_params q = *p;
    // the layout without pool entries must fit; the default pool is cut to
    // what the array holds (sub-blocks past it take the rebuild path, with
    // identical results), a pool size the caller set must fit as it is
    if (fwd_layout(B, E_max, N_out, 0).total > kScratchBytes) return LIF_ERR_SIZE;
    if (q.pool_cap < 0) {
        size_t cap = fwd_layout(B, E_max, N_out, -1).pool_cap;
        if (cap > 0x7fffffff) cap = 0x7fffffff;
        size_t lo = 0, hi = cap;                      // largest fitting slice size
        while (lo < hi) {
            const size_t mid = hi - (hi - lo) / 2;
            if (fwd_layout(B, E_max, N_out, (int)mid).total <= kScratchBytes) lo = mid;
            else hi = mid - 1;
        }
        q.pool_cap = (int32_t)lo;
    }
    if (fwd_layout(B, E_max, N_out, q.pool_cap).total > kScratchBytes) return LIF_ERR_SIZE;
    void* ws = nullptr;
    rc = scratch_address(&ws);
    if (rc) return rc;
    return forward_impl(false, ev_t, ev_src, ev_n, B, E_max, WT, C_in, N_out, &q, out_t, out_n, out_i, out_k, status,
                        ws, kScratchBytes, (hipStream_t)stream);
}
