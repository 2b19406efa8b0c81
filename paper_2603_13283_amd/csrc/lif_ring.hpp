// lif_ring.hpp -- the resolve pass of the forward for calls with few flagged
// sub-blocks: one workgroup per neuron, whose staging waves prepare windows of
// intervals in a ring of LDS buffers ahead of the wave that follows the
// neuron's serial chain of spikes.  Included by lif_forward.hip after the
// helpers that both resolve passes share.
#pragma once

namespace lif {

// A wait inside a workgroup that does not end within this many polls is an
// internal error (reported in the status words instead of waiting for ever).
constexpr int kSpinLimit = 1 << 22;

// ---------------------------------------------------------------------------
// Resolve pass by rings: one workgroup of four waves per neuron that has
// flagged sub-blocks (the work lists of the check pass).  Intervals outside flagged
// sub-blocks provably hold no spike.  The flagged sub-blocks are taken in
// time order:
//   * Candidate list: per chunk of kChunkEv events, the sub-block masks (two
//     segments per lane) are compacted into a time-ordered list in LDS with
//     one wave prefix sum, with the pool slot of every candidate.
//   * Windows of kWinCand candidates (kWinIv intervals) in a ring of kRing
//     LDS buffers: the staging waves (waves 1..3, windows in turn) walk the
//     window's sub-blocks and fill its buffer while the chain wave (wave 0)
//     works on an earlier one; a ready word per buffer and a consumed count
//     hand the buffers over (no barrier per window).
//   * The chain searches a window 64 intervals at a time: interval i crosses
//     iff key_i >= K, the key of the current reset deficit (crossing_key), so
//     one ballot finds the earliest crossing.  Its spike time is solved
//     wave-uniform, the deficit and K are raised, and the search resumes at
//     the same interval (a second spike in it, App. E.2 restart).
//   * The open interval after the sample's last event is one more slot of
//     the window holding the sample's last sub-block.
//   * Spikes are buffered in LDS and written out kWave at a time.
// ---------------------------------------------------------------------------
constexpr int kWinIv = kWinCand * kSub;          // intervals per window
static_assert(kWinIv == kWave, "one window interval per lane");
constexpr int kOpenIv = kWinIv;                  // window slot of the open interval
constexpr int kRing = 8;                         // window buffers
constexpr int kRingWaves = 4;                    // the chain wave and three staging waves

struct WinBuf {
    double key[kWinIv + 1];                      // crossing key (NaN: no interval)
    double v0[kWinIv + 1], i0[kWinIv + 1];       // no-reset (V, I) at the interval start
    float t0[kWinIv + 1];                        // interval start (time of the event before it; 0 for the first)
    float t1[kWinIv + 1];                        // interval end (its closing event's time)
};

struct RingLds {
    uint32_t cand[kCandCap];                     // (segment in chunk << 3) | sub-block
    uint32_t slot[kCandCap];                     // pool slot of each candidate (kNoSlot: none)
    WinBuf win[kRing];
    double sp_t0[kWave], sp_y[kWave];            // spike buffer: interval start, e^{-u/tm},
    float si[kWave];                             // I at the spike,
    int32_t sk[kWave];                           // events consumed before the spike
    double open_len;                             // length of the open interval (t_end - last event)
    int ntot;                                    // candidates of the chunk (chain wave -> all)
    int ready[kRing];                            // 1 + window index staged in each buffer
    double kmax[kRing];                          // largest key of each buffer's window (NaN keys left out)
    int consumed;                                // windows the chain has finished
    int stop;                                    // the chain reached s_max
    unsigned long long kpub;                     // bits of the chain's current deficit key K
};

__device__ __forceinline__ int lds_load(const int* p)
{
    return __hip_atomic_load(const_cast<int*>(p), __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void lds_store(int* p, int v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A staging wave's window: candidates c0 .. c0 + kWinCand - 1 of the chunk,
// lane l taking interval j = l % kSub of candidate c0 + l / kSub.  Every lane
// loads its own interval's closing event (source, decays, times) and its
// candidate's entering state (stage_load, issued before the wait for the
// window's buffer), then its weight; the 16
// lanes of a candidate (one row) take the no-reset states of the sub-block by
// a scan of its event maps (row_states), lane j the state at its interval's
// start (after event j - 1) and end, and the interval's crossing key.  Candidates past the pool's capacity take
// their entering state from rebuild_entry.  open_last: the window holds the
// sample's last sub-block, and the open interval after its last event is
// staged too.
struct StageIn {
    int k, sc;
    bool ok;
    uint32_t slot;
    double A, D;
    float ta, tb;
    double2 u0;
};

__device__ __forceinline__ StageIn stage_load(const RingLds& sh, int c0, int tot, int seg0, int nb,
                                              const float* __restrict__ tt, const int32_t* __restrict__ src,
                                              const Decay* __restrict__ d, const double2* __restrict__ pool)
{
    const int lane = (int)threadIdx.x % kWave;
    const int j = lane % kSub, r = lane / kSub;
    const int c = c0 + r;
    const int cc = min(c, tot - 1);
    const uint32_t cw = sh.cand[cc];
    StageIn in;
    in.slot = sh.slot[cc];
    const int kq = (seg0 + (int)(cw >> 3)) * kSeg + (int)(cw & 7u) * kSub;
    in.ok = c < tot && kq + j < nb;
    in.k = min(kq + j, nb - 1);
    in.sc = src[in.k];
    const Decay dk = d[in.k];
    in.A = dk.A;
    in.D = dk.D;
    in.ta = tt[max(in.k - 1, 0)];
    in.tb = tt[in.k];
    in.u0 = pool[in.slot != kNoSlot ? in.slot : 0u];    // the pool holds at least one entry
    return in;
}

__device__ __forceinline__ void stage_window(RingLds& sh, WinBuf& w, const Model& m, const StageIn& in, int c0,
                                             int tot, int seg0, int b, int n, int nb, int S, int N, int C_in,
                                             const int32_t* __restrict__ src, const Decay* __restrict__ d,
                                             const float* __restrict__ WT, const double2* __restrict__ carry,
                                             bool open_last, double& kmax)
{
    const int lane = (int)threadIdx.x % kWave;
    const int r = lane / kSub;
    const int c = c0 + r;
    const int k = in.k, sc = in.sc;
    const bool ok = in.ok;
    const double2 ad = make_double2(in.A, in.D);
    const float ta = in.ta, tb = in.tb;
    double2 u0 = in.u0;
    const float wv = WT[(size_t)clamp_src(sc, C_in) * (size_t)N + n];
    if (__ballot(c < tot && in.slot == kNoSlot)) {
        const int nc = min(kWinCand, tot - c0);
        for (int x = 0; x < nc; ++x) {
            if (sh.slot[c0 + x] != kNoSlot) continue;
            const uint32_t cx = sh.cand[c0 + x];
            const int seg = seg0 + (int)(cx >> 3);
            const double2 cs = carry[((size_t)b * S + seg) * N + n];
            const double2 e = rebuild_entry(cs.x, cs.y, seg * kSeg, seg * kSeg + (int)(cx & 7u) * kSub, n, N, C_in,
                                            src, d, WT);
            if (x == r) u0 = e;
        }
    }
    double U0, J0, U, J;
    row_states(u0, ad.x, ad.y, wv, U0, J0, U, J);
    const double V0 = v_of(m, U0, J0), I0 = J0;
    const double V1 = v_of(m, U, J);
    const double t0 = k > 0 ? (double)ta : 0.0, t1 = (double)tb;
    // The deficit of the spikes the chain has found so far, decayed to the
    // interval's start, bounds the true deficit there from below (the chain
    // works on earlier windows, and later spikes only add to it), so the
    // no-crossing screen of the true state is safe with it (with a lower
    // bound of that deficit, exp_lower).  Most intervals of a neuron that has
    // fired fail it; the crossing key is computed only when some lane passes.
    const double Kp = __longlong_as_double((long long)__hip_atomic_load(&sh.kpub, __ATOMIC_RELAXED,
                                                                        __HIP_MEMORY_SCOPE_WORKGROUP));
    const double L = t1 - t0;
    const bool maybe = ok && L > 0.0 &&
                       (V0 - exp_lower(Kp - t0 * m.inv_tm)) + (I0 > m.th ? (I0 - m.th) * (L * m.inv_tm) : 0.0) >=
                           m.th_lo;
    double key = __builtin_nan("");
    double crit, hi, fhi;
    if (__ballot(maybe)) {
        crossing_data(m, V0, I0, V1, L, ad.x, ad.y, crit, hi, fhi);
        if (maybe) key = crossing_key(m, crit, t0);
    }
    w.key[lane] = key;
    double km = key;
    w.v0[lane] = V0;
    w.i0[lane] = I0;
    w.t0[lane] = k > 0 ? ta : 0.0f;
    w.t1[lane] = tb;
    if (open_last && ok && k == nb - 1) {
        // the open interval after the sample's last event (the same screen)
        const double Lo = m.t_end - t1;
        const bool mo = Lo > 0.0 &&
                        (V1 - exp_lower(Kp - t1 * m.inv_tm)) + (J > m.th ? (J - m.th) * (Lo * m.inv_tm) : 0.0) >=
                            m.th_lo;
        double ko = __builtin_nan("");
        if (mo) {
            open_interval_data(m, V1, J, Lo, crit, hi, fhi);
            ko = crossing_key(m, crit, t1);
        }
        w.key[kOpenIv] = ko;
        w.v0[kOpenIv] = V1;
        w.i0[kOpenIv] = J;
        w.t0[kOpenIv] = tb;
        sh.open_len = m.t_end - t1;
        km = fmax(km, w.key[kOpenIv]);
    }
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) km = fmax(km, __shfl_xor(km, off, kWave));
    if (lane == 0) kmax = km;
}

// Wave-uniform resolve state of one neuron: the reset deficit of the spikes
// so far is D(t) = dref e^{-(t - tref)/tm} for t after the latest spike,
// with tref the start of the interval that spike lies in (the deficit is
// carried in that interval's frame), and K = ln(dref) + tref/tm its key.
struct RingChain {
    int ns;              // spikes so far
    double dref, tref, K;
    double ylast;        // e^{-u/tm} of the latest spike (its offset u in its interval)
    int lastw, lasti;    // window and interval of the latest spike
    bool capped;
};

// Spikes [from, to) from the LDS buffer to the outputs (coalesced); the
// spike times t0 - tm ln y are taken here, 64 at a time, off the chain.
__device__ __forceinline__ void ring_flush(RingLds& sh, const Model& m, int from, int to, float* __restrict__ st,
                                             float* __restrict__ si, int32_t* __restrict__ sk)
{
    const int lane = (int)threadIdx.x % kWave;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (from + lane < to) {
        const int q = (from + lane) % kWave;
        st[from + lane] = (float)(sh.sp_t0[q] - m.tm * log(sh.sp_y[q]));
        if (si) si[from + lane] = sh.si[q];
        if (sk) sk[from + lane] = sh.sk[q];
    }
    __builtin_amdgcn_wave_barrier();
}

// The spike in window interval i (the earliest crossing the search found):
// the deficit at the interval start, the spike time (polynomial solve when
// tau_m / tau_s is an integer plus one, else bracketed Newton on the
// interval's closed-form maximum), the spike into the LDS buffer, and the
// raised deficit in the interval's frame.  Returns false at s_max.
template <int PI>
__device__ bool spike_at(RingLds& sh, const WinBuf& w, const Model& m, int i, int wg, int c0, int seg0, int nb,
                         RingChain& ch, float* __restrict__ st, float* __restrict__ si, int32_t* __restrict__ sk)
{
    const int lane = (int)threadIdx.x % kWave;
    const double V0 = rl_double(w.v0[i], 0), I0 = rl_double(w.i0[i], 0);
    const double t0 = (double)__builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, w.t0[i])));
    const double Dk = ch.ns > 0 ? ch.dref * exp(-(t0 - ch.tref) * m.inv_tm) : 0.0;
    const double ylo = (ch.ns > 0 && ch.lastw == wg && ch.lasti == i) ? ch.ylast : 1.0;
    const double kI = m.kappa * I0, c0v = V0 - Dk + kI;
    double y = 0.0, E1 = 0.0, E2 = 0.0;
    bool ok = false;
    if constexpr (PI > 0) {
        ok = root_poly<PI>(m, c0v, kI, ylo, y);
        if (ok) E2 = ipow<PI>(y);
    }
    if (ok) {
        E1 = rcp_refined(y);
    } else {
        // the exponential solve brackets the root in [0, hi] with the
        // interval's closed-form maximum (interval_max)
        const double L = i == kOpenIv ? sh.open_len : (double)w.t1[i] - t0;
        double A = 0.0, D = 0.0, V1 = 0.0;
        if (!isinf(L)) {
            A = exp(-L * m.inv_tm);
            D = exp(-L * m.inv_ts);
            V1 = V0 * A + unit_kernel(m, L, A) * I0;
        }
        const IntervalMax im = interval_max(m, V0, I0, V1, L, A, D);
        root_h(m, c0v, kI, 0.0, V0 - m.th - Dk, im.hi, im.Fhi - Dk, &E1, &E2, nullptr);
        y = rcp_refined(E1);
    }
    int kev = nb;
    if (i != kOpenIv) {
        const uint32_t cw = sh.cand[c0 + i / kSub];
        kev = (seg0 + (int)(cw >> 3)) * kSeg + (int)(cw & 7u) * kSub + i % kSub;
    }
    if (lane == 0) {
        const int q = ch.ns % kWave;
        sh.sp_t0[q] = t0;
        sh.sp_y[q] = y;
        sh.si[q] = (float)(I0 * (E2 * y));
        sh.sk[q] = kev;
    }
    const double Dnew = Dk + m.dth * E1;
    ch.dref = Dnew;
    ch.tref = t0;
    ch.K = log(Dnew) + t0 * m.inv_tm;
    if (lane == 0)
        __hip_atomic_store(&sh.kpub, (unsigned long long)__double_as_longlong(ch.K), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
    ch.ylast = y;
    ch.lastw = wg;
    ch.lasti = i;
    ++ch.ns;
    if (ch.ns % kWave == 0) ring_flush(sh, m, ch.ns - kWave, ch.ns, st, si, sk);
    if (ch.ns >= m.s_max) {
        ch.capped = true;
        return false;
    }
    return true;
}

// The chain wave's work on one window: its n_iv intervals (one per lane),
// then (open_last) the open interval; one call site of the spike solve keeps
// the kernel's code small.
template <int PI>
__device__ __forceinline__ void chain_window(RingLds& sh, const WinBuf& w, const Model& m, int wg, int c0, int n_iv,
                                             bool open_last, int seg0, int nb, RingChain& ch, float* __restrict__ st,
                                             float* __restrict__ si, int32_t* __restrict__ sk)
{
    const int lane = (int)threadIdx.x % kWave;
    const int nh = n_iv > 0 ? 1 : 0;
    const int hend = open_last ? nh + 1 : nh;
    const double kb = w.key[lane], ko = w.key[kOpenIv];
    for (int h = 0; h < hend; ++h) {
        const bool open = h == nh;
        const double key = open ? ko : kb;
        int from = 0;
        for (;;) {
            const unsigned long long cm = __ballot((open ? lane == 0 : lane >= from) && key >= ch.K);
            if (cm == 0ull) break;
            const int kl = __ffsll((long long)cm) - 1;
            if (!spike_at<PI>(sh, w, m, open ? kOpenIv : h * kWave + kl, wg, c0, seg0, nb, ch, st, si, sk)) return;
            from = kl;
        }
    }
}

// The four waves of the workgroup call this for the same neuron and pass the
// same barriers (one per chunk; candidate counts and the stop flag pass
// through LDS).  Returns the spike count on the chain wave, 0 on the three
// staging waves.
template <int PI>
__device__ int ring_neuron(RingLds& sh, int b, int n, const float* __restrict__ ev_t,
                              const int32_t* __restrict__ ev_src, const int32_t* __restrict__ ev_n, int E_max,
                              const float* __restrict__ WT, int C_in, int N, int E_pad, int S, const Model& m,
                              const Decay* __restrict__ dec, const double2* __restrict__ carry,
                              const uint32_t* __restrict__ mask, uint32_t pool_cap, const double2* __restrict__ pool,
                              float* __restrict__ out_t, int32_t* __restrict__ out_n, float* __restrict__ out_i,
                              int32_t* __restrict__ out_k, int32_t* __restrict__ status)
{
    const int lane = (int)threadIdx.x % kWave;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const bool chain = wv == 0;               // wave 0 resolves, waves 1.. stage (wave-uniform)
    // the chain is the critical path: its instructions go first on its SIMD
    if (chain) __builtin_amdgcn_s_setprio(3);
    // a wait that does not end within kSpinLimit polls is an internal error:
    // it is reported and the neuron is stopped instead of waiting for ever
    auto give_up = [&]() {
        if (lane == 0) atomicOr(&status[LIF_ST_FLAGS], LIF_WARN_INTERNAL);
        lds_store(&sh.stop, 1);
    };
    if (threadIdx.x == 0) {
        sh.consumed = 0;
        sh.stop = 0;
        sh.kpub = (unsigned long long)__double_as_longlong(-INFINITY);
        for (int r = 0; r < kRing; ++r) sh.ready[r] = 0;
    }
    // the first chunk's mask words are loaded together with the event count
    // (words past the sample's segments are dropped below)
    uint32_t mw[kSegPerLane];
#pragma unroll
    for (int h = 0; h < kSegPerLane; ++h) {
        const int sj = lane * kSegPerLane + h;
        mw[h] = chain && sj < S ? mask[((size_t)b * S + sj) * N + n] : 0u;
    }
    const int nb = __builtin_amdgcn_readfirstlane(clamp_count(ev_n[b], E_max));
    const float* tt = ev_t + (size_t)b * E_max;
    const int32_t* src = ev_src + (size_t)b * E_max;
    const Decay* d = dec + (size_t)b * E_pad;
    const size_t idx = (size_t)b * N + n;
    float* st = out_t + idx * (size_t)m.s_max;
    float* si = out_i ? out_i + idx * (size_t)m.s_max : nullptr;
    int32_t* sk = out_k ? out_k + idx * (size_t)m.s_max : nullptr;
    const int Sb = (nb + kSeg - 1) / kSeg;
    const bool has_open = __builtin_amdgcn_readfirstlane(nb > 0 && m.t_end > (double)tt[max(nb - 1, 0)] ? 1 : 0) != 0;
    __syncthreads();                          // the ring is reset

    RingChain ch{0, 0.0, 0.0, -INFINITY, 1.0, -1, -1, false};
    int wbase = 0;                            // windows of earlier chunks
    bool stop = false;
    for (int seg0 = 0; seg0 < Sb && !stop; seg0 += kChunkSeg) {
        // ---- this chunk's flagged sub-blocks as a time-ordered list, with
        // slots; lane l takes segments seg0 + kSegPerLane l + h
        if (chain) {
            uint32_t mv[kSegPerLane];
            int pc = 0;
#pragma unroll
            for (int h = 0; h < kSegPerLane; ++h) {
                const int sj = seg0 + lane * kSegPerLane + h;
                if (seg0 > 0) mw[h] = sj < Sb ? mask[((size_t)b * S + sj) * N + n] : 0u;
                mv[h] = sj < Sb ? (mw[h] & ((1u << kSubPerSeg) - 1u)) : 0u;
                pc += __popc(mv[h]);
            }
            int ex = pc;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const int v = __shfl_up(ex, off, kWave);
                if (lane >= off) ex += v;
            }
            const int ctot = rl_int(ex, kWave - 1);
            ex -= pc;
            // candidates and their pool slots (consecutive per segment)
            int o = ex;
#pragma unroll
            for (int h = 0; h < kSegPerLane; ++h) {
                uint32_t mm = mv[h], rel = mw[h] >> kMaskBits;
                while (mm) {
                    sh.cand[o] = ((uint32_t)(lane * kSegPerLane + h) << 3) | (uint32_t)__builtin_ctz(mm);
                    sh.slot[o] = rel < pool_cap ? (uint32_t)b * pool_cap + rel : kNoSlot;
                    ++o;
                    ++rel;
                    mm &= mm - 1u;
                }
            }
            if (lane == 0) sh.ntot = ctot;
        }
        __syncthreads();
        const int tot = __builtin_amdgcn_readfirstlane(sh.ntot);
        const int nwin = (tot + kWinCand - 1) / kWinCand;
        if (tot > 0) {
            // the open interval is taken after the window holding the sample's
            // last sub-block, when that sub-block is flagged (it is the last
            // candidate of the last chunk)
            const uint32_t cwl = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.cand[tot - 1]);
            const bool open_here = has_open && (seg0 + (int)(cwl >> 3)) * kSeg + (int)(cwl & 7u) * kSub + kSub >= nb;
            if (!chain) {
                for (int wi = wv - 1; wi < nwin; wi += kRingWaves - 1) {
                    const int wg = wbase + wi, buf = wg % kRing;
                    // this window's loads go out before the wait for its buffer
                    const StageIn cur = stage_load(sh, wi * kWinCand, tot, seg0, nb, tt, src, d, pool);
                    bool halt = false;
                    for (int spin = 0;; ++spin) {
                        halt = lds_load(&sh.stop) != 0;
                        if (halt || lds_load(&sh.consumed) >= wg - kRing + 1) break;
                        if (spin >= kSpinLimit) {
                            give_up();
                            halt = true;
                            break;
                        }
                        __builtin_amdgcn_s_sleep(1);
                    }
                    if (halt) break;
                    stage_window(sh, sh.win[buf], m, cur, wi * kWinCand, tot, seg0, b, n, nb, S, N, C_in, src, d,
                                 WT, carry, open_here && wi == nwin - 1, sh.kmax[buf]);
                    lds_store(&sh.ready[buf], wg + 1);
                }
            } else {
                for (int wi = 0; wi < nwin;) {
                    const int wg = wbase + wi, buf = wg % kRing;
                    bool late = false;
                    for (int spin = 0; lds_load(&sh.ready[buf]) != wg + 1; ++spin) {
                        if (spin >= kSpinLimit || lds_load(&sh.stop) != 0) {
                            if (spin >= kSpinLimit) give_up();
                            late = true;
                            break;
                        }
                        __builtin_amdgcn_s_sleep(1);
                    }
                    if (late) break;
                    // the run of windows wi, wi + 1, ... staged already (lane q
                    // looks at window wi + q), and the first of them whose
                    // largest key reaches the current deficit's key: the
                    // windows before it hold no crossing and are passed over
                    const int bq = (wg + lane) % kRing;
                    const bool rdy = lane < kRing && wi + lane < nwin && lds_load(&sh.ready[bq]) == wg + lane + 1;
                    const int nr = __builtin_ctzll(~__ballot(rdy));
                    const unsigned long long hit = __ballot(lane < nr && sh.kmax[bq] >= ch.K);
                    if (hit == 0ull) {
                        wi += nr;
                        lds_store(&sh.consumed, wg + nr);
                        continue;
                    }
                    wi += __builtin_ctzll(hit);
                    const int wh = wbase + wi, c0 = wi * kWinCand;
                    chain_window<PI>(sh, sh.win[wh % kRing], m, wh, c0, min(kWinCand, tot - c0) * kSub,
                                     open_here && wi == nwin - 1, seg0, nb, ch, st, si, sk);
                    ++wi;
                    lds_store(&sh.consumed, wh + 1);
                    if (ch.capped) {
                        lds_store(&sh.stop, 1);
                        break;
                    }
                }
            }
        }
        wbase += nwin;
        __syncthreads();                      // all waves are done with the chunk's list
        stop = __builtin_amdgcn_readfirstlane(lds_load(&sh.stop)) != 0;
    }
    if (!chain) return 0;
    ring_flush(sh, m, ch.ns - ch.ns % kWave, ch.ns, st, si, sk);
    if (lane == 0) out_n[idx] = ch.ns;
    return ch.ns;
}

// Work-list driven: the per-sample lists of neurons built by the check pass
// are taken as one concatenated list, entry w by workgroup w mod gridDim.x.
// Status counts are added once per workgroup.
template <int PI>
__global__ __launch_bounds__(kWave * kRingWaves) void k_resolve_ring(
    const float* __restrict__ ev_t, const int32_t* __restrict__ ev_src, const int32_t* __restrict__ ev_n, int B,
    int E_max, const float* __restrict__ WT, int C_in, int N, int E_pad, int S, Model m,
    const Decay* __restrict__ dec, const double2* __restrict__ carry, const uint32_t* __restrict__ mask,
    uint32_t pool_cap, const double2* __restrict__ pool, const uint32_t* __restrict__ pool_count,
    const uint32_t* __restrict__ work, const uint32_t* __restrict__ nwork, unsigned long long most,
    float* __restrict__ out_t, int32_t* __restrict__ out_n, float* __restrict__ out_i, int32_t* __restrict__ out_k,
    int32_t* __restrict__ status)
{
    __shared__ RingLds sh;
    const int lane = (int)threadIdx.x % kWave;
    resolve_status(ev_n, B, E_max, pool_count, pool_cap, status);
    if (most != ~0ull && flagged_total(pool_count, B) > most) return;     // k_resolve's
    // spikes and capped neurons of this workgroup's neurons, added to the
    // status words once at its end
    unsigned long long spikes = 0;
    uint32_t capped = 0;
    // All waves walk the list the same way.  Running sum of the list
    // lengths over groups of 64 samples (one load per lane, a wave prefix
    // sum): entry w of the concatenated lists belongs to the first sample
    // whose running sum exceeds w.
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
    for (uint32_t w = blockIdx.x;; w += gridDim.x) {
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
        const uint32_t bn = (uint32_t)__builtin_amdgcn_readfirstlane((int)work[(size_t)b * N + (w - before)]);
        const int ns = ring_neuron<PI>(sh, (int)(bn / (uint32_t)N), (int)(bn % (uint32_t)N), ev_t, ev_src, ev_n,
                                      E_max, WT, C_in, N, E_pad, S, m, dec, carry, mask, pool_cap, pool, out_t, out_n,
                                      out_i, out_k, status);
        spikes += (unsigned long long)ns;
        capped += ns >= m.s_max ? 1u : 0u;
    }
    if (threadIdx.x == 0) {
        const int32_t sp = (int32_t)(spikes > 0x7fffffffull ? 0x7fffffffull : spikes);
        if (sp) {
            atomicAdd(&status[LIF_ST_SPIKES], sp);
            atomicAdd(&status[LIF_ST_ROOT_SOLVES], sp);
        }
        if (capped) {
            atomicAdd(&status[LIF_ST_CAPPED], (int32_t)capped);
            atomicOr(&status[LIF_ST_FLAGS], LIF_WARN_SPIKE_CAP);
        }
    }
}


}  // namespace lif
