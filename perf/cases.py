"""The calls whose speed is measured: one entry point (or one short sequence
of them) per case, on seeded inputs made on the GPU.

Kinds of case and what each stands for in use:

  forward        a LIF layer's forward pass: inference, and the first half of
                 every training step
  backward       the layer's spike-time gradient to weights and input times
  delayed        a layer with synaptic delays: queue build, forward, backward
  reg            the spike-count regularisers' loss and gradient of a layer
  delayed_reg    the same for a layer with delays, on its queues
  readout        the tail of a network: spike merge, weighted leaky-integrator
                 readout with cross-entropy and gradients, gradient scatter
  train          a whole two-layer training step's loss and gradients (the
                 weights stay, so that every pass does the same work)

``exact`` computes the same results in 64 bits with plain torch, one input
event at a time, directly from the model: exponential decay between events,
the interval's maximum, a root per threshold crossing, a hard reset.
"""
import math

import torch

import paper_2603_13283_amd as lif
from paper_2603_13283_amd.train import DelayConfig, RegConfig, TwoLayerNet

DEV = "cuda:0"
F64 = torch.float64
TAU_MEM, V_TH, SOLVER_REG = 0.02, 1.0, 0.01
C_TARGET, LAM_REG, LAM_OVER = 14.0, 1e-3, 5e-5      # the regularisers' target and weights
LI = dict(tau_li=0.5, tau_max=1.0, beta=0.05)       # the readout's constants

# What a case leaves out.  median_hz: median rate of the input channels
# (log-normal, sigma 1); events: uniform events per sample instead; bursts:
# event-camera input; ragged: samples of any length up to the full one, one of
# them empty.
DEFAULTS = dict(B=1, C=64, N=32, s_max=64, gain=4.0, T=1.0, median_hz=0.0, events=0, bursts=False, ragged=False,
                tau_syn=0.005, v_reset=0.0, t_end=math.inf, d_max=0.1, rate=0.0, K=20, N2=0, gain2=12.0, reg=False,
                delays=False, time_grad=True)


def listed():
    return [
        # one sample through a small layer: latency of a streaming call
        dict(name="forward_64x32_b1", kind="forward", B=1, C=64, N=32, events=256, gain=8.0),
        # the headline layer: audio-like input, 700 channels, ~5 k events a sample
        dict(name="forward_700x256_b32", kind="forward", B=32, C=700, N=256, median_hz=4.33),
        # odd sizes, samples of any length, a time-constant ratio that is no integer, a reset below rest
        dict(name="forward_odd_ragged", kind="forward", B=13, C=1001, N=387, events=6000, gain=9.0, ragged=True,
             tau_syn=0.006, v_reset=-0.3, t_end=1.2),
        # event-camera input in bursts, 2312 polarity channels
        dict(name="forward_2312x1024_b64", kind="forward", B=64, C=2312, N=1024, bursts=True, gain=3.0, T=0.3),
        # a large layer on long streams, ~100 k events a sample, driven so that it fires
        dict(name="forward_32768x2048_b16", kind="forward", B=16, C=32768, N=2048, median_hz=1.851, gain=16.0),
        # gradients of a hidden layer of the two-layer network
        dict(name="backward_700x512_b128", kind="backward", B=128, C=700, N=512, s_max=128, median_hz=8.66),
        # gradients of the large layer
        dict(name="backward_32768x2048_b16", kind="backward", B=16, C=32768, N=2048, median_hz=1.851, gain=16.0),
        # a layer with learnable delays: queues, forward and backward
        dict(name="delayed_700x256_b32", kind="delayed", B=32, C=700, N=256, median_hz=4.33),
        # regularisers of a hidden layer of the two-layer network
        dict(name="reg_700x512_b128", kind="reg", B=128, C=700, N=512, s_max=128, median_hz=8.66),
        # the same with delays
        dict(name="delayed_reg_700x512_b128", kind="delayed_reg", B=128, C=700, N=512, s_max=128, median_hz=8.66),
        # merge, readout and their gradients at the network's output, ~14 spikes a neuron
        dict(name="readout_512x20_b128", kind="readout", B=128, N=512, s_max=128, rate=14.0),
        # the training step of the two-layer network with its regularisers
        dict(name="train_700x512x512_b128", kind="train", B=128, C=700, N=512, N2=512, s_max=128, median_hz=8.66,
             reg=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward", "forward", "backward", "delayed", "reg", "delayed_reg", "readout", "train"])
    if kind == "readout":
        return dict(kind=kind, B=_log_int(rng, 1, 128), N=_log_int(rng, 20, 512), K=_log_int(rng, 2, 64),
                    s_max=rng.choice([32, 64, 128]), rate=math.exp(rng.uniform(0.0, math.log(14.0))))
    top = dict(forward=3e9, backward=3e9, delayed=3e8, reg=6e8, delayed_reg=3e8, train=3e8)[kind]
    while True:
        B, N = _log_int(rng, 1, 128), _log_int(rng, 20, 2048)
        C, events = _log_int(rng, 20, 8192), _log_int(rng, 60, 60000)
        if kind == "train":
            N, events = min(N, 600), min(events, 14000)
        if 3e4 <= B * N * events <= top:
            break
    T = round(max(0.1, min(1.0, events / 6000)), 3)
    # the layer's drive, (events per second) gain^2 / C: 114 in the headline layer, ~230 in the two-layer network, 780
    # in the large one
    drive = math.exp(rng.uniform(math.log(150.0), math.log(900.0)))
    case = dict(kind=kind, B=B, C=C, N=N, events=events, T=T, ragged=rng.random() < 0.4,
                gain=round(math.sqrt(drive * C * T / events), 2), s_max=rng.choice([64, 128]))
    if rng.random() < 0.3:
        case.update(tau_syn=rng.choice([0.004, 0.006, 0.01]), v_reset=rng.choice([0.0, -0.3]), t_end=case["T"] * 1.25)
    if kind in ("backward", "reg", "delayed", "delayed_reg"):
        case["time_grad"] = rng.random() < 0.7
    if kind == "train":
        case.update(N2=_log_int(rng, 20, 600), reg=rng.random() < 0.5, delays=rng.random() < 0.5)
    return case


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _full(case):
    return dict(DEFAULTS, **case)


def _params(c):
    return lif.Params(tau_mem=TAU_MEM, tau_syn=c["tau_syn"], v_th=V_TH, v_reset=c["v_reset"], t_end=c["t_end"],
                      s_max=c["s_max"], solver_reg=SOLVER_REG)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _capacity(c):
    """Queue length: as many events as a sample of the case's input may have."""
    if c["events"]:
        return c["events"]
    if c["bursts"]:
        on = 0.3 * c["C"]                                 # active channels of a window
        return int(3 * on * 9.606 + 6 * math.sqrt(3 * on * (9.606 + 0.7 * 9.606 ** 2)))
    m = c["median_hz"] * c["T"]
    mean, var = m * math.exp(0.5) * c["C"], m * m * math.e * (math.e - 1) * c["C"]
    return int(mean + 6 * math.sqrt(mean + var))


def _pack(b, t, src, B, E):
    """Per-sample queues of E entries, sorted by time, from flat (sample, time,
    source) lists (events past a full queue are dropped)."""
    n = torch.bincount(b, minlength=B)
    order = torch.sort(b * (1 << 32) + t.view(torch.int32).to(torch.int64), stable=True).indices
    b, t, src = b[order], t[order], src[order]
    at = torch.arange(b.numel(), device=DEV) - (torch.cumsum(n, 0) - n)[b]
    b, t, src, at = (x[at < E] for x in (b, t, src, at))
    ev_t = torch.full((B, E), math.inf, dtype=torch.float32, device=DEV)
    ev_s = torch.zeros((B, E), dtype=torch.int32, device=DEV)
    ev_t[b, at] = t
    ev_s[b, at] = src.to(torch.int32)
    return ev_t, ev_s, n.clamp(max=E).to(torch.int32)


def _events(c, g):
    B, C, T = c["B"], c["C"], c["T"]
    if c["bursts"]:
        # three windows; in each 30 % of the channels fire ~9.6 times around its middle (sigma 15 ms)
        on = torch.rand((3, B, C), generator=g, device=DEV) < 0.3
        cnt = torch.poisson(torch.where(on, 9.606, 0.0), generator=g).long().flatten()
        cell = torch.repeat_interleave(torch.arange(3 * B * C, device=DEV), cnt)
        u = torch.rand(cell.numel(), generator=g, dtype=F64, device=DEV) * 2 - 1
        win = T / 3
        edge = math.erf(0.5 * win / (0.015 * math.sqrt(2)))
        t = ((cell // (B * C)) + 0.5) * win + 0.015 * math.sqrt(2) * torch.erfinv(u * edge)
        b, src = (cell // C) % B, cell % C
    elif c["events"]:
        n = torch.full((B,), c["events"], dtype=torch.int64, device=DEV)
        if c["ragged"] and B > 1:
            n = torch.randint(0, c["events"] + 1, (B,), generator=g, device=DEV)
            n[0], n[B - 1] = c["events"], 0
        b = torch.repeat_interleave(torch.arange(B, device=DEV), n)
        src = torch.randint(0, C, (b.numel(),), generator=g, device=DEV)
        t = torch.rand(b.numel(), generator=g, dtype=F64, device=DEV) * T
    else:
        rate = c["median_hz"] * torch.exp(torch.randn((B, C), generator=g, device=DEV))
        cnt = torch.poisson(rate * T, generator=g).long().flatten()
        cell = torch.repeat_interleave(torch.arange(B * C, device=DEV), cnt)
        b, src = cell // C, cell % C
        t = torch.rand(b.numel(), generator=g, dtype=F64, device=DEV) * T
    return _pack(b, t.to(torch.float32), src, B, _capacity(c))


def _weights(g, C, N, gain):
    return torch.randn((C, N), generator=g, device=DEV) * (gain / math.sqrt(C))


def _bytes(n):
    return torch.empty(max(int(n), 1), dtype=torch.uint8, device=DEV)


def _trains(c, g):
    """Sorted random spike trains with Poisson counts (a layer's output)."""
    B, N, S = c["B"], c["N"], c["s_max"]
    n = torch.poisson(torch.full((B, N), c["rate"], device=DEV), generator=g).clamp(max=S).to(torch.int32)
    t = torch.rand((B, N, S), generator=g, device=DEV) * 0.98 + 0.01
    live = torch.arange(S, device=DEV) < n[..., None]
    t = torch.where(live, t, math.inf).sort(-1).values.contiguous()
    return lif.ForwardOut(t, n, None, None)


def _inputs(c, seed):
    """The layer's inputs alone: events and weights (and delays)."""
    g = _gen(seed)
    s = {"c": c, "g": g, "P": _params(c), "ev": _events(c, g), "W": _weights(g, c["C"], c["N"], c["gain"])}
    if c["kind"] in ("delayed", "delayed_reg"):
        s["D"] = torch.rand((c["C"], c["N"]), generator=g, device=DEV) * c["d_max"]
    return s


def prepare(case, seed):
    c = _full(case)
    kind = c["kind"]
    if kind == "readout":
        g = _gen(seed)
        s = {"c": c, "fwd": _trains(c, g), "W": _weights(g, c["N"], c["K"], 4.0),
             "labels": torch.randint(0, c["K"], (c["B"],), generator=g, device=DEV, dtype=torch.int32)}
        s["E2"] = min(lif.LIF_MERGE_MAX, c["N"] * c["s_max"])
        s["ws"] = _bytes(lif.lif_li_readout_workspace_size(c["B"], s["E2"], c["N"], c["K"]))
        return s
    s = _inputs(c, seed)
    g, P, W = s["g"], s["P"], s["W"]
    B, E = s["ev"][0].shape
    C, N = W.shape
    if kind == "train":
        kw = {}
        if c["reg"]:
            kw["reg"] = RegConfig(c_target=(C_TARGET, C_TARGET), lam_reg=LAM_REG, lam_over=LAM_OVER)
        if c["delays"]:
            raw = lambda *sh: torch.log(torch.expm1(5.0 * (torch.rand(sh, generator=g, device=DEV) * 0.099 + 1e-3))) / 5.0
            kw["delays"] = DelayConfig(raw(C, N), raw(N, c["N2"]), beta=5.0)
        s["W2"], s["Wo"] = _weights(g, N, c["N2"], c["gain2"]), _weights(g, c["N2"], c["K"], 4.0)
        s["labels"] = torch.randint(0, c["K"], (B,), generator=g, device=DEV, dtype=torch.int32)
        q = lif.LiParams(tau_mem=TAU_MEM, tau_syn=c["tau_syn"], **LI)
        s["net"] = TwoLayerNet(W, s["W2"], s["Wo"], B=B, E_max=E, P1=P, P2=P, q=q, **kw)
        return s
    fws = lambda: _bytes(lif.lif_layer_forward_workspace_size(B, E, C, N, P.c()))
    if kind == "forward":
        s["ws"] = fws()
        new = lambda dt: torch.empty((B, N, c["s_max"]), dtype=dt, device=DEV)
        s["out"] = lif.ForwardOut(new(torch.float32), torch.empty((B, N), dtype=torch.int32, device=DEV),
                                  new(torch.float32), torch.empty(lif.LIF_STATUS_WORDS, dtype=torch.int32, device=DEV),
                                  new(torch.int32))
        return s
    upstream = lambda: torch.randn((B, N, c["s_max"]), generator=g, device=DEV)
    if kind in ("backward", "reg"):
        s["fwd"] = lif.forward(*s["ev"], W, P, ws=fws())
    if kind == "backward":
        s["g_out"] = upstream()
        s["ws"] = _bytes(lif.lif_layer_backward_workspace_size(B, E, C, N, P.c()))
    elif kind == "reg":
        s["ws"] = _bytes(lif.lif_spike_count_reg_backward_workspace_size(B, E, C, N))
    elif kind == "delayed":
        s["g_out"] = upstream()
        s["qws"] = _bytes(lif.lif_delay_queues_workspace_size(B, E, N))
        s["ws"] = _bytes(lif.lif_layer_backward_delayed_workspace_size(B, E, C, N, P.c()))
    elif kind == "delayed_reg":
        s["q"] = lif.delay_queues(*s["ev"], s["D"])
        s["fwd"] = lif.forward_delayed(s["q"], s["ev"][1], s["ev"][2], W, P)
        s["ws"] = _bytes(lif.lif_spike_count_reg_delayed_workspace_size(B, E, C, N))
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _spikes(o):
    return {"t": o.out_t, "n": o.out_n, "i": o.out_i, "k": o.out_k}


def run(s):
    c = s["c"]
    kind, tg = c["kind"], c["time_grad"]
    if kind == "readout":
        N, S = c["N"], c["s_max"]
        t2, s2, n2, perm, _ = lif.merge(s["fwd"], s["E2"])
        logits, loss, gW, gT = lif.li_readout(t2, s2, n2, s["W"], lif.LiParams(**LI), labels=s["labels"], ws=s["ws"])
        g = lif.merge_grad(gT, perm, n2, N, S)
        return {"t": t2, "src": s2, "n": n2, "perm": perm, "logits": logits, "loss": loss, "gW": gW, "gT": gT, "g": g}
    ev, W, P = s["ev"], s["W"], s["P"]
    if kind == "forward":
        return _spikes(lif.forward(*ev, W, P, ws=s["ws"], out=s["out"]))
    if kind == "backward":
        gW, gT = lif.backward(*ev, W, s["fwd"], s["g_out"], P, want_time_grad=tg, ws=s["ws"])
        return {"gW": gW, "gT": gT}
    if kind == "reg":
        loss, gs, gW, gT = lif.spike_count_reg_backward(*ev, W, s["fwd"], C_TARGET, LAM_REG, LAM_OVER, P,
                                                        want_time_grad=tg, ws=s["ws"])
        return {"loss": loss, "gs": gs, "gW": gW, "gT": gT}
    if kind == "delayed":
        q = lif.delay_queues(*ev, s["D"], ws=s["qws"])
        o = lif.forward_delayed(q, ev[1], ev[2], W, P)
        gW, gD, gT = lif.backward_delayed(q, ev[1], ev[2], W, o, s["g_out"], P, want_time_grad=tg, ws=s["ws"])
        # the queues hold the events of each sample; entries past them are not written
        return {"spikes": _spikes(o), "gW": gW, "gD": gD, "gT": gT}
    if kind == "delayed_reg":
        loss, gs, gW, gD, gT = lif.spike_count_reg_delayed_backward(s["q"], ev[1], ev[2], W, s["fwd"], C_TARGET, LAM_REG,
                                                                    LAM_OVER, P, want_time_grad=tg, ws=s["ws"])
        return {"loss": loss, "gs": gs, "gW": gW, "gD": gD, "gT": gT}
    r = s["net"].step(*ev, s["labels"], update=False)
    return {"loss": r.loss, "logits": r.logits, "grads": r.grads, "reg": list(r.reg_losses), "spikes1": _spikes(r.fwd1),
            "spikes2": _spikes(r.fwd2)}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _mean_events(c):
    if c["bursts"]:
        return 3 * 0.3 * c["C"] * 9.606
    if c["events"]:
        return c["events"] * (0.5 if c["ragged"] and c["B"] > 2 else 1.0)
    return c["median_hz"] * math.exp(0.5) * c["C"] * c["T"]


def work(case):
    """Bytes: inputs read once, outputs written once.  Flops: per (event,
    neuron) the two-state decay and jump (4), and for a gradient its adjoint
    recurrence and products (8); the regularisers also take each interval's
    maximum (20)."""
    c = _full(case)
    B, C, N, S, kind = c["B"], c["C"], c["N"], c["s_max"], c["kind"]
    if kind == "readout":
        ev = B * N * c["rate"]
        return {"bytes": ev * (4 + 12 + 8) + 8 * N * c["K"] + 4.0 * B * N * S, "flops": ev * 6.0 * c["K"]}
    E = _mean_events(c)
    ne, weights, events, spikes = B * N * E, 4.0 * C * N, 8.0 * B * E, 12.0 * B * N * S
    if kind == "forward":
        return {"bytes": events + weights + spikes, "flops": 4 * ne}
    if kind == "backward":
        return {"bytes": 1.5 * events + 2 * weights + spikes + 4.0 * B * N * S, "flops": 8 * ne}
    if kind == "reg":
        return {"bytes": 1.5 * events + 2 * weights + spikes, "flops": 32 * ne}
    if kind == "delayed":
        return {"bytes": 1.5 * events + 4 * weights + 4 / 3 * spikes + 8.0 * ne, "flops": 12 * ne}
    if kind == "delayed_reg":
        return {"bytes": 0.5 * events + 3 * weights + spikes + 8.0 * ne, "flops": 32 * ne}
    ne2 = B * c["N2"] * N * 2.5                          # ~2.5 spikes a neuron reach the second layer
    per = 12 + (28 if c["reg"] else 0)
    W2 = 4.0 * N * c["N2"]
    return {"bytes": events + (4 if c["delays"] else 2) * (weights + W2) + 12.0 * B * (N + c["N2"]) * S,
            "flops": per * (ne + ne2)}


# The state is float64 and the outputs are float32, so another correct
# implementation differs by the outputs' rounding (6e-8; measured against
# exact: 2.5e-8 in norm) where a result is well conditioned.  A gradient sums
# terms that cancel; the regularisers take an interval's maximum and its
# records in float32 (measured 1.3e-7, with delays 2.4e-6); a training step
# hands spike times on in float32.
def tolerance(case):
    return {"forward": {"rel": 1e-6, "max": 1e-5}, "readout": {"rel": 1e-6, "max": 1e-5},
            "backward": {"rel": 1e-6, "max": 1e-4}, "delayed": {"rel": 2e-6, "max": 2e-4},
            "reg": {"rel": 1e-6, "max": 1e-4}, "delayed_reg": {"rel": 1e-5, "max": 1e-3},
            "train": {"rel": 5e-5, "max": 5e-3}}[case["kind"]]


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------
class _Stream:
    """The input a layer's neurons see, event by event: at(k) gives times
    [B, 1] (or [B, N] of a layer with delays), weights [B, N] and the
    channels and sample event indices that they come from."""

    def __init__(self, c, s):
        self.c, self.W, (t, src, n) = c, s["W"].double(), s["ev"]
        self.n, self.src, self.t = n.long()[:, None], src.long(), t.double()
        self.B, self.E = t.shape
        self.C, self.N = self.W.shape
        self.tm, self.ts = TAU_MEM, c["tau_syn"]
        self.kappa = self.ts / (self.tm - self.ts)
        self.col = torch.arange(self.N, device=DEV)
        self.q = None
        if "D" in s:
            a = torch.empty((self.B, self.N, self.E), dtype=torch.float32, device=DEV)
            for b in range(self.B):
                a[b] = t[b] + s["D"].t()[:, self.src[b]]                     # float32 arrivals, as the queues hold them
            a.masked_fill_(torch.arange(self.E, device=DEV) >= self.n[:, :, None], math.inf)
            a, k = torch.sort(a, dim=-1, stable=True)
            self.q, self.qk = a.permute(2, 0, 1).contiguous(), k.permute(2, 0, 1).to(torch.int32).contiguous()

    def time(self, k):
        return self.t[:, k:k + 1] if self.q is None else self.q[k].double()

    def channel(self, k):
        return self.src[:, k:k + 1] if self.q is None else torch.gather(self.src, 1, self.qk[k].long())

    def weight(self, k):
        return self.W[self.src[:, k]] if self.q is None else self.W[self.channel(k), self.col]

    def interval(self, k, tp):
        """(has interval k, its length): it ends at event k, or at t_end after the last one."""
        te = self.time(k) if k < self.E else torch.full_like(tp, math.inf)
        L = torch.where(self.n > k, te, self.c["t_end"]) - tp
        return (self.n >= k) & (L > 0), L

    def decays(self, L):
        return torch.exp(-L / self.tm), torch.exp(-L / self.ts)

    def zeros(self):
        return torch.zeros((self.B, self.N), dtype=F64, device=DEV)


def _exact_forward(x):
    c, tm, ts, ka = x.c, x.tm, x.ts, x.kappa
    S, th, r = c["s_max"], V_TH, 1.0 / x.ts - 1.0 / x.tm
    V, I, tp = x.zeros(), x.zeros(), x.zeros()
    out_t = torch.full((x.B, x.N, S), math.inf, dtype=F64, device=DEV)
    out_i, out_k = torch.zeros_like(out_t), torch.zeros_like(out_t, dtype=torch.int32)
    out_n = torch.zeros((x.B, x.N), dtype=torch.int64, device=DEV)
    ft, fi, fk, fn = out_t.view(-1, S), out_i.view(-1, S), out_k.view(-1, S), out_n.view(-1)
    for k in range(x.E + 1):
        ok, L = x.interval(k, tp)
        # a crossing needs I > th, or V at th already: the rest is skipped
        A, D = x.decays(L)
        V1 = V * A + ka * I * (A - D)
        at = (ok & (out_n < S) & ((I > th) | (V >= th))).flatten().nonzero().flatten()
        v, i, l, u0 = V.view(-1)[at], I.view(-1)[at], L.expand_as(V).reshape(-1)[at], torch.zeros(at.numel(), dtype=F64, device=DEV)
        t0 = tp.view(-1)[at]
        while at.numel():
            # the maximum over the interval's rest, of (V_lin - th) e^{u/tm}: at ts ln(I / th) when inside
            us = torch.minimum(ts * torch.log((i / th).clamp(min=1.0)), l)
            peak = v * torch.exp(-us / tm) + ka * i * (torch.exp(-us / tm) - torch.exp(-us / ts))
            go = (peak >= th).nonzero().flatten()
            if not go.numel():
                break
            at, v, i, l, u0, t0, us = at[go], v[go], i[go], l[go], u0[go], t0[go], us[go]
            # Newton from the left on a concave function: it rises to the first root
            c0, u = v + ka * i, torch.zeros_like(v)
            for _ in range(60):
                e1, e2 = torch.exp(u / tm), ka * i * torch.exp(-u * r)
                F = c0 - th * e1 - e2
                du = (-F / (r * e2 - th / tm * e1)).nan_to_num(0.0).clamp(min=0.0)
                un = torch.minimum(u + du, us)
                done = not bool((un - u > 1e-16 + 1e-15 * u).any())
                u = un
                if done:
                    break
            n = fn[at]
            u0, i, l = u0 + u, i * torch.exp(-u / ts), l - u
            v = torch.full_like(v, c["v_reset"])
            ft[at, n], fi[at, n], fk[at, n] = t0 + u0, i, k
            fn[at] = n + 1
            # the state at the interval's end, after this spike
            V1.view(-1)[at] = v * torch.exp(-l / tm) + ka * i * (torch.exp(-l / tm) - torch.exp(-l / ts))
            more = ((fn[at] < S) & (l > 0) & (i > th)).nonzero().flatten()
            at, v, i, l, u0, t0 = at[more], v[more], i[more], l[more], u0[more], t0[more]
        if k < x.E:
            has = x.n > k
            V = torch.where(has, V1, V)
            I = torch.where(has, I * D + x.weight(k), I)
            tp = torch.where(has, x.time(k), tp)
    return {"t": out_t, "n": out_n.to(torch.int32), "i": out_i, "k": out_k}


class _Spikes:
    """Given spikes grouped by the interval that holds them: of(k) gives the
    flat (sample, neuron) indices, slots and times of interval k's spikes."""

    def __init__(self, fwd, extra=None):
        B, N, S = fwd["t"].shape
        live = torch.arange(S, device=DEV) < fwd["n"].long()[..., None]
        flat = live.view(-1).nonzero().flatten()
        k = fwd["k"].reshape(-1)[flat].long()
        order = torch.sort(k, stable=True).indices
        flat, k = flat[order], k[order]
        self.i, self.s, self.t = flat // S, flat % S, fwd["t"].reshape(-1)[flat].double()
        self.extra = None if extra is None else extra.reshape(-1)[flat]
        edges = torch.searchsorted(k, torch.arange(int(k.max()) + 2 if k.numel() else 1, device=DEV))
        self.edges = edges.tolist()

    def of(self, k):
        return slice(self.edges[k], self.edges[k + 1]) if k + 1 < len(self.edges) else slice(0, 0)


def _adjoints(x, fwd, g):
    """d(loss)/d(constraint) of every spike, last spike first, through the resets."""
    t, i, n = fwd["t"].double(), fwd["i"].double(), fwd["n"].long()
    jump = (V_TH - x.c["v_reset"]) / x.tm
    mu, Q = torch.zeros_like(t), x.zeros()
    for s in range(t.shape[2] - 1, -1, -1):
        live = n > s
        if s + 1 < t.shape[2]:
            nxt = n > s + 1
            Q = torch.where(nxt, (Q + mu[..., s + 1]) * torch.exp(-(t[..., s + 1] - t[..., s]) / x.tm).nan_to_num(0.0), 0.0)
        m = -(g[..., s].double() - jump * Q) / ((i[..., s] - V_TH) / x.tm).clamp(min=SOLVER_REG)
        mu[..., s] = torch.where(live, m, 0.0)
    return mu


class _Grads:
    """Sums of per-event gradient terms over the batch."""

    def __init__(self, x):
        self.x = x
        self.W = torch.zeros((x.C, x.N), dtype=F64, device=DEV)
        self.D = torch.zeros_like(self.W) if x.q is not None else None
        self.T = torch.zeros((x.B, x.E), dtype=F64, device=DEV)

    def add(self, k, gw, ga):
        x, has = self.x, self.x.n > k
        gw, ga = torch.where(has, gw, 0.0), torch.where(has, ga, 0.0)
        if x.q is None:
            self.W.index_add_(0, x.src[:, k], gw)
            self.T[:, k] += ga.sum(1)
        else:
            at = (x.channel(k) * x.N + x.col).flatten()
            self.W.view(-1).index_add_(0, at, gw.flatten())
            self.D.view(-1).index_add_(0, at, ga.flatten())
            self.T.scatter_add_(1, torch.where(has, x.qk[k].long(), 0), ga)

    def out(self, time_grad):
        r = {"gW": self.W, "gT": self.T if time_grad else None}
        return r if self.D is None else dict(r, gD=self.D)


def _exact_backward(x, fwd, g, time_grad):
    mu = _adjoints(x, fwd, g)
    sp = _Spikes(fwd, mu)
    Pm, Ps, out = x.zeros(), x.zeros(), _Grads(x)
    for k in range(x.E - 1, -1, -1):
        tk = x.time(k)
        if k + 1 < x.E:
            L = torch.where(x.n > k + 1, x.time(k + 1) - tk, 0.0)
            A, D = x.decays(L)
            Pm, Ps = Pm * A, Ps * D
        at = sp.of(k + 1)
        if at.stop > at.start:
            i = sp.i[at]
            u = (sp.t[at] - tk.expand(x.B, x.N).reshape(-1)[i]).clamp(min=0.0)
            Pm.view(-1).index_add_(0, i, sp.extra[at] * torch.exp(-u / x.tm))
            Ps.view(-1).index_add_(0, i, sp.extra[at] * torch.exp(-u / x.ts))
        out.add(k, x.kappa * (Pm - Ps), x.weight(k) * x.kappa * (Pm / x.tm - Ps / x.ts))
    return out.out(time_grad)


def _exact_reg(x, fwd, time_grad):
    """Loss terms and gradient of lam_reg L_reg + lam_over L_over: each
    interval's largest V from its true start state, the hinge means, the
    gates, and the adjoint of a pseudo-spike at every active maximum."""
    c, tm, ts, ka, th = x.c, x.tm, x.ts, x.kappa, V_TH
    dth, c_tv = th - c["v_reset"], x.tm * x.ts / (x.tm - x.ts)
    sp = _Spikes(fwd)
    V, I, Dft, tp = x.zeros(), x.zeros(), x.zeros(), x.zeros()
    su, so, nsil, nspk = x.zeros(), x.zeros(), x.zeros(), x.zeros()
    sgn, em_, es_, vs_, ve_ = [], [], [], [], []
    for k in range(x.E + 1):
        here = x.n >= k
        _, L = x.interval(k, tp)
        L = torch.where(here, L, 0.0)
        A, D = x.decays(L)
        V0 = V - Dft
        V1 = torch.where(torch.isinf(L), -math.inf, V0 * A + ka * I * (A - D))
        best = torch.maximum(V0, V1)
        a = V0 + ka * I
        u = torch.where((I > 0) & (a > 0), c_tv * torch.log((ka * I * tm / (a * ts)).clamp(min=1.0)), 0.0)
        inside = (u > 0) & (u < L)
        eu, fu = x.decays(u)
        Vu = torch.where(inside, V0 * eu + ka * I * (eu - fu), -math.inf)
        inner = Vu > best
        vmax = torch.where(inner, Vu, best)
        start, end = ~inner & (V0 >= V1), ~inner & (V1 > V0)
        at, spiked = sp.of(k), torch.zeros((x.B, x.N), dtype=torch.bool, device=DEV)
        spiked.view(-1)[sp.i[at]] = True
        su += torch.where(here & ~spiked, (th - vmax).clamp(min=0.0), 0.0)
        so += torch.where(here & spiked, (vmax - th).clamp(min=0.0), 0.0)
        nsil += here & ~spiked
        nspk += here & spiked
        s_ = torch.where(spiked, torch.where(vmax > th, -1, 0), torch.where(vmax < th, 1, 0))
        sgn.append(torch.where(here, s_, 0).to(torch.int8))
        em_.append(torch.where(start, 1.0, torch.where(end, A.expand_as(V), eu)))
        es_.append(torch.where(start, 1.0, torch.where(end, D.expand_as(V), fu)))
        vs_.append(torch.where(start & (k > 0), (I - V0) / tm, 0.0) if k else x.zeros())
        ve_.append(torch.where(end & (x.n > k), (I * D - vmax) / tm, 0.0))
        te = torch.where(x.n > k, x.time(k), tp) if k < x.E else tp
        Dft = Dft * A
        if at.stop > at.start:
            i = sp.i[at]
            Dft.view(-1).index_add_(0, i, dth * torch.exp(-(te.expand(x.B, x.N).reshape(-1)[i] - sp.t[at]) / tm))
        if k < x.E:
            has = x.n > k
            V = torch.where(has, V * A + ka * I * (A - D), V)
            I = torch.where(has, I * D + x.weight(k), I)
            tp = torch.where(has, te, tp)
    ub, ob = su / nsil.clamp(min=1), so / nspk.clamp(min=1)
    n = fwd["n"].double()
    cb = n.mean(0)
    gu, go = (1 - cb / C_TARGET).clamp(min=0.0), (cb / C_TARGET - 1).clamp(min=0.0)
    gi = (n / C_TARGET - 1).clamp(min=0.0)
    loss = torch.stack([(gu * ub.mean(0) + go * ob.mean(0)).mean(), (gi * ob).sum(0).mean()])
    Gu = -LAM_REG * gu / (x.N * x.B) / nsil.clamp(min=1)
    Go = (LAM_REG * go / (x.N * x.B) + LAM_OVER * gi / x.N) / nspk.clamp(min=1)
    Gu, Go = torch.where(nsil > 0, Gu, 0.0), torch.where(nspk > 0, Go, 0.0)
    mu = lambda k: torch.where(sgn[k] > 0, Gu, torch.where(sgn[k] < 0, Go, 0.0))
    Pm, Ps, out, gs = x.zeros(), x.zeros(), _Grads(x), torch.zeros_like(fwd["t"], dtype=F64)
    nxt = mu(x.E)
    for k in range(x.E - 1, -1, -1):
        tk = x.time(k)
        # the pseudo-spikes after event k: those of interval k + 1 and, decayed over it, the later ones
        L = torch.where(x.n > k + 1, x.time(k + 1) - tk, 0.0) if k + 1 < x.E else torch.zeros_like(tk)
        A, D = x.decays(L)
        Pm, Ps = Pm * A + nxt * em_[k + 1], Ps * D + nxt * es_[k + 1]
        m = mu(k)
        out.add(k, ka * (Pm - Ps), x.weight(k) * ka * (Pm / tm - Ps / ts) + nxt * vs_[k + 1] + m * ve_[k])
        at = sp.of(k)
        if at.stop > at.start:
            i = sp.i[at]
            w = -(dth / tm) * Pm.view(-1)[i] * torch.exp(-(tk.expand(x.B, x.N).reshape(-1)[i] - sp.t[at]) / tm)
            gs.view(-1, gs.shape[2])[i, sp.s[at]] = w
        nxt = m
    return dict(out.out(time_grad), loss=loss, gs=gs)


def _exact_readout(c, s):
    B, N, S, K, E2 = c["B"], c["N"], c["s_max"], c["K"], s["E2"]
    t = s["fwd"].out_t.reshape(B, -1)
    v, perm = torch.sort(t, dim=1, stable=True)
    v, perm = v[:, :E2], perm[:, :E2]
    n = s["fwd"].out_n.long().sum(1).clamp(max=E2)
    live = torch.arange(E2, device=DEV) < n[:, None]
    src = torch.where(live, perm // S, 0)
    t0 = torch.where(live, v, 0.0).double()
    tm, ts, li, tmax = TAU_MEM, DEFAULTS["tau_syn"], LI["tau_li"], LI["tau_max"]
    Tm, Ts, ka = li * tm / (li + tm), li * ts / (li + ts), ts / (tm - ts)
    use = live & (t0 < tmax)
    r, w0 = tmax - t0, torch.exp(-t0 / li)
    G = torch.where(use, ka * w0 * (-Tm * torch.expm1(-r / Tm) + Ts * torch.expm1(-r / Ts)), 0.0)
    dG = torch.where(use, -G / li + ka * w0 * (torch.exp(-r / Ts) - torch.exp(-r / Tm)), 0.0)
    W = s["W"].double()
    H = torch.zeros((B, N), dtype=F64, device=DEV).scatter_add_(1, src, G)
    z = H @ W
    lab = s["labels"].long()
    p = torch.softmax(LI["beta"] * z, 1)
    dz = LI["beta"] * (p - torch.nn.functional.one_hot(lab, K)) / B
    gT = dG * torch.gather(dz @ W.t(), 1, src)
    g = torch.zeros((B, N * S), dtype=F64, device=DEV)
    g.scatter_add_(1, torch.where(live, perm, 0), torch.where(live, gT, 0.0))
    return {"t": None, "src": None, "n": None, "perm": None, "logits": z, "gW": H.t() @ dz, "gT": gT,
            "loss": torch.nn.functional.cross_entropy(LI["beta"] * z, lab).reshape(1), "g": g.view(B, N, S)}


def exact(case, seed):
    c = _full(case)
    if c["kind"] == "train":
        return None                                       # two layers' events in turn, forwards and backwards: minutes
    s = prepare(case, seed)
    if c["kind"] == "readout":
        return _exact_readout(c, s)
    x = _Stream(c, s)
    if x.E > 30000 and c["kind"] != "backward":
        return None                                       # a step per event: over 20 seconds
    if c["kind"] == "forward":
        return _exact_forward(x)
    if c["kind"] == "delayed":
        fwd = _exact_forward(x)
        handed = {k: (v.float() if v.dtype == F64 else v) for k, v in fwd.items()}
        return dict(_exact_backward(x, handed, s["g_out"], c["time_grad"]), spikes=fwd)
    fwd = _spikes(s["fwd"])
    if c["kind"] == "backward":
        return _exact_backward(x, fwd, s["g_out"], c["time_grad"])
    return _exact_reg(x, fwd, c["time_grad"])
