"""The backward walk at the edges of its split: channel ranges (318 channels
fill a workgroup's LDS block), list chunks of 1024 events, blocks of 64 events,
groups of 8, tiles of 64 neurons; calls below and above 4096 events (the two
fixed-point conversions); spike bursts (several spikes of a neuron within a
group), streams so sparse that a block of 64 events spans many time constants,
and times far from 0.  Against the oracle, with the tolerances of the other
gradient tests (_fwd_bwd)."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests.parity import compare_grad
from tests.test_gpu_backward import _dev, _dev_fwd, _fwd_bwd, env  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,C,N,n,T,gain", [
    (1, 1, 1, 40, 0.05, 3.0),            # one channel, one neuron, less than a block
    (2, 318, 64, 1024, 0.2, 14.0),       # one full range, one full list chunk
    (2, 319, 65, 1025, 0.2, 14.0),       # two ranges, a chunk and an event, a tile and a neuron
    (3, 637, 33, 2100, 0.3, 12.0),       # three ranges, over 4096 events in all
    (5, 700, 130, 3000, 0.4, 12.0),      # the two-layer network's channels
    (2, 40, 70, 2500, 0.05, 60.0),       # bursts: many spikes per group of events
])
def test_adjoint_edges(env, B, C, N, n, T, gain):
    cfg = W.random_small(61, B=B, C=C, N=N, n_events=n, T=T, gain=gain)
    _fwd_bwd(env, cfg.events, cfg.layers[0].WT, 61, s_max=512, label=f"B{B} C{C} N{N} n{n} T{T}")


def _padded(ev, E):
    pad = ((0, 0), (0, E - ev.E_max))
    return W.EventBatch(np.pad(ev.ev_t, pad, constant_values=np.inf), np.pad(ev.ev_src, pad), ev.ev_n)


# Calls large enough for the walk over LDS blocks: past 2^23 (event, neuron) pairs
# with the queues' padding, and with adjoints on more than N events / 13 + 2^21 of
# the pairs without it.  The sizes are those at which the blocks, lists, tiles and
# groups end.
@pytest.mark.parametrize("B,C,N,n,T,gain,e_max", [
    (50, 318, 64, 1024, 0.2, 14.0, 7000),        # one range, a full list chunk
    (50, 319, 65, 1025, 0.2, 14.0, 7000),        # two ranges, a chunk and an event, a tile and a neuron
    (26, 637, 70, 1999, 0.3, 12.0, 7000),        # three ranges
    (9, 700, 130, 3000, 0.4, 12.0, 9000),        # workgroups that share a block
    (28, 40, 70, 2500, 0.05, 60.0, 9000),        # bursts: more than two spikes per lane and group
    (7, 3000, 200, 3000, 30.0, 60.0, 9000),      # ten ranges, lists over many references
])
@pytest.mark.parametrize("early", [False, True])
def test_adjoint_blocks(env, B, C, N, n, T, gain, e_max, early):
    """early: the backward alone, with some spike times moved before events that
    the spikes follow."""
    torch, lif = env
    cfg = W.random_small(67, B=B, C=C, N=N, n_events=n, T=T, gain=gain, ragged=False)
    ev, WT = _padded(cfg.events, e_max), cfg.layers[0].WT
    r = oracle.forward(ev.ev_t, ev.ev_src, ev.ev_n, WT, oracle.LifParams(s_max=256))
    live, events = int((r.out_n > 0).sum()), int(ev.ev_n.sum())
    assert B * e_max * N > 1 << 23 and live * events > B * events * N / 13 + (B << 21)
    label = f"blocks B{B} C{C} N{N} n{n} live {live / (B * N):.2f}"
    if not early and T < 1.0:
        _fwd_bwd(env, ev, WT, 67, s_max=256, label=label)
        return
    # (the long stream alone too: its train's own rounding, an ulp of 1.9e-6 s at
    # 30 s, is above the end-to-end bound)
    rng = np.random.default_rng(67)
    r = r.rounded()
    t = r.out_t - np.where(rng.random(r.out_t.shape) < (0.02 if early else 0.0), rng.random(r.out_t.shape) * 1e-3, 0.0)
    t = np.maximum.accumulate(np.maximum(t, 0.0).astype(np.float32), -1).astype(np.float64)
    _handmade(torch, lif, label, ev.ev_t, ev.ev_src, WT, t, r.out_k, 67, ev_n=ev.ev_n, out_i=r.out_i)


def test_adjoint_one_neuron_fires(env):
    """A wide call in which few neurons have adjoints, and one in which none has."""
    torch, lif = env
    cfg = W.random_small(68, B=9, C=700, N=130, n_events=3000, T=0.4, gain=12.0, ragged=False)
    ev, WT = _padded(cfg.events, 9000), cfg.layers[0].WT.copy()
    d = [_dev(torch, a) for a in (ev.ev_t, ev.ev_src, ev.ev_n, WT)]
    P, OP = lif.Params(s_max=128), oracle.LifParams(s_max=128)
    out = lif.forward(*d, P)
    r32 = oracle.forward(ev.ev_t, ev.ev_src, ev.ev_n, WT, OP).rounded()
    rng = np.random.default_rng(68)
    g = (rng.standard_normal(r32.out_t.shape) * np.isfinite(r32.out_t)).astype(np.float32)
    for keep in ([77], [0, 64, 129], []):
        h = g.copy()
        h[:, [i for i in range(130) if i not in keep]] = 0.0
        h[1:5] = 0.0                                     # samples without any
        oW, oT = oracle.backward(ev.ev_t, ev.ev_src, ev.ev_n, WT, r32, h.astype(np.float64), OP)
        for time_grad in (True, False):
            gW, gT = lif.backward(*d, _dev_fwd(torch, lif, r32), _dev(torch, h), P, want_time_grad=time_grad)
            torch.cuda.synchronize()
            compare_grad(gW.cpu().numpy(), oW, label=f"gW {keep}")
            if time_grad:
                compare_grad(gT.cpu().numpy(), oT, label=f"gT {keep}")


def test_adjoint_ways_under_capture(env):
    """One captured call replayed with upstream gradients on all, few, none and
    all neurons again: the way is the device's choice on every replay."""
    torch, lif = env
    cfg = W.random_small(69, B=9, C=700, N=130, n_events=3000, T=0.4, gain=12.0, ragged=False)
    ev = _padded(cfg.events, 9000)
    d = [_dev(torch, a) for a in (ev.ev_t, ev.ev_src, ev.ev_n, cfg.layers[0].WT)]
    P = lif.Params(s_max=128)
    out = lif.forward(*d, P)
    full = torch.randn(out.out_t.shape, generator=torch.Generator(device="cuda:0").manual_seed(2), device="cuda:0")
    few = torch.zeros_like(full)
    few[:, 70:73] = full[:, 70:73]
    g = full.clone()
    ws = torch.empty(lif.lif_layer_backward_workspace_size(9, 9000, 700, 130, P.c()), dtype=torch.uint8, device="cuda:0")
    ws2 = torch.empty_like(ws)
    lif.backward(*d, out, g, P, ws=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gW, gT = lif.backward(*d, out, g, P, ws=ws)
    for h in (full, few, torch.zeros_like(full), full):
        g.copy_(h)
        graph.replay()
        want = lif.backward(*d, out, h, P, ws=ws2)
        torch.cuda.synchronize()
        assert torch.equal(gW, want[0]) and torch.equal(gT, want[1])


# (B, C, N, n, T, gain, t0): 64 events over thousands of tau_s; a stream that
# starts 1500 s in (references far from 0 and, in float32, many spike times
# rounded onto or before the event just before them)
@pytest.mark.parametrize("B,C,N,n,T,gain,t0", [(2, 12, 20, 300, 90.0, 30.0, 0.0), (2, 60, 70, 3000, 0.4, 14.0, 1500.0)])
def test_adjoint_long_and_late(env, B, C, N, n, T, gain, t0):
    """The backward alone, both sides on the oracle's float32 spike train: at
    such times the train's own rounding (an ulp is 7.6e-6 s at 90 s, 1.5e-3
    of tau_s) is above the end-to-end bound."""
    torch, lif = env
    cfg = W.random_small(62, B=B, C=C, N=N, n_events=n, T=T, gain=gain)
    ev, WT = cfg.events, cfg.layers[0].WT
    ev_t = (ev.ev_t.astype(np.float64) + t0).astype(np.float32)
    OP = oracle.LifParams(s_max=128)
    r32 = oracle.forward(ev_t, ev.ev_src, ev.ev_n, WT, OP).rounded()
    g = (np.random.default_rng(62).standard_normal(r32.out_t.shape) * np.isfinite(r32.out_t)).astype(np.float32)
    oW, oT = oracle.backward(ev_t, ev.ev_src, ev.ev_n, WT, r32, g.astype(np.float64), OP)
    d = [_dev(torch, a) for a in (ev_t, ev.ev_src, ev.ev_n, WT)]
    gW, gT = lif.backward(*d, _dev_fwd(torch, lif, r32), _dev(torch, g), lif.Params(s_max=128))
    torch.cuda.synchronize()
    sW, sT = compare_grad(gW.cpu().numpy(), oW, label="gW"), compare_grad(gT.cpu().numpy(), oT, label="gT")
    print(f"[case] t0={t0} T={T} spikes={int(r32.out_n.sum())} rel(gW)={sW:.2e} rel(gT)={sT:.2e}", flush=True)


# From several events to a reference (100 tau_s) to a thousand references between
# events, as one list and as the lists of three channel ranges, where a group of
# eight events spans more of them; groups that lie in one reference next to ones
# that do not; bursts between long silences.
@pytest.mark.parametrize("C", [40, 700])
@pytest.mark.parametrize("tau_syn", [0.005, 0.0038])
@pytest.mark.parametrize("kind,T", [("even", 6.0), ("even", 40.0), ("even", 3000.0), ("bursts", 40.0)])
def test_adjoint_sparse_streams(env, C, tau_syn, kind, T):
    torch, lif = env
    B, N, E = 2, 70, 700
    rng = np.random.default_rng(66)
    t = rng.random((B, E)) * T
    if kind == "bursts":
        t = np.floor(t / 5.0) * 5.0 + rng.random((B, E)) * 0.03
    ev_t = np.sort(t, -1).astype(np.float32)
    ev_src = rng.integers(0, C, (B, E)).astype(np.int32)
    WT = (rng.standard_normal((C, N)) * 5.0).astype(np.float32)
    # one to three spikes of a neuron after some of the events
    out_t, out_k = np.full((B, N, 256), np.inf), np.zeros((B, N, 256), np.int32)
    for b in range(B):
        for i in range(N):
            ks = np.sort(rng.choice(np.arange(1, E + 1), 60, replace=False))
            ks = np.repeat(ks, rng.integers(1, 4, ks.size))[:200]
            ts = ev_t[b, ks - 1].astype(np.float64)
            nxt = np.append(ev_t[b], ev_t[b, -1] + 1.0)[ks].astype(np.float64)
            ts = ts + np.minimum(nxt - ts, 4 * tau_syn) * (0.2 + 0.3 * rng.random(ks.size))
            out_t[b, i, :ks.size] = np.maximum.accumulate(ts.astype(np.float32))
            out_k[b, i, :ks.size] = ks
    _handmade(torch, lif, f"C={C} tau_s={tau_syn} {kind} T={T}", ev_t, ev_src, WT, out_t, out_k, 66, tau_syn=tau_syn)


def _handmade(torch, lif, label, ev_t, ev_src, WT, out_t, out_k, seed, ev_n=None, out_i=None, **kw):
    """The backward alone on a spike train given by hand, out_t and out_k
    [B][N][S] with infinite times past the last spike."""
    B, E = ev_t.shape
    ev_n = np.full(B, E, np.int32) if ev_n is None else ev_n
    rng = np.random.default_rng(seed)
    valid = np.isfinite(out_t)
    out_n = valid.sum(-1).astype(np.int32)
    if out_i is None:
        out_i = np.where(valid, 1.5 + rng.random(out_t.shape), 0.0)
    out_i = out_i.astype(np.float32)
    g = (rng.standard_normal(out_t.shape) * valid).astype(np.float32)
    S = out_t.shape[-1]
    r = oracle.ForwardResult(out_t.astype(np.float64), out_i.astype(np.float64), out_n, None, None, None, out_k.astype(np.int32))
    oW, oT = oracle.backward(ev_t, ev_src, ev_n, WT, r, g.astype(np.float64), oracle.LifParams(s_max=S, **kw))
    d = [_dev(torch, a) for a in (ev_t, ev_src, ev_n, WT)]
    fwd = lif.ForwardOut(_dev(torch, out_t.astype(np.float32)), _dev(torch, out_n), _dev(torch, out_i), None,
                         _dev(torch, out_k.astype(np.int32)))
    gW, gT = lif.backward(*d, fwd, _dev(torch, g), lif.Params(s_max=S, **kw))
    torch.cuda.synchronize()
    sW, sT = compare_grad(gW.cpu().numpy(), oW, label="gW"), compare_grad(gT.cpu().numpy(), oT, label="gT")
    print(f"[case] {label} spikes={int(out_n.sum())} rel(gW)={sW:.2e} rel(gT)={sT:.2e}", flush=True)


@pytest.mark.parametrize("tau_syn", [0.0038, 0.0076, 0.005])
def test_adjoint_spikes_on_references(env, tau_syn):
    """A stream over many references (multiples of 100 tau_s, to which the
    exponentials are referred) with spikes at exactly such times: 25 of them
    are 9.5 s and 19 s, which their reciprocals put on either side."""
    torch, lif = env
    rng = np.random.default_rng(64)
    B, C, N, E = 2, 9, 66, 200
    at = np.float32(2500 * tau_syn)
    ev_t = np.sort(rng.random((B, E)) * 2 * at, -1).astype(np.float32)
    ev_t[:, E // 2:] = np.maximum(ev_t[:, E // 2:], at)
    ev_t[:, :E // 2] = np.minimum(ev_t[:, :E // 2], np.nextafter(at, np.float32(0)))
    ev_t[:, E // 2 - 4:E // 2] = at - np.linspace(3, 0.5, 4, dtype=np.float32) * np.float32(tau_syn)
    ev_t.sort(-1)
    out_t = np.full((B, N, 2), np.inf)
    out_k = np.zeros((B, N, 2), np.int32)
    out_t[:, :, 0], out_k[:, :, 0] = at, E // 2
    out_t[:, ::2, 1] = ev_t[:, -1:] + 0.5 * tau_syn
    out_k[:, ::2, 1] = E
    _handmade(torch, lif, f"tau_s={tau_syn}", ev_t, rng.integers(0, C, (B, E)).astype(np.int32),
              rng.standard_normal((C, N)).astype(np.float32), out_t, out_k, 64, tau_syn=tau_syn)


@pytest.mark.parametrize("C,n", [(40, 1500), (700, 3000)])
@pytest.mark.parametrize("back", [2e-4, 5e-3])
def test_adjoint_spike_times_before_their_events(env, C, n, back):
    """Spike times moved back past some of the events that the spikes follow
    (within a group of eight, across groups and blocks): out_k decides which
    events count, with offsets of 0."""
    torch, lif = env
    B, N = 2, 70
    cfg = W.random_small(65, B=B, C=C, N=N, n_events=n, T=0.5, gain=10.0, ragged=False)
    ev, WT = cfg.events, cfg.layers[0].WT
    r = oracle.forward(ev.ev_t, ev.ev_src, ev.ev_n, WT, oracle.LifParams(s_max=64)).rounded()
    rng = np.random.default_rng(65)
    t = r.out_t - np.where(rng.random(r.out_t.shape) < 0.5, rng.random(r.out_t.shape) * back, 0.0)
    # (times stay in order, also in float32)
    t = np.maximum.accumulate(np.maximum(t, 0.0).astype(np.float32), -1).astype(np.float64)
    assert int((t < r.out_t).sum()) > 50
    _handmade(torch, lif, f"C={C} back={back}", ev.ev_t, ev.ev_src, WT, t, r.out_k, 65)


@pytest.mark.parametrize("n", [500, 5000])
@pytest.mark.parametrize("scale", [1.0, 1e6])
@pytest.mark.parametrize("bad", [("nan", "inf"), ("nan",), ("inf",)])
def test_adjoint_not_finite(env, n, scale, bad):
    """A NaN and an infinite upstream gradient on one neuron each leave every
    other neuron's dL/dW column as it is without them, whatever the size of
    their own (at 1e6 their fixed-point sums need the scale of the finite
    neurons)."""
    torch, lif = env
    cfg = W.random_small(63, B=2, C=30, N=66, n_events=n, T=0.4, gain=14.0)
    ev, WT = cfg.events, cfg.layers[0].WT
    d = [_dev(torch, a) for a in (ev.ev_t, ev.ev_src, ev.ev_n, WT)]
    P = lif.Params(s_max=128)
    out = lif.forward(*d, P)
    g = scale * torch.randn(out.out_t.shape, generator=torch.Generator(device="cuda:0").manual_seed(1), device="cuda:0")
    base, _ = lif.backward(*d, out, g, P)
    fired = (out.out_n[0] > 0).nonzero().flatten().tolist()
    h = g.clone()
    for i, v in zip(fired, bad):
        h[0, i, 0] = float(v)
    got, gT = lif.backward(*d, out, h, P)
    torch.cuda.synchronize()
    keep = [i for i in range(66) if i not in fired[:len(bad)]]
    # the bound of the fixed-point scale is not the same in the two calls
    assert torch.allclose(got[:, keep], base[:, keep], rtol=1e-5, atol=1e-6 * float(base.abs().max()))
    if "nan" in bad:
        assert torch.isnan(gT[0]).any()


@pytest.mark.parametrize("C", [1, 318, 319, 700])
@pytest.mark.parametrize("time_grad", [True, False])
def test_adjoint_empty_queues(env, C, time_grad):
    """Queues without room for an event: dL/dW is zero whatever the workspace
    held, on both sides of one channel range."""
    torch, lif = env
    B, N, P = 3, 70, lif.Params(s_max=8)
    print(f"[case] empty queues C={C} time_grad={time_grad}", flush=True)
    ev_t = torch.empty((B, 0), device="cuda:0")
    ev_s = torch.empty((B, 0), dtype=torch.int32, device="cuda:0")
    ev_n = torch.zeros(B, dtype=torch.int32, device="cuda:0")
    WT = torch.ones((C, N), device="cuda:0")
    out = lif.forward(ev_t, ev_s, ev_n, WT, P)
    ws = torch.full((lif.lif_layer_backward_workspace_size(B, 0, C, N, P.c()),), 1, dtype=torch.uint8, device="cuda:0")
    gW, gT = lif.backward(ev_t, ev_s, ev_n, WT, out, torch.ones_like(out.out_t), P, want_time_grad=time_grad, ws=ws)
    torch.cuda.synchronize()
    assert int(out.out_n.sum()) == 0 and not gW.any()
    assert gT is None if not time_grad else gT.numel() == 0
