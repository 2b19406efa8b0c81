"""The forward's wave-per-neuron resolve pass (calls that flag many sub-blocks):
against the oracle and, bit for bit where both apply, across pool sizes; bursts
of spikes within an interval's window, caps, both root solvers, resets below
rest, open intervals, and streams longer than a candidate chunk.  Every case is
above the pass's line in size; the last one flags too few sub-blocks for it."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_forward import _dev, check, env  # noqa: F401

pytestmark = pytest.mark.gpu

MOST = 65536            # flagged sub-blocks from which the pass runs


def _layer(seed, n, gain, B=64, C=50, N=256, T=0.7):
    cfg = W.random_small(seed, B=B, C=C, N=N, n_events=n, T=T, gain=gain)
    return cfg.events, cfg.layers[0].WT


@pytest.mark.parametrize("kw", [
    dict(s_max=256),
    dict(s_max=256, tau_syn=0.0061),                     # the exponential solve
    dict(s_max=256, v_reset=-0.4, t_end=0.69),           # queues that go on past t_end
    dict(s_max=256, v_reset=-0.4, t_end=0.9),
    dict(s_max=5),                                       # the cap binds
])
def test_wave_pass(env, kw):
    ev, WT = _layer(71, 4300, 9.0)
    s = check(env, ev, WT, f"wave {kw}", both=False, **kw)
    assert s["par"]["status"][3] > MOST and s["par"]["spikes"] > 2000


def test_wave_pass_long_streams(env):
    ev, WT = _layer(72, 20000, 7.0, B=8, N=520, T=1.6)   # three candidate chunks
    s = check(env, ev, WT, "wave long", both=False, s_max=256)
    assert s["par"]["status"][3] > MOST


def test_wave_pass_pools(env):
    torch, lif = env
    ev, WT = _layer(73, 4300, 9.0)
    d = [_dev(torch, a) for a in (ev.ev_t, ev.ev_src, ev.ev_n, WT)]
    outs = [lif.forward(*d, lif.Params(s_max=256, pool_cap=pc)) for pc in (-1, 0, 700)]
    torch.cuda.synchronize()
    assert int(outs[0].status[3]) > MOST and int(outs[1].status[7]) > MOST
    for o in outs[1:]:
        for a, b in ((o.out_t, outs[0].out_t), (o.out_i, outs[0].out_i), (o.out_n, outs[0].out_n), (o.out_k, outs[0].out_k)):
            assert torch.equal(a, b)


def test_few_flagged_take_the_ring(env):
    ev, WT = _layer(74, 4300, 0.6)
    s = check(env, ev, WT, "few flagged", both=False)
    assert s["par"]["status"][3] <= MOST


def test_many_flagged_of_few_stay_on_the_ring(env):
    """Below 2^22 sub-blocks in all the ring takes every call, also one that flags
    more than the line between the passes."""
    ev, WT = _layer(75, 4300, 9.0, B=20)
    assert 20 * 256 * 4 * -(-ev.E_max // 64) <= 1 << 22
    s = check(env, ev, WT, "dense ring", both=False, s_max=256)
    assert s["par"]["status"][3] > MOST
