"""The merge's bucket sort and its bitonic fallback, and the readout's chunks
and class groups, at their edges: the merge bit for bit against numpy's sort of
(time, neuron, spike), the readout against the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import loss as OL
from tests.test_gpu_loss import _dev, env, run_case  # noqa: F401

pytestmark = pytest.mark.gpu


def _trains(rng, B, N, S, kind):
    n = rng.integers(0, S + 1, (B, N)).astype(np.int32)
    n[0] = 0                                             # an empty sample
    if kind == "uniform":
        t = rng.random((B, N, S))
    elif kind == "piled":                                # all spikes at a few times: bins of thousands
        t = rng.integers(1, 4, (B, N, S)) / 8.0
    elif kind == "outlier":                              # one far spike: nearly all others in one bin
        t = rng.random((B, N, S)) * 1e-3
        n[1, 0] = max(int(n[1, 0]), 1)
        t[1, 0, 0] = 1e6
    else:                                                # "bursts": volleys of a few hundred microseconds
        t = rng.integers(0, 40, (B, N, S)) * 0.02 + rng.random((B, N, S)) * 3e-4
    t = np.sort(t.astype(np.float32), -1)
    t[np.arange(S) >= n[..., None]] = np.inf
    return np.sort(t, -1), n


@pytest.mark.parametrize("N,S,E2", [(1, 2, 2), (3, 5, 9), (64, 16, 1024), (97, 40, 16384), (200, 96, 16384), (512, 64, 5000)])
@pytest.mark.parametrize("kind", ["uniform", "piled", "outlier", "bursts"])
def test_merge_sorts(env, N, S, E2, kind):
    torch, lif = env
    rng = np.random.default_rng(5)
    t, n = _trains(rng, 3, N, S, kind)
    print(f"[case] merge N={N} S={S} E2={E2} {kind}", flush=True)
    t2, s2, n2, perm, _ = lif.merge(lif.ForwardOut(_dev(torch, t), _dev(torch, n), None, None), E2)
    torch.cuda.synchronize()
    for b in range(3):
        flat = t[b].reshape(-1)
        order = np.argsort(flat, kind="stable")          # equal times in (neuron, spike) order
        k = min(int(n[b].sum()), E2)
        assert int(n2[b]) == k
        assert np.array_equal(perm[b].cpu().numpy()[:k], order[:k])
        assert np.array_equal(t2[b].cpu().numpy()[:k], flat[order[:k]])
        assert np.array_equal(s2[b].cpu().numpy()[:k], order[:k] // S)
        assert np.all(np.isinf(t2[b].cpu().numpy()[k:])) and np.all(perm[b].cpu().numpy()[k:] == -1)


@pytest.mark.parametrize("B,C,K,n", [(1, 1, 1, 1), (2, 7, 2, 255), (3, 40, 3, 256), (9, 300, 33, 257), (70, 20, 64, 1100)])
def test_readout_edges(env, B, C, K, n):
    ev = W.random_small(7, B=B, C=C, N=2, n_events=n, T=1.0, gain=1.0).events
    rng = np.random.default_rng(8)
    WT = (rng.normal(0, 1, (C, K)) * 2).astype(np.float32)
    run_case(env, ev, WT, OL.LiParams(), rng.integers(0, K, B).astype(np.int32), f"B{B} C{C} K{K} n{n}")
