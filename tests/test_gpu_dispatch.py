"""Dispatch by size: launches on either side of a size rule give the same results,
and those of the oracle."""
import numpy as np
import pytest

from paper_2606_17081_amd import workload as wl
from test_gpu_parity import _compare_episode, _oracle_episode, gpu, say  # noqa: F401

pytestmark = pytest.mark.gpu


def _mixed_workload():
    """Every option of an episode on a single-turn and a multi-turn trace, caches under pressure."""
    traces = {1: wl.tiny_trace(1, 700), 2: wl.multiturn_trace(2, 40)}
    options = [dict(), dict(controller=1, ctrl_window=40, cap=300), dict(controller=2),
               dict(policy=wl.POLICY_SOFTMAX, tau=16.0),
               dict(policy=wl.POLICY_P2C), dict(policy=wl.POLICY_RANDOM), dict(policy=wl.POLICY_ROUND_ROBIN),
               dict(evict_policy=wl.EVICT_FREQ, decay_steps=5), dict(evict_policy=wl.EVICT_FREQ, decay_steps=200),
               dict(tier_g1=150, tier_g2=250)]
    eps = [wl.EpisodeSpec(**{**dict(seed=s, concurrency=C, cap=2048), **o}) for s in traces for C in (8, 100)
           for o in options]
    return wl.Workload("mixed", W=5, cache_blocks=700, traces=traces, episodes=eps)


def test_workgroup_widths(gpu, orc):
    """Up to one workgroup per compute unit the episodes run on 512 threads, beyond on 256."""
    torch, rk = gpu
    from paper_2606_17081_amd.episodes import EpisodeRunner
    w = _mixed_workload()
    n = len(w.episodes)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    many = w.episodes * (cus // n + 1)
    assert n < cus < len(many)
    ref, cache = None, {}
    for label, eps, slots in (("wide", w.episodes, 0), ("narrow", many, 0), ("wide, queued", w.episodes, 7),
                              ("narrow, queued", many, cus + 3)):
        say(label, len(eps), "episodes,", slots, "workspaces")
        r = EpisodeRunner(w, eps, ws_slots=slots)
        r.step()
        torch.cuda.synchronize()
        assert rk.device_status(reset=True) == 0
        got = [r.episode_results(e) for e in (range(n) if len(eps) == n else range(len(eps) - n, len(eps)))]
        if ref is None:
            ref = got
            for e, sp in enumerate(eps):
                o = _oracle_episode(orc, w, sp, cache)
                assert o["totals"][1] > 0
                _compare_episode(got[e], o, w.W, window=sp.concurrency, label=f"{label} {e}")
        order = range(n) if len(eps) == n else [(len(eps) - n + k) % n for k in range(n)]
        for k, e in enumerate(order):
            for key, v in ref[e].items():
                assert np.array_equal(got[k][key], v), (label, e, key)
