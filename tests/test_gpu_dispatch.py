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


@pytest.mark.parametrize("cache,option", [(c, o) for c in (60, 400, 2500)
                                          for o in (dict(), dict(evict_policy=wl.EVICT_FREQ, decay_steps=3))])
def test_eviction_rounds(gpu, orc, cache, option):
    """An eviction reads its log in rounds, a short one first where it looks for few victims: few and many,
    live records spread evenly, crowded at the tail by conversations read again and again, and kept
    at the head by their frequency."""
    torch, rk = gpu
    from paper_2606_17081_amd.episodes import EpisodeRunner
    traces = {1: wl.tiny_trace(1, 400), 2: wl.multiturn_trace(2, 30), 3: wl.saturation_trace(3, 150)}
    eps = [wl.EpisodeSpec(seed=s, concurrency=C, cap=2048, **option) for s in traces for C in (8, 64)]
    w = wl.Workload("evictions", W=3, cache_blocks=cache, traces=traces, episodes=eps)
    r = EpisodeRunner(w)
    r.step()
    torch.cuda.synchronize()
    assert rk.device_status(reset=True) == 0
    oracle, evicted = {}, 0
    for e, sp in enumerate(eps):
        o = _oracle_episode(orc, w, sp, oracle)
        evicted = max(evicted, int(o["evict_count"].max()))
        _compare_episode(r.episode_results(e), o, w.W, window=sp.concurrency, label=f"{cache} {e}")
    assert evicted > 64                                # more than one group of records in an eviction


@pytest.mark.parametrize("W,m,spare", [(1, 9, 0), (3, 64, 0), (6, 32, 0), (6, 300, 40), (16, 8, 0), (16, 65, 3),
                                       (16, 256, 0), (16, 256, 4), (16, 256, 20), (32, 255, 1), (33, 130, 0),
                                       (64, 64, 0), (64, 200, 1), (64, 512, 0)])
@pytest.mark.parametrize("levels", [(0.0,), (0.0, 0.5), (0.0, 0.1, 0.3, 0.35, 0.7, 1.0)])
def test_poa_free_places(gpu, orc, W, m, spare, levels):
    """The optimum starts from priced placements when nearly all of the K W places are taken and
    without prices otherwise; spare adds places to K = ceil(m / W).  Overlaps from few levels tie
    whole rows, and workers of very unequal counts make the prices matter."""
    torch, rk = gpu
    rng = np.random.default_rng([W, m, spare, len(levels)])
    K = -(-m // W) + spare
    n = 3 * m
    P = rng.integers(1, 300, n).astype(np.int32)
    am = np.minimum(rng.integers(0, W, n), rng.integers(0, W, n)).astype(np.int32)
    ov = np.floor(rng.choice(levels, size=(n, W)) * P[:, None]).astype(np.int32)
    ov[m: 2 * m] = ov[m: 2 * m, :1]                    # a window of rows cached alike everywhere
    up, pp = rk.to_device, dict(wl.POA_PARAMS)
    sel, coo = (torch.zeros(3, dtype=torch.float64, device="cuda") for _ in range(2))
    hat = torch.zeros(1, dtype=torch.float64, device="cuda")
    params = rk.PoaParams(pp["a"], pp["b"], pp["d"], pp["beta"], pp["C_cap"], pp["w_c"], K)
    ws = torch.empty(rk.poa_workspace_size(n, W), dtype=torch.uint8, device="cuda")
    rk.poa_estimate(up(np.arange(0, n + 1, m, dtype=np.int64)), up(np.array([0, 3], np.int64)), n, m, W, up(am), up(ov),
                    up(P), params, sel, coo, hat, ws)
    torch.cuda.synchronize()
    assert rk.device_status(reset=True) == 0
    for w in range(3):
        r = slice(w * m, (w + 1) * m)
        s, c, _ = orc.poa_window(am[r], ov[r], P[r], W, K=K, **pp)
        # sums of at most 512 fp32 costs in fp64 on both sides
        assert float(sel[w]) == pytest.approx(s, rel=1e-13) and float(coo[w]) == pytest.approx(c, rel=1e-13)


@pytest.mark.parametrize("W,m,spare", [(8, 20, 1), (16, 256, 2), (17, 40, 0), (32, 256, 0), (33, 70, 0), (40, 3, 0),
                                       (48, 130, 1), (49, 4, 0), (49, 5, 0), (64, 3, 0), (64, 64, 0)])
def test_poa_many_windows(gpu, orc, W, m, spare):
    """Few windows, in index order, and many, ordered by length, choose their wavefronts by other
    rules; either side gives a window's sums, and those of the oracle."""
    torch, rk = gpu
    rng = np.random.default_rng([W, m, spare])
    lens = rng.integers(1, m + 1, 10)
    lens[0] = m
    n, K = int(lens.sum()), (-(-m // W) + spare) if spare else 0
    P = rng.integers(1, 300, n).astype(np.int32)
    am = np.minimum(rng.integers(0, W, n), rng.integers(0, W, n)).astype(np.int32)
    ov = np.floor(rng.choice((0.0, 0.25, 0.5, 0.9), size=(n, W)) * P[:, None]).astype(np.int32)
    up, pp = rk.to_device, dict(wl.POA_PARAMS)
    params = rk.PoaParams(pp["a"], pp["b"], pp["d"], pp["beta"], pp["C_cap"], pp["w_c"], K)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    sums = []
    for copies in (1, 4 * cus // len(lens) + 2):
        nw, rows = len(lens) * copies, n * copies
        win = np.concatenate([[0], np.cumsum(np.tile(lens, copies))]).astype(np.int64)
        sel, coo = (torch.zeros(nw, dtype=torch.float64, device="cuda") for _ in range(2))
        hat = torch.zeros(1, dtype=torch.float64, device="cuda")
        ws = torch.empty(rk.poa_workspace_size(rows, W), dtype=torch.uint8, device="cuda")
        rk.poa_estimate(up(win), up(np.array([0, nw], np.int64)), rows, m, W, up(np.tile(am, copies)),
                        up(np.tile(ov, (copies, 1))), up(np.tile(P, copies)), params, sel, coo, hat, ws)
        torch.cuda.synchronize()
        assert rk.device_status(reset=True) == 0
        sums.append((sel.cpu().numpy().reshape(copies, -1), coo.cpu().numpy().reshape(copies, -1)))
    assert len(lens) <= 2 * cus < 4 * cus < nw
    at = np.concatenate([[0], np.cumsum(lens)])
    for w in range(len(lens)):
        r = slice(at[w], at[w + 1])
        s, c, _ = orc.poa_window(am[r], ov[r], P[r], W, K=K or -(-int(lens[w]) // W), **pp)
        for sel, coo in sums:                       # sums of at most 256 fp32 costs in fp64 on both sides
            np.testing.assert_allclose(sel[:, w], s, rtol=1e-13)
            np.testing.assert_allclose(coo[:, w], c, rtol=1e-13)


def test_poa_largest_window(gpu):
    """4,096 rows on 64 workers, the most LDS a window takes: without overlaps every worker's 64 places
    are taken at its base cost."""
    torch, rk = gpu
    W, m = 64, 4096
    am = np.random.default_rng(1).integers(0, W, m).astype(np.int32)
    up, pp = rk.to_device, dict(wl.POA_PARAMS)
    sel, coo, hat = (torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(3))
    ws = torch.empty(rk.poa_workspace_size(m, W), dtype=torch.uint8, device="cuda")
    rk.poa_estimate(up(np.array([0, m], np.int64)), up(np.array([0, 1], np.int64)), m, m, W, up(am),
                    up(np.zeros((m, W), np.int32)), up(np.ones(m, np.int32)),
                    rk.PoaParams(pp["a"], pp["b"], pp["d"], pp["beta"], pp["C_cap"], pp["w_c"], 0), sel, coo, hat, ws)
    torch.cuda.synchronize()
    assert rk.device_status(reset=True) == 0
    n = np.bincount(am, minlength=W).astype(np.float32)
    gap = np.maximum(np.float32(pp["C_cap"]) - n, 1).astype(np.float32)
    base = (np.float32(pp["a"]) * n + np.float32(pp["b"])) + np.float32(pp["d"]) / (gap * gap)
    assert float(sel) == pytest.approx(float(base[am].astype(np.float64).sum()), rel=1e-13)
    assert float(coo) == pytest.approx(64 * float(base.astype(np.float64).sum()), rel=1e-13)


@pytest.mark.parametrize("n_seq", [1, 3, 8192, 8193])
def test_hash_few_and_many_sequences(gpu, orc, n_seq):
    """Up to 8,192 sequences take a workgroup each, more a lane each: lengths around the spans of
    64 and 256 blocks, partial blocks, token ranges at odd addresses and ranges that are too short."""
    torch, rk = gpu
    rng = np.random.default_rng(n_seq)
    edges = np.array([0, 1, 2, 63, 64, 65, 255, 256, 257, 511, 512, 513, 700])
    blocks = np.concatenate([edges, rng.integers(0, 40, n_seq)])[:n_seq] if n_seq > 3 else np.array([513, 700, 65])[:n_seq]
    short = rng.random(n_seq) < 0.05                       # a token short of the last block
    length = np.maximum(16 * blocks + rng.integers(0, 16, n_seq) - 16 * (short & (blocks > 0)), 0)
    tok_off, chain_off = (np.concatenate([[3 * k], 3 * k + np.cumsum(x)]).astype(np.int64)
                          for k, x in ((1, length), (0, blocks)))
    tokens = rng.integers(-2 ** 31, 2 ** 31, int(tok_off[-1]) + 1).astype(np.int32)
    ch = torch.full((int(chain_off[-1]) + 1,), 77, dtype=torch.int64, device="cuda")
    rk.hash_chains(rk.to_device(tokens), rk.to_device(tok_off), rk.to_device(chain_off), ch)
    torch.cuda.synchronize()
    bits = rk.device_status(reset=True)
    assert bits == (2 if (length // 16 < blocks).any() else 0)
    got = rk.to_host_u64(ch)
    assert got[-1] == 77
    for s in range(n_seq):
        n = int(min(blocks[s], length[s] // 16))
        row = got[chain_off[s]: chain_off[s + 1]]
        assert not row[n:].any()
        ref = orc.hash_chains(tokens[tok_off[s]: tok_off[s] + 16 * n], [0, 16 * n], [n])
        assert np.array_equal(row[:n], np.asarray(ref, np.uint64)[:n]), s


def _index_slots(rk, idx):
    """The occupied slots of an index: {key: mask}, and the slot of each key."""
    a = idx.cpu().numpy().view(np.uint64).reshape(-1, 2)
    s = np.nonzero(a[:, 0])[0]
    assert not a[a[:, 0] == 0, 1].any()
    return {int(k): int(m) for k, m in a[s]}, dict(zip(a[s, 0].tolist(), s.tolist())), a[:, 0] != 0


@pytest.mark.parametrize("log2,W,kind", [(19, 5, "uniform"), (20, 64, "uniform"), (20, 3, "dense"), (21, 64, "shared"),
                                         (22, 7, "uniform"), (22, 2, "ends"), (20, 2, "skewed"), (20, 1, "zeros"),
                                         (22, 40, "uniform")])
def test_index_build_partitioned(gpu, log2, W, kind):
    """From 2^20 slots on the index is partitioned and built in LDS: every key in its probe order from
    its home slot with the workers that hold it, at load 0.5, for uniform keys, keys shared by all
    workers, keys whose home slots run on over the ends of sub-bins, bins and the table, keys that
    crowd into a few bins (built by atomics instead) and zero keys."""
    torch, rk = gpu
    rng = np.random.default_rng([log2, W])
    slots = 1 << log2
    n = slots // 2 // W
    hi = rng.permutation(np.arange(1, W * n + 1, dtype=np.uint64)) << np.uint64(32)
    if kind == "shared":
        keys = np.tile(hi[:n] | rng.integers(0, 2 ** 32, n, dtype=np.uint64), W)
    elif kind == "dense":
        keys = hi | np.arange(W * n, dtype=np.uint64)
    elif kind == "ends":
        # 40 keys at the last slots of every 8,192, among them the table's last
        m = min(W * n, 40 * (slots >> 13))
        low = (np.arange(m, dtype=np.uint64) // np.uint64(40) << np.uint64(13)) + np.uint64(8185) + rng.integers(
            0, 7, m, dtype=np.uint64)
        n = m // W
        keys = (hi[:m] | low)[: W * n]
    elif kind == "skewed":
        keys = hi | rng.integers(0, slots >> 6, W * n, dtype=np.uint64)
    else:
        keys = hi | rng.integers(0, 2 ** 32, W * n, dtype=np.uint64)
    keys = np.where(rng.random(keys.size) < 0.001, 0, keys) if kind == "zeros" else keys
    off = np.arange(W + 1, dtype=np.int64) * n
    want = {}
    for j in range(W):
        for k in keys[off[j]: off[j + 1]].tolist():
            want[k] = want.get(k, 0) | 1 << j
    zeros = want.pop(0, None)
    up = rk.to_device(np.ascontiguousarray(keys))
    for turn in range(2):                           # over whatever the buffer held
        idx = torch.full((2 * slots,), -1 if turn else 5, dtype=torch.int64, device="cuda")
        rk.index_build(up, off, log2, idx)
        torch.cuda.synchronize()
        assert rk.device_status(reset=True) == (4 if zeros else 0)
        got, where, full = _index_slots(rk, idx)
        assert got == want
        # no empty slot between a key's home and its slot
        holes = np.concatenate([[0], np.cumsum(~np.concatenate([full, full]))])
        at = np.array([where[k] for k in want])
        home = (np.array(list(want), np.uint64) & np.uint64(slots - 1)).astype(np.int64)
        at = np.where(at < home, at + slots, at)
        assert (holes[at] == holes[home]).all()


def _assert_index(torch, keys, off, log2, out):
    """The index holds the key sets and nothing else, every key in its probe order from its home slot."""
    W = len(off) - 1
    worker = torch.repeat_interleave(torch.arange(W, device="cuda"), torch.from_numpy(np.diff(off)).cuda())
    want, at = torch.unique(keys, return_inverse=True)
    mask = torch.zeros_like(want).index_add_(0, at, torch.ones_like(worker) << worker)    # (no pair twice)
    slot = torch.nonzero(out.view(-1, 2)[:, 0]).flatten()
    key, k = torch.sort(out.view(-1, 2)[slot, 0])
    assert torch.equal(key, want) and torch.equal(out.view(-1, 2)[slot, 1][k], mask)
    empty = out.view(-1, 2)[:, 0] == 0
    assert not (out.view(-1, 2)[:, 1] != 0).logical_and_(empty).any()
    holes = torch.cumsum(empty, 0, dtype=torch.int32)         # empty slots up to each
    home, total = out.view(-1, 2)[slot, 0] & ((1 << log2) - 1), holes[-1]
    wrapped = (slot < home).int()
    assert torch.equal(holes[slot] + wrapped * total, holes[home] - empty[home].int())


# low bits of keys that every worker holds (shared) and of the first worker's own; what they reach
_CROWDED = {
    "64 past a sub-bin's end": lambda lg: ([8191] * 5, [8191] * 60),
    "65 past a sub-bin's end": lambda lg: ([8191] * 5, [8191] * 61),
    "64 out of a bin": lambda lg: ([], [*range(8192, 16384), *[16383] * 30, *[8191] * 35]),
    "65 out of a bin": lambda lg: ([], [*range(8192, 16384), *[16383] * 30, *[8191] * 36]),
    "through three sub-bins": lambda lg: ([], [*range(8192, 24576), *[8191] * 50, *[24575] * 20]),
    "out of the index": lambda lg: ([(1 << lg) - 1] * 9, [(1 << lg) - 2] * 30),
    "a first sub-bin's entries to the limit": lambda lg: ([7 + 30 * i for i in range(256)], []),
    "a first sub-bin's entries past it": lambda lg: ([7 + 30 * i for i in range(257)], []),
}


@pytest.mark.parametrize("log2,W,kind", [
    (25, 64, "uniform"), (25, 3, "uniform"), (29, 2, "uniform"),
    (22, 9, "64 past a sub-bin's end"), (22, 9, "65 past a sub-bin's end"), (22, 1, "64 out of a bin"),
    (22, 1, "65 out of a bin"), (25, 2, "through three sub-bins"), (22, 9, "out of the index"),
    (29, 9, "out of the index"), (23, 64, "a first sub-bin's entries to the limit"),
    (23, 64, "a first sub-bin's entries past it")])
def test_index_build_sub_bins(gpu, log2, W, kind):
    """The partitioned index with 2 to 256 sub-bins of 8,192 slots in each of its 256 bins: uniform keys,
    and keys that fill what may pass an end (64 keys) or lie before a sub-bin's place (16,384 entries),
    or run it over by one, which is found after other bins have been written."""
    torch, rk = gpu
    g = torch.Generator(device="cuda").manual_seed(log2 + W)
    if kind == "uniform":
        n = min((1 << log2) // 2, 1 << 24) // W
        low = torch.randint(0, 1 << 32, (W * n,), generator=g, device="cuda")
        keys, off = (torch.arange(1, W * n + 1, device="cuda") << 32) | low, np.arange(W + 1, dtype=np.int64) * n
    else:
        shared, own = (torch.tensor(x, dtype=torch.int64, device="cuda") for x in _CROWDED[kind](log2))
        number = torch.randperm(shared.numel() + own.numel(), generator=g, device="cuda") + 1
        shared, own = shared | number[: shared.numel()] << 32, own | number[shared.numel():] << 32
        keys = torch.cat([own] + [shared[torch.randperm(shared.numel(), generator=g, device="cuda")] for _ in range(W)])
        off = np.concatenate([[0], own.numel() + shared.numel() * np.arange(1, W + 1)]).astype(np.int64)
    out = torch.full((2 << log2,), 5, dtype=torch.int64, device="cuda")
    for _ in range(2):
        rk.index_build(keys, off, log2, out)
        torch.cuda.synchronize()
        assert rk.device_status(reset=True) == 0
        _assert_index(torch, keys, off, log2, out)


def test_index_build_streams_and_capture(gpu):
    """Builds on several streams at once, and one captured into a graph, give the same index."""
    torch, rk = gpu
    rng = np.random.default_rng(9)
    log2, W, n = 20, 16, 20000
    sets = [(np.arange(1, W * n + 1, dtype=np.uint64) << np.uint64(32)) | rng.integers(0, 2 ** 32, W * n, dtype=np.uint64)
            for _ in range(6)]
    off = np.arange(W + 1, dtype=np.int64) * n
    ups = [rk.to_device(k) for k in sets]
    idx = [torch.empty(2 << log2, dtype=torch.int64, device="cuda") for _ in sets]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in sets]
    for _ in range(3):
        for k, s in enumerate(streams):
            rk.index_build(ups[k], off, log2, idx[k], stream=s)
    torch.cuda.synchronize()
    ref = [_index_slots(rk, i)[0] for i in idx]
    for k, keys in enumerate(sets):
        assert ref[k] == {int(x): 1 << (i // n) for i, x in enumerate(keys)}
    g = torch.cuda.CUDAGraph()
    cap = torch.empty(2 << log2, dtype=torch.int64, device="cuda")
    with torch.cuda.graph(g):
        rk.index_build(ups[0], off, log2, cap)
    for _ in range(3):
        cap.fill_(3)
        g.replay()
        torch.cuda.synchronize()
        assert _index_slots(rk, cap)[0] == ref[0]
    assert rk.device_status(reset=True) == 0


@pytest.mark.parametrize("log2,W,kind", [(14, 140, "uniform"), (15, 63, "uniform"), (15, 70, "uniform"), (15, 64, "ends"),
                                         (16, 32, "dense"), (18, 8, "skewed"), (20, 3, "uniform"), (22, 1, "zeros"),
                                         (23, 1, "uniform"), (17, 66, "few"), (15, 64, "500 past an end"),
                                         (15, 64, "600 past an end"), (15, 70, "600 past an end")])
def test_table_build_partitioned(gpu, log2, W, kind):
    """Tables of 2^15 to 2^22 slots, 2^21 in all or more, are partitioned and built in LDS, others by
    atomics: every key of a worker in its probe order from its home slot, at load 0.5 or below.  Of the
    partitioned ones, "dense" fills bins' lists to the last entry, "skewed" runs one over, and the keys
    past the bins' ends fill their buffer (2^15) almost, or run it over."""
    torch, rk = gpu
    rng = np.random.default_rng([log2, W, 3])
    slots = 1 << log2
    assert (15 <= log2 <= 22 and W * slots >= 1 << 21) == ((log2, W) not in ((14, 140), (15, 63), (23, 1)))
    n = np.full(W, slots // 2)
    if kind == "skewed":
        n = np.full(W, 20000)                       # in the first of the 2^14 slots of a bin
    if "past" in kind:
        n = np.full(W, int(kind[:3]))
        assert (W * (n[0] - 1) > 1 << 15) == (kind[:3] == "600")
    if kind == "few":
        n = rng.integers(0, 5, W)
    if kind == "ends":
        n = np.full(W, 20 * (slots >> 13))
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    hi = rng.permutation(np.arange(1, off[-1] + 1, dtype=np.uint64)) << np.uint64(32)
    if kind == "dense":
        low = np.arange(off[-1], dtype=np.uint64)
    elif kind == "ends":
        low = (rng.integers(0, slots >> 13, off[-1], dtype=np.uint64) << np.uint64(13)) + np.uint64(8185)
    elif kind == "skewed":
        low = rng.integers(0, slots >> 5, off[-1], dtype=np.uint64)
    elif "past" in kind:
        low = np.full(off[-1], (1 << 14) - 1, np.uint64)
    else:
        low = rng.integers(0, 2 ** 32, off[-1], dtype=np.uint64)
    keys = hi | low
    if kind == "zeros":
        keys[rng.random(keys.size) < 0.001] = 0
    if off[-1] > 10 and W > 1 and "past" not in kind:
        keys[off[1] - 1] = keys[off[0]]             # a worker's key twice
    up = rk.to_device(keys)
    for fill in (-1, 5):
        t = torch.full((W * slots,), fill, dtype=torch.int64, device="cuda")
        rk.table_build(up, off, log2, t)
        torch.cuda.synchronize()
        assert rk.device_status(reset=True) == (4 if kind == "zeros" else 0)
        got = t.cpu().numpy().view(np.uint64).reshape(W, slots)
        for j in range(W):
            want = np.unique(keys[off[j]: off[j + 1]])
            want = want[want != 0]
            at = np.nonzero(got[j])[0]
            assert np.array_equal(np.sort(got[j][at]), want), j
            empty = got[j] == 0
            holes = np.concatenate([[0], np.cumsum(np.concatenate([empty, empty]))])
            home = (got[j][at] & np.uint64(slots - 1)).astype(np.int64)
            at = np.where(at < home, at + slots, at)
            assert (holes[at] == holes[home]).all(), j


def _ms(torch, f):
    """Median time of f in milliseconds, after a first run."""
    t = []
    for _ in range(6):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        t.append(a.elapsed_time(b))
    return sorted(t[1:])[2]


@pytest.mark.parametrize("layout,log2,W", [("index", 24, 1), ("index", 24, 3), ("tables", 21, 1), ("tables", 20, 5)])
def test_crowded_keys_fill_the_chip(gpu, layout, log2, W):
    """Keys that crowd at one place are inserted by atomics after a partition that did not fit: by the
    whole chip, as under capture, where there is no partition (before, 16 workgroups a worker took 6
    to 60 times as long)."""
    torch, rk = gpu
    g = torch.Generator(device="cuda").manual_seed(log2 + W)
    n = (1 << log2) // 2 // (W if layout == "index" else 1)
    keys = (torch.arange(1, W * n + 1, device="cuda") << 32) | torch.randint(0, 1 << 32, (W * n,), generator=g, device="cuda")
    if layout == "index":                           # more than the 64 that may pass a sub-bin's end
        keys[:200] = (torch.arange(1 << 30, (1 << 30) + 200, device="cuda") << 32) | 8191
    else:                                           # more than the 2^14 of a bin's list
        keys[:17000] = (torch.arange(1 << 30, (1 << 30) + 17000, device="cuda") << 32) | torch.randint(
            0, 1 << 14, (17000,), generator=g, device="cuda")
    off = np.arange(W + 1, dtype=np.int64) * n
    build = rk.index_build if layout == "index" else rk.table_build
    out = torch.empty((2 if layout == "index" else W) << log2, dtype=torch.int64, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        build(keys, off, log2, out)
    whole = _ms(torch, graph.replay)
    ref = torch.sort(out.view(-1, 2)[:, 0] if layout == "index" else out.view(W, -1))[0]
    out.fill_(3)
    split = _ms(torch, lambda: build(keys, off, log2, out))
    say(layout, log2, W, "captured", whole, "ms, partition first", split, "ms")
    assert torch.equal(torch.sort(out.view(-1, 2)[:, 0] if layout == "index" else out.view(W, -1))[0], ref)
    assert rk.device_status(reset=True) == 0
    assert split < 2.5 * whole                      # 1.1 to 1.3 measured


@pytest.mark.parametrize("shared,at", [(2, 8191), (20, 8191), (20, (1 << 24) - 1)])
def test_shared_keys_past_an_end(gpu, shared, at):
    """Blocks that every worker caches pass the end of a sub-bin, and of the index, as one key each:
    the partitioned build holds them (before, two of them sent the whole build back to atomics, six
    times the time)."""
    torch, rk = gpu
    log2, W = 24, 64
    g = torch.Generator(device="cuda").manual_seed(shared)
    n = (1 << log2) // 2 // W
    keys = (torch.arange(1, W * n + 1, device="cuda") << 32) | torch.randint(0, 1 << 32, (W * n,), generator=g, device="cuda")
    off = np.arange(W + 1, dtype=np.int64) * n
    out = torch.empty(2 << log2, dtype=torch.int64, device="cuda")
    plain = _ms(torch, lambda: rk.index_build(keys, off, log2, out))
    keys.view(W, n)[:, :shared] = (torch.arange(1 << 30, (1 << 30) + shared, device="cuda") << 32) | at
    ms = _ms(torch, lambda: rk.index_build(keys, off, log2, out))
    say(shared, "shared keys at", at, ms, "ms, none", plain, "ms")
    slots = out.view(-1, 2)
    slots = slots[slots[:, 0] != 0]
    assert slots.shape[0] == W * n - (W - 1) * shared
    slots = slots[torch.argsort(slots[:, 0])]
    want, worker = torch.sort(keys.view(W, n)[:, shared:].reshape(-1))
    k = torch.searchsorted(slots[:, 0].contiguous(), want)
    assert torch.equal(slots[k, 0], want) and torch.equal(slots[k, 1], 1 << (worker // (n - shared)))
    k = torch.searchsorted(slots[:, 0].contiguous(), torch.sort(keys[:shared])[0])
    assert (slots[k, 1] == -1).all()                # every worker's bit
    assert rk.device_status(reset=True) == 0
    assert ms < 3 * plain                           # 1.0 to 1.6 measured, 6.3 to 7.4 before


def _sleep_cycles(torch, ms):
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    a.record()
    torch.cuda._sleep(10_000_000)
    b.record()
    torch.cuda.synchronize()
    return int(ms / a.elapsed_time(b) * 1e7)


def _build_inputs(torch, rk, layout, sets, seed):
    """Key sets on the device, key offsets, log2 slots and the partitioned build of a layout."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    W, log2 = 4, 20
    n = (1 << log2) // 2 // (W if layout == "index" else 1)
    keys = [((torch.arange(1, W * n + 1, device="cuda") + k * W * n) << 32)
            | torch.randint(0, 1 << 32, (W * n,), generator=g, device="cuda") for k in range(sets)]
    out = [torch.empty((2 if layout == "index" else W) << log2, dtype=torch.int64, device="cuda") for _ in keys]
    return keys, np.arange(W + 1, dtype=np.int64) * n, log2, out, rk.index_build if layout == "index" else rk.table_build


def _assert_built(torch, layout, keys, out):
    """Every key of the set and no other, in its worker's table or with its worker's bit."""
    W = 4
    if layout == "index":
        slots = out.view(-1, 2)
        slots = slots[slots[:, 0] != 0]
        key, k = torch.sort(slots[:, 0])
        want, worker = torch.sort(keys)
        assert torch.equal(key, want) and torch.equal(slots[k, 1], 1 << (worker // (keys.numel() // W)))
    else:
        got = torch.sort(out.view(W, -1), dim=1)[0]
        want = torch.sort(keys.view(W, -1), dim=1)[0]
        assert torch.equal(got[:, -want.shape[1]:], want) and not got[:, : -want.shape[1]].any()


def _stream_beside(torch, busy, cycles):
    """A stream whose work does not share busy's hardware queue."""
    x = torch.zeros(8, device="cuda")
    for _ in range(8):
        s, ended = torch.cuda.Stream(), torch.cuda.Event()
        torch.cuda.synchronize()
        with torch.cuda.stream(busy):
            torch.cuda._sleep(cycles)
            ended.record()
        with torch.cuda.stream(s):
            x.add_(1)
        s.synchronize()
        if not ended.query():
            return s
    pytest.skip("every stream shares the busy one's hardware queue")


@pytest.mark.parametrize("layout", ["index", "tables"])
def test_builds_wait_for_no_other_stream(gpu, layout):
    """A build ends while builds of another stream wait behind 200 ms of other work (before, the fifth
    build waited for the first one's stream)."""
    import time
    torch, rk = gpu
    keys, off, log2, out, build = _build_inputs(torch, rk, layout, 5, 1)
    busy, cycles = torch.cuda.Stream(), _sleep_cycles(torch, 200)
    free = _stream_beside(torch, busy, cycles // 4)
    build(keys[4], off, log2, out[4], stream=free)
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        torch.cuda._sleep(cycles)
        ended = torch.cuda.Event()
        ended.record()
    t = time.perf_counter()
    for k in range(4):
        build(keys[k], off, log2, out[k], stream=busy)
    for _ in range(3):
        build(keys[4], off, log2, out[4], stream=free)
    free.synchronize()
    ms = (time.perf_counter() - t) * 1e3
    early = not ended.query()
    torch.cuda.synchronize()
    say(layout, "ended after", ms, "ms, before the other stream's work:", early)
    for k in range(5):
        _assert_built(torch, layout, keys[k], out[k])
    assert rk.device_status(reset=True) == 0
    assert early


@pytest.mark.parametrize("layout", ["index", "tables"])
def test_builds_on_many_streams_and_captured(gpu, layout):
    """More streams with builds under way than there are side buffers, builds on one stream while
    another is captured, and a captured build."""
    torch, rk = gpu
    keys, off, log2, out, build = _build_inputs(torch, rk, layout, 7, 2)
    cycles = _sleep_cycles(torch, 20)
    streams = [torch.cuda.Stream() for _ in keys]
    for _ in range(3):
        for s, k, o in zip(streams, keys, out):
            with torch.cuda.stream(s):
                torch.cuda._sleep(cycles // 10)
            build(k, off, log2, o, stream=s)
            build(k, off, log2, o, stream=s)
    torch.cuda.synchronize()
    for k, o in zip(keys, out):
        _assert_built(torch, layout, k, o)
        o.fill_(5)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        build(keys[0], off, log2, out[0])
        for i in (1, 2, 1, 2, 3, 4, 5, 6):
            build(keys[i], off, log2, out[i], stream=streams[i])
    for _ in range(3):
        torch.cuda.synchronize()
        for k, o in zip(keys[1:], out[1:]):
            _assert_built(torch, layout, k, o)
        out[0].fill_(3)
        graph.replay()
        torch.cuda.synchronize()
        _assert_built(torch, layout, keys[0], out[0])
        for i in range(1, 7):
            out[i].fill_(3)
            build(keys[i], off, log2, out[i])
    assert rk.device_status(reset=True) == 0


def test_scoring_right_after_a_large_build(gpu):
    """The first scoring of hashed requests after an index larger than the caches is built still finds
    the requests there (before, it took 1.3 times a repeated one's time)."""
    torch, rk = gpu
    g = torch.Generator(device="cuda").manual_seed(3)
    log2, W, B, L = 27, 64, 65536, 256
    n = (1 << log2) // 4 // W
    rand = lambda k: (torch.arange(1, k + 1, device="cuda") << 32) | torch.randint(  # noqa: E731
        0, 1 << 32, (k,), generator=g, device="cuda")
    shared = rand(256 * L).view(256, L)
    chains = (rand(B * L) + (1 << 60)).view(B, L)
    chains[:, : L // 2] = shared[torch.randint(0, 256, (B,), generator=g, device="cuda"), : L // 2]
    keys = (rand(W * n) + (1 << 61)).view(W, n)
    keys[:, : shared.numel()] = shared.view(-1)
    off, chains = torch.arange(B + 1, device="cuda") * L, chains.reshape(-1)
    active = torch.zeros(W, dtype=torch.int32, device="cuda")
    keys, key_off = keys.reshape(-1), np.arange(W + 1, dtype=np.int64) * n
    index = rk.index_build(keys, key_off, log2)
    ov, cost, am = rk.route_score_index(chains, off, index, log2, active)
    assert (ov == L // 2).all()
    first, again = [], []
    for _ in range(9):
        rk.index_build(keys, key_off, log2, index)
        for t in (first, again):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            rk.route_score_index(chains, off, index, log2, active, overlap=ov, cost=cost, argmin=am)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b) * 1e3)
    first, again = sorted(first)[4], sorted(again)[4]
    say("first", first, "us, again", again, "us")
    assert rk.device_status(reset=True) == 0
    assert first < 1.25 * again
