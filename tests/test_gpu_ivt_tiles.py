"""Saccade extraction at the edges of its tiles: streams that end around a chunk of 2048 samples, runs
across chunks, longer than a bit word, a chunk and the longest trace, one-sample runs in every
position, outputs past the records written to host memory, and streams of several chunks per tile;
exactly against a vectorised reference that is itself checked against the oracle's loop."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")


def reference(g, min_dur=6.0, min_amp=0.0, max_T=2048):
    """(first sample, T) of the kept runs, 30 deg/s at 1 kHz, in the stream's own FP32."""
    thr = np.float32(30.0) * np.float32(1.0) * np.float32(1e-3)
    d = np.diff(g, axis=0)
    fast = np.concatenate([[False], d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1] > thr * thr])
    edge = np.flatnonzero(np.diff(np.concatenate([[False], fast, [False]]).astype(np.int8)))
    first, last = edge[0::2] - 1, edge[1::2] - 1
    T = last - first + 1
    v = g[last] - g[first]
    amp = np.sqrt(v[:, 0] * v[:, 0] + v[:, 1] * v[:, 1])
    keep = (T - 1 >= min_dur) & (amp >= np.float32(min_amp)) & (T <= max_T)
    return first[keep], T[keep]


def stream(moving):
    """Gaze that moves 0.05 deg in every sample of `moving` (a flag per sample)."""
    step = np.where(moving, np.float32(0.05), np.float32(0.0)).astype(np.float64)
    sign = np.where((np.arange(len(moving)) // 3000) % 2 == 0, 1.0, -1.0)
    x = np.cumsum(step * sign)
    return np.stack([x, 0.5 * x], 1).astype(np.float32)


def random_flags(N, seed, p_on, p_off):
    rng = np.random.default_rng(seed)
    lengths_on = rng.geometric(p_off, N // 2 + 2)
    lengths_off = rng.geometric(p_on, N // 2 + 2)
    ends = np.cumsum(np.stack([lengths_off, lengths_on], 1).reshape(-1))
    k = np.searchsorted(ends, np.arange(N), side="right")
    f = (k % 2) == 1
    f[0] = False
    return f


def test_reference_matches_the_oracle():
    for seed, p_on, p_off in ((1, 0.05, 0.05), (2, 0.5, 0.5), (3, 0.02, 0.01)):
        g = stream(random_flags(1500, seed, p_on, p_off))
        for md, mt in ((0.0, 2048), (6.0, 2048), (6.0, 40)):
            want = oracle.ivt(g, min_dur=md, max_T=mt)
            f, T = reference(g, md, 0.0, mt)
            assert [(w["start"], w["T"]) for w in want] == list(zip(f, T))


def flags_for(case):
    if case.startswith("n"):                       # stream ends around a chunk, moving up to its last sample
        N = int(case[1:])
        f = random_flags(N, N, 0.02, 0.05)
        f[max(1, N - 9):] = True
        return f
    if case == "alternate":                        # one-sample runs in every other position
        f = np.zeros(5000, bool)
        f[1::2] = True
        return f
    if case == "long":                             # runs of 64, 65, 2047, 2048, 2049 and 5000 samples
        f = np.zeros(30000, bool)
        k = 1
        for n in (64, 65, 127, 2046, 2047, 2048, 2049, 5000, 7):
            f[k:k + n] = True
            k += n + 13
        return f
    if case == "from_start":
        f = np.zeros(4096, bool)
        f[1:1900] = True
        f[2047:2050] = True
        f[2060:2070] = True
        return f
    return random_flags(300000, 11, 0.5, 0.3)      # "dense": tens of thousands of short runs


@pytest.mark.gpu
@pytest.mark.parametrize("min_dur,max_T,min_amp", [(6.0, 2048, 0.0), (0.0, 2048, 0.0), (3.0, 65, 0.3)])
@pytest.mark.parametrize("case", ["n2", "n63", "n64", "n65", "n2047", "n2048", "n2049", "n4097", "alternate", "long",
                                  "from_start", "dense"])
def test_tiles(case, min_dur, max_T, min_amp):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_09884_amd import opmm
    ctx = opmm.Context(0)
    g = stream(flags_for(case))
    first, T = reference(g, min_dur, min_amp, max_T)
    d = torch.from_numpy(g).cuda()
    pos = torch.zeros(3 * g.shape[0] + 16, device="cuda")
    kw = dict(min_dur=min_dur, max_T=max_T, min_amp=min_amp)
    recs, src = ctx.ivt_extract(d, pos, max_out=len(T) + 5, **kw)
    assert np.array_equal(src, first) and np.array_equal(recs["T"], T)
    off = np.cumsum(2 * T) - 2 * T
    assert np.array_equal(recs["pos_offset"], off)
    P = pos.cpu().numpy()
    for i in range(0, len(T), max(1, len(T) // 200)):
        a = int(first[i])
        assert np.array_equal(P[off[i]:off[i] + 2 * T[i]].reshape(-1, 2), g[a:a + T[i]] - g[a])
    # both bounds cut a prefix: the record count, and the room for traces
    if len(T) > 2:
        n = len(T) // 2
        recs, src = ctx.ivt_extract(d, pos, max_out=n, **kw)
        assert np.array_equal(src, first[:n])
        recs, src = ctx.ivt_extract(d, pos[:int(off[n]) + 2 * int(T[n]) - 1], max_out=len(T), **kw)
        assert np.array_equal(src, first[:n])
    ctx.close()


@pytest.mark.gpu
def test_several_chunks_per_tile_and_odd_alignment():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_09884_amd import opmm
    ctx = opmm.Context(0)
    N = 2048 * 4096 + 5000                         # two chunks per tile
    g = stream(random_flags(N, 5, 0.004, 0.02))
    first, T = reference(g)
    buf = torch.zeros(2 * N + 1, device="cuda")    # samples at an odd float: 4-byte alignment
    buf[1:].copy_(torch.from_numpy(g.reshape(-1)))
    pos = torch.zeros(2 * int(T.sum()) + 1, device="cuda")[1:]
    recs, src = ctx.ivt_extract(buf[1:].view(N, 2), pos, max_out=len(T) + 1)
    assert len(T) > 20000 and np.array_equal(src, first) and np.array_equal(recs["T"], T)
    P = pos.cpu().numpy()
    want = np.concatenate([g[a:a + t] - g[a] for a, t in zip(first, T)]).reshape(-1)
    assert np.array_equal(P, want)
    ctx.close()


@pytest.mark.gpu
def test_many_short_runs_take_no_turns():
    """A stream that moves in every other sample takes a few times as long as a still one, not ten times (a chunk's
    thousand runs are emitted side by side)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import time
    from paper_2007_09884_amd import opmm
    ctx = opmm.Context(0)
    N = 100000
    flags = np.zeros(N, bool)
    pos = torch.zeros(2 * N, device="cuda")
    best = {}
    for name in ("still", "alternate"):
        flags[1::2] = name == "alternate"
        d = torch.from_numpy(stream(flags)).cuda()
        times = []
        for _ in range(30):
            t = time.perf_counter()
            recs, _src = ctx.ivt_extract(d, pos, min_dur=0.0, max_out=4096)
            times.append(time.perf_counter() - t)
        assert len(recs) == (4096 if name == "alternate" else 0)
        best[name] = min(times)
    assert best["alternate"] < 6 * best["still"], best
    ctx.close()
