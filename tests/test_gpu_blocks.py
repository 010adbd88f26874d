"""The recurrence advances four samples per step, aligned to each candidate's own pulse end.  Its edges:
traces shorter than a block and with every remainder, pulses that end before the trace, on a sample, in
every position of a block and past the trace, side by side in one wave; against the FP64 oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def opmm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_09884_amd import opmm as m
    return m


@pytest.fixture(scope="module")
def ctx(opmm):
    c = opmm.Context(0)
    yield c
    c.close()


def candidates(T):
    """OPCs whose pulses end all over a trace of T samples (and before and after it)."""
    rng = np.random.default_rng(T)
    pw = [-1.0, 0.0, 0.25, 0.999]
    for k in range(min(T, 9)):
        pw += [k + 0.0, k + 0.5]
    pw += [T - 1.5, T - 1.0, T - 0.5, float(T), T + 0.5, T + 7.0]
    p = np.stack([oracle.nominal(2.2 * 12.0 + 21.0) * rng.uniform(0.75, 1.25, 18) for _ in pw]).astype(np.float32)
    p[:, 17] = pw
    return p


@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 14, 17, 60, 131])
def test_trajectories_and_costs_at_block_edges(ctx, opmm, T):
    p = candidates(T)
    n = len(p)
    ref = np.stack([oracle.simulate(p[i].astype(np.float64), 12.0, T) for i in range(n)])
    out = torch.full((n, T), float("nan"), device="cuda")
    d = torch.from_numpy(p).cuda()
    ctx.simulate(d, torch.full((n,), 12.0, device="cuda"), T, out)
    torch.cuda.synchronize()
    # half an FP32 ulp of the largest angle, and the transition's truncation (~5e-9 deg, 1e-7 at most)
    tol = 0.5 * np.spacing(np.float32(np.abs(ref).max())) + 1e-7
    assert np.abs(out.cpu().numpy() - ref).max() <= tol
    # costs against a noisy trace of the first candidates' family, 2-D
    rng = np.random.default_rng(100 + T)
    pos = oracle.make_target(oracle.nominal(47.4), 12.0, 30.0, T, 2, rng.standard_normal((T, 2)), 0.05)
    rec = opmm.saccade_records([T], 2, [12.0], [30.0], [47.4], [1])
    want, _ = oracle.score(p, pos, 12.0, 30.0)
    dpos = torch.from_numpy(np.ascontiguousarray(pos, np.float32).reshape(-1)).cuda()
    got = torch.zeros(n, device="cuda")
    ctx.score(d, dpos, rec, got)
    assert np.allclose(got.cpu().numpy(), want, rtol=1e-6, atol=1e-6)
    scr = torch.zeros(n, device="cuda")
    ctx.score(d, dpos, rec, scr, screen=True)
    # the screening pass: within half the default tolerance of the FP64 cost
    assert np.abs(scr.cpu().numpy().astype(np.float64) - want).max() <= 2.5e-5
