"""Nelder-Mead with three tasks per wave (the automatic choice for large batches): values, iterations,
decisions and status are those of one task per wave, bit for bit, with tasks that stop at different
iterations, shrink, hold a NaN trace, and a last wave that is not full."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def batch(S):
    rng = np.random.default_rng(S)
    T = rng.integers(1, 64, S)
    T[:4] = (1, 2, 3, 4)
    amp = rng.uniform(2.0, 20.0, S).astype(np.float32)
    dur = np.maximum(T, 12).astype(np.float32)
    phi = rng.uniform(0.0, 360.0, S).astype(np.float32)
    base = oracle.simulate(oracle.nominal(40.0), 10.0, 64)
    pos = [np.outer(base[:t] * a / 10.0, [np.cos(np.radians(p)), np.sin(np.radians(p))])
           + rng.uniform(0.0, 0.6) * rng.standard_normal((t, 2)) for t, a, p in zip(T, amp, phi)]
    pos[7][0, 0] = np.nan
    return T, amp, phi, dur, np.concatenate([q.reshape(-1) for q in pos]).astype(np.float32)


@pytest.mark.parametrize("S", [1027, 1096])
@pytest.mark.parametrize("max_iter,tol_x,tol_f", [(0, 1e-4, 1e-6), (60, 2e-2, 1e-2), (150, 1e-4, 1e-6)])
def test_three_tasks_per_wave(S, max_iter, tol_x, tol_f):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_09884_amd import opmm
    ctx = opmm.Context(0)
    assert S > 4 * torch.cuda.get_device_properties(0).multi_processor_count  # the automatic choice is three
    T, amp, phi, dur, pos = batch(S)
    recs = opmm.saccade_records(T, 2, amp, phi, dur, np.arange(S, dtype=np.uint64))
    d = torch.from_numpy(pos).cuda()
    got = {}
    for tpw in (0, 1, 2):
        o = dict(opc=torch.zeros(S, 18, device="cuda"), rmse=torch.zeros(S, device="cuda"),
                 it=torch.zeros(S, dtype=torch.int32, device="cuda"),
                 dec=torch.full((S, max(max_iter, 1)), -1, dtype=torch.int8, device="cuda"),
                 st=torch.zeros(S, dtype=torch.int32, device="cuda"))
        prm = opmm.nm_params(max_iter=max_iter, tol_x=tol_x, tol_f=tol_f, tasks_per_wave=tpw)
        ctx.fit_nm(d, recs, prm, o["opc"], o["rmse"], o["it"], o["dec"], o["st"])
        torch.cuda.synchronize()
        got[tpw] = {k: v.cpu().numpy() for k, v in o.items()}
    for tpw in (1, 2):
        for k in got[0]:
            a, b = got[0][k], got[tpw][k]
            assert np.array_equal(a.view(np.uint32) if a.dtype == np.float32 else a,
                                  b.view(np.uint32) if b.dtype == np.float32 else b), (tpw, k)
    assert np.isnan(got[0]["rmse"][7]) and got[0]["it"][7] == 0
    if max_iter == 60:
        assert len(np.unique(got[0]["it"])) > 1        # tasks end at different iterations
    if max_iter:
        assert np.count_nonzero(got[0]["dec"] == 4) > 0  # some shrinks
    ctx.close()


def test_long_traces_keep_one_task_per_wave():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2007_09884_amd import opmm
    ctx = opmm.Context(0)
    S = 1100
    T, amp, phi, dur, pos = batch(S)
    T = np.append(T, opmm.MAX_T)
    amp, phi, dur = np.append(amp, np.float32(10.0)), np.append(phi, np.float32(0.0)), np.append(dur, np.float32(40.0))
    long = np.stack([oracle.simulate(oracle.nominal(40.0), 10.0, opmm.MAX_T), np.zeros(opmm.MAX_T)], 1)
    d = torch.from_numpy(np.concatenate([pos, long.reshape(-1).astype(np.float32)])).cuda()
    recs = opmm.saccade_records(T, 2, amp, phi, dur, np.arange(S + 1, dtype=np.uint64))
    got = []
    for tpw in (0, 1, 2):
        opc, rmse = torch.zeros(S + 1, 18, device="cuda"), torch.zeros(S + 1, device="cuda")
        ctx.fit_nm(d, recs, opmm.nm_params(max_iter=3, tasks_per_wave=tpw), opc, rmse)
        torch.cuda.synchronize()
        got.append((opc.cpu().numpy().tobytes(), rmse.cpu().numpy().tobytes()))
    assert got[0] == got[1] == got[2]
    ctx.close()


@pytest.mark.parametrize("max_iter", [0, 60])
def test_three_tasks_per_wave_past_two_waves_per_simd(max_iter):
    """Beyond two waves per SIMD the automatic choice is three tasks per wave whatever the traces' lengths."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    test_three_tasks_per_wave(8 * torch.cuda.get_device_properties(0).multi_processor_count + 3, max_iter, 2e-2, 1e-2)
