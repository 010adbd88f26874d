"""Polish at the edges of the block recurrence and of the polish's staging of Jacobian rows:
traces shorter than a block, around every remainder, around the staged 25-32 samples and several
fillings; alone and three to a wave."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENGTHS = [1, 2, 3, 4, 5, 6, 7, 8, 9, 23, 24, 25, 26, 27, 28, 29, 30, 31, 32, 33, 49, 56, 57, 64, 65, 97, 130]


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


def problem(opmm, pw=None):
    rng = np.random.default_rng(5)
    S = len(LENGTHS)
    T = np.array(LENGTHS)
    dur = np.maximum(T, 20).astype(np.float32)
    recs = opmm.saccade_records(T, 2, np.full(S, 11.0, np.float32), np.full(S, 25.0, np.float32), dur,
                                np.arange(S, dtype=np.uint64))
    nom = np.stack([oracle.nominal(float(d)) for d in dur])
    true = (nom * rng.uniform(0.85, 1.15, nom.shape)).astype(np.float32)
    start = np.clip(true * (1 + 0.02 * rng.standard_normal(nom.shape)), 0.76 * nom, 1.24 * nom).astype(np.float32)
    u = np.array([np.cos(np.radians(25.0)), np.sin(np.radians(25.0))])
    traces = [(oracle.simulate(true[s].astype(np.float64), 11.0, int(T[s]))[:, None] * u
               + 0.05 * rng.standard_normal((T[s], 2))).astype(np.float32) for s in range(S)]
    return recs, start, traces


@pytest.mark.parametrize("objective", [0, 1])
def test_polish_alone_and_three_to_a_wave(ctx, opmm, objective):
    """A batch of one (a wave of its own) gives the bits of the same saccade among thousands (three to a
    wave), and the result is no worse than the start and its costs are those of opmm_score."""
    recs, start, traces = problem(opmm)
    S = len(LENGTHS)
    copies = 3000 // S + 1
    pos = np.concatenate([t.reshape(-1) for t in traces])
    d = torch.from_numpy(np.tile(pos, copies)).cuda()
    many = np.concatenate([recs] * copies)
    for c in range(copies):
        many["pos_offset"][c * S:(c + 1) * S] += c * pos.size
    prm = opmm.polish_params(max_iter=3, objective=objective)
    opc = torch.from_numpy(np.tile(start, (copies, 1))).cuda()
    rm, ma = torch.zeros(S * copies, device="cuda"), torch.zeros(S * copies, device="cuda")
    ctx.polish(d, many, prm, opc, rm, ma)
    torch.cuda.synchronize()
    opc, rm, ma = opc.cpu().numpy(), rm.cpu().numpy(), ma.cpu().numpy()
    for s in range(S):
        o1, r1, m1 = torch.from_numpy(start[s:s + 1].copy()).cuda(), torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
        ctx.polish(d, recs[s:s + 1], prm, o1, r1, m1)
        torch.cuda.synchronize()
        for c in (0, copies // 2, copies - 1):
            k = c * S + s
            assert opc[k].tobytes() == o1.cpu().numpy()[0].tobytes() and rm[k] == r1.item() and ma[k] == m1.item(), LENGTHS[s]
        both = np.stack([start[s], opc[s]])
        want, _ = oracle.score(both, traces[s], 11.0, 25.0)
        assert abs(rm[s] - want[1]) <= 1e-6 * want[1] + 1e-6
        if objective == 0:
            assert rm[s] <= want[0] + 1e-6


@pytest.mark.parametrize("copies", [1, 112])
def test_polish_lowers_the_mean_absolute_difference(ctx, opmm, copies):
    """Objective MAE: mae_out is the oracle's mean absolute difference of the result, and no larger than the
    start's; one saccade per wave, and three."""
    recs, start, traces = problem(opmm)
    S = len(LENGTHS)
    pos = np.concatenate([t.reshape(-1) for t in traces])
    d = torch.from_numpy(np.tile(pos, copies)).cuda()
    many = np.concatenate([recs] * copies)
    for c in range(copies):
        many["pos_offset"][c * S:(c + 1) * S] += c * pos.size
    opc = torch.from_numpy(np.tile(start, (copies, 1))).cuda()
    rm, ma = torch.zeros(S * copies, device="cuda"), torch.zeros(S * copies, device="cuda")
    ctx.polish(d, many, opmm.polish_params(max_iter=3, objective=opmm.OBJ_MAE), opc, rm, ma)
    torch.cuda.synchronize()
    opc, rm, ma = opc.cpu().numpy()[-S:], rm.cpu().numpy()[-S:], ma.cpu().numpy()[-S:]
    for s in range(S):
        rmse, mae = oracle.score(np.stack([start[s], opc[s]]), traces[s], 11.0, 25.0)
        # FP32 outputs of costs of a few hundredths of a degree; the plant's truncation is far below
        assert abs(rm[s] - rmse[1]) <= 1e-6 * rmse[1] + 1e-6, LENGTHS[s]
        assert abs(ma[s] - mae[1]) <= 1e-6 * mae[1] + 1e-6, LENGTHS[s]
        assert mae[1] <= mae[0] + 1e-6, LENGTHS[s]
    assert np.mean([oracle.score(opc[s:s + 1], traces[s], 11.0, 25.0)[1][0] for s in range(S)]) < \
        np.mean([oracle.score(start[s:s + 1], traces[s], 11.0, 25.0)[1][0] for s in range(S)])
