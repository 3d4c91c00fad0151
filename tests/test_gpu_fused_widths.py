"""The single-launch passes at every number of (sequence, hand) pairs per thread and
hands per block that a game can have: the smoothed best response in FP64 and FP32
and the regret update, each on the layout it is meant for.

Tolerances are those of the operations elsewhere: strategies 1e-12 absolute and
values 1e-13 of the size of the terms they add, in FP32 1e-5 and 1e-6; CFR
iterates 1e-10 of the largest entry."""
import numpy as np
import pytest

from instances.efg import random_efg
from instances.endgames import river
from oracle import Cfr as OracleCfr
from oracle import Problem
from oracle.general import GeneralProblem
from tests.layout import Layout
from tests.test_gpu_fused_pass import HALVES, QUARTERS, check

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIX = (0.25, 0.5, 0.75, 1.0, 2.0)


def tree(ranks, fracs, raises):
    return lambda: river("x", 7, ranks, "ranking_ties10", 0.5, 1000.0, 20000.0, fracs, raises)


# hands per block, pairs per thread (of 512 threads): game
GAMES = {
    (16, 1): tree(5, (0.5, 1.0), 0),
    (16, 2): tree(5, HALVES, 1),
    (16, 3): tree(5, QUARTERS, 1),
    (4, 1): tree(5, SIX, 1),
    (4, 2): tree(13, HALVES, 3),
    (4, 3): tree(13, QUARTERS, 2),
    (4, 5): tree(8, SIX, 2),
    (1, 1): lambda: random_efg(1, 6, 4, 4),
    (1, 2): lambda: random_efg(0, 8, 3, 6),
    (1, 3): lambda: random_efg(0, 7, 4, 4),
}


@pytest.fixture(scope="module")
def egt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_03063_amd import egt as mod

    return mod


def setup(egt, hands, pairs):
    inst = GAMES[hands, pairs]()
    P, G = (GeneralProblem(inst), egt.GeneralGame(inst)) if hands == 1 else (Problem(inst), egt.Game(inst))
    assert G.routes()["pass_hands"] == hands
    per_thread = -(-max(G.n_seq) * hands // 512)
    assert (5 if per_thread == 4 else per_thread) == pairs
    print(f"[case] {hands} hands per block, {pairs} pairs per thread: {P.n} hands, {G.n_seq} sequences", flush=True)
    return P, G, Layout(G, P)


@pytest.mark.parametrize("hands,pairs", list(GAMES))
def test_smoothed_br(egt, hands, pairs):
    P, G, L = setup(egt, hands, pairs)
    rng = np.random.default_rng(16)
    for p in (0, 1):
        g = 10.0 * rng.standard_normal((P.n_seq[p], P.n))
        if hands > 1:
            check(egt, G, P, L, g, p, 0.5)
        g32 = torch.from_numpy(np.ascontiguousarray(L.to_lib(p, g))).float().cuda()
        q, val = egt.smoothed_br_mixed(G, p, g32, 0.5)
        q, val = q.double().cpu().numpy(), float(val.item())
        q_o, val_o, _, V = P.sbr(p, L.from_lib(p, g32.double().cpu().numpy()), 0.5)
        assert np.all(q[:, P.n:] == 0)
        assert np.abs(L.from_lib(p, q) - q_o).max() <= 1e-5
        scale = abs(val_o) + np.abs(V).sum()
        if hands == 1:  # the value adds terms of size mu beta log n that cancel
            scale += 0.5 * max(n.beta for n in P.tp[p].nodes) * np.log(16.0)
        assert abs(val - val_o) <= 1e-6 * scale
    G.close()


@pytest.mark.parametrize("hands,pairs", list(GAMES))
def test_regret_update(egt, hands, pairs):
    P, G, L = setup(egt, hands, pairs)
    C, D = OracleCfr(P, "CFR_PLUS"), egt.Cfr(G, "CFR_PLUS")
    for _ in range(3):
        C.step()
        D.step(1)
        got = D.get()
        for p, key in ((0, "x"), (1, "y")):
            for mine, want in ((got[key], C.cur[p]), (got[key + "_avg"], C.avg[p])):
                assert torch.all(mine[:, P.n:] == 0)
                assert np.abs(L.from_lib(p, mine.cpu().numpy()) - want).max() <= 1e-10 * np.abs(want).max()
    D.close()
    G.close()
