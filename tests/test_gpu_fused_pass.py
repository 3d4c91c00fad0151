"""The single-launch smoothed best response and regret update at the sizes where its layout
changes: 1, 2, 3 and 5 (sequence, hand) pairs per thread with 16 and 4 hands
per block and with one live slot, trees just below and above the switch to a
launch per level, nodes of one to ten actions (lane pairs and quads past their
first round), and temperatures and gradients at the ends of the range, where
the shift's quotient cannot be formed from a reciprocal.

Tolerances are those of the operations elsewhere: strategies 1e-12 absolute,
values 1e-13 of the size of the terms they add, CFR iterates 1e-10 of the
largest entry."""
import numpy as np
import pytest

from instances import make_instance
from instances.efg import random_efg
from instances.endgames import river
from oracle import Cfr as OracleCfr
from oracle import Problem
from oracle.general import GeneralProblem
from tests.layout import Layout

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

HALVES, QUARTERS, SEVEN = (0.5, 1.0, 2.0), (0.25, 0.5, 1.0, 2.0), (0.25, 0.5, 0.75, 1.0, 1.5, 2.0, 3.0)
# ranks, bet fractions, raises: sequences per player in the comment
RIVER = [
    (5, (0.5, 1.0), 0),  # 10, 16 hands per block
    (5, HALVES, 1),      # 49
    (5, (0.5, 1.0), 2),  # 64, two pairs per thread
    (5, HALVES, 2),      # 127, over three: 4 hands per block
    (5, QUARTERS, 2),    # 286
    (8, (0.25, 0.5, 0.75, 1.0, 2.0), 2),  # 520, 5 pairs per thread
    (8, QUARTERS, 3),    # 808, a launch per level
    (10, SEVEN, 1),      # 190, 595 hands, ten actions
    (13, QUARTERS, 2),   # 286, 1081 hands
    (13, (0.25, 0.5, 0.75, 1.0, 2.0), 2),  # 520, a launch per level
]


@pytest.fixture(scope="module")
def egt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_03063_amd import egt as mod

    return mod


def check(egt, G, P, L, g, p, mu):
    q, val = egt.smoothed_br(G, p, torch.from_numpy(np.ascontiguousarray(L.to_lib(p, g))).cuda(), mu)
    br = egt.best_response(G, p, torch.from_numpy(np.ascontiguousarray(L.to_lib(p, g))).cuda())
    q, val, br = q.cpu().numpy(), float(val.cpu()[0]), float(br.cpu()[0])
    q_o, val_o, _, V = P.sbr(p, g, mu)
    assert np.all(q[:, P.n:] == 0)
    assert np.abs(L.from_lib(p, q) - q_o).max() <= 1e-12
    assert abs(val - val_o) <= 1e-13 * (np.abs(V).sum() + 1.0)
    assert abs(br - P.br(p, g)) <= 1e-13 * (np.abs(g).sum() + 1.0)


@pytest.mark.parametrize("ranks,fracs,raises", RIVER)
def test_river_sizes(egt, ranks, fracs, raises):
    inst = river("x", 3, ranks, "ranking_ties10", 0.5, 1000.0, 20000.0, fracs, raises)
    P, G = Problem(inst), egt.Game(inst)
    L = Layout(G, P)
    rng = np.random.default_rng(11)
    for p in (0, 1):
        print(f"[case] {inst.n_hands} hands, {G.n_seq[p]} sequences, player {p}", flush=True)
        check(egt, G, P, L, 10.0 * rng.standard_normal((P.n_seq[p], P.n)), p, 0.5)
    G.close()


@pytest.mark.parametrize("variant", ["CFR", "CFR_PLUS"])
@pytest.mark.parametrize("ranks,fracs,raises", RIVER[:3] + RIVER[4:7] + RIVER[8:9])
def test_regret_update_sizes(egt, ranks, fracs, raises, variant):
    inst = river("x", 4, ranks, "ranking_ties10", 0.5, 1000.0, 20000.0, fracs, raises)
    P, G = Problem(inst), egt.Game(inst)
    L, C, D = Layout(G, P), OracleCfr(P, variant), egt.Cfr(G, variant)
    print(f"[case] {variant} {inst.n_hands} hands, {G.n_seq} sequences", flush=True)
    for _ in range(4):
        C.step()
        D.step(1)
        got = D.get()
        for p, key in ((0, "x"), (1, "y")):
            for mine, want in ((got[key], C.cur[p]), (got[key + "_avg"], C.avg[p])):
                assert torch.all(mine[:, P.n:] == 0)
                assert np.abs(L.from_lib(p, mine.cpu().numpy()) - want).max() <= 1e-10 * np.abs(want).max()
    D.close()
    G.close()


@pytest.mark.parametrize("args", [(1, 6, 4, 4), (0, 8, 3, 6), (0, 7, 4, 4), (3, 8, 4, 6)])
def test_general_sizes(egt, args):
    inst = random_efg(*args)
    P, G = GeneralProblem(inst), egt.GeneralGame(inst)
    L = Layout(G, P)
    rng = np.random.default_rng(12)
    for p in (0, 1):
        print(f"[case] general {args}, {G.n_seq[p]} sequences, player {p}", flush=True)
        g = rng.standard_normal((P.n_seq[p], 1))
        q, val = egt.smoothed_br(G, p, torch.from_numpy(np.ascontiguousarray(L.to_lib(p, g))).cuda(), 0.3)
        q = q.cpu().numpy()
        q_o, val_o, _, _ = P.sbr(p, g, 0.3)
        assert np.all(q[:, 1:] == 0)
        assert np.abs(L.from_lib(p, q) - q_o).max() <= 1e-12
        # the value adds terms of size mu beta log n that cancel: bound relative to them
        scale = abs(val_o) + 0.3 * max(n.beta for n in P.tp[p].nodes) * np.log(16.0) + np.abs(g).sum()
        assert abs(float(val.item()) - val_o) <= 1e-13 * scale
    G.close()


@pytest.mark.parametrize("mu,scale", [(1e-290, 1.0), (1e290, 1.0), (1e-3, 1e304), (0.5, 1e-300), (3.0, 1.0)])
def test_ends_of_the_range(egt, mu, scale):
    inst = make_instance("c0", 2)
    P, G = Problem(inst), egt.Game(inst)
    L = Layout(G, P)
    rng = np.random.default_rng(13)
    for p in (0, 1):
        g = scale * rng.standard_normal((P.n_seq[p], P.n))
        leaf = max(range(len(P.tp[p].nodes)), key=lambda v: P.tp[p].nodes[v].first_seq)
        if scale == 1.0:  # an action that is never taken
            g[P.tp[p].nodes[leaf].first_seq] = np.inf
        q, _ = egt.smoothed_br(G, p, torch.from_numpy(np.ascontiguousarray(L.to_lib(p, g))).cuda(), mu)
        with np.errstate(all="ignore"):
            q_o = P.sbr(p, g, mu)[0]
        print(f"[case] mu {mu:g} scale {scale:g} player {p}", flush=True)
        got = L.from_lib(p, q.cpu().numpy())
        assert np.array_equal(np.isnan(got), np.isnan(q_o))
        assert np.nanmax(np.abs(got - q_o)) <= 1e-12
    G.close()
