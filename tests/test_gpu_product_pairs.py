"""The paired product kernel (large trees) at the edges of its ranges: one, two
and five hands per thread, hand counts around whole threads and rows, odd
numbers of sequences of a kind, trees just below and above the switch, open
folds (sequences with other terminals than one fold and one showdown), one-card
hands, and the form that also yields max |g| (CFR on a large tree).

Tolerance: 1e-12 of the sum of the absolute terms an entry adds, as for the
products elsewhere; CFR iterates 1e-10 of the largest entry."""
import numpy as np
import pytest

from instances.endgames import BetAbstraction, Instance, river
from oracle import Cfr as OracleCfr
from oracle import Problem
from tests.layout import Layout
from tests.test_gpu_ops import grad_bound

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES = (0.25, 0.5, 0.75, 1.0, 2.0)
OPEN = BetAbstraction(fracs=((SIZES, SIZES, SIZES, SIZES), (SIZES, SIZES, SIZES, (0.5, 1.0))),
                      allin=((True,) * 4, (True,) * 4), open_fold=(True, True))


def one_card(n):
    rng = np.random.default_rng(n)
    return Instance(name="one_card", n_cards=n, cards_per_hand=1, board=np.zeros(0, np.int32),
                    hand_cards=np.arange(n, dtype=np.int32).reshape(n, 1), strength=rng.integers(0, n // 2, n).astype(np.int32),
                    belief=np.stack([rng.dirichlet(np.ones(n)) for _ in range(2)]), pot=100.0, stack=5000.0,
                    bet_fracs=SIZES, allin=True, max_raises=3)


CASES = {
    "105h": lambda: river("x", 1, 5, "int30", 1.0, 100.0, 5000.0, SIZES, 3),
    "276h": lambda: river("x", 2, 7, "ranking_ties10", 0.5, 100.0, 5000.0, SIZES, 3, n_board=4),
    "528h": lambda: river("x", 3, 9, "ranking_ties10", 0.5, 100.0, 5000.0, SIZES, 3, n_board=3),
    "1081h_808": lambda: river("x", 4, 13, "ranking_ties10", 0.5, 1000.0, 20000.0, (0.25, 0.5, 1.0, 2.0), 3),
    "1081h_520": lambda: river("x", 4, 13, "ranking_ties10", 0.5, 1000.0, 20000.0, SIZES, 2),
    "1176h": lambda: river("x", 5, 13, "ranking_ties10", 0.5, 1000.0, 20000.0, (0.25, 0.5, 1.0, 2.0), 3, n_board=3),
    "open_fold": lambda: river("x", 6, 8, "ranking_ties10", 0.5, 100.0, 5000.0, (), 3, abstraction=OPEN),
    "one_card": lambda: one_card(60),
}


@pytest.fixture(scope="module")
def egt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_03063_amd import egt as mod

    return mod


@pytest.mark.parametrize("name", list(CASES))
def test_products(egt, name):
    inst = CASES[name]()
    P, G = Problem(inst), egt.Game(inst)
    L = Layout(G, P)
    print(f"[case] {name}: {inst.n_hands} hands, {G.n_seq} sequences", flush=True)
    rng = np.random.default_rng(21)
    v = [rng.standard_normal((P.n_seq[p], P.n)) for p in (0, 1)]
    for p in (0, 1):
        lib = L.to_lib(1 - p, v[1 - p])
        lib[:, P.n:] = np.nan  # the padding of an input is not read
        got = egt.gradient(G, p, torch.from_numpy(lib).cuda(), torch.full((G.n_seq[p], G.ld), np.nan, dtype=torch.float64, device="cuda"))
        got = got.cpu().numpy()
        want = P.grad_x(v[1]) if p == 0 else P.grad_y(v[0])
        assert np.all(got[:, P.n:] == 0)
        assert np.all(np.abs(L.from_lib(p, got) - want) <= 1e-12 * grad_bound(P, p, v[1 - p]) + 1e-300)
    G.close()


@pytest.mark.parametrize("name", ["105h", "1081h_808"])
def test_cfr_on_paired_products(egt, name):
    inst = CASES[name]()
    P, G = Problem(inst), egt.Game(inst)
    L, C, D = Layout(G, P), OracleCfr(P, "CFR_PLUS"), egt.Cfr(G, "CFR_PLUS")
    print(f"[case] CFR+ {name}", flush=True)
    for _ in range(3):
        C.step()
        D.step(1)
        got = D.get()
        for p, key in ((0, "x"), (1, "y")):
            for mine, want in ((got[key], C.cur[p]), (got[key + "_avg"], C.avg[p])):
                assert np.abs(L.from_lib(p, mine.cpu().numpy()) - want).max() <= 1e-10 * np.abs(want).max()
    D.close()
    G.close()
