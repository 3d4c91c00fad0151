"""The precision form's products where their layout changes: the column-block
GEMM with one, two and three tiles of hands per wavefront, last column blocks of
any fill, few hands, more hands than a block's LDS holds (the tiled GEMM), and
the fold kernel with two, five and eight hands per thread, groups of fewer than
four sequences, open folds and one-card hands.

Tolerance, per entry, relative to the sum of the absolute terms: the BF16 hi + lo
split of a reach is off by 2^-18 of it, FP32 sums of up to 2048 terms by at most
2048 x 2^-24: together below 1.3e-4."""
import numpy as np
import pytest

from instances.endgames import Instance, river
from oracle import Problem
from tests.layout import Layout
from tests.test_gpu_ops import grad_bound
from tests.test_gpu_product_pairs import OPEN, SIZES, one_card

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SEVEN = (0.25, 0.5, 0.75, 1.0, 1.5, 2.0, 3.0)


def many_hands(n, raises):
    """n two-card hands of a 90-card deck, in random order of strength."""
    rng = np.random.default_rng(n)
    pairs = np.array([(a, b) for a in range(90) for b in range(a + 1, 90)], dtype=np.int32)
    hands = pairs[np.sort(rng.choice(len(pairs), n, replace=False))]
    return Instance(name="many", n_cards=90, cards_per_hand=2, board=np.zeros(0, np.int32), hand_cards=hands,
                    strength=rng.integers(0, n, n).astype(np.int32),
                    belief=np.stack([rng.dirichlet(np.ones(n)) for _ in range(2)]), pot=100.0, stack=5000.0,
                    bet_fracs=SIZES, allin=True, max_raises=raises)


CASES = {
    "1684_sequences": lambda: river("x", 1, 13, "ranking_ties10", 0.5, 1000.0, 20000.0, (0.25, 0.5, 1.0, 2.0), 4),
    "3001_sequences": lambda: river("x", 2, 13, "ranking_ties10", 0.5, 1000.0, 20000.0, SEVEN, 3),
    "520_sequences": lambda: river("x", 7, 13, "ranking_ties10", 0.5, 1000.0, 20000.0, SIZES, 2),
    "105h": lambda: river("x", 3, 5, "int30", 1.0, 100.0, 5000.0, SEVEN, 3),
    "351h": lambda: river("x", 4, 8, "ranking_ties10", 0.5, 1000.0, 20000.0, SEVEN, 4),
    "1300h": lambda: many_hands(1300, 3),
    "2048h": lambda: many_hands(2048, 1),
    "1300h_few": lambda: many_hands(1300, 0),
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
    rng = np.random.default_rng(31)
    for p in (0, 1):
        v = rng.random((P.n_seq[1 - p], P.n)).astype(np.float32)
        lib = torch.from_numpy(L.to_lib(1 - p, v.astype(np.float64))).float().cuda()
        out = torch.full((G.n_seq[p], G.ld), np.nan, dtype=torch.float32, device="cuda")
        got = egt.gradient_mixed(G, p, lib, out).double().cpu().numpy()
        want = P.grad_x(v.astype(np.float64)) if p == 0 else P.grad_y(v.astype(np.float64))
        assert np.all(got[:, P.n:] == 0)
        assert np.all(np.abs(L.from_lib(p, got) - want) <= 1.3e-4 * grad_bound(P, p, v.astype(np.float64)) + 1e-30)
    G.close()
