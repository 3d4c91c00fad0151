"""Which kernels a game's operations run, on both sides of every line between them,
and the benchmark's rooflines naming the kernels that ran."""
import pytest

import bench
from instances.efg import random_efg
from instances.endgames import river
from tests.test_gpu_fused_pass import QUARTERS, SEVEN
from tests.test_gpu_mixed_columns import many_hands
from tests.test_gpu_product_pairs import SIZES, one_card

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def tree(ranks, fracs, raises, **kw):
    return lambda: river("x", 3, ranks, "ranking_ties10", 0.5, 1000.0, 20000.0, fracs, raises, **kw)


# name: game, sequences of the larger tree, product by pairs, hands per block of the single launch, column GEMM
GAMES = {
    "three_pairs_16_hands": (tree(5, QUARTERS, 1), 76, 0, 16, 0),
    "four_hands": (tree(5, SIZES, 1), 109, 0, 4, 0),
    "five_pairs": (tree(8, SIZES, 2), 520, 0, 4, 0),
    "six_pairs": (tree(8, QUARTERS, 3), 808, 1, 0, 1),
    "595h_209_tiles": (tree(10, SIZES, 2), 520, 0, 0, 0),
    "741h_264_tiles": (tree(11, SIZES, 2), 520, 0, 0, 1),
    "1081h_three_pairs": (tree(13, QUARTERS, 2), 286, 0, 4, 0),
    "1081h_five_pairs": (tree(13, SIZES, 2), 520, 0, 0, 1),
    "1081h_columns": (tree(13, SEVEN, 3), 3001, 1, 0, 1),
    "1176h": (tree(13, QUARTERS, 3, n_board=3), 808, 1, 0, 1),
    "1300h": (lambda: many_hands(1300, 3), 2524, 0, 0, 0),
    "one_card_few": (lambda: one_card(60), None, 1, 0, 1),
}


@pytest.fixture(scope="module")
def egt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_03063_amd import egt as mod

    return mod


@pytest.mark.parametrize("name", list(GAMES))
def test_routes(egt, name):
    make, seqs, pairs, hands, columns = GAMES[name]
    G = egt.Game(make())
    print(f"[case] {name}: {G.n} hands, {G.n_seq} sequences", flush=True)
    assert seqs is None or max(G.n_seq) == seqs
    assert G.routes() == dict(paired_product=pairs, pass_hands=hands, column_gemm=columns)
    product = bench.product_roofline(egt, torch, G, 2, name)
    assert product["kernel"] == ("product_pairs_kernel" if pairs else "product_kernel")
    sbr = bench.sbr_roofline(egt, torch, G, 2, name)
    assert sbr["kernel"] == ("sbr_fused_kernel" if hands else "level-path passes")
    G.close()


@pytest.mark.parametrize("args,seqs,hands", [((1, 6, 4, 4), 84, 1), ((0, 7, 4, 4), 1240, 1), ((5, 8, 4, 20), None, 0)])
def test_general_routes(egt, args, seqs, hands):
    G = egt.GeneralGame(random_efg(*args))
    print(f"[case] general {args}: {G.n_seq} sequences", flush=True)
    assert seqs is None or max(G.n_seq) == seqs
    assert G.routes() == dict(paired_product=0, pass_hands=hands, column_gemm=0)
    G.close()
