"""The precision form's products on both sides of the lines between the showdown
GEMMs: K-split tiles of 32 columns x 32 hands in one round and column blocks where
they would take two, and column blocks from 512 columns on.

Tolerance, per entry, relative to the sum of the absolute terms: the BF16 hi + lo
split of a reach is off by 2^-18 of it, FP32 sums of up to 2048 terms by at most
2048 x 2^-24: together below 1.3e-4."""
import numpy as np
import pytest

from instances.endgames import river
from oracle import Problem
from tests.layout import Layout
from tests.test_gpu_mixed_columns import many_hands
from tests.test_gpu_ops import grad_bound
from tests.test_gpu_product_pairs import SIZES

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

QUARTERS = (0.25, 0.5, 1.0, 2.0)


def tree(ranks, fracs, raises):
    return lambda: river("x", 8, ranks, "ranking_ties10", 0.5, 1000.0, 20000.0, fracs, raises)


# name: game, by column blocks
GAMES = {
    "105h_520": (tree(5, SIZES, 2), 0),      # 347 columns, 44 tiles
    "105h_808": (tree(5, QUARTERS, 3), 1),   # 539 columns, 68 tiles
    "595h_520": (tree(10, SIZES, 2), 0),     # 347 columns, 209 tiles
    "741h_520": (tree(11, SIZES, 2), 1),     # 347 columns, 264 tiles
    "1300h_few": (lambda: many_hands(1300, 1), 0),
}


@pytest.fixture(scope="module")
def egt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_03063_amd import egt as mod

    return mod


@pytest.mark.parametrize("name", list(GAMES))
def test_products(egt, name):
    make, columns = GAMES[name]
    inst = make()
    P, G = Problem(inst), egt.Game(inst)
    L = Layout(G, P)
    print(f"[case] {name}: {inst.n_hands} hands, {G.n_seq} sequences", flush=True)
    assert G.routes()["column_gemm"] == columns
    rng = np.random.default_rng(32)
    for p in (0, 1):
        v = rng.random((P.n_seq[1 - p], P.n)).astype(np.float32)
        lib = torch.from_numpy(L.to_lib(1 - p, v.astype(np.float64))).float().cuda()
        out = torch.full((G.n_seq[p], G.ld), np.nan, dtype=torch.float32, device="cuda")
        got = egt.gradient_mixed(G, p, lib, out).double().cpu().numpy()
        want = P.grad_x(v.astype(np.float64)) if p == 0 else P.grad_y(v.astype(np.float64))
        assert np.all(got[:, P.n:] == 0)
        assert np.all(np.abs(L.from_lib(p, got) - want) <= 1.3e-4 * grad_bound(P, p, v.astype(np.float64)) + 1e-30)
    G.close()
