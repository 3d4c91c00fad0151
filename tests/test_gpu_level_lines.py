"""The launch-per-level smoothed best response on both sides of two lines: the
lowest level with one and with two hands per lane, and the top-down pass with a
wavefront per sequence and per part of a node (16 wavefronts per compute unit
each; those of a tree in the comment, lowest level and top-down pass, in FP64).
Rows that are aligned to one element only take the other forms, with the same
bits.

Tolerances are those of the operations elsewhere: strategies 1e-12 absolute and
values 1e-13 of the size of the terms they add."""
import numpy as np
import pytest

from instances.endgames import river
from oracle import Problem
from tests.layout import Layout
from tests.test_gpu_fused_pass import QUARTERS, SEVEN, check
from tests.test_gpu_level_path import offset

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TREES = [
    (5, QUARTERS, 3),  # 1 and 3, 105 hands
    (5, SEVEN, 3),     # 4 and 12
    (5, SEVEN, 4),     # 7 and 23
    (8, SEVEN, 3),     # 11 and 35, 351 hands
    (8, SEVEN, 4),     # 21 and 70
]


@pytest.fixture(scope="module")
def egt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_03063_amd import egt as mod

    return mod


@pytest.mark.parametrize("ranks,fracs,raises", TREES)
def test_forms(egt, ranks, fracs, raises):
    inst = river("x", 9, ranks, "ranking_ties10", 0.5, 1000.0, 20000.0, fracs, raises)
    P, G = Problem(inst), egt.Game(inst)
    assert G.routes()["pass_hands"] == 0
    L = Layout(G, P)
    rng = np.random.default_rng(17)
    for p in (0, 1):
        print(f"[case] {inst.n_hands} hands, {G.n_seq[p]} sequences, player {p}", flush=True)
        g = 10.0 * rng.standard_normal((P.n_seq[p], P.n))
        check(egt, G, P, L, g, p, 0.5)
        rows = torch.from_numpy(np.ascontiguousarray(L.to_lib(p, g))).cuda()
        for dtype, run in ((torch.float64, egt.smoothed_br), (torch.float32, egt.smoothed_br_mixed)):
            x = rows.to(dtype)
            q, val = run(G, p, x, 0.5)
            q1, val1 = run(G, p, offset(x, 1), 0.5, strat_out=offset(torch.zeros_like(x), 1))
            assert torch.equal(q, q1) and torch.equal(val, val1)
    G.close()
