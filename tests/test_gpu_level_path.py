"""The launch-per-level smoothed best response where its layout changes: levels of
a few nodes (a wavefront per action), of some hundreds (a wavefront per node, one
hand per lane) and of a thousand (two hands per lane), nodes of up to twenty
children and up to ten actions (past the four that the lowest level keeps in
registers), the top-down pass with rows that allow accesses of 16, 8 and 4 bytes,
and temperatures and gradients at the ends of the range.

Tolerances are those of the operations elsewhere: strategies 1e-12 absolute and
values 1e-13 of the size of the terms they add, in FP32 1e-5 and 1e-6; the forms
of one pass evaluate the same operations, so between them the bits agree."""
import numpy as np
import pytest

from instances.endgames import river
from oracle import Problem
from tests.layout import Layout
from tests.test_gpu_fused_pass import QUARTERS, SEVEN, check

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# ranks, bet fractions, raises, stack: nodes one level above the lowest in the comment
TREES = [
    (8, QUARTERS, 3, 20000.0),    # 20, 351 hands
    (13, QUARTERS, 6, 20000.0),   # 198, 1081 hands
    (10, QUARTERS, 6, 200000.0),  # 1045, 595 hands
    (13, SEVEN, 3, 20000.0),      # 51, nodes of ten actions
]


@pytest.fixture(scope="module")
def egt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_03063_amd import egt as mod

    return mod


def offset(t, elements):
    """t on rows that begin `elements` elements past the allocation's alignment."""
    buf = torch.zeros(t.numel() + elements, dtype=t.dtype, device=t.device)
    view = buf[elements:].view(t.shape)
    view.copy_(t)
    return view


@pytest.mark.parametrize("ranks,fracs,raises,stack", TREES)
def test_tree_sizes(egt, ranks, fracs, raises, stack):
    inst = river("x", 5, ranks, "ranking_ties10", 0.5, 1000.0, stack, fracs, raises)
    P, G = Problem(inst), egt.Game(inst)
    L = Layout(G, P)
    rng = np.random.default_rng(14)
    for p in (0, 1):
        print(f"[case] {inst.n_hands} hands, {G.n_seq[p]} sequences, player {p}", flush=True)
        g = 10.0 * rng.standard_normal((P.n_seq[p], P.n))
        check(egt, G, P, L, g, p, 0.5)
        g32 = torch.from_numpy(np.ascontiguousarray(L.to_lib(p, g))).float().cuda()
        q_o, val_o, _, V = P.sbr(p, L.from_lib(p, g32.double().cpu().numpy()), 0.5)
        first = None
        for e in (0, 2, 1):
            q, val = egt.smoothed_br_mixed(G, p, offset(g32, e), 0.5, strat_out=offset(torch.zeros_like(g32), e))
            q, val = q.double().cpu().numpy(), float(val.item())
            assert np.all(q[:, P.n:] == 0)
            assert np.abs(L.from_lib(p, q) - q_o).max() <= 1e-5
            assert abs(val - val_o) <= 1e-6 * (abs(val_o) + np.abs(V).sum())
            first = first or (q, val)
            assert np.array_equal(q, first[0]) and val == first[1]
    G.close()


@pytest.mark.parametrize("mu,scale", [(1e-290, 1.0), (1e290, 1.0), (1e-3, 1e304), (0.5, 1e-300), (3.0, 1.0)])
def test_ends_of_the_range(egt, mu, scale):
    inst = river("x", 6, 5, "ranking_ties10", 0.5, 1000.0, 20000.0, SEVEN, 4)
    P, G = Problem(inst), egt.Game(inst)
    L = Layout(G, P)
    rng = np.random.default_rng(15)
    for p in (0, 1):
        g = scale * rng.standard_normal((P.n_seq[p], P.n))
        leaf = max(range(len(P.tp[p].nodes)), key=lambda v: P.tp[p].nodes[v].first_seq)
        if scale == 1.0:  # an action that is never taken
            g[P.tp[p].nodes[leaf].first_seq] = np.inf
        print(f"[case] mu {mu:g} scale {scale:g} {G.n_seq[p]} sequences, player {p}", flush=True)
        rows = torch.from_numpy(np.ascontiguousarray(L.to_lib(p, g))).cuda()
        q, val = egt.smoothed_br(G, p, rows, mu)
        q1, val1 = egt.smoothed_br(G, p, offset(rows, 1), mu, strat_out=offset(torch.zeros_like(rows), 1))
        with np.errstate(all="ignore"):
            q_o = P.sbr(p, g, mu)[0]
        got = L.from_lib(p, q.cpu().numpy())
        assert np.array_equal(np.isnan(got), np.isnan(q_o))
        assert np.nanmax(np.abs(got - q_o)) <= 1e-12
        assert np.array_equal(q.cpu().numpy(), q1.cpu().numpy(), equal_nan=True)
        assert np.array_equal(val.cpu().numpy(), val1.cpu().numpy(), equal_nan=True)
    G.close()
