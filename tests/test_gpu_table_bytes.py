"""The device tables of a game stay within what its description has been charged
for: a batch whose budget is the state plus those bytes admits the solve.  Bytes
per game (FP64, precision form) as charged with per-player node, sequence and
terminal arrays and no tables that only one route reads."""
import pytest

from instances import make_instance
from instances.endgames import river

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

QUARTERS, FIVE, SEVEN = (0.25, 0.5, 1.0, 2.0), (0.25, 0.5, 0.75, 1.0, 2.0), (0.25, 0.5, 0.75, 1.0, 1.5, 2.0, 3.0)


def tree(ranks, fracs, raises):
    return lambda: river("x", 3, ranks, "ranking_ties10", 0.5, 1000.0, 20000.0, fracs, raises)


GAMES = {
    "kuhn": (lambda: make_instance("kuhn", 0), 11520, 15616),
    "micro": (lambda: make_instance("micro", 0), 14080, 18176),
    "c0": (lambda: make_instance("c0", 0), 20480, 55808),
    "c1": (lambda: make_instance("c1", 0), 134656, 2516480),
    "c3": (lambda: make_instance("c3", 0), 2403328, 4906496),
    "lib": (lambda: make_instance("lib", 0), 106496, 2486784),
    "1081h_286": (tree(13, QUARTERS, 2), 157696, 2540032),
    "1081h_520": (tree(13, FIVE, 2), 251904, 2639872),
    "1081h_808": (tree(13, QUARTERS, 3), 366080, 2760192),
    "105h_808": (tree(5, QUARTERS, 3), 331264, 382976),
    "595h_190": (tree(10, SEVEN, 1), 100608, 849152),
}


@pytest.fixture(scope="module")
def egt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_03063_amd import egt as mod

    return mod


@pytest.mark.parametrize("name", list(GAMES))
def test_admitted_at_the_same_budget(egt, name):
    make, *charged = GAMES[name]
    inst = make()
    G = egt.Game(inst)
    for precision, tables in zip(("fp64", "mixed"), charged):
        print(f"[case] {name} {precision}", flush=True)
        b = egt.Batch(budget_bytes=egt.state_bytes(G, precision=precision) + tables, max_slots=1)
        slot = b.admit_desc(inst, precision=precision, max_iters=1)
        assert slot is not None, "refused"
        print(f"tables: {b.usage()[0] - egt.state_bytes(G, precision=precision)} of {tables} bytes", flush=True)
        while b.poll(slot) is None:
            b.tick()
        b.retire(slot)
        b.close()
    G.close()
