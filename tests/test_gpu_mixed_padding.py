"""The padding of the precision form's products, entries n_hands .. ld - 1 of
every row: written 0 whatever the other entries are (an infinite strategy entry
reaches its rows, not their padding), and not read from an input.  Games for
each of the three showdown GEMMs, with hand counts that leave a partly filled
unit of eight hands, and one-card hands whose rows are mostly padding."""
import numpy as np
import pytest

from instances import make_instance
from instances.endgames import Instance, river
from tests.test_gpu_mixed_columns import many_hands

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def two_hands():
    return Instance(name="two-hands", n_cards=2, cards_per_hand=1, board=np.zeros(0, dtype=np.int32),
                    hand_cards=np.arange(2, dtype=np.int32).reshape(2, 1), strength=np.arange(2, dtype=np.int32),
                    belief=np.full((2, 2), 0.5), pot=2.0, stack=4.0, bet_fracs=(0.5, 1.0), allin=True, max_raises=2)


GAMES = {
    "k_split_105h": lambda: make_instance("c0", 0),
    "k_split_two_hands": two_hands,
    "columns_351h": lambda: river("x", 1, 8, "ranking_ties10", 0.5, 1000.0, 20000.0, (0.25, 0.5, 1.0, 2.0), 4),
    "columns_1081h": lambda: river("x", 2, 13, "ranking_ties10", 0.5, 1000.0, 20000.0,
                                   (0.25, 0.5, 0.75, 1.0, 1.5, 2.0, 3.0), 3),
    "tiled_1300h": lambda: many_hands(1300, 3),
}


@pytest.fixture(scope="module")
def egt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_03063_amd import egt as mod

    return mod


def strategy(G, p, seed):
    gen = torch.Generator().manual_seed(seed)
    v = torch.zeros((G.n_seq[p], G.ld))
    v[:, :G.n] = torch.rand((G.n_seq[p], G.n), generator=gen)
    return v


def product(egt, G, p, v):
    out = torch.full((G.n_seq[p], G.ld), float("nan"), dtype=torch.float32, device="cuda")
    return egt.gradient_mixed(G, p, v.cuda(), out).cpu()


@pytest.mark.parametrize("value", [None, np.inf, np.nan])
@pytest.mark.parametrize("name", list(GAMES))
def test_written_zero(egt, name, value):
    G = egt.Game(GAMES[name]())
    print(f"[case] {name}: {G.n} hands, {G.n_seq} sequences, a hand's entries {value}", flush=True)
    for p in (0, 1):
        v = strategy(G, 1 - p, 3)
        if value is not None:
            v[:, G.n // 2] = value
        out = product(egt, G, p, v)
        if value is not None:
            assert not torch.isfinite(out[:, :G.n]).all()
        assert torch.all(out[:, G.n:].contiguous().view(torch.int32) == 0), "the padding holds +0.0"
    G.close()


@pytest.mark.parametrize("name", list(GAMES))
def test_input_padding_is_ignored(egt, name):
    G = egt.Game(GAMES[name]())
    print(f"[case] {name}: {G.n} hands, {G.n_seq} sequences", flush=True)
    for p in (0, 1):
        v = strategy(G, 1 - p, 4)
        want = product(egt, G, p, v)
        assert torch.isfinite(want).all()
        for value in (np.nan, np.inf):
            v[:, G.n:] = value
            assert torch.equal(product(egt, G, p, v), want)
    G.close()
