"""The precision form's products on rows that are aligned to 8 bytes, as callers
promise, and to 4: the same bits as on aligned rows, for each of the three
showdown GEMMs (their 16-byte loads, and the column form's 16-byte stores)."""
import pytest

from tests.test_gpu_level_path import offset
from tests.test_gpu_mixed_padding import GAMES, strategy

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def egt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1810_03063_amd import egt as mod

    return mod


@pytest.mark.parametrize("elements", [2, 1])
@pytest.mark.parametrize("name", list(GAMES))
def test_products(egt, name, elements):
    G = egt.Game(GAMES[name]())
    print(f"[case] {name}: {G.n} hands, {G.n_seq} sequences, rows {4 * elements}-byte aligned", flush=True)
    for p in (0, 1):
        v = strategy(G, 1 - p, 5).cuda()
        want = egt.gradient_mixed(G, p, v)
        got = egt.gradient_mixed(G, p, offset(v, elements), offset(torch.full_like(want, float("nan")), elements))
        assert got.data_ptr() % 16 == 4 * elements
        assert torch.equal(got, want)
    G.close()
