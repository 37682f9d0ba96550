"""Objectives of many tiles: what counting a tile costs, and that overlapping
launches of one model (whose values may then be wrong) leave the next right."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from exa_modeling import DataSet, Model
from parity_util import dev

pytestmark = pytest.mark.gpu
TILE = 2048


def _model(tiles):
    from paper_2608_16265_amd import ExaModel
    n = tiles * TILE
    m = Model("many")
    x = m.add_var(n)
    d = DataSet(n, i=np.arange(n))
    m.add_obj(x[d.i] ** 2, d)
    return ExaModel(m), dev(np.random.default_rng(tiles).uniform(-1, 1, n))


def _best_us(fn, calls=50, rounds=20):
    fn()
    best = float("inf")
    for _ in range(rounds):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            fn()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / calls)
    return best


def test_cost_of_many_tiles():
    """On one address a tile's count takes about 20 ns after the last one's; a
    tile's 16 KB take under 4 ns at the rate of a copy."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    (few, xf), (many, xm) = _model(65), _model(2049)
    of, om = (torch.empty(1, dtype=torch.float64, device="cuda:0") for _ in range(2))
    ns = 1e3 * (_best_us(lambda: many.obj(xm, om)) - _best_us(lambda: few.obj(xf, of))) / (2049 - 65)
    assert ns < 10, ns


@pytest.mark.parametrize("tiles", [2, 33, 489])
def test_after_overlapping_launches(tiles):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    em, x = _model(tiles)
    want = em.obj(x).clone()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [torch.empty(1, dtype=torch.float64, device="cuda:0") for _ in streams]
    for _ in range(5):
        for s, o in zip(streams, outs):
            with torch.cuda.stream(s):
                for _ in range(20):
                    em.obj(x, o)
        torch.cuda.synchronize()
        got = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda:0")
        assert torch.equal(em.obj(x, got), want)
