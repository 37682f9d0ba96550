"""The objective of several tiles, added up by the tile that finishes last:
the bits of a batch's reduction launch, call after call, under replay, beside
other callbacks and for every workgroup width."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from exa_modeling import DataSet, Model, exp
from parity_util import dev

pytestmark = pytest.mark.gpu
TILE = 2048


@pytest.mark.parametrize("sizes", [(TILE - 1,), (TILE,), (TILE + 1,), (2 * TILE,), (1, 1), (TILE, 1), (5, 3 * TILE + 7, 64),
                                   (255 * TILE + 1,), (256 * TILE + 1,), (600 * TILE - 3,)], ids=str)
def test_objective(sizes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_16265_amd import ExaModel
    from paper_2608_16265_amd.batch import ExaBatch
    rng = np.random.default_rng(4)
    m = Model("terms")
    n = max(sizes)
    x = m.add_var(n)
    for k in sizes:
        d = DataSet(k, i=np.arange(k), c=rng.uniform(0.5, 1.5, k))
        m.add_obj(d.c * exp(0.1 * x[d.i]) * x[d.i], d)
    em = ExaModel(m)
    xs = [dev(rng.uniform(-1, 1, n)) for _ in range(3)]
    b = ExaBatch([em], autotune=False)
    want = []
    for v in xs:
        f = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda:0")
        b.evaluate(v, None, f=f)
        want.append(f)
    for _ in range(3):
        for v, f in zip(xs, want):
            assert torch.equal(em.obj(v).reshape(1), f)
    for block in (64, 128, 256):
        alt = ExaModel(m, block=block, epl=1)
        for v, f in zip(xs, want):
            o = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda:0")
            g = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda:0")
            alt.evaluate(v, f=o, g=g)
            assert torch.equal(o, f) and not bool(torch.isnan(g).any())
    # a captured graph, with eager calls between its replays
    o, v = torch.zeros(1, dtype=torch.float64, device="cuda:0"), xs[0].clone()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        em.obj(v, o)
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        em.obj(v, o)
    for u, f in zip(xs, want):
        v.copy_(u)
        o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, f) and torch.equal(em.obj(u).reshape(1), f)
    b.close()
