"""Sums pulled through incidence lists (references in no order, such as a
network's branch ends): against the oracle at the sizes where the tiles of
entries and variables can go wrong, the longest list a unit takes and one
longer, points that hit a variable twice, variables without entries, and every
way of calling them bit for bit the same."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from exa_modeling import DataSet, Model, cos, sin
from exa_modeling.generators import Workload
from parity_util import dev
from test_parity_gpu import check_all
from test_sums_gpu import inputs, nan

pytestmark = pytest.mark.gpu


def network(kind, nb, nl, seed=1):
    """nl links between nb nodes; two values per node."""
    rng = np.random.default_rng(seed)
    m = Model("net-" + kind)
    a = m.add_var(nb + 2)
    v = m.add_var(nb + 2)
    th = m.add_par(rng.uniform(0.5, 1.5, nb))
    f, t = rng.integers(0, nb, nl), rng.integers(0, nb, nl)
    if kind == "hub":           # one node with 64 entries, the longest list
        f[:], t[:] = 1 + np.arange(nl) % (nb - 1), 1 + (np.arange(nl) + 1) % (nb - 1)
        f[:64] = 0
    elif kind == "long":        # 65: stays in the reduction
        f[:], t[:] = 1 + np.arange(nl) % (nb - 1), 1 + (np.arange(nl) + 1) % (nb - 1)
        f[:65] = 0
    elif kind == "loops":       # both ends of a point at one node
        t[::3] = f[::3]
    elif kind == "holes":       # most nodes have no entry
        f, t = f // 9 * 9, t // 9 * 9
    elif kind == "ring":        # in the points' order, too many bytes for one L2
        f, t = np.arange(nl) % nb, (np.arange(nl) + 1) % nb
    nodes = DataSet(nb, b=np.arange(nb), c=rng.uniform(0.5, 1.5, nb))
    links = DataSet(nl, f=f, t=t, g=rng.uniform(0.5, 1.5, nl))
    d, n = links, nodes
    if kind in ("before", "both"):
        m.add_con(v[n.b] ** 2 * n.c, nodes)
    e = v[d.f] * v[d.t] * (d.g * cos(a[d.f] - a[d.t]) + sin(a[d.f] - a[d.t]))
    m.add_con(e - v[d.f] ** 2, links)
    m.add_con(e * d.g, links)
    if kind in ("after", "both"):
        m.add_con(a[n.b + 1] * th[n.b] * v[n.b], DataSet(nb, b=np.arange(nb)))
    if kind == "inverse":       # nodes that a strictly increasing column picks
        few = np.sort(rng.choice(nb, max(1, nb // 2), replace=False))
        m.add_con(sin(v[n.b]), DataSet(few.size, b=few))
    m.add_obj(n.c * v[n.b] ** 2, nodes)
    return Workload(m, rng.uniform(0.5, 1.5, m.nvar), rng.standard_normal(m.ncon), 0.7)


CASES = [("plain", 2, 1), ("plain", 2, 3), ("plain", 63, 64), ("plain", 64, 32), ("plain", 65, 200), ("plain", 255, 128),
         ("plain", 257, 129), ("plain", 1000, 1400), ("hub", 100, 300), ("long", 100, 300), ("loops", 50, 120),
         ("ring", 60000, 80000), ("plain", 60000, 80000),  # the second stays in the reduction
         ("holes", 2000, 300), ("before", 130, 260), ("after", 130, 260), ("both", 300, 400), ("inverse", 200, 300)]


@pytest.fixture(scope="module")
def cache(tmp_path_factory):
    return str(tmp_path_factory.mktemp("code"))


@pytest.mark.parametrize("kind,nb,nl", CASES, ids=lambda v: str(v))
def test_lists(kind, nb, nl, cache):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_16265_amd import ExaModel
    w = network(kind, nb, nl)
    em, _ = check_all(w, ExaModel(w.model, cache_dir=cache), tag=f"{kind} {nb} {nl}: ")
    X, Y, V, W = inputs(w, em)
    sig = 0.6
    ref = dict(jtw=em.jtprod(X, W, nan(em.nvar)), hv=em.hprod(X, Y, sig, V, nan(em.nvar)))
    lag = em.lag_grad(X, Y, sig, nan(em.nvar))
    # the products from the coordinate values: a sum of at most 65 products
    # per variable on each side
    assert not any(bool(torch.isnan(t).any()) for t in (*ref.values(), lag))
    for b, e, fu in ((64, 1, False), (64, 4, True), (128, 3, True), (256, 8, False)):
        alt = ExaModel(w.model, cache_dir=cache, block=b, epl=e, fuse=fu)
        out = {k: nan(em.nvar) for k in ref}
        alt.set_eval_schedule(("jtprod", "hprod"), b, e, fu, "per_callback")
        alt.evaluate(X, Y, sig, V, W, **out)
        for k in ref:
            assert torch.equal(out[k], ref[k]), (k, b, e)
        assert torch.equal(alt.lag_grad(X, Y, sig, nan(em.nvar)), lag), (b, e)
        assert torch.equal(alt.jtprod(X, W, nan(em.nvar)), ref["jtw"]), (b, e)
        assert torch.equal(alt.hprod(X, Y, sig, V, nan(em.nvar)), ref["hv"]), (b, e)


def test_batch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_16265_amd import ExaModel
    from paper_2608_16265_amd.batch import ExaBatch
    wls = [network("plain", nb, nl, seed=nb) for nb, nl in ((70, 100), (33, 40), (300, 700), (2, 2), (1000, 1300))]
    wls.append(network("hub", 100, 300))
    wls.append(network("long", 100, 300))
    for w in wls:
        w.model.name = "nets"
    ems = [ExaModel(w.model) for w in wls]
    b = ExaBatch(ems, autotune=False)
    ins = [inputs(w, em, seed=k) for k, (w, em) in enumerate(zip(wls, ems))]
    X, Y, V, W = (torch.cat(t) for t in zip(*ins))
    jtw, hv, lag = nan(b.total("x")), nan(b.total("x")), nan(b.total("x"))
    for _ in range(3):
        b.evaluate(X, Y, 0.4, V, W, jtw=jtw, hv=hv)
        b.evaluate(X, Y, 0.4, lag=lag)
    for i, (em, (x, y, v, u)) in enumerate(zip(ems, ins)):
        s = b.slice("x", i)
        assert torch.equal(jtw[s], em.jtprod(x, u)) and torch.equal(hv[s], em.hprod(x, y, 0.4, v)), i
        assert torch.equal(lag[s], em.lag_grad(x, y, 0.4)), i
    b.close()
