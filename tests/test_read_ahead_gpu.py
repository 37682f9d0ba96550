"""Launches that store enough to read their next inputs ahead (read-ahead
tiles): the outputs are those of the callbacks called one by one at a size
that reads nothing ahead, bit for bit, and every entry is written."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from exa_modeling import DataSet, Model, sin
from exa_modeling.generators import Workload, goddard
from parity_util import dev

pytestmark = pytest.mark.gpu


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def formulation(n, seed=2):
    """n points with dense derivatives: a gathered, a reversed and an
    increasing index column (whose last reference ends at the last variable),
    data and parameter values, a weight per point."""
    rng = np.random.default_rng(seed)
    m = Model("ahead")
    x = m.add_var(n + 3)
    d = DataSet(n, i=np.arange(n), r=np.arange(n)[::-1] + 1, g=rng.integers(0, n + 3, n), c=rng.uniform(0.5, 1.5, n))
    p = x[d.i] * x[d.i + 3]
    q = x[d.r] * d.c + x[d.g]
    m.add_con(sin(p + q), d)
    m.add_con(p * q * sin(p - q), d)
    m.add_obj(p ** 2 * q, d)
    return Workload(m, rng.uniform(-1, 1, m.nvar), rng.standard_normal(m.ncon), 0.7)


def nan(n):
    return torch.full((n,), float("nan"), dtype=torch.float64, device="cuda:0")


def outputs(em):
    return dict(f=nan(1), g=nan(em.nvar), c=nan(em.ncon), jac=nan(em.nnzj), hess=nan(em.nnzh), jv=nan(em.ncon),
                jtw=nan(em.nvar), hv=nan(em.nvar))


# 96 MiB of Hessian values are about 466,000 points (27 slots); the first
# size stays below, the last has the Jacobian above it as well
@pytest.mark.parametrize("n", [300_001, 500_001, 1_600_003])
def test_large_launches(n, tmp_path):
    _gpu()
    from paper_2608_16265_amd import ExaModel
    w = formulation(n)
    em = ExaModel(w.model, cache_dir=str(tmp_path))
    rng = np.random.default_rng(1)
    X, Y, V, W = dev(w.x), dev(w.y), dev(rng.standard_normal(em.nvar)), dev(rng.standard_normal(em.ncon))
    one = ExaModel(w.model, cache_dir=str(tmp_path), block=64, epl=1, fuse=False)
    ref = dict(g=one.grad(X, nan(em.nvar)), c=one.cons(X, nan(em.ncon)), jac=one.jac_coord(X, nan(em.nnzj)),
               hess=one.hess_coord(X, Y, 0.7, nan(em.nnzh)), jv=one.jprod(X, V, nan(em.ncon)),
               jtw=one.jtprod(X, W, nan(em.nvar)), hv=one.hprod(X, Y, 0.7, V, nan(em.nvar)))
    for sel in (("jac",), ("hess",), ("jac", "hess"), ("f", "g", "c", "jac", "hess", "jv", "jtw", "hv")):
        out = {k: v for k, v in outputs(em).items() if k in sel}
        em.evaluate(X, Y, 0.7, V, W, **out)
        for k in sel:
            assert not bool(torch.isnan(out[k]).any()), (sel, k)
            assert k == "f" or torch.equal(out[k], ref[k]), (sel, k)
    assert torch.equal(em.hess_coord(X, Y, 0.7, nan(em.nnzh)), ref["hess"])


def test_large_batch():
    """Instances of several sizes, each read ahead during the one before it
    in its XCD's list; the second batch is one list of small instances."""
    _gpu()
    from paper_2608_16265_amd import ExaModel
    from paper_2608_16265_amd.batch import ExaBatch
    wls = [goddard(n, seed=n) for n in (60_000, 9, 30_001, 41_000, 64, 20_000, 70_003, 1_000, 50_000, 12_345, 3)]
    ems = [ExaModel(w.model) for w in wls]
    rng = np.random.default_rng(3)
    for order in (ems, ems[::-1]):
        b = ExaBatch(order, autotune=False)
        x, y, v, w = (dev(rng.uniform(0.5, 1.5, b.total(s))) for s in "xyxy")
        out = dict(f=b.empty("B"), g=nan(b.total("x")), c=nan(b.total("y")), jac=nan(b.total("jac")),
                   hess=nan(b.total("hess")), jv=nan(b.total("y")), jtw=nan(b.total("x")), hv=nan(b.total("x")))
        for _ in range(2):
            b.evaluate(x, y, 0.6, v, w, **out)
        for i, em in enumerate(order):
            xs, ys = x[b.slice("x", i)].clone(), y[b.slice("y", i)].clone()
            vs, ws = v[b.slice("x", i)].clone(), w[b.slice("y", i)].clone()
            ref = dict(g=em.grad(xs), c=em.cons(xs), jac=em.jac_coord(xs), hess=em.hess_coord(xs, ys, 0.6),
                       jv=em.jprod(xs, vs), jtw=em.jtprod(xs, ws), hv=em.hprod(xs, ys, 0.6, vs))
            where = dict(g="x", c="y", jac="jac", hess="hess", jv="y", jtw="x", hv="x")
            for k in ref:
                assert torch.equal(out[k][b.slice(where[k], i)], ref[k]), (k, i)
        b.close()
