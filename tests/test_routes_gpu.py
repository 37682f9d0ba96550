"""What runs, beside what comes out: no reduction where units finish every sum,
read-ahead tiles where a launch stores enough, the products against the
coordinate values, each instance's objective in a batch, and infinities and
NaN where bilinear terms put them and nowhere else."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from exa_modeling import DataSet, Model
from exa_modeling.generators import Workload, acopf, goddard, pde, rosenbrock
from parity_util import dev, host
from test_incidence_gpu import network
from test_read_ahead_gpu import formulation
from test_sums_gpu import forms, inputs, nan

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("make,left", [
    (lambda: acopf(300, 1), False), (lambda: pde(66, 1), False), (lambda: rosenbrock(4100, 1), False),
    (lambda: network("both", 300, 400), False), (lambda: network("long", 100, 300), True),
    (lambda: goddard(700, 1), True)], ids=["acopf", "pde", "rosenbrock", "lists", "long list", "shared step"])
def test_what_the_reduction_is_left(make, left):
    _gpu()
    from paper_2608_16265_amd import ExaModel
    em = ExaModel(make().model)
    b = em.eval_bytes(("grad", "jtprod", "hprod"))
    assert (b["reduce_read"] + b["reduce_write"] > 0) == left, b


@pytest.mark.parametrize("n,ahead", [(300_001, False), (500_001, True)])
def test_read_ahead_tiles(n, ahead, tmp_path):
    """27 Hessian values a point: 65 and 108 MB."""
    _gpu()
    from paper_2608_16265_amd import ExaModel
    em = ExaModel(formulation(n).model, cache_dir=str(tmp_path))
    em.set_eval_schedule(("hess",), 256, 4, True)
    points = -(-n // 1024)
    tiles = em.eval_schedule(("hess",))["tiles"]
    # x, y, the two index columns and the data column, 256 KB and less a tile
    assert tiles - points in (range(40, 2000) if ahead else range(1)), (tiles, points)


@pytest.mark.parametrize("kind,nb,nl", [("hub", 100, 300), ("loops", 50, 120), ("both", 300, 400), ("ring", 60000, 80000)])
def test_products_from_coordinate_values(kind, nb, nl, tmp_path):
    """J^T w and H v against sums of the Jacobian's and Hessian's entries."""
    _gpu()
    from paper_2608_16265_amd import ExaModel
    w = network(kind, nb, nl)
    em = ExaModel(w.model, cache_dir=str(tmp_path))
    X, Y, V, W = inputs(w, em)
    v, u = host(V), host(W)
    r, c = em.jac_structure()
    jac = host(em.jac_coord(X))
    ref, mag = np.zeros(em.nvar), np.zeros(em.nvar)
    np.add.at(ref, c, jac * u[r])
    np.add.at(mag, c, np.abs(jac * u[r]))
    # an entry may be the sum of a few terms of up to 10 times its size; at
    # most 130 additions on either side
    assert np.all(np.abs(host(em.jtprod(X, W)) - ref) <= 200 * EPS * mag)
    r, c = em.hess_structure()
    h = host(em.hess_coord(X, Y, 0.6))
    ref, mag = np.zeros(em.nvar), np.zeros(em.nvar)
    for i, j in ((r, c), (c, r)):
        on = r != c if i is c else np.ones(r.size, bool)
        np.add.at(ref, i[on], (h * v[j])[on])
        np.add.at(mag, i[on], np.abs(h * v[j])[on])
    # entries of several derivative terms each
    assert np.all(np.abs(host(em.hprod(X, Y, 0.6, V)) - ref) <= 2000 * EPS * (mag + np.abs(mag).max() * 1e-3))


def test_objective_of_each_instance():
    _gpu()
    from paper_2608_16265_amd import ExaModel
    from paper_2608_16265_amd.batch import ExaBatch
    wls = [forms("plain", 70), forms("gaps", 90), forms("reversed", 130), forms("plain", 5000)]
    ems = [ExaModel(w.model) for w in wls]
    b = ExaBatch(ems, autotune=False)
    x, f = torch.cat([dev(w.x) for w in wls]), nan(len(wls))
    for _ in range(3):
        f.fill_(float("nan"))
        b.evaluate(x, f=f)
        for i, em in enumerate(ems):
            assert torch.equal(f[i:i + 1], em.obj(x[b.slice("x", i)].clone()).reshape(1)), i
    b.close()


def bilinear(kind, n, rng):
    """Rows a[i] b[j] over one data set; the two variables of every point."""
    m = Model("bilinear " + kind)
    x = m.add_var(3 * n + 40)
    k = np.arange(n)
    i, j = dict(chain=(k, k + 1), gaps=(3 * k, 3 * k + 1), lists=(rng.integers(0, n, n), rng.integers(0, n, n)),
                shared=(k, np.full(n, 3 * n + 5)), period=(k, 3 * n + 8 + k % 8),
                map=(np.where(k < 80, 0, k), (k * 7) % n))[kind]
    if kind == "chain":
        d = DataSet(n, i=i)
        m.add_con(x[d.i] * x[d.i + 1], d)
    elif kind == "gaps":
        d = DataSet(n, i=i)
        m.add_con(x[d.i] * x[d.i + 1], d)
    elif kind == "shared":
        d = DataSet(n, i=i)
        m.add_con(x[d.i] * x[3 * n + 5], d)
    else:
        d = DataSet(n, i=i, j=j)
        m.add_con(x[d.i] * x[d.j], d)
    return m, i, j


@pytest.mark.parametrize("n", [64, 200, 1031])
@pytest.mark.parametrize("kind", ["chain", "gaps", "lists", "shared", "period", "map"])
def test_nonfinite_values_stay_where_they_belong(kind, n):
    """J^T w adds w x[j] to i and w x[i] to j, H v adds y v[j] to i and y v[i]
    to j: NaN, infinities and finite values, entry by entry."""
    _gpu()
    from paper_2608_16265_amd import ExaModel
    rng = np.random.default_rng(n)
    m, i, j = bilinear(kind, n, rng)
    em = ExaModel(m)

    def with_bad(size):
        a = rng.uniform(0.5, 1.5, size)
        at = np.unique(np.concatenate([[0, size - 1], rng.integers(0, size, 3)]))
        a[at] = rng.choice([np.nan, np.inf, -np.inf], at.size)
        return a
    fine = lambda size: rng.uniform(0.5, 1.5, size)  # noqa: E731
    for bad in ("x", "w", "v", "y", "all"):
        x, w, v, y = (with_bad(s) if bad in (name, "all") else fine(s)
                      for name, s in (("x", em.nvar), ("w", n), ("v", em.nvar), ("y", n)))
        with np.errstate(invalid="ignore", over="ignore"):
            for got, p, q, wt in ((em.jtprod(dev(x), dev(w), nan(em.nvar)), x[j], x[i], w),
                                  (em.hprod(dev(x), dev(y), 0.6, dev(v), nan(em.nvar)), v[j], v[i], y)):
                ref = np.zeros(em.nvar)
                np.add.at(ref, i, wt * p)
                np.add.at(ref, j, wt * q)
                g = host(got)
                assert np.array_equal(np.isnan(g), np.isnan(ref)), (bad, np.flatnonzero(np.isnan(g) != np.isnan(ref)))
                inf = np.isinf(ref)
                assert np.array_equal(g[inf], ref[inf]), bad
                ok = np.isfinite(ref)
                # at most 2 n additions of products of up to 1.5 squared
                assert np.all(np.abs(g[ok] - ref[ok]) <= 2 * n * EPS * np.maximum(1.0, np.abs(ref[ok]))), bad
