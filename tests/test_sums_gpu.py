"""Sums (gradient, J^T w, H v, Lagrangian gradient) that the evaluation units
finish themselves: against the oracle at the sizes where their lane mapping
can go wrong (chunks of 64 - S owners, runs of several chunks, first and last
points of a chain, gaps in index columns, variables nothing contributes to),
and every way of calling them bit for bit the same."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from exa_modeling import DataSet, Model, exp, sin
from exa_modeling.generators import Workload, acopf, goddard, pde, rosenbrock, two_stage
from parity_util import dev, host
from test_parity_gpu import check_all

pytestmark = pytest.mark.gpu


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def forms(kind, n, seed=1):
    """One data set of n points over columns of every shape the rule tells
    apart, variables before, between and behind the ones it reaches."""
    rng = np.random.default_rng(seed)
    m = Model(kind)
    lead, tail = 5, 7
    i = np.arange(n)
    cols = dict(i=i + lead)
    size = n + lead + 40 + tail
    if kind == "gaps":          # strictly increasing, not by one
        cols["i"] = np.sort(rng.choice(2 * n, n, replace=False)) + lead
        size = 2 * n + lead + 40 + tail
    elif kind == "reversed":    # every variable hit once, points descending
        cols["i"] = i[::-1] + lead
    elif kind == "shared":      # a literal and a period of 4 beside a chain
        cols["s"] = i % 4
    x = m.add_var(size)
    z = m.add_var(6)
    th = m.add_par(rng.uniform(0.5, 1.5, n))
    d = DataSet(n, c=rng.uniform(0.5, 1.5, n), t=i, **cols)
    one = DataSet(1, k=np.zeros(1, dtype=np.int64))
    j = d.i
    if kind == "far":           # one chain of span 3 and one 30 further up
        e = x[j] * x[j + 3] + d.c * sin(x[j + 30])
    elif kind == "wide":        # shift of 8 and of 9: the second is a chain of its own
        e = x[j] * x[j + 8] + d.c * x[j + 17] ** 2
    elif kind == "shared":
        e = x[j] * exp(0.1 * z[5]) + z[d.s] * x[j + 1] ** 2 * d.c
    else:
        e = x[j] * x[j + 1] * d.c + sin(x[j + 2])
    m.add_con(e, d)
    m.add_con(x[j + 1] ** 2 * th[d.t], d)
    m.add_con(x[lead] * x[lead + 1], one)           # hits the chain's first variables
    m.add_con_aug(0, d.t, -x[j], DataSet(n, t=i, **cols))  # weight entries over the same variables
    m.add_obj(d.c * x[j] ** 2, d)                   # at most one objective term per variable
    m.add_obj(z[4] ** 2, one)
    return Workload(m, rng.uniform(-1, 1, m.nvar), rng.standard_normal(m.ncon), 0.7)


CASES = [("rosen", n) for n in (2, 3, 64, 65, 127, 4100)]
CASES += [("goddard", n) for n in (1, 2, 62, 63, 64, 127, 700)]
CASES += [("goddard", 300000)]                      # runs of several chunks
CASES += [("two_stage", n) for n in (4, 33, 9000)]  # periodic columns, runs of several chunks
CASES += [("pde", n) for n in (3, 4, 9, 66)]
CASES += [(k, n) for k in ("plain", "gaps", "reversed", "far", "wide", "shared") for n in (1, 2, 64, 65, 513)]


def case(kind, n):
    make = dict(rosen=rosenbrock, goddard=goddard, pde=pde, two_stage=two_stage)
    return make[kind](n, seed=4) if kind in make else forms(kind, n)


def inputs(w, em, seed=3):
    rng = np.random.default_rng(seed)
    y = w.y if w.y.size == em.ncon else rng.standard_normal(em.ncon)
    return dev(w.x), dev(y), dev(rng.standard_normal(em.nvar)), dev(rng.standard_normal(em.ncon))


def nan(n):
    return torch.full((n,), float("nan"), dtype=torch.float64, device="cuda:0")


@pytest.fixture(scope="module")
def cache(tmp_path_factory):
    """Sizes of one kind share their generated code: compiled once."""
    return str(tmp_path_factory.mktemp("code"))


@pytest.mark.parametrize("kind,n", CASES, ids=lambda v: str(v))
def test_sums_finished_by_units(kind, n, cache):
    _gpu()
    from paper_2608_16265_amd import ExaModel
    w = case(kind, n)
    em, _ = check_all(w, ExaModel(w.model, cache_dir=cache), tag=f"{kind} {n}: ")
    X, Y, V, W = inputs(w, em)
    sig = 0.6
    ref = dict(g=em.grad(X, nan(em.nvar)), jtw=em.jtprod(X, W, nan(em.nvar)), hv=em.hprod(X, Y, sig, V, nan(em.nvar)))
    lag = em.lag_grad(X, Y, sig, nan(em.nvar))
    if n <= 4100:
        alts = [dict(block=b, epl=e, fuse=f) for b, e, f in ((64, 1, False), (128, 3, True), (256, 8, False))]
        for kw in alts:
            alt = ExaModel(w.model, cache_dir=cache, **kw)
            out = {k: nan(em.nvar) for k in ref}
            alt.evaluate(X, Y, sig, V, W, **out)
            for k in ref:
                assert torch.equal(out[k], ref[k]), (k, kw)
            assert torch.equal(alt.lag_grad(X, Y, sig, nan(em.nvar)), lag), kw
            assert torch.equal(alt.hprod(X, Y, sig, V, nan(em.nvar)), ref["hv"]), kw
    # the one-pass units leave these sums to the same units
    cbs = ("obj", "grad", "cons", "jac", "hess", "jprod", "jtprod", "hprod")
    em.set_eval_schedule(cbs, 128, 2, True, "one_pass")
    out = dict(f=nan(1), g=nan(em.nvar), c=nan(em.ncon), jac=nan(em.nnzj), hess=nan(em.nnzh), jv=nan(em.ncon),
               jtw=nan(em.nvar), hv=nan(em.nvar))
    em.evaluate(X, Y, sig, V, W, **out)
    for k in ref:
        assert torch.equal(out[k], ref[k]), k
    assert not any(bool(torch.isnan(t).any()) for t in out.values())


def test_batch_of_instances_whose_sums_differ():
    """Instances of one formulation whose index columns take different forms:
    each keeps its own units, and its own bits."""
    _gpu()
    from paper_2608_16265_amd import ExaModel
    from paper_2608_16265_amd.batch import ExaBatch
    wls = [forms("plain", 70), forms("gaps", 90), forms("reversed", 130), forms("plain", 20), forms("gaps", 33)]
    for w in wls:
        w.model.name = "mixed"
    ems = [ExaModel(w.model) for w in wls]
    b = ExaBatch(ems, autotune=False)
    ins = [inputs(w, em, seed=k) for k, (w, em) in enumerate(zip(wls, ems))]
    X, Y, V, W = (torch.cat(t) for t in zip(*ins))
    sig = 0.4
    out = dict(f=b.empty("B"), g=nan(b.total("x")), c=nan(b.total("y")), jac=nan(b.total("jac")),
               hess=nan(b.total("hess")), jv=nan(b.total("y")), jtw=nan(b.total("x")), hv=nan(b.total("x")))
    lag = nan(b.total("x"))
    for _ in range(3):
        b.evaluate(X, Y, sig, V, W, **out)
        b.evaluate(X, Y, sig, lag=lag)
    for i, (em, (x, y, v, w)) in enumerate(zip(ems, ins)):
        s = b.slice("x", i)
        assert torch.equal(out["g"][s], em.grad(x)) and torch.equal(out["jtw"][s], em.jtprod(x, w)), i
        assert torch.equal(out["hv"][s], em.hprod(x, y, sig, v)) and torch.equal(lag[s], em.lag_grad(x, y, sig)), i
        assert torch.equal(out["jac"][b.slice("jac", i)], em.jac_coord(x)), i
        assert torch.equal(out["hess"][b.slice("hess", i)], em.hess_coord(x, y, sig)), i
        assert torch.equal(out["c"][b.slice("y", i)], em.cons(x)) and torch.equal(out["jv"][b.slice("y", i)], em.jprod(x, v)), i
    b.close()


@pytest.mark.parametrize("sigma", [float("inf"), -0.0, float("nan")])
def test_lagrangian_gradient_keeps_nonfinite_weights(sigma):
    """sigma * gradient is formed for every variable, also where the
    gradient is zero: infinities and NaN come out as the composition gives."""
    _gpu()
    from paper_2608_16265_amd import ExaModel
    for w in (acopf(70, 3), goddard(65, 2), forms("plain", 65)):
        em = ExaModel(w.model)
        X, Y, _, _ = inputs(w, em)
        got = host(em.lag_grad(X, Y, sigma))
        ref = host(em.grad(X).mul_(sigma).add_(em.jtprod(X, Y)))
        assert np.array_equal(got, ref, equal_nan=True)


def test_large_map_beside_middling_segments():
    """A map of one lane per segment (over 2^22 entries) with two segments of
    some 300 entries, which blocks of their own add."""
    _gpu()
    from paper_2608_16265_amd import ExaModel
    N, K = (1 << 22) + 77, 600
    rng = np.random.default_rng(8)
    m = Model("large")
    x = m.add_var(N + 2)
    perm, hub = rng.permutation(N), N + rng.integers(0, 2, K)
    d, e = DataSet(N, i=perm), DataSet(K, h=hub)
    m.add_con(sin(x[d.i]), d)
    m.add_con(exp(x[e.h]), e)
    em = ExaModel(m)
    xv, wv = rng.uniform(-1, 1, N + 2), rng.standard_normal(N + K)
    got = host(em.jtprod(dev(xv), dev(wv), nan(N + 2)))
    ref = np.zeros(N + 2)
    ref[perm] = np.cos(xv[perm]) * wv[:N]
    for h in (N, N + 1):
        ref[h] = np.exp(xv[h]) * wv[N:][hub == h].sum()
    # two cosines (a few ulp of 1) and products on each side; 600 additions
    # behind a factor of at most e for the two long segments
    assert np.abs(got[:N] - ref[:N]).max() <= 8 * 2.0 ** -53 * np.abs(wv).max()
    assert np.abs(got[N:] - ref[N:]).max() <= 2.0 ** -53 * K * np.e * np.abs(wv[N:]).sum()
