"""Models under a device-memory budget: the estimate bounds what is allocated,
and a model that does without the units that finish sums gives the same bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from exa_modeling import DataSet, sin
from exa_modeling.generators import Workload, goddard, rosenbrock
from test_incidence_gpu import network
from test_sums_gpu import forms, inputs, nan

pytestmark = pytest.mark.gpu


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("make", [lambda: rosenbrock(2, 1), lambda: rosenbrock(20000, 1), lambda: goddard(1, 1),
                                  lambda: goddard(3000, 1), lambda: forms("gaps", 2), lambda: forms("shared", 513),
                                  lambda: network("hub", 100, 300), lambda: network("plain", 60000, 80000)])
def test_estimate_bounds_allocation(make):
    _gpu()
    from paper_2608_16265_amd import ExaModel
    m = make().model
    est = ExaModel(m, host_only=True).device_bytes()
    em = ExaModel(m, max_device_bytes=est)
    assert 0 < em.device_bytes() <= est


def test_without_finishing_units():
    _gpu()
    from paper_2608_16265_amd import ExaModel
    from paper_2608_16265_amd.batch import ExaBatch
    # links in the map, an objective of 30 tiles, and a short chain whose units
    # take a little more than they save
    w = network("plain", 60000, 80000)
    m = w.model
    z, d = m.add_var(3), DataSet(2, i=np.arange(2))
    m.add_con(z[d.i] * sin(z[d.i + 1]), d)
    w = Workload(m, np.concatenate([w.x, [0.3, -0.7, 1.1]]), np.zeros(0), 0.7)
    full = ExaModel(w.model)
    budget = ExaModel(w.model, host_only=True).device_bytes()
    for _ in range(2):  # first the tiles, then the units give way
        budget = ExaModel(w.model, host_only=True, max_device_bytes=budget - 1).device_bytes()
    lean = ExaModel(w.model, max_device_bytes=budget)
    sums = lambda em: em.generated_source().split("sums finished by units: ")[1].split("\n")[0]
    assert lean.device_bytes() <= budget and "U" not in sums(lean) and "U" in sums(full)
    X, Y, V, W = inputs(w, full)
    want = dict(f=full.obj(X), g=full.grad(X), jtw=full.jtprod(X, W), hv=full.hprod(X, Y, 0.6, V))
    lag = full.lag_grad(X, Y, 0.6)
    assert torch.equal(lean.obj(X), want["f"]) and lean.obj_host(X) == float(want["f"])
    assert torch.equal(lean.jtprod(X, W), want["jtw"]) and torch.equal(lean.hprod(X, Y, 0.6, V), want["hv"])
    out = dict(f=nan(1), g=nan(full.nvar), jtw=nan(full.nvar), hv=nan(full.nvar))
    lean.evaluate(X, Y, 0.6, V, W, **out)
    assert all(torch.equal(out[k], want[k].reshape(out[k].shape)) for k in out)
    b = ExaBatch([lean, full], autotune=False)
    x, y, v, u = (torch.cat((t, t)) for t in (X, Y, V, W))
    out = dict(f=b.empty("B"), jtw=nan(b.total("x")), hv=nan(b.total("x")))
    l2 = nan(b.total("x"))
    b.evaluate(x, y, 0.6, v, u, **out)
    b.evaluate(x, y, 0.6, lag=l2)
    for i in range(2):
        s = b.slice("x", i)
        assert torch.equal(out["f"][i:i + 1], want["f"].reshape(1)), i
        assert torch.equal(out["jtw"][s], want["jtw"]) and torch.equal(out["hv"][s], want["hv"]), i
        assert torch.equal(l2[s], lag), i
    b.close()
