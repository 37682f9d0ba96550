"""Points per lane that a caller fixes: a launch nobody has timed keeps them
whatever its size."""
import pytest

torch = pytest.importorskip("torch")

from exa_modeling.generators import pde
from parity_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epl,exact,points", [(4, True, 4), (16, True, 16), (4, False, 1)])
def test_kept_as_given(epl, exact, points):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_16265_amd import ExaModel
    from paper_2608_16265_amd.batch import ExaBatch
    w = pde(40, seed=1)
    em = ExaModel(w.model, epl=epl, epl_exact=exact)
    assert em.schedule("hess")["points_per_lane"] == points
    x, y = dev(w.x), dev(w.y)
    hess = torch.empty(em.nnzh, dtype=torch.float64, device="cuda:0")
    em.evaluate(x, y, 0.7, hess=hess)
    assert em.eval_schedule(("hess",))["points_per_lane"] == points
    b = ExaBatch([em], autotune=False, epl=epl, epl_exact=exact)
    out = torch.empty_like(hess)
    b.evaluate(x, y, 0.7, hess=out)
    assert b.schedule(("hess",))["points_per_lane"] == points
    assert torch.equal(out, hess)
    b.close()


@pytest.mark.parametrize("given,flag,points", [(4, 0, 4), (4, 1, 1), (0, 0, 1)])
def test_options_record(given, flag, points, monkeypatch):
    """The C options: a nonzero epl is kept unless epl_most is set; zero
    leaves the choice to the library."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_16265_amd import ExaModel, model as binding

    def options(*a):
        o = binding._lib.Options(*a)
        o.epl, o.epl_most = given, flag
        return o
    monkeypatch.setattr(binding, "Options", options)
    assert ExaModel(pde(40, seed=1).model).schedule("hess")["points_per_lane"] == points
