"""exa_lag_grad and exa_eval of the gradient and J^T w: the first eager call of
either is enough for the other to be captured."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from exa_modeling.generators import acopf, rosenbrock
from parity_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tuned", [False, True])
@pytest.mark.parametrize("make", [lambda: acopf(60, 3), lambda: rosenbrock(300, 3)], ids=["acopf", "rosenbrock"])
def test_the_other_is_ready(make, tuned):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_16265_amd import ExaModel
    w = make()
    ref = ExaModel(w.model)
    x, y = dev(w.x), dev(np.random.default_rng(1).standard_normal(ref.ncon))
    want = dict(g=ref.grad(x), jtw=ref.jtprod(x, y), lag=ref.lag_grad(x, y, 0.6))
    nan = lambda: torch.full((ref.nvar,), float("nan"), dtype=torch.float64, device="cuda:0")  # noqa: E731
    for eager, captured in (("eval", "lag"), ("lag", "eval")):
        em = ExaModel(w.model, autotune=tuned)
        g, jtw, lag = nan(), nan(), nan()
        call = dict(eval=em.bind(x, None, 0.6, None, y, g=g, jtw=jtw), lag=lambda: em.lag_grad(x, y, 0.6, lag))
        call[eager]()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call[captured]()
        for _ in range(3):
            for t in (g, jtw, lag):
                t.fill_(float("nan"))
            call[eager]()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(g, want["g"]) and torch.equal(jtw, want["jtw"]) and torch.equal(lag, want["lag"])
