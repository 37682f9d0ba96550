"""exa_eval_timing counts the reduction launches there are: none where the
evaluation launch finishes every sum."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from exa_modeling.generators import acopf, goddard
from parity_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("make,reduced", [(lambda: acopf(60, 1), 0), (lambda: goddard(300, 1), 3)], ids=["acopf", "goddard"])
def test_launches_recorded(make, reduced):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_16265_amd import ExaModel
    w = make()
    em = ExaModel(w.model)
    x, u = dev(w.x), dev(np.random.default_rng(1).standard_normal(em.ncon))
    call = em.bind(x, None, 1.0, None, u, jtw=torch.empty(em.nvar, dtype=torch.float64, device="cuda:0"))
    call()
    em.eval_timing(True)
    for _ in range(3):
        call()
    t = em.eval_timing_read()
    em.eval_timing(False)
    assert (t["calls"], t["reduce_calls"]) == (3, reduced), t
    b = em.eval_bytes(("jtprod",))
    assert (b["reduce_read"] + b["reduce_write"] > 0) == (reduced > 0), b
