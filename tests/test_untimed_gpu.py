"""Schedules nobody has timed: the options' points per lane, halved while a
launch has fewer than 768 workgroups; the values are the same."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from exa_modeling.generators import pde
from parity_util import dev, host

pytestmark = pytest.mark.gpu


# from one workgroup to far more than 768, and numbers that halve to 1 unevenly
@pytest.mark.parametrize("n,epl", [(3, 4), (250, 4), (260, 3), (330, 4), (470, 4), (700, 4), (700, 16), (700, 1)])
def test_points_per_lane(n, epl):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_16265_amd import ExaModel
    w = pde(n, seed=1)
    em = ExaModel(w.model, epl=epl)
    s = em.schedule("hess")
    pats = [em.pattern_info(p) for p in range(len(w.model.patterns))]
    sizes = [p["ndata"] for p in pats if p["o2step"] > 0]
    tiles = lambda e: sum(-(-k // (256 * e)) for k in sizes)
    want = epl
    while want > 1 and tiles(want) < 768:
        want //= 2
    assert (s["block"], s["points_per_lane"], s["tiles"]) == (256, want, tiles(want)), s
    x, y = dev(w.x), dev(w.y)
    ref = ExaModel(w.model, block=64, epl=1)
    rng = np.random.default_rng(2)
    v, u = dev(rng.standard_normal(em.nvar)), dev(rng.standard_normal(em.ncon))
    assert torch.equal(em.hess_coord(x, y, 0.7), ref.hess_coord(x, y, 0.7))
    for cb in ("c", "jac", "hess", "jv", "jtw", "hv"):
        size = dict(c=em.ncon, jac=em.nnzj, hess=em.nnzh, jv=em.ncon, jtw=em.nvar, hv=em.nvar)
        a, b = (torch.full((size[cb],), float("nan"), dtype=torch.float64, device="cuda:0") for _ in range(2))
        em.evaluate(x, y, 0.7, v, u, **{cb: a})
        ref.evaluate(x, y, 0.7, v, u, **{cb: b})
        assert torch.equal(a, b), cb
