"""A chain beside data sets of two far points (the first and last variables):
pulled behind a branch, or too many tables and left to the reduction."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from exa_modeling.generators import Workload
from test_parity_gpu import check_all
from test_plans_cpu import edges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(64, 1), (200, 2), (200, 25), (5000, 3)])
def test_edges(n, k, tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_16265_amd import ExaModel
    rng = np.random.default_rng(n + k)
    m = edges(n, k)
    w = Workload(m, rng.uniform(-1, 1, m.nvar), rng.standard_normal(m.ncon), 0.7)
    check_all(w, ExaModel(m, cache_dir=str(tmp_path)), tag=f"edges {n} {k}: ")
