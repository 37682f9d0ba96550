"""A bound batch call owns its batch: it works when nothing else holds the batch
any more, and refuses once the batch is closed."""
import gc

import pytest

torch = pytest.importorskip("torch")

from exa_modeling.generators import acopf
from parity_util import dev

pytestmark = pytest.mark.gpu


def test_bound_call_keeps_its_batch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_16265_amd import ExaError, ExaModel
    from paper_2608_16265_amd.batch import ExaBatch
    w = acopf(40, 2)
    em = ExaModel(w.model)
    x = dev(w.x)
    c = torch.full((em.ncon,), float("nan"), dtype=torch.float64, device="cuda:0")
    call = ExaBatch([em], autotune=False).bind(x, c=c)  # the batch itself is dropped here
    gc.collect()
    for _ in range(4):
        call()
    assert torch.equal(c, em.cons(x))
    b = ExaBatch([em], autotune=False)
    call = b.bind(x, c=c)
    call()
    torch.cuda.synchronize()
    b.close()
    with pytest.raises(ExaError, match="null batch"):
        call()
