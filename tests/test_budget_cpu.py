"""Footprint estimates and budgets of host-only models: what a model is charged
follows from the tables its plan uses, and budgets that sufficed while every
sum went through a map still do."""
import numpy as np
import pytest

from exa_modeling import DataSet, Model, sin
from exa_modeling.generators import acopf, goddard, pde, rosenbrock, two_stage
from paper_2608_16265_amd import ExaModel


def links(nb, nl, seed=1):
    """Links between random nodes, too many for incidence lists."""
    rng = np.random.default_rng(seed)
    m = Model("links")
    x = m.add_var(nb)
    d = DataSet(nl, f=rng.integers(0, nb, nl), t=rng.integers(0, nb, nl))
    m.add_con(sin(x[d.f] - x[d.t]), d)
    return m


def columns(n, cols):
    """n points over x[i], i = 0 .. n-1, beside columns that nothing uses."""
    m = Model("columns")
    x = m.add_var(n)
    d = DataSet(n, i=np.arange(n), **cols)
    m.add_con(sin(x[d.i]), d)
    return m


# footprints estimated when every sum had a map and no unit a table
BUDGETS = [("acopf 118", lambda: acopf(118, 118).model, 156880), ("acopf 3000", lambda: acopf(3000, 3000).model, 2856424),
           ("pde 66", lambda: pde(66, 1).model, 1431104), ("goddard 1000", lambda: goddard(1000, 1).model, 611732),
           ("two-stage 64", lambda: two_stage(64, seed=1).model, 604168),
           ("rosenbrock 1000", lambda: rosenbrock(1000, 1).model, 176588)]


@pytest.mark.parametrize("make,budget", [b[1:] for b in BUDGETS], ids=[b[0] for b in BUDGETS])
def test_budgets_that_sufficed(make, budget):
    m = make()
    em = ExaModel(m, host_only=True, max_device_bytes=budget)
    assert em.device_bytes() <= budget
    assert ExaModel(m, host_only=True).device_bytes() <= budget  # and with room for every table


def test_column_without_a_table_is_charged_its_bytes():
    """An index column that no sum needs inverted takes 4 bytes a point, in
    whatever order its values are."""
    n = 5000
    base = ExaModel(columns(n, {}), host_only=True).device_bytes()
    for col in (np.arange(n), np.arange(n) * 400000, np.random.default_rng(2).permutation(n)):
        got = ExaModel(columns(n, dict(u=col)), host_only=True).device_bytes()
        assert 0 <= got - base <= 4 * n + 64, (got, base)


def test_what_speed_added_is_given_up_first():
    """Under a budget that only the options' tiles fit, launches keep them."""
    m = links(100_000, 150_000)
    full = ExaModel(m, host_only=True).device_bytes()
    less = ExaModel(m, host_only=True, max_device_bytes=full - 1).device_bytes()
    assert less < full
    with pytest.raises(Exception, match="budget"):
        ExaModel(m, host_only=True, max_device_bytes=less // 2)
