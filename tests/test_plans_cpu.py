"""Which sums the evaluation units take over, read from the generated source
of host-only models ("sums finished by units: ..."): values alone cannot tell,
since the reduction gives the same ones."""
import re

import numpy as np
import pytest

from exa_modeling import DataSet, Model, sin
from paper_2608_16265_amd import ExaModel

JT, HV, GRAD = range(3)


def plan(m):
    """Per sum the text of its units (empty: every sum goes through the map)."""
    line = ExaModel(m, host_only=True).generated_source().split("// sums finished by units: ")[1].split("\n")[0]
    parts = re.split(r"[012][+-]L?", line)[1:]
    assert len(parts) == 3, line
    return parts


def sources(text):
    """(data set, reference, how, sparse) of every pulled source; how 0: counted
    from the variable, 1: through an inverse table."""
    return [(int(g), int(r), int(h), bool(s))
            for g, r, h, s in re.findall(r"(\d+)\.(\d+)\.(\d+)\.-?\d+\.-?\d+(s?),", text)]


def edges(n, k):
    """A chain over n variables beside k data sets of two points each."""
    m = Model("edges")
    x = m.add_var(n)
    d = DataSet(n - 1, i=np.arange(n - 1))
    m.add_con(sin(x[d.i] * x[d.i + 1]), d)
    for j in range(k):
        e = DataSet(2, i=np.array([j, n - 1 - j]))
        m.add_con(sin(x[e.i]), e)
    return m


@pytest.mark.parametrize("k,pulled", [(1, True), (4, True), (5, False)])
def test_few_far_points_are_pulled_behind_a_branch(k, pulled):
    for text in plan(edges(10_000, k))[:2]:
        assert len(sources(text)) == (k if pulled else 0), text
        assert all(s[2:] == (1, True) for s in sources(text)), text


def test_tables_for_a_few_points_are_bounded():
    """25 tables of 100,000 entries for 50 points: their variables, and the
    chain they lie on, stay in the map; the code and the footprint stay small."""
    few, many = edges(100_000, 2), edges(100_000, 25)
    assert not any(sources(t) for t in plan(many))
    a, b = (ExaModel(m, host_only=True) for m in (few, many))
    assert len(b.generated_source()) < 8 * len(a.generated_source())
    assert b.device_bytes() < 1.2 * a.device_bytes()


def test_gaps_that_pay_keep_their_table():
    n = 1000
    m = Model("gaps")
    x = m.add_var(4 * n)
    d = DataSet(n, i=np.arange(n) * 3)
    m.add_con(sin(x[d.i]), d)
    assert sources(plan(m)[JT]) == [(0, 0, 1, True)]


def units(text):
    return re.findall(r"U(\d+)S(\d+)", text)


def lists(text):
    """Data sets whose contributions are pulled through incidence lists."""
    return [int(g) for g in re.findall(r"l(\d+)\.\d+:", text)]


def chain_shifts(text):
    """Lane shifts of every chain."""
    chains = re.findall(r"c\d+:((?:\d+/\d+,)+)b", text)
    return [[int(r.split("/")[0]) for r in c.split(",")[:-1]] for c in chains]


def test_list_length_limit():
    from test_incidence_gpu import network
    for kind, want in (("hub", True), ("long", False)):  # 64 and 65 entries
        text = plan(network(kind, 100, 300).model)
        assert bool(lists(text[JT])) == want and bool(lists(text[HV])) == want, text


def test_lists_in_the_points_order_or_small():
    from test_incidence_gpu import network
    for kind, nb, nl, want in (("ring", 60000, 80000, True), ("plain", 60000, 80000, False), ("plain", 1000, 1400, True)):
        assert bool(lists(plan(network(kind, nb, nl).model)[JT])) == want, (kind, nb)


def shifted(n, s):
    m = Model("shifted")
    x = m.add_var(n + s)
    d = DataSet(n, i=np.arange(n))
    m.add_con(sin(x[d.i] * x[d.i + s]), d)
    return m


def test_chain_span_limit():
    assert chain_shifts(plan(shifted(500, 8))[JT]) == [[0, 8]]
    assert not chain_shifts(plan(shifted(500, 9))[JT])  # overlapping, too far for a shift: a unit over variables
    assert [s for s in sources(plan(shifted(500, 9))[JT]) if s[2] == 0]


@pytest.mark.parametrize("period", [0, 1, 2, 4, 32, 64])
def test_shared_references(period):
    """Partial sums for a literal index (0) and a period of 2 to 32 points;
    a period of 1 (every point the same entry) repeats with 2; one of 64 is
    left to lists or the map."""
    n = 640
    m = Model("shared")
    x, z = m.add_var(n), m.add_var(64)
    d = DataSet(n, i=np.arange(n), s=np.arange(n) % max(1, period))
    m.add_con(x[d.i] * sin(z[3] if period == 0 else z[d.s]), d)
    got = re.findall(r"s(\d+)/(\d+),", plan(m)[JT])
    want = {0: [("1", "1")], 1: [("1", "2")], 64: []}.get(period, [("1", str(period))])
    assert got == want, plan(m)[JT]


def test_gaps_take_a_table():
    from test_sums_gpu import forms
    assert [s for s in sources(plan(forms("gaps", 513).model)[JT]) if s[2] == 1]
    assert not [s for s in sources(plan(forms("plain", 513).model)[JT]) if s[2] == 1]


def test_one_read_ahead_loop_per_kernel():
    """Kernels that may read ahead hold the loop once, not once per callback:
    copies cost compile time on every model."""
    src = ExaModel(edges(100, 1), host_only=True).generated_source()
    body = src[src.index("exa_ahead(const double* x"):]
    kernels = re.split(r'extern "C" __global__', body)[1:]
    calls = [k.count("exa_ahead(") for k in kernels]
    assert max(calls) == 1 and sum(calls) == 6, calls
