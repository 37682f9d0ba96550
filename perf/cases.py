"""What the performance of this evaluator is measured on.

A case is one thing a solver's program does at every iterate, through the
package's public entry points: every callback of a point (``ExaModel.bind``),
the set an interior-point method asks for, the products a matrix-free method
asks for, the values of a KKT matrix in compressed columns, the Lagrangian
gradient and H v of an augmented-Lagrangian method, a batch of uneven
instances, and the parameter adjoint of a batch through torch.autograd.

The models are the synthetic families of ``exa_modeling.generators`` at the
sizes of the benchmark, its ladders and the tests.  They are stated here as
plain data (:class:`Form`): variable blocks, data sets and patterns whose
expressions are functions that accept both the modeling package's expressions
(to build the model) and torch tensors (to compute exact values).
"""
import math
import os
import tempfile

import numpy as np
import torch

# ------------------------------------------------------------------ the cases

# every callback of a point in one bound call / an interior-point iterate
ALL = "f,g,c,jac,hess,jv,jtw,hv"
IPM = "f,g,c,jac,hess"


def listed():
    return [
        # the smallest call a solver makes in a loop: a 118-bus network, every
        # callback, default options; launches and latency are all it costs
        dict(name="all_acopf_118", family="acopf", size=118, call="bind", outs=ALL, autotune=False),
        # an interior-point iterate of a mid-size network, tuned as a solver's
        # long loop would
        dict(name="ipm_acopf_1354", family="acopf", size=1354, call="bind", outs=IPM, autotune=True),
        # the 10,000-bus model of the benchmark: every callback of an iterate
        dict(name="all_acopf_10000", family="acopf", size=10000, call="bind", outs=ALL, autotune=True),
        # assembling a KKT system: coordinate values, then compressed columns
        dict(name="kkt_acopf_10000", family="acopf", size=10000, call="kkt", outs="", autotune=False),
        # the largest network of the ladder, matrix-free: J v, J^T w, H v
        dict(name="products_acopf_78484", family="acopf", size=78484, call="products", outs="", autotune=True),
        # the grid model of the benchmark: every callback of an iterate
        dict(name="all_pde_1000", family="pde", size=1000, call="bind", outs=ALL, autotune=True),
        # an odd grid, matrix-free, default options
        dict(name="products_pde_517", family="pde", size=517, call="products", outs="", autotune=False),
        # a long trajectory with one variable (the step) shared by every point
        dict(name="all_goddard_1000000", family="goddard", size=1000000, call="bind", outs=ALL, autotune=True),
        # the largest two-stage model of the ladder: Lagrangian gradient and
        # H v, every root variable shared by a quarter of the scenario rows
        dict(name="lag_two_stage_65536", family="two_stage", size=65536, call="lag_hprod", outs="", autotune=True),
        # Newton-CG on the unconstrained problem: f, the gradient, H v
        dict(name="newton_rosenbrock_200000", family="rosenbrock", size=200000, call="newton", outs="", autotune=False),
        # uneven networks of 500 to 20,000 buses, every callback of all of them
        dict(name="all_batch_64", family="batch", size=64, lo=500, hi=20000, call="batch", outs=ALL, autotune=True),
        # differentiating the Lagrangian gradient of a batch with respect to
        # the parameters (branch data among them): forward and backward
        dict(name="theta_batch_32", family="batch", size=32, lo=1000, hi=4000, call="theta", outs="", autotune=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["acopf", "acopf", "pde", "goddard", "two_stage", "rosenbrock", "batch"])
    tuned = rng.random() < 0.5
    if family == "batch":
        lo = _log_int(rng, 100, 2000)
        return dict(family=family, size=rng.randint(3, 48), lo=lo, hi=_log_int(rng, 2 * lo, 10 * lo),
                    call=rng.choice(["batch", "theta"]), outs=ALL, autotune=tuned)
    if family == "rosenbrock":
        return dict(family=family, size=_log_int(rng, 20, 1000000), call="newton", outs="", autotune=tuned)
    lo, hi = dict(acopf=(30, 78484), pde=(10, 1000), goddard=(20, 1000000), two_stage=(16, 65536))[family]
    call = rng.choice(["bind", "bind", "kkt", "products", "lag_hprod"])
    if call == "kkt":  # the compressed form is analysed on the host: a quarter of the largest sizes
        hi = hi // 4 if family != "pde" else hi // 2
    return dict(family=family, size=_log_int(rng, lo, hi), call=call, outs=rng.choice([ALL, IPM]), autotune=tuned)


# ----------------------------------------------------------- models as plain data


class Pat:
    """One pattern: refs are its distinct variable references in the order of
    the Jacobian's slots, each (block, index column or None, offset); pairs
    the Hessian's slots (positions in refs); fn(F, r, p, d) its expression
    over references, parameters and data values, F giving sin, cos, exp."""

    def __init__(self, kind, ds, fn, refs=(), pars=(), cols=(), pairs=(), target=None, row=None):
        self.kind, self.ds, self.fn = kind, ds, fn
        self.refs, self.pars, self.cols, self.pairs = refs, pars, cols, pairs
        self.target, self.row = target, row


class Form:
    """blocks: variable blocks {name: values}; params {name: values}; sets:
    data sets {name: {column: array}}; pats: patterns in declaration order."""

    def __init__(self, blocks, params, sets, pats, y):
        self.blocks, self.params, self.sets, self.pats = blocks, params, sets, pats
        self.x = np.concatenate(list(blocks.values()))
        self.theta = np.concatenate(list(params.values())) if params else np.zeros(0)
        self.y = y
        self.start, at = {}, 0
        for d in (blocks, params):
            at = 0
            for k, v in d.items():
                self.start[k] = at
                at += len(v)
        self.ncon = sum(self.n(p) for p in pats if p.kind == "con")

    def n(self, p):
        return len(next(iter(self.sets[p.ds].values())))

    def index(self, p, ref):
        name, col, off = ref
        if col is None:
            return np.full(self.n(p), self.start[name] + off, dtype=np.int64)
        return self.sets[p.ds][col].astype(np.int64) + (self.start[name] + off)


FLOW_PAIRS = ((1, 1), (1, 2), (3, 3), (4, 4), (3, 4), (1, 3), (1, 4), (2, 3), (2, 4))


def acopf(rng, nb, branch_params=False, scale_loads=False):
    """AC power flow in polar form: a ring plus random chords (0.35 per bus),
    a generator at every fifth bus."""
    nc, ng = (35 * nb + 99) // 100, (nb + 2) // 5
    a, b = rng.integers(0, nb, (2, 3 * nc + 64))
    lo, hi = np.minimum(a, b), np.maximum(a, b)
    keep = (lo != hi) & (hi - lo != 1) & ~((lo == 0) & (hi == nb - 1))
    _, first = np.unique(lo * nb + hi, return_index=True)
    first = np.sort(first[keep[first]])[:nc]
    fr = np.concatenate([np.arange(nb), a[first]])
    to = np.concatenate([(np.arange(nb) + 1) % nb, b[first]])
    nl = fr.size
    gen_bus = rng.choice(nb, ng, replace=False)
    g, bs = rng.uniform(1, 10, nl), rng.uniform(-20, -5, nl)
    blocks = dict(va=rng.uniform(-.3, .3, nb), vm=rng.uniform(.9, 1.1, nb), pg=rng.uniform(0, 2, ng),
                  qg=rng.uniform(-1, 1, ng), p=rng.uniform(-1, 1, 2 * nl), q=rng.uniform(-1, 1, 2 * nl))
    load = rng.uniform(0, 1, (2, nb)) * (rng.uniform(.9, 1.1, nb) if scale_loads else 1.0)
    params = dict(pd=load[0], qd=load[1], c1=rng.uniform(10, 40, ng), c2=rng.uniform(.01, .1, ng))
    sets = dict(gens=dict(i=np.arange(ng), bus=gen_bus, c0=rng.uniform(0, 1, ng)),
                br=dict(l=np.arange(nl), f=fr, t=to, g=g, b=bs), buses=dict(b=np.arange(nb)),
                arcs=dict(a=np.arange(2 * nl), bus=np.concatenate([fr, to])))
    bp = dict(pars=(("gpar", "l", 0), ("bpar", "l", 0))) if branch_params else dict(cols=("g", "b"))
    if branch_params:
        params.update(gpar=g, bpar=bs)

    def flow_p(F, r, p, d):
        (pi, vi, vj, ai, aj), (G, B) = r, p or d
        return pi - (G * vi ** 2 - vi * vj * (G * F.cos(ai - aj) + B * F.sin(ai - aj)))

    def flow_q(F, r, p, d):
        (qi, vi, vj, ai, aj), (G, B) = r, p or d
        return qi - (-B * vi ** 2 - vi * vj * (G * F.sin(ai - aj) - B * F.cos(ai - aj)))

    vf, vt, af, at = ("vm", "f", 0), ("vm", "t", 0), ("va", "f", 0), ("va", "t", 0)
    flow = dict(pairs=FLOW_PAIRS, **bp)
    square = dict(pairs=((0, 0), (1, 1)))

    def limit(F, r, p, d):
        return r[0] ** 2 + r[1] ** 2

    pats = [
        Pat("obj", "gens", lambda F, r, p, d: p[0] * r[0] ** 2 + p[1] * r[0] + d[0], (("pg", "i", 0),),
            (("c2", "i", 0), ("c1", "i", 0)), ("c0",), ((0, 0),)),
        Pat("con", "br", flow_p, (("p", "l", 0), vf, vt, af, at), **flow),
        Pat("con", "br", flow_q, (("q", "l", 0), vf, vt, af, at), **flow),
        Pat("con", "br", flow_p, (("p", "l", nl), vt, vf, at, af), **flow),
        Pat("con", "br", flow_q, (("q", "l", nl), vt, vf, at, af), **flow),
        Pat("con", "buses", lambda F, r, p, d: p[0], (), (("pd", "b", 0),)),
        Pat("con", "buses", lambda F, r, p, d: p[0], (), (("qd", "b", 0),)),
        Pat("aug", "gens", lambda F, r, p, d: -r[0], (("pg", "i", 0),), target=5, row="bus"),
        Pat("aug", "gens", lambda F, r, p, d: -r[0], (("qg", "i", 0),), target=6, row="bus"),
        Pat("aug", "arcs", lambda F, r, p, d: r[0], (("p", "a", 0),), target=5, row="bus"),
        Pat("aug", "arcs", lambda F, r, p, d: r[0], (("q", "a", 0),), target=6, row="bus"),
        Pat("con", "br", limit, (("p", "l", 0), ("q", "l", 0)), **square),
        Pat("con", "br", limit, (("p", "l", nl), ("q", "l", nl)), **square),
    ]
    return Form(blocks, params, sets, pats, rng.standard_normal(6 * nl + 2 * nb))


def pde(rng, n):
    """Distributed control of -Laplace(u) + exp(u) = f on an n x n grid."""
    N, s = n * n, np.arange(n) / (n - 1)
    ut = np.outer(np.sin(math.pi * s), np.sin(math.pi * s)).reshape(-1)
    inner = np.arange(N).reshape(n, n)[1:-1, 1:-1].reshape(-1)
    ih2 = float((n - 1) ** 2)

    def row(F, r, p, d):
        c, w, e, nn, ss, f = r
        return (4 * c - w - e - nn - ss) * ih2 + F.exp(c) - f

    refs = (("u", "c", 0), ("u", "c", -n), ("u", "c", n), ("u", "c", 1), ("u", "c", -1), ("f", "c", 0))
    pats = [Pat("obj", "pts", lambda F, r, p, d: 0.5 * (r[0] - d[0]) ** 2, (("u", "c", 0),), (), ("ut",), ((0, 0),)),
            Pat("obj", "pts", lambda F, r, p, d: 1e-4 * r[0] ** 2, (("f", "c", 0),), pairs=((0, 0),)),
            Pat("con", "inn", row, refs, pairs=((0, 0),))]
    blocks = dict(u=ut + 0.1 * rng.standard_normal(N), f=rng.uniform(0, 10, N))
    return Form(blocks, {}, dict(pts=dict(c=np.arange(N), ut=ut), inn=dict(c=inner)), pats,
                rng.standard_normal(inner.size))


def goddard(rng, T):
    """The Goddard rocket over T trapezoidal steps; the step dt is one
    variable of every row."""
    hc, Dc, ce, mf, thrust = 500.0, 310.0, 0.5, 0.6, 3.5

    def drag(F, h, v):
        return Dc * v ** 2 * F.exp(-hc * (h - 1.0) / 1.0)

    def alt(F, r, p, d):
        h, hp, dt, v, vp = r
        return h - hp - 0.5 * dt * (v + vp)

    def vel(F, r, p, d):
        v, vp, dt, tau, h, m, taup, hp, mp = r
        return v - vp - 0.5 * dt * ((tau - drag(F, h, v)) / m - (1.0 / h) ** 2
                                    + (taup - drag(F, hp, vp)) / mp - (1.0 / hp) ** 2)

    def mass(F, r, p, d):
        m, mp, dt, tau, taup = r
        return m - mp + 0.5 * dt / ce * (tau + taup)

    def now(b):
        return (b, "t", 0)

    def before(b):
        return (b, "t", -1)

    dt = ("dt", None, 0)
    dyn = ((2, 3), (2, 4))
    vel_pairs = ((0, 0), (4, 4), (0, 4), (5, 5), (3, 5), (0, 5), (4, 5), (1, 1), (7, 7), (1, 7), (8, 8), (6, 8),
                 (1, 8), (7, 8), (2, 3), (2, 0), (2, 4), (2, 5), (2, 6), (2, 1), (2, 7), (2, 8))
    pats = [
        Pat("con", "steps", alt, (now("h"), before("h"), dt, now("v"), before("v")), pairs=dyn),
        Pat("con", "steps", vel, (now("v"), before("v"), dt, now("tau"), now("h"), now("m"), before("tau"),
                                  before("h"), before("m")), pairs=vel_pairs),
        Pat("con", "steps", mass, (now("m"), before("m"), dt, now("tau"), before("tau")), pairs=dyn),
        Pat("con", "one", lambda F, r, p, d: r[0] - 1.0, (("h", None, 0),)),
        Pat("con", "one", lambda F, r, p, d: r[0] - 0.0, (("v", None, 0),)),
        Pat("con", "one", lambda F, r, p, d: r[0] - 1.0, (("m", None, 0),)),
        Pat("con", "one", lambda F, r, p, d: r[0] - p[0], (("m", None, T),), (("mf", None, 0),)),
        Pat("obj", "one", lambda F, r, p, d: -r[0], (("h", None, T),)),
    ]
    s = np.arange(T + 1) / T
    blocks = dict(h=1.0 + 0.01 * rng.uniform(0, 1, T + 1), v=s * (1 - s) + 0.01 * rng.standard_normal(T + 1),
                  m=1.0 + (mf - 1.0) * s + 0.004 * rng.uniform(0, 1, T + 1),
                  tau=thrust / 2 + 0.1 * rng.standard_normal(T + 1), dt=np.full(1, 1.0 / T))
    return Form(blocks, dict(mf=np.full(1, mf)), dict(steps=dict(t=np.arange(1, T + 1)), one=dict(k=np.zeros(1, int))),
                pats, rng.standard_normal(3 * T + 4))


def two_stage(rng, S, n0=8, nz=32):
    """A two-stage stochastic program: n0 root variables shared by S
    scenarios of nz variables each."""
    j, s = np.tile(np.arange(nz), S), np.repeat(np.arange(S), nz)
    sets = dict(root=dict(i=np.arange(n0), i1=(np.arange(n0) + 1) % n0),
                sc=dict(k=j + nz * s, xi=j % n0, xn=(j + 1) % n0, scen=s + 1, p=np.full(nz * S, 1.0 / S)))
    z, d = ("z", "k", 0), ("d", "k", 0)
    pats = [
        Pat("obj", "root", lambda F, r, p, d: 0.5 * r[0] ** 2, (("x", "i", 0),), pairs=((0, 0),)),
        Pat("con", "root", lambda F, r, p, d: r[0] * r[1], (("x", "i", 0), ("x", "i1", 0)), pairs=((0, 1),)),
        Pat("obj", "sc", lambda F, r, p, d: d[0] * (r[0] - p[0]) ** 2, (z,), (d,), ("p",), ((0, 0),)),
        Pat("con", "sc", lambda F, r, p, d: r[0] * F.exp(r[1]) - r[2] ** 2 + p[0] * r[0],
            (z, ("x", "xi", 0), ("x", "xn", 0)), (d,), (), ((1, 1), (0, 1), (2, 2))),
    ]
    dd = rng.standard_normal(nz * S)
    blocks = dict(x=rng.uniform(-1, 1, n0), z=rng.standard_normal(nz * S))
    return Form(blocks, dict(d=dd), sets, pats, rng.standard_normal(n0 + nz * S))


def rosenbrock(rng, N):
    """The extended Rosenbrock function of N variables."""
    pats = [Pat("obj", "d", lambda F, r, p, d: 100 * (r[0] ** 2 - r[1]) ** 2 + (r[0] - 1) ** 2,
                (("x", "i", -1), ("x", "i", 0)), pairs=((0, 0), (1, 1), (0, 1)))]
    return Form(dict(x=rng.uniform(-2, 2, N)), {}, dict(d=dict(i=np.arange(1, N))), pats, np.zeros(0))


FAMILIES = dict(acopf=acopf, pde=pde, goddard=goddard, two_stage=two_stage, rosenbrock=rosenbrock)


def forms(case, seed):
    """The case's model (or a batch's models) and the vectors v and w."""
    rng = np.random.Generator(np.random.PCG64(seed))
    if case["family"] == "batch":
        # bus counts spread log-uniformly over [lo, hi], in a mixed order that
        # the case fixes
        spread = np.random.Generator(np.random.PCG64(case["size"]))
        sizes = np.exp(spread.uniform(math.log(case["lo"]), math.log(case["hi"]), case["size"])).round().astype(int)
        fs = [acopf(rng, int(nb), case["call"] == "theta", True) for nb in sizes]
    else:
        fs = [FAMILIES[case["family"]](rng, case["size"])]
    v = rng.standard_normal(sum(f.x.size for f in fs))
    w = rng.standard_normal(sum(f.ncon for f in fs))
    return fs, v, w


# ------------------------------------------------------------- the user's program


class _Ops:
    """sin, cos, exp of the modeling package's expressions."""

    def __init__(self):
        from exa_modeling import ir
        self.sin, self.cos, self.exp = ir.sin, ir.cos, ir.exp


# a program that comes back keeps its compiled kernels on disk
CACHE = os.path.join(tempfile.gettempdir(), "exa_cases_cache_%d" % os.getuid())


def build(form, autotune):
    """The form as a model of this package."""
    from exa_modeling import DataSet, Model
    from paper_2608_16265_amd import ExaModel
    m, F = Model("case"), _Ops()
    blk = {k: m.add_var(len(v), name=k) for k, v in form.blocks.items()}
    par = {k: m.add_par(v, k) for k, v in form.params.items()}
    sets = {k: DataSet(len(next(iter(c.values()))), **c) for k, c in form.sets.items()}

    def ref(table, ds, name, col, off):
        return table[name][off if col is None else getattr(ds, col) + off]

    for p in form.pats:
        ds = sets[p.ds]
        e = p.fn(F, [ref(blk, ds, *r) for r in p.refs], [ref(par, ds, *r) for r in p.pars],
                 [getattr(ds, c) for c in p.cols])
        if p.kind == "obj":
            m.add_obj(e, ds)
        elif p.kind == "con":
            m.add_con(e, ds)
        else:
            m.add_con_aug(p.target, getattr(ds, p.row), e, ds)
    os.makedirs(CACHE, exist_ok=True)
    return ExaModel(m, autotune=autotune, cache_dir=CACHE)


SIZES = dict(f="B", g="x", c="y", jac="jac", hess="hess", jv="y", jtw="x", hv="x")


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0")


def _empty(n):
    return torch.empty(n, dtype=torch.float64, device="cuda:0")


def prepare(case, seed):
    from paper_2608_16265_amd.batch import ExaBatch
    fs, v, w = forms(case, seed)
    x, y = _dev(np.concatenate([f.x for f in fs])), _dev(np.concatenate([f.y for f in fs]))
    v, w, sigma = _dev(v), _dev(w), 0.75
    models = [build(f, case["autotune"]) for f in fs]
    if case["family"] == "batch":
        handle = ExaBatch(models, autotune=case["autotune"])
        call, out = _batch(case, handle, fs, x, y, sigma, v, w)
    else:
        handle = models[0]
        call, out = _single(case, handle, x, y, sigma, v, w)
    if case["autotune"]:
        call()  # the solver's first iterate tunes the schedules
    return dict(call=call, out=out, handle=handle)  # a bound call does not keep its batch alive


def _batch(case, b, fs, x, y, sigma, v, w):
    from paper_2608_16265_amd.adjoint import batch_lagrangian_gradient
    if case["call"] == "batch":
        out = {k: b.empty(SIZES[k]) for k in case["outs"].split(",")}
        return b.bind(x, y, sigma, v, w, **out), out
    theta, out = _dev(np.concatenate([f.theta for f in fs])), {}

    def call():
        t = theta.detach().requires_grad_(True)
        lag = batch_lagrangian_gradient(t, b, x, y, sigma)
        lag.backward(v)
        out["lag"], out["theta_bar"] = lag.detach(), t.grad
    return call, out


def _single(case, em, x, y, sigma, v, w):
    n = dict(B=1, x=em.nvar, y=em.ncon, jac=em.nnzj, hess=em.nnzh)
    kind = case["call"]
    if kind == "bind":
        out = {k: _empty(n[SIZES[k]]) for k in case["outs"].split(",")}
        return em.bind(x, y, sigma, v, w, **out), out
    if kind == "kkt":
        out = dict(jac=_empty(em.nnzj), hess=_empty(em.nnzh))
        for k in ("jac", "hess"):  # the solver's symbolic factorisation has read the structure
            out[k + "_csc"] = _empty(em.csc_structure(k)[1].size)

        def call():
            em.jac_hess_coord(x, y, sigma, out["jac"], out["hess"])
            em.csc_values("jac", out["jac"], out["jac_csc"])
            em.csc_values("hess", out["hess"], out["hess_csc"])
    elif kind == "products":
        out = dict(jv=_empty(em.ncon), jtw=_empty(em.nvar), hv=_empty(em.nvar))

        def call():
            em.jprod(x, v, out["jv"])
            em.jtprod(x, w, out["jtw"])
            em.hprod(x, y, sigma, v, out["hv"])
    elif kind == "lag_hprod":
        out = dict(lag=_empty(em.nvar), hv=_empty(em.nvar))

        def call():
            em.lag_grad(x, y, sigma, out["lag"])
            em.hprod(x, y, sigma, v, out["hv"])
    else:
        out = dict(f=_empty(1), g=_empty(em.nvar), hv=_empty(em.nvar))

        def call():
            em.obj(x, out["f"])
            em.grad(x, out["g"])
            em.hprod(x, y, sigma, v, out["hv"])
    return call, out


def run(state):
    state["call"]()
    return state["out"]


# ------------------------------------------------------------------- what it takes

CALL_OUTS = dict(kkt=("jac", "hess", "jac_csc", "hess_csc"), products=("jv", "jtw", "hv"), lag_hprod=("lag", "hv"),
                 newton=("f", "g", "hv"), theta=("lag", "theta_bar"))


def outputs_of(case):
    return CALL_OUTS.get(case["call"]) or tuple(case["outs"].split(","))


def work(case):
    """Each input (point, multipliers, directions, parameters, data columns
    that are not the point's own number) read once, each output written once;
    about 4 operations a value and derivative."""
    want = outputs_of(case)
    fs, _, _ = forms(case, 1)
    nbytes = flops = 0
    for f in fs:
        n, m = f.x.size, f.ncon
        nj = sum(f.n(p) * len(p.refs) for p in f.pats if p.kind != "obj")
        nh = sum(f.n(p) * len(p.pairs) for p in f.pats)
        size = dict(f=1, g=n, c=m, jac=nj, hess=nh, jv=m, jtw=n, hv=n, lag=n, theta_bar=f.theta.size,
                    jac_csc=nj, hess_csc=nh)
        used = {(p.ds, c) for p in f.pats for c in p.cols + tuple(r[1] for r in p.refs + p.pars if r[1])}
        used |= {(p.ds, p.row) for p in f.pats if p.row}
        for ds, c in used:
            a = f.sets[ds][c]
            if a.dtype.kind == "f":
                nbytes += 8 * a.size
            elif not np.array_equal(a, np.arange(a.size)):
                nbytes += 4 * a.size
        vectors = n + f.theta.size
        vectors += m if {"hess", "hv", "lag", "theta_bar"} & set(want) else 0
        vectors += n if {"jv", "hv", "theta_bar"} & set(want) else 0
        vectors += m if "jtw" in want else 0
        nbytes += 8 * (vectors + sum(size[k] for k in want))
        flops += 4 * (nj + nh + m + n)
    return dict(bytes=nbytes, flops=flops)


# ----------------------------------------------------------------- exact values


def _grad(t, leaf):
    """d t / d leaf of elementwise t, zeros where t does not depend on it."""
    if not t.requires_grad:
        return torch.zeros_like(leaf)
    g, = torch.autograd.grad(t.sum(), leaf, create_graph=True, allow_unused=True)
    return torch.zeros_like(leaf) if g is None else g


def _exact_form(f, sigma, y, v, w, want):
    """The outputs `want` of one model, from torch's derivatives of each
    pattern at all its data points."""
    x, th = torch.as_tensor(f.x), torch.as_tensor(f.theta)
    y, v, w = (torch.as_tensor(a) for a in (y, v, w))
    second = {"hess", "hess_csc", "hv", "theta_bar"} & set(want)
    z = lambda k: torch.zeros(k, dtype=torch.float64)  # noqa: E731
    o = dict(f=z(1), g=z(x.numel()), c=z(f.ncon), jv=z(f.ncon), jtw=z(x.numel()), hv=z(x.numel()),
             jty=z(x.numel()), theta_bar=z(th.numel()))
    jac, hess, jpos, hpos = [], [], [], []
    rows, at = {}, 0
    for i, p in enumerate(f.pats):
        if p.kind == "con":
            rows[i] = torch.arange(at, at + f.n(p))
            at += f.n(p)
    for i, p in enumerate(f.pats):
        ix = [torch.as_tensor(f.index(p, r)) for r in p.refs]
        ip = [torch.as_tensor(f.index(p, r)) for r in p.pars]
        r = [x[k].requires_grad_(True) for k in ix]
        q = [th[k].requires_grad_(True) for k in ip]
        d = [torch.as_tensor(f.sets[p.ds][c]) for c in p.cols]
        t = p.fn(torch, r, q, d)
        J = [_grad(t, k) for k in r]
        if p.kind == "obj":
            row, wy, ww = None, torch.full((f.n(p),), sigma, dtype=torch.float64), None
            o["f"] += t.detach().sum()
            for k, g in zip(ix, J):
                o["g"].index_add_(0, k, g.detach())
        else:
            row = rows[i] if p.kind == "con" else rows[p.target][torch.as_tensor(f.sets[p.ds][p.row])]
            wy, ww = y[row], w[row]
            o["c"].index_add_(0, row, t.detach())
            for k, g in zip(ix, J):
                o["jv"].index_add_(0, row, g.detach() * v[k])
                o["jtw"].index_add_(0, k, g.detach() * ww)
                o["jty"].index_add_(0, k, g.detach() * wy)
            if J:
                jac.append(torch.stack([g.detach() for g in J], 1).reshape(-1))
                jpos.append((torch.stack([row] * len(J), 1).reshape(-1), torch.stack(ix, 1).reshape(-1)))
        if not second:
            continue
        H = [(_grad(J[a], r[b])).detach() * wy for a, b in p.pairs]
        for (a, b), h in zip(p.pairs, H):
            o["hv"].index_add_(0, ix[a], h * v[ix[b]])
            if a != b:
                o["hv"].index_add_(0, ix[b], h * v[ix[a]])
        if H:
            hess.append(torch.stack(H, 1).reshape(-1))
            pa = torch.stack([torch.maximum(ix[a], ix[b]) for a, b in p.pairs], 1).reshape(-1)
            pb = torch.stack([torch.minimum(ix[a], ix[b]) for a, b in p.pairs], 1).reshape(-1)
            hpos.append((pa, pb))
        if "theta_bar" in want:
            for a, k in enumerate(ix):
                for s, kp in enumerate(ip):
                    o["theta_bar"].index_add_(0, kp, _grad(J[a], q[s]).detach() * wy * v[k])
    o["jac"] = torch.cat(jac) if jac else z(0)
    o["hess"] = torch.cat(hess) if hess else z(0)
    o["lag"] = sigma * o["g"] + o["jty"]
    for k, pos, nrow in (("jac", jpos, max(f.ncon, 1)), ("hess", hpos, x.numel())):
        if k + "_csc" in want:  # columns ascending, rows ascending in a column
            key = torch.cat([c * nrow + r for r, c in pos]) if pos else torch.zeros(0, dtype=torch.int64)
            cells, inv = torch.unique(key, return_inverse=True)
            o[k + "_csc"] = z(cells.numel()).index_add_(0, inv, o[k])
    return {k: o[k].detach() for k in want}


def exact(case, seed):
    fs, v, w = forms(case, seed)
    want, got, nx, ny = outputs_of(case), [], 0, 0
    for f in fs:
        got.append(_exact_form(f, 0.75, f.y, v[nx:nx + f.x.size], w[ny:ny + f.ncon], want))
        nx, ny = nx + f.x.size, ny + f.ncon
    return {k: torch.cat([g[k] for g in got]) for k in want}
