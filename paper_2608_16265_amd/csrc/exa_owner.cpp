// Which variables' sums (J^T w, H v, gradient) the evaluation units finish
// themselves, and the reduction maps of the others (see OwnPlan).
#include <algorithm>
#include <map>
#include <sstream>

#include "exa_internal.h"

namespace exa {

namespace {

// A unit over variables evaluates every contribution anew, so it only pays
// while that is little work; a host unit's pulled contributions come on top
// of the host's own sweep.  Limits in tree nodes of the patterns pulled from.
// (The grid model's J^T w pulls 5 references of a 21-node row: 5 x 21 = 105
// nodes, of which the constant derivatives cost nothing once emitted.)
constexpr int kPullNodes = 160, kHostPullNodes = 64;
// A unit that pulls through incidence lists evaluates a point once per slot
// (a branch once for each end); longest list (a lane adds it from LDS, and it
// has to fit the smallest tile), and limit of the points' nodes.
constexpr int kListLength = 64, kListNodes = 400, kListSlots = 4;
// A list's points are gathered, line by line, where the data set's own unit
// streams them and leaves one number per reference to gather.  That pays while
// the points' data fits in an XCD's L2 beside the rest (kListBytes), or while
// the lists follow the points' order: 256 entries in turn touch at most
// kListSpread times the lines that 256 points in a row would.  Measured, map /
// lists: networks of nodes linked at random J^T w 20,000 nodes and 30,000
// links (1 MB) 7.8 / 5.2 us, H v 9.5 / 5.5; 100,000 and 150,000 (5 MB, spread
// 16) 17.0 / 17.5 and 19 / 25; 500,000 and 700,000 75 / 146 and 125 / 194; a
// ring of 78,484 buses with chords (spread 5) 18.2 / 13.4 and 16.7 / 12.6.
constexpr int64_t kListBytes = (int64_t)2 << 20;
constexpr int kListSpread = 8;
// Runs per data set, so that one workgroup can add a variable's partial sums.
// Each run is kOwnWaves waves' work (8192 waves at most: more than the chip
// holds), added through LDS: 65,536 scenarios' J^T w 25.8 us with 4096 runs of
// one wave, 23.2 with 2048 of four, H v 31.9 / 30.3; 4096 scenarios 9.3 / 8.1
// and 9.7 / 8.4 (the reduction reads a quarter); a trajectory of 10,000 steps,
// every callback 9.4 / 8.1.  1024 and 4096 runs of four: J^T w 22.7 and 24.5.
constexpr int64_t kMaxRuns = 2048;
// A column with gaps costs the unit that pulls through it one 4-byte table
// entry per variable it spans, in memory and in every launch, however few points
// it has.  A cluster is left to the map when these come to more than the map's own
// pointer per variable and kEntryBytes per contribution.  Measured on a chain
// of two references over 1,000,000 variables beside k data sets of two far
// points each, units / map: J^T w k = 1 8.3 / 15.7 us, 3 12.7 / 15.7, 9
// 24.6 / 15.7 (2 us a table: equal at 4.7), and 25 with every pull evaluated
// in full 252 / 15.7.
constexpr int64_t kEntryBytes = 6;
// Doubles a workgroup holds for its waves' partial sums.
constexpr int kMaxPartials = 2048;

struct Src {
    OwnSrc s;
    int kind = 0;         // 0 usable, 1 shared, 2 other (its variables stay in the map), 3 by incidence lists
    int64_t lo = 0, hi = 0;  // first and last variable
    int nodes = 0;
    bool grad = false;
};

const std::vector<int32_t>& col_of(const Model& M, const Group& G, int c) { return M.pats[G.members[0]].icols[c]; }

bool increasing(const std::vector<int32_t>& c) {
    for (size_t k = 1; k < c.size(); ++k)
        if (c[k] <= c[k - 1]) return false;
    return true;
}

// The smallest period 2, 4, ..., 32 with which the column repeats, or 0.
int period_of(const std::vector<int32_t>& c) {
    for (int P = 2; P <= 32; P *= 2) {
        if ((int64_t)c.size() < 4 * P) return 0;
        bool ok = true;
        for (size_t k = P; k < c.size() && ok; ++k) ok = c[k] == c[k - P];
        if (ok) return P;
    }
    return 0;
}

bool in_sum(const Pattern& P, SumKind s) {
    if (P.ndata == 0) return false;
    if (s == SUM_HV) return !P.hvs.empty();
    return (P.kind == EXA_OBJ) == (s == SUM_GRAD) && P.o1step() > 0;
}

// Group references that patterns of the group contribute to a sum through.
std::vector<int> refs_of(const Model& M, const Group& G, SumKind s) {
    if (s == SUM_HV) return G.hv_refs;
    std::vector<char> hit(G.vrefs.size(), 0);
    for (int p : G.members)
        if (in_sum(M.pats[p], s))
            for (int r : M.pats[p].vg) hit[r] = 1;
    std::vector<int> out;
    for (size_t r = 0; r < hit.size(); ++r)
        if (hit[r]) out.push_back((int)r);
    return out;
}

int nodes_of(const Model& M, const Group& G, SumKind s, int r) {
    int n = 0;
    for (int p : G.members) {
        const Pattern& P = M.pats[p];
        if (in_sum(P, s) && std::find(P.vg.begin(), P.vg.end(), r) != P.vg.end()) n += (int)P.nodes.size();
    }
    return n;
}

Src make_src(const Model& M, int g, int r, SumKind s, const std::vector<std::vector<char>>& inc,
             const std::vector<std::vector<int>>& period) {
    const Group& G = M.groups[g];
    const Pattern& P0 = M.pats[G.members[0]];
    const RefKey& k = G.vrefs[r];
    Src o;
    o.s.group = g;
    o.s.ref = r;
    o.nodes = nodes_of(M, G, s, r);
    if (G.vrefs.size() > EXA_MAX_REFS) {
        o.kind = 2;  // more references than the tables hold
    } else if (k.col < 0) {
        o.kind = G.ndata == 1 ? 0 : 1;
    } else if (P0.affine[k.col]) {
        o.kind = 0;
    } else if (inc[g][k.col]) {
        o.s.how = OWN_INVERSE;
    } else {
        o.kind = period[g][k.col] ? 1 : s == SUM_GRAD ? 2 : 3;
        if (o.kind == 3) o.s.how = OWN_LIST;
    }
    if (G.ndata > 0) {
        if (k.col < 0) {
            o.lo = o.hi = k.off;
        } else if (o.kind == 0) {
            o.lo = P0.icols[k.col].front() + k.off;
            o.hi = P0.icols[k.col].back() + k.off;
        } else if (o.kind == 3) {
            o.lo = G.range[k.col].first + k.off;
            o.hi = G.range[k.col].second + k.off;
        }
    }
    return o;
}

// Variable of an affine source at point 0.
int64_t shift_of(const Src& s) { return s.lo; }

struct Cluster {
    std::vector<Src> src, grad;
    int64_t lo = 0, hi = -1;
    bool ok = true;
};

// Sources of several groups in summation order: groups in order, within a
// group ascending points (descending offsets), then references.
bool order_pulled(std::vector<Src>& v, SumKind s) {
    std::stable_sort(v.begin(), v.end(), [s](const Src& a, const Src& b) {
        const int ga = s == SUM_GRAD ? a.s.pat : a.s.group, gb = s == SUM_GRAD ? b.s.pat : b.s.group;
        if (ga != gb) return ga < gb;
        if (a.lo != b.lo) return a.lo > b.lo;
        return a.s.ref < b.s.ref;
    });
    return true;
}

// References of one data set whose points' order does not follow from their
// offsets: an inverse column beside any other column.
bool order_known(const Model& M, const std::vector<Src>& v) {
    std::map<int, std::pair<int, bool>> col;  // group -> (column, some inverse)
    for (const Src& s : v) {
        const int c = M.groups[s.s.group].vrefs[s.s.ref].col;
        auto it = col.find(s.s.group);
        if (it == col.end()) {
            col[s.s.group] = {c, s.s.how == OWN_INVERSE};
            continue;
        }
        it->second.second |= s.s.how == OWN_INVERSE;
        if (it->second.second && it->second.first != c) return false;
    }
    return true;
}

int weight_nodes(const Model& M, const std::vector<Src>& v) {
    int n = 0;
    for (const Src& s : v)
        if (s.s.wread < 0 && M.groups[s.s.group].ndata > 1) n += s.nodes;
    return n;
}

// A source as one unit over variables lo..hi pulls it.
OwnSrc within(const Model& M, const Src& x, int64_t lo, int64_t hi) {
    OwnSrc s = x.s;
    int64_t hit = std::min(hi, x.hi) - std::max(lo, x.lo) + 1;
    if (s.how == OWN_INVERSE) {
        const RefKey& k = M.groups[s.group].vrefs[s.ref];
        const std::vector<int32_t>& c = col_of(M, M.groups[s.group], k.col);
        hit = std::upper_bound(c.begin(), c.end(), hi - k.off) - std::lower_bound(c.begin(), c.end(), lo - k.off);
    }
    s.sparse = 4 * hit < 3 * (hi - lo + 1);
    return s;
}

// Whether the tables a cluster's sources need are worth it (kEntryBytes).
bool tables_pay(const Model& M, const Cluster& c) {
    int64_t entries = 0, table = 0;
    std::map<std::pair<int, int>, int64_t> span;  // a column's references share its table
    for (const Src& x : c.src) entries += M.groups[x.s.group].ndata;
    for (const std::vector<Src>* v : {&c.src, &c.grad})
        for (const Src& x : *v)
            if (x.s.how == OWN_INVERSE) span[{x.s.group, M.groups[x.s.group].vrefs[x.s.ref].col}] = x.hi - x.lo + 1;
    for (auto& t : span) table += 4 * t.second;
    return table <= 4 * (c.hi - c.lo + 1) + kEntryBytes * entries;
}

// The chains of host group g over a cluster, or none when g cannot host it.
std::vector<OwnChain> host_chains(const Model& M, const Cluster& C, int g, SumKind s) {
    std::vector<Src> mine, others;
    for (const Src& x : C.src) (x.s.group == g && x.s.wread < 0 ? mine : others).push_back(x);
    for (const Src& x : mine)
        if (x.s.how != OWN_AFFINE) return {};
    for (const Src& x : others)
        if (x.s.group == g) return {};  // a weight read of the host's own data set: order interleaved
    if (!order_known(M, others) || weight_nodes(M, others) > kHostPullNodes) return {};
    std::stable_sort(mine.begin(), mine.end(), [](const Src& a, const Src& b) {
        return a.lo != b.lo ? a.lo > b.lo : a.s.ref < b.s.ref;
    });
    const int64_t n = M.groups[g].ndata;
    std::vector<OwnChain> out;
    std::vector<std::pair<int64_t, int64_t>> dom;
    for (size_t i = 0; i < mine.size();) {
        OwnChain c;
        c.top = mine[i].s.ref;
        const int64_t top = shift_of(mine[i]);
        int64_t low = top;
        for (; i < mine.size() && top - shift_of(mine[i]) <= kOwnSpan; ++i) {
            low = shift_of(mine[i]);
            c.refs.emplace_back((int)(top - low), mine[i].s.ref);
        }
        dom.emplace_back(low, top + n - 1);
        out.push_back(c);
    }
    // the chains' variables: disjoint, and the whole cluster
    std::vector<std::pair<int64_t, int64_t>> d = dom;
    std::sort(d.begin(), d.end());
    int64_t at = C.lo;
    for (auto& x : d) {
        if (x.first != at) return {};
        at = x.second + 1;
    }
    if (at != C.hi + 1) return {};
    order_pulled(others, s);
    for (size_t i = 0; i < out.size(); ++i) {
        const int here = s == SUM_GRAD ? mine[0].s.pat : g;
        for (const Src& x : others)
            if (x.lo <= dom[i].second && x.hi >= dom[i].first) {
                const int there = s == SUM_GRAD ? x.s.pat : x.s.group;
                (there < here ? out[i].before : out[i].after).push_back(within(M, x, dom[i].first, dom[i].second));
            }
        for (const Src& x : C.grad)
            if (x.lo <= dom[i].second && x.hi >= dom[i].first)
                out[i].grad.push_back(within(M, x, dom[i].first, dom[i].second));
    }
    return out;
}

// The lists of U's slots over data set G (none when one is too long), and how
// far they are from the points' order.
void fill_lists(const Model& M, const Group& G, OwnUnit& U) {
    auto at = [&](const std::pair<int, int64_t>& sl, int64_t k) {
        return (sl.first < 0 ? 0 : (int64_t)col_of(M, G, sl.first)[k]) + sl.second;
    };
    U.lptr.assign(U.n + 1, 0);
    for (int64_t k = 0; k < G.ndata; ++k)
        for (auto& sl : U.slots) ++U.lptr[at(sl, k) + 1];
    for (int64_t i = 0; i < U.n; ++i) {
        if (U.lptr[i + 1] > kListLength) {
            U.lptr.clear();
            return;
        }
        U.lptr[i + 1] += U.lptr[i];
    }
    U.lent.assign(U.lptr[U.n] + 1, 0);
    std::vector<int32_t> fill(U.lptr.begin(), U.lptr.end() - 1);
    for (int64_t k = 0; k < G.ndata; ++k)
        for (size_t j = 0; j < U.slots.size(); ++j) U.lent[fill[at(U.slots[j], k)]++] = (int32_t)(4 * k + j);
    int64_t lines = 0;
    const int64_t ne = U.lptr[U.n];
    std::vector<int32_t> w;
    for (int64_t e = 0; e < ne; e += 256) {
        w.assign(U.lent.begin() + e, U.lent.begin() + std::min(ne, e + 256));
        for (int32_t& x : w) x >>= 6;  // 16 points: 128 bytes of a column
        std::sort(w.begin(), w.end());
        lines += std::unique(w.begin(), w.end()) - w.begin();
    }
    U.spread = ne ? 16.0 * lines / ne : 0.0;
}

// The unit that pulls a cluster through incidence lists (of the one data set
// with references in no order), or one without a data set.  Lists made before
// (another sum's, another of the cluster's ranges) are taken from `made`.
OwnUnit list_unit(const Model& M, const Cluster& C, SumKind s, std::vector<OwnUnit>& made) {
    OwnUnit U;
    int g = -1;
    for (const Src& x : C.src)
        if (x.kind == 3) {
            if (g >= 0 && x.s.group != g) return U;
            g = x.s.group;
        }
    const Group& G = M.groups[g];
    std::vector<Src> mine, others;
    for (const Src& x : C.src) (x.s.group == g ? mine : others).push_back(x);
    const int64_t entries = (int64_t)mine.size() * G.ndata;
    if (mine.size() > kListSlots || G.ndata >= (int64_t)1 << 29 || entries >= INT32_MAX) return U;
    std::stable_sort(mine.begin(), mine.end(), [](const Src& a, const Src& b) { return a.s.ref < b.s.ref; });
    std::vector<int> hit(M.pats.size(), 0);
    OwnUnit::Out o;
    o.lo = C.lo;
    for (const Src& x : mine) {
        if (x.s.wread >= 0) return U;
        const RefKey& k = G.vrefs[x.s.ref];
        U.slots.emplace_back(k.col, k.off - C.lo);
        o.refs.push_back(x.s.ref);
        for (int p : G.members)
            if (in_sum(M.pats[p], s) && std::find(M.pats[p].vg.begin(), M.pats[p].vg.end(), x.s.ref) != M.pats[p].vg.end())
                hit[p] = (int)M.pats[p].nodes.size();
    }
    int nodes = 0;
    for (int n : hit) nodes += n;
    if (nodes * (int)mine.size() > kListNodes || !order_known(M, others) || weight_nodes(M, others) > kPullNodes) return U;
    U.lo = C.lo;
    U.n = C.hi - C.lo + 1;
    if (U.n > 8 * entries + 64) return U;  // mostly variables without entries
    auto same = std::find_if(made.begin(), made.end(), [&](const OwnUnit& V) {
        return V.lgroup == g && V.n == U.n && V.slots == U.slots;
    });
    if (same == made.end()) {
        OwnUnit V;
        V.lgroup = g;
        V.n = U.n;
        V.slots = U.slots;
        fill_lists(M, G, V);
        same = made.insert(made.end(), std::move(V));
    }
    if (same->lptr.empty()) return U;
    int64_t bytes = 0;
    for (size_t p = 0; p < hit.size(); ++p) bytes += hit[p] ? 8 * G.ndata : 0;
    const Pattern& P0 = M.pats[G.members[0]];
    bytes += G.ndata * (4 * P0.n_icols + 8 * P0.n_fcols);
    if (bytes > kListBytes && same->spread > kListSpread) return U;
    U.lptr = same->lptr;
    U.lent = same->lent;
    order_pulled(others, s);
    for (const Src& x : others) (x.s.group < g ? o.before : o.after).push_back(within(M, x, C.lo, C.hi));
    for (const Src& x : C.grad) o.grad.push_back(within(M, x, C.lo, C.hi));
    U.outs.push_back(o);
    U.lgroup = g;
    return U;
}

void plan_one(Model& M, SumKind s, const std::vector<std::vector<char>>& inc,
              const std::vector<std::vector<int>>& period, std::vector<OwnUnit>& made) {
    OwnPlan& plan = M.own[s];
    plan = OwnPlan();
    if (s == SUM_GRAD && M.grad_direct) return;
    const bool with_grad = s == SUM_JT && M.grad_direct;
    // ---- sources
    std::vector<Src> all;
    std::vector<std::vector<int>> refs(M.groups.size());
    for (size_t g = 0; g < M.groups.size(); ++g) {
        const Group& G = M.groups[g];
        if (G.ndata == 0) continue;
        refs[g] = refs_of(M, G, s);
        if (s == SUM_GRAD) {
            int n = 0, pat = -1;
            for (int p : G.members)
                if (in_sum(M.pats[p], s)) ++n, pat = p;
            if (n > 1) return;  // the gradient's order is by pattern, not by data set
            for (int r : refs[g]) {
                all.push_back(make_src(M, (int)g, r, s, inc, period));
                all.back().s.pat = pat;
            }
            continue;
        }
        std::map<int, int> wr;
        for (int p : G.members)
            if (s == SUM_JT && M.pats[p].wread) wr[M.pats[p].vg[0]] = p;
        for (int r : refs[g]) {
            if (s == SUM_HV) {
                const size_t j = std::find(G.hv_refs.begin(), G.hv_refs.end(), r) - G.hv_refs.begin();
                if (G.hv_direct[j]) continue;
            }
            Src x = make_src(M, (int)g, r, s, inc, period);
            auto w = wr.find(r);
            if (w != wr.end()) {
                x.s.wread = w->second;
                if (x.kind == 1 || x.kind == 3) x.kind = 2;
            }
            all.push_back(x);
        }
    }
    if (s == SUM_GRAD)
        // the whole gradient or nothing: its units replace the patterns' own
        for (const Src& x : all)
            if (x.kind != 0) return;
    std::vector<Src> grads;
    if (with_grad)
        for (size_t p = 0; p < M.pats.size(); ++p) {
            const Pattern& P = M.pats[p];
            if (!in_sum(P, SUM_GRAD)) continue;
            for (int r : P.vg) {
                Src x = make_src(M, P.group, r, SUM_GRAD, inc, period);
                x.s.pat = (int)p;
                x.grad = true;
                x.nodes = (int)P.nodes.size();
                if (x.kind == 1) x.kind = 2;
                grads.push_back(x);
            }
        }
    // ---- variables of the sources that cannot be owned, and of any source
    std::vector<char> touched(M.nvar, 0);
    auto each_var = [&](const Src& x, auto&& f) {
        const Group& G = M.groups[x.s.group];
        const RefKey& k = G.vrefs[x.s.ref];
        if (k.col < 0) {
            f(k.off);
            return;
        }
        for (int32_t c : col_of(M, G, k.col)) f((int64_t)c + k.off);
    };
    std::vector<char> direct(M.nvar, 0);
    if (s == SUM_HV)
        for (const Group& G : M.groups)
            for (size_t j = 0; j < G.hv_refs.size(); ++j)
                if (G.hv_direct[j]) {
                    const RefKey& k = G.vrefs[G.hv_refs[j]];
                    for (int64_t q = 0; q < G.ndata; ++q)
                        direct[k.col < 0 ? k.off : (int64_t)M.pats[G.members[0]].icols[k.col][q] + k.off] = 1;
                }
    std::vector<Cluster> cl;
    std::vector<std::vector<OwnChain>> chains;
    std::vector<int> host;
    std::vector<OwnUnit> lists;
    for (;;) {
        std::vector<char> poison(M.nvar + 1, 0);
        for (const std::vector<Src>* v : {&all, &grads})
            for (const Src& x : *v) each_var(x, [&](int64_t i) {
                touched[i] = 1;
                if (x.kind == 1 || x.kind == 2) poison[i] = 1;
            });
        std::vector<int64_t> npoison(M.nvar + 1, 0), ntouched(M.nvar + 1, 0), ndirect(M.nvar + 1, 0);
        for (int64_t v = 0; v < M.nvar; ++v) {
            npoison[v + 1] = npoison[v] + poison[v];
            ntouched[v + 1] = ntouched[v] + touched[v];
            ndirect[v + 1] = ndirect[v] + direct[v];
        }
        // ---- clusters: unions of overlapping intervals
        std::vector<Src> order;
        for (const std::vector<Src>* v : {&all, &grads})
            for (const Src& x : *v)
                if (x.kind == 0 || x.kind == 3) order.push_back(x);
        std::stable_sort(order.begin(), order.end(), [](const Src& a, const Src& b) { return a.lo < b.lo; });
        cl.clear();
        for (const Src& x : order) {
            if (cl.empty() || x.lo > cl.back().hi) {
                cl.emplace_back();
                cl.back().lo = x.lo;
                cl.back().hi = x.hi;
            }
            Cluster& c = cl.back();
            c.hi = std::max(c.hi, x.hi);
            (x.grad ? c.grad : c.src).push_back(x);
        }
        // H v variables stored by the kernel never lie inside a cluster
        for (Cluster& c : cl)
            c.ok = npoison[c.hi + 1] == npoison[c.lo] && (s != SUM_HV || ndirect[c.hi + 1] == ndirect[c.lo]);
        // ---- units: a host where one can, else over the variables
        chains.assign(cl.size(), {});
        host.assign(cl.size(), -1);
        lists.assign(cl.size(), OwnUnit());
        bool again = false;
        for (size_t i = 0; i < cl.size(); ++i) {
            Cluster& c = cl[i];
            if (!c.ok) continue;
            if (weight_nodes(M, c.grad) > kHostPullNodes || !tables_pay(M, c)) {
                c.ok = false;
                continue;
            }
            if (std::any_of(c.src.begin(), c.src.end(), [](const Src& x) { return x.kind == 3; })) {
                lists[i] = list_unit(M, c, s, made);
                c.ok = lists[i].lgroup >= 0;
                continue;
            }
            std::vector<std::pair<int, int>> cand;  // (nodes, group)
            for (const Src& x : c.src)
                if (x.s.wread < 0 && x.s.how == OWN_AFFINE) {
                    int n = 0;
                    for (int p : M.groups[x.s.group].members)
                        if (in_sum(M.pats[p], s)) n += (int)M.pats[p].nodes.size();
                    if (M.groups[x.s.group].ndata > 1) cand.emplace_back(-n, x.s.group);
                }
            std::sort(cand.begin(), cand.end());
            for (auto& x : cand)
                if (host[i] < 0) {
                    chains[i] = host_chains(M, c, x.second, s);
                    if (!chains[i].empty()) host[i] = x.second;
                }
            if (host[i] < 0 && (!order_known(M, c.src) || weight_nodes(M, c.src) > kPullNodes)) c.ok = false;
        }
        // references in no order that no unit can pull: their variables stay in the
        // map, and those beside them are looked at again
        for (const Cluster& c : cl)
            for (const Src& x : c.src)
                if (!c.ok && x.kind == 3)
                    for (Src& y : all)
                        if (y.s.group == x.s.group && y.s.ref == x.s.ref) y.kind = 2, again = true;
        if (!again) break;
    }
    int nv = 0, nl = 0;
    for (size_t i = 0; i < cl.size(); ++i)
        if (cl[i].ok && host[i] < 0 && (++nv > EXA_MAX_VUNITS || (lists[i].lgroup >= 0 && ++nl > EXA_MAX_LISTS)))
            cl[i].ok = false;
    // the Lagrangian gradient: an objective pattern is owned whole or not at all
    for (bool again = with_grad; again;) {
        again = false;
        for (size_t p = 0; p < M.pats.size(); ++p) {
            if (!in_sum(M.pats[p], SUM_GRAD)) continue;
            int in = 0, total = 0;
            for (const Src& x : grads) total += x.s.pat == (int)p;
            for (const Cluster& c : cl)
                for (const Src& x : c.grad) in += c.ok && x.s.pat == (int)p;
            if (in == 0 || in == total) continue;
            for (Cluster& c : cl)
                for (const Src& x : c.grad)
                    if (c.ok && x.s.pat == (int)p) c.ok = false, again = true;
        }
    }
    if (s == SUM_GRAD)
        for (const Cluster& c : cl)
            if (!c.ok) return;
    // ---- what is owned: per (group, reference), per variable
    std::vector<std::vector<char>> owned(M.groups.size());
    for (size_t g = 0; g < M.groups.size(); ++g) owned[g].assign(M.groups[g].vrefs.size(), 0);
    plan.skip = direct;
    plan.drop.assign(M.pats.size(), 0);
    bool any = false;
    for (size_t i = 0; i < cl.size(); ++i) {
        const Cluster& c = cl[i];
        if (!c.ok) continue;
        any = true;
        for (const Src& x : c.src) owned[x.s.group][x.s.ref] = 1;
        for (const Src& x : c.grad) plan.drop[x.s.pat] = 1;
        std::fill(plan.skip.begin() + c.lo, plan.skip.begin() + c.hi + 1, 1);
    }
    // ---- fills: nothing contributes (a few long ranges; many short ones stay
    // in the map, whose reduction writes their zeros)
    std::vector<std::pair<int64_t, int64_t>> gaps;
    for (int64_t v = 0; v < M.nvar;) {
        if (touched[v] || plan.skip[v]) {
            ++v;
            continue;
        }
        int64_t e = v;
        while (e < M.nvar && !touched[e] && !plan.skip[e]) ++e;
        gaps.emplace_back(v, e - v);
        v = e;
    }
    if (gaps.size() <= 64) {
        plan.fill = gaps;
        for (auto& z : gaps) std::fill(plan.skip.begin() + z.first, plan.skip.begin() + z.first + z.second, 1);
        any = any || !gaps.empty();
    }
    // ---- host units, with the buffer, shared and direct references of their data sets
    for (size_t g = 0; g < M.groups.size(); ++g) {
        const Group& G = M.groups[g];
        OwnUnit U;
        U.code = EXA_OWN_CODE + (int)g;
        U.group = (int)g;
        U.npts = G.ndata;
        for (size_t i = 0; i < cl.size(); ++i)
            if (cl[i].ok && host[i] == (int)g) U.chains.insert(U.chains.end(), chains[i].begin(), chains[i].end());
        for (const OwnChain& c : U.chains)
            for (auto& r : c.refs) U.S = std::max(U.S, r.first);
        const int64_t W = 64 - U.S, chunks = (G.ndata + U.S + W - 1) / W;
        const int64_t runl = std::max<int64_t>(1, (chunks + kMaxRuns * kOwnWaves - 1) / (kMaxRuns * kOwnWaves)),
                      nrun = (chunks + runl * kOwnWaves - 1) / (runl * kOwnWaves);
        int partials = 0;
        const std::vector<int>& list = s == SUM_JT ? G.jt_refs : s == SUM_HV ? G.hv_refs : refs[g];
        if (G.ndata == 0) continue;
        for (size_t j = 0; j < list.size(); ++j) {
            const int r = list[j];
            if (s == SUM_HV && G.hv_direct[j]) {
                U.direct.push_back(r);
                continue;
            }
            if (owned[g][r]) continue;
            const RefKey& k = G.vrefs[r];
            const int64_t bs = (G.ndata + 15) & ~(int64_t)15;
            int P = 0;
            if (s != SUM_GRAD && k.col < 0)
                P = G.ndata > 1 ? 1 : 0;
            else if (s != SUM_GRAD)
                P = period[g][k.col];
            // a chunk's phases are its lanes' only when chunks start at
            // multiples of 64; the partial sums take the reference's slot
            if (P && (P == 1 || U.S == 0) && nrun * P <= bs && kOwnWaves * (partials + P) <= kMaxPartials) {
                partials += P;
                U.shared.emplace_back(r, P);
                any = true;
            } else {
                U.bufrefs.push_back(r);
            }
        }
        U.nrun = chunks;
        if (!U.shared.empty()) U.runl = runl, U.nrun = nrun;
        if (!U.chains.empty() || !U.bufrefs.empty() || !U.shared.empty() || !U.direct.empty()) plan.units.push_back(U);
    }
    int j = 0;
    for (size_t i = 0; i < cl.size(); ++i) {
        if (!cl[i].ok || host[i] >= 0 || lists[i].lgroup >= 0) continue;
        OwnUnit U;
        U.vunit = j;
        U.code = EXA_OWN_VCODE + j++;
        U.lo = cl[i].lo;
        U.n = cl[i].hi - cl[i].lo + 1;
        std::vector<Src> v = cl[i].src;
        order_pulled(v, s);
        for (const Src& x : v) U.srcs.push_back(within(M, x, cl[i].lo, cl[i].hi));
        for (const Src& x : cl[i].grad) U.grad.push_back(within(M, x, cl[i].lo, cl[i].hi));
        plan.units.push_back(U);
    }
    // lists: clusters with the same ones share a unit (a bus's angle and magnitude)
    std::vector<OwnUnit> with_lists;
    for (size_t i = 0; i < cl.size(); ++i) {
        if (!cl[i].ok || lists[i].lgroup < 0) continue;
        OwnUnit& U = lists[i];
        U.outs[0].vunit = j++;
        auto same = std::find_if(with_lists.begin(), with_lists.end(), [&](const OwnUnit& V) {
            return V.lgroup == U.lgroup && V.n == U.n && V.slots == U.slots && V.outs.size() < 2;
        });
        if (same != with_lists.end()) {
            same->outs.push_back(U.outs[0]);
            continue;
        }
        U.vunit = U.outs[0].vunit;
        U.code = EXA_OWN_VCODE + U.vunit;
        U.lunit = (int)with_lists.size();
        with_lists.push_back(std::move(U));
    }
    plan.units.insert(plan.units.end(), with_lists.begin(), with_lists.end());
    plan.on = any;
    if (!any) {
        plan = OwnPlan();
        return;
    }
    if (with_grad) {
        // zero entries of the gradient that the Lagrangian gradient's own
        // units do not write
        for (auto& z : M.grad_zero)
            for (int64_t v = z.first; v < z.first + z.second;) {
                if (plan.skip[v]) {
                    ++v;
                    continue;
                }
                int64_t e = v;
                while (e < z.first + z.second && !plan.skip[e]) ++e;
                plan.lag_zero.emplace_back(v, e - v);
                v = e;
            }
    }
}

void sign(std::ostringstream& os, const OwnSrc& s) {
    os << s.group << "." << s.ref << "." << s.how << "." << s.wread << "." << s.pat << (s.sparse ? "s," : ",");
}

}  // namespace

void plan_sums(Model& M) {
    for (Pattern& P : M.pats) {
        P.affine.assign(P.n_icols, 0);
        for (int c = 0; c < P.n_icols; ++c) {
            bool a = P.ndata > 0;
            for (int64_t k = 1; k < P.ndata && a; ++k) a = P.icols[c][k] == P.icols[c][0] + k;
            P.affine[c] = a ? 1 : 0;
        }
    }
    std::vector<std::vector<char>> inc(M.groups.size());
    std::vector<std::vector<int>> period(M.groups.size());
    for (size_t g = 0; g < M.groups.size(); ++g) {
        const Pattern& P0 = M.pats[M.groups[g].members[0]];
        for (int c = 0; c < P0.n_icols; ++c) {
            inc[g].push_back(P0.ndata > 0 && increasing(P0.icols[c]) ? 1 : 0);
            period[g].push_back(inc[g].back() ? 0 : period_of(P0.icols[c]));
        }
    }
    for (size_t g = 0; g < M.groups.size(); ++g) {
        M.groups[g].inc = inc[g];
        for (const auto& c : M.pats[M.groups[g].members[0]].icols) {
            auto mm = std::minmax_element(c.begin(), c.end());
            M.groups[g].range.emplace_back(c.empty() ? 0 : *mm.first, c.empty() ? 0 : *mm.second);
        }
    }
    std::vector<OwnUnit> made;
    for (int s = 0; s < SUM_COUNT; ++s) plan_one(M, (SumKind)s, inc, period, made);
    M.lag_units = M.own[SUM_JT].on && M.grad_direct;
    std::ostringstream os;
    for (int s = 0; s < SUM_COUNT; ++s) {
        const OwnPlan& p = M.own[s];
        os << s << (p.on ? "+" : "-") << (M.lag_units ? "L" : "");
        for (const OwnUnit& U : p.units) {
            os << "U" << U.code << "S" << U.S;
            for (const OwnChain& c : U.chains) {
                os << "c" << c.top << ":";
                for (auto& r : c.refs) os << r.first << "/" << r.second << ",";
                os << "b";
                for (auto& x : c.before) sign(os, x);
                os << "a";
                for (auto& x : c.after) sign(os, x);
                os << "g";
                for (auto& x : c.grad) sign(os, x);
            }
            os << "B";
            for (int r : U.bufrefs) os << r << ",";
            os << "s";
            for (auto& r : U.shared) os << r.first << "/" << r.second << ",";
            os << "d";
            for (int r : U.direct) os << r << ",";
            if (U.lgroup >= 0) {
                os << "l" << U.lgroup << "." << U.lunit << ":";
                for (auto& x : U.slots) os << x.first << ",";
            }
            for (const OwnUnit::Out& o : U.outs) {
                os << "o" << o.vunit << ":";
                for (int r : o.refs) os << r << ",";
                os << "b";
                for (auto& x : o.before) sign(os, x);
                os << "a";
                for (auto& x : o.after) sign(os, x);
                os << "g";
                for (auto& x : o.grad) sign(os, x);
            }
            os << "v";
            for (auto& x : U.srcs) sign(os, x);
            os << "g";
            for (auto& x : U.grad) sign(os, x);
        }
    }
    M.own_sig = os.str();
}

void drop_plans(Model& M) {
    const bool grad = M.use_own && M.own[SUM_GRAD].on;
    for (OwnPlan& p : M.own) p = OwnPlan();
    M.use_own = M.lag_units = false;
    M.lean = true;
    M.epl_most = false;
    M.own_sig = "0-1-2-";
    sum_map(M, SUM_JT, false, M.jt_map);
    sum_map(M, SUM_HV, false, M.h_map);
    if (grad) sum_map(M, SUM_GRAD, false, M.grad_map);
}

const OwnPlan* own_plan(const Model& M, int mode, bool own) {
    if (!own) return nullptr;
    const OwnPlan* p = mode == M_JTPROD || mode == M_LAG || mode == M_GRADL ? &M.own[SUM_JT]
                       : mode == M_HPROD                                  ? &M.own[SUM_HV]
                       : mode == M_GRAD                                   ? &M.own[SUM_GRAD]
                                                                          : nullptr;
    return p && p->on ? p : nullptr;
}

// Entries (variable, position) in summation order: data sets in declaration
// order, ascending points, then references (the gradient: patterns, points,
// slots); with own, only what the plan leaves to the reduction, a data set's
// partial sums (run by run) after its per-point entries.
void sum_map(const Model& M, SumKind s, bool own, SegMap& out) {
    const OwnPlan* plan = own && M.own[s].on ? &M.own[s] : nullptr;
    std::vector<std::pair<int64_t, int64_t>> e;
    auto var = [&](const Group& G, int r, int64_t k) {
        const RefKey& rk = G.vrefs[r];
        return rk.col < 0 ? rk.off : (int64_t)M.pats[G.members[0]].icols[rk.col][k] + rk.off;
    };
    std::vector<char> skip;
    if (plan) {
        skip = plan->skip;
    } else if (s == SUM_HV) {
        skip.assign(M.nvar, 0);
        for (const Group& G : M.groups)
            for (size_t j = 0; j < G.hv_refs.size(); ++j)
                for (int64_t k = 0; G.hv_direct[j] && k < G.ndata; ++k) skip[var(G, G.hv_refs[j], k)] = 1;
    }
    if (s == SUM_GRAD) {
        for (const Pattern& P : M.pats)
            if (P.kind == EXA_OBJ && !plan)
                for (int64_t k = 0; k < P.ndata; ++k)
                    for (int q = 0; q < P.o1step(); ++q) e.emplace_back(P.var_index(q, k), P.ob + q * P.bstride() + k);
    } else {
        for (size_t g = 0; g < M.groups.size(); ++g) {
            const Group& G = M.groups[g];
            const int64_t bs = (G.ndata + 15) & ~(int64_t)15;
            const int64_t base = s == SUM_JT ? M.fo_obj_len + G.ob : G.oh;
            const std::vector<int>& list = s == SUM_JT ? G.jt_refs : G.hv_refs;
            const OwnUnit* U = nullptr;
            if (plan)
                for (const OwnUnit& u : plan->units)
                    if (u.group == (int)g) U = &u;
            // (reference, position of its slot array or -1, weight pattern or -1)
            struct Ent {
                int r;
                int64_t pos;
                int w;
            };
            std::vector<Ent> ent;
            std::vector<char> shared(G.vrefs.size(), 0);
            if (U)
                for (auto& x : U->shared) shared[x.first] = 1;
            for (size_t j = 0; j < list.size(); ++j) {
                const int r = list[j];
                if (s == SUM_HV && G.hv_direct[j]) continue;
                if (plan && (!U || std::find(U->bufrefs.begin(), U->bufrefs.end(), r) == U->bufrefs.end())) continue;
                ent.push_back({r, base + (int64_t)j * bs, -1});
            }
            // weight entries ~(2 row + negated) of augmentation terms that are
            // one variable; owned ones are written by their units
            for (int p : G.members)
                if (s == SUM_JT && M.pats[p].wread) {
                    const int r = M.pats[p].vg[0];
                    if (plan && G.ndata > 0 && plan->skip[var(G, r, 0)]) continue;
                    ent.push_back({r, -1, p});
                }
            std::sort(ent.begin(), ent.end(), [](const Ent& a, const Ent& b) { return a.r < b.r; });
            for (int64_t k = 0; k < G.ndata && !ent.empty(); ++k)
                for (const Ent& x : ent) {
                    if (x.w < 0) {
                        e.emplace_back(var(G, x.r, k), x.pos + k);
                        continue;
                    }
                    const Pattern& A = M.pats[x.w];
                    const int64_t row = A.tgt0 + (int64_t)A.icols[A.row_icol][k] + A.row_off;
                    e.emplace_back(var(G, x.r, k), ~(2 * row + (A.wread < 0 ? 1 : 0)));
                }
            if (U)
                for (auto& x : U->shared) {
                    const int64_t j = std::find(list.begin(), list.end(), x.first) - list.begin();
                    for (int64_t run = 0; run < U->nrun; ++run)
                        for (int ph = 0; ph < x.second && ph < G.ndata; ++ph)
                            e.emplace_back(var(G, x.first, ph), base + j * bs + ph * U->nrun + run);
                }
        }
    }
    out = SegMap();
    out.ptr.assign(M.nvar + 1, 0);
    for (auto& x : e) out.ptr[x.first + 1]++;
    for (int64_t v = 0; v < M.nvar; ++v) out.ptr[v + 1] += out.ptr[v];
    out.idx.assign(e.size(), 0);
    std::vector<int64_t> fill(out.ptr.begin(), out.ptr.end() - 1);
    for (auto& x : e) out.idx[fill[x.first]++] = x.second;
    if (std::find(skip.begin(), skip.end(), 1) != skip.end()) {
        for (int64_t v = 0; v < M.nvar; ++v)
            if (skip[v] && out.ptr[v + 1] > out.ptr[v])
                fail(EXA_EINVAL, "internal: a variable written by a unit has reduction entries");
        out.skip = std::move(skip);
    }
}

}  // namespace exa
