// Internal declarations of the evaluator library (not part of the C ABI).
#pragma once

#include <atomic>
#include <cstdint>
#include <map>
#include <memory>
#include <stdexcept>
#include <string>
#include <vector>

#include "../../include/exa.h"

namespace exa {

// ---------------------------------------------------------------------------
// Errors: thrown inside the library, turned into exa_status at the ABI.
struct Error : std::runtime_error {
    exa_status code;
    Error(exa_status c, const std::string& m) : std::runtime_error(m), code(c) {}
};
[[noreturn]] void fail(exa_status code, const std::string& msg);
void set_last_error(const std::string& msg);

// ---------------------------------------------------------------------------
// Device-side layout.  The same text defines the structs for the host
// compiler and, stringified, for the run-time compiled kernels, so the two
// layouts cannot drift apart.
// Index into ExaInstDev::off: where an instance's slice starts in each of
// the arrays a call reads or writes.
#define EXA_OFF_ROWS 0    /* constraint rows (ncon)                          */
#define EXA_OFF_AUG 1     /* augmentation term buffer (naug)                 */
#define EXA_OFF_JAC 2     /* Jacobian values (nnzj)                          */
#define EXA_OFF_HESS 3    /* Hessian values (nnzh)                           */
#define EXA_OFF_PAR 4     /* parameter-adjoint buffer (nnzp)                 */
#define EXA_OFF_TILE 5    /* per-tile partial sums of the objective          */
#define EXA_OFF_X 6       /* x and v/w vectors (nvar)                        */
#define EXA_OFF_Y 7       /* y (ncon)                                        */
#define EXA_OFF_FO_OBJ 8  /* first-order buffer, objective part (nnzg)       */
#define EXA_OFF_FO_CON 9  /* first-order buffer, constraint part (nnzj)      */
#define EXA_OFF_HV 10     /* H v buffer (curved slots)                       */
#define EXA_NOFF 12
// Index offsets of a pattern's unique references live in ExaPatDev::roff
// (variable slots first, then parameter slots), so that every instance of a
// formulation runs the same code whatever its block offsets.
#define EXA_MAX_REFS 48
// Tile code of a zero-fill tile (entries of g no objective term touches).
#define EXA_ZERO_TILE 1023
// Codes of the units that finish variables themselves (OwnUnit): data set g
// -> EXA_OWN_CODE + g, the j-th unit over variables -> EXA_OWN_VCODE + j.
#define EXA_OWN_CODE 128
#define EXA_OWN_VCODE 256
#define EXA_MAX_VUNITS 32
// Units over variables that pull through incidence lists: at most this many
// per sum, of at most EXA_LIST_TILE entries and variables per tile.
#define EXA_MAX_LISTS 4
#define EXA_LIST_TILE 256
#define EXA_PAD_TILE 4095  // a tile that matches no unit: does nothing
// A tile that only reads T.count bytes of input ahead of the tiles that need
// them: from entry T.start of x, y, v or the J^T w weights of its launch
// (T.slot = EXA_AHEAD_*), or from byte T.start of the device address T.slot.
#define EXA_AHEAD_TILE 4094
#define EXA_AHEAD_X 0
#define EXA_AHEAD_Y 1
#define EXA_AHEAD_V 2
#define EXA_AHEAD_W 3

// ExaPatDev::hvd: bit r set when the pattern's group stores H v reference r
// straight into the output (Group::hv_direct, for this instance's data).
// ExaPatDev::vd, inv, icmin, icmax, runl, nrun are filled for the first
// pattern of a data set: vd[r] is the shift of group reference r (variable =
// data point + vd[r] when its index column counts up by one; variable =
// column value + vd[r] when the column's inverse table inv[c] is used), inv[c]
// maps column values icmin[c] .. icmax[c] to their data point or -1, runl[s]
// and nrun[s] are the 64-lane chunks per wave and the runs of the data set's
// unit for sum s (SumKind).  ExaInstDev::vlo[s][j]: the first variable of the
// j-th unit over variables of sum s.  ExaInstDev::nobj: objective tiles, whose
// partial sums the last of them adds (ExaCall::direct, EXA_ARRIVAL).
// ExaMulti::in: the launch's inputs by EXA_AHEAD_*, for read-ahead tiles.  ExaInstDev::lptr[s][j], lent[s][j] (J^T w
// and H v): incidence lists of its j-th list unit, entries lptr[i] .. lptr[i+1]
// of the unit's i-th variable, each a data point * 4 + the slot (OwnUnit::slots).
// EXA_G and EXA_K name the address spaces of data (global memory) and of the
// tables (read-only for a launch) in the generated code; the host has one.
// Without them a pointer read from a table is generic: its loads are flat ones
// (which hold back every later wait, LDS included), and a table field behind a
// store is read by a vector load, into registers: the network's jtprod kernel
// took 90 vector registers instead of 60, exa_k_multi 119 instead of 91, the
// trajectory's 149 instead of 120.  Before / after, inputs from HBM: every
// callback of the trajectory 159 / 130 us, of the grid 61.7 / 54.4, of 64
// networks 183 / 170, of 10,000 buses 10.3 / 8.8; Lagrangian gradient and H v
// of 65,536 scenarios 79 / 62.
#define EXA_DEVICE_STRUCTS                                                       \
    struct ExaPatDev {                                                           \
        const EXA_G int* ic[8];                                                  \
        const EXA_G double* fc[8];                                               \
        long long ndata;                                                         \
        long long o0;                                                            \
        long long o1;                                                            \
        long long o2;                                                            \
        long long op;                                                            \
        long long oh;                                                            \
        long long ob;                                                            \
        long long tgt0;                                                          \
        long long row_off;                                                       \
        int row_ic;                                                              \
        int hvd;                                                                 \
        const EXA_G int* rptr;                                                   \
        const EXA_G int* ridx;                                                   \
        long long roff[48];                                                      \
        long long vd[48];                                                        \
        const EXA_G int* inv[8];                                                 \
        int icmin[8];                                                            \
        int icmax[8];                                                            \
        int runl[4];                                                             \
        int nrun[4];                                                             \
    };                                                                           \
    struct ExaInstDev {                                                          \
        long long off[12];                                                       \
        const EXA_G double* theta;                                               \
        long long nobj;                                                          \
        long long vlo[4][32];                                                    \
        const EXA_G int* lptr[2][4];                                             \
        const EXA_G int* lent[2][4];                                             \
        struct ExaPatDev pat[32];                                                \
    };                                                                           \
    struct ExaTile {                                                             \
        int pat;                                                                 \
        int inst;                                                                \
        long long start;                                                         \
        long long count;                                                         \
        long long slot;                                                          \
    };                                                                           \
    struct ExaCall {                                                             \
        const struct ExaTile* tiles;                                             \
        long long ntiles;                                                        \
        long long per_xcd;                                                       \
        const EXA_K struct ExaInstDev* inst;                                     \
        const double* x;                                                         \
        const double* y;                                                         \
        const double* v;                                                         \
        double* out0;                                                            \
        double* out1;                                                            \
        double sigma;                                                            \
        int direct;                                                              \
        int unstaged;                                                            \
    };                                                                           \
    struct ExaMulti {                                                            \
        const struct ExaTile* tiles;                                             \
        long long ntiles;                                                        \
        long long per_xcd;                                                       \
        const EXA_K struct ExaInstDev* inst;                                     \
        struct ExaCall c[10];                                                    \
        const double* in[4];                                                     \
    };

#define EXA_G
#define EXA_K
EXA_DEVICE_STRUCTS
#undef EXA_G
#undef EXA_K

// Counting the objective's tiles as they finish, so that the last one adds
// their partial sums (exa_obj_finish).  Tiles count in groups of 32 in a row,
// each group on a 128-byte line of its own (line 1 + slot / 32), and whoever
// completes a group counts it on line 0.  One count on one address took 20 ns
// a tile, one after another: 65,536 scenarios (1025 tiles) 24.1 us, 8,000,000
// Rosenbrock terms (3907 tiles) 60.8, against 13.3 and 24.8 with a launch that
// adds the sums; in two levels 13.1 and 18.4.
// Counts are never cleared: a group of fewer tiles has its last tile weigh the
// rest, and a count is complete when it passes a multiple of its power of two.
// L launches that overlap pass L multiples whatever their order, so they leave
// the counts as they found them (a launch's result may then be formed too
// early; the next call's is right).
#define EXA_ARRIVAL                                                                  \
    struct ExaArrival {                                                              \
        unsigned line, weight, bits, group_weight, group_bits;                       \
    };                                                                               \
    EXA_FN struct ExaArrival exa_arrival(long long slot, long long n) {              \
        struct ExaArrival a;                                                         \
        const unsigned g = (unsigned)(slot >> 5), last = (unsigned)((n - 1) >> 5);   \
        a.line = 1 + g;                                                              \
        a.bits = 5;                                                                  \
        a.weight = slot == n - 1 ? 32u - (unsigned)(slot & 31) : 1u;                 \
        a.group_bits = 0;                                                            \
        while ((1u << a.group_bits) < last + 1) ++a.group_bits;                      \
        a.group_weight = g == last ? (1u << a.group_bits) - last : 1u;               \
        return a;                                                                    \
    }                                                                                \
    EXA_FN bool exa_completes(unsigned before, unsigned weight, unsigned bits) {     \
        return ((before + weight) >> bits) != (before >> bits);                      \
    }
#define EXA_FN static inline
EXA_ARRIVAL
#undef EXA_FN
// First 8-byte word of the counts behind n partial sums, and words in all.
#define EXA_COUNT_AT(n) (((n) + 15) & ~15LL)
inline int64_t count_words(int64_t n) { return n > 1 ? EXA_COUNT_AT(n) + 16 * (1 + (n + 31) / 32) : 1; }

#define EXA_STR2(...) #__VA_ARGS__
#define EXA_STR(...) EXA_STR2(__VA_ARGS__)

// ---------------------------------------------------------------------------
// Host-side model.

enum Mode : int {
    M_OBJ = 0,    // objective terms -> per-tile partial sums
    M_CONS = 1,   // constraint rows; each pulls its augmentation terms
    M_GRAD = 2,   // objective gradient: in place, or first-order buffer
    M_JAC = 3,    // Jacobian values
    M_HESS = 4,   // Lagrangian Hessian values
    M_JPROD = 5,  // J v rows; each pulls its augmentation terms
    M_JTPROD = 6, // w[row] * J -> first-order buffer (jac part)
    M_HPROD = 7,  // local (w H) v on curved slots -> H v buffer
    M_ADJ = 8,    // mixed partials -> parameter buffer
    M_JH = 9,     // Jacobian and Hessian values of each data point in one pass
    M_COUNT = 10
};
static_assert(M_COUNT == 10, "ExaMulti holds one call per mode");
// Units that run several callbacks' jobs at one point from one set of loads
// and sweeps, used by the several-callback kernel only (their jobs take
// inputs and outputs from the per-mode calls of an ExaMulti):
// M_SFULL: grad, cons, jac, hess, jprod, hprod (a J^T w of the same call is
//          summed from the Jacobian values by the reduction launch);
// M_SIPM:  grad, cons, jac, hess (an interior-point iterate).
constexpr int M_SFULL = 10, M_SIPM = 11;
inline bool multi_unit_mode(int mode) { return mode == M_SFULL || mode == M_SIPM; }
// The Lagrangian gradient of variables whose J^T y and objective gradient the
// units finish themselves: M_LAG runs the J^T w units with sigma * gradient
// added (call record of M_JTPROD), M_GRADL the gradient's tiles of the other
// variables (call record and code of M_GRAD).
constexpr int M_LAG = 12, M_GRADL = 13;
// Tiles of the several-callback kernel carry their mode above this bit of
// the unit code (unit codes stay below 1 << EXA_MODE_SHIFT).
#define EXA_MODE_SHIFT 12

struct TNode {            // node of a simplified tree
    int op = 0;
    int a = -1, b = -1;   // children (positions in the node list)
    int col = -1;         // data column (DATA) or index column (VAR/PARAM)
    int64_t off = 0;      // index offset (VAR/PARAM)
    double val = 0.0;     // literal (CONST)
    int slot = -1;        // VAR: unique var slot; PARAM: unique param slot
};

struct RefKey {           // symbolic identity of a var/param reference
    int col;
    int64_t off;
    bool operator==(const RefKey& o) const { return col == o.col && off == o.off; }
};

struct Pattern {
    int kind = 0;
    int index = 0;                    // declaration position
    std::vector<TNode> nodes;         // simplified tree, post-order, root last
    int64_t ndata = 0;
    int n_icols = 0, n_fcols = 0;
    std::vector<std::vector<int32_t>> icols;   // host copies (index columns)
    // index column c holds c0, c0 + 1, ..., c0 + ndata - 1 (at least kIdentMin
    // points): the generated code uses the data point itself instead of
    // loading it (c0 sits in the references' offsets)
    std::vector<char> ident;
    // index column c holds c0, c0 + 1, ... (any length); c0 = icols[c][0].
    // The generated code counts such columns of at least kIdentMin points
    // from the data point (ident), with c0 folded into the index offsets
    std::vector<char> affine;
    std::vector<const double*> fcols_src;      // caller's float columns (create only)
    std::vector<RefKey> vslots;       // unique var refs, first-visit order
    std::vector<RefKey> pslots;       // unique param refs
    std::vector<std::pair<int, int>> hslots;   // unique pairs of var slots
    // layout
    int64_t o0 = 0;   // CON first row; OBJ first term; AUG first aug entry
    int64_t o1 = 0;   // CON/AUG first jac entry; OBJ first grad-buffer entry
    int64_t o2 = 0;   // first hess entry
    int64_t op = 0;   // first param-buffer entry
    int64_t ob = 0;   // first entry of this pattern's block in its part of the first-order buffer
    int target = -1;
    int row_icol = -1;
    int64_t row_off = 0;
    int64_t tgt0 = 0; // AUG: first row of the target block
    std::vector<double> lcon, ucon;
    // data-set group (patterns over the same data arrays) and the group-level
    // reference each of this pattern's var / param slots maps to
    int group = -1;
    std::vector<int> vg, pg;
    // AUG: data points grouped by the target row they add to (CSR over the
    // target block's rows, points ascending): the row's lane pulls them
    std::vector<int32_t> rptr, ridx;
    // CON: augmentation patterns adding to this block, declaration order
    std::vector<int> augs;
    // var slots that occur in some Hessian pair (the only ones H v reaches)
    std::vector<int> hvs;
    // AUG whose expression is plus or minus one variable, the only J^T w
    // contribution of its data set to that reference: its contribution is
    // +-w[row], which the reduction reads from w itself (no J^T w job)
    int wread = 0;  // +1, -1, or 0
    int64_t oh = 0;   // first entry of this pattern in the H v buffer

    // work buffers (first-order, H v, parameter) hold each pattern's block
    // slot-major: slot s of data point k at block + s * bstride() + k, with
    // every slot array padded to whole 128-byte lines
    int64_t bstride() const { return (ndata + 15) & ~(int64_t)15; }
    int o1step() const { return (int)vslots.size(); }
    int o2step() const { return (int)hslots.size(); }
    int pstep() const { return (int)pslots.size(); }
    int64_t row(int64_t k) const {
        return kind == EXA_CON ? o0 + k : tgt0 + (int64_t)icols[row_icol][k] + row_off;
    }
    int64_t var_index(int s, int64_t k) const {
        const RefKey& r = vslots[s];
        return r.col < 0 ? r.off : (int64_t)icols[r.col][k] + r.off;
    }
    int64_t par_index(int s, int64_t k) const {
        const RefKey& r = pslots[s];
        return r.col < 0 ? r.off : (int64_t)icols[r.col][k] + r.off;
    }
};

// Patterns declared over the very same data arrays (same ndata, same column
// arrays in the same order).  Their evaluations can share one lane: the data
// loads, the gathers of x and common subexpressions are then done once.
struct Group {
    std::vector<int> members;          // pattern positions, declaration order
    std::vector<RefKey> vrefs, prefs;  // distinct references over all members
    std::vector<std::pair<int, int>> vsrc, psrc;  // first (member, slot) of each
    int64_t ndata = 0;
    std::vector<char> inc;  // index columns that increase strictly (plan_sums)
    std::vector<std::pair<int32_t, int32_t>> range;  // least and greatest value of each index column
    // J^T w and H v contributions are summed over the members of a point
    // before they leave the lane: one buffer slot per group-level reference
    // that some member contributes to (ascending reference index), blocks at
    // ob (constraint part of the first-order buffer) and oh (H v buffer)
    std::vector<int> jt_refs, hv_refs;
    int64_t ob = 0, oh = 0;
    // per H v reference: every entry it stores is the only H v contribution
    // to its variable (at most 32 references).  Code generated with the flag
    // set writes the output entry itself when the instance's bit in
    // ExaPatDev::hvd is set, and the buffer entry otherwise; code generated
    // without it always writes the buffer entry (no index kept live)
    std::vector<char> hv_direct;
};

// A unit of generated code for one callback: one pattern, or the members of
// a group evaluated together.  Tile codes: pattern p -> p, group g -> 32 + g.
struct Unit {
    int code = 0;
    int group = 0;
    std::vector<int> members;
    int64_t ndata = 0;
};

// Inputs a unit's generated code really reads for one data point (after
// dead-code elimination), used to report algorithmic traffic.
struct UnitLive {
    std::vector<int> icols, fcols;     // data columns
    std::vector<int> vrefs, vseeds, prefs;  // group-level references
    int weights = 0;                   // y entries (one per member that needs it)
    int64_t outputs = 0;               // doubles written per data point
    bool pulls = false;                // base rows pull augmentation terms
    int64_t extra = 0;                 // bytes per point or variable of pulled contributions
};

// Sorted reduction map (CSR): segment s sums buf[idx[ptr[s] .. ptr[s+1])].
struct SegMap {
    std::vector<int64_t> ptr, idx;
    // segments the reduction leaves alone (empty: none); such a segment has
    // no entries, its output is written by the evaluation kernel
    std::vector<char> skip;
    int64_t nseg() const { return ptr.empty() ? 0 : (int64_t)ptr.size() - 1; }
};

// ---- sums finished by the units themselves -----------------------------------
// A variable whose contributions to a sum all come through strictly increasing
// index columns gets at most one from each (data set, reference), at a data
// point that follows from the variable; one data set's columns in no order
// give a variable a list of points (incidence lists).  Such a variable needs
// no work buffer and no map: a unit adds its contributions in the map's order
// (data set, point, reference) and stores the sum.  plan_sums finds these variables per
// sum, in clusters (intervals of variables whose references overlap), and the
// units that own them:
//  * the unit of a host data set whose columns count up by one: lane of point
//    k owns variable k + top, takes the contributions of the references whose
//    offset is smaller by s from the lane s further up (a wave's last lanes
//    recompute the next wave's first points: W = 64 - S owners per wave), and
//    evaluates ("pulls") the contributions of other data sets itself;
//  * where a data set's references come in no order, a unit over the cluster's
//    variables that pulls its contributions through incidence lists;
//  * otherwise a unit over the cluster's variables, one lane each, which pulls
//    every contribution (through the column's inverse table where a column
//    has gaps).
// References that few variables share (a literal index, or a column that
// repeats with a period of 2 to 32 points) leave one partial sum per run of
// chunks instead of one entry per point: a wave adds its lanes.
enum SumKind : int { SUM_JT = 0, SUM_HV = 1, SUM_GRAD = 2, SUM_COUNT = 3 };
struct OwnSrc {
    int group = 0, ref = 0;  // data set and group reference
    int how = 0;             // OWN_AFFINE, OWN_INVERSE or OWN_LIST
    int wread = -1;          // augmentation pattern whose +-w[row] this is
    int pat = -1;            // objective pattern (gradient contributions)
    bool sparse = false;     // contributes to under three quarters of the unit's variables: behind a branch
};
constexpr int OWN_AFFINE = 0, OWN_INVERSE = 1, OWN_LIST = 2;
constexpr int kOwnWaves = 4;
constexpr int kOwnSpan = 8;  // largest lane shift of a chain
struct OwnChain {
    int top = 0;                             // reference with the largest offset
    std::vector<std::pair<int, int>> refs;   // (lane shift, reference), summation order
    std::vector<OwnSrc> before, after;       // pulled, from data sets before / after the host
    std::vector<OwnSrc> grad;                // pulled objective gradient (Lagrangian gradient only)
};
struct OwnUnit {
    int code = 0;
    int group = -1;                  // host data set, or -1: a unit over variables
    std::vector<OwnChain> chains;    // host units
    int S = 0;                       // largest lane shift
    std::vector<int> bufrefs;        // references that go to the work buffer, one entry per point
    std::vector<std::pair<int, int>> shared;  // (reference, period): partial sums
    std::vector<int> direct;         // H v references stored straight into the output
    int vunit = -1;                  // units over variables: index j, and their pulled sources in order
    std::vector<OwnSrc> srcs, grad;
    int64_t lo = 0, n = 0;           // units over variables: this instance's range
    // units over variables that pull data set lgroup's contributions through
    // incidence lists: an entry is a point and one of up to four slots (an
    // index column and an offset), its contribution to output o that of
    // reference outs[o].refs[slot]; output o's variables are lo .. lo + n - 1
    // of range vunit, its other sources before / after the data set's
    int lgroup = -1, lunit = -1;
    struct Out {
        int vunit = 0;
        int64_t lo = 0;
        std::vector<int> refs;
        std::vector<OwnSrc> before, after, grad;
    };
    std::vector<Out> outs;
    std::vector<std::pair<int, int64_t>> slots;  // (column, offset from the range's first variable)
    std::vector<int32_t> lptr, lent;             // this instance's lists
    double spread = 0;  // 128-byte lines 256 entries touch, over those of 256 points in a row
    // host units: this instance's points, chunks a wave takes in turn, and
    // runs of one wave, or with shared references of kOwnWaves waves whose
    // partial sums are added in order into one
    int64_t npts = 0;
    int64_t runl = 1, nrun = 0;
    int64_t points_per_run() const { return runl * (64 - S) * (shared.empty() ? 1 : kOwnWaves); }
    // lanes take points as in any unit (no shifts, no sums over a wave)
    bool plain() const { return S == 0 && shared.empty(); }
};
struct OwnPlan {
    bool on = false;
    std::vector<OwnUnit> units;
    std::vector<std::pair<int64_t, int64_t>> fill;  // (first, count): variables nothing contributes to
    std::vector<char> skip;   // variables the units write (owned, filled or direct)
    std::vector<char> drop;   // per objective pattern: its gradient is owned (M_GRADL leaves it out)
    std::vector<std::pair<int64_t, int64_t>> lag_zero;  // gradient zero ranges of M_GRADL
};

struct DeviceState;  // defined in exa_runtime.cpp

struct Model {
    int64_t nvar = 0, ncon = 0, ntheta = 0;
    int64_t nnzj = 0, nnzh = 0, nnzg = 0, naug = 0, nnzp = 0, nobj = 0, nhv = 0;
    // work-buffer lengths (entries, slot arrays padded): first-order buffer
    // (objective part, then constraint part), H v buffer, parameter buffer
    int64_t fo_obj_len = 0, fo_con_len = 0, hv_len = 0, par_len = 0;
    // every variable gets at most one objective-gradient contribution: the
    // gradient kernel writes g directly (plus zero tiles for the rest)
    bool grad_direct = false;
    std::vector<std::pair<int64_t, int64_t>> grad_zero;  // untouched ranges of g
    std::vector<Pattern> pats;
    std::vector<Group> groups;
    std::vector<double> xl, xu, theta;
    // reduction maps (positions in the first-order buffer: grad part first)
    SegMap grad_map, jt_map, h_map, par_map;
    // sums finished by the units (per SumKind); device models run them, and
    // their maps hold the other variables only (host-only and lean models use
    // the general maps and units).  A batch runs instances of one plan
    // (own_sig) in one launch, each with its own plan's units
    OwnPlan own[SUM_COUNT];
    bool use_own = false;
    // a device-memory budget left no room for what finishing units need beside
    // the buffers: every sum goes through its map, objectives of several tiles
    // through the reduction launch
    bool lean = false;
    std::string own_sig;     // what the plans fix in the generated code
    bool lag_units = false;  // the Lagrangian gradient runs M_LAG units
    bool host_only = false;
    int block = 256, epl = 4;
    bool epl_most = true;  // untimed launches may take fewer points per lane than epl
    bool autotune = false, fuse = false;
    bool eval_per_mode = false;  // exa_eval: per-callback tiles only
    std::string signature;   // hash of the simplified trees (shared code)
    std::string cache_dir;   // code-object cache directory ("" : none)
    int64_t max_device_bytes = 0;  // device memory budget (0: none)
    // build statistics: host analysis, code generation and compilation (or
    // cache read) in milliseconds; whether the code object came from the
    // on-disk cache; whether it was shared with a live model
    double host_ms = 0, codegen_ms = 0, compile_ms = 0;
    bool cache_hit = false, module_shared = false;
    // inputs each generated unit really reads, per (mode, unit code)
    std::map<std::pair<int, int>, UnitLive> live;
    std::atomic<int64_t> counters[9];
    // compressed sparse columns of the Jacobian (0) and of the Hessian's
    // lower triangle (1), analysed on first use: colptr [nvar+1], rowval,
    // and the COO positions each entry sums (ascending)
    struct Csc {
        bool ready = false;
        std::vector<int32_t> colptr, rowval;
        SegMap map;
    };
    Csc csc[2];
    std::unique_ptr<DeviceState> dev;
    Model();
    ~Model();
};

// exa_model.cpp
void build_host(Model& M, const exa_pattern_desc* pats, int32_t npats);
std::string pattern_signature(const Model& M);
// Augmentations a and b have the same row lists (rptr / ridx): the same data
// arrays, rows from the same index column plus the same offset, and targets
// of one size.  The generated pulls of such augmentations share one walk.
bool same_walk(const Model& M, int a, int b);

// exa_owner.cpp
void plan_sums(Model& M);
// No sums finished by units (Model::lean).
void drop_plans(Model& M);
// Every source that a unit pulls from or counts its variables by.
template <class F>
void each_source(const OwnUnit& U, F&& f) {
    for (const std::vector<OwnSrc>* v : {&U.srcs, &U.grad})
        for (const OwnSrc& x : *v) f(x);
    for (const OwnUnit::Out& o : U.outs)
        for (const std::vector<OwnSrc>* v : {&o.before, &o.after, &o.grad})
            for (const OwnSrc& x : *v) f(x);
    for (const OwnChain& c : U.chains) {
        OwnSrc top;
        top.group = U.group;
        top.ref = c.top;
        f(top);
        for (const std::vector<OwnSrc>* v : {&c.before, &c.after, &c.grad})
            for (const OwnSrc& x : *v) f(x);
    }
}
// The map of a sum: with own, of the variables the plan's units leave to the
// reduction; without, of every variable.
void sum_map(const Model& M, SumKind s, bool own, SegMap& out);
// The plan a mode's launch runs on (nullptr: general units).
const OwnPlan* own_plan(const Model& M, int mode, bool own);

// exa_codegen.cpp
// Component modes of a unit mode (itself for plain modes, jac + hess for JH);
// one-pass units leave out the gradient or H v when own units finish them.
const std::vector<int>& job_modes(const Model& M, int mode);
const std::vector<int>& job_modes(int mode);
#define EXA_BLOCK_MAX 256
bool pattern_in_mode(const Pattern& P, int mode);
// Single-callback launches whose stores can outweigh their reads; only their
// kernels hold code for read-ahead tiles (in the others it costs registers:
// the constraints' kernel of the network model took 102 instead of 74).
inline bool mode_reads_ahead(int mode) { return mode == M_JAC || mode == M_HESS || mode == M_JH; }
// Modes the several-callback kernels evaluate: exa_k_multi (Jacobian and
// Hessian apart) or exa_k_multijh (with Jacobian + Hessian units).
const std::vector<int>& multi_modes(bool jh);
std::vector<Unit> units_for(const Model& M, int mode, bool fused);
// Generated source for all callbacks; fills live[(mode, unit code)].
// ident_flags: per pattern and index column, whether the code may use the
// data point itself (default: each pattern's own flags); hvd_flags: per
// group and H v reference, whether the code may store the reference into
// the output (default: each group's own Group::hv_direct)
std::string generate_source(const Model& M, std::map<std::pair<int, int>, UnitLive>* live = nullptr,
                            const std::vector<std::vector<char>>* ident_flags = nullptr,
                            const std::vector<std::vector<char>>* hvd_flags = nullptr);

// exa_runtime.cpp
// Objective tiles always hold kObjBlock * kObjEpl points (256 virtual lanes
// of 8 points), so the objective's summation order is fixed; its own launch
// uses kObjBlock-wide workgroups.
constexpr int kObjBlock = 256, kObjEpl = 8;
constexpr int64_t kIdentMin = 64;
constexpr bool kObjFused = true;
void build_device(Model& M);
// Device memory a model needs (data columns, tables, work buffers, maps),
// estimated from the host analysis before anything is allocated: as it is, or
// lean (Model::lean).
int64_t estimate_device_bytes(Model& M, bool lean);
// The larger of the two, which any budget has room for.
int64_t estimate_device_bytes(Model& M);

}  // namespace exa

struct exa_model {
    exa::Model impl;
};
