// Device state of a model and the helpers shared by the runtime and batching.
#pragma once
#include <hip/hip_runtime.h>

#include <functional>
#include <map>
#include <memory>
#include <string>
#include <vector>

#include "exa_internal.h"

namespace exa {

struct Module {
    hipModule_t mod = nullptr;
    hipFunction_t fn[M_COUNT] = {};
    hipFunction_t fn_multi = nullptr;    // tiles of several callbacks in one launch (Jacobian and Hessian apart)
    hipFunction_t fn_multijh = nullptr;  // the same with Jacobian + Hessian units
    hipFunction_t fn_onepass = nullptr;  // one pass per point for several callbacks
    std::string source;
    std::vector<char> code;
    ~Module();
};

struct DevMap {
    const void* ptr = nullptr;  // int32 entries unless wide
    const void* idx = nullptr;
    int64_t nseg = 0;
    int wide = 0;
    // chunked sums (see ExaSegJob) for maps with long segments
    int chunked = 0;
    const int32_t* lanes = nullptr;  // 2 per lane: segment, count | chunks << 4
    const int32_t* lidx = nullptr;   // 4 per lane: the chunk's positions
    int64_t nlanes = 0;
    const int32_t* longs = nullptr;
    const int32_t* lpart = nullptr;
    int64_t nparts = 0, nlong = 0;
    int32_t long_len = 0;
    double* lsum = nullptr;
};

struct DeviceState {
    int device = 0;
    std::shared_ptr<Module> module;
    std::vector<void*> allocs;
    std::vector<int64_t> sizes;       // bytes of each allocation
    int64_t allocated = 0;            // bytes allocated now
    int64_t budget = 0;               // 0: no limit; else alloc fails past it (EXA_ENOMEM)
    double* theta = nullptr;
    ExaInstDev* inst = nullptr;       // device copy of the single-instance table
    ExaInstDev inst_host;             // host copy (device pointers), reused by batches
    // schedule of each callback's evaluation kernel
    struct Sched {
        int block = 256, epl = 4;
        bool fused = false, tuned = false;
        bool unstaged = false;  // each lane stores its own output slice (no LDS staging)
        ExaTile* tiles = nullptr;
        int64_t ntiles = 0;
    } sched[M_COUNT];
    // schedule of the several-callback launch, per exa_eval mask
    struct MultiSched {
        int block = 256, epl = 4;
        bool fused = false, tuned = false;
        bool unstaged = false;  // each lane stores its own output slices
        int units = EXA_UNITS_PER_CALLBACK;  // EXA_UNITS_*: which kernel and units run the tiles
        ExaTile* tiles = nullptr;
        int64_t ntiles = 0;
    };
    std::map<uint32_t, MultiSched> multi;
    // HIP events around exa_eval's two launches while timing is on: four per
    // recorded call (evaluation start/end, reduction start/end)
    struct EvalTiming {
        bool on = false;
        std::vector<hipEvent_t> ev;
        std::vector<char> reduced;  // per recorded call: a reduction was launched
        int64_t used = 0;
    } timing;
    void timing_off();
    double* fo = nullptr;             // first-order buffer: grad part, then jac part
    double* par = nullptr;
    double* hv = nullptr;             // H v contributions (curved slots only)
    double* tilesum = nullptr;
    double* lag_tmp = nullptr;  // J^T y of exa_lag_grad (nvar)
    double* fval = nullptr;     // objective of exa_obj_host (device)
    double* fhost = nullptr;    // its pinned host copy
    DevMap csc_map[2];          // uploaded on the first exa_csc_values call
    bool csc_up[2] = {false, false};
    DevMap grad_map, jt_map, h_map, par_map;

    void* alloc(size_t bytes);
    void* upload(const void* src, size_t bytes);
    void release(void* p);
    ~DeviceState();
};

void hip_check(hipError_t e, const char* what);
// The model's own checks of a live (device) model, for entry points in other
// source files: EXA_EINVAL / EXA_ESTATE as the callbacks raise them.
Model& live_model(exa_model* m);
// One callback's evaluation launch under its current schedule (no tuning,
// no allocation).
void launch_mode_untuned(Model& M, int mode, ExaCall call, hipStream_t s);
// The segment sums of a map from `buf` into `out` (one reduction launch,
// plus one for long segments).
void segsum(const DevMap& m, const double* buf, double* out, hipStream_t s, const double* w = nullptr);
exa_status guard_status(const std::function<void()>& f);
// Points per lane of a launch whose schedule nobody has timed, where the
// options leave it open (epl_most, or no epl given): theirs, halved while the launch would have fewer than kFullLaunch workgroups (three
// per compute unit).  With fewer, a tile's points per lane are a serial chain
// of loads on a chip that has room for them side by side.  Measured at 256
// lanes, four points / one point per lane (iterates in turn): 10,000 buses
// Jacobian + Hessian 10.4 / 5.4 us, J^T w 15.2 / 8.6, every callback but the
// objective 30.1 / 14.8; 1354 buses 26.5 / 13.8; trajectory of 10,000 steps
// Hessian 9.6 / 5.4.  From about three per compute unit on more workgroups
// gain nothing: the 1000 x 1000 grid's J^T w (977) 15.6 / 18.2, every callback
// of the 517 x 517 grid (over 2000) 15.5 / 18.0, 300,000 steps 49.3 / 51.3.
constexpr int64_t kFullLaunch = 768;
template <class Tiles>
int untimed_epl(int epl, bool most, const Tiles& tiles) {
    while (most && epl > 1 && tiles(epl) < kFullLaunch) epl /= 2;
    return epl;
}
// Tiles that write zeros to the gradient entries no objective term touches,
// kZeroTileEntries entries each (more when a tile of points is larger).
constexpr int64_t kZeroTileEntries = 4096;
void add_zero_tiles(const Model& M, int64_t tp, std::vector<ExaTile>& tiles);
// Bytes one read-ahead tile covers (EXA_AHEAD_TILE).
constexpr int64_t kAheadBytes = 256 * 1024;
// Inputs of one round of tiles on one XCD (interleave_units).
constexpr int64_t kRoundBytes = 512 * 1024;
// Which inputs beside x a launch of `modes` has: v, y and the J^T w weights.
struct AheadIn {
    bool v = false, y = false, w = false;
};
AheadIn ahead_in(const Model& M, const std::vector<int>& modes);
// Input ranges to be read ahead of some tiles: per array (EXA_AHEAD_* or a
// data column's device address), [first, last) in bytes.
struct Ahead {
    std::map<int64_t, std::vector<std::pair<int64_t, int64_t>>> spans;
    void add(bool has, int64_t slot, int64_t lo, int64_t hi) {
        if (hi > lo && has) spans[slot].emplace_back(lo, hi);
    }
    int64_t bytes() const;  // of their union
    void tiles(int inst, std::vector<ExaTile>& out);  // their union as tiles
};
// Fills ExaMulti::in and inst from the call records.
void multi_inputs(ExaMulti& mc);
// Whether a launch reads ahead: its stores outweigh its reads, and with three
// sets of buffers in turn they sweep the last-level cache (256 MB), so that the
// next iterate's inputs come from HBM.  One set's inputs stay in that cache,
// and the extra workgroups then cost a few per cent.  Every callback, us
// without / with the tiles, three sets in turn and one: the 1,000,000-step
// trajectory 158 / 126 and 103 / 107, its interior-point set 91 / 73 and
// 69 / 70, the 1000 x 1000 grid 63 / 52 and 39 / 38, 64 networks 169 / 145 and
// 121 / 130.  Launches that mostly read, or write less, find their inputs in the
// cache either way, and the workgroups cost them up to 20% (64 networks:
// constraints 23 / 27 us, J v 26 / 32).
inline bool reads_ahead(int64_t in, int64_t out) { return out >= in && out >= (int64_t)96 << 20; }
// Bytes a unit's tiles write as outputs.
int64_t tile_outputs(const Model& M, int mode, const ExaTile* t, size_t n);
void ahead_unit(const Model& M, int mode, const ExaTile* t, size_t n, const AheadIn& has, Ahead& in);
bool has_fusable_group(const Model& M, int mode);
// Modes of an exa_eval mask (with jh: Jacobian + Hessian as JH units), the
// one-pass unit mode covering a mask (or -1), whether a mask has both the
// Jacobian and the Hessian, the units a mask can run as asked, and the modes
// whose tiles make up a mask's launch under those units.
std::vector<int> eval_modes(uint32_t mask, bool jh);
int combined_mode_of(uint32_t mask);
bool has_jh(uint32_t mask);
int valid_units(uint32_t mask, int units);
std::vector<int> launch_modes(const Model& M, uint32_t mask, int units);
// The mode in a tile's code: M_GRADL runs the gradient's units.
inline int tile_mode(int mode) { return mode == M_GRADL ? (int)M_GRAD : mode; }
// Algorithmic bytes of the reduction launch of a mask (maps, buffer entries,
// outputs, objective partials when there are several).
void reduce_bytes(const Model& M, uint32_t mask, int64_t& rd, int64_t& wr);
std::vector<char> compile_code(const std::string& src);
// The code object of a source through the on-disk cache in `dir` (empty: no
// cache); *hit tells whether it was read from the cache.
std::vector<char> cached_code(const std::string& src, const std::string& dir, bool* hit);
// The cache directory: the option's, else $EXA_CACHE_DIR, else none.
std::string cache_dir_of(const char* opt_dir);
// shared: whether a live model had it already.
std::shared_ptr<Module> compile_module(const std::string& src, const std::string& cache_dir, bool* cache_hit,
                                       bool* shared = nullptr);
// One line to stderr when the environment variable EXA_LOG is set (not "0").
bool log_on();
void log_msg(const std::string& msg);
// Tiles of tile_pts points per unit.  With fills, a unit whose code reads
// nothing (constant derivatives only) gets tiles of kZeroTileEntries points
// (the batch, which is throughput-bound); without, only when its tiles
// would far outnumber the workgroups the chip holds at once.
std::vector<ExaTile> make_tiles(const Model& M, int mode, int inst, int64_t tile_pts, bool fused,
                                bool fills = false);
std::string kernel_name(int mode);
int mode_lds_doubles(const Model& M, int mode);
void set_schedule(Model& M, int mode, int block, int epl, bool fused);
// How a map's segments are summed (see ExaSegJob): one lane per segment
// when no segment is longer than 2 * kExaChunk (or positions need 64 bits);
// otherwise parts of kExaLongSeg entries for segments longer than that, and
// for the others chunk lanes, except on large maps whose other segments are
// all short (at most kExaShortSeg entries), where one lane per segment reads
// fewer bytes than a 24-byte lane record per segment.
struct ChunkPlan {
    int32_t long_len = 0;  // segments longer than this have blocks of their own (0: none do)
    int64_t nsplit = 0;    // long segments summed in parts (the others by one workgroup each)
    bool chunked = false;  // chunk lanes (else one lane per segment)
    std::vector<int32_t> meta, lidx;    // 2 and 4 per lane, a multiple of 256 lanes
    std::vector<int32_t> longs, lpart;  // 5 per long segment; 2 per part block
    int64_t nlanes() const { return (int64_t)meta.size() / 2; }
    int64_t nlong() const { return (int64_t)longs.size() / 5; }
    int64_t nparts() const { return (int64_t)lpart.size() / 2; }
};
ChunkPlan chunk_plan(const SegMap& S, bool own = false);
// live: the liveness records of the code that runs (default: the model's own)
void kernel_bytes(const Model& M, const std::vector<int>& modes, bool fused, int64_t& rd, int64_t& wr,
                  const std::map<std::pair<int, int>, UnitLive>* live = nullptr);
// Map and tables of a segment map on the device (int32 when positions fit,
// chunked when segments are long).
void upload_map(DeviceState& D, const SegMap& S, DevMap& d, bool own = false);
// CSC analysis of the Jacobian (which = 0) or Hessian (1) on first use.
Model::Csc& csc_form(Model& M, int which);
void jac_structure_host(const Model& M, int32_t* rows, int32_t* cols);
void hess_structure_host(const Model& M, int32_t* rows, int32_t* cols);
const char* last_error();

}  // namespace exa
