// Host-side internal types of libompd.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <condition_variable>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "../../include/ompd.h"
#include "ompd_device.h"

struct ServingState;

struct ompd_ctx {
    int device = 0;
    hipDeviceProp_t prop{};
    int n_cu = 1;
    int lds_max = 64 * 1024;
    uint64_t budget = 0;
    int64_t wall_khz = 100000;     // device wall-clock rate (s_memrealtime)
    int32_t wait_ticks = 0;        // bound of a kernel wait without progress, in wall-clock ticks
    char* static_scratch = nullptr;   // this device's copy of the allocation-free entry point's scratch
    std::mutex mu;                 // serialises API calls
    ServingState* srv = nullptr;   // created on first submit
    std::mutex srv_mu;
};

// Launch sizes of one solve: slots of the result ring, each phase kernel's
// LDS bytes and grid, and the grid of the pass kernels.
struct LaunchDims {
    int ring_slots = 16;
    bool split = true;           // one kernel per phase and pass (else the per-tile kernel)
    size_t lds[ompd::N_PHASES] = {0, 0, 0, 0, 0, 0};
    int grid[ompd::N_PHASES] = {1, 1, 1, 1, 1, 1};
    bool refine = false;         // some CFG runs the loop-entry refinement (phase and pass launched)
    int grid_edge = 1;
    size_t lds_tile = 0;         // the per-tile kernel: LDS of its largest phase
    int grid_tile = 1;
    int n_walk = 0;              // CFGs on the walk
    // strip schedule
    int n_strip = 0;             // CFGs on it
    int n_level = 0;             // strip tiles: the last n_level entries of the tile array
    int n_tblock = 0, n_tedge = 0;   // transpose items: the last entries of the item array, blocks first
    int prep_threads = 256;      // threads of the strip ingest
    size_t lds_prep = 0;         // LDS of the strip ingest (the largest CFG's peel that fits)
    // launches of each strip kernel: consecutive strip tiles whose workgroups have the same number
    // of wavefronts and whose records hold edge entries in the same way
    struct Bucket { int first, n, waves, by_rows; size_t lds; };
    static constexpr int MAX_BUCKETS = 8;
    int n_buckets = 0;
    bool first_half = false;     // the strips stop after eager validity
    Bucket bucket[MAX_BUCKETS] = {};
};

// Tunable launch configuration of a plan; results never depend on it.
struct PlanConfig {
    size_t lds_bytes = 0;   // bytes of the result ring per phase workgroup (0 = default)
    int wg_per_cu = 0;      // phase workgroups per CU (0 = as many as fit)
    bool split = true;      // one kernel per phase and pass (else one per-tile kernel)
    bool use_graph = true;  // replay a captured HIP graph
    // schedule per size bucket (ompd_sched_bucket): -1 the default rule, else SCHED_WALK or
    // SCHED_LEVEL; CFGs whose schedule the plan's flags name keep it
    int bucket_sched[OMPD_SCHED_BUCKETS] = {-1, -1, -1, -1, -1};
    int only_bucket = -1;   // autotuning: solve only the CFGs of this bucket (-1: all)
    bool roomy = false;     // fail rather than take a smaller layout where memory is short
    bool first_half = false; // the caller reads next use and eager validity only (strips stop there)
};
// Size bucket of a CFG for the schedule choice: blocks below 256, 1,024, 4,096, 16,384, or more.
inline int ompd_sched_bucket(int n_blocks)
{
    return n_blocks < 256 ? 0 : n_blocks < 1024 ? 1 : n_blocks < 4096 ? 2 : n_blocks < 16384 ? 3 : 4;
}

struct ompd_plan {
    ompd_ctx* ctx = nullptr;
    int n = 0;
    uint32_t flags = 0;
    PlanConfig cfg;
    std::vector<ompd::DevCfg> h_cfgs;
    std::vector<ompd_result> res;
    std::vector<int32_t> h_info;
    int32_t* d_info = nullptr;            // [n][INFO_WORDS]: every CFG's status words, gathered for one copy
    ompd::DevCfg* d_cfgs = nullptr;
    std::vector<ompd::Tile> h_tiles;
    ompd::Tile* d_tiles = nullptr;
    int n_tiles = 0;
    ompd::EdgeItem* d_items = nullptr;
    int n_items = 0;
    int32_t* d_counter = nullptr;
    void* scratch = nullptr;
    size_t scratch_bytes = 0;
    int max_nb = 2;
    LaunchDims dims;
    hipGraph_t g_prep = nullptr, g_solve = nullptr;
    hipGraphExec_t gx_prep = nullptr, gx_solve = nullptr;
    hipStream_t last_stream = nullptr;
    hipEvent_t ev0 = nullptr, ev1 = nullptr, ev2 = nullptr;
    bool profile = false;          // launch directly and time every kernel
    hipEvent_t evk[ompd::N_SOLVE_KERNELS] = {};   // after each solve kernel (profile runs)
};

int ompd_fail(int code, const std::string& msg);
// The message for CFG i's info words (status, and for OMPD_E_DEVICE which wait gave up).
std::string ompd_status_message(int i, const int32_t* info);

struct ScratchOff {
    // the walk's arrays
    size_t aveout, mayp, later, flg, eag, both, pp, pi, pe, tmp, recf, recb, stf, stb, lorder, loff;
    // the strips' arrays, in the same bytes (strip: the CFG can take the strip schedule)
    bool strip;
    int rows;    // rows of a pass its lane records have room for
    size_t s_rw, s_1, s_2, s_3, s_g, s_b, s_recf, s_recb, s_link, s_eid, s_erec, s_ebwd, s_xf, s_xb, s_estf, s_estb, s_locf,
        s_locb, s_kc, s_lorder, s_loff, s_pos, s_lastf, s_lastb, s_facts, s_hdr;
    // both schedules
    size_t nu, ave, ie, ig, avf, vk, bnd, fp, info;
};
// Scratch of one CFG, offsets relative to its base.  The strips' arrays take the walk's place; a
// CFG with many edges per block needs more for them, which `rows` grants: at least that many rows of a pass
// in the lane records (0: no more bytes than the walk, or the CFG is left to it).
size_t ompd_cfg_scratch(const ompd_cfg& g, const ompd_result& r, ScratchOff& o, int rows);
void ompd_fill_devcfg(const ompd_cfg& g, const ompd_result& r, char* base, const ScratchOff& o, uint32_t flags,
                      int32_t wait_ticks, ompd::DevCfg& d, uint64_t* bnd_host, uint64_t* bnd_dev = nullptr);
// WANT_* bits of the outputs a caller asked for.
int32_t ompd_want(const ompd_result& r);
// Transpose items of a CFG on the strip schedule.
inline size_t ompd_transpose_items(size_t nb, size_t ne, size_t wd)
{
    const size_t runs = wd ? (wd + ompd::STRIP_T_WORDS - 1) / ompd::STRIP_T_WORDS : 1;
    auto chunks = [](size_t rows) { return (rows + ompd::STRIP_T_ROWS - 1) / ompd::STRIP_T_ROWS; };
    return runs * (chunks(nb) + (wd ? chunks(ne + 1) : 0));
}
int ompd_strip_rows(const ompd_cfg* g, int n, uint32_t flags);
// Settle the schedule of each CFG of a launch (a CFG whose schedule the caller names, or that the
// strips cannot hold, keeps the walk or the strips; the others take the strips, or the walk when
// a launch that fills the GPU asks for the per-tile kernel), and the shape of its strips.
constexpr int STRIP_ANYWAY_BLOCKS = 12288;   // ... and the CFG has fewer blocks than this
void ompd_settle_sched(ompd::DevCfg* h, int n, int n_cu, bool split = true);
// Default bound of a kernel wait without progress (the longest legitimate wait is one step of
// the other wavefront, microseconds).
constexpr int64_t OMPD_WAIT_DEFAULT_NS = 2000000000ll;
// Launch shape of a set of CFGs: tiles (longest first), edge-step items and grids.
struct Shape {
    std::vector<ompd::Tile> tiles;
    std::vector<ompd::EdgeItem> items;
    LaunchDims dims;
};
int ompd_make_shape(ompd_ctx* ctx, const std::vector<ompd::DevCfg>& cfgs, const PlanConfig& pc, Shape& sh);
int ompd_launch_prep(const ompd::DevCfg* d_cfgs, int n, int32_t* d_counter, const LaunchDims& dims, hipStream_t s);
int ompd_launch_solve(const ompd::DevCfg* d_cfgs, const ompd::Tile* d_tiles, int n_tiles, const ompd::EdgeItem* d_items,
                      int n_items, int32_t* d_counter, const LaunchDims& dims, hipStream_t s,
                      hipEvent_t* after = nullptr);
int ompd_plan_build(ompd_ctx* ctx, const ompd_cfg* cfgs, ompd_result* res, int32_t n, uint32_t flags,
                    const PlanConfig& pc, ompd_plan** out);
int ompd_plan_retile(ompd_plan* p, const PlanConfig& pc);
int ompd_plan_run_locked(ompd_plan* p, hipStream_t s);
// Run a plan again whose last run succeeded and whose CFGs have kept their edges, spaces, calls and
// the variables no block may touch (rows, boundaries and summaries may have changed): the ingest's
// tables still hold.
int ompd_plan_rerun_locked(ompd_plan* p, hipStream_t s);
int ompd_plan_collect(ompd_plan* p, int32_t* per_cfg);
int ompd_batch_locked(ompd_ctx* ctx, const ompd_cfg* cfgs, ompd_result* res, int32_t n, uint32_t flags,
                      hipStream_t s);
void ompd_serving_shutdown(ompd_ctx* ctx);
