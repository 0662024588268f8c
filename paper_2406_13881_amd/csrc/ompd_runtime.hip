// Host runtime of libompd: contexts, resident plans (scratch arena, tiles,
// captured HIP graph), the host-pointer batch path and the autotuner.
// The serving loop lives in ompd_serving.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/ompd.h"
#include "ompd_device.h"
#include "ompd_internal.h"

namespace ompd {
extern "C" __global__ void ompd_k_prep(const DevCfg*, int, int32_t*, int);
extern "C" __global__ void ompd_k_nu(const DevCfg*, const Tile*, int, int32_t*, int);
extern "C" __global__ void ompd_k_ave(const DevCfg*, const Tile*, int, int32_t*, int);
extern "C" __global__ void ompd_k_mayp(const DevCfg*, const Tile*, int, int32_t*, int);
extern "C" __global__ void ompd_k_later(const DevCfg*, const Tile*, int, int32_t*, int);
extern "C" __global__ void ompd_k_avf(const DevCfg*, const Tile*, int, int32_t*, int);
extern "C" __global__ void ompd_k_post_ave(const DevCfg*, const Tile*, const EdgeItem*, int, int32_t*);
extern "C" __global__ void ompd_k_post_mayp(const DevCfg*, const Tile*, const EdgeItem*, int, int32_t*);
extern "C" __global__ void ompd_k_post_later(const DevCfg*, const Tile*, const EdgeItem*, int, int32_t*);
extern "C" __global__ void ompd_k_post_avf(const DevCfg*, const Tile*, const EdgeItem*, int, int32_t*);
extern "C" __global__ void ompd_k_live(const DevCfg*, const Tile*, int, int32_t*, int);
extern "C" __global__ void ompd_k_post_live(const DevCfg*, const Tile*, const EdgeItem*, int, int32_t*);
extern "C" __global__ void ompd_k_varkind(const DevCfg*, const Tile*, int, int32_t*);
extern "C" __global__ void ompd_k_solve(const DevCfg*, const Tile*, int, int32_t*, int);
extern "C" __global__ void ompd_k_sprep(const DevCfg*, int, int);
extern "C" __global__ void ompd_k_tin(const DevCfg*, const EdgeItem*);
extern "C" __global__ void ompd_k_strip_a(const DevCfg*, const Tile*);
extern "C" __global__ void ompd_k_tmid(const DevCfg*, const EdgeItem*);
extern "C" __global__ void ompd_k_strip_b(const DevCfg*, const Tile*);
extern "C" __global__ void ompd_k_strip_b_rows(const DevCfg*, const Tile*);
extern "C" __global__ void ompd_k_tout(const DevCfg*, const EdgeItem*);
static const void* const k_phases[N_PHASES] = {(const void*)ompd_k_nu, (const void*)ompd_k_ave,
                                               (const void*)ompd_k_mayp, (const void*)ompd_k_later,
                                               (const void*)ompd_k_avf, (const void*)ompd_k_live};
// threads of a phase workgroup: the compute and the helper wavefront
constexpr int PHASE_THREADS = 128;
}  // namespace ompd

using namespace ompd;

static thread_local std::string g_err;

// Scratch of the allocation-free batch entry point (ompd_analyze_batch_noalloc):
// every device the library runs on holds its own copy, from the first context
// on it until the process ends.  Host code never passes this name to a kernel
// or a copy: it uses the device address that hipGetSymbolAddress returns for
// the current device (ompd_ctx::static_scratch).
constexpr size_t OMPD_STATIC_SCRATCH_BYTES = (size_t)OMPD_NOALLOC_SCRATCH_MIB << 20;
static __device__ __align__(256) char scratch[OMPD_STATIC_SCRATCH_BYTES];
static std::mutex g_scratch_mu[64];   // one caller at a time per device (the scratch is shared)

int ompd_fail(int code, const std::string& msg)
{
    g_err = msg;
    return code;
}

#define CK(x)                                                                                   \
    do {                                                                                        \
        hipError_t e_ = (x);                                                                    \
        if (e_ != hipSuccess)                                                                   \
            return ompd_fail(OMPD_E_DEVICE, std::string(#x) + ": " + hipGetErrorString(e_));    \
    } while (0)

// An allocation: device memory that there is not is OMPD_E_NOMEM, so that a caller can free some
// and call again.
#define CK_MALLOC(x)                                                                            \
    do {                                                                                        \
        hipError_t e_ = (x);                                                                    \
        if (e_ != hipSuccess) {                                                                 \
            (void)hipGetLastError();                                                            \
            return ompd_fail(OMPD_E_NOMEM, std::string(#x) + ": " + hipGetErrorString(e_));     \
        }                                                                                       \
    } while (0)

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
static void drop_graphs(ompd_plan* p);

// ---------------------------------------------------------------------------
// context
// ---------------------------------------------------------------------------
extern "C" int ompd_ctx_create(ompd_ctx** out, int device_ordinal, uint64_t budget)
{
    if (!out) return ompd_fail(OMPD_E_INVAL, "out is NULL");
    int ndev = 0;
    CK(hipGetDeviceCount(&ndev));
    if (device_ordinal < 0 || device_ordinal >= ndev) return ompd_fail(OMPD_E_DEVICE, "no such device");
    ompd_ctx* c = new ompd_ctx();
    c->device = device_ordinal;
    c->budget = budget ? budget : (64ull << 30);
    hipError_t e = hipSetDevice(device_ordinal);
    if (e == hipSuccess) e = hipGetDeviceProperties(&c->prop, device_ordinal);
    if (e != hipSuccess) {
        delete c;
        return ompd_fail(OMPD_E_DEVICE, hipGetErrorString(e));
    }
    c->n_cu = c->prop.multiProcessorCount;
    int khz = 0;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, device_ordinal) == hipSuccess && khz > 0)
        c->wall_khz = khz;
    (void)hipGetLastError();
    c->wait_ticks = (int32_t)std::min<int64_t>(OMPD_WAIT_DEFAULT_NS / 1000 * c->wall_khz / 1000, INT32_MAX);
    // this device's address of the static scratch (the device is current)
    void* sp = nullptr;
    e = hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !sp) {
        delete c;
        return ompd_fail(OMPD_E_DEVICE, std::string("static scratch address: ") + hipGetErrorString(e));
    }
    c->static_scratch = (char*)sp;
    size_t lds_max = c->prop.maxSharedMemoryPerMultiProcessor;
    if (!lds_max) lds_max = c->prop.sharedMemPerBlock;
    lds_max = std::min<size_t>(lds_max ? lds_max : 64 * 1024, 160 * 1024);
    // dynamic LDS limit per kernel = device limit minus the kernel's static LDS
    int dyn = (int)lds_max;
    for (const void* k : {k_phases[0], k_phases[1], k_phases[2], k_phases[3], k_phases[4], k_phases[5],
                          (const void*)ompd_k_prep, (const void*)ompd_k_solve, (const void*)ompd_k_sprep,
                          (const void*)ompd_k_strip_a, (const void*)ompd_k_strip_b, (const void*)ompd_k_strip_b_rows}) {
        hipFuncAttributes fa{};
        int st = 0;
        if (hipFuncGetAttributes(&fa, k) == hipSuccess) st = (int)fa.sharedSizeBytes;
        int want = (int)lds_max - st;
        if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, want) != hipSuccess) {
            (void)hipGetLastError();
            want = std::min(want, 64 * 1024 - st);
        }
        dyn = std::min(dyn, want);
    }
    (void)hipGetLastError();
    c->lds_max = dyn;
    *out = c;
    return OMPD_OK;
}

extern "C" int ompd_set_wait_limit(ompd_ctx* c, int64_t ns)
{
    if (!c) return ompd_fail(OMPD_E_INVAL, "ctx is NULL");
    if (ns < 0) return ompd_fail(OMPD_E_INVAL, "wait limit is negative");
    std::lock_guard<std::mutex> lk(c->mu);
    if (ns == 0) ns = OMPD_WAIT_DEFAULT_NS;
    const int64_t t = ns / 1000 * c->wall_khz / 1000 + (ns % 1000) * c->wall_khz / 1000000;
    c->wait_ticks = (int32_t)std::max<int64_t>(1, std::min<int64_t>(t, INT32_MAX));
    return OMPD_OK;
}

extern "C" void ompd_ctx_destroy(ompd_ctx* c)
{
    if (!c) return;
    ompd_serving_shutdown(c);
    delete c;
}

extern "C" const char* ompd_last_error(const ompd_ctx*) { return g_err.c_str(); }

extern "C" int ompd_device_info(ompd_ctx* c, int32_t* n_cu, int32_t* lds_bytes, int64_t* mem_bytes)
{
    if (!c) return ompd_fail(OMPD_E_INVAL, "ctx is NULL");
    if (n_cu) *n_cu = c->n_cu;
    if (lds_bytes) *lds_bytes = c->lds_max;
    if (mem_bytes) *mem_bytes = (int64_t)c->prop.totalGlobalMem;
    return OMPD_OK;
}

// ---------------------------------------------------------------------------
// tile rules
// ---------------------------------------------------------------------------
// Cut one CFG into tiles: ceil(wd / TILE_WORDS) runs of words, split evenly.
static void make_tiles(int ci, int nv, std::vector<Tile>& out)
{
    int wd = (nv + 63) / 64;
    int t = tiles_of(wd);
    if (wd == 0) {
        out.push_back(Tile{ci, 0, 0, 0});
        return;
    }
    int s0 = 0;
    for (int k = 0; k < t; ++k) {
        int n = wd / t + (k < wd % t ? 1 : 0);
        out.push_back(Tile{ci, s0, n, k});
        s0 += n;
    }
}

// ---------------------------------------------------------------------------
// plan
// ---------------------------------------------------------------------------
static int check_cfg_host(const ompd_cfg& g, int i)
{
    char buf[160];
    auto bad = [&](const char* why) {
        snprintf(buf, sizeof buf, "cfg %d: %s", i, why);
        return ompd_fail(OMPD_E_INVAL, buf);
    };
    if (g.n_blocks < 2) return bad("n_blocks < 2");
    if (g.n_edges < 0 || g.n_vars < 0) return bad("negative size");
    if (g.entry < 0 || g.entry >= g.n_blocks || g.exit < 0 || g.exit >= g.n_blocks || g.entry == g.exit)
        return bad("entry/exit out of range");
    if (!g.succ_ptr || !g.space) return bad("succ_ptr/space missing");
    if (g.n_edges > 0 && (!g.succ_idx || !g.edge_kind)) return bad("succ_idx/edge_kind missing");
    if (g.n_vars > 0 && (!g.read_bits || !g.write_bits)) return bad("read/write bits missing");
    if (g.call_summary && (g.n_summaries <= 0 || !g.summaries)) return bad("call summaries missing");
    return OMPD_OK;
}

size_t ompd_cfg_scratch(const ompd_cfg& g, const ompd_result& r, ScratchOff& o, int rows)
{
    size_t total = 0;
    auto take = [&](size_t bytes) { size_t x = total; total += align256(bytes); return x; };
    const size_t wd = (size_t)(g.n_vars + 63) / 64, nb = (size_t)g.n_blocks, ne = (size_t)g.n_edges;
    const size_t bv = nb * wd * 8, ev = ne * wd * 8;
    o.aveout = take(2 * bv);
    o.mayp = take(2 * bv);
    o.later = take(2 * bv);
    o.eag = take(2 * ev);
    o.both = take(ev);
    o.flg = take((size_t)tiles_of((int)wd) * 4 * nb * 8);
    o.pp = take(4 * (nb + 1));
    o.pi = take(4 * std::max<size_t>(ne, 1));
    o.pe = take(4 * std::max<size_t>(ne, 1));
    o.tmp = take(4 * (nb + 1));
    o.recf = take(32 * nb);
    o.recb = take(32 * nb);
    o.stf = take(32 * nb);
    o.stb = take(32 * nb);
    o.lorder = take(4 * nb);
    o.loff = take(4 * (nb + 1));
    const size_t walk = total;
    total = 0;
    auto put = [&](size_t bytes) { size_t x = total; total += (bytes + 63) & ~(size_t)63; return x; };
    const size_t units = wd + 1, nrec = (size_t)strip_records(g.n_edges);
    o.rows = std::max(rows, 4 / strip_units(g.n_blocks, (int)wd));
    const size_t recs = 128 * nb * o.rows;   // (at most a pass per block)
    o.s_rw = put(16 * units * nb);
    o.s_1 = put(16 * units * nb);
    o.s_2 = put(16 * units * nb);
    o.s_3 = put(16 * units * nb);
    o.s_g = put(16 * wd * nrec);
    o.s_b = put(8 * wd * nrec);
    o.s_recf = put(recs);
    o.s_recb = put(recs);
    o.s_link = put(4 * nrec);
    o.s_eid = put(4 * nrec);
    o.s_erec = put(4 * ne);
    o.s_ebwd = put(ne >= STRIP_ROW_EDGES ? 4 * nrec : 0);
    o.s_xf = put(4 * (ne + 2));
    o.s_xb = put(4 * (ne + 2));
    o.s_estf = put(4 * (nb + 1));
    o.s_estb = put(4 * (nb + 1));
    o.s_locf = put(4 * nb);
    o.s_locb = put(4 * nb);
    o.s_kc = put(4 * (nb + 1));
    o.s_lorder = put(4 * nb);
    o.s_loff = put(4 * (nb + 1));
    o.s_pos = put(2 * nb);
    o.s_lastf = put(2 * nb);
    o.s_lastb = put(2 * nb);
    o.s_facts = put(nb);
    o.s_hdr = put(4 * SH_WORDS);
    o.strip = nb <= (size_t)STRIP_MAX_BLOCKS && ne <= (size_t)STRIP_MAX_EDGES && (rows > 0 || total <= walk);
    total = align256(o.strip ? std::max(walk, total) : walk);
    o.nu = (r.nu_host && r.nu_dev) ? SIZE_MAX : take(2 * bv);
    o.ave = (r.ave_host && r.ave_dev) ? SIZE_MAX : take(2 * bv);
    o.ie = (r.ins_entry_to_host && r.ins_entry_to_dev) ? SIZE_MAX : take(2 * bv);
    o.ig = (r.ins_edge_to_host && r.ins_edge_to_dev) ? SIZE_MAX : take(2 * ev);
    o.avf = (!r.avf_host == !r.avf_dev) ? SIZE_MAX : take(2 * bv);
    o.vk = r.var_kind ? take(4 * wd * 8) : SIZE_MAX;
    o.fp = take(wd * 8 + 8);
    o.bnd = take(4 * wd * 8);
    o.info = take(4 * INFO_WORDS);
    return total;
}

int32_t ompd_want(const ompd_result& r)
{
    return (r.nu_host ? WANT_NU_H : 0) | (r.nu_dev ? WANT_NU_D : 0) | (r.ave_host ? WANT_AVE_H : 0) |
           (r.ave_dev ? WANT_AVE_D : 0) | (r.avf_host ? WANT_AVF_H : 0) | (r.avf_dev ? WANT_AVF_D : 0) |
           (r.ins_entry_to_host ? WANT_IE_H : 0) | (r.ins_entry_to_dev ? WANT_IE_D : 0) |
           (r.ins_edge_to_host ? WANT_IG_H : 0) | (r.ins_edge_to_dev ? WANT_IG_D : 0);
}

// Rows of a pass for a launch.  A pass holds 4 rows of 16 lanes: one row of edges for 4 words of
// variables does the least work per word, 4 rows for one word the fewest passes.  A lone CFG of 8002
// blocks and 24 words solves in 3.1 ms with one row, 2.6 ms with four; 1024 CFGs (4266 strips of 4
// words) in 12.1 ms with one row, 16.4 ms with two, 27.2 ms with four.
int ompd_strip_rows(const ompd_cfg* g, int n, uint32_t flags)
{
    if (flags & OMPD_F_SCHED_WALK) return 0;   // (no room for what the walk does not use)
    int64_t words = 0;
    for (int i = 0; i < n; ++i) words += (g[i].n_vars + 63) / 64 + 1;
    return words <= 64 ? 4 : words <= 256 ? 2 : 1;
}

void ompd_settle_sched(DevCfg* h, int n, int n_cu, bool split)
{
    std::vector<int> order(n);
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return h[a].nb > h[b].nb; });
    for (int i = 0; i < n; ++i) h[i].by_size = order[i];
    auto strips_of = [](const DevCfg& d) -> int64_t { return (d.wd + d.units) / d.units; };
    int64_t strips = 0;
    for (int i = 0; i < n; ++i)
        if (h[i].sched_rule ? h[i].strip_ok : h[i].sched == SCHED_LEVEL) strips += strips_of(h[i]);
    // Who asks for the per-tile kernel gets it, on the walk, where the launch fills the GPU.  One that
    // leaves it idle, and a large CFG, take the strips all the same (us, strips / per-tile kernel alone:
    // 66 blocks 239 / 573, 2002 blocks x 300 variables 845 / 16,347, 14002 x 300 3,333 / 118,526).
    if (!split) {
        const bool room = strips <= n_cu;
        strips = 0;
        for (int i = 0; i < n; ++i) {
            DevCfg& d = h[i];
            if (d.sched_rule) d.sched = d.strip_ok && (room || d.nb >= STRIP_ANYWAY_BLOCKS) ? SCHED_LEVEL : SCHED_WALK;
            if (d.sched == SCHED_LEVEL) strips += strips_of(d);
        }
    } else
        for (int i = 0; i < n; ++i)
            if (h[i].sched_rule) h[i].sched = h[i].strip_ok ? SCHED_LEVEL : SCHED_WALK;
    // Blocks per wavefront: the fewer, the shorter a strip's chain of passes, and the more rounds
    // until what one wavefront changed has reached the others.  While the GPU has room for every
    // strip at once (a workgroup each) 32 blocks and up to 8 wavefronts are best; where strips queue
    // for the compute units, their total work counts and longer runs cost less, and 4 wavefronts:
    // 8 of them fill a compute unit's registers, which idles while they wait for each other, where
    // two workgroups of 4 fill each other's waits.  Solve kernels, us, at 32 / 64 / 200 / 400 blocks
    // and up to 8 wavefronts: a lone CFG of 66 blocks 163 / 185 / 257 / 257, of 779 blocks 579 / 579 /
    // 625 / 1060; 96 CFGs (242 strips) 1415 / 1795 / 3020 / 4420; 2048 CFGs of about 60 blocks (2377
    // strips) 1170 / 841 / 493 / 493.  1024 CFGs (4266 strips) at 200 blocks: up to 8 wavefronts
    // 12.2 ms, 4 9.9 ms, 2 10.6 ms.  (All measured before cross links read the states of the round
    // before, which adds 4-11 %.)
    const bool idle = strips <= n_cu;
    const int busy_per = (int)std::min<int64_t>(200, 32 * strips / std::max(n_cu, 1));
    int most = 1;
    for (int i = 0; i < n; ++i) {
        DevCfg& d = h[i];
        d.spread = d.sched == SCHED_LEVEL && idle;
        const int per = d.spread ? 32 : std::max(32, busy_per), limit = idle ? STRIP_MAX_WAVES : STRIP_BUSY_WAVES;
        // (a caller's sweep cap counts sweeps in which each block sees what comes before it, as the walk
        // does: one run of passes.  Several see each other's results a round late and take more rounds,
        // 10 where the walk takes 4 on CFGs of 66 blocks, and would stop calls that the walk finishes)
        d.waves = 1;
        if (d.sweep_cap == 0)
            while (d.waves < limit && d.nb > per * d.waves) d.waves *= 2;
        if (d.sched == SCHED_LEVEL) most = std::max(most, d.waves);
    }
    // One launch holds strips of one wavefront count, and two launches take the longest of each in
    // turn.  So all take the largest CFG's count while the GPU has room for every strip (a small CFG
    // with more wavefronts than it likes still ends first), or where the CFGs that would rather have
    // fewer are at most a quarter of the work (the 1024 CFGs: 9.9 ms in three launches, 9.3 in one).
    int64_t work = 0, less = 0;
    auto takes_most = [&](const DevCfg& d) { return d.sched == SCHED_LEVEL && d.sweep_cap == 0; };
    for (int i = 0; i < n; ++i)
        if (takes_most(h[i])) {
            const int64_t k = (int64_t)((h[i].wd + h[i].units) / h[i].units) * h[i].nb;
            work += k;
            if (h[i].waves < most) less += k;
        }
    if (idle || 4 * less <= work)
        for (int i = 0; i < n; ++i)
            if (takes_most(h[i])) h[i].waves = most;
}

// Fill the kernels' descriptor of one CFG whose scratch starts at `base`.
// Default boundary values (for NULL boundaries) are written to bnd_host
// ([4*wd] words: entry valid H, D, exit live H, D), to be copied by the
// caller to bnd_dev (default: base + o.bnd), where the descriptor points.
void ompd_fill_devcfg(const ompd_cfg& g, const ompd_result& r, char* base, const ScratchOff& o, uint32_t flags,
                      int32_t wait_ticks, DevCfg& d, uint64_t* bnd_host, uint64_t* bnd_dev)
{
    int wd = (g.n_vars + 63) / 64;
    memset(&d, 0, sizeof d);
    d.wait_ticks = wait_ticks > 0 ? wait_ticks : 1;
    d.nb = g.n_blocks; d.ne = g.n_edges; d.nv = g.n_vars; d.entry = g.entry; d.exit = g.exit; d.wd = wd;
    d.n_sums = g.call_summary ? g.n_summaries : 0;
    d.placement = ((flags & OMPD_F_PLACEMENT_EAGER) ? PL_EAGER : 0) | ((flags & OMPD_F_SUMMARY) ? PL_SUMMARY : 0) |
                  ((flags & OMPD_F_PLACEMENT_LAZY) ? PL_LAZY : 0) | ((flags & OMPD_F_PLACEMENT_REFINE) ? PL_REFINE : 0);
    d.sweep_cap = (int)((flags >> 16) & 0xFFFFu);
    d.strip_ok = o.strip;
    d.by_rows = g.n_edges >= STRIP_ROW_EDGES;
    d.sched_rule = !(flags & (OMPD_F_SCHED_LEVEL | OMPD_F_SCHED_WALK));
    d.sched = o.strip && !(flags & OMPD_F_SCHED_WALK) ? SCHED_LEVEL : SCHED_WALK;
    d.units = 4 / o.rows;
    d.waves = 1;
    d.succ_ptr = g.succ_ptr; d.succ_idx = g.succ_idx; d.kind = g.edge_kind; d.space = g.space;
    d.R = g.read_bits; d.W = g.write_bits;
    uint64_t* bnd = bnd_dev ? bnd_dev : (uint64_t*)(base + o.bnd);
    d.ev_h = g.entry_valid_host ? g.entry_valid_host : bnd;
    d.ev_d = g.entry_valid_dev ? g.entry_valid_dev : bnd + wd;
    d.lx_h = g.exit_live_host ? g.exit_live_host : bnd + 2 * wd;
    d.lx_d = g.exit_live_dev ? g.exit_live_dev : bnd + 3 * wd;
    d.call = g.call_summary; d.sums = g.summaries;
    d.scalar = g.scalar;
    d.fp = (uint64_t*)(base + o.fp);
    d.fpc = r.fp_clause;
    size_t bvw = (size_t)g.n_blocks * wd, evw = (size_t)g.n_edges * wd;
    auto at = [&](size_t off) { return off == SIZE_MAX ? (uint64_t*)nullptr : (uint64_t*)(base + off); };
    uint64_t *nu = at(o.nu), *ave = at(o.ave), *ie = at(o.ie), *ig = at(o.ig), *avf = at(o.avf);
    // a requested half is written in place; a missing half goes to scratch
    d.nu_h = r.nu_host ? r.nu_host : nu;               d.nu_d = r.nu_dev ? r.nu_dev : nu + bvw;
    d.ave_h = r.ave_host ? r.ave_host : ave;           d.ave_d = r.ave_dev ? r.ave_dev : ave + bvw;
    d.ie_h = r.ins_entry_to_host ? r.ins_entry_to_host : ie;
    d.ie_d = r.ins_entry_to_dev ? r.ins_entry_to_dev : ie + bvw;
    d.ig_h = r.ins_edge_to_host ? r.ins_edge_to_host : ig;
    d.ig_d = r.ins_edge_to_dev ? r.ins_edge_to_dev : ig + evw;
    if (r.avf_host || r.avf_dev) {
        d.avf_h = r.avf_host ? r.avf_host : avf;
        d.avf_d = r.avf_dev ? r.avf_dev : avf + bvw;
    }
    d.var_kind = r.var_kind; d.after_dev = r.after_dev; d.before_dev = r.before_dev;
    uint64_t* ao = at(o.aveout);
    uint64_t* mp = at(o.mayp);
    uint64_t* la = at(o.later);
    d.aveout_h = ao; d.aveout_d = ao + bvw; d.mayp_h = mp; d.mayp_d = mp + bvw;
    d.later_h = la; d.later_d = la + bvw;
    uint64_t* ea = at(o.eag);
    d.eag_h = ea; d.eag_d = ea + evw; d.both = at(o.both);
    d.flg = at(o.flg);
    d.vk_acc = at(o.vk);
    d.pred_ptr = (int32_t*)(base + o.pp); d.pred_idx = (int32_t*)(base + o.pi);
    d.pred_eid = (int32_t*)(base + o.pe); d.tmp = (int32_t*)(base + o.tmp);
    d.rec_f = (int32_t*)(base + o.recf); d.rec_b = (int32_t*)(base + o.recb);
    d.step_f = (int32_t*)(base + o.stf); d.step_b = (int32_t*)(base + o.stb);
    d.lorder = (int32_t*)(base + o.lorder); d.loff = (int32_t*)(base + o.loff);
    d.want = ompd_want(r);
    // (the final validity behind a call reads next use by rows)
    if (g.call_summary) d.want |= WANT_NU_H | WANT_NU_D;
    auto u64p = [&](size_t off) { return (uint64_t*)(base + off); };
    auto u32p = [&](size_t off) { return (uint32_t*)(base + off); };
    auto i32p = [&](size_t off) { return (int32_t*)(base + off); };
    auto u16p = [&](size_t off) { return (uint16_t*)(base + off); };
    d.p_rw = u64p(o.s_rw); d.p_1 = u64p(o.s_1); d.p_2 = u64p(o.s_2); d.p_3 = u64p(o.s_3);
    d.p_g = u64p(o.s_g); d.p_b = u64p(o.s_b);
    d.rec_sf = u32p(o.s_recf); d.rec_sb = u32p(o.s_recb);
    d.link = u32p(o.s_link); d.eid = i32p(o.s_eid); d.erec = i32p(o.s_erec); d.ebwd = i32p(o.s_ebwd);
    d.x_f = u32p(o.s_xf); d.x_b = u32p(o.s_xb);
    d.est_f = i32p(o.s_estf); d.est_b = i32p(o.s_estb);
    d.loc_f = u32p(o.s_locf); d.loc_b = u32p(o.s_locb);
    d.pos = u16p(o.s_pos); d.last_f = u16p(o.s_lastf); d.last_b = u16p(o.s_lastb);
    d.s_kc = i32p(o.s_kc); d.s_lorder = i32p(o.s_lorder); d.s_loff = i32p(o.s_loff);
    d.facts = (uint8_t*)(base + o.s_facts);
    d.hdr = i32p(o.s_hdr);
    d.info = i32p(o.info);
    if (bnd_host && wd > 0) {
        uint64_t last = (g.n_vars & 63) ? ((1ull << (g.n_vars & 63)) - 1) : ~0ull;
        for (int w = 0; w < 4 * wd; ++w) bnd_host[w] = 0;
        for (int w = 0; w < wd; ++w) {
            uint64_t m = (w == wd - 1) ? last : ~0ull;
            bnd_host[w] = m;            // entry valid on the host
            bnd_host[2 * wd + w] = m;   // live on the host after exit
        }
    }
}

// Default result ring of one phase workgroup (recently computed blocks, STATE_BYTES each).
constexpr size_t RING_BYTES_DEFAULT = 64 * STATE_BYTES;

// Tiles for a set of CFGs, longest first, the edge-step items and the launch
// sizes that go with them under a configuration.
int ompd_make_shape(ompd_ctx* ctx, const std::vector<DevCfg>& cfgs, const PlanConfig& pc, Shape& sh)
{
    std::vector<Tile>& tiles = sh.tiles;
    tiles.clear();
    sh.items.clear();
    auto in_plan = [&](int i) { return pc.only_bucket < 0 || ompd_sched_bucket(cfgs[i].nb) == pc.only_bucket; };
    for (int i = 0; i < (int)cfgs.size(); ++i)
        if (in_plan(i) && cfgs[i].sched != SCHED_LEVEL) make_tiles(i, cfgs[i].nv, tiles);
    // a tile's work ~ its blocks times the sweeps, which grow with the CFG: longest first
    std::stable_sort(tiles.begin(), tiles.end(),
                     [&](const Tile& a, const Tile& b) { return cfgs[a.cfg].nb > cfgs[b.cfg].nb; });
    const int walk_tiles = (int)tiles.size();
    LaunchDims& dm = sh.dims;
    // strip tiles (after the walk tiles), launch by launch: CFGs with the same wavefronts and records
    // of the same kind, the ones that need most time first
    {
        std::vector<int> order;
        dm.n_walk = dm.n_strip = 0;
        for (int i = 0; i < (int)cfgs.size(); ++i) {
            if (cfgs[i].sched != SCHED_LEVEL) { ++dm.n_walk; continue; }
            ++dm.n_strip;
            if (in_plan(i)) order.push_back(i);
        }
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
            if (cfgs[a].waves != cfgs[b].waves) return cfgs[a].waves > cfgs[b].waves;
            if (cfgs[a].by_rows != cfgs[b].by_rows) return cfgs[a].by_rows > cfgs[b].by_rows;
            return cfgs[a].nb > cfgs[b].nb;
        });
        dm.n_buckets = 0;
        for (int i : order) {
            const DevCfg& d = cfgs[i];
            if (!dm.n_buckets || dm.bucket[dm.n_buckets - 1].waves != d.waves ||
                dm.bucket[dm.n_buckets - 1].by_rows != d.by_rows)
                dm.bucket[dm.n_buckets++] = LaunchDims::Bucket{(int)tiles.size() - walk_tiles, 0, d.waves, d.by_rows, 0};
            LaunchDims::Bucket& k = dm.bucket[dm.n_buckets - 1];
            for (int u = 0; u <= d.wd; u += d.units) {
                tiles.push_back(Tile{i, u, std::min(d.units, d.wd + 1 - u), 0});
                ++k.n;
            }
            k.lds = std::max(k.lds, strip_lds(d.nb, d.waves));
        }
    }
    dm.n_level = (int)tiles.size() - walk_tiles;
    dm.first_half = pc.first_half;
    int max_nb = 0;
    // pass items: runs of up to PASS_WORDS words (the passes need no LDS, so a full wavefront of
    // words each), 64-block chunks, longest CFGs first
    {
        std::vector<int> order(cfgs.size());
        for (int i = 0; i < (int)order.size(); ++i) order[i] = i;
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cfgs[a].nb > cfgs[b].nb; });
        for (int i : order) {
            const int wd = cfgs[i].wd;
            if (wd <= 0 || !in_plan(i) || cfgs[i].sched == SCHED_LEVEL) continue;
            const int runs = (wd + PASS_WORDS - 1) / PASS_WORDS;
            for (int r = 0; r < runs; ++r) {
                const int s0 = (int)((int64_t)wd * r / runs), s1 = (int)((int64_t)wd * (r + 1) / runs);
                for (int b0 = 0; b0 < cfgs[i].nb; b0 += 64) sh.items.push_back(EdgeItem{i, s0, s1 - s0, b0});
            }
        }
        max_nb = order.empty() ? 0 : cfgs[order[0]].nb;
        // transpose items of the strip CFGs: block chunks, then record chunks
        dm.n_tblock = dm.n_tedge = 0;
        dm.lds_prep = 0;
        for (int edges = 0; edges < 2; ++edges)
            for (int i : order) {
                const DevCfg& d = cfgs[i];
                if (d.sched != SCHED_LEVEL || !in_plan(i)) continue;
                for (size_t pl : {strip_prep_lds(d.nb, d.ne), strip_prep_lds(d.nb, 0)})
                    if (pl <= (size_t)ctx->lds_max) {
                        dm.lds_prep = std::max(dm.lds_prep, pl);
                        break;
                    }
                if (edges && d.wd == 0) continue;
                const int rows = edges ? strip_records(d.ne) : d.nb;
                for (int s0 = 0; s0 < std::max(d.wd, 1); s0 += STRIP_T_WORDS)
                    for (int r = 0; r < rows; r += STRIP_T_ROWS) {
                        sh.items.push_back(EdgeItem{i, s0, std::min(STRIP_T_WORDS, d.wd - s0), edges ? ~r : r});
                        ++(edges ? dm.n_tedge : dm.n_tblock);
                    }
            }
    }
    // Threads of the strip ingest: what follows the peel is by block and by level, each a few dependent
    // loads from L2 (8002 blocks: 570 us of 256 threads, 220 us of 1024); a small CFG has no work for more
    // than 256, and a workgroup's barriers and start cost more with them.
    dm.prep_threads = max_nb < 200 ? 256 : max_nb < 1000 ? 512 : 1024;
    // result ring: a power of two of STATE_BYTES slots in [8, 64], as large as every phase's LDS allows
    const size_t want = pc.lds_bytes ? pc.lds_bytes : RING_BYTES_DEFAULT;
    int rs = 8;
    while (rs < 64 && (size_t)(2 * rs) * STATE_BYTES <= want) rs *= 2;
    while (rs > 1 && phase_lds(PH_LATER, rs) > (size_t)ctx->lds_max) rs /= 2;
    dm.ring_slots = rs;
    // each phase kernel: as many workgroups as it keeps resident
    for (int ph = 0; walk_tiles && ph < N_PHASES; ++ph) {
        dm.lds[ph] = phase_lds(ph, rs);
        int n = 0;
        CK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_phases[ph], PHASE_THREADS, dm.lds[ph]));
        n = std::max(1, n);
        if (pc.wg_per_cu > 0) n = std::min(n, pc.wg_per_cu);
        dm.grid[ph] = std::max(1, std::min(walk_tiles, n * ctx->n_cu));
    }
    dm.split = pc.split;
    dm.lds_tile = 0;
    for (int ph = 0; ph < N_PHASES; ++ph) dm.lds_tile = std::max(dm.lds_tile, dm.lds[ph]);
    dm.refine = false;
    for (int i = 0; i < (int)cfgs.size(); ++i)
        dm.refine |= in_plan(i) && cfgs[i].sched != SCHED_LEVEL && refines(cfgs[i].placement);
    if (walk_tiles) {
        int n = 0;
        CK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void*)ompd_k_solve, PHASE_THREADS, dm.lds_tile));
        n = std::max(1, n);
        if (pc.wg_per_cu > 0) n = std::min(n, pc.wg_per_cu);
        dm.grid_tile = std::max(1, std::min(walk_tiles, n * ctx->n_cu));
    }
    if (dm.n_level) dm.split = true;   // the per-tile kernel does not run strip tiles
    if (!walk_tiles) return OMPD_OK;
    int pe = 1;
    CK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&pe, (const void*)ompd_k_post_ave, 64, 0));
    dm.grid_edge = std::max(1, std::min((int)std::max<size_t>(sh.items.size() - dm.n_tblock - dm.n_tedge, walk_tiles),
                                        std::max(1, pe) * ctx->n_cu));
    return OMPD_OK;
}

int ompd_plan_build(ompd_ctx* ctx, const ompd_cfg* cfgs, ompd_result* res, int32_t n, uint32_t flags,
                    const PlanConfig& pc, ompd_plan** out)
{
    if (!ctx || !out || n < 0 || (n > 0 && !cfgs)) return ompd_fail(OMPD_E_INVAL, "bad arguments");
    for (int i = 0; i < n; ++i) {
        int rc = check_cfg_host(cfgs[i], i);
        if (rc) return rc;
    }
    CK(hipSetDevice(ctx->device));
    ompd_plan* p = new ompd_plan();
    p->ctx = ctx;
    p->n = n;
    p->flags = flags;
    p->cfg = pc;
    if (flags & OMPD_F_TILE_KERNEL) p->cfg.split = false;
    if (const uint32_t r = (flags >> 8) & 7u) p->cfg.lds_bytes = (size_t)(4u << r) * STATE_BYTES;   // 8 .. 64 slots
    p->res.assign(res, res + n);
    p->h_cfgs.resize(n);

    std::vector<ScratchOff> off(n);
    std::vector<size_t> base(n);
    // default boundaries of every CFG, side by side (one upload)
    std::vector<size_t> boff(n);
    size_t bnd_words = 0, counter_off = 0, bnd_off = 0, total = 0;
    int max_nb = 2;
    for (int i = 0; i < n; ++i) {
        boff[i] = bnd_words;
        bnd_words += 4 * (size_t)((cfgs[i].n_vars + 63) / 64);
        max_nb = std::max(max_nb, cfgs[i].n_blocks);
    }
    // (a plan that does not fit with the room the strips like may still fit without)
    hipError_t e = hipSuccess;
    for (int rows : {ompd_strip_rows(cfgs, n, flags), 0}) {
        total = 0;
        for (int i = 0; i < n; ++i) {
            base[i] = total;
            total += ompd_cfg_scratch(cfgs[i], res[i], off[i], rows);
        }
        counter_off = total;
        total += 256;
        bnd_off = total;
        total += (8 * bnd_words + 255) & ~(size_t)255;
        e = hipMalloc(&p->scratch, std::max<size_t>(total, 256));
        if (e == hipSuccess) break;
        p->scratch = nullptr;
        (void)hipGetLastError();
        if (pc.roomy) break;
    }
    p->scratch_bytes = total;
    if (e != hipSuccess) {
        delete p;
        return ompd_fail(OMPD_E_NOMEM, std::string("scratch allocation: ") + hipGetErrorString(e));
    }
    char* S = (char*)p->scratch;
    p->d_counter = (int32_t*)(S + counter_off);
    std::vector<uint64_t> bnd(std::max<size_t>(bnd_words, 1), 0);
    uint64_t* bnd_dev = (uint64_t*)(S + bnd_off);
    for (int i = 0; i < n; ++i)
        ompd_fill_devcfg(cfgs[i], res[i], S + base[i], off[i], flags, ctx->wait_ticks, p->h_cfgs[i], bnd.data() + boff[i],
                         bnd_dev + boff[i]);
    if (bnd_words) {
        e = hipMemcpy(bnd_dev, bnd.data(), 8 * bnd_words, hipMemcpyHostToDevice);
        if (e != hipSuccess) { ompd_plan_destroy(p); return ompd_fail(OMPD_E_DEVICE, hipGetErrorString(e)); }
    }
    p->max_nb = max_nb;
    p->h_info.assign((size_t)n * INFO_WORDS, 0);
    auto tables = [&]() -> int {
        CK_MALLOC(hipMalloc(&p->d_cfgs, sizeof(DevCfg) * std::max(n, 1)));   // (filled by ompd_plan_retile)
        CK_MALLOC(hipMalloc(&p->d_info, 4 * INFO_WORDS * (size_t)std::max(n, 1)));
        return ompd_plan_retile(p, p->cfg);
    };
    const int rc = tables();
    if (rc) { ompd_plan_destroy(p); return rc; }
    CK(hipEventCreate(&p->ev0));
    CK(hipEventCreate(&p->ev1));
    CK(hipEventCreate(&p->ev2));
    *out = p;
    return OMPD_OK;
}

// (Re)build tiles and launch shapes for a configuration (drops captured graphs).  The plan changes
// only once everything new is in device memory and its last run is over: on an error it stays as it
// was.
int ompd_plan_retile(ompd_plan* p, const PlanConfig& pc)
{
    ompd_ctx* ctx = p->ctx;
    // the schedule of each CFG the plan's flags leave open: the bucket's choice, else the rule
    std::vector<DevCfg> cfgs = p->h_cfgs;
    for (DevCfg& d : cfgs) {
        if (p->flags & (OMPD_F_SCHED_LEVEL | OMPD_F_SCHED_WALK)) break;
        const int want = pc.bucket_sched[ompd_sched_bucket(d.nb)];
        d.sched_rule = want < 0;
        if (want >= 0) d.sched = d.strip_ok ? want : SCHED_WALK;
    }
    ompd_settle_sched(cfgs.data(), p->n, ctx->n_cu, pc.split);
    Shape sh;
    int rc = ompd_make_shape(ctx, cfgs, pc, sh);
    if (rc) return rc;
    struct Tables {
        Tile* tiles = nullptr;
        EdgeItem* items = nullptr;
        ~Tables()
        {
            if (tiles) (void)hipFree(tiles);
            if (items) (void)hipFree(items);
        }
    } t;
    CK_MALLOC(hipMalloc(&t.tiles, sizeof(Tile) * std::max<size_t>(sh.tiles.size(), 1)));
    CK_MALLOC(hipMalloc(&t.items, sizeof(EdgeItem) * std::max<size_t>(sh.items.size(), 1)));
    if (!sh.tiles.empty()) CK(hipMemcpy(t.tiles, sh.tiles.data(), sizeof(Tile) * sh.tiles.size(), hipMemcpyHostToDevice));
    if (!sh.items.empty()) CK(hipMemcpy(t.items, sh.items.data(), sizeof(EdgeItem) * sh.items.size(), hipMemcpyHostToDevice));
    if (p->ev2) CK(hipEventSynchronize(p->ev2));   // (the last run, on whatever stream, reads the descriptors)
    if (p->n) CK(hipMemcpy(p->d_cfgs, cfgs.data(), sizeof(DevCfg) * p->n, hipMemcpyHostToDevice));
    drop_graphs(p);
    std::swap(p->d_tiles, t.tiles);
    std::swap(p->d_items, t.items);
    p->h_cfgs.swap(cfgs);
    p->cfg = pc;
    p->dims = sh.dims;
    p->n_tiles = (int)sh.tiles.size();
    p->n_items = (int)sh.items.size();
    p->h_tiles.swap(sh.tiles);
    return OMPD_OK;
}

int ompd_launch_prep(const DevCfg* d_cfgs, int n, int32_t* d_counter, const LaunchDims& dm, hipStream_t s)
{
    if (n <= 0) return OMPD_OK;
    if (dm.n_walk)
        hipLaunchKernelGGL(ompd_k_prep, dim3(n), dim3(256), 0, s, d_cfgs, n, d_counter, dm.ring_slots);
    if (dm.n_strip)
        hipLaunchKernelGGL(ompd_k_sprep, dim3(n), dim3(dm.prep_threads), dm.lds_prep, s, d_cfgs, n, (int)dm.lds_prep);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return ompd_fail(OMPD_E_DEVICE, std::string("ingest launch (lds ") + std::to_string(dm.lds_prep) + "): " +
                                            hipGetErrorString(e));
    return OMPD_OK;
}

int ompd_launch_solve(const DevCfg* d_cfgs, const Tile* d_tiles, int n_tiles, const EdgeItem* d_items, int n_items,
                      int32_t* d_counter, const LaunchDims& dm, hipStream_t s, hipEvent_t* after)
{
    if (n_tiles <= 0) return OMPD_OK;
    // the walk's tiles and items, then the strips'
    n_tiles -= dm.n_level;
    n_items -= dm.n_tblock + dm.n_tedge;
    const Tile* d_strips = d_tiles + n_tiles;
    const EdgeItem* d_titems = d_items + n_items;
    const int rs = dm.ring_slots, grid_edge = dm.grid_edge;
    int k = 0;
    auto mark = [&]() { if (after) (void)hipEventRecord(after[k], s); ++k; };
    if (!dm.split) {
        // every phase and pass of a tile in one persistent kernel
        hipLaunchKernelGGL(ompd_k_solve, dim3(dm.grid_tile), dim3(PHASE_THREADS), dm.lds_tile, s, d_cfgs, d_tiles,
                           n_tiles, d_counter, rs);
        mark();
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return ompd_fail(OMPD_E_DEVICE, std::string("solve launch (ring slots ") + std::to_string(rs) + "): " +
                                                hipGetErrorString(e));
        return OMPD_OK;
    }
    // (a phase or pass that no CFG needs is not launched; its profile mark is still taken)
    auto phase = [&](int ph, bool launch) {
        if (launch && n_tiles > 0) {
            void* args[] = {(void*)&d_cfgs, (void*)&d_tiles, (void*)&n_tiles, (void*)&d_counter, (void*)&rs};
            (void)hipLaunchKernel(k_phases[ph], dim3(dm.grid[ph]), dim3(PHASE_THREADS), args, dm.lds[ph], s);
        }
        mark();
    };
    auto pass = [&](const void* fn, bool launch) {
        if (launch && n_items > 0) {
            void* args[] = {(void*)&d_cfgs, (void*)&d_tiles, (void*)&d_items, (void*)&n_items, (void*)&d_counter};
            (void)hipLaunchKernel(fn, dim3(grid_edge), dim3(64), args, 0, s);
        }
        mark();
    };
    phase(PH_NU, true);
    phase(PH_AVE, true);
    pass((const void*)ompd_k_post_ave, true);
    phase(PH_MAYP, true);
    pass((const void*)ompd_k_post_mayp, true);
    phase(PH_LATER, true);
    pass((const void*)ompd_k_post_later, true);
    phase(PH_LIVE, dm.refine);
    pass((const void*)ompd_k_post_live, dm.refine);
    phase(PH_AVF, true);
    pass((const void*)ompd_k_post_avf, true);
    if (n_tiles > 0) hipLaunchKernelGGL(ompd_k_varkind, dim3(grid_edge), dim3(64), 0, s, d_cfgs, d_tiles, n_tiles, d_counter);
    mark();
    auto transpose = [&](const void* fn, int n) {
        if (n > 0) {
            void* args[] = {(void*)&d_cfgs, (void*)&d_titems};
            (void)hipLaunchKernel(fn, dim3(n), dim3(256), args, 0, s);
        }
        mark();
    };
    auto strips = [&](const void* fn, const void* fn_rows) {
        for (int b = 0; b < dm.n_buckets; ++b) {
            const LaunchDims::Bucket& k = dm.bucket[b];
            const Tile* t = d_strips + k.first;
            void* args[] = {(void*)&d_cfgs, (void*)&t};
            (void)hipLaunchKernel(k.by_rows ? fn_rows : fn, dim3(k.n), dim3(64 * k.waves), args, k.lds, s);
        }
        mark();
    };
    transpose((const void*)ompd_k_tin, dm.n_tblock);
    strips((const void*)ompd_k_strip_a, (const void*)ompd_k_strip_a);
    transpose((const void*)ompd_k_tmid, dm.n_tblock);
    if (!dm.first_half) strips((const void*)ompd_k_strip_b, (const void*)ompd_k_strip_b_rows);
    else mark();
    transpose((const void*)ompd_k_tout, dm.first_half ? 0 : dm.n_tblock + dm.n_tedge);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return ompd_fail(OMPD_E_DEVICE, std::string("solve launch (ring slots ") + std::to_string(rs) + "): " +
                                            hipGetErrorString(e));
    return OMPD_OK;
}

static int launch_prep(ompd_plan* p, hipStream_t s)
{
    return ompd_launch_prep((const DevCfg*)p->d_cfgs, p->n, p->d_counter, p->dims, s);
}

static int launch_solve(ompd_plan* p, hipStream_t s)
{
    return ompd_launch_solve((const DevCfg*)p->d_cfgs, (const Tile*)p->d_tiles, p->n_tiles,
                             (const EdgeItem*)p->d_items, p->n_items, p->d_counter, p->dims, s);
}

// Capture one launch function into an executable graph (nullptr if capture
// is not available here).
static hipGraphExec_t capture(ompd_plan* p, int (*fn)(ompd_plan*, hipStream_t), hipGraph_t* keep)
{
    hipStream_t cs;
    if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) return nullptr;
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    int rc = (e == hipSuccess) ? fn(p, cs) : OMPD_E_DEVICE;
    hipGraph_t g = nullptr;
    hipError_t e2 = hipStreamEndCapture(cs, &g);
    (void)hipStreamDestroy(cs);
    (void)hipGetLastError();
    if (e != hipSuccess || e2 != hipSuccess || rc != OMPD_OK || !g) {
        if (g) (void)hipGraphDestroy(g);
        return nullptr;
    }
    hipGraphExec_t x = nullptr;
    if (hipGraphInstantiate(&x, g, nullptr, nullptr, 0) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipGraphDestroy(g);
        return nullptr;
    }
    *keep = g;
    return x;
}

static void drop_graphs(ompd_plan* p)
{
    if (p->gx_prep) (void)hipGraphExecDestroy(p->gx_prep);
    if (p->gx_solve) (void)hipGraphExecDestroy(p->gx_solve);
    if (p->g_prep) (void)hipGraphDestroy(p->g_prep);
    if (p->g_solve) (void)hipGraphDestroy(p->g_solve);
    p->gx_prep = p->gx_solve = nullptr;
    p->g_prep = p->g_solve = nullptr;
}

// Enqueue one solve: HIP events on the caller's stream around the ingest
// kernel and around the persistent solve (events stay outside the graphs).
static int launch_all(ompd_plan* p, hipStream_t s)
{
    (void)hipGetLastError();
    if (p->cfg.use_graph && !p->gx_prep) {
        p->gx_prep = capture(p, launch_prep, &p->g_prep);
        p->gx_solve = capture(p, launch_solve, &p->g_solve);
        if (!p->gx_prep || !p->gx_solve) {
            drop_graphs(p);
            p->cfg.use_graph = false;   // capture unavailable: launch directly
        }
    }
    CK(hipEventRecord(p->ev0, s));
    if (p->profile) {
        // direct launches with an event after every kernel, all on the caller's stream
        int rc = launch_prep(p, s);
        if (rc) return rc;
        CK(hipEventRecord(p->ev1, s));
        rc = ompd_launch_solve((const DevCfg*)p->d_cfgs, (const Tile*)p->d_tiles, p->n_tiles,
                               (const EdgeItem*)p->d_items, p->n_items, p->d_counter, p->dims, s, p->evk);
        if (rc) return rc;
        CK(hipEventRecord(p->ev2, s));
        return OMPD_OK;
    }
    if (p->cfg.use_graph) CK(hipGraphLaunch(p->gx_prep, s));
    else { int rc = launch_prep(p, s); if (rc) return rc; }
    CK(hipEventRecord(p->ev1, s));
    if (p->cfg.use_graph) CK(hipGraphLaunch(p->gx_solve, s));
    else { int rc = launch_solve(p, s); if (rc) return rc; }
    CK(hipEventRecord(p->ev2, s));
    return OMPD_OK;
}

extern "C" int ompd_plan_create(ompd_ctx* ctx, const ompd_cfg* cfgs, ompd_result* res, int32_t n, uint32_t flags,
                                ompd_plan** out)
{
    if (!(flags & OMPD_F_DEVICE_PTRS)) return ompd_fail(OMPD_E_INVAL, "plans need OMPD_F_DEVICE_PTRS");
    if (!ctx) return ompd_fail(OMPD_E_INVAL, "ctx is NULL");
    std::lock_guard<std::mutex> lk(ctx->mu);
    PlanConfig pc;
    return ompd_plan_build(ctx, cfgs, res, n, flags, pc, out);
}

int ompd_plan_run_locked(ompd_plan* p, hipStream_t s)
{
    CK(hipSetDevice(p->ctx->device));
    p->last_stream = s;
    return launch_all(p, s);
}

// The status words of a launch as its ingest left them.
__global__ void __launch_bounds__(256) ompd_k_info_clear(const DevCfg* __restrict__ cfgs, int n)
{
    const int total = n * INFO_WORDS;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < total; t += gridDim.x * blockDim.x) {
        const int w = t % INFO_WORDS;
        if (w != INFO_LEVELS && w != INFO_ORDER) cfgs[t / INFO_WORDS].info[w] = 0;
    }
}

int ompd_plan_rerun_locked(ompd_plan* p, hipStream_t s)
{
    if (p->dims.n_walk) return ompd_plan_run_locked(p, s);
    CK(hipSetDevice(p->ctx->device));
    p->last_stream = s;
    CK(hipEventRecord(p->ev0, s));
    hipLaunchKernelGGL(ompd_k_info_clear, dim3(std::min((p->n * INFO_WORDS + 255) / 256, 1024)), dim3(256), 0, s,
                       (const DevCfg*)p->d_cfgs, p->n);
    CK(hipEventRecord(p->ev1, s));
    int rc = launch_solve(p, s);
    if (rc) return rc;
    CK(hipEventRecord(p->ev2, s));
    return OMPD_OK;
}

extern "C" int ompd_plan_run(ompd_plan* p, void* stream)
{
    if (!p) return ompd_fail(OMPD_E_INVAL, "plan is NULL");
    std::lock_guard<std::mutex> lk(p->ctx->mu);
    return ompd_plan_run_locked(p, (hipStream_t)stream);
}

std::string ompd_status_message(int i, const int32_t* inf)
{
    const int st = inf[INFO_STATUS];
    char buf[320];
    if (st == OMPD_E_DEVICE && inf[INFO_PM_PHASE] > 0) {
        static const char* const ph[5] = {"next use", "eager validity", "pending copies", "delayed placement",
                                          "final validity"};
        static const char* const what[5] = {"?", "inputs of a step (in_ready)", "a free ring slot (consumed)",
                                            "stored states (flushed)", "a produced step (produced, helper)"};
        const int k = inf[INFO_PM_PHASE] - 1, w = inf[INFO_PM_WHAT];
        snprintf(buf, sizeof buf,
                 "cfg %d: a kernel wait gave up (phase %s, tile %d of the CFG, waiting for %s: counter at %d, "
                 "needed %d, after %d wall-clock ticks)",
                 i, (k >= 0 && k < 5) ? ph[k] : "?", inf[INFO_PM_TILE], (w >= 0 && w < 5) ? what[w] : "?",
                 inf[INFO_PM_SEEN], inf[INFO_PM_TARGET], inf[INFO_PM_TICKS]);
    } else
        snprintf(buf, sizeof buf, "cfg %d: %s", i,
                 st == OMPD_E_INVAL ? "malformed CFG" : st == OMPD_E_NOCONVERGE ? "sweep cap reached" : "device error");
    return buf;
}

// The status words of every CFG of a launch (each in its own scratch) into one array, so that
// they come back in one copy instead of one per CFG.
__global__ void __launch_bounds__(256) ompd_k_info(const DevCfg* __restrict__ cfgs, int n, int32_t* __restrict__ out)
{
    const int total = n * INFO_WORDS;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < total; t += gridDim.x * blockDim.x)
        out[t] = cfgs[t / INFO_WORDS].info[t % INFO_WORDS];
}

static int gather_info(const DevCfg* d_cfgs, int n, int32_t* d_out, int32_t* h_out, hipStream_t s)
{
    if (n <= 0) return OMPD_OK;
    const int total = n * INFO_WORDS;
    hipLaunchKernelGGL(ompd_k_info, dim3(std::min((total + 255) / 256, 1024)), dim3(256), 0, s, d_cfgs, n, d_out);
    CK(hipGetLastError());
    CK(hipMemcpyAsync(h_out, d_out, 4 * (size_t)total, hipMemcpyDeviceToHost, s));
    return OMPD_OK;
}

int ompd_plan_collect(ompd_plan* p, int32_t* per_cfg)
{
    CK(hipSetDevice(p->ctx->device));
    if (p->n == 0) {
        CK(hipStreamSynchronize(p->last_stream));
        return OMPD_OK;
    }
    // info words live per CFG inside the scratch arena
    int rg = gather_info(p->d_cfgs, p->n, p->d_info, p->h_info.data(), p->last_stream);
    if (rg) return rg;
    CK(hipStreamSynchronize(p->last_stream));
    int first = OMPD_OK;
    for (int i = 0; i < p->n; ++i) {
        const int32_t* inf = &p->h_info[(size_t)i * INFO_WORDS];
        int st = inf[INFO_STATUS];
        if (per_cfg) per_cfg[i] = st;
        for (int k = 0; k < 6; ++k) p->res[i].sweeps[k] = inf[INFO_SWEEPS + k];
        if (st && first == OMPD_OK) {
            first = st;
            g_err = ompd_status_message(i, inf);
        }
    }
    return first;
}

extern "C" int ompd_plan_status(ompd_plan* p, int32_t* per_cfg)
{
    if (!p) return ompd_fail(OMPD_E_INVAL, "plan is NULL");
    std::lock_guard<std::mutex> lk(p->ctx->mu);
    return ompd_plan_collect(p, per_cfg);
}

extern "C" int ompd_plan_last_ms(ompd_plan* p, float* total_ms, float* solve_ms)
{
    if (!p) return ompd_fail(OMPD_E_INVAL, "plan is NULL");
    CK(hipEventSynchronize(p->ev2));
    float a = 0, b = 0;
    CK(hipEventElapsedTime(&a, p->ev0, p->ev2));
    CK(hipEventElapsedTime(&b, p->ev1, p->ev2));
    if (total_ms) *total_ms = a;
    if (solve_ms) *solve_ms = b;
    return OMPD_OK;
}

extern "C" int ompd_plan_profile(ompd_plan* p, int32_t enable)
{
    if (!p) return ompd_fail(OMPD_E_INVAL, "plan is NULL");
    std::lock_guard<std::mutex> lk(p->ctx->mu);
    if (enable && !p->evk[0])
        for (hipEvent_t& e : p->evk) CK(hipEventCreate(&e));
    p->profile = enable != 0;
    return OMPD_OK;
}

extern "C" int ompd_plan_kernel_ms(ompd_plan* p, float* ms, int32_t capacity, int32_t* n_kernels)
{
    if (!p || !ms) return ompd_fail(OMPD_E_INVAL, "bad arguments");
    if (!p->profile) return ompd_fail(OMPD_E_INVAL, "profiling is off for this plan");
    CK(hipEventSynchronize(p->ev2));
    const int n = 1 + (p->dims.split ? N_SOLVE_KERNELS : 1);
    if (n_kernels) *n_kernels = n;
    hipEvent_t marks[2 + N_SOLVE_KERNELS] = {p->ev0, p->ev1};
    for (int k = 0; k < N_SOLVE_KERNELS; ++k) marks[2 + k] = p->evk[k];
    for (int k = 0; k < n && k < capacity; ++k) {
        float x = 0;
        CK(hipEventElapsedTime(&x, marks[k], marks[k + 1]));
        ms[k] = x;
    }
    return OMPD_OK;
}

extern "C" int ompd_plan_configure(ompd_plan* p, int64_t lds_bytes, int32_t wg_per_cu)
{
    if (!p || lds_bytes < 0 || wg_per_cu < 0) return ompd_fail(OMPD_E_INVAL, "bad plan configuration");
    std::lock_guard<std::mutex> lk(p->ctx->mu);
    PlanConfig c = p->cfg;
    c.lds_bytes = (size_t)lds_bytes;
    c.wg_per_cu = wg_per_cu;
    c.use_graph = true;
    return ompd_plan_retile(p, c);
}

extern "C" int ompd_plan_split_kernels(ompd_plan* p, int32_t split)
{
    if (!p) return ompd_fail(OMPD_E_INVAL, "plan is NULL");
    std::lock_guard<std::mutex> lk(p->ctx->mu);
    PlanConfig c = p->cfg;
    c.split = split != 0;
    c.use_graph = true;
    return ompd_plan_retile(p, c);
}

extern "C" int ompd_plan_describe(ompd_plan* p, char* buf, int32_t len)
{
    if (!p || !buf || len <= 0) return ompd_fail(OMPD_E_INVAL, "bad arguments");
    long lanes = 0;
    for (size_t i = 0; i + p->dims.n_level < p->h_tiles.size(); ++i) lanes += p->h_tiles[i].nw;
    // strip_cfgs: the CFGs solved by level; level_cfgs: those of them in the shape of a launch that leaves
    // the GPU idle
    int level_cfgs = 0;
    for (const DevCfg& d : p->h_cfgs) level_cfgs += d.spread;
    snprintf(buf, len,
             "{\"cfgs\": %d, \"tiles\": %d, \"words\": %ld, \"ring_slots\": %d, \"split\": %d, \"grid_tile\": %d, "
             "\"grid_phases\": [%d, %d, %d, %d, %d], "
             "\"lds_bytes\": %zu, \"wg_per_cu\": %d, \"graph\": %d, \"graph_captured\": %d, "
             "\"scratch_bytes\": %zu, \"bucket_sched\": [%d, %d, %d, %d, %d], \"level_cfgs\": %d, "
             "\"strip_cfgs\": %d, \"level_tiles\": %d, \"lds_level\": %zu, \"strip_launches\": %d}",
             p->n, p->n_tiles - p->dims.n_level, lanes, p->dims.ring_slots, (int)p->dims.split, p->dims.grid_tile,
             p->dims.grid[0], p->dims.grid[1], p->dims.grid[2],
             p->dims.grid[3], p->dims.grid[4], p->cfg.lds_bytes, p->cfg.wg_per_cu,
             p->cfg.use_graph ? 1 : 0, p->gx_solve ? 1 : 0, p->scratch_bytes, p->cfg.bucket_sched[0],
             p->cfg.bucket_sched[1], p->cfg.bucket_sched[2], p->cfg.bucket_sched[3], p->cfg.bucket_sched[4],
             level_cfgs, p->dims.n_strip, p->dims.n_level, p->dims.n_buckets ? p->dims.bucket[0].lds : 0, p->dims.n_buckets);
    return OMPD_OK;
}

extern "C" void ompd_plan_destroy(ompd_plan* p)
{
    if (!p) return;
    (void)hipSetDevice(p->ctx->device);
    if (p->last_stream || p->gx_prep) (void)hipDeviceSynchronize();
    drop_graphs(p);
    if (p->d_tiles) (void)hipFree(p->d_tiles);
    if (p->d_items) (void)hipFree(p->d_items);
    if (p->d_cfgs) (void)hipFree(p->d_cfgs);
    if (p->d_info) (void)hipFree(p->d_info);
    if (p->scratch) (void)hipFree(p->scratch);
    if (p->ev0) (void)hipEventDestroy(p->ev0);
    if (p->ev1) (void)hipEventDestroy(p->ev1);
    if (p->ev2) (void)hipEventDestroy(p->ev2);
    for (hipEvent_t e : p->evk)
        if (e) (void)hipEventDestroy(e);
    delete p;
}

// ---------------------------------------------------------------------------
// autotuner
// ---------------------------------------------------------------------------
// Time the plan under configuration c: `trials` runs after one that warms up the graph.
static int time_config(ompd_plan* p, const PlanConfig& c, hipStream_t s, int trials, float& avg)
{
    int rc = ompd_plan_retile(p, c);
    if (rc) return rc;
    float tot = 0;
    for (int t = 0; t < trials + 1; ++t) {
        rc = ompd_plan_run_locked(p, s);
        if (rc) return rc;
        CK(hipEventSynchronize(p->ev2));
        float ms = 0;
        CK(hipEventElapsedTime(&ms, p->ev0, p->ev2));
        if (t > 0) tot += ms;
    }
    avg = tot / trials;
    return OMPD_OK;
}

extern "C" int ompd_plan_autotune(ompd_plan* p, void* stream, int32_t trials, float* best_ms)
{
    if (!p) return ompd_fail(OMPD_E_INVAL, "plan is NULL");
    std::lock_guard<std::mutex> lk(p->ctx->mu);
    hipStream_t s = (hipStream_t)stream;
    trials = std::max(1, trials);
    PlanConfig base = p->cfg;
    base.only_bucket = -1;
    // 1. the schedule of each size bucket, its CFGs timed alone under both schedules
    if (!(p->flags & (OMPD_F_SCHED_LEVEL | OMPD_F_SCHED_WALK))) {
        int count[OMPD_SCHED_BUCKETS] = {0}, small[OMPD_SCHED_BUCKETS] = {0};
        for (const DevCfg& d : p->h_cfgs) {
            const int b = ompd_sched_bucket(d.nb);
            ++count[b];
            small[b] += d.strip_ok;
        }
        for (int b = 0; b < OMPD_SCHED_BUCKETS; ++b) {
            if (!count[b]) continue;
            float best = 1e30f;
            int pick = SCHED_WALK;
            for (int sc : {(int)SCHED_WALK, (int)SCHED_LEVEL}) {
                if (sc == SCHED_LEVEL && small[b] == 0) continue;
                PlanConfig c = base;
                c.bucket_sched[b] = sc;
                c.only_bucket = b;
                float ms = 0;
                if (time_config(p, c, s, trials, ms) != OMPD_OK) continue;
                if (ms < best) { best = ms; pick = sc; }
            }
            base.bucket_sched[b] = pick;
        }
    }
    // the buckets were timed alone, where the lower latency wins; on the whole plan the throughput
    // may favour the default rule instead: keep whichever runs the plan faster (there is nothing to
    // compare where the rule puts every CFG on the schedule picked for it)
    if (!(p->flags & (OMPD_F_SCHED_LEVEL | OMPD_F_SCHED_WALK))) {
        PlanConfig rule = base;
        for (int b = 0; b < OMPD_SCHED_BUCKETS; ++b) rule.bucket_sched[b] = -1;
        auto schedules = [&](const PlanConfig& c, std::vector<int>& of) -> bool {
            if (ompd_plan_retile(p, c) != OMPD_OK) return false;
            for (const DevCfg& d : p->h_cfgs) of.push_back(d.sched);
            return true;
        };
        std::vector<int> picked, ruled;
        float t_pick = 0, t_rule = 0;
        if (schedules(base, picked) && schedules(rule, ruled) && picked != ruled &&
            time_config(p, base, s, trials, t_pick) == OMPD_OK && time_config(p, rule, s, trials, t_rule) == OMPD_OK &&
            t_rule < t_pick)
            base = rule;
    }
    // 2. the launch configuration of the whole plan with those schedules; it is the walk's, so a plan
    // without a CFG on it keeps the one it has
    PlanConfig best = base;
    float best_t = 1e30f;
    int rc = ompd_plan_retile(p, base);
    if (rc) return rc;
    std::vector<PlanConfig> candidates;
    if (p->dims.n_walk == 0) candidates.push_back(base);
    else
        for (size_t lds : {(size_t)16 * STATE_BYTES, (size_t)32 * STATE_BYTES, (size_t)64 * STATE_BYTES})
            for (int wpc : {0, 4}) {
                PlanConfig c = base;
                c.lds_bytes = lds;
                c.wg_per_cu = wpc;
                candidates.push_back(c);
            }
    for (const PlanConfig& c : candidates) {
        float ms = 0;
        if (time_config(p, c, s, trials, ms) != OMPD_OK) continue;
        if (ms < best_t) { best_t = ms; best = c; }
    }
    rc = ompd_plan_retile(p, best);
    if (rc) return rc;
    if (best_t >= 1e30f) return ompd_fail(OMPD_E_DEVICE, "autotune: no configuration ran");
    if (best_ms) *best_ms = best_t;
    return OMPD_OK;
}

extern "C" int ompd_plan_set_schedule(ompd_plan* p, const int32_t* per_bucket)
{
    if (!p || !per_bucket) return ompd_fail(OMPD_E_INVAL, "bad arguments");
    for (int b = 0; b < OMPD_SCHED_BUCKETS; ++b)
        if (per_bucket[b] < -1 || per_bucket[b] > 1) return ompd_fail(OMPD_E_INVAL, "schedule must be -1, 0 or 1");
    std::lock_guard<std::mutex> lk(p->ctx->mu);
    PlanConfig c = p->cfg;
    for (int b = 0; b < OMPD_SCHED_BUCKETS; ++b) c.bucket_sched[b] = per_bucket[b];
    c.only_bucket = -1;
    c.use_graph = true;
    return ompd_plan_retile(p, c);
}

// ---------------------------------------------------------------------------
// host-pointer batch path (and the device-pointer one-shot path)
// ---------------------------------------------------------------------------
namespace {
struct Staged {
    std::vector<ompd_cfg> dcfg;
    std::vector<ompd_result> dres;
    void* dmem = nullptr;
    size_t bytes = 0;
    // output copies back: (device offset, host pointer, bytes)
    struct Back { size_t off; void* host; size_t bytes; };
    std::vector<Back> back;
    ~Staged() { if (dmem) (void)hipFree(dmem); }
};
}  // namespace

static int stage_inputs(const ompd_cfg* cfgs, ompd_result* res, int n, Staged& st, hipStream_t s)
{
    // layout: inputs then outputs, each 256-aligned
    std::vector<uint8_t> host;
    size_t total = 0;
    auto reserve = [&](size_t bytes) { size_t o = total; total += align256(bytes); return o; };
    struct In { size_t sp, si, kd, spc, R, W, evh, evd, lxh, lxd, call, sums, sc; };
    struct OutO { size_t nu_h, nu_d, ave_h, ave_d, avf_h, avf_d, ie_d, ie_h, ig_d, ig_h, vk, ad, bd, fpc; };
    std::vector<In> in(n);
    std::vector<OutO> oo(n);
    for (int i = 0; i < n; ++i) {
        const ompd_cfg& g = cfgs[i];
        const ompd_result& r = res[i];
        size_t wd = (size_t)(g.n_vars + 63) / 64;
        size_t bv = (size_t)g.n_blocks * wd * 8, ev = (size_t)g.n_edges * wd * 8;
        In& a = in[i];
        a.sp = reserve(4 * ((size_t)g.n_blocks + 1));
        a.si = reserve(4 * (size_t)g.n_edges);
        a.kd = reserve((size_t)g.n_edges);
        a.spc = reserve((size_t)g.n_blocks);
        a.R = reserve(bv);
        a.W = reserve(bv);
        a.evh = g.entry_valid_host ? reserve(wd * 8) : SIZE_MAX;
        a.evd = g.entry_valid_dev ? reserve(wd * 8) : SIZE_MAX;
        a.lxh = g.exit_live_host ? reserve(wd * 8) : SIZE_MAX;
        a.lxd = g.exit_live_dev ? reserve(wd * 8) : SIZE_MAX;
        a.call = g.call_summary ? reserve(4 * (size_t)g.n_blocks) : SIZE_MAX;
        a.sums = g.call_summary ? reserve((size_t)g.n_summaries * 16 * wd * 8) : SIZE_MAX;
        a.sc = g.scalar ? reserve(wd * 8) : SIZE_MAX;
        (void)r;
        (void)ev;
    }
    size_t in_bytes = total;
    for (int i = 0; i < n; ++i) {
        const ompd_cfg& g = cfgs[i];
        const ompd_result& r = res[i];
        size_t wd = (size_t)(g.n_vars + 63) / 64;
        size_t bv = (size_t)g.n_blocks * wd * 8, ev = (size_t)g.n_edges * wd * 8;
        OutO& o = oo[i];
        auto opt = [&](const void* ptr, size_t bytes) { return ptr ? reserve(bytes) : SIZE_MAX; };
        o.nu_h = opt(r.nu_host, bv); o.nu_d = opt(r.nu_dev, bv);
        o.ave_h = opt(r.ave_host, bv); o.ave_d = opt(r.ave_dev, bv);
        o.avf_h = (r.avf_host || r.avf_dev) ? reserve(bv) : SIZE_MAX;
        o.avf_d = (r.avf_host || r.avf_dev) ? reserve(bv) : SIZE_MAX;
        o.ie_d = opt(r.ins_entry_to_dev, bv); o.ie_h = opt(r.ins_entry_to_host, bv);
        o.ig_d = opt(r.ins_edge_to_dev, ev); o.ig_h = opt(r.ins_edge_to_host, ev);
        o.vk = opt(r.var_kind, (size_t)g.n_vars); o.ad = opt(r.after_dev, g.n_blocks); o.bd = opt(r.before_dev, g.n_blocks);
        o.fpc = opt(r.fp_clause, bv);
    }
    st.bytes = total;
    hipError_t e = hipMalloc(&st.dmem, std::max<size_t>(total, 256));
    if (e != hipSuccess) return ompd_fail(OMPD_E_NOMEM, std::string("device staging: ") + hipGetErrorString(e));
    host.assign(in_bytes, 0);
    char* D = (char*)st.dmem;
    st.dcfg.resize(n);
    st.dres.resize(n);
    for (int i = 0; i < n; ++i) {
        const ompd_cfg& g = cfgs[i];
        const ompd_result& r = res[i];
        size_t wd = (size_t)(g.n_vars + 63) / 64;
        size_t bv = (size_t)g.n_blocks * wd * 8, ev = (size_t)g.n_edges * wd * 8;
        const In& a = in[i];
        auto put = [&](size_t o, const void* src, size_t bytes) { if (bytes && src) memcpy(host.data() + o, src, bytes); };
        put(a.sp, g.succ_ptr, 4 * ((size_t)g.n_blocks + 1));
        put(a.si, g.succ_idx, 4 * (size_t)g.n_edges);
        put(a.kd, g.edge_kind, (size_t)g.n_edges);
        put(a.spc, g.space, (size_t)g.n_blocks);
        put(a.R, g.read_bits, bv);
        put(a.W, g.write_bits, bv);
        if (a.evh != SIZE_MAX) put(a.evh, g.entry_valid_host, wd * 8);
        if (a.evd != SIZE_MAX) put(a.evd, g.entry_valid_dev, wd * 8);
        if (a.lxh != SIZE_MAX) put(a.lxh, g.exit_live_host, wd * 8);
        if (a.lxd != SIZE_MAX) put(a.lxd, g.exit_live_dev, wd * 8);
        if (a.call != SIZE_MAX) put(a.call, g.call_summary, 4 * (size_t)g.n_blocks);
        if (a.sums != SIZE_MAX) put(a.sums, g.summaries, (size_t)g.n_summaries * 16 * wd * 8);
        if (a.sc != SIZE_MAX) put(a.sc, g.scalar, wd * 8);
        ompd_cfg d = g;
        d.succ_ptr = (const int32_t*)(D + a.sp);
        d.succ_idx = (const int32_t*)(D + a.si);
        d.edge_kind = (const uint8_t*)(D + a.kd);
        d.space = (const uint8_t*)(D + a.spc);
        d.read_bits = (const uint64_t*)(D + a.R);
        d.write_bits = (const uint64_t*)(D + a.W);
        d.entry_valid_host = a.evh != SIZE_MAX ? (const uint64_t*)(D + a.evh) : nullptr;
        d.entry_valid_dev = a.evd != SIZE_MAX ? (const uint64_t*)(D + a.evd) : nullptr;
        d.exit_live_host = a.lxh != SIZE_MAX ? (const uint64_t*)(D + a.lxh) : nullptr;
        d.exit_live_dev = a.lxd != SIZE_MAX ? (const uint64_t*)(D + a.lxd) : nullptr;
        d.call_summary = a.call != SIZE_MAX ? (const int32_t*)(D + a.call) : nullptr;
        d.summaries = a.sums != SIZE_MAX ? (const uint64_t*)(D + a.sums) : nullptr;
        d.scalar = a.sc != SIZE_MAX ? (const uint64_t*)(D + a.sc) : nullptr;
        st.dcfg[i] = d;
        const OutO& o = oo[i];
        ompd_result dr;
        memset(&dr, 0, sizeof dr);
        auto outp = [&](size_t off, void* hp, size_t bytes) -> void* {
            if (off == SIZE_MAX) return nullptr;
            if (hp) st.back.push_back({off, hp, bytes});
            return D + off;
        };
        dr.nu_host = (uint64_t*)outp(o.nu_h, r.nu_host, bv);
        dr.nu_dev = (uint64_t*)outp(o.nu_d, r.nu_dev, bv);
        dr.ave_host = (uint64_t*)outp(o.ave_h, r.ave_host, bv);
        dr.ave_dev = (uint64_t*)outp(o.ave_d, r.ave_dev, bv);
        dr.avf_host = (uint64_t*)outp(o.avf_h, r.avf_host, bv);
        dr.avf_dev = (uint64_t*)outp(o.avf_d, r.avf_dev, bv);
        dr.ins_entry_to_dev = (uint64_t*)outp(o.ie_d, r.ins_entry_to_dev, bv);
        dr.ins_entry_to_host = (uint64_t*)outp(o.ie_h, r.ins_entry_to_host, bv);
        dr.ins_edge_to_dev = (uint64_t*)outp(o.ig_d, r.ins_edge_to_dev, ev);
        dr.ins_edge_to_host = (uint64_t*)outp(o.ig_h, r.ins_edge_to_host, ev);
        dr.var_kind = (uint8_t*)outp(o.vk, r.var_kind, (size_t)g.n_vars);
        dr.after_dev = (uint8_t*)outp(o.ad, r.after_dev, (size_t)g.n_blocks);
        dr.before_dev = (uint8_t*)outp(o.bd, r.before_dev, (size_t)g.n_blocks);
        dr.fp_clause = (uint64_t*)outp(o.fpc, r.fp_clause, bv);
        st.dres[i] = dr;
    }
    if (in_bytes) CK(hipMemcpyAsync(st.dmem, host.data(), in_bytes, hipMemcpyHostToDevice, s));
    CK(hipStreamSynchronize(s));
    return OMPD_OK;
}

int ompd_batch_locked(ompd_ctx* ctx, const ompd_cfg* cfgs, ompd_result* res, int32_t n, uint32_t flags,
                      hipStream_t s)
{
    if (n < 0 || (n > 0 && (!cfgs || !res))) return ompd_fail(OMPD_E_INVAL, "bad arguments");
    CK(hipSetDevice(ctx->device));
    for (int i = 0; i < n; ++i) {
        int rc = check_cfg_host(cfgs[i], i);
        if (rc) return rc;
    }
    PlanConfig pc;
    pc.use_graph = false;
    if (flags & OMPD_F_DEVICE_PTRS) {
        ompd_plan* p = nullptr;
        int rc = ompd_plan_build(ctx, cfgs, res, n, flags, pc, &p);
        if (rc) return rc;
        rc = ompd_plan_run_locked(p, s);
        if (rc == OMPD_OK) rc = ompd_plan_collect(p, nullptr);
        for (int i = 0; i < n; ++i) memcpy(res[i].sweeps, p->res[i].sweeps, sizeof res[i].sweeps);
        ompd_plan_destroy(p);
        return rc;
    }
    Staged st;
    int rc = stage_inputs(cfgs, res, n, st, s);
    if (rc) return rc;
    ompd_plan* p = nullptr;
    rc = ompd_plan_build(ctx, st.dcfg.data(), st.dres.data(), n, flags | OMPD_F_DEVICE_PTRS, pc, &p);
    if (rc) return rc;
    rc = ompd_plan_run_locked(p, s);
    int rc2 = (rc == OMPD_OK) ? ompd_plan_collect(p, nullptr) : rc;
    if (rc == OMPD_OK) {
        for (int i = 0; i < n; ++i) memcpy(res[i].sweeps, p->res[i].sweeps, sizeof res[i].sweeps);
        // copy outputs back (also for invalid CFGs: their buffers hold unspecified values)
        std::vector<uint8_t> host(st.bytes);
        hipError_t e = hipMemcpy(host.data(), st.dmem, st.bytes, hipMemcpyDeviceToHost);
        if (e != hipSuccess) rc2 = ompd_fail(OMPD_E_DEVICE, hipGetErrorString(e));
        else
            for (const auto& b : st.back) memcpy(b.host, host.data() + b.off, b.bytes);
    }
    ompd_plan_destroy(p);
    return rc2;
}

extern "C" int ompd_analyze_batch(ompd_ctx* ctx, const ompd_cfg* cfgs, ompd_result* res, int32_t n, uint32_t flags,
                                  void* stream)
{
    if (!ctx) return ompd_fail(OMPD_E_INVAL, "ctx is NULL");
    std::lock_guard<std::mutex> lk(ctx->mu);
    return ompd_batch_locked(ctx, cfgs, res, n, flags, (hipStream_t)stream);
}

extern "C" int ompd_analyze_batch_noalloc(ompd_ctx* ctx, const ompd_cfg* cfgs, ompd_result* res, int32_t n,
                                          uint32_t flags, void* stream)
{
    if (!ctx) return ompd_fail(OMPD_E_INVAL, "ctx is NULL");
    if (!(flags & OMPD_F_DEVICE_PTRS)) return ompd_fail(OMPD_E_INVAL, "noalloc: needs OMPD_F_DEVICE_PTRS");
    if (n < 0 || (n > 0 && (!cfgs || !res))) return ompd_fail(OMPD_E_INVAL, "bad arguments");
    std::lock_guard<std::mutex> lk(ctx->mu);
    std::lock_guard<std::mutex> sk(g_scratch_mu[ctx->device & 63]);
    if (!ctx->static_scratch) return ompd_fail(OMPD_E_DEVICE, "noalloc: no static scratch on this device");
    CK(hipSetDevice(ctx->device));
    for (int i = 0; i < n; ++i) {
        int rc = check_cfg_host(cfgs[i], i);
        if (rc) return rc;
    }
    if (n == 0) return OMPD_OK;
    hipStream_t s = (hipStream_t)stream;
    PlanConfig pc;
    pc.use_graph = false;
    if (flags & OMPD_F_TILE_KERNEL) pc.split = false;
    if (const uint32_t r = (flags >> 8) & 7u) pc.lds_bytes = (size_t)(4u << r) * STATE_BYTES;
    // layout of the static scratch: each CFG's solver scratch, the work counters, the default
    // boundaries, then the launch tables (descriptors, tiles, items) and the gathered status words;
    // a batch whose strip tables do not fit takes the walk
    char* S = ctx->static_scratch;
    std::vector<ScratchOff> off(n);
    std::vector<size_t> base(n), boff(n);
    std::vector<DevCfg> h(n);
    std::vector<uint64_t> bnd;
    Shape sh;
    int rc = OMPD_OK;
    size_t total = 0, bnd_words = 0, counter_off = 0, bnd_off = 0, cfg_off = 0, tile_off = 0, item_off = 0, info_off = 0;
    const int rows = ompd_strip_rows(cfgs, n, flags);
    for (uint32_t walk : {0u, OMPD_F_SCHED_WALK}) {
        total = bnd_words = 0;
        for (int i = 0; i < n; ++i) {
            base[i] = total;
            total += ompd_cfg_scratch(cfgs[i], res[i], off[i], walk ? 0 : rows);
            boff[i] = bnd_words;
            bnd_words += 4 * (size_t)((cfgs[i].n_vars + 63) / 64);
        }
        counter_off = total;
        total += 256;
        bnd_off = total;
        total += align256(8 * bnd_words);
        bnd.assign(std::max<size_t>(bnd_words, 1), 0);
        for (int i = 0; i < n; ++i)
            ompd_fill_devcfg(cfgs[i], res[i], S + base[i], off[i], flags | walk, ctx->wait_ticks, h[i],
                             bnd.data() + boff[i], (uint64_t*)(S + bnd_off) + boff[i]);
        ompd_settle_sched(h.data(), n, ctx->n_cu, pc.split);
        sh = Shape();
        rc = ompd_make_shape(ctx, h, pc, sh);
        if (rc) return rc;
        cfg_off = total;
        total += align256(sizeof(DevCfg) * n);
        tile_off = total;
        total += align256(sizeof(Tile) * std::max<size_t>(sh.tiles.size(), 1));
        item_off = total;
        total += align256(sizeof(EdgeItem) * std::max<size_t>(sh.items.size(), 1));
        info_off = total;
        total += align256(4 * INFO_WORDS * (size_t)n);
        if (total <= OMPD_STATIC_SCRATCH_BYTES || !sh.dims.n_strip) break;
    }
    if (total > OMPD_STATIC_SCRATCH_BYTES) {
        char buf[200];
        snprintf(buf, sizeof buf, "noalloc: the batch needs %zu bytes of scratch, the static scratch holds %zu",
                 total, OMPD_STATIC_SCRATCH_BYTES);
        return ompd_fail(OMPD_E_NOMEM, buf);
    }
    // nothing here needs zeroed memory: the ingest kernel clears the counters and status words
    if (bnd_words) CK(hipMemcpyAsync(S + bnd_off, bnd.data(), 8 * bnd_words, hipMemcpyHostToDevice, s));
    CK(hipMemcpyAsync(S + cfg_off, h.data(), sizeof(DevCfg) * n, hipMemcpyHostToDevice, s));
    if (!sh.tiles.empty())
        CK(hipMemcpyAsync(S + tile_off, sh.tiles.data(), sizeof(Tile) * sh.tiles.size(), hipMemcpyHostToDevice, s));
    if (!sh.items.empty())
        CK(hipMemcpyAsync(S + item_off, sh.items.data(), sizeof(EdgeItem) * sh.items.size(), hipMemcpyHostToDevice,
                          s));
    const DevCfg* dc = (const DevCfg*)(S + cfg_off);
    int32_t* counter = (int32_t*)(S + counter_off);
    rc = ompd_launch_prep(dc, n, counter, sh.dims, s);
    if (rc == OMPD_OK)
        rc = ompd_launch_solve(dc, (const Tile*)(S + tile_off), (int)sh.tiles.size(), (const EdgeItem*)(S + item_off),
                               (int)sh.items.size(), counter, sh.dims, s);
    std::vector<int32_t> info((size_t)n * INFO_WORDS, 0);
    if (rc == OMPD_OK) rc = gather_info(dc, n, (int32_t*)(S + info_off), info.data(), s);
    CK(hipStreamSynchronize(s));   // the host tables above stay alive until the copies are done
    if (rc) return rc;
    int first = OMPD_OK;
    for (int i = 0; i < n; ++i) {
        const int32_t* inf = &info[(size_t)i * INFO_WORDS];
        for (int k = 0; k < 6; ++k) res[i].sweeps[k] = inf[INFO_SWEEPS + k];
        if (inf[INFO_STATUS] && first == OMPD_OK) {
            first = inf[INFO_STATUS];
            g_err = ompd_status_message(i, inf);
        }
    }
    return first;
}

extern "C" int ompd_analyze_cfg(ompd_ctx* ctx, const ompd_cfg* cfg, ompd_result* res, uint32_t flags, void* stream)
{
    if (!ctx || !cfg || !res) return ompd_fail(OMPD_E_INVAL, "bad arguments");
    std::lock_guard<std::mutex> lk(ctx->mu);
    return ompd_batch_locked(ctx, cfg, res, 1, flags, (hipStream_t)stream);
}
