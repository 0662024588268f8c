// Strip schedule (gfx950): the blocks of a level in parallel, a wavefront's last passes in LDS.
//
// A block's level is one more than the highest level of its predecessors over edges other than
// BACK; no such edge joins two blocks of a level.  ompd_k_sprep sorts the blocks by level and lays
// out, for each direction, passes: what a wavefront does at once, 4 rows of 16 lanes.  A row holds
// the edges of some blocks of one level (whole blocks, their edges side by side) for one word of
// variables; the meet over a block's edges is a segmented reduction with DPP moves, and its last
// lane applies the block's transfer.  With `units` words per strip a pass takes 4 / units groups
// of a level.
//
// A pass's results go to the state array and to a ring of the wavefront's last 8 passes in LDS
// (1 KiB each).  A neighbour up to 8 passes back is read from there; one further back, or not yet
// visited in the round, from the state array.  That and the other inputs (constants of the phase)
// lie in arrays by word and position ([word][block by level], host and device word together), so
// that a row's lanes read neighbouring pairs, and are loaded 6-8 passes ahead.  What is left on
// the chain from pass to pass is the LDS read, the meet, the transfer and the LDS write: a pass is
// bound by the instructions one wavefront issues, so a pass takes as many words as fit.
//
// ompd_k_tin transposes the accesses into that layout, ompd_k_tmid and ompd_k_tout the results
// back to the caller's rows (bound by memory: 3.5-5.1 TB/s on 4096 CFGs).  One workgroup runs all
// phases of its words (ompd_k_strip_a: next use and eager validity; ompd_k_strip_b: pending copies,
// placement, refinement, final validity, map kinds).
//
// A phase is a sequence of rounds.  The passes of a direction are cut into one run per wavefront;
// a round visits every run in level order.  After a round only readers of a neighbour that is not
// visited before them in a round (a BACK edge, or the neighbour in another wavefront's run) can
// see a state they have not seen: the ingest kernel lists these links, and a pass with such a link
// whose neighbour changed is marked.  Such a link reads its neighbour as it was before the round.  The
// next round visits, from each marked pass on, as far as
// the changes of this round reach; without a mark the states are the fixed point.  The phases are
// monotone from the same start, so every order of visits reaches the walk's fixed point, bit for
// bit.
#include <type_traits>

#include "ompd_common.h"

namespace ompd {

typedef uint64_t u64;
typedef uint32_t hw;
#define LDS3 __attribute__((address_space(3)))

// Lane record, first word: where the neighbour's state is (near: its place in the ring; far: its
// position), the block's position, whether the lane is the block's last (its writer).
constexpr uint32_t R0_REF = 0x7FFFu, R0_FAR = 1u << 15, R0_LAST = 1u << 31;
constexpr int R0_POS = 16;   // 15 bits
// Second word: the edge's entry, whether the lanes 1, 2, 4, 8 before belong to the same block, the
// edge's and block's flags, and (the same in a pass's every lane) whether the pass holds a block
// with a special rule and the reduction steps its longest block needs.  A CFG with more entries than 16
// bits number (by_rows): a row's edges follow each other in the forward order (link) and in the
// backward one (ebwd), so lanes 0 and 1 of a row hold the low and high half of where its first one is.
constexpr uint32_t R1_EDGE = 0xFFFFu;
constexpr int R1_SAME = 16, R1_LE = 20, R1_DEV = 21, R1_NOEDGE = 22, R1_XSRC = 23, R1_SPECIAL = 24, R1_CROSS = 25,
              R1_KIND = 26, R1_STEPS = 29;
// kinds (3 bits): + K_MULTI for a block with more edges than a group's lanes (EXIT and calls too)
constexpr uint32_t K_ENTRY = 1, K_EXIT = 2, K_CALL = 3, K_MULTI = 4;
constexpr int ROW = 16;                   // lanes of a group
// Place of a block: its pass, its first lane among the pass's groups, and in the place of a pass's
// first block the pass's facts.
constexpr int LOC_LANE = 16, LOC_STEPS = 23;
constexpr uint32_t LOC_SPECIAL = 1u << 22;

// --------------------------------------------------------------------------
// ingest
// --------------------------------------------------------------------------
// Peel from ENTRY over the edges other than BACK by one wavefront: lorder gets the blocks by level,
// loff where each level starts; returns the blocks placed, *nl the levels.  rec: per block, low half
// the count of those edges into it, high half its successors over them, two of 15 bits (none: the
// entry nb, whose count does not run out), or PEEL_LIST and where its list in si starts (bit 15 marks
// a list's last entry; without si the list is read from the CSR).
//
// The levels are a chain, a CFG has hundreds to thousands of them and most hold a few blocks: a
// lane holds a block of the level and its record, and one LDS operation counts down a successor and
// returns its record, so that a level costs one LDS latency and few instructions.  A freed block
// stays in its lane, a lane's second one moves to an idle lane.  Levels with lists go on through `fr`
// (the first 64 blocks of the next level), wider ones through lorder.  (Order, CSR range, edges and
// counts read one after another: 0.44 us a level of a 8002-block CFG; this: 0.29 us.)
constexpr uint32_t PEEL_LIST = 1u << 31;
__device__ __noinline__ int peel_lds(int entry, LDS3 u64* rec, const LDS3 uint16_t* si, LDS3 uint16_t* fr,
                                     GAS int32_t* lorder, GAS int32_t* loff, const GAS int32_t* succ_ptr,
                                     const GAS int32_t* succ_idx, const GAS uint8_t* kind, LDS3 int* nl_out)
{
    const int lane = threadIdx.x & 63;
    const u64 below = (1ull << lane) - 1ull;
    auto down = [&](uint32_t q) -> u64 {
        return __hip_atomic_fetch_sub(&rec[q], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    int fa = 0, fb, tail = 1, nl = 0;
    auto append = [&](bool free, uint32_t q) {
        const u64 m = __ballot(free);
        const int at = tail + __popcll(m & below);
        if (free) {
            lorder[at] = (int32_t)q;
            if (at - fb < 64) fr[at - fb] = (uint16_t)q;
        }
        tail += __popcll(m);
    };
    // the successors of the lanes' blocks (records w), however many
    auto step = [&](int b, uint32_t w, bool on) {
        const bool list = on && (w & PEEL_LIST) != 0, two = on && !list;
        bool f0 = false, f1 = false;
        if (two) {
            f0 = (uint32_t)down(w & 0x7FFFu) == 1u;
            f1 = (uint32_t)down(w >> 16) == 1u;
        }
        append(f0, w & 0x7FFFu);
        append(f1, w >> 16);
        on = list;
        int e = !on ? 0 : si ? (int)(w & ~PEEL_LIST) : succ_ptr[b];
        const int z = on && !si ? succ_ptr[b + 1] : 0;
        while (__ballot(on)) {
            uint32_t q = 0;
            bool take = on;
            if (on && si) {
                const uint32_t v = si[e++];
                q = v & 0x7FFFu;
                on = !(v >> 15);
            } else if (on) {
                take = kind[e] != 1;
                q = (uint32_t)succ_idx[e];
                on = ++e < z;
            }
            append(take && (uint32_t)down(q) == 1u, q);
        }
    };
    if (lane == 0) lorder[0] = entry;
    int cur = lane == 0 ? entry : -1;
    uint32_t w = (uint32_t)(rec[entry] >> 32);
    for (bool wide = false;;) {
        // narrow levels of blocks with up to two successors
        while (!wide) {
            if (__ballot(cur >= 0 && (int32_t)w < 0)) break;
            if (lane == 0) loff[nl] = fa;
            const uint32_t q0 = w & 0x7FFFu, q1 = w >> 16;
            u64 r0 = 0, r1 = 0;
            if (cur >= 0) { r0 = down(q0); r1 = down(q1); }
            const bool f0 = (uint32_t)r0 == 1u, f1 = (uint32_t)r1 == 1u;
            const u64 m0 = __ballot(f0), m1 = __ballot(f1);
            const int n0 = __popcll(m0), n1 = __popcll(m1);
            if (f0) lorder[(uint32_t)(tail + __popcll(m0 & below))] = (int32_t)q0;
            if (f1) lorder[(uint32_t)(tail + n0 + __popcll(m1 & below))] = (int32_t)q1;
            fa = tail;
            tail += n0 + n1;
            ++nl;
            cur = f0 ? (int)q0 : f1 ? (int)q1 : -1;
            w = (uint32_t)((f0 ? r0 : r1) >> 32);
            if (n0 + n1 == 0) {
                if (lane == 0) *nl_out = nl;
                return tail;
            }
            wide = n0 + n1 > 64;
            if (wide) break;
            for (u64 more = m0 & m1, idle = ~(m0 | m1); more; more &= more - 1, idle &= idle - 1) {
                const int from = __builtin_ctzll(more), to = __builtin_ctzll(idle);
                const int q = __builtin_amdgcn_readlane((int)q1, from), r = __builtin_amdgcn_readlane((int)(r1 >> 32), from);
                if (lane == to) { cur = q; w = (uint32_t)r; }
            }
        }
        // one level of any kind
        fb = tail;
        if (lane == 0) loff[nl] = fa;
        if (!wide) step(cur, w, cur >= 0);
        else {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            for (int i = fa; i < fb; i += 64) {
                const bool on = i + lane < fb;
                const int b = on ? lorder[i + lane] : 0;
                step(b, (uint32_t)(rec[b] >> 32), on);
            }
        }
        // (else the narrow levels wait for their stores: a load that this level left unused counts
        // with them)
        __builtin_amdgcn_s_waitcnt(0);
        ++nl;
        const int n = tail - fb;
        if (n == 0) {
            if (lane == 0) *nl_out = nl;
            return tail;
        }
        fa = fb;
        wide = n > 64;
        if (!wide) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            cur = lane < n ? (int)fr[lane] : -1;
            w = (uint32_t)(rec[cur >= 0 ? cur : 0] >> 32);
        }
    }
}

extern "C" __global__ void __launch_bounds__(1024, 8) ompd_k_sprep(const DevCfg* __restrict__ cfgs, int n_cfgs, int lds_bytes)
{
    extern __shared__ __align__(16) uint32_t smem[];
    __shared__ int s_err, s_tail, s_nl, s_x[2];
    __shared__ int32_t s_scan[16];
    __shared__ uint16_t s_fr[64];
    if ((int)blockIdx.x >= n_cfgs) return;
    const int ci = cfgs[blockIdx.x].by_size;
    if (cfgs[ci].sched != SCHED_LEVEL) return;
    const DevCfg c = cfgs[ci];
    const int tid = threadIdx.x, nt = blockDim.x;
    const int nb = c.nb, ne = c.ne;
    if (!validate_cfg(c, s_err)) return;
    int32_t* kc = c.s_kc;          // edges into each block, later a cursor
    const bool lists = strip_prep_lds(nb, ne) <= (size_t)lds_bytes, in_lds = lists || strip_prep_lds(nb, 0) <= (size_t)lds_bytes;
    LDS3 u64* rec = (LDS3 u64*)smem;
    LDS3 uint32_t* rec32 = (LDS3 uint32_t*)smem;
    LDS3 uint16_t* si = lists ? (LDS3 uint16_t*)(rec + nb + 1) : nullptr;
    for (int b = tid; b < nb; b += nt) kc[b] = 0;
    if (in_lds) for (int b = tid; b <= nb; b += nt) rec[b] = b < nb ? 0ull : 1ull << 30;
    else for (int b = tid; b < nb; b += nt) c.est_b[b] = 0;                   // (the counts, in global memory)
    if (tid == 0) { s_x[0] = s_x[1] = 0; s_tail = 1; s_err = 0; }
    __syncthreads();
    for (int b = tid; b < nb; b += nt) {
        const int e0 = c.succ_ptr[b], z = c.succ_ptr[b + 1];
        uint32_t w = (uint32_t)nb | ((uint32_t)nb << 16);
        int k = 0, first[2] = {0, 0};
        for (int e = e0; e < z; ++e) {
            const int q = c.succ_idx[e];
            atomicAdd(&kc[q], 1);
            if (c.kind[e] == 1) continue;
            if (!in_lds) { atomicAdd(&c.est_b[q], 1); continue; }
            __hip_atomic_fetch_add(&rec32[2 * q], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (k < 2) first[k] = q;
            if (k == 0) w = (w & 0xFFFF0000u) | (uint32_t)q;
            else if (k == 1) w = (w & 0xFFFFu) | ((uint32_t)q << 16);
            if (si && k == 2) { si[e0] = (uint16_t)first[0]; si[e0 + 1] = (uint16_t)first[1]; }
            if (si && k >= 2) si[e0 + k] = (uint16_t)q;
            ++k;
        }
        if (k > 2) {
            w = PEEL_LIST | (uint32_t)e0;
            if (si) si[e0 + k - 1] |= 0x8000u;
        }
        if (in_lds) rec32[2 * b + 1] = w;
    }
    __syncthreads();
    // a block that no edge enters, or one without a way out, is malformed (and has no record)
    for (int b = tid; b < nb; b += nt)
        if ((b != c.entry && __hip_atomic_load(&kc[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) ||
            (b != c.exit && c.succ_ptr[b] == c.succ_ptr[b + 1]))
            s_err = 1;
    __syncthreads();
    if (s_err) { if (tid == 0) c.info[INFO_STATUS] = OMPD_E_INVAL_; return; }
    int32_t* lorder = c.s_lorder;
    int32_t* loff = c.s_loff;
    int nl = 0, placed = 0;
    if (in_lds) {
        if (tid < 64) {
            const int p = peel_lds(c.entry, rec, si, (LDS3 uint16_t*)s_fr, G(c.s_lorder), G(c.s_loff), G(c.succ_ptr),
                                   G(c.succ_idx), G(c.kind), (LDS3 int*)&s_nl);
            if (tid == 0) s_tail = p;
        }
        __syncthreads();
        nl = s_nl;
        placed = s_tail;
    } else {
        int32_t* dg = c.est_b;
        if (tid == 0) lorder[0] = c.entry;
        __syncthreads();
        int fa = 0, fb = 1;
        while (fa < fb) {
            if (tid == 0) loff[nl] = fa;
            for (int i = fa + tid; i < fb; i += nt) {
                const int b = lorder[i];
                for (int e = c.succ_ptr[b]; e < c.succ_ptr[b + 1]; ++e) {
                    if (c.kind[e] == 1) continue;
                    const int q = c.succ_idx[e];
                    if (atomicSub(&dg[q], 1) == 1) lorder[atomicAdd(&s_tail, 1)] = q;
                }
            }
            __syncthreads();
            fa = fb;
            fb = s_tail;
            ++nl;
            __syncthreads();
        }
        placed = fb;
    }
    __syncthreads();
    if (placed < nb) {
        // blocks of a cycle without a BACK edge: a level each, in id order
        for (int b = tid; b < nb; b += nt) c.pos[b] = 0xFFFFu;
        __syncthreads();
        for (int i = tid; i < placed; i += nt) c.pos[lorder[i]] = (uint16_t)i;
        __syncthreads();
        if (tid == 0) {
            int n = placed;
            for (int b = 0; b < nb; ++b)
                if (c.pos[b] == 0xFFFFu) { lorder[n] = b; loff[nl++] = n++; }
            s_nl = nl;
        }
        __syncthreads();
        nl = s_nl;
    }
    if (tid == 0) {
        loff[nl] = nb;
        c.info[INFO_LEVELS] = nl;
        c.info[INFO_ORDER] = 1;
    }
    for (int i = tid; i < nb; i += nt) c.pos[lorder[i]] = (uint16_t)i;
    // first edge of each position: forward by position, backward by position from the last
    // (est_b[s]: the block at position nb - 1 - s)
    if (tid == 0) { c.est_f[0] = 0; c.est_b[0] = 0; }
    __syncthreads();
    for (int i = tid; i < nb; i += nt) {
        const int b = lorder[i], k = __hip_atomic_load(&kc[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int d = c.succ_ptr[b + 1] - c.succ_ptr[b];
        c.est_f[i + 1] = k > 0 ? k : 1;
        c.est_b[nb - i] = d > 0 ? d : 1;
    }
    __syncthreads();
    block_scan_inclusive(c.est_f + 1, nb, s_scan);
    block_scan_inclusive(c.est_b + 1, nb, s_scan);
    // Groups and passes: a level's blocks in order, whole blocks to a group of up to 16 edges (a
    // block with more has a group of its own), R groups to a pass; one thread per level, its
    // groups counted first.  loc: the place of each position.
    const int C = c.units, R = 4 / C;
    int32_t* lp = reinterpret_cast<int32_t*>(c.x_f);   // [levels + 1] first pass of each level (the links come later)
    uint2* const RECS[2] = {reinterpret_cast<uint2*>(c.rec_sf), reinterpret_cast<uint2*>(c.rec_sb)};
    int np[2], sl[2];   // passes; passes of a wavefront's run
    for (int dir = 0; dir < 2; ++dir) {
        const int32_t* es = dir ? c.est_b : c.est_f;
        uint32_t* loc = dir ? c.loc_b : c.loc_f;
        for (int phase = 0; phase < 2; ++phase) {
            for (int l = tid; l < nl; l += nt) {
                const int lv = dir ? nl - 1 - l : l;
                const int a = dir ? nb - loff[lv + 1] : loff[lv], z = dir ? nb - loff[lv] : loff[lv + 1];
                const int base = phase ? lp[l] : 0;
                int g = 0, fill = 0, at = es[a], most = 1, first = 0;
                uint32_t special = 0;
                auto facts = [&]() {   // of a finished pass, to its first block's place
                    const uint32_t steps = most > 8 ? 4u : most > 4 ? 3u : most > 2 ? 2u : most > 1 ? 1u : 0u;
                    loc[first] |= special | (steps << LOC_STEPS);
                    most = 1;
                    special = 0;
                };
                for (int s = a; s < z; ++s) {
                    const int nx = es[s + 1], k = nx - at, lanes = min(k, ROW), i = dir ? nb - 1 - s : s;
                    if (fill + lanes > ROW) {
                        ++g;
                        fill = 0;
                        if (phase && g % R == 0) facts();
                    }
                    if (phase) {
                        const int b = lorder[i];
                        if (g % R == 0 && fill == 0) first = i;
                        if (c.by_rows && fill == 0)   // (of a row with one edge; else its record follows)
                            RECS[dir][((size_t)(base + g / R) * R + g % R) * ROW + 1] = make_uint2(0u, (uint32_t)at >> 16);
                        loc[i] = (uint32_t)(base + g / R) | ((uint32_t)((g % R) * ROW + fill) << LOC_LANE);
                        if (b == c.entry || b == c.exit || k > ROW || (c.call && c.call[b] >= 0)) special = LOC_SPECIAL;
                        most = max(most, k);
                    }
                    fill += lanes;
                    at = nx;
                }
                if (phase) facts();
                else lp[l + 1] = g / R + 1;
            }
            if (phase == 0) {
                if (tid == 0) lp[0] = 0;
                __syncthreads();
                block_scan_inclusive(lp + 1, nl, s_scan);
                np[dir] = lp[nl];
                sl[dir] = (np[dir] + c.waves - 1) / c.waves;
                // lanes without an edge
                uint4* z = reinterpret_cast<uint4*>(RECS[dir]);
                for (int i = tid; i < np[dir] * R * ROW / 2; i += nt) z[i] = make_uint4(0, 0, 0, 0);
            }
            __syncthreads();
        }
    }
    auto pass_of = [&](uint32_t l) -> int { return (int)(l & 0xFFFFu); };
    // is a reader's visit not always after its neighbour's in a round?
    auto cross = [&](int dir, int pn, int pr) { return pn >= pr || pn / sl[dir] != pr / sl[dir]; };
    auto kind_of = [&](int b, int k) -> uint32_t {
        return (b == c.entry ? K_ENTRY : b == c.exit ? K_EXIT : (c.call && c.call[b] >= 0) ? K_CALL : 0u) + (k > ROW ? K_MULTI : 0u);
    };
    // the record of edge `slot` of the k of the block at position i (place l) whose neighbour is at
    // position in (place ln, kn edges); `fl`: flags of the second word; `entry`: the edge's (by_rows: its
    // place in the direction's order)
    auto record = [&](int dir, int i, uint32_t l, int k, int slot, int in, uint32_t ln, int kn, int entry, uint32_t fl) {
        const int lanes = min(k, ROW), pr = pass_of(l), pn = pass_of(ln), lane = (int)(l >> LOC_LANE) & 63;
        uint32_t w0 = (uint32_t)i << R0_POS;
        if (slot == lanes - 1) w0 |= R0_LAST;
        const bool x = in >= 0 && cross(dir, pn, pr);
        if (in >= 0 && !x && pr - pn <= STRIP_RING) {
            // the neighbour's writer: its lane in the first unit's row of its group
            const uint32_t ll = ((ln >> LOC_LANE) & 63u) + (uint32_t)min(kn, ROW) - 1u;
            w0 |= (uint32_t)((pn % STRIP_RING) * 64) + (ll / ROW) * (uint32_t)(C * ROW) + ll % ROW;
        } else if (in >= 0) w0 |= R0_FAR | (uint32_t)in;
        for (int t = 0; t < 4; ++t) fl |= slot >= (1 << t) ? 1u << (R1_SAME + t) : 0u;
        if (c.by_rows) {
            const int in_row = (lane + slot) % ROW;
            const uint32_t row = (uint32_t)(entry - in_row);
            entry = in_row == 0 ? (int)(row & R1_EDGE) : in_row == 1 ? (int)(row >> 16) : 0;
        }
        fl |= (x ? 1u << R1_CROSS : 0u) | (uint32_t)entry;
        if (lane + slot == 0) fl |= ((l & LOC_SPECIAL) ? 1u << R1_SPECIAL : 0u) | ((l >> LOC_STEPS) << R1_STEPS);
        RECS[dir][(size_t)pr * R * ROW + lane + slot] = make_uint2(w0, fl);
    };
    auto flags_of = [&](int b, int k) -> uint32_t {
        return (c.space[b] ? 1u << R1_DEV : 0u) | (kind_of(b, k) << R1_KIND);
    };
    // A thread takes a block and its edges [e, z); past the first WIDE of them (a switch, its join)
    // the wavefront's lanes share what is left of each such block, one after another: `first` per
    // edge of the lane's own block, `rest` per edge of lane l's block, `end` after it.  (One thread
    // per block throughout: 1.1 / 10.2 ms for a switch of 300 / 3000 cases in a loop; this: 0.6 / 5.5 ms.)
    constexpr int WIDE = 16;
    const int wl = tid & 63;
    auto edges = [&](int e, int z, auto&& first, auto&& rest, auto&& end) {
        const int own = min(z, e + WIDE);
        for (int k = e; k < own; ++k) first(k);
        for (u64 m = __ballot(z - e > WIDE); m; m &= m - 1) {
            const int l = __builtin_ctzll(m);
            const int from = __builtin_amdgcn_readlane(e, l) + WIDE, to = __builtin_amdgcn_readlane(z, l);
            for (int k = from + wl; k < to; k += 64) rest(k, l);
            end(l);
        }
    };
    auto of = [](auto v, int l) { return (decltype(v))__builtin_amdgcn_readlane((int)v, l); };
    // the last reader of a block, gathered over a wide block's lanes into lane l's
    struct Readers { int last = 0; uint32_t xs = 0; };
    auto gather = [&](Readers& mine, Readers& part, int l) {
        int v = part.last;
        for (int d = 1; d < 64; d <<= 1) v = max(v, __shfl_xor(v, d, 64));
        const bool x = __ballot(part.xs != 0u) != 0ull;
        if (wl == l) {
            mine.last = max(mine.last, v);
            if (x) mine.xs = 0x8000u;
        }
        part = Readers{};
    };
    auto reader = [&](int dir, Readers& r, int p, int pr) {
        if (cross(dir, p, pr)) r.xs = 0x8000u;
        else r.last = max(r.last, pr);
    };
    // what a block's writer needs to know of its readers: the last pass of its run that reads it
    // later in a round, and (bit 15) whether a cross link does; forward first
    for (int b0 = 0; b0 < nb; b0 += nt) {
        const int b = b0 + tid;
        const bool on = b < nb;
        const int i = on ? c.pos[b] : 0, pf = on ? pass_of(c.loc_f[i]) : 0;
        Readers mine, part;
        auto look = [&](Readers& r, int p, int e) { reader(0, r, p, pass_of(c.loc_f[c.pos[c.succ_idx[e]]])); };
        edges(on ? c.succ_ptr[b] : 0, on ? c.succ_ptr[b + 1] : 0, [&](int e) { look(mine, pf, e); },
              [&](int e, int l) { look(part, of(pf, l), e); }, [&](int l) { gather(mine, part, l); });
        if (on) c.last_f[i] = (uint16_t)((uint32_t)mine.last | mine.xs);
    }
    __syncthreads();
    // forward records, entries and cross links, by edge
    for (int b0 = 0; b0 < nb; b0 += nt) {
        const int b = b0 + tid;
        const bool on = b < nb;
        const int i = on ? c.pos[b] : 0, kb = on ? c.est_f[i + 1] - c.est_f[i] : 0;
        const uint32_t lb = on ? c.loc_f[i] : 0u;
        auto edge = [&](int i, int kb, uint32_t lb, int e) {
            const int q = c.succ_idx[e], iq = c.pos[q], a = c.est_f[iq], k = c.est_f[iq + 1] - a;
            const int slot = atomicSub(&kc[q], 1) - 1;
            const uint32_t lq = c.loc_f[iq];
            const bool le = is_le(c, c.kind[e]);
            c.link[a + slot] = (uint32_t)i | (le ? 0x8000u : 0u) | ((uint32_t)iq << 16);
            c.eid[a + slot] = e;
            c.erec[e] = a + slot;
            if (slot < ROW)
                record(0, iq, lq, k, slot, i, lb, kb, a + slot,
                       flags_of(q, k) | (le ? 1u << R1_LE : 0u) | ((c.last_f[iq] & 0x8000u) ? 1u << R1_XSRC : 0u));
            if (cross(0, pass_of(lb), pass_of(lq))) c.x_f[atomicAdd(&s_x[0], 1)] = (uint32_t)i | ((uint32_t)pass_of(lq) << 16);
        };
        edges(on ? c.succ_ptr[b] : 0, on ? c.succ_ptr[b + 1] : 0, [&](int e) { edge(i, kb, lb, e); },
              [&](int e, int l) { edge(of(i, l), of(kb, l), of(lb, l), e); }, [](int) {});
        if (on && b == c.entry) {
            const int a = c.est_f[i];
            c.link[a] = (uint32_t)i | ((uint32_t)i << 16);
            c.eid[a] = -1;
            record(0, i, lb, 1, 0, -1, 0, 0, a,
                   flags_of(b, 1) | (1u << R1_NOEDGE) | ((c.last_f[i] & 0x8000u) ? 1u << R1_XSRC : 0u));
        }
    }
    __syncthreads();
    // backward records and cross links: a block reads its successors, its readers are its
    // predecessors
    for (int b0 = 0; b0 < nb; b0 += nt) {
        const int b = b0 + tid;
        const bool on = b < nb;
        const int i = on ? c.pos[b] : 0, e0 = on ? c.succ_ptr[b] : 0, d = on ? c.succ_ptr[b + 1] - e0 : 0;
        const uint32_t lb = on ? c.loc_b[i] : 0u;
        const int pb = pass_of(lb), at = on ? c.est_b[nb - 1 - i] : 0;
        Readers mine, part;
        auto look = [&](Readers& r, int p, int e) { reader(1, r, p, pass_of(c.loc_b[c.link[e] & 0x7FFFu])); };
        const bool read = on && b != c.entry;
        edges(read ? c.est_f[i] : 0, read ? c.est_f[i + 1] : 0, [&](int e) { look(mine, pb, e); },
              [&](int e, int l) { look(part, of(pb, l), e); }, [&](int l) { gather(mine, part, l); });
        if (on) c.last_b[i] = (uint16_t)((uint32_t)mine.last | mine.xs);
        const uint32_t fl = on ? flags_of(b, d) | (mine.xs ? 1u << R1_XSRC : 0u) : 0u;
        auto crosses = [&](int iq, uint32_t lq, int p) {
            if (cross(1, pass_of(lq), p)) c.x_b[atomicAdd(&s_x[1], 1)] = (uint32_t)iq | ((uint32_t)p << 16);
        };
        static_assert(WIDE >= ROW, "the records of a block are its own thread's");
        edges(e0, e0 + d,
              [&](int e) {
                  const int j = e - e0, iq = c.pos[c.succ_idx[e]];
                  const uint32_t lq = c.loc_b[iq];
                  if (c.by_rows) c.ebwd[at + j] = c.erec[e];
                  if (j < ROW)
                      record(1, i, lb, d, j, iq, lq, c.est_b[nb - iq] - c.est_b[nb - 1 - iq], c.by_rows ? at + j : c.erec[e], fl);
                  crosses(iq, lq, pb);
              },
              [&](int e, int l) {
                  const int iq = c.pos[c.succ_idx[e]];
                  if (c.by_rows) c.ebwd[of(at, l) + e - of(e0, l)] = c.erec[e];
                  crosses(iq, c.loc_b[iq], of(pb, l));
              },
              [](int) {});
        if (on && d == 0) {
            if (c.by_rows) c.ebwd[at] = 0;
            record(1, i, lb, 1, 0, -1, 0, 0, c.by_rows ? at : 0, fl | (1u << R1_NOEDGE));
        }
    }
    __syncthreads();
    if (tid == 0) {
        c.hdr[SH_PASS_F] = np[0];
        c.hdr[SH_PASS_B] = np[1];
        c.hdr[SH_X_F] = s_x[0];
        c.hdr[SH_X_B] = s_x[1];
    }
}

// --------------------------------------------------------------------------
// solve
// --------------------------------------------------------------------------
// A pair of words, host and device.
struct __attribute__((aligned(16))) Pair { u64 h, d; };
__device__ __forceinline__ bool operator!=(const Pair& a, const Pair& b) { return a.h != b.h || a.d != b.d; }
typedef u64 v2u __attribute__((ext_vector_type(2)));
__device__ __forceinline__ Pair ldp(const u64* a, u64 i)   // pair i of an array
{
    const v2u v = *reinterpret_cast<const GAS v2u*>(G(a) + 2 * i);
    return Pair{v.x, v.y};
}
__device__ __forceinline__ void stp(u64* a, u64 i, Pair p)
{
    v2u v;
    v.x = p.h;
    v.y = p.d;
    *reinterpret_cast<GAS v2u*>(G(a) + 2 * i) = v;
}
// the same at a 32-bit byte offset from a wave-uniform start
__device__ __forceinline__ Pair ldp32(const GAS char* a, uint32_t off)
{
    const v2u v = *reinterpret_cast<const GAS v2u*>(a + off);
    return Pair{v.x, v.y};
}

// The strip of a workgroup as one lane sees it.
struct Strip {
    LDS3 char* ring;       // the wavefront's ring: STRIP_RING passes of 64 pairs
    LDS3 uint32_t* chg;    // blocks changed in this round
    LDS3 uint32_t* mark;   // passes to visit in this round
    LDS3 int* ctl;         // control word, map-kind masks
    int lane, wave, waves; // lane of the wavefront, wavefront of the workgroup
    int i, row;            // lane of the group, row of the wavefront
    int R;                 // groups of a pass
    int nb, nv, nrec;
    int u0, nu;            // the workgroup's first unit, its units
    int unit;              // the lane's unit (the last one again past the end)
    bool on;               // the unit is the lane's own
    bool flg;              // the word of reachability facts
    uint32_t ro;           // LDS offset of the unit's row in a pass of the ring
    u64 vm, fp, evh, evd, lxh, lxd;
    uint32_t cn, ce;       // start of the lane's unit in the workgroup's part of a block / an edge array (entries)
    size_t bn, be;         // start of the workgroup's part (entries)
};

__device__ __forceinline__ uint32_t sld(const LDS3 uint32_t* p) { return __hip_atomic_load(const_cast<LDS3 uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ int sld(const LDS3 int* p) { return __hip_atomic_load(const_cast<LDS3 int*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
template <class T> __device__ __forceinline__ void sst(LDS3 T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ void sor(LDS3 uint32_t* p, uint32_t v) { __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ __forceinline__ u64 wide(uint32_t m) { return (u64)m | ((u64)m << 32); }   // a mask for both halves
// all ones if bit `bit` is set
__device__ __forceinline__ u64 bit_mask(uint32_t w, int bit) { return wide((uint32_t)((int32_t)(w << (31 - bit)) >> 31)); }

template <int S>
__device__ __forceinline__ u64 row_shr(u64 v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, 0x110 + S, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), 0x110 + S, 0xF, 0xF, true);
    return (u64)lo | ((u64)hi << 32);
}
// lane L's value in every lane of its row
template <int L>
__device__ __forceinline__ uint32_t row_lane(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + L, 0xF, 0xF, true);   // row_newbcast
}
// Segmented reduction over the lanes of a block's edges: the last one gets the result (the first
// NA words by AND, the others by OR).  w1: the lane's record, steps: of its pass.
template <int NA, int N>
__device__ __forceinline__ void meet(uint32_t w1, uint32_t steps, u64 (&a)[N])
{
    auto step = [&](auto kc) {
        constexpr int K = decltype(kc)::value;
        const u64 same = bit_mask(w1, R1_SAME + K);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const u64 o = row_shr<1 << K>(a[j]);
            if (j < NA) a[j] &= o | ~same;
            else a[j] |= o & same;
        }
    };
    if (steps > 0) {
        step(std::integral_constant<int, 0>{});
        if (steps > 1) {
            step(std::integral_constant<int, 1>{});
            if (steps > 2) {
                step(std::integral_constant<int, 2>{});
                if (steps > 3) step(std::integral_constant<int, 3>{});
            }
        }
    }
}

constexpr bool backward(int ph) { return ph == PH_NU || ph == PH_LIVE; }
// Per phase: the words an edge contributes and how they meet (NA by AND, then N - NA by OR).
template <int PH> struct Terms { static constexpr int NA = 0, N = 2; };
template <> struct Terms<PH_AVE> { static constexpr int NA = 2, N = 2; };
template <> struct Terms<PH_LATER> { static constexpr int NA = 2, N = 4; };
template <> struct Terms<PH_AVF> { static constexpr int NA = 2, N = 2; };

// A record's inputs: the block's accesses, what the phase knows of the block (next use, copies
// before it), the edge's copies, its valid-in-both word.
template <int PH> struct In {
    static constexpr bool NODE = PH == PH_AVE || PH == PH_AVF || PH == PH_LIVE, EDGE = PH != PH_NU && PH != PH_AVE,
                          BOTH = PH == PH_LATER;
    Pair rw, nd, g;
    u64 b;
};
// arrays of a phase, from the workgroup's part on
template <int PH> struct Src {
    const GAS char *rw, *nd, *g, *b;
    GAS char* st;    // the phase's states
    GAS char* sh;    // what a round's cross links read: their sources' states before the round
};
template <int PH>
__device__ __forceinline__ Src<PH> sources(const DevCfg& c, const Strip& t)
{
    Src<PH> s;
    auto blk = [&](u64* a) { return reinterpret_cast<GAS char*>(G(a) + 2 * t.bn); };
    s.rw = blk(c.p_rw);
    s.nd = blk(PH == PH_AVE ? c.p_1 : c.p_2);
    s.g = reinterpret_cast<const GAS char*>(G(c.p_g) + 2 * t.be);
    s.b = reinterpret_cast<const GAS char*>(G(c.p_b) + t.be);
    s.st = blk(PH == PH_AVE || PH == PH_MAYP ? c.p_2 : c.p_1);
    s.sh = blk(c.p_3);   // (written after the phases that give it its contents, read out before the others)
    return s;
}
template <int PH>
__device__ __forceinline__ void load_in(const Src<PH>& s, uint32_t n, uint32_t e, In<PH>& x)   // n, e: entries
{
    x.rw = ldp32(s.rw, 16u * n);
    if constexpr (In<PH>::NODE) x.nd = ldp32(s.nd, 16u * n);
    if constexpr (In<PH>::EDGE) x.g = ldp32(s.g, 16u * e);
    if constexpr (In<PH>::BOTH) x.b = *reinterpret_cast<const GAS u64*>(s.b + 8u * e);
}

// The term of one edge from its neighbour's state and the edge's words; has / nle: the edge exists
// / exists and does not enter a loop.
template <int PH>
__device__ __forceinline__ void edge_term(u64 has, u64 nle, const Pair& s, const Pair& g, u64 b, u64 (&a)[Terms<PH>::N])
{
    if constexpr (PH == PH_NU) { a[0] = s.h & has; a[1] = s.d & has; }
    else if constexpr (PH == PH_AVE) { a[0] = s.h; a[1] = s.d; }
    else if constexpr (PH == PH_MAYP) { a[0] = (g.h | s.h) & nle; a[1] = (g.d | s.d) & nle; }
    else if constexpr (PH == PH_LATER) {
        const u64 lh = g.h | s.h, ld = g.d | s.d;
        a[0] = lh | b; a[1] = ld | b; a[2] = lh & nle; a[3] = ld & nle;
    }
    else if constexpr (PH == PH_AVF) { a[0] = s.h | g.h; a[1] = s.d | g.d; }
    else { a[0] = ((s.h & ~g.h) | g.d) & has; a[1] = ((s.d & ~g.d) | g.h) & has; }   // PH_LIVE
}

__device__ __forceinline__ u64 tselect(u64 a, u64 l, u64 t00, u64 t01, u64 t10, u64 t11)
{
    return (~a & ~l & t00) | (~a & l & t01) | (a & ~l & t10) | (a & l & t11);
}
// the unit's word of row r of the summary of call ci
__device__ __forceinline__ u64 sum_row(const DevCfg& c, const Strip& t, int ci, int r)
{
    return G(c.sums)[((size_t)ci * SUM_ROWS + r) * (size_t)c.wd + t.unit];
}
// validity behind a call: the callee's exit-validity tables by the validity before it and the
// next use after it (the OR over the block's successors; from the states while the strips hold
// them, from the rows ompd_k_tmid wrote once the placement has taken their place)
template <bool ROWS>
__device__ __forceinline__ void call_valid(const DevCfg& c, const Strip& t, int pos, u64& ah, u64& ad)
{
    const int b = G(c.s_lorder)[pos], ci = G(c.call)[b];
    u64 lh = 0, ld = 0;
    for (int e = G(c.succ_ptr)[b]; e < G(c.succ_ptr)[b + 1]; ++e) {
        const int q = G(c.succ_idx)[e];
        if constexpr (ROWS) {
            lh |= G(c.nu_h)[(size_t)q * c.wd + t.unit];
            ld |= G(c.nu_d)[(size_t)q * c.wd + t.unit];
        } else {
            const Pair p = ldp(c.p_1, (size_t)t.unit * t.nb + G(c.pos)[q]);
            lh |= p.h;
            ld |= p.d;
        }
    }
    ah = tselect(ah, lh, sum_row(c, t, ci, SUM_TH), sum_row(c, t, ci, SUM_TH + 1), sum_row(c, t, ci, SUM_TH + 2),
                 sum_row(c, t, ci, SUM_TH + 3));
    ad = tselect(ad, ld, sum_row(c, t, ci, SUM_TD), sum_row(c, t, ci, SUM_TD + 1), sum_row(c, t, ci, SUM_TD + 2),
                 sum_row(c, t, ci, SUM_TD + 3));
}
// what a block uses on the host and on the device (a call whose callee may touch a variable uses it)
__device__ __forceinline__ Pair uses(const DevCfg& c, const Strip& t, uint32_t kind, int pos, u64 dev, u64 rr)
{
    Pair u{rr & (~dev | t.fp), rr & dev & ~t.fp};
    if ((kind & 3u) == K_EXIT) u = Pair{t.lxh, t.lxd};
    if ((kind & 3u) == K_CALL) {
        const int ci = G(c.call)[G(c.s_lorder)[pos]];
        const u64 mw = sum_row(c, t, ci, SUM_MAYW_H) | sum_row(c, t, ci, SUM_MAYW_D);
        u.h |= sum_row(c, t, ci, SUM_MAYR_H) | mw;
        u.d |= sum_row(c, t, ci, SUM_MAYR_D) | mw;
    }
    return u;
}

// The block's new state from the met terms and its inputs (SPECIAL: by the rules of ENTRY, EXIT and
// calls too).
template <int PH, bool SPECIAL>
__device__ __forceinline__ Pair block_state(const DevCfg& c, const Strip& t, uint32_t w1, int pos,
                                            const u64 (&a)[Terms<PH>::N], const In<PH>& x)
{
    const u64 dev = bit_mask(w1, R1_DEV), rr = x.rw.h, ww = x.rw.d;
    const uint32_t kind = SPECIAL ? (w1 >> R1_KIND) & 3u : 0u;
    Pair v;
    if constexpr (PH == PH_NU) {
        u64 oh = a[0], od = a[1];
        if (kind == K_CALL && !t.flg) {
            const int ci = G(c.call)[G(c.s_lorder)[pos]];
            oh = sum_row(c, t, ci, SUM_NU0_H) | (sum_row(c, t, ci, SUM_NU1_H) & oh);
            od = sum_row(c, t, ci, SUM_NU0_D) | (sum_row(c, t, ci, SUM_NU1_D) & od);
        }
        v.h = (rr & (~dev | t.fp)) | (~ww & oh);
        v.d = (rr & dev & ~t.fp) | (~ww & od);
        if (kind == K_EXIT) v = Pair{t.lxh, t.lxd};
    } else if constexpr (PH == PH_AVE || PH == PH_AVF) {
        u64 ih = (x.nd.h | a[0]) & t.vm, id = (x.nd.d | a[1]) & t.vm;
        if (kind == K_ENTRY) { ih = t.evh; id = t.evd; }
        u64 ah = (ih & ~ww & dev) | ((ih | ww) & ~dev);
        u64 ad = ((id | ww) & dev & ~(rr & t.fp)) | (id & ~ww & ~dev);
        if (kind == K_CALL && !t.flg) call_valid<PH == PH_AVF>(c, t, pos, ah, ad);
        v.h = ah & t.vm;
        v.d = ad & t.vm;
    } else if constexpr (PH == PH_MAYP || PH == PH_LATER) {
        u64 sh = ((rr | ww) & ~dev) | (rr & t.fp & dev), sd = ((rr & ~t.fp) | ww) & dev;
        if (kind == K_EXIT || kind == K_CALL) {
            const Pair u = uses(c, t, kind, pos, dev, rr);
            sh = u.h | (kind == K_CALL ? sh : 0ull);
            sd = u.d | (kind == K_CALL ? sd : 0ull);
        }
        if constexpr (PH == PH_MAYP) v = Pair{a[0] & ~sh & t.vm, a[1] & ~sd & t.vm};
        else v = Pair{a[0] & a[2] & ~sh & t.vm, a[1] & a[3] & ~sd & t.vm};
    } else {   // PH_LIVE
        u64 rh = rr & (~dev | t.fp), rd = rr & dev & ~t.fp;
        const u64 kh = ww & ~dev, kd = (ww | (rr & t.fp)) & dev;
        if (kind == K_EXIT) { rh = t.lxh; rd = t.lxd; }
        if (kind == K_CALL) { rh = ~0ull; rd = ~0ull; }
        const u64 ah = rh | (a[0] & ~kh), ad = rd | (a[1] & ~kd);
        v.h = ((ah & ~x.nd.h) | x.nd.d) & t.vm;
        v.d = ((ad & ~x.nd.d) | x.nd.h) & t.vm;
    }
    return v;
}

// Edges past the first 16 of a block with more, in the forward order of `link` or the backward one
// of the successor CSR: visit(neighbour position, entry, loop entry) for those of the lane.
template <bool BWD, class Visit>
__device__ __forceinline__ void more_edges(const DevCfg& c, const Strip& t, int pos, Visit&& visit)
{
    if constexpr (BWD) {
        const int b = G(c.s_lorder)[pos], e0 = G(c.succ_ptr)[b], d = G(c.succ_ptr)[b + 1] - e0;
        for (int j = t.i + ROW; j < d; j += ROW)
            visit((int)G(c.pos)[G(c.succ_idx)[e0 + j]], G(c.erec)[e0 + j], false);
    } else {
        const int a = G(c.est_f)[pos], k = G(c.est_f)[pos + 1] - a;
        for (int j = t.i + ROW; j < k; j += ROW) {
            const uint32_t l = G(c.link)[a + j];
            visit((int)(l & 0x7FFFu), a + j, (l & 0x8000u) != 0);
        }
    }
}

// the wavefront's run of a direction's passes
__device__ __forceinline__ void my_run(const Strip& t, int np, int& p0, int& p1)
{
    const int len = (np + t.waves - 1) / t.waves;
    p0 = min(np, t.wave * len);
    p1 = min(np, p0 + len);
}

// Highest value of a wavefront's lanes.
__device__ __forceinline__ int wave_max(int v)
{
    auto step = [&](int o) { v = max(v, o); };
    step(__builtin_amdgcn_update_dpp(v, v, 0x111, 0xF, 0xF, false));   // row_shr 1, 2, 4, 8
    step(__builtin_amdgcn_update_dpp(v, v, 0x112, 0xF, 0xF, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x114, 0xF, 0xF, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x118, 0xF, 0xF, false));
    const int a = max(__builtin_amdgcn_readlane(v, 15), __builtin_amdgcn_readlane(v, 31));
    return max(a, max(__builtin_amdgcn_readlane(v, 47), __builtin_amdgcn_readlane(v, 63)));
}

// One wavefront's visit of passes p0 .. p1 - 1 in a round.  A pass's records are loaded two groups
// of AHEAD passes before it runs, its inputs one group before: a pass takes ~500 cycles, a load
// that misses L2 three or more of them.  FIRST: the first round, from `init`.  Else the ring is
// refilled with the passes before p0 (from pass `back` on), `reach` is the wavefront's horizon (the
// last pass that reads a block changed in this round), and `more(p)`, asked before a group of
// passes beyond it, ends the run early; true if a state of the lane's blocks changed.
template <int PH, bool BY_ROWS, bool FIRST, class More>
__device__ __forceinline__ bool run_passes(const DevCfg& c, const Strip& t, const Src<PH>& src, int p0, int p1, int back,
                                           u64 init, int& reach, More&& more)
{
    constexpr bool BWD = backward(PH);
    constexpr int NA = Terms<PH>::NA, N = Terms<PH>::N;
    constexpr int AHEAD = PH == PH_NU || FIRST ? 8 : 6;
    static_assert(AHEAD <= STRIP_RING, "a far state is stored before it is loaded ahead");
    const uint32_t stride = (uint32_t)__builtin_amdgcn_readfirstlane(t.R * ROW * 8);   // bytes of a pass's records
    const GAS char* RC = reinterpret_cast<const GAS char*>(G(BWD ? c.rec_sb : c.rec_sf));
    const uint32_t ro = (uint32_t)(((t.row / (4 / t.R)) * ROW + t.i) * 8);
    const GAS char* LAST = reinterpret_cast<const GAS char*>(G(BWD ? c.last_b : c.last_f));
    uint32_t changed = 0;
    int far_reader = -1;   // last reader of the lane's changed blocks
    struct Rec { uint32_t x, y; };
    auto record = [&](int p) -> Rec {
        typedef uint32_t v2 __attribute__((ext_vector_type(2)));
        const GAS char* at = RC + (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(p < p1 ? p : p1 - 1) * stride));
        const v2 v = *reinterpret_cast<const GAS v2*>(at + ro);
        return Rec{v.x, v.y};
    };
    struct Slot { In<PH> x; Pair far, old; uint32_t last; };
    auto load = [&](const Rec& r, Slot& s) {
        const uint32_t pos = (r.x >> R0_POS) & 0x7FFFu, n = t.cn + pos;
        uint32_t e = r.y & R1_EDGE;
        if constexpr (BY_ROWS && In<PH>::EDGE) {
            // (lanes without an edge take another one's entry)
            const uint32_t row = row_lane<0>(e) | (row_lane<1>(e) << 16);
            e = min(row + (uint32_t)t.i, (uint32_t)t.nrec - 1u);
            if constexpr (BWD) e = (uint32_t)G(c.ebwd)[e];
        }
        load_in<PH>(src, n, t.ce + e, s.x);
        const uint32_t far = 16u * (t.cn + ((r.x & R0_FAR) ? r.x & R0_REF : 0u));
        if constexpr (FIRST) s.far = ldp32(src.st, far);
        else s.far = ldp32(((r.y >> R1_CROSS) & 1u) ? src.sh : src.st, far);
        if constexpr (!FIRST) {
            s.old = ldp32(src.st, 16u * n);
            s.last = *reinterpret_cast<const GAS uint16_t*>(LAST + 2u * pos);
        }
    };
    auto ring = [&](int p) -> LDS3 v2u* {
        return reinterpret_cast<LDS3 v2u*>(t.ring + (((uint32_t)p % STRIP_RING) * 1024u + (uint32_t)t.lane * 16u));
    };
    auto visit = [&](int p, const Rec& r, const Slot& q) {
        const uint32_t w1 = r.y, facts = (uint32_t)__builtin_amdgcn_readfirstlane((int)w1);
        const v2u nr = *reinterpret_cast<const LDS3 v2u*>(t.ring + ((r.x & 0x1FFu) * 16u + t.ro));
        const bool far = r.x & R0_FAR;
        Pair s{far ? q.far.h : nr.x, far ? q.far.d : nr.y};
        if constexpr (FIRST) {
            // (a neighbour that may not have been visited yet has the start's state)
            const u64 x = bit_mask(w1, R1_CROSS);
            s.h = (s.h & ~x) | (init & x);
            s.d = (s.d & ~x) | (init & x);
        }
        const u64 has = ~bit_mask(w1, R1_NOEDGE), nle = has & ~bit_mask(w1, R1_LE);
        u64 a[N];
        edge_term<PH>(has, nle, s, q.x.g, q.x.b, a);
        const int pos = (int)((r.x >> R0_POS) & 0x7FFFu);
        const bool special = (facts >> R1_SPECIAL) & 1u;
        if (special) {
            asm volatile("; special");   // (one scalar branch around what few passes need)
            if ((w1 >> R1_KIND) & K_MULTI)
                more_edges<BWD>(c, t, pos, [&](int in, int entry, bool le) {
                    const uint32_t* loc = BWD ? c.loc_b : c.loc_f;
                    const int pn = (int)(G(loc)[in] & 0xFFFFu), len = (G(c.hdr)[BWD ? SH_PASS_B : SH_PASS_F] + t.waves - 1) / t.waves;
                    const bool cross = pn >= p || pn / len != p / len;
                    const Pair st = !cross ? ldp32(src.st, 16u * (t.cn + in))
                                    : FIRST ? Pair{init, init} : ldp32(src.sh, 16u * (t.cn + in));
                    In<PH> x{};
                    if constexpr (In<PH>::EDGE) x.g = ldp32(src.g, 16u * (t.ce + entry));
                    if constexpr (In<PH>::BOTH) x.b = *reinterpret_cast<const GAS u64*>(src.b + 8u * (t.ce + entry));
                    u64 o[N];
                    edge_term<PH>(~0ull, le ? 0ull : ~0ull, st, x.g, x.b, o);
#pragma unroll
                    for (int n = 0; n < N; ++n) a[n] = n < NA ? (a[n] & o[n]) : (a[n] | o[n]);
                });
        }
        meet<NA, N>(w1, facts >> R1_STEPS, a);
        Pair v = block_state<PH, false>(c, t, w1, pos, a, q.x);
        if (special) {
            asm volatile("; special");
            v = block_state<PH, true>(c, t, w1, pos, a, q.x);
        }
        v2u o;
        o.x = v.h;
        o.y = v.d;
        *ring(p) = o;
        if ((int32_t)r.x < 0) {   // the block's last lane
            if constexpr (FIRST) {
                *reinterpret_cast<GAS v2u*>(src.st + 16u * (t.cn + pos)) = o;
                if ((w1 >> R1_XSRC) & 1u)
                    if (v != Pair{init, init}) sor(t.chg + (pos >> 5), 1u << (pos & 31));
            } else if (v != q.old) {
                *reinterpret_cast<GAS v2u*>(src.st + 16u * (t.cn + pos)) = o;
                far_reader = max(far_reader, (int)(q.last & 0x7FFFu));
                changed = 1u;
                if ((w1 >> R1_XSRC) & 1u) sor(t.chg + (pos >> 5), 1u << (pos & 31));
            }
        }
    };
    Rec r[AHEAD], rn[AHEAD];
    Slot s[AHEAD];
#pragma unroll
    for (int v = 0; v < AHEAD; ++v) r[v] = record(p0 + v);
    if constexpr (!FIRST) {
        // the passes before the run, as they are
        Rec k[STRIP_RING];
        Pair o[STRIP_RING];
        const int first = max(back, p0 - STRIP_RING);
#pragma unroll
        for (int v = 0; v < STRIP_RING; ++v) k[v] = record(min(first + v, p0));
#pragma unroll
        for (int v = 0; v < STRIP_RING; ++v) o[v] = ldp32(src.st, 16u * (t.cn + ((k[v].x >> R0_POS) & 0x7FFFu)));
#pragma unroll
        for (int v = 0; v < STRIP_RING; ++v) {
            v2u x;
            x.x = o[v].h;
            x.y = o[v].d;
            *ring(min(first + v, p0)) = x;
        }
    }
#pragma unroll
    for (int v = 0; v < AHEAD; ++v) rn[v] = record(p0 + AHEAD + v);
#pragma unroll
    for (int v = 0; v < AHEAD; ++v) load(r[v], s[v]);
    for (int p = p0;;) {
#pragma unroll
        for (int v = 0; v < AHEAD; ++v) {
            if (p + v < p1) visit(p + v, r[v], s[v]);
            r[v] = rn[v];
            load(r[v], s[v]);
            rn[v] = record(p + v + 2 * AHEAD);
        }
        p += AHEAD;
        if (p >= p1) break;
        if constexpr (!FIRST)
            if (p > reach) {
                reach = max(reach, wave_max(far_reader));
                if (p > reach && !more(p)) break;
            }
    }
    if constexpr (!FIRST) reach = max(reach, wave_max(far_reader));
    return changed != 0u;
}

// The fixed point of a phase; false when the sweep cap stops it.  BY_ROWS: the records hold their rows'
// edge entries.
template <int PH, bool BY_ROWS>
__device__ __forceinline__ bool fixed_point(const DevCfg& c, const Strip& t)
{
    constexpr bool BWD = backward(PH);
    const int np = G(c.hdr)[BWD ? SH_PASS_B : SH_PASS_F], nx = G(c.hdr)[BWD ? SH_X_B : SH_X_F];
    const GAS uint32_t* links = G(BWD ? c.x_b : c.x_f);
    const int tid = threadIdx.x, nt = blockDim.x, nw = strip_bit_words(t.nb);
    const Src<PH> src = sources<PH>(c, t);
    // start: next use, pending and delayed copies and the refinement from nothing, validity from
    // everything
    const u64 init = PH == PH_AVE || PH == PH_AVF ? t.vm : 0ull;
    for (int b = tid; b < nw; b += nt) sst(t.chg + b, 0u);
    // Cross links read their sources from `sh`, which changes between rounds only, so that the rounds
    // (and the sweeps reported) do not depend on which wavefront is ahead (reading the states as they
    // are took 4-11 % less in these kernels, and a round more or less from run to run).
    for (int j = tid; j < nx; j += nt) {
        const uint32_t q = links[j] & 0xFFFFu;
        for (int u = 0; u < t.nu; ++u) {
            const int unit = t.u0 + u, bits = t.nv - 64 * unit;
            v2u v;
            v.x = v.y = !(PH == PH_AVE || PH == PH_AVF) ? 0ull : unit == c.wd ? 3ull : bits >= 64 ? ~0ull : (1ull << bits) - 1ull;
            *reinterpret_cast<GAS v2u*>(src.sh + 16u * (uint32_t)(u * t.nb + (int)q)) = v;
        }
    }
    __syncthreads();
    int p0, p1;
    my_run(t, np, p0, p1);
    const int cap = c.sweep_cap > 0 ? c.sweep_cap : 2 * t.nb + 2;
    int sweeps = 1;
    bool changed = false, good = true;
    int reach = -1;
    if (p0 < p1) (void)run_passes<PH, BY_ROWS, true>(c, t, src, p0, p1, p0, init, reach, [](int) { return true; });
    for (int round = 1;; ++round) {
        if (round > 1) {
            const bool any = __syncthreads_or(changed);
            if (any && ++sweeps > cap) { good = false; sweeps = cap; break; }
        } else __syncthreads();
        for (int b = tid; b < nw; b += nt) sst(t.mark + b, 0u);
        __syncthreads();
        bool found = false;
        for (int j = tid; j < nx; j += nt) {
            const uint32_t l = links[j], q = l & 0xFFFFu, p = l >> 16;
            if ((sld(t.chg + (q >> 5)) >> (q & 31)) & 1u) {
                sor(t.mark + (p >> 5), 1u << (p & 31));
                found = true;
                for (int u = 0; u < t.nu; ++u) {
                    const uint32_t at = 16u * (uint32_t)(u * t.nb + (int)q);
                    *reinterpret_cast<GAS v2u*>(src.sh + at) = *reinterpret_cast<const GAS v2u*>(src.st + at);
                }
            }
        }
        if (!__syncthreads_or(found)) break;
        for (int b = tid; b < nw; b += nt) sst(t.chg + b, 0u);
        __syncthreads();
        changed = false;
        reach = -1;
        // the first marked pass at or after p in the run, or p1
        auto next_mark = [&](int p) -> int {
            for (int w0 = p >> 5; (w0 << 5) < p1; w0 += 64) {
                const int w = w0 + t.lane;
                uint32_t m = w < nw ? sld(t.mark + w) : 0u;
                const int low = p - 32 * w;   // bits before p
                if (low > 0) m = low >= 32 ? 0u : m & (~0u << low);
                const u64 some = __builtin_amdgcn_ballot_w64(m != 0u);
                if (some) {
                    const int l = (int)__builtin_ctzll(some);
                    const uint32_t mm = (uint32_t)__builtin_amdgcn_readlane((int)m, l);
                    return min(p1, 32 * (w0 + l) + (int)__builtin_ctz(mm));
                }
            }
            return p1;
        };
        for (int p = next_mark(p0); p < p1;) {
            int end = p1;   // the passes go on to the horizon and over short gaps
            changed |= run_passes<PH, BY_ROWS, false>(c, t, src, p, p1, p0, init, reach, [&](int q) {
                const int m = next_mark(q);
                if (m < p1 && m < q + 32) return true;
                end = m;
                return false;
            });
            p = end;
        }
    }
    __syncthreads();
    if (tid == 0) {
        atomicMax(&c.info[INFO_SWEEPS + PH], sweeps);
        if (!good) set_status(c.info, OMPD_E_NOCONVERGE_);
    }
    return good;
}

// The strip of this workgroup; false if there is nothing to do (the CFG failed).
__device__ __forceinline__ bool open_strip(const DevCfg& c, int u0, int nu, uint32_t* smem, Strip& t)
{
    const int C = c.units, nb = c.nb, nw = strip_bit_words(nb);
    t.lane = threadIdx.x & 63;
    t.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    t.waves = blockDim.x >> 6;
    LDS3 char* base = (LDS3 char*)smem;
    t.ring = base + t.wave * (STRIP_RING * 1024);
    t.chg = (LDS3 uint32_t*)(base + t.waves * (STRIP_RING * 1024));
    t.mark = t.chg + nw;
    t.ctl = (LDS3 int*)(t.mark + nw);
    t.i = t.lane & (ROW - 1);
    t.row = t.lane / ROW;
    const int k = t.row % C;
    t.R = 4 / C;
    t.nb = nb;
    t.nv = c.nv;
    t.nrec = strip_records(c.ne);
    t.u0 = u0;
    t.nu = nu;
    t.on = k < nu;
    t.unit = u0 + min(k, nu - 1);
    t.flg = t.unit == c.wd;
    t.ro = (uint32_t)(k * ROW * 16);
    t.cn = (uint32_t)((t.unit - u0) * nb);
    t.ce = (uint32_t)((t.flg ? 0 : t.unit - u0) * t.nrec);
    t.bn = (size_t)u0 * nb;
    t.be = u0 < c.wd ? (size_t)u0 * t.nrec : 0;
    const int bits = c.nv - 64 * t.unit;
    t.vm = t.flg ? 3ull : bits >= 64 ? ~0ull : (1ull << bits) - 1ull;
    auto word = [&](const u64* a) -> u64 { return t.flg ? 0ull : G(a)[t.unit]; };
    t.fp = word(c.fp);
    t.evh = t.flg ? 2ull : word(c.ev_h);
    t.evd = word(c.ev_d);
    t.lxh = t.flg ? 1ull : word(c.lx_h);
    t.lxd = word(c.lx_d);
    if (threadIdx.x == 0) sst(t.ctl, (int)(G(c.info)[INFO_STATUS] != 0));
    __syncthreads();
    const int skip = __builtin_amdgcn_readfirstlane(sld(t.ctl));
    __syncthreads();
    return !skip;
}

// ---- what follows from a fixed point, block by block ------------------------------------------
// One thread per block and all units of the strip: a block's loads depend on each other (its edges'
// range, their ends, the ends' states) and nothing else does, so a thread takes the units, and two
// blocks, together.
template <class F>
__device__ __forceinline__ void by_units(int nu, F&& f)
{
    if (nu == 1) f(std::integral_constant<int, 1>{});
    else if (nu == 2) f(std::integral_constant<int, 2>{});
    else if (nu > 2) f(std::integral_constant<int, 4>{});
}
// starts of the units in the block and edge arrays (the last one again past the end) and their masks
template <int U> struct UnitRun {
    size_t bo[U], eo[U];
    u64 vm[U];
    int unit[U];
    __device__ __forceinline__ UnitRun(const Strip& t, int wd, int nu)
    {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            unit[u] = t.u0 + (u < nu ? u : nu - 1);
            bo[u] = (size_t)unit[u] * t.nb;
            eo[u] = (size_t)unit[u] * t.nrec;
            const int bits = t.nv - 64 * unit[u];
            vm[u] = bits >= 64 ? ~0ull : (1ull << bits) - 1ull;
        }
    }
};
// The edges into two blocks per thread: first(k, block position, its edges' range, the first edge's
// ends word) for k = 0, 1 after both blocks' words are loaded.
template <class F>
__device__ __forceinline__ void two_blocks(const DevCfg& c, int nb, F&& f)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int b0 = tid; b0 < nb; b0 += 2 * nt) {
        int b[2], a[2], z[2];
        uint32_t l[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            b[k] = min(b0 + k * nt, nb - 1);
            a[k] = G(c.est_f)[b[k]];
            z[k] = G(c.est_f)[b[k] + 1];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) l[k] = G(c.link)[a[k]];
        f(b, a, z, l, b0 + nt < nb);
    }
}

// After eager validity: eager validity in; per edge the eager copies EAG_s(p->q) = NU_s(q) &
// ~AVEout_s(p) and the part of "valid in both spaces" that the pending copies do not change (a loop
// entry: valid before the edge or made so on it; else valid before).
template <int U>
__device__ __forceinline__ void after_ave(const DevCfg& c, const Strip& t, int wd)
{
    const int nu = min(t.u0 + t.nu, wd) - t.u0;
    const UnitRun<U> w(t, wd, nu);
    two_blocks(c, t.nb, [&](const int* b, const int* a, const int* z, const uint32_t* l, bool two) {
        Pair n[2][U], p[2][U];
        int blk[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            blk[k] = G(c.s_lorder)[b[k]];
#pragma unroll
            for (int u = 0; u < U; ++u) { n[k][u] = ldp(c.p_1, w.bo[u] + b[k]); p[k][u] = ldp(c.p_2, w.bo[u] + (l[k] & 0x7FFFu)); }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (k && !two) break;
            Pair m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) m[u] = Pair{~0ull, ~0ull};
            auto edge = [&](int e, uint32_t le, const Pair* q) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    m[u].h &= q[u].h;
                    m[u].d &= q[u].d;
                    if (u >= nu) continue;
                    const Pair nn = n[k][u];
                    stp(c.p_g, w.eo[u] + e, Pair{nn.h & ~q[u].h, nn.d & ~q[u].d});
                    G(c.p_b)[w.eo[u] + e] = (le & 0x8000u) ? ((q[u].h | nn.h) & (q[u].d | nn.d)) : (q[u].h & q[u].d);
                }
            };
            edge(a[k], l[k], p[k]);
            for (int e = a[k] + 1; e < z[k]; ++e) {
                const uint32_t le = G(c.link)[e];
                Pair q[U];
#pragma unroll
                for (int u = 0; u < U; ++u) q[u] = ldp(c.p_2, w.bo[u] + (le & 0x7FFFu));
                edge(e, le, q);
            }
            const bool entry = blk[k] == c.entry;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u < nu)
                    stp(c.p_3, w.bo[u] + b[k], Pair{(entry ? G(c.ev_h)[w.unit[u]] : n[k][u].h | m[u].h) & w.vm[u],
                                                    (entry ? G(c.ev_d)[w.unit[u]] : n[k][u].d | m[u].d) & w.vm[u]});
        }
    });
}

// After the delayed placement: the copies, before a block what reaches it delayed and it uses, on
// an edge what does not go on into the block.
template <int U>
__device__ __forceinline__ void after_later(const DevCfg& c, const Strip& t, int nu)
{
    const UnitRun<U> w(t, c.wd, nu);
    u64 fp[U];
#pragma unroll
    for (int u = 0; u < U; ++u) fp[u] = G(c.fp)[w.unit[u]];
    two_blocks(c, t.nb, [&](const int* b, const int* a, const int* z, const uint32_t* l, bool two) {
        Pair p[2][U], g[2][U];
        u64 bo[2][U], rr[2][U];
        int blk[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            blk[k] = G(c.s_lorder)[b[k]];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                p[k][u] = ldp(c.p_1, w.bo[u] + (l[k] & 0x7FFFu));
                g[k][u] = ldp(c.p_g, w.eo[u] + a[k]);
                bo[k][u] = G(c.p_b)[w.eo[u] + a[k]];
                rr[k][u] = ldp(c.p_rw, w.bo[u] + b[k]).h;
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (k && !two) break;
            if (blk[k] == c.entry) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (u < nu) stp(c.p_2, w.bo[u] + b[k], Pair{0, 0});
                continue;
            }
            u64 m[U][4];
#pragma unroll
            for (int u = 0; u < U; ++u) { m[u][0] = m[u][1] = ~0ull; m[u][2] = m[u][3] = 0ull; }
            auto meet_edge = [&](uint32_t le, int u, const Pair& q, const Pair& gq, u64 bq) {
                u64 o[4];
                edge_term<PH_LATER>(~0ull, ~bit_mask(le, 15), q, gq, bq, o);
                m[u][0] &= o[0]; m[u][1] &= o[1]; m[u][2] |= o[2]; m[u][3] |= o[3];
            };
#pragma unroll
            for (int u = 0; u < U; ++u) meet_edge(l[k], u, p[k][u], g[k][u], bo[k][u]);
            for (int e = a[k] + 1; e < z[k]; ++e) {
                const uint32_t le = G(c.link)[e];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    meet_edge(le, u, ldp(c.p_1, w.bo[u] + (le & 0x7FFFu)), ldp(c.p_g, w.eo[u] + e), G(c.p_b)[w.eo[u] + e]);
            }
            Pair in[U];
#pragma unroll
            for (int u = 0; u < U; ++u) in[u] = Pair{m[u][0] & m[u][2] & w.vm[u], m[u][1] & m[u][3] & w.vm[u]};
            auto edge = [&](int e, uint32_t le, int u, const Pair& q, const Pair& gq) {
                const u64 x = bit_mask(le, 15);
                if (u < nu)
                    stp(c.p_g, w.eo[u] + e, Pair{(gq.h | q.h) & (x | ~in[u].h) & w.vm[u], (gq.d | q.d) & (x | ~in[u].d) & w.vm[u]});
            };
#pragma unroll
            for (int u = 0; u < U; ++u) edge(a[k], l[k], u, p[k][u], g[k][u]);
            for (int e = a[k] + 1; e < z[k]; ++e) {
                const uint32_t le = G(c.link)[e];
                Pair q[U], gq[U];
#pragma unroll
                for (int u = 0; u < U; ++u) { q[u] = ldp(c.p_1, w.bo[u] + (le & 0x7FFFu)); gq[u] = ldp(c.p_g, w.eo[u] + e); }
#pragma unroll
                for (int u = 0; u < U; ++u) edge(e, le, u, q[u], gq[u]);
            }
            const u64 dev = G(c.space)[blk[k]] ? ~0ull : 0ull;
            const int ci = c.call ? G(c.call)[blk[k]] : -1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                Pair us{rr[k][u] & (~dev | fp[u]), rr[k][u] & dev & ~fp[u]};
                if (blk[k] == c.exit) us = Pair{G(c.lx_h)[w.unit[u]], G(c.lx_d)[w.unit[u]]};
                if (ci >= 0) {
                    const GAS u64* sm = G(c.sums) + (size_t)ci * SUM_ROWS * c.wd + w.unit[u];
                    const u64 mw = sm[SUM_MAYW_H * c.wd] | sm[SUM_MAYW_D * c.wd];
                    us.h |= sm[SUM_MAYR_H * c.wd] | mw;
                    us.d |= sm[SUM_MAYR_D * c.wd] | mw;
                }
                if (u < nu) stp(c.p_2, w.bo[u] + b[k], Pair{in[u].h & us.h, in[u].d & us.d});
            }
        }
    });
}

// After the final validity: final validity in, and the map-kind masks ([units][to, from, used on the
// device, firstprivate], two LDS words each).
template <int U>
__device__ __forceinline__ void after_avf(const DevCfg& c, const Strip& t, int nu, LDS3 uint32_t* kinds)
{
    const UnitRun<U> w(t, c.wd, nu);
    u64 fp[U], acc[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        fp[u] = G(c.fp)[w.unit[u]];
        acc[u][0] = acc[u][1] = acc[u][2] = acc[u][3] = 0ull;
    }
    two_blocks(c, t.nb, [&](const int* b, const int* a, const int* z, const uint32_t* l, bool two) {
        Pair p[2][U], g[2][U], ie[2][U], rw[2][U];
        int blk[2];
        u64 no_dev[2], clear[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            blk[k] = G(c.s_lorder)[b[k]];
            no_dev[k] = (G(c.facts)[b[k]] & FACT_BEFORE) ? 0ull : ~0ull;           // no DEVICE block follows
            clear[k] = (G(c.facts)[l[k] & 0x7FFFu] & FACT_AFTER) ? 0ull : ~0ull;   // ... or comes before the edge
#pragma unroll
            for (int u = 0; u < U; ++u) {
                p[k][u] = ldp(c.p_1, w.bo[u] + (l[k] & 0x7FFFu));
                g[k][u] = ldp(c.p_g, w.eo[u] + a[k]);
                ie[k][u] = ldp(c.p_2, w.bo[u] + b[k]);
                rw[k][u] = ldp(c.p_rw, w.bo[u] + b[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (k && !two) break;
            const bool entry = blk[k] == c.entry, kernel = G(c.space)[blk[k]] && blk[k] != c.exit;
            Pair m[U];
            u64 none = ~0ull;
#pragma unroll
            for (int u = 0; u < U; ++u) m[u] = Pair{~0ull, ~0ull};
            auto edge = [&](int u, const Pair& q, const Pair& gq, u64 cl) {
                m[u].h &= q.h | gq.h;
                m[u].d &= q.d | gq.d;
                acc[u][0] |= gq.d & cl;
                acc[u][1] |= gq.h & no_dev[k];
            };
            if (!entry) {
                none &= clear[k];
#pragma unroll
                for (int u = 0; u < U; ++u) edge(u, p[k][u], g[k][u], clear[k]);
                for (int e = a[k] + 1; e < z[k]; ++e) {
                    const int q = (int)(G(c.link)[e] & 0x7FFFu);
                    const u64 cl = (G(c.facts)[q] & FACT_AFTER) ? 0ull : ~0ull;
                    none &= cl;
#pragma unroll
                    for (int u = 0; u < U; ++u) edge(u, ldp(c.p_1, w.bo[u] + q), ldp(c.p_g, w.eo[u] + e), cl);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                Pair in{G(c.ev_h)[w.unit[u]], G(c.ev_d)[w.unit[u]]};
                if (!entry) {
                    in = Pair{ie[k][u].h | m[u].h, ie[k][u].d | m[u].d};
                    acc[u][0] |= ie[k][u].d & none;
                    acc[u][1] |= ie[k][u].h & no_dev[k];
                }
                if (kernel) {
                    acc[u][2] |= (rw[k][u].h & ~fp[u]) | rw[k][u].d;
                    acc[u][3] |= rw[k][u].h & fp[u];
                }
                if (u < nu) stp(c.p_3, w.bo[u] + b[k], Pair{in.h & w.vm[u], in.d & w.vm[u]});
            }
        }
    });
    if (!c.var_kind) return;
#pragma unroll
    for (int u = 0; u < U; ++u)
        for (int k = 0; k < 4; ++k) {
            if (u >= nu) continue;
            LDS3 uint32_t* o = kinds + 8 * u + 2 * k;
            if ((uint32_t)acc[u][k]) sor(o, (uint32_t)acc[u][k]);
            if ((uint32_t)(acc[u][k] >> 32)) sor(o + 1, (uint32_t)(acc[u][k] >> 32));
        }
}

// Next use and eager validity of a strip, and what follows from them.
//
// What bounds it: alone on a compute unit a visit is a chain of ~100 vector instructions and one
// LDS round trip, 0.27-0.33 us, and a CFG's rounds are as long as its wavefronts' runs; the
// registers (the inputs loaded ahead) leave room for two wavefronts per SIMD, whose visits then take
// 0.4 us.  A batch's strips also wait for memory: each round reads a strip's arrays again (about 1 MB
// for 4,000 blocks and 4 words), the resident ones exceed the last-level cache, and both strip
// kernels move data at 3.3-3.8 TB/s (a copy: 4.9).  Rows of 8 lanes and 8 words per strip need a quarter
// fewer passes but twice the arrays per strip: 1024 CFGs the same or slower (strip_b 8.0 -> 8.8 ms);
// 4 wavefronts per SIMD with inputs loaded 3-4 passes ahead are no faster either.
// Both strip kernels, before (the phase and pass kernels of the walk or of the old level schedule) ->
// now: 66 blocks x 32 variables 0.55 -> 0.17 ms, 8002 x 1500 31 -> 2.8 ms, 16386 x
// 2048 68 -> 5.7 ms, 1024 CFGs 76 -> 10.5 ms.
extern "C" __global__ void __launch_bounds__(64 * STRIP_MAX_WAVES)
ompd_k_strip_a(const DevCfg* __restrict__ cfgs, const Tile* __restrict__ tiles)
{
    extern __shared__ __align__(16) uint32_t smem[];
    const Tile tl = tiles[blockIdx.x];
    const DevCfg& c = cfgs[tl.cfg];
    Strip t;
    if (!open_strip(c, tl.s0, tl.nw, smem, t)) return;
    const int tid = threadIdx.x, nt = blockDim.x, nb = t.nb, wd = c.wd;
    const bool with_facts = tl.s0 + tl.nw == wd + 1;
    const size_t fo = (size_t)wd * nb;
    if (!fixed_point<PH_NU, false>(c, t)) return;
    if (with_facts) {
        // bit 0 of the host word: the block reaches EXIT; bit 1 of the device word: it reaches a
        // DEVICE block; the word takes part in the validity without next use
        bool bad = false;
        for (int b = tid; b < nb; b += nt) {
            const Pair v = ldp(c.p_1, fo + b);
            stp(c.p_1, fo + b, Pair{0, 0});
            G(c.facts)[b] = (v.d & 2) ? FACT_BEFORE : 0;
            if (!(v.h & 1)) bad = true;
        }
        if (bad) set_status(c.info, OMPD_E_INVAL_);
        __syncthreads();
    }
    if (!fixed_point<PH_AVE, false>(c, t)) return;
    if (with_facts) {
        // bit 0 of the host word: not reached from ENTRY; bit 1: no DEVICE block reaches the block
        bool bad = false;
        for (int b = tid; b < nb; b += nt) {
            const Pair v = ldp(c.p_2, fo + b);
            const uint8_t before = G(c.facts)[b], after = (v.h & 2) ? 0 : FACT_AFTER;
            G(c.facts)[b] = before | after;
            if (v.h & 1) bad = true;
            const int blk = G(c.s_lorder)[b];
            if (c.after_dev) G(c.after_dev)[blk] = after ? 1 : 0;
            if (c.before_dev) G(c.before_dev)[blk] = before ? 1 : 0;
        }
        if (bad) set_status(c.info, OMPD_E_INVAL_);
    }
    by_units(min(tl.s0 + tl.nw, wd) - tl.s0, [&](auto uc) { after_ave<decltype(uc)::value>(c, t, wd); });
}

// Pending copies, placement, refinement and final validity of a strip, and the map kinds of its
// variables.  BY_ROWS has kernels of its own: a branch around those few instructions in the others
// costs them 3 % (strip_b, 2048 small CFGs: 331 -> 343 us, 779 blocks 412 -> 424 us).
template <bool BY_ROWS>
__device__ __forceinline__ void strip_b(const DevCfg* __restrict__ cfgs, const Tile* __restrict__ tiles, uint32_t* smem)
{
    const Tile tl = tiles[blockIdx.x];
    const DevCfg& c = cfgs[tl.cfg];
    const int wd = c.wd, nu = min(tl.nw, wd - tl.s0);   // (the word of facts is done)
    if (nu <= 0) return;
    Strip t;
    if (!open_strip(c, tl.s0, nu, smem, t)) return;
    const int tid = threadIdx.x, nt = blockDim.x, nb = t.nb;
    if (c.placement & PL_EAGER) {
        // every eager copy stays on its edge
        for (int b = tid; b < nu * nb; b += nt) stp(c.p_2, (size_t)tl.s0 * nb + b, Pair{0, 0});
    } else {
        if (!fixed_point<PH_MAYP, BY_ROWS>(c, t)) return;
        // valid in both spaces on an edge: no copy pending across it
        by_units(nu, [&](auto uc) {
            constexpr int U = decltype(uc)::value;
            const UnitRun<U> w(t, c.wd, nu);
#pragma unroll 2
            for (int e = tid; e < t.nrec; e += nt) {
                const uint32_t l = G(c.link)[e];
                const u64 keep = bit_mask(l, 15);
                Pair p[U];
                u64 b[U];
#pragma unroll
                for (int u = 0; u < U; ++u) { p[u] = ldp(c.p_2, w.bo[u] + (l & 0x7FFFu)); b[u] = G(c.p_b)[w.eo[u] + e]; }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (u < nu) G(c.p_b)[w.eo[u] + e] = b[u] & (keep | ~(p[u].h | p[u].d));
            }
        });
        __syncthreads();
        if (!fixed_point<PH_LATER, BY_ROWS>(c, t)) return;
        by_units(nu, [&](auto uc) { after_later<decltype(uc)::value>(c, t, nu); });
        __syncthreads();
        if (refines(c.placement)) {
            if (!fixed_point<PH_LIVE, BY_ROWS>(c, t)) return;
            // a copy on a loop entry whose value nothing reads is dropped
            for (int u = tl.s0; u < tl.s0 + nu; ++u)
                for (int e = tid; e < t.nrec; e += nt) {
                    const uint32_t l = G(c.link)[e];
                    if (!(l & 0x8000u)) continue;
                    const size_t at = (size_t)u * t.nrec + e;
                    const Pair p = ldp(c.p_1, (size_t)u * nb + (l >> 16)), g = ldp(c.p_g, at);
                    stp(c.p_g, at, Pair{g.h & p.h, g.d & p.d});
                }
        }
    }
    __syncthreads();
    if (!fixed_point<PH_AVF, BY_ROWS>(c, t)) return;
    LDS3 uint32_t* kinds = (LDS3 uint32_t*)(t.ctl + 16);   // [units][to, from, used on the device, firstprivate]
    if (tid < 32) sst(kinds + tid, 0u);
    __syncthreads();
    by_units(nu, [&](auto uc) { after_avf<decltype(uc)::value>(c, t, nu, kinds); });
    if (!c.var_kind) return;
    __syncthreads();
    for (int j = tid; j < 64 * nu; j += nt) {
        const int v = 64 * tl.s0 + j;
        if (v >= c.nv) continue;
        const LDS3 uint32_t* o = kinds + 8 * (j >> 6) + ((j >> 5) & 1);
        auto bit = [&](int k) -> uint32_t { return (sld(o + 2 * k) >> (j & 31)) & 1u; };
        const uint32_t t1 = bit(0), f1 = bit(1), d1 = bit(2), q1 = bit(3);
        G(c.var_kind)[v] = (uint8_t)(t1 | (f1 << 1) | ((d1 && !t1 && !f1) ? 4u : 0u) | (q1 << 3));
    }
}

extern "C" __global__ void __launch_bounds__(64 * STRIP_MAX_WAVES)
ompd_k_strip_b(const DevCfg* __restrict__ cfgs, const Tile* __restrict__ tiles)
{
    extern __shared__ __align__(16) uint32_t smem[];
    strip_b<false>(cfgs, tiles, smem);
}

extern "C" __global__ void __launch_bounds__(64 * STRIP_MAX_WAVES)
ompd_k_strip_b_rows(const DevCfg* __restrict__ cfgs, const Tile* __restrict__ tiles)
{
    extern __shared__ __align__(16) uint32_t smem[];
    strip_b<true>(cfgs, tiles, smem);
}

// --------------------------------------------------------------------------
// transposes between the caller's rows and the strips' pairs
// --------------------------------------------------------------------------
// An item: a CFG, a run of up to T_WORDS words and a chunk of T_ROWS positions (b0 >= 0) or of
// T_ROWS edge entries (b0 < 0: from ~b0).
constexpr int T_WORDS = STRIP_T_WORDS, T_ROWS = STRIP_T_ROWS;
struct TTile { u64 h[T_ROWS][T_WORDS + 1], d[T_ROWS][T_WORDS + 1]; };

extern "C" __global__ void __launch_bounds__(256) ompd_k_tin(const DevCfg* __restrict__ cfgs, const EdgeItem* __restrict__ items)
{
    __shared__ TTile tile;
    const EdgeItem it = items[blockIdx.x];
    const DevCfg& c = cfgs[it.cfg];
    if (G(c.info)[INFO_STATUS] != 0) return;
    const int tid = threadIdx.x, nb = c.nb, wd = c.wd;
    const int n = min(T_ROWS, nb - it.b0);
    if (it.s0 == 0)
        // the word of facts: every block "reads" bit 1, DEVICE blocks "write" it
        for (int j = tid; j < n; j += 256)
            stp(c.p_rw, (size_t)wd * nb + it.b0 + j, Pair{2ull, G(c.space)[G(c.s_lorder)[it.b0 + j]] ? 2ull : 0ull});
    const int w = tid % T_WORDS;
    if (w < it.nw)
        for (int r = tid / T_WORDS; r < n; r += 256 / T_WORDS) {
            const size_t at = (size_t)G(c.s_lorder)[it.b0 + r] * wd + it.s0 + w;
            tile.h[r][w] = G(c.R)[at];
            tile.d[r][w] = G(c.W)[at];
        }
    __syncthreads();
    const int r = tid % T_ROWS;
    if (r < n)
        for (int k = tid / T_ROWS; k < it.nw; k += 256 / T_ROWS)
            stp(c.p_rw, (size_t)(it.s0 + k) * nb + it.b0 + r, Pair{tile.h[r][k], tile.d[r][k]});
}

// n pairs of each of `words` words (stride `str`, from entry `at`) to the caller's rows (NULL: not
// asked for), entry r to row row_of(r) (negative: none)
template <class RowOf>
__device__ __forceinline__ void pairs_to_rows(TTile& tile, const u64* src, u64* h, u64* d, int n, size_t str, size_t at,
                                              int s0, int words, int wd, RowOf&& row_of)
{
    if (!h && !d) return;
    const int tid = threadIdx.x, r = tid % T_ROWS;
    if (r < n)
        for (int k = tid / T_ROWS; k < words; k += 256 / T_ROWS) {
            const Pair p = ldp(src, (size_t)(s0 + k) * str + at + r);
            tile.h[r][k] = p.h;
            tile.d[r][k] = p.d;
        }
    __syncthreads();
    const int w = tid % T_WORDS;
    if (w < words)
        for (int q = tid / T_WORDS; q < n; q += 256 / T_WORDS) {
            const int to = row_of(q);
            if (to < 0) continue;
            if (h) G(h)[(size_t)to * wd + s0 + w] = tile.h[q][w];
            if (d) G(d)[(size_t)to * wd + s0 + w] = tile.d[q][w];
        }
    __syncthreads();
}

// next use and eager validity
extern "C" __global__ void __launch_bounds__(256) ompd_k_tmid(const DevCfg* __restrict__ cfgs, const EdgeItem* __restrict__ items)
{
    __shared__ TTile tile;
    const EdgeItem it = items[blockIdx.x];
    const DevCfg& c = cfgs[it.cfg];
    if (G(c.info)[INFO_STATUS] != 0 || it.nw == 0) return;
    const int n = min(T_ROWS, c.nb - it.b0);
    auto block = [&](int q) -> int { return G(c.s_lorder)[it.b0 + q]; };
    auto asked = [&](int bit, u64* a) -> u64* { return (c.want & bit) ? a : nullptr; };
    pairs_to_rows(tile, c.p_1, asked(WANT_NU_H, c.nu_h), asked(WANT_NU_D, c.nu_d), n, c.nb, it.b0, it.s0, it.nw, c.wd, block);
    pairs_to_rows(tile, c.p_3, asked(WANT_AVE_H, c.ave_h), asked(WANT_AVE_D, c.ave_d), n, c.nb, it.b0, it.s0, it.nw, c.wd, block);
}

// final validity, the copies, the firstprivate clauses
extern "C" __global__ void __launch_bounds__(256) ompd_k_tout(const DevCfg* __restrict__ cfgs, const EdgeItem* __restrict__ items)
{
    __shared__ TTile tile;
    const EdgeItem it = items[blockIdx.x];
    const DevCfg& c = cfgs[it.cfg];
    if (G(c.info)[INFO_STATUS] != 0 || it.nw == 0) return;
    auto asked = [&](int bit, u64* a) -> u64* { return (c.want & bit) ? a : nullptr; };
    if (it.b0 < 0) {
        const int e0 = ~it.b0, nrec = strip_records(c.ne), n = min(T_ROWS, nrec - e0);
        pairs_to_rows(tile, c.p_g, asked(WANT_IG_H, c.ig_h), asked(WANT_IG_D, c.ig_d), n, nrec, e0, it.s0, it.nw, c.wd,
                      [&](int q) -> int { return G(c.eid)[e0 + q]; });
        return;
    }
    const int n = min(T_ROWS, c.nb - it.b0);
    auto block = [&](int q) -> int { return G(c.s_lorder)[it.b0 + q]; };
    pairs_to_rows(tile, c.p_3, asked(WANT_AVF_H, c.avf_h), asked(WANT_AVF_D, c.avf_d), n, c.nb, it.b0, it.s0, it.nw, c.wd, block);
    pairs_to_rows(tile, c.p_2, asked(WANT_IE_H, c.ie_h), asked(WANT_IE_D, c.ie_d), n, c.nb, it.b0, it.s0, it.nw, c.wd, block);
    if (c.fpc) {
        const int w = threadIdx.x % T_WORDS;
        if (w < it.nw)
            for (int q = threadIdx.x / T_WORDS; q < n; q += 256 / T_WORDS) {
                const int b = block(q);
                const size_t at = (size_t)b * c.wd + it.s0 + w;
                G(c.fpc)[at] = G(c.space)[b] ? (G(c.R)[at] & G(c.fp)[it.s0 + w]) : 0ull;
            }
    }
}

}  // namespace ompd
