// Device code shared by the ingest kernels and the solvers (internal).
#pragma once
#include <hip/hip_runtime.h>

#include "ompd_device.h"

#define OMPD_E_INVAL_ (-1)
#define OMPD_E_DEVICE_ (-3)
#define OMPD_E_NOCONVERGE_ (-4)

namespace ompd {

// Views of generic pointers as global-memory pointers: loads and stores
// through them compile to global_load/global_store, which only count
// against vmcnt, so a wait for LDS does not also drain outstanding
// global prefetches (flat accesses would count against both).
#define GAS __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ const GAS T* G(const T* p) { return (const GAS T*)p; }
template <typename T>
__device__ __forceinline__ GAS T* G(T* p) { return (GAS T*)p; }

__device__ __forceinline__ void set_status(int32_t* info, int32_t code)
{
    atomicCAS(&info[INFO_STATUS], 0, code);
}

// Does an edge of kind k stop the delay?  Loop entries do, unless the placement is pure lazy.
__device__ __forceinline__ bool is_le(const DevCfg& c, uint8_t k) { return k == 2 && !(c.placement & PL_LAZY); }

// Inclusive prefix sum of a[0..n) in global memory by one workgroup.
__device__ void block_scan_inclusive(int32_t* a, int n, int32_t* sh)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int carry = 0;
    for (int base = 0; base < n; base += blockDim.x) {
        int i = base + threadIdx.x;
        int x = (i < n) ? a[i] : 0;
        for (int d = 1; d < 64; d <<= 1) {
            int y = __shfl_up(x, d, 64);
            if (lane >= d) x += y;
        }
        if (lane == 63) sh[wv] = x;
        __syncthreads();
        int off = carry, tot = 0;
        for (int j = 0; j < nw; ++j) {
            if (j < wv) off += sh[j];
            tot += sh[j];
        }
        __syncthreads();
        if (i < n) a[i] = x + off;
        carry += tot;
    }
    __syncthreads();
}

// Ingest of one CFG by its workgroup: clears the status words and the CFG's masks, checks the CSR,
// the boundary rules and the rows (stage 1: what the later stages index with; stage 2: the rest),
// and finds the firstprivate variables.  False (status set) for a malformed CFG.
__device__ inline bool validate_cfg(const DevCfg& c, int& s_err)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    const int nb = c.nb, ne = c.ne, wd = c.wd;
    if (tid == 0) s_err = 0;
    for (int i = tid; i < INFO_WORDS; i += nt) c.info[i] = 0;
    if (c.var_kind)
        for (int i = tid; i < 4 * wd; i += nt) c.vk_acc[i] = 0;
    for (int w = tid; w < wd; w += nt) c.fp[w] = 0;
    __syncthreads();

    // validation, stage 1: pointers, kinds, spaces
    int err = 0;
    if (tid == 0 && (c.succ_ptr[0] != 0 || c.succ_ptr[nb] != ne)) err = 1;
    for (int b = tid; b < nb; b += nt) {
        int a = c.succ_ptr[b], z = c.succ_ptr[b + 1];
        if (z < a || a < 0 || z > ne) err = 1;
        if (c.space[b] > 1) err = 1;
    }
    for (int e = tid; e < ne; e += nt)
        if (c.kind[e] > 2) err = 1;
    if (tid == 0 && (c.space[c.entry] != 0 || c.space[c.exit] != 0)) err = 1;
    if (err) atomicOr(&s_err, 1);
    __syncthreads();
    if (s_err) { if (tid == 0) c.info[INFO_STATUS] = OMPD_E_INVAL_; return false; }

    // stage 2: successor targets, ENTRY/EXIT rules, bit rows, boundaries, calls
    if (tid == 0 && c.succ_ptr[c.exit + 1] != c.succ_ptr[c.exit]) err = 1;
    for (int e = tid; e < ne; e += nt) {
        int q = c.succ_idx[e];
        if (q < 0 || q >= nb || q == c.entry) err = 1;
        else if (q == c.exit && c.kind[e] != 0) err = 1;
    }
    for (int e = c.succ_ptr[c.entry] + tid; e < c.succ_ptr[c.entry + 1]; e += nt)
        if (c.kind[e] == 1) err = 1;
    for (int b = tid; b < nb; b += nt)
        if (c.succ_ptr[b + 1] - c.succ_ptr[b] > (int)REC_COUNT) err = 1;
    if (wd > 0) {
        const uint64_t last = (c.nv & 63) ? ((1ull << (c.nv & 63)) - 1ull) : ~0ull;
        for (int w = tid; w < wd; w += nt) {
            uint64_t m = (w == wd - 1) ? last : ~0ull;
            if (c.R[(size_t)c.entry * wd + w] | c.W[(size_t)c.entry * wd + w] |
                c.R[(size_t)c.exit * wd + w] | c.W[(size_t)c.exit * wd + w]) err = 1;
            uint64_t eh = c.ev_h[w], ed = c.ev_d[w];
            if ((eh | ed | c.lx_h[w] | c.lx_d[w]) & ~m) err = 1;
            if (!(c.placement & PL_SUMMARY) && ((eh | ed) & m) != m) err = 1;   // a summary evaluation may leave gaps
        }
        for (int b = tid; b < nb; b += nt)
            if ((c.R[(size_t)b * wd + wd - 1] | c.W[(size_t)b * wd + wd - 1]) & ~last) err = 1;
    }
    if (c.call) {
        for (int b = tid; b < nb; b += nt) {
            int k = c.call[b];
            if (k >= 0 && (k >= c.n_sums || c.space[b] != 0 || b == c.entry || b == c.exit)) err = 1;
        }
    }
    if (err) atomicOr(&s_err, 1);
    __syncthreads();
    if (s_err) { if (tid == 0) c.info[INFO_STATUS] = OMPD_E_INVAL_; return false; }

    // firstprivate variables: marked scalars that no DEVICE block writes (the OR of the device
    // blocks' writes gathers in c.fp first)
    if (c.scalar && wd > 0) {
        for (size_t i = tid; i < (size_t)nb * wd; i += nt) {
            const int b = (int)(i / wd), w = (int)(i % wd);
            if (c.space[b]) {
                const uint64_t x = c.W[i];
                if (x) atomicOr((unsigned long long*)&c.fp[w], (unsigned long long)x);
            }
        }
        __syncthreads();
        const uint64_t last = (c.nv & 63) ? ((1ull << (c.nv & 63)) - 1ull) : ~0ull;
        for (int w = tid; w < wd; w += nt) {
            // the atomics above ran in L2: read their result there, past this CU's cache
            const uint64_t dw = __hip_atomic_load(&c.fp[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            c.fp[w] = c.scalar[w] & ~dw & (w == wd - 1 ? last : ~0ull);
        }
        __syncthreads();
    }
    return true;
}

}  // namespace ompd
