// tj_kernels.hip - gfx950 kernels of the tensor-path sort and equi-join.
//
// Everything here is integer work bound by memory traffic (the paper places
// the cost of joins and sorts in data movement and intermediate results, not
// arithmetic: Sec. I, Sec. II.C), so no matrix cores are used. The building
// blocks are wave64 primitives:
//   - ballot-based match: lanes holding the same digit find each other with one
//     ballot per digit bit, which gives each row its stable rank among equal
//     digits in the wavefront;
//   - DPP prefix sums (row_shr 1/2/4/8, row_bcast 15/31) for offsets;
//   - LDS staging so that rows leave a tile as per-digit runs (coalesced).
//
// Keys are mapped to "ordinals" that compare as unsigned integers in the same
// order as the signed keys (flip the sign bit); digits are taken from
// (ordinal - base) so that only the bits that vary inside a bucket are used.
#include "tj_internal.h"
#include "tj_rmi.h"

#include <algorithm>
#include <type_traits>

namespace tj {

// ---------------------------------------------------------------------------
// key <-> ordinal
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t ord_of(int32_t k) { return (uint64_t)((uint32_t)k ^ 0x80000000u); }
__device__ __forceinline__ uint64_t ord_of(int64_t k) { return (uint64_t)k ^ 0x8000000000000000ull; }
template <typename K> __device__ __forceinline__ K key_of(uint64_t o);
template <> __device__ __forceinline__ int32_t key_of<int32_t>(uint64_t o)
{
    return (int32_t)((uint32_t)o ^ 0x80000000u);
}
template <> __device__ __forceinline__ int64_t key_of<int64_t>(uint64_t o)
{
    return (int64_t)(o ^ 0x8000000000000000ull);
}

// Workgroup barrier that orders LDS traffic only. Blocks here never hand data
// to each other through global memory inside a launch (global reads that feed
// LDS complete before their LDS write, by data dependence), so outstanding
// global stores need not drain at a barrier; a plain __syncthreads() would wait
// for them (vmcnt(0)) and serialise store latency into every tile.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---------------------------------------------------------------------------
// wave64 primitives
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// number of set bits of m in lanes below this lane
__device__ __forceinline__ uint32_t mbcnt(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint32_t lane_id() { return mbcnt(~0ull); }

// p[min(q, n - 1)], n >= 1. The load is unconditional (the clamped index
// always names a real element), so an unrolled batch of them is issued before
// the first wait; a guarded load would wait on each one in turn.
template <typename T>
__device__ __forceinline__ T ld_clamp(const T* __restrict__ p, uint64_t q, uint64_t n)
{
    return p[q < n ? q : n - 1];
}

// p[i] for a byte offset below 2^32: a uniform base and a 32-bit offset a lane,
// where 64-bit addresses would take two registers for every load in flight.
template <typename T>
__device__ __forceinline__ T at32(const T* __restrict__ p, uint32_t i)
{
    return *(const T*)((const char*)p + (uint32_t)(i * (uint32_t)sizeof(T)));
}

// at32, issued where it stands: the compiler moves plain loads to their first
// use and waits on each one there.
template <typename T>
__device__ __forceinline__ T ld_now(const T* __restrict__ p, uint32_t i)
{
    return __hip_atomic_load((const T*)((const char*)p + (uint32_t)(i * (uint32_t)sizeof(T))), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// A value that is the same in all lanes, for scalar registers (arguments of a
// call that is not inlined arrive in vector registers).
template <typename T>
__device__ __forceinline__ T uniform(T x)
{
    if constexpr (sizeof(T) == 8) {
        const uint64_t v = (uint64_t)x;
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
        return (T)((uint64_t)hi << 32 | lo);
    } else {
        return (T)__builtin_amdgcn_readfirstlane((int)x);
    }
}

// Inclusive prefix sum across the 64 lanes with DPP: shifts of 1, 2, 4, 8
// inside each row of 16 lanes, then row_bcast:15 carries row totals into rows
// 1 and 3 and row_bcast:31 carries the first half's total into rows 2 and 3.
// Lanes whose DPP source is out of range (or whose row is masked off) read the
// `old` operand, 0, so every step is v += shifted-or-zero.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

__device__ __forceinline__ uint64_t wave_incl_scan64(uint64_t v)
{
    const uint32_t l = lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint64_t t = __shfl_up(v, (unsigned)d, 64);
        if (l >= (uint32_t)d) v += t;
    }
    return v;
}

__device__ __forceinline__ uint64_t wave_sum64(uint64_t v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

__device__ __forceinline__ uint64_t wave_min64(uint64_t v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        uint64_t t = __shfl_xor(v, d, 64);
        v = t < v ? t : v;
    }
    return v;
}

__device__ __forceinline__ uint64_t wave_max64(uint64_t v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        uint64_t t = __shfl_xor(v, d, 64);
        v = t > v ? t : v;
    }
    return v;
}

__device__ __forceinline__ uint64_t wave_or64(uint64_t v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v |= __shfl_xor(v, d, 64);
    return v;
}

// Exclusive prefix of one value per thread over the block (NT threads);
// `tmp` holds NT/64 words of LDS. Returns the prefix; *total gets the sum.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* tmp, uint32_t* total)
{
    constexpr int NW = NT / 64;
    const uint32_t w = threadIdx.x / 64;
    uint32_t inc = wave_incl_scan(v);
    if ((threadIdx.x & 63) == 63) tmp[w] = inc;
    lds_barrier();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NW; i++) {
        uint32_t t = tmp[i];
        off += ((uint32_t)i < w) ? t : 0u;
        tot += t;
    }
    lds_barrier();
    *total = tot;
    return off + inc - v;
}

template <int NT>
__device__ __forceinline__ uint64_t block_sum64(uint64_t v, uint64_t* tmp)
{
    constexpr int NW = NT / 64;
    v = wave_sum64(v);
    if ((threadIdx.x & 63) == 0) tmp[threadIdx.x / 64] = v;
    lds_barrier();
    uint64_t tot = 0;
#pragma unroll
    for (int i = 0; i < NW; i++) tot += tmp[i];
    lds_barrier();
    return tot;
}

// Smallest and largest ordinal of the block's rows, from each thread's own.
template <int NT>
__device__ __forceinline__ void block_minmax64(uint64_t& lo, uint64_t& hi, uint64_t* tmp)
{
    constexpr int NW = NT / 64;
    lo = wave_min64(lo);
    hi = wave_max64(hi);
    if ((threadIdx.x & 63) == 0) tmp[threadIdx.x / 64] = lo;
    lds_barrier();
#pragma unroll
    for (int i = 0; i < NW; i++) lo = tmp[i] < lo ? tmp[i] : lo;
    lds_barrier();
    if ((threadIdx.x & 63) == 0) tmp[threadIdx.x / 64] = hi;
    lds_barrier();
#pragma unroll
    for (int i = 0; i < NW; i++) hi = tmp[i] > hi ? tmp[i] : hi;
    lds_barrier();
}

// Inclusive running maximum across the wave (same DPP pattern as the sum; 0 is
// the identity, values are non-negative).
__device__ __forceinline__ uint32_t wave_incl_max(uint32_t v)
{
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
    return v;
}

// Maximum over the values of all threads before this one (0 for thread 0).
template <int NT>
__device__ __forceinline__ uint32_t block_excl_max(uint32_t v, uint32_t* tmp)
{
    constexpr int NW = NT / 64;
    const uint32_t w = threadIdx.x / 64, l = threadIdx.x & 63;
    const uint32_t inc = wave_incl_max(v);
    if (l == 63) tmp[w] = inc;
    uint32_t prev = (uint32_t)__shfl_up((int)inc, 1u, 64);
    if (l == 0) prev = 0;
    lds_barrier();
    uint32_t off = 0;
#pragma unroll
    for (int i = 0; i < NW; i++) off = ((uint32_t)i < w && tmp[i] > off) ? tmp[i] : off;
    lds_barrier();
    return max(off, prev);
}

// Maximum over the block.
template <int NT>
__device__ __forceinline__ uint32_t block_max(uint32_t v, uint32_t* tmp)
{
    constexpr int NW = NT / 64;
    const uint32_t inc = wave_incl_max(v);
    if ((threadIdx.x & 63) == 63) tmp[threadIdx.x / 64] = inc;
    lds_barrier();
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < NW; i++) m = tmp[i] > m ? tmp[i] : m;
    lds_barrier();
    return m;
}

// Stable rank of one row per lane among the rows of this wavefront with the
// same digit: rows of earlier rounds (counted in this wave's private LDS
// histogram `hist`) and lower lanes of this round. The lanes sharing a digit
// are found with one ballot per digit bit. Invalid lanes take no part.
__device__ __forceinline__ uint32_t wave_rank(uint32_t d, bool valid, int nbits, uint32_t* hist)
{
    uint64_t peers = ballot(valid);
    for (int b = 0; b < nbits; b++) {
        const bool bit = (d >> b) & 1u;
        const uint64_t m = ballot(bit);
        peers &= bit ? m : ~m;
    }
    const uint32_t below = mbcnt(peers);
    uint32_t base = 0;
    if (valid) base = hist[d];
    if (valid && below == 0) hist[d] = base + (uint32_t)__popcll(peers);
    return base + below;
}

// Per-wave digit counters live in LDS as cnt[w * (BINS + 1) + d]; the padding
// word spreads both a wave's random digits and the column walk below across
// banks. scan_counts turns them, by one block-wide exclusive scan in
// (digit, wave) order, into offsets inside the tile:
//   cnt[w][d] = rows with a smaller digit + rows of digit d in earlier waves.
// Returns the tile's row total. Ends with a barrier.
template <int NT, int NW, int BINS>
__device__ __forceinline__ uint32_t scan_counts(uint32_t* cnt, uint32_t* tmp)
{
    constexpr int STRIDE = BINS + 1;
    constexpr int E = BINS * NW;
    constexpr int EPT = E / NT;
    static_assert(E % NT == 0, "counter matrix must split evenly over the block");
    uint32_t v[EPT];
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < EPT; i++) {
        const int e = threadIdx.x * EPT + i;
        v[i] = cnt[(e % NW) * STRIDE + e / NW];
        s += v[i];
    }
    uint32_t tot;
    uint32_t ex = block_excl_scan<NT>(s, tmp, &tot);
#pragma unroll
    for (int i = 0; i < EPT; i++) {
        const int e = threadIdx.x * EPT + i;
        cnt[(e % NW) * STRIDE + e / NW] = ex;
        ex += v[i];
    }
    lds_barrier();
    return tot;
}

// ---------------------------------------------------------------------------
// small utility kernels
// ---------------------------------------------------------------------------
__global__ void k_fill_u64(uint64_t* p, uint64_t n, uint64_t v)
{
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

hipError_t launch_fill_u64(uint64_t* p, uint64_t n, uint64_t v, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    uint64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_u64, dim3((uint32_t)blocks), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

__global__ void k_wave_scan_test(const uint32_t* in, uint32_t* out, uint64_t n)
{
    const uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    const uint32_t v = i < n ? in[i] : 0u;
    const uint32_t s = wave_incl_scan(v);
    if (i < n) out[i] = s;
}

hipError_t launch_wave_scan_test(const uint32_t* in, uint32_t* out, uint64_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_wave_scan_test, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, st, in, out, n);
    return hipGetLastError();
}

// Copies the planner's tables from pinned host memory into the workspace (16
// bytes a lane) and sets the regions a launch needs cleared: one launch in
// place of a copy per table and a fill per region, each of which costs about
// as much as the launch (10 us between two small launches).
__device__ __forceinline__ void stage_slice(const StageArgs& a, uint64_t i0, uint64_t step)
{
    for (uint64_t i = i0; i < a.n16; i += step) ((uint4*)a.dst)[i] = ((const uint4*)a.src)[i];
#pragma unroll
    for (int f = 0; f < STAGE_FILLS; f++)
        for (uint64_t i = i0; i < a.fill_n[f]; i += step) a.fill_p[f][i] = a.fill_v[f];
}

__global__ __launch_bounds__(256) void k_stage(StageArgs a)
{
    stage_slice(a, blockIdx.x * 256ull + threadIdx.x, (uint64_t)gridDim.x * 256);
}

hipError_t launch_stage(const StageArgs& a, hipStream_t st)
{
    uint64_t n = a.n16;
    for (int f = 0; f < STAGE_FILLS; f++) n = a.fill_n[f] > n ? a.fill_n[f] : n;
    if (n == 0) return hipSuccess;
    uint64_t blocks = (n + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(k_stage, dim3((uint32_t)blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

// dst[i] = src[i] (a few words; dst is pinned host memory)
__global__ void k_publish(uint64_t* __restrict__ dst, const uint64_t* __restrict__ src, uint32_t n)
{
    if (threadIdx.x < n) dst[threadIdx.x] = src[threadIdx.x];
}

hipError_t launch_publish(uint64_t* dst, const uint64_t* src, uint32_t n, hipStream_t st)
{
    if (n > 64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, st, dst, src, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// range probe: minimum and maximum ordinal over one or two key columns
// ---------------------------------------------------------------------------
// step_a, step_b > 1: the minimum and maximum of every step-th element of the
// column only (a sample), and of its last. vary: minmax[2] receives the bits in
// which any of them differs from a's first.
template <typename K>
__global__ __launch_bounds__(256) void k_probe(const K* __restrict__ a, uint64_t na,
                                               const K* __restrict__ b, uint64_t nb,
                                               uint64_t* __restrict__ minmax, uint64_t step_a, uint64_t step_b,
                                               bool vary)
{
    __shared__ uint64_t smin[4], smax[4], svary[4];
    uint64_t mn = ~0ull, mx = 0, vr = 0;
    const uint64_t first = vary && na ? ord_of(a[0]) : 0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t t0 = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    // U loads in flight per thread; a clamped index re-reads a real element,
    // which leaves the minimum and maximum unchanged.
    constexpr int U = 8;
    const uint64_t sa = (na + step_a - 1) / step_a, sb = (nb + step_b - 1) / step_b;  // sampled elements
    for (uint64_t i0 = t0; i0 < sa; i0 += stride * U) {
        K v[U];
#pragma unroll
        for (int u = 0; u < U; u++) v[u] = ld_clamp(a, (i0 + u * stride) * step_a, na);
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint64_t o = ord_of(v[u]);
            mn = o < mn ? o : mn;
            mx = o > mx ? o : mx;
            vr |= o ^ first;
        }
    }
    for (uint64_t i0 = t0; i0 < sb; i0 += stride * U) {
        K v[U];
#pragma unroll
        for (int u = 0; u < U; u++) v[u] = ld_clamp(b, (i0 + u * stride) * step_b, nb);
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint64_t o = ord_of(v[u]);
            mn = o < mn ? o : mn;
            mx = o > mx ? o : mx;
            vr |= o ^ first;
        }
    }
    mn = wave_min64(mn);
    mx = wave_max64(mx);
    vr = wave_or64(vr);
    if ((threadIdx.x & 63) == 0) {
        smin[threadIdx.x / 64] = mn;
        smax[threadIdx.x / 64] = mx;
        svary[threadIdx.x / 64] = vr;
    }
    lds_barrier();
    if (threadIdx.x == 0) {
        for (int i = 0; i < 4; i++) {
            mn = smin[i] < mn ? smin[i] : mn;
            mx = smax[i] > mx ? smax[i] : mx;
            vr |= svary[i];
        }
        // (atomics of all blocks on a word take their turns, 10 ns each; few blocks
        // beat what they read there, which only gets nearer to the result. 54.6M
        // int64 keys: 157 us; 308 when every block made them, 218 without the third word)
        auto now = [&](int i) { return __hip_atomic_load(&minmax[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        if (mn < now(0)) atomicMin((unsigned long long*)&minmax[0], (unsigned long long)mn);
        if (mx > now(1)) atomicMax((unsigned long long*)&minmax[1], (unsigned long long)mx);
        if (vary && (vr & ~now(2))) atomicOr((unsigned long long*)&minmax[2], (unsigned long long)vr);
    }
}

hipError_t launch_probe_step(int key_bytes, const void* a, uint64_t na, const void* b, uint64_t nb,
                             uint64_t step_a, uint64_t step_b, uint64_t* minmax, bool vary, hipStream_t st)
{
    hipError_t e = launch_fill_u64(minmax, 1, ~0ull, st);
    if (e != hipSuccess) return e;
    e = launch_fill_u64(minmax + 1, vary ? 2 : 1, 0ull, st);
    if (e != hipSuccess) return e;
    if (step_a < 1) step_a = 1;
    if (step_b < 1) step_b = 1;
    const uint64_t ma = (na + step_a - 1) / step_a, mb = (nb + step_b - 1) / step_b, n = ma > mb ? ma : mb;
    uint64_t blocks = (n + 256 * 16 - 1) / (256 * 16);
    if (blocks < 1) blocks = 1;
    if (blocks > 8192) blocks = 8192;
    if (key_bytes == 4)
        hipLaunchKernelGGL(k_probe<int32_t>, dim3((uint32_t)blocks), dim3(256), 0, st,
                           (const int32_t*)a, na, (const int32_t*)b, nb, minmax, step_a, step_b, vary);
    else
        hipLaunchKernelGGL(k_probe<int64_t>, dim3((uint32_t)blocks), dim3(256), 0, st,
                           (const int64_t*)a, na, (const int64_t*)b, nb, minmax, step_a, step_b, vary);
    return hipGetLastError();
}

hipError_t launch_probe(int key_bytes, const void* a, uint64_t na, const void* b, uint64_t nb,
                        uint64_t* minmax, hipStream_t st)
{
    return launch_probe_step(key_bytes, a, na, b, nb, 1, 1, minmax, false, st);
}

// The probe of a call whose first pass plans its digit on the device: each
// block leaves its minimum and maximum in parts[2 * block], which the histogram
// reduces (k_hist, ROOT), and stages its slice of the pass's tables.
template <typename K>
__global__ __launch_bounds__(256) void k_probe_root(const K* __restrict__ a, uint64_t na,
                                                    const K* __restrict__ b, uint64_t nb,
                                                    uint64_t* __restrict__ parts, StageArgs sa)
{
    __shared__ uint64_t tmp[4];
    const uint64_t stride = (uint64_t)gridDim.x * 256, t0 = blockIdx.x * 256ull + threadIdx.x;
    uint64_t mn = ~0ull, mx = 0;
    constexpr int U = 8;
    auto column = [&](const K* __restrict__ p, uint64_t n) {
        for (uint64_t i0 = t0; i0 < n; i0 += stride * U) {
            K v[U];
#pragma unroll
            for (int u = 0; u < U; u++) v[u] = ld_clamp(p, i0 + u * stride, n);
#pragma unroll
            for (int u = 0; u < U; u++) {
                const uint64_t o = ord_of(v[u]);
                mn = o < mn ? o : mn;
                mx = o > mx ? o : mx;
            }
        }
    };
    stage_slice(sa, t0, stride);
    column(a, na);
    column(b, nb);
    block_minmax64<256>(mn, mx, tmp);
    if (threadIdx.x == 0) {
        parts[2 * blockIdx.x] = mn;
        parts[2 * blockIdx.x + 1] = mx;
    }
}

uint32_t probe_root_blocks(uint64_t na, uint64_t nb)
{
    const uint64_t n = na > nb ? na : nb, blocks = (n + 256 * 8 - 1) / (256 * 8);
    return (uint32_t)(blocks < 1 ? 1 : blocks > PROBE_PARTS ? PROBE_PARTS : blocks);
}

hipError_t launch_probe_root(int key_bytes, const void* a, uint64_t na, const void* b, uint64_t nb, uint64_t* parts,
                             const StageArgs& sa, hipStream_t st)
{
    const dim3 grid(probe_root_blocks(na, nb)), block(256);
    if (key_bytes == 4)
        hipLaunchKernelGGL(k_probe_root<int32_t>, grid, block, 0, st, (const int32_t*)a, na, (const int32_t*)b, nb,
                           parts, sa);
    else
        hipLaunchKernelGGL(k_probe_root<int64_t>, grid, block, 0, st, (const int64_t*)a, na, (const int64_t*)b, nb,
                           parts, sa);
    return hipGetLastError();
}

// Every step-th key of a column, as its ordinal: out[i] = ord(a[i * step]) for
// i < ceil(n / step).
template <typename K>
__global__ __launch_bounds__(256) void k_gather_step(const K* __restrict__ a, uint64_t n, uint64_t step,
                                                     uint64_t* __restrict__ out)
{
    const uint64_t m = (n + step - 1) / step;
    for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < m; i += (uint64_t)gridDim.x * 256) out[i] = ord_of(a[i * step]);
}

hipError_t launch_gather_step(int key_bytes, const void* a, uint64_t n, uint64_t step, uint64_t* out, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    if (step < 1) step = 1;
    const uint64_t m = (n + step - 1) / step;
    uint64_t blocks = (m + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    if (key_bytes == 4)
        hipLaunchKernelGGL(k_gather_step<int32_t>, dim3((uint32_t)blocks), dim3(256), 0, st, (const int32_t*)a, n,
                           step, out);
    else
        hipLaunchKernelGGL(k_gather_step<int64_t>, dim3((uint32_t)blocks), dim3(256), 0, st, (const int64_t*)a, n,
                           step, out);
    return hipGetLastError();
}

// Ordinals of single keys anywhere in the buffers: out[i] = ord of the key at
// refs[i] (4 or 8 bytes). Used to sample a few rows of crowded buckets.
__global__ __launch_bounds__(256) void k_read_ords(const KeyRef* __restrict__ refs, uint32_t n,
                                                   uint64_t* __restrict__ out)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= n) return;
    const KeyRef r = refs[i];
    out[i] = r.kb == 8 ? ord_of(*(const int64_t*)r.p) : ord_of(*(const int32_t*)r.p);
}

hipError_t launch_read_ords(const KeyRef* refs, uint32_t n, uint64_t* out, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_read_ords, dim3((n + 255) / 256), dim3(256), 0, st, refs, n, out);
    return hipGetLastError();
}

// Digit of ordinal o in a group: its radix digit, or in a pivot group
// (GROUP_PIVOT) its side of the pivot key `base`: 0 below, 1 equal, 2 above.
// With a multiplier (GroupDesc::mul) the digits cut the key range into any
// number of equal parts instead of a power of two.
__device__ __forceinline__ uint32_t group_digit(uint64_t o, uint64_t base, uint32_t shift, uint32_t mask,
                                                bool pivot, uint32_t mul = 0)
{
    if (pivot) return (uint32_t)(o >= base) + (uint32_t)(o > base);
    const uint64_t t = (o - base) >> shift;
    return (mul ? __umulhi((uint32_t)t, mul) : (uint32_t)t) & mask;
}

// ---------------------------------------------------------------------------
// radix histogram: per chunk, the digit counts of its rows (and, per group
// and digit, the smallest and largest ordinal, so that every child bucket
// knows its exact key range and single-key buckets are recognised)
// ---------------------------------------------------------------------------
// LEARNED: the digit is the learned bucket of the row's key (model copied to
// LDS), and every row's bucket is stored in bkt for the scatter. The learned
// variant runs 1024-thread blocks: its 34 KiB of LDS per block would cap
// 256-thread blocks at half the waves a CU can hold.
// ROOT: the pass's one segment takes its digit here, from the probe's partial
// extremes (every block reduces them and plans the same digit); the first
// block of each group writes it to the group for the kernels that follow, and
// block 0 the extremes to root.hdr (pinned) for the host. The host then plans
// no launch before the probe is done: a call of 10^5 rows saves the wait.
// Inputs of one key need no pass: nothing is counted (the scan adds up stale
// counts, which nobody reads) and range_miss stops the scatter. (Counting a join
// of 10^4 x 10^4 rows of one key: 56 us with the wait, 64 with the whole pass, 39 so.)
template <typename K, bool LEARNED, int NT = PART_THREADS, bool ROOT = false>
__global__ __launch_bounds__(NT) void k_hist(const ChunkDesc* __restrict__ chunks,
                                                       GroupDesc* __restrict__ groups,
                                                       BufSet bufs, uint32_t* __restrict__ hist,
                                                       uint64_t* __restrict__ gmin,
                                                       uint64_t* __restrict__ gmax,
                                                       const tj_rmi_t* __restrict__ model, BktSet bkt,
                                                       uint32_t* __restrict__ range_miss, RootArgs root)
{
    __shared__ uint32_t cnt[NB];
    __shared__ uint64_t mn[NB], mx[NB];
    __shared__ __align__(16) char lm_raw[LEARNED ? sizeof(tj_rmi_t) : 16];
    const tj_rmi_t& lm = *(const tj_rmi_t*)lm_raw;
    const ChunkDesc ch = chunks[blockIdx.x];
    GroupDesc g = groups[ch.group];
    if constexpr (ROOT) {
        __shared__ uint64_t rtmp[NT / 64];
        static_assert((uint32_t)NT >= PROBE_PARTS, "one partial a thread");
        uint64_t lo = ~0ull, hi = 0;
        if (threadIdx.x < root.nparts) {
            lo = root.parts[2 * threadIdx.x];
            hi = root.parts[2 * threadIdx.x + 1];
        }
        block_minmax64<NT>(lo, hi, rtmp);
        plan_digit(hi - lo, root.rows, FULL_DIGIT, g.shift, g.bits);
        g.base = lo;
        if (threadIdx.x == 0 && blockIdx.x == g.chunk0) {  // (no block of this launch uses what another one writes here)
            GroupDesc* w = groups + ch.group;
            w->base = lo;
            w->shift = g.shift;
            w->bits = g.bits;
            w->flags = root.flags | (root.narrow && g.shift > 32 ? GROUP_WIDE : 0u);
            if (blockIdx.x == 0) {
                root.hdr[0] = lo;
                root.hdr[1] = hi;
                if (lo == hi) *range_miss = 1u;  // stops the scatter
            }
        }
        if (lo == hi) return;
    }
    const K* __restrict__ src = (const K*)bufs.key[g.src][g.side] + g.src_koff + ch.start;
    uint16_t* __restrict__ bk = LEARNED ? bkt.b[g.side] + ch.start : nullptr;
    const uint32_t nbins = 1u << g.bits;
    for (uint32_t d = threadIdx.x; d < nbins; d += NT) {
        cnt[d] = 0;
        mn[d] = ~0ull;
        mx[d] = 0;
    }
    if (LEARNED) rmi_to_lds<NT>((tj_rmi_t*)lm_raw, model);
    lds_barrier();
    // GROUP_CHECK_RANGE: the digit range came from a sample; a row below base, or
    // whose digit is not below ndig (by shift, and multiplier if there is one),
    // would take a wrong digit, so it is flagged (the planner then takes the exact
    // range and repeats the pass).
    const bool check = !LEARNED && (g.flags & GROUP_CHECK_RANGE) != 0;
    const bool pivot = (g.flags & GROUP_PIVOT) != 0;
    bool miss = false;
    // Rows are counted with LDS atomics. When every valid row of a wave's round
    // falls in one bin (skewed inputs: buckets dominated by one key), the wave
    // reduces them first and one lane updates the bin.
    constexpr int U = 4;
    const uint32_t lane = threadIdx.x & 63;
    for (uint32_t b0 = 0; b0 < ch.len; b0 += NT * U) {  // trip count uniform over the block
        const uint32_t q0 = b0 + threadIdx.x;
        K k[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t q = q0 + u * NT;
            k[u] = ld_clamp(src, q, ch.len);  // rows past the chunk are masked below
        }
        // learned buckets of the round's rows first: independent chains of LDS
        // reads that the compiler interleaves
        uint32_t lb[LEARNED ? U : 1];
        if (LEARNED) {
#pragma unroll
            for (int u = 0; u < U; u++) lb[LEARNED ? u : 0] = min(rmi_bucket(lm, ord_of(k[u])), nbins - 1u);
#pragma unroll
            for (int u = 0; u < U; u++) {
                const uint32_t q = q0 + u * NT;
                if (q < ch.len) bk[q] = (uint16_t)lb[LEARNED ? u : 0];
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t q = q0 + u * NT;
            const uint64_t o = ord_of(k[u]);
            const bool valid = q < ch.len && o >= g.flo && o <= g.fhi;
            uint32_t d;
            if (LEARNED) d = valid ? lb[LEARNED ? u : 0] : 0u;
            else d = valid ? group_digit(o, g.base, g.shift, nbins - 1u, pivot, g.mul) : 0u;
            if (check) {
                const uint64_t t = (o - g.base) >> g.shift;
                miss = miss || (valid && (o < g.base || t > 0xffffffffull ||
                                          (g.mul ? __umulhi((uint32_t)t, g.mul) : (uint32_t)t) >= g.ndig));
            }
            const uint64_t vm = ballot(valid);
            if (vm == 0) continue;
            const int first = __ffsll((unsigned long long)vm) - 1;
            const uint32_t d0 = (uint32_t)__shfl((int)d, first, 64);
            if (ballot(valid && d != d0) == 0) {
                const uint64_t lo = wave_min64(valid ? o : ~0ull);
                const uint64_t hi = wave_max64(valid ? o : 0ull);
                if ((int)lane == first) {
                    atomicAdd(&cnt[d0], (uint32_t)__popcll(vm));
                    atomicMin((unsigned long long*)&mn[d0], (unsigned long long)lo);
                    atomicMax((unsigned long long*)&mx[d0], (unsigned long long)hi);
                }
            } else if (valid) {
                atomicAdd(&cnt[d], 1u);
                // The minimum only falls and the maximum only rises, so a row
                // that does not beat a value read (atomically) at any moment
                // cannot change them; most rows skip the 64-bit atomics.
                if (o < __hip_atomic_load(&mn[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
                    atomicMin((unsigned long long*)&mn[d], (unsigned long long)o);
                if (o > __hip_atomic_load(&mx[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
                    atomicMax((unsigned long long*)&mx[d], (unsigned long long)o);
            }
        }
    }
    if (check && ballot(miss) && (threadIdx.x & 63) == 0) atomicOr(range_miss, 1u);
    lds_barrier();
    for (uint32_t d = threadIdx.x; d < nbins; d += NT) {
        hist[(uint64_t)blockIdx.x * NB + d] = cnt[d];
        if (cnt[d]) {
            atomicMin((unsigned long long*)&gmin[g.child0 + d], (unsigned long long)mn[d]);
            atomicMax((unsigned long long*)&gmax[g.child0 + d], (unsigned long long)mx[d]);
        }
    }
}

hipError_t launch_hist(int key_bytes, const ChunkDesc* chunks, uint32_t nchunks,
                       GroupDesc* groups, BufSet bufs, uint32_t* hist, uint64_t* gmin,
                       uint64_t* gmax, uint32_t* range_miss, const RootArgs* root, hipStream_t st)
{
    if (nchunks == 0) return hipSuccess;
    const BktSet none{};
    if (root) {
        if (key_bytes == 4)
            hipLaunchKernelGGL((k_hist<int32_t, false, PART_THREADS, true>), dim3(nchunks), dim3(PART_THREADS), 0, st,
                               chunks, groups, bufs, hist, gmin, gmax, nullptr, none, range_miss, *root);
        else
            hipLaunchKernelGGL((k_hist<int64_t, false, PART_THREADS, true>), dim3(nchunks), dim3(PART_THREADS), 0, st,
                               chunks, groups, bufs, hist, gmin, gmax, nullptr, none, range_miss, *root);
        return hipGetLastError();
    }
    if (key_bytes == 4)
        hipLaunchKernelGGL((k_hist<int32_t, false>), dim3(nchunks), dim3(PART_THREADS), 0, st, chunks, groups,
                           bufs, hist, gmin, gmax, nullptr, none, range_miss, RootArgs{});
    else
        hipLaunchKernelGGL((k_hist<int64_t, false>), dim3(nchunks), dim3(PART_THREADS), 0, st, chunks, groups,
                           bufs, hist, gmin, gmax, nullptr, none, range_miss, RootArgs{});
    return hipGetLastError();
}

constexpr int LEARNED_HIST_THREADS = 1024;

hipError_t launch_learned_hist(int key_bytes, const ChunkDesc* chunks, uint32_t nchunks,
                               GroupDesc* groups, BufSet bufs, const tj_rmi_t* model, BktSet bkt,
                               uint32_t* hist, uint64_t* gmin, uint64_t* gmax, hipStream_t st)
{
    if (nchunks == 0) return hipSuccess;
    if (key_bytes == 4)
        hipLaunchKernelGGL((k_hist<int32_t, true, LEARNED_HIST_THREADS>), dim3(nchunks), dim3(LEARNED_HIST_THREADS), 0, st,
                           chunks, groups,
                           bufs, hist, gmin, gmax, model, bkt, nullptr, RootArgs{});
    else
        hipLaunchKernelGGL((k_hist<int64_t, true, LEARNED_HIST_THREADS>), dim3(nchunks), dim3(LEARNED_HIST_THREADS), 0, st,
                           chunks, groups,
                           bufs, hist, gmin, gmax, model, bkt, nullptr, RootArgs{});
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// offset scan, two levels. Level 1 (one block per scan block of <= CBLOCK
// chunks): hist[c][d] becomes the exclusive prefix of digit d over the scan
// block's earlier chunks; cbsum[b][d] the scan block's total. Level 2 (one
// block per group): cbsum[b][d] becomes the prefix over the group's earlier
// scan blocks, ccount[d] the group's digit totals and cstart[d] the first
// destination row of digit d (digit-major, so buckets are in key order).
// A row of chunk c with digit d and rank r inside the chunk goes to
// cstart[d] + cbsum[b][d] + hist[c][d] + r.
// ---------------------------------------------------------------------------
// A digit a thread, and all loads of a step before its stores: both levels are
// chains of memory latencies (level 2 of a 2^29-row pass, 64 scan blocks: 30 us
// with two digits a thread, each block's total loaded after the last one's prefix
// was stored, 11 so; one pass of 100k rows, scan blocks scanned here: 9 -> 6 us).
constexpr int SCAN_THREADS = NB;

// Exclusive prefix of digit d over `n` chunks from hist row `c0`, in place; returns the total.
__device__ __forceinline__ uint32_t scan_chunks(uint32_t* __restrict__ hist, uint64_t c0, uint32_t n, uint32_t d)
{
    uint32_t run = 0;
    uint32_t v[CBLOCK];
#pragma unroll
    for (int c = 0; c < CBLOCK; c++) v[c] = (uint32_t)c < n ? hist[(c0 + c) * NB + d] : 0u;
#pragma unroll
    for (int c = 0; c < CBLOCK; c++) {
        if ((uint32_t)c < n) hist[(c0 + c) * NB + d] = run;
        run += v[c];
    }
    return run;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_l1(const CBlockDesc* __restrict__ cblocks,
                                                          uint32_t* __restrict__ hist,
                                                          uint32_t* __restrict__ cbsum)
{
    const CBlockDesc cb = cblocks[blockIdx.x];
    cbsum[(uint64_t)blockIdx.x * NB + threadIdx.x] = scan_chunks(hist, cb.chunk0, cb.nchunks, threadIdx.x);
}

// One block per segment: level 2 of the scan for each of its sides, and its
// children folded into one record each (rows per side, key range), written to
// the device table `out` and, when the host plans them, to pinned host memory
// `hout` as well. It runs before the scatter, so that the host reads the
// records and prepares what follows while the scatter runs. direct: every
// group has one scan block, whose chunks are scanned here instead of by
// k_scan_l1.
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_l2(const GroupDesc* __restrict__ groups, int nside, int direct,
                                                          uint32_t* __restrict__ hist,
                                                          uint32_t* __restrict__ cbsum,
                                                          uint32_t* __restrict__ ccount,
                                                          uint64_t* __restrict__ cstart,
                                                          const uint64_t* __restrict__ gmin,
                                                          const uint64_t* __restrict__ gmax,
                                                          ChildRec* __restrict__ out, ChildRec* __restrict__ hout,
                                                          const uint32_t* __restrict__ miss,
                                                          uint64_t* __restrict__ hmiss)
{
    __shared__ uint32_t tmp[SCAN_THREADS / 64];
    const uint32_t d = threadIdx.x;
    ChildRec rec{0, 0, ~0ull, 0};
    GroupDesc g[2];
    uint32_t tot[2];
    uint64_t lo[2], hi[2];
    g[0] = groups[blockIdx.x * nside];
    g[1] = groups[blockIdx.x * nside + nside - 1];
    const uint32_t nbins = 1u << g[0].bits, dc = min(d, nbins - 1);
    const uint64_t at0 = g[0].child0 / nside;
    // both sides' memory first, then their scans
#pragma unroll
    for (int side = 0; side < 2; side++) {
        if (side >= nside) break;
        lo[side] = ld_now(gmin + g[side].child0, dc);
        hi[side] = ld_now(gmax + g[side].child0, dc);
        uint32_t run = 0;
        if (direct) {
            run = scan_chunks(hist, g[side].chunk0, g[side].nchunks, d);
            if (g[side].nchunks) cbsum[(uint64_t)g[side].cblock0 * NB + d] = 0;
        } else {
            uint32_t* const cs = cbsum + (uint64_t)g[side].cblock0 * NB;
            const uint32_t n = g[side].ncblocks;
            for (uint32_t b0 = 0; b0 < n; b0 += 16) {  // (16 loads in flight: a store stops the next load)
                uint32_t v[16];
#pragma unroll
                for (int b = 0; b < 16; b++) v[b] = b0 + b < n ? cs[(uint64_t)(b0 + b) * NB + d] : 0u;
#pragma unroll
                for (int b = 0; b < 16; b++) {
                    if (b0 + b < n) cs[(uint64_t)(b0 + b) * NB + d] = run;
                    run += v[b];
                }
            }
        }
        tot[side] = d < nbins ? run : 0u;
    }
#pragma unroll
    for (int side = 0; side < 2; side++) {
        if (side >= nside) break;
        uint32_t all;
        const uint64_t ex = block_excl_scan<SCAN_THREADS>(tot[side], tmp, &all);
        if (d < nbins) {
            ccount[g[side].child0 + d] = tot[side];
            cstart[g[side].child0 + d] = g[side].dst_start + ex;
            if (side == 0) rec.rn = tot[side];
            else rec.sn = tot[side];
            rec.lo = lo[side] < rec.lo ? lo[side] : rec.lo;
            rec.hi = hi[side] > rec.hi ? hi[side] : rec.hi;
        }
    }
    if (d < nbins) {
        out[at0 + d] = rec;
        if (hout) hout[at0 + d] = rec;
    }
    if (hmiss && blockIdx.x == 0 && threadIdx.x == 0) *hmiss = *miss;
}

// ---------------------------------------------------------------------------
// Leaf batching of a level on the device, for levels of many segments whose
// children mostly fit one LDS block: the host then reads back four summary
// words and the few children too large for a leaf instead of one record per
// child. One wave per segment. Adjacent children are batched
// greedily into leaves of at most LEAF_CAP rows (a child whose keys were
// narrowed into another 2^32 window starts a new leaf), as the host planner
// does. A child over LEAF_CAP closes the open leaf and is listed for the host
// (BigChild records at the top of the leaf table, counted in summary[4]): the
// host plans only those. The greedy choice is the only sequential part: a
// uniform loop over the children's row counts marks where leaves start (a
// 512-bit mask in scalar registers). Everything else is per child, across the
// lanes: exclusive prefix sums of the rows give each leaf its first rows and
// sizes, the last non-empty child before the leaf's end gives its largest key,
// and a prefix count of children with rows on both sides tells whether a join
// leaf can produce pairs. Pass 0 counts the useful leaves and the listed
// children of each segment; pass 1 writes them after those of the earlier
// segments of the batch (leaves upwards from leaf_base, listed children
// downwards from the top of the table; a slot below leaf_base sets
// BATCH_OVERFLOW, and so does a collision, which the host detects from the
// totals).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_batch_leaves(const GroupDesc* __restrict__ groups,
                                                     const ChildRec* __restrict__ crec, BatchArgs a,
                                                     uint32_t* __restrict__ seg_count,
                                                     LeafDesc* __restrict__ leaves,
                                                     unsigned long long* __restrict__ summary, int pass)
{
    constexpr int RPL = NB / 64;  // children per lane: child d = j*64 + lane
    __shared__ uint32_t s_rpre[NB + 1], s_spre[NB + 1], s_both[NB + 1];  // exclusive prefixes
    __shared__ uint32_t s_last[NB];  // last non-empty child at or before d
    __shared__ uint64_t s_hi[NB];
    const uint32_t sgi = blockIdx.x, l = threadIdx.x;
    const GroupDesc g0 = groups[sgi * a.nside];
    const uint64_t s_start = a.nside == 2 ? groups[sgi * 2 + 1].dst_start : 0;
    const uint64_t koff_s = a.nside == 2 ? groups[sgi * 2 + 1].dst_koff : 0;
    const uint32_t nb = 1u << g0.bits;
    const ChildRec* cr = crec + g0.child0 / a.nside;
    uint32_t rows[RPL], win[RPL];
    uint64_t lo[RPL];
    uint64_t bigm[RPL];  // children over LEAF_CAP, one bit each
    uint32_t rc = 0, sc = 0, bc = 0, lastc = 0;  // carries of the prefixes across slots
#pragma unroll
    for (int j = 0; j < RPL; j++) {
        const uint32_t d = j * 64 + l;
        const ChildRec c = d < nb ? cr[d] : ChildRec{0, 0, ~0ull, 0};
        rows[j] = c.rn + c.sn;
        bigm[j] = ballot(rows[j] > (uint32_t)LEAF_CAP);
        uint64_t clo = c.lo, chi = c.hi;
        win[j] = 0;
        if (a.narrowing && rows[j]) {
            if (g0.flags & GROUP_DIGIT_WINDOWS) {  // each child has its own window, from its first key
                const uint64_t w0 = g0.base + digit_start(d, g0.shift, g0.mul);
                win[j] = d;
                clo -= w0;
                chi -= w0;
            } else {
                const uint64_t off = clo - g0.base;
                win[j] = (uint32_t)(off >> 32);
                clo = off & 0xffffffffull;
                chi = (chi - g0.base) & 0xffffffffull;
            }
        }
        lo[j] = clo;
        const uint32_t both = c.rn > 0 && c.sn > 0 ? 1u : 0u;
        const uint32_t ri = wave_incl_scan(c.rn), si = wave_incl_scan(c.sn), bi = wave_incl_scan(both);
        const uint32_t li = wave_incl_max(rows[j] ? d + 1 : 0u);  // 1 + last non-empty child so far
        if (d < nb) {
            s_rpre[d] = rc + ri - c.rn;
            s_spre[d] = sc + si - c.sn;
            s_both[d] = bc + bi - both;
            const uint32_t lst = li > lastc ? li : lastc;
            s_last[d] = lst ? lst - 1 : 0u;
            s_hi[d] = chi;
        }
        rc += (uint32_t)__shfl((int)ri, 63, 64);
        sc += (uint32_t)__shfl((int)si, 63, 64);
        bc += (uint32_t)__shfl((int)bi, 63, 64);
        const uint32_t lm = (uint32_t)__shfl((int)li, 63, 64);
        lastc = lm > lastc ? lm : lastc;
    }
    if (l == 0) {
        s_rpre[nb] = rc;
        s_spre[nb] = sc;
        s_both[nb] = bc;
    }
    // greedy batching: bit d of start[] marks a child that opens a leaf
    uint64_t start[RPL];
    {
        bool open = false;
        uint32_t acc = 0, lwin = 0;
#pragma unroll
        for (int j = 0; j < RPL; j++) {
            uint64_t m = 0;
            const uint64_t ne = ballot(rows[j] > 0);
            uint64_t todo = ne;
            while (todo) {
                const uint32_t ln = (uint32_t)__builtin_ctzll(todo);
                todo &= todo - 1;
                const uint32_t r = (uint32_t)__builtin_amdgcn_readlane((int)rows[j], (int)ln);
                if (r > (uint32_t)LEAF_CAP) {  // listed for the host; the next child opens a leaf
                    open = false;
                    continue;
                }
                const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)win[j], (int)ln);
                if (!open || w != lwin || acc + r > (uint32_t)LEAF_CAP) {
                    m |= 1ull << ln;
                    open = true;
                    lwin = w;
                    acc = 0;
                }
                acc += r;
            }
            start[j] = m;
        }
    }
    lds_barrier();  // the prefix tables are complete
    // per leaf (its starting child): extent, sizes, key range, usefulness
    uint32_t useful[RPL], e_of[RPL];
#pragma unroll
    for (int j = 0; j < RPL; j++) {
        const uint32_t d = j * 64 + l;
        const bool st = (start[j] >> l) & 1ull;
        // the leaf ends at the next start or listed child after d, else at
        // the end of the segment's children
        uint32_t e = nb;
        const uint64_t above = l == 63 ? 0ull : (start[j] | bigm[j]) & (~0ull << (l + 1));
        if (above) {
            e = j * 64 + (uint32_t)__builtin_ctzll(above);
        } else {
#pragma unroll
            for (int k = j + 1; k < RPL; k++)
                if (e == nb && (start[k] | bigm[k])) e = k * 64 + (uint32_t)__builtin_ctzll(start[k] | bigm[k]);
        }
        e_of[j] = e;
        useful[j] = st && (!a.join || s_both[e] - s_both[d] > 0) ? 1u : 0u;
    }
    // emission order: useful leaves, and listed children, in child order
    uint32_t idx[RPL], bidx[RPL], nleaf = 0, nbig = 0;
#pragma unroll
    for (int j = 0; j < RPL; j++) {
        const uint64_t um = ballot(useful[j] != 0);
        idx[j] = nleaf + mbcnt(um);
        nleaf += (uint32_t)__popcll(um);
        bidx[j] = nbig + mbcnt(bigm[j]);
        nbig += (uint32_t)__popcll(bigm[j]);
    }
    if (pass == 0) {
        if (l == 0) seg_count[sgi] = nleaf | (nbig << 16);
        return;
    }
    uint64_t before = 0, before_big = 0;
    for (uint32_t i = l; i < sgi; i += 64) {
        before += seg_count[i] & 0xffffu;
        before_big += seg_count[i] >> 16;
    }
    before = wave_sum64(before);
    before_big = wave_sum64(before_big);
    uint64_t rows_all = 0;
    bool wide = false, over = false;
#pragma unroll
    for (int j = 0; j < RPL; j++) {
        if (!((bigm[j] >> l) & 1ull)) continue;
        const uint32_t d = j * 64 + l;
        const uint64_t k = before_big + bidx[j];
        if (a.leaf_base + k + 1 > a.leaf_cap) {
            over = true;
            continue;
        }
        const ChildRec c = cr[d];
        BigChild b;
        b.seg = sgi;
        b.child = d;
        b.r_off = s_rpre[d];
        b.s_off = s_spre[d];
        b.rn = c.rn;
        b.sn = c.sn;
        b.lo = c.lo;
        b.hi = c.hi;
        *(BigChild*)(leaves + (a.leaf_cap - 1 - k)) = b;
    }
#pragma unroll
    for (int j = 0; j < RPL; j++) {
        if (!useful[j]) continue;
        const uint32_t d = j * 64 + l, e = e_of[j];
        const uint32_t rn = s_rpre[e] - s_rpre[d], sn = s_spre[e] - s_spre[d];
        rows_all += (uint64_t)rn + sn;
        const uint64_t slot = a.leaf_base + before + idx[j];
        if (slot >= a.leaf_cap) {
            over = true;
            continue;
        }
        const uint64_t llo = lo[j], lhi = s_hi[s_last[e - 1]];
        const uint64_t span = lhi - llo;
        const uint32_t bits = span ? 64u - (uint32_t)__clzll((long long)span) : 0u;
        wide = wide || bits > 32;
        LeafDesc L;
        L.r0 = g0.dst_start + s_rpre[d];
        L.s0 = s_start + s_spre[d];
        L.kr0 = L.r0 + g0.dst_koff;
        L.ks0 = L.s0 + koff_s;
        L.base = llo;
        L.out = a.join ? 0 : L.r0 + a.out_delta;
        L.rn = rn;
        L.sn = sn;
        L.bits = (uint16_t)bits;
        L.kb = (uint16_t)a.kb;
        L.buf = (uint16_t)a.buf;
        L.flags = (uint16_t)a.flags;
        leaves[slot] = L;
    }
    rows_all = wave_sum64(rows_all);
    const uint64_t fl = (ballot(wide) ? BATCH_WIDE : 0ull) | (ballot(over) ? BATCH_OVERFLOW : 0ull);
    if (l != 0) return;
    atomicAdd(&summary[0], (unsigned long long)nleaf);
    atomicAdd(&summary[1], (unsigned long long)rows_all);
    if (fl) atomicOr(&summary[2], (unsigned long long)fl);
    if (nbig) atomicAdd(&summary[4], (unsigned long long)nbig);
}

hipError_t launch_batch_leaves(const GroupDesc* groups, const ChildRec* crec, const BatchArgs& a,
                               uint32_t* seg_count, LeafDesc* leaves, uint64_t* summary, int pass,
                               hipStream_t st)
{
    if (a.nseg == 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_leaves, dim3(a.nseg), dim3(64), 0, st, groups, crec, a, seg_count, leaves,
                       (unsigned long long*)summary, pass);
    return hipGetLastError();
}

hipError_t launch_scan(const CBlockDesc* cblocks, uint32_t ncblocks, const GroupDesc* groups, uint32_t ngroups,
                       int nside, bool direct, uint32_t* hist, uint32_t* cbsum, uint32_t* ccount, uint64_t* cstart,
                       const uint64_t* gmin, const uint64_t* gmax, ChildRec* out, ChildRec* hout,
                       const uint32_t* miss, uint64_t* hmiss, hipStream_t st)
{
    if (ncblocks == 0 || ngroups == 0) return hipSuccess;
    if (!direct) {
        hipLaunchKernelGGL(k_scan_l1, dim3(ncblocks), dim3(SCAN_THREADS), 0, st, cblocks, hist, cbsum);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_scan_l2, dim3(ngroups / nside), dim3(SCAN_THREADS), 0, st, groups, nside, direct ? 1 : 0, hist,
                       cbsum, ccount, cstart, gmin, gmax, out, hout, miss, hmiss);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// stable LDS-staged scatter. Each block walks its chunk in tiles of
// SC_TILE rows. Per tile: rows are ranked within their wave by ballot match,
// offset across waves and digits by one block scan, staged in LDS grouped by
// digit, and written out as per-digit runs while the next tile's loads are in
// flight. Wave w of the tile owns rows [w*SC_KI*64, (w+1)*SC_KI*64); round r
// of a wave covers 64 consecutive rows, so (wave, round, lane) is input order
// and the partition is stable.
// KO is the written key type. KO = int32 with K = int64 narrows the keys: a
// row is written as the low 32 bits of (ord - g.base), stored so that ord_of
// of the stored int32 gives them back. Every child of such a pass spans at
// most 2^32 ordinals and lies inside one window g.base + [j*2^32, (j+1)*2^32),
// so inside a child (and among children of one window) the narrowed keys
// order as the originals.
// ---------------------------------------------------------------------------
constexpr int SC_NT = 512, SC_KI = 18, SC_NW = SC_NT / 64, SC_TILE = SC_NT * SC_KI;
constexpr int SC_STRIDE = NB + 1;
static_assert(SC_TILE == PART_TILE, "chunk sizes are planned in scatter tiles");

// DIGIN (learned pass): each row's digit is read from bkt instead of being
// computed from its key; rows are ranked by ballot match, which is stable by
// construction, and the staged digit replaces the staged tile index.
template <typename K, typename KO, bool RIDS, bool WKEYS, bool DIGIN>
__global__ __launch_bounds__(SC_NT) void k_scatter(const ChunkDesc* __restrict__ chunks,
                                                   const GroupDesc* __restrict__ groups,
                                                   const uint32_t* __restrict__ hist,
                                                   const uint32_t* __restrict__ cbsum,
                                                   const uint64_t* __restrict__ cstart,
                                                   BufSet bufs, BktSet bkt, const uint32_t* __restrict__ skip)
{
    // (a row outside the sampled digit range: the call starts again, nothing is to be moved)
    if (skip && *skip) return;
    constexpr int NT = SC_NT, KI = SC_KI, NW = SC_NW, TILE = SC_TILE;
    __shared__ uint32_t cnt[NW * SC_STRIDE];
    __shared__ uint32_t spare[NT];  // one private counter per thread for rows that take no part
    __shared__ uint32_t run[NB], delta[NB];
    __shared__ uint32_t tmp[NW];
    __shared__ uint32_t s_unordered;
    // staging, with one spare slot per lane of a wave for rows that take no part
    __shared__ K skey[TILE + 64];
    __shared__ int32_t srid[RIDS ? TILE + 64 : 1];
    __shared__ uint16_t sidx[TILE + 64];  // the staged row's index inside the tile (DIGIN: its digit)

    const ChunkDesc ch = chunks[blockIdx.x];
    const GroupDesc g = groups[ch.group];
    const K* __restrict__ src_k = (const K*)bufs.key[g.src][g.side] + g.src_koff + ch.start;
    const int32_t* __restrict__ src_r = bufs.rid[g.src][g.side] + ch.start;
    KO* __restrict__ dst_k = (KO*)bufs.key[g.dst][g.side] + g.dst_koff;
    int32_t* __restrict__ dst_r = (int32_t*)bufs.rid[g.dst][g.side];
    const uint16_t* __restrict__ src_b = DIGIN ? bkt.b[g.side] + ch.start : nullptr;
    const uint32_t nbins = 1u << g.bits, mask = nbins - 1u;
    const uint32_t w = threadIdx.x / 64, l = threadIdx.x & 63;
    const bool force_reorder = (g.flags & GROUP_FORCE_REORDER) != 0;

    const bool pivot = (g.flags & GROUP_PIVOT) != 0;
    auto digit_of = [&](K k) { return group_digit(ord_of(k), g.base, g.shift, mask, pivot); };
    // a narrowing launch may hold groups that keep their 8-byte keys (uniform per block)
    const bool wide = sizeof(KO) < sizeof(K) && (g.flags & GROUP_WIDE) != 0;
    K* __restrict__ dst_kw = (K*)bufs.key[g.dst][g.side] + g.dst_koff;
    auto write_row = [&](uint32_t dst, K k, int32_t rid) {
        if (WKEYS) {
            if (sizeof(KO) == sizeof(K)) dst_k[dst] = (KO)k;
            else if (wide) dst_kw[dst] = k;
            else dst_k[dst] = (KO)((uint32_t)(ord_of(k) - g.base) ^ 0x80000000u);
        }
        if (RIDS) dst_r[dst] = rid;
    };

    for (uint32_t d = threadIdx.x; d < NB; d += NT)
        run[d] = d < nbins ? (uint32_t)(cstart[g.child0 + d] + cbsum[(uint64_t)ch.cblock * NB + d] +
                                        hist[(uint64_t)blockIdx.x * NB + d])
                           : 0u;
    K key[KI];
    int32_t rid[KI];
    uint32_t bin[DIGIN ? KI : 1];
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = (w * KI + r) * 64 + l;
        key[r] = q < ch.len ? src_k[q] : K(0);
        if (RIDS) rid[r] = q < ch.len ? src_r[q] : 0;
        if (DIGIN) bin[DIGIN ? r : 0] = ld_clamp(src_b, q, ch.len);  // rows past the chunk are masked
    }
    for (uint32_t t0 = 0; t0 < ch.len; t0 += TILE) {
        uint32_t dig[KI], rk[KI];
        bool val[KI];
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const uint32_t q = t0 + (w * KI + r) * 64 + l;
            const uint64_t o = ord_of(key[r]);
            val[r] = q < ch.len && o >= g.flo && o <= g.fhi;
            if (DIGIN) dig[r] = val[r] ? bin[DIGIN ? r : 0] & mask : 0u;
            else dig[r] = val[r] ? group_digit(o, g.base, g.shift, mask, pivot) : 0u;
        }
        for (uint32_t i = l; i < NB; i += 64) cnt[w * SC_STRIDE + i] = 0;
        // Rank inside the wave: one LDS atomic per row on the wave's own
        // counters. The wave issues its rounds in row order; within a round the
        // hardware applies the lanes that hit one counter in lane order, which
        // makes the ranks stable. Nothing relies on that order: the write-out
        // checks it and the tile is written again, ranked by ballots, if a
        // digit's rows ever come out of input order.
        if (DIGIN) {
#pragma unroll
            for (int r = 0; r < KI; r++) rk[r] = wave_rank(dig[r], val[r], (int)g.bits, &cnt[w * SC_STRIDE]);
        } else {
#pragma unroll
            for (int r = 0; r < KI; r++)
                rk[r] = atomicAdd(val[r] ? &cnt[w * SC_STRIDE + dig[r]] : &spare[threadIdx.x], 1u);
        }
        if (threadIdx.x == 0) s_unordered = 0;
        lds_barrier();
        const uint32_t total = scan_counts<NT, NW, NB>(cnt, tmp);
        for (uint32_t d = threadIdx.x; d < NB; d += NT) {
            const uint32_t tex = cnt[d];
            const uint32_t nxt = d + 1 < NB ? cnt[d + 1] : total;
            delta[d] = run[d] - tex;
            run[d] += nxt - tex;
        }
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const uint32_t p = val[r] ? cnt[w * SC_STRIDE + dig[r]] + rk[r] : TILE + l;
            skey[p] = key[r];
            if (RIDS) srid[p] = rid[r];
            sidx[p] = (uint16_t)(DIGIN ? dig[r] : (w * KI + r) * 64 + l);
        }
        lds_barrier();
        // next tile's loads overlap the write-out of this one
        const uint32_t n0 = t0 + TILE;
        if (n0 < ch.len) {
#pragma unroll
            for (int r = 0; r < KI; r++) {
                const uint32_t q = n0 + (w * KI + r) * 64 + l;
                key[r] = q < ch.len ? src_k[q] : K(0);
                if (RIDS) rid[r] = q < ch.len ? src_r[q] : 0;
                if (DIGIN) bin[DIGIN ? r : 0] = ld_clamp(src_b, q, ch.len);
            }
        }
        bool unordered = false;
        if (total) {
            // the KI rows of each thread are read together (a position past the
            // tile's rows re-reads its last row and writes nothing)
#pragma unroll
            for (int j = 0; j < KI; j++) {
                const uint32_t p = threadIdx.x + j * NT;
                const uint32_t pc = p < total ? p : total - 1;
                const K k = skey[pc];
                const int32_t rv = RIDS ? srid[pc] : 0;
                const uint32_t x = sidx[pc], xp = DIGIN ? 0u : sidx[pc ? pc - 1 : 0];
                const uint32_t d = DIGIN ? x : digit_of(k);
                if (p < total) {
                    write_row(delta[d] + p, k, rv);
                    // cnt[d] (wave 0's entry) is where digit d starts inside the tile
                    if (!DIGIN) unordered = unordered || (p > cnt[d] && xp > x);
                }
            }
        }
        if (unordered) s_unordered = 1;
        lds_barrier();
        if (!DIGIN && (s_unordered || force_reorder)) {
            // Rare path: rank the tile again by ballot match (from its rows in
            // the source) and write it over the same destination rows.
            K k2[KI];
            int32_t r2[KI];
#pragma unroll
            for (int r = 0; r < KI; r++) {
                const uint32_t q = t0 + (w * KI + r) * 64 + l;
                k2[r] = q < ch.len ? src_k[q] : K(0);
                r2[r] = RIDS && q < ch.len ? src_r[q] : 0;
                const uint64_t o = ord_of(k2[r]);
                val[r] = q < ch.len && o >= g.flo && o <= g.fhi;
                dig[r] = val[r] ? group_digit(o, g.base, g.shift, mask, pivot) : 0u;
            }
            for (uint32_t i = l; i < NB; i += 64) cnt[w * SC_STRIDE + i] = 0;
#pragma unroll
            for (int r = 0; r < KI; r++) rk[r] = wave_rank(dig[r], val[r], (int)g.bits, &cnt[w * SC_STRIDE]);
            lds_barrier();
            scan_counts<NT, NW, NB>(cnt, tmp);  // same counts, so delta[] still holds
#pragma unroll
            for (int r = 0; r < KI; r++) {
                if (val[r]) {
                    const uint32_t p = cnt[w * SC_STRIDE + dig[r]] + rk[r];
                    skey[p] = k2[r];
                    if (RIDS) srid[p] = r2[r];
                }
            }
            lds_barrier();
            for (uint32_t p = threadIdx.x; p < total; p += NT) {
                const K k = skey[p];
                write_row(delta[digit_of(k)] + p, k, RIDS ? srid[p] : 0);
            }
            lds_barrier();
        }
    }
}

// ---------------------------------------------------------------------------
// scatter in whole lines, for passes whose chunks are several tiles long and
// whose groups have at most LN_D digits. What bounds a scatter is its writes:
// at 512 digits a 9216-row tile ends 18 rows a digit, and runs that begin and
// end inside 128-byte lines reach 2.7 TB/s (reads and writes together) whatever
// the tile does meanwhile, while the same rows cut at line boundaries (16 keys
// of 8 bytes, 32 of 4, 32 row ids) reach 5.0, at any number of digits. So the
// rows of a digit that do not fill a line stay behind in LDS until the next
// tile: each digit has room for one line of keys and one of row ids (256
// bytes; 320 digits: 80 KiB), and only a chunk's first and last line of a
// digit are written in part. Keys and row ids are staged one after the other
// in the same 64 KiB.
//
// One block fills a CU, so nothing else hides its waits, and a wave's loads and
// stores count in one counter, so that a load which stores follow is waited for
// together with them. So a tile's rows are loaded while the tile before leaves,
// a third of them at a time, and waited for once, at the tile's start. (Loads
// issued where they are next used, with a wait for keys and one for row ids a
// tile: 3.2 TB/s; all at once: 3.4; in thirds: 3.7. Half of the waves loading
// and half writing: 16-row threads spill, 0.8.)
//
// Measured, 2^29 rows of a 64-bit key and a row id, a pass: 4.80 ms in
// k_scatter, 3.50 here (3.7 TB/s of 24 bytes a row); 2^27 + 2^29 join rows, two
// passes (8-byte keys narrowed, then 4-byte ones): 10.3 -> 9.0 ms. What is left
// over the 5.0 TB/s is the tile's LDS work, mostly of the ranking and staging.
//
// Ranks, stability and narrowed keys as in k_scatter, with 16-bit counters (in
// the staging space, which is free then); a row's order is checked on staged
// (digit, index) words, which increase strictly over the whole tile.
// Destination rows are counted from the line boundary at or before the column's
// start: v = row + phase. Line v / G of a digit is written by consecutive
// lanes, from the carried rows (v below the digit's cursor) and the staged ones.
// ---------------------------------------------------------------------------
constexpr int LN_NT = 1024, LN_KI = 8, LN_NW = LN_NT / 64;
constexpr int LN_CS = LN_D + 2;  // 16-bit counters of a wave
static_assert(LN_TILE == LN_NT * LN_KI, "chunk sizes are planned in tiles");
static_assert(LN_D * LN_NW % LN_NT == 0 && LN_D <= LN_NT && LN_D % 2 == 0, "counters split evenly over the block");

// One line of a tile's output, for G = 2^LG rows of one column:
//   x: line number << LG | first slot that is this chunk's;
//   y: digit | (staged position of slot 0 + 32) << 9 | carried slots << 23.
// The thread t of digit t writes its lines' words; `at`, `n`: its first line in
// the tile's list and their number; cur, first: destination rows of its first
// staged row and of the chunk's first row; tex: its first staged position.
template <int LG>
__device__ __forceinline__ void list_lines(uint2* lin, uint32_t at, uint32_t n, uint32_t cur, uint32_t first,
                                           uint32_t tex, uint32_t phase, uint32_t t, uint32_t l)
{
    constexpr uint32_t G = 1u << LG;
    const uint32_t line = (cur + phase) >> LG, c = (cur + phase) & (G - 1);
    const uint32_t skip = (first + phase) >> LG == line ? (first + phase) & (G - 1) : 0u;
    const uint32_t pos = tex + 32u - c;
    auto put = [&](uint32_t i, uint32_t at_, uint32_t line_, uint32_t skip_, uint32_t pos_, uint32_t c_, uint32_t d) {
        lin[at_ + i] = uint2{(line_ + i) << LG | (i ? 0u : skip_), d | (pos_ + (i << LG)) << 9 | (i ? 0u : c_) << 23};
    };
    constexpr uint32_t OWN = 6;
    for (uint32_t i = 0; i < OWN && i < n; i++) put(i, at, line, skip, pos, c, t);
    uint64_t m = ballot(n > OWN);  // a digit of many lines: by its whole wave
    while (m) {
        const int src = __ffsll((unsigned long long)m) - 1;
        m &= m - 1;
        const uint32_t n_ = __shfl(n, src, 64), at_ = __shfl(at, src, 64), line_ = __shfl(line, src, 64),
                       pos_ = __shfl(pos, src, 64), d = __shfl(t, src, 64);
        for (uint32_t i = OWN + l; i < n_; i += 64) put(i, at_, line_, 0, pos_, 0, d);
    }
}

// The listed lines of one column leave. The staged rows and the carried ones
// are both in `lds` (carry: the latter's offset), so that each row is one read.
template <typename T, int LG>
__device__ __forceinline__ void write_lines(T* __restrict__ dst, uint32_t phase, const T* lds, uint32_t carry,
                                            const uint2* lin, uint32_t lines, const uint32_t* s_end, bool last,
                                            bool redo, uint32_t t)
{
    constexpr int U = 2;
    constexpr uint32_t G = 1u << LG;
    const uint32_t n = lines << LG;
    for (uint32_t q0 = t; q0 < n; q0 += LN_NT * U) {
        uint32_t at[U];
        T val[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t q = q0 + u * LN_NT, qc = q < n ? q : n - 1, j = qc & (G - 1);
            const uint2 L = lin[qc >> LG];
            const uint32_t d = L.y & 0x1ffu, row = (L.x & ~(G - 1)) + j - phase;
            const bool staged = j >= L.y >> 23;
            ok[u] = q < n && j >= (L.x & (G - 1)) && (!last || row < s_end[d]) && (staged || !redo);
            val[u] = lds[staged ? min(((L.y >> 9) & 0x3fffu) + j - 32u, (uint32_t)LN_TILE - 1u) : carry + (d << LG) + j];
            at[u] = row;
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (ok[u]) dst[at[u]] = val[u];
    }
}

template <typename K, typename KO, bool RIDS>
__global__ __launch_bounds__(LN_NT) void k_scatter_lines(const ChunkDesc* __restrict__ chunks,
                                                         const GroupDesc* __restrict__ groups,
                                                         const uint32_t* __restrict__ hist,
                                                         const uint32_t* __restrict__ cbsum,
                                                         const uint64_t* __restrict__ cstart, BufSet bufs,
                                                         const uint32_t* __restrict__ skip)
{
    if (skip && *skip) return;
    constexpr int NT = LN_NT, KI = LN_KI, NW = LN_NW, TILE = LN_TILE, D = LN_D, CS = LN_CS;
    constexpr int LGK = sizeof(KO) == 8 ? 4 : 5, LGR = 5;
    constexpr int GK = 1 << LGK, GR = 1 << LGR;
    constexpr bool NARROW = sizeof(KO) < sizeof(K);
    // staged keys, or staged row ids and order words, or the rank counters;
    // then each digit's carried line of keys, and of row ids
    constexpr int STAGE = TILE * (RIDS || sizeof(KO) == 8 ? 8 : 4);
    __shared__ __align__(16) char lds[STAGE + D * 128 + (RIDS ? D * 128 : 0)];
    // lines: a digit's n rows, up to G - 1 carried and, at a chunk's end, up to G - 1 that are not there
    __shared__ uint2 lin[TILE / GK + 2 * D];
    __shared__ uint32_t s_first[D], s_end[D], s_keep[D];
    __shared__ uint32_t s_sub[NARROW ? D : 1];
    __shared__ uint32_t tmp[NW];
    __shared__ uint32_t s_unordered;
    static_assert(STAGE >= NW * CS * 2, "the counters share the staging space");
    uint16_t* const cnt = (uint16_t*)lds;
    KO* const skey = (KO*)lds;
    int32_t* const srid = (int32_t*)lds;
    uint32_t* const stag = (uint32_t*)lds + TILE;
    constexpr uint32_t CK = STAGE / sizeof(KO), CR = (STAGE + D * 128) / 4;  // offsets of the carried rows

    const ChunkDesc ch = chunks[blockIdx.x];
    const GroupDesc g = groups[ch.group];
    const K* __restrict__ src_k = (const K*)bufs.key[g.src][g.side] + g.src_koff + ch.start;
    const int32_t* __restrict__ src_r = RIDS ? bufs.rid[g.src][g.side] + ch.start : nullptr;
    KO* __restrict__ dst_k = (KO*)bufs.key[g.dst][g.side] + g.dst_koff;
    int32_t* __restrict__ dst_r = (int32_t*)bufs.rid[g.dst][g.side];
    const uint32_t phk = (uint32_t)((uintptr_t)dst_k % 128 / sizeof(KO));
    const uint32_t phr = RIDS ? (uint32_t)((uintptr_t)dst_r % 128 / 4) : 0u;
    const uint32_t nbins = min(1u << g.bits, (uint32_t)D);
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
    uint32_t t = threadIdx.x, l = t & 63;
    const bool pivot = (g.flags & GROUP_PIVOT) != 0, force = (g.flags & GROUP_FORCE_REORDER) != 0;

    // thread d keeps digit d's cursor
    uint32_t cur = 0;
    if (t < nbins)
        cur = (uint32_t)(cstart[g.child0 + t] + cbsum[(uint64_t)ch.cblock * NB + t] + hist[(uint64_t)blockIdx.x * NB + t]);
    if (t < nbins) s_first[t] = cur;
    if (NARROW && t < D)
        s_sub[t] = (uint32_t)(g.base + (g.flags & GROUP_DIGIT_WINDOWS ? digit_start(t, g.shift, g.mul) : 0));

    K key[KI];
    int32_t rid[RIDS ? KI : 1], next_rid[RIDS ? KI : 1];
    auto load_keys = [&](uint32_t t0, int r0, int r1) {
#pragma unroll
        for (int r = r0; r < r1; r++) key[r] = at32(src_k, min(t0 + (w * KI + r) * 64 + l, ch.len - 1));
    };
    auto load_rids = [&](int32_t (&to)[RIDS ? KI : 1], uint32_t t0) {
        if constexpr (RIDS) {
#pragma unroll
            for (int r = 0; r < KI; r++) to[r] = at32(src_r, min(t0 + (w * KI + r) * 64 + l, ch.len - 1));
        }
    };
    load_keys(0, 0, KI);
    load_rids(rid, 0);
    for (uint32_t t0 = 0; t0 < ch.len; t0 += TILE) {
        const uint32_t rows = ch.len - t0 < (uint32_t)TILE ? ch.len - t0 : (uint32_t)TILE;
        const bool last = t0 + TILE >= ch.len;
        for (int redo = 0;; redo++) {
            // (addresses derived from t and l are formed anew for every tile:
            // kept across tiles, they would take the registers the rows need)
            asm volatile("" : "+v"(t), "+v"(l));
            uint32_t pd[KI];  // digit << 16 | rank in the wave, then | staged position
            // rank inside the wave (redo: by ballots)
            for (uint32_t i = l; i < CS / 2; i += 64) ((uint32_t*)cnt)[w * (CS / 2) + i] = 0;
            if (redo) lds_barrier();  // (the ballots' counters are read as 16-bit words)
            uint32_t* const cw = (uint32_t*)cnt + w * (CS / 2);
#pragma unroll
            for (int r = 0; r < KI; r++)
                pd[r] = min(group_digit(ord_of(key[r]), g.base, g.shift, (1u << g.bits) - 1u, pivot, g.mul), (uint32_t)D - 1u);
            if (!redo) {
                uint32_t old[KI];
#pragma unroll
                for (int r = 0; r < KI; r++) {
                    old[r] = 0;
                    if ((w * KI + r) * 64 + l < rows) old[r] = atomicAdd(cw + pd[r] / 2, 1u << (pd[r] & 1) * 16);
                }
#pragma unroll
                for (int r = 0; r < KI; r++) pd[r] = pd[r] << 16 | (old[r] >> (pd[r] & 1) * 16 & 0xffffu);
            } else {
#pragma unroll
                for (int r = 0; r < KI; r++) {
                    const bool val = (w * KI + r) * 64 + l < rows;
                    const uint32_t d = pd[r];
                    uint64_t peers = ballot(val);
#pragma unroll 1
                    for (int b = 0; b < MAX_DIGIT_BITS; b++) {
                        const bool bit = (d >> b) & 1u;
                        const uint64_t m = ballot(bit);
                        peers &= bit ? m : ~m;
                    }
                    const uint32_t below = mbcnt(peers);
                    const uint32_t base = val ? cnt[w * CS + d] : 0u;
                    if (val && below == 0) cnt[w * CS + d] = (uint16_t)(base + __popcll(peers));
                    pd[r] = d << 16 | (base + below);
                }
            }
            // The next tile's rows arrive while this one leaves: a third of the
            // loads here and two more below, so that they do not queue at once.
            if (!last) load_rids(next_rid, t0 + TILE);
            lds_barrier();
            if (t == 0) s_unordered = 0;
            {
                // offsets of (digit, wave) inside the tile
                constexpr int EPT = D * NW / NT;
                uint32_t v[EPT], sum = 0, total;
#pragma unroll
                for (int i = 0; i < EPT; i++) {
                    const int e = t * EPT + i;
                    v[i] = cnt[(e % NW) * CS + e / NW];
                    sum += v[i];
                }
                uint32_t ex = block_excl_scan<NT>(sum, tmp, &total);
#pragma unroll
                for (int i = 0; i < EPT; i++) {
                    const int e = t * EPT + i;
                    cnt[(e % NW) * CS + e / NW] = (uint16_t)ex;
                    ex += v[i];
                }
            }
            lds_barrier();
#pragma unroll
            for (int r = 0; r < KI; r++) pd[r] += cnt[w * CS + (pd[r] >> 16)];
            uint32_t tex = 0, end = 0, ngk = 0, ngr = 0;
            if (t < nbins) {
                tex = cnt[t];
                end = cur + (t + 1 < (uint32_t)D ? cnt[t + 1] : rows) - tex;
                ngk = (end + phk + (last ? GK - 1 : 0)) / GK - (cur + phk) / GK;
                if (RIDS) ngr = (end + phr + (last ? GR - 1 : 0)) / GR - (cur + phr) / GR;
            }
            uint32_t lines;
            const uint32_t g0 = block_excl_scan<NT>(ngk | ngr << 16, tmp, &lines);  // barriers: the counters are read
            asm volatile("" : "+v"(t), "+v"(l));
            list_lines<LGK>(lin, g0 & 0xffffu, ngk, cur, t < nbins ? s_first[t] : 0u, tex, phk, t, l);
            if (t < nbins) {
                // rows from these staged positions (+ 32) on do not fill a line
                const uint32_t kk = tex + 32u + (end + phk) / GK * GK - (cur + phk);
                const uint32_t kr = RIDS ? tex + 32u + (end + phr) / GR * GR - (cur + phr) : 0u;
                s_keep[t] = kk | kr << 16;
                s_end[t] = end;
            }
#pragma unroll
            for (int r = 0; r < KI; r++) {
                if ((w * KI + r) * 64 + l < rows) {
                    if constexpr (NARROW) skey[pd[r] & 0xffffu] = (KO)(((uint32_t)ord_of(key[r]) - s_sub[pd[r] >> 16]) ^ 0x80000000u);
                    else skey[pd[r] & 0xffffu] = (KO)key[r];
                }
            }
            if (!last) load_keys(t0 + TILE, 0, KI / 2);
            lds_barrier();
            write_lines<KO, LGK>(dst_k, phk, skey, CK, lin, lines & 0xffffu, s_end, last, redo != 0, t);
            lds_barrier();
            if (!last) {
                load_keys(t0 + TILE, KI / 2, KI);
                // (a tile that is not the last is full)
#pragma unroll
                for (int r = 0; r < KI; r++) {
                    const uint32_t d = pd[r] >> 16, p = pd[r] & 0xffffu, s = p + 32u - (s_keep[d] & 0xffffu);
                    if ((int32_t)s >= 0) skey[CK + d * GK + s] = skey[p];
                }
            }
            if constexpr (!RIDS) {
                lds_barrier();
                break;  // (a count does not depend on the order of equal digits)
            }
            if constexpr (RIDS) {
                asm volatile("" : "+v"(t), "+v"(l));
                lds_barrier();
                {
                    // (formed again from LDS: kept, they would cost registers)
                    uint32_t n = 0, at = 0, f = 0;
                    if (t < nbins) {
                        const uint32_t e = s_end[t];
                        n = (e + phr + (last ? GR - 1 : 0)) / GR - (cur + phr) / GR;
                        at = (s_keep[t] >> 16) - 32u - (e + phr) / GR * GR + (cur + phr);  // its first staged position
                        f = s_first[t];
                    }
                    list_lines<LGR>(lin, g0 >> 16, n, cur, f, at, phr, t, l);
                }
#pragma unroll
                for (int r = 0; r < KI; r++) {
                    const uint32_t x = (w * KI + r) * 64 + l;
                    if (x < rows) {
                        srid[pd[r] & 0xffffu] = rid[r];
                        stag[pd[r] & 0xffffu] = (pd[r] & 0xffff0000u) | x;
                    }
                }
                lds_barrier();
                bool unordered = false;
#pragma unroll
                for (int r = 0; r < KI; r++) {
                    const uint32_t p = r * NT + t;
                    const uint32_t tag = stag[p];
                    uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)tag, 0x138, 0xf, 0xf, false);  // wave_shr:1
                    if (l == 0 && p) prev = stag[p - 1];
                    unordered = unordered || (p > 0 && p < rows && prev >= tag);
                }
                if (unordered) s_unordered = 1;
                write_lines<int32_t, LGR>(dst_r, phr, srid, CR, lin, lines >> 16, s_end, last, redo != 0, t);
                lds_barrier();
                if (!last) {
#pragma unroll
                    for (int r = 0; r < KI; r++) {
                        const uint32_t d = pd[r] >> 16, s = (pd[r] & 0xffffu) + 32u - (s_keep[d] >> 16);
                        if ((int32_t)s >= 0) srid[CR + d * GR + s] = rid[r];
                    }
                }
                if (redo || !(s_unordered || force)) break;
                load_keys(t0, 0, KI);
            }
        }
        if constexpr (RIDS) {
#pragma unroll
            for (int r = 0; r < KI; r++) rid[r] = next_rid[r];
        }
        if (t < nbins) cur = s_end[t];
    }
}

hipError_t launch_scatter_lines(int key_bytes, int out_key_bytes, bool rids, const ChunkDesc* chunks, uint32_t nchunks,
                                const GroupDesc* groups, const uint32_t* hist, const uint32_t* cbsum,
                                const uint64_t* cstart, BufSet bufs, const uint32_t* skip, hipStream_t st)
{
    if (nchunks == 0) return hipSuccess;
    if (out_key_bytes > key_bytes) return hipErrorInvalidValue;
#define TJ_SL(K, KO, R) \
    hipLaunchKernelGGL((k_scatter_lines<K, KO, R>), dim3(nchunks), dim3(LN_NT), 0, st, chunks, groups, hist, cbsum, cstart, bufs, skip)
    if (key_bytes == 4) {
        if (rids) TJ_SL(int32_t, int32_t, true);
        else TJ_SL(int32_t, int32_t, false);
    } else if (out_key_bytes == 8) {
        if (rids) TJ_SL(int64_t, int64_t, true);
        else TJ_SL(int64_t, int64_t, false);
    } else {
        if (rids) TJ_SL(int64_t, int32_t, true);
        else TJ_SL(int64_t, int32_t, false);
    }
#undef TJ_SL
    return hipGetLastError();
}

hipError_t launch_scatter(int key_bytes, int out_key_bytes, bool rids, bool keys, const ChunkDesc* chunks,
                          uint32_t nchunks, const GroupDesc* groups, const uint32_t* hist,
                          const uint32_t* cbsum, const uint64_t* cstart, BufSet bufs, const uint32_t* skip,
                          hipStream_t st)
{
    if (nchunks == 0) return hipSuccess;
    if (out_key_bytes > key_bytes) return hipErrorInvalidValue;
    const dim3 grid(nchunks), block(SC_NT);
    const BktSet none{};
#define TJ_SC(K, KO, R, W)                                                                           \
    hipLaunchKernelGGL((k_scatter<K, KO, R, W, false>), grid, block, 0, st, chunks, groups, hist, cbsum, cstart, \
                       bufs, none, skip)
    if (key_bytes == 4) {
        if (!keys) TJ_SC(int32_t, int32_t, true, false);
        else if (rids) TJ_SC(int32_t, int32_t, true, true);
        else TJ_SC(int32_t, int32_t, false, true);
    } else if (out_key_bytes == 8 || !keys) {
        if (!keys) TJ_SC(int64_t, int64_t, true, false);
        else if (rids) TJ_SC(int64_t, int64_t, true, true);
        else TJ_SC(int64_t, int64_t, false, true);
    } else {
        if (rids) TJ_SC(int64_t, int32_t, true, true);
        else TJ_SC(int64_t, int32_t, false, true);
    }
#undef TJ_SC
    return hipGetLastError();
}

hipError_t launch_learned_scatter(int key_bytes, bool rids, const ChunkDesc* chunks, uint32_t nchunks,
                                  const GroupDesc* groups, const uint32_t* hist, const uint32_t* cbsum,
                                  const uint64_t* cstart, BufSet bufs, BktSet bkt, hipStream_t st)
{
    if (nchunks == 0) return hipSuccess;
    const dim3 grid(nchunks), block(SC_NT);
#define TJ_SCL(K, R)                                                                                  \
    hipLaunchKernelGGL((k_scatter<K, K, R, true, true>), grid, block, 0, st, chunks, groups, hist, cbsum,  \
                       cstart, bufs, bkt, nullptr)
    if (key_bytes == 4) {
        if (rids) TJ_SCL(int32_t, true);
        else TJ_SCL(int32_t, false);
    } else {
        if (rids) TJ_SCL(int64_t, true);
        else TJ_SCL(int64_t, false);
    }
#undef TJ_SCL
    return hipGetLastError();
}

// Expansion of a single-key join range straight in the output columns.
// mode 0: dst[t] = src[t / b] for t in [0, n); mode 1: dst[t] = dst[t mod b] for t in [b, n).
__global__ __launch_bounds__(256) void k_expand(int32_t* __restrict__ dst, const int32_t* __restrict__ src,
                                                uint64_t n, uint64_t b, int mode)
{
    for (uint64_t t = blockIdx.x * 256ull + threadIdx.x; t < n; t += (uint64_t)gridDim.x * 256) {
        uint64_t i = (uint64_t)((double)t / (double)b);
        while (i * b > t) i--;
        while ((i + 1) * b <= t) i++;
        if (mode == 0) dst[t] = src[i];
        else if (t >= b) dst[t] = dst[t - i * b];
    }
}

hipError_t launch_expand(int32_t* dst, const int32_t* src, uint64_t n, uint64_t b, int mode, hipStream_t st)
{
    if (n == 0 || b == 0) return hipSuccess;
    uint64_t blocks = (n + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(k_expand, dim3((uint32_t)blocks), dim3(256), 0, st, dst, src, n, b, mode);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// per-bucket LDS sort: a stable LSD radix sort, 8-bit digits, of NT*KI items
// held in registers, items exchanged through LDS after every digit. KW is the
// relative-key word: 32 bits when the bucket's keys span < 2^32, else 64.
// On return the sorted items are in lds_key / lds_idx. Padding items carry
// the all-ones key and the largest positions, so they sort last.
// ---------------------------------------------------------------------------
constexpr int LBINS = 256, LSTRIDE = LBINS + 1;
// Block shape of a leaf of at most C rows, per key word. C = LEAF_CAP: 32-bit
// keys use 512 threads x 16 rows (in k_leaf_sort_narrow 64 KiB of LDS, two blocks
// per CU); 64-bit keys 1024 threads x 8 rows. The smaller capacities are for inputs
// of one block, where nothing but the block's own latency counts: 4 rows a thread.
// (A join block has 1024 threads x 8 rows with either key word: FULL.)
template <typename KW, int C = LEAF_CAP, bool FULL = false> struct LeafShape {
    static constexpr int NT = C < LEAF_CAP ? C / 4 : sizeof(KW) == 4 && !FULL ? 512 : 1024;
    static constexpr int KI = C / NT;
    static constexpr int NW = NT / 64;
    static constexpr int NBB = C == 1024 ? 10 : C == 4096 ? 12 : sizeof(KW) == 4 ? 12 : 13;  // bin bits of block_bin_sort
    static constexpr int NBIN = 1 << NBB;
    // LDS words shared by the bin counters and the LSD digit counters
    static constexpr int CNT_WORDS = NBIN > NW * LSTRIDE ? NBIN : NW * LSTRIDE;
};

// LDS array whose element i sits at i + (i / G) * S: S spare elements after
// every G. With G = the items per thread, a wave reading its items in blocked
// order (lane l at l*G + i) has an odd stride in 4-byte words and so spreads
// its lanes over the banks; consecutive-lane access stays conflict-free.
template <typename T, int G, int S>
struct LdsPad {
    T* p;
    __device__ __forceinline__ T& operator[](uint32_t i) const { return p[i + (i / G) * S]; }
    // element t*G + i, i < G (thread t's i-th item in blocked order)
    __device__ __forceinline__ T& blk(uint32_t t, uint32_t i) const { return p[t * (G + S) + i]; }
    // all G items of thread t; 16-byte loads for an unpadded 16-bit array (a
    // wave then reads 16 bytes per lane instead of 2, with 8x fewer conflicts)
    __device__ __forceinline__ void blk_all(uint32_t t, uint32_t (&out)[G]) const
    {
        if constexpr (S == 0 && sizeof(T) == 2 && (G * 2) % 16 == 0) {
            const uint4* v = (const uint4*)(p + t * G);
#pragma unroll
            for (int j = 0; j < G * 2 / 16; j++) {
                const uint4 w = v[j];
                const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int h = 0; h < 4; h++) {
                    out[j * 8 + 2 * h] = ws[h] & 0xffffu;
                    out[j * 8 + 2 * h + 1] = ws[h] >> 16;
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < G; i++) out[i] = p[t * (G + S) + i];
        }
    }
    static constexpr uint32_t size(uint32_t n) { return n + (n / G) * S; }
};
// sort blocks read their sorted items across lanes: plain layout (for the join's, see JoinLds)
template <typename KW, int C = LEAF_CAP> using KeyPlain = LdsPad<KW, LeafShape<KW, C>::KI, 0>;
template <typename KW, int C = LEAF_CAP> using IdxPlain = LdsPad<uint16_t, LeafShape<KW, C>::KI, 0>;

// Largest bin block_bin_sort accepts: the exact ranking inside a bin costs
// every item of the bin one pass over it.
constexpr uint32_t BIN_MAXC = 48;  // < 64: the bin size is packed in 6 bits

// Stable sort of the block's items in one counting pass. Item key[r] sits at
// position q = (w*KI + r)*64 + l; items with q < n are sorted, the rest are
// padding and stay at q (their keys are all ones and their positions the
// largest, so that is their sorted place too). An item's index is its
// position q, so the stable order is the order of the pairs (key, q).
//  1. Each item is counted into one of 2^NBB bins by the top bits of its key
//     (LDS atomics; the slot an item gets inside its bin is arbitrary).
//  2. An exclusive scan of the bin counts gives each bin's first position;
//     the items are written there in slot order.
//  3. Each item of a bin with two or more items counts the items of its bin
//     that precede it in (key, q) order and moves to that rank.
// The result, in lds_key / lds_idx, is exact whatever order the atomics take.
// Returns false, having written nothing to lds_key / lds_idx, when some bin
// holds more than BIN_MAXC items; the caller then sorts another way.
template <typename KW, int NT, int KI, int NBB, typename KA, typename IA>
__device__ __forceinline__ bool block_bin_sort(const KW (&key)[KI], int bits, uint32_t n, KA lds_key,
                                               IA lds_idx, uint32_t* hist, uint32_t* tmp)
{
    constexpr int NBIN = 1 << NBB, BPT = NBIN / NT;
    static_assert(NBIN % NT == 0, "bins must split evenly over the block");
    static_assert(NT * KI <= 8192, "positions are packed in 13 bits");
    const uint32_t w = threadIdx.x / 64, l = threadIdx.x & 63;
    const int hb = bits < NBB ? bits : NBB;
    const int sh = bits - hb;
    for (uint32_t i = threadIdx.x; i < (uint32_t)NBIN; i += NT) hist[i] = 0;
    lds_barrier();
    // per item: bin | slot << 16, then pos | first of bin << 13 | bin size << 26,
    // then (1 << 31 | final position) for the items that move
    // (array elements are only ever assigned unconditionally: a conditional
    // assignment makes the compiler copy the whole array through every branch)
    uint32_t info[KI];
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = (w * KI + r) * 64 + l;
        const KW kb = key[r] >> sh;  // < 2^NBB when the keys span `bits` bits
        const uint32_t b = kb < (KW)NBIN ? (uint32_t)kb : (uint32_t)NBIN - 1u;
        uint32_t slot = 0;
        if (q < n) slot = atomicAdd(&hist[b], 1u);
        info[r] = b | (slot << 16);
    }
    lds_barrier();
    uint32_t c[BPT], sum = 0, mx = 0;
#pragma unroll
    for (int i = 0; i < BPT; i++) {
        c[i] = hist[threadIdx.x * BPT + i];
        sum += c[i];
        mx = c[i] > mx ? c[i] : mx;
    }
    if (block_max<NT>(mx, tmp) > BIN_MAXC) return false;
    uint32_t tot;
    uint32_t ex = block_excl_scan<NT>(sum, tmp, &tot);
#pragma unroll
    for (int i = 0; i < BPT; i++) {
        hist[threadIdx.x * BPT + i] = ex;
        ex += c[i];
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = (w * KI + r) * 64 + l;
        const uint32_t b = info[r] & 0xffffu;
        const uint32_t s0 = hist[b];
        const uint32_t e0 = b + 1 < (uint32_t)NBIN ? hist[b + 1] : n;
        const bool valid = q < n;
        const uint32_t pos = valid ? s0 + (info[r] >> 16) : q;
        info[r] = valid ? pos | (s0 << 13) | ((e0 - s0) << 26) : 0u;
        lds_key[pos] = key[r];
        lds_idx[pos] = (uint16_t)q;
    }
    lds_barrier();
    // The thread's items walk their bins in step, so that the LDS reads of all
    // of them are in flight together: step j reads element j of each bin (an
    // item whose bin is shorter re-reads its bin's first element and ignores it).
    uint32_t rank[KI], cbmax = 0;
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t cb = info[r] >> 26;
        rank[r] = 0;
        cbmax = cb > 1 && cb > cbmax ? cb : cbmax;
    }
    for (uint32_t j = 0; j < cbmax; j++) {
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const uint32_t q = (w * KI + r) * 64 + l;
            const uint32_t s0 = (info[r] >> 13) & 0x1fffu, cb = info[r] >> 26;
            const bool act = j < cb;
            const uint32_t e = act ? s0 + j : s0;
            const KW kj = lds_key[e];
            const uint32_t ij = lds_idx[e];
            rank[r] += (act && (kj < key[r] || (kj == key[r] && ij < q))) ? 1u : 0u;
        }
    }
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t pos = info[r] & 0x1fffu, s0 = (info[r] >> 13) & 0x1fffu, cb = info[r] >> 26;
        info[r] = (cb > 1 && s0 + rank[r] != pos) ? 0x80000000u | (s0 + rank[r]) : 0u;
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < KI; r++) {
        if (info[r] >> 31) {
            const uint32_t q = (w * KI + r) * 64 + l;
            lds_key[info[r] & 0x1fffu] = key[r];
            lds_idx[info[r] & 0x1fffu] = (uint16_t)q;
        }
    }
    lds_barrier();
    return true;
}

// ATOMIC ranks with one LDS atomic per item (in lane order on this hardware,
// which makes every pass stable); the caller must then check that the result
// is ordered by (key, idx) and sort again with ATOMIC = false if it is not.
// SHARED: cnt and tmp lie inside lds_key / lds_idx (two more barriers a pass).
template <typename KW, int NT, int KI, bool ATOMIC = false, bool SHARED = false, typename KA, typename IA>
__device__ __forceinline__ void block_lsd_sort(KW (&key)[KI], uint16_t (&idx)[KI], int bits,
                                               KA lds_key, IA lds_idx, uint32_t* cnt,
                                               uint32_t* tmp, int lo_bit = 0)
{
    constexpr int NW = NT / 64;
    const uint32_t w = threadIdx.x / 64, l = threadIdx.x & 63;
    const int passes = (bits + 7) / 8;
    if (passes == 0) {
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const uint32_t q = (w * KI + r) * 64 + l;
            lds_key[q] = key[r];
            lds_idx[q] = idx[r];
        }
        lds_barrier();
        return;
    }
    for (int p = 0; p < passes; p++) {
        const int sh = lo_bit + 8 * p;
        const int nb = bits - 8 * p < 8 ? bits - 8 * p : 8;
        const uint32_t mask = (1u << nb) - 1u;
        uint32_t dig[KI], rk[KI];
#pragma unroll
        for (int r = 0; r < KI; r++) dig[r] = (uint32_t)(key[r] >> sh) & mask;
        for (uint32_t i = l; i < LBINS; i += 64) cnt[w * LSTRIDE + i] = 0;
        if (ATOMIC) {
#pragma unroll
            for (int r = 0; r < KI; r++) rk[r] = atomicAdd(&cnt[w * LSTRIDE + dig[r]], 1u);
        } else {
#pragma unroll
            for (int r = 0; r < KI; r++) rk[r] = wave_rank(dig[r], true, nb, &cnt[w * LSTRIDE]);
        }
        lds_barrier();
        scan_counts<NT, NW, LBINS>(cnt, tmp);
#pragma unroll
        for (int r = 0; r < KI; r++) {
            rk[r] += cnt[w * LSTRIDE + dig[r]];
        }
        if (SHARED) lds_barrier();
#pragma unroll
        for (int r = 0; r < KI; r++) {
            lds_key[rk[r]] = key[r];
            lds_idx[rk[r]] = idx[r];
        }
        lds_barrier();
        // (reloaded after the last pass too: a conditional reload would make
        // the compiler copy both arrays through the branch)
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const uint32_t q = (w * KI + r) * 64 + l;
            key[r] = lds_key[q];
            idx[r] = lds_idx[q];
        }
        if (SHARED) lds_barrier();
    }
}

// True (the same on every thread) when the first n items of lds_key/lds_idx
// are in strictly increasing (key, idx) order. *flag must be 0 on entry and
// is 0 again on return; ends with a barrier.
template <typename KW, int NT, int KI, typename KA, typename IA>
__device__ __forceinline__ bool block_check_order(KA lds_key, IA lds_idx, uint32_t n, uint32_t* flag)
{
    const uint32_t t = threadIdx.x, p0 = t * KI;
    KW kp = t ? lds_key.blk(t - 1, KI - 1) : (KW)0;
    uint32_t ip = t ? lds_idx.blk(t - 1, KI - 1) : 0u;
    uint32_t xs[KI];
    lds_idx.blk_all(t, xs);
    bool bad = false;
#pragma unroll
    for (int i = 0; i < KI; i++) {
        const uint32_t p = p0 + i;
        const KW k = lds_key.blk(t, i);
        const uint32_t x = xs[i];
        bad = bad || (p > 0 && p < n && !(kp < k || (kp == k && ip < x)));
        kp = k;
        ip = x;
    }
    if (bad) *flag = 1;
    lds_barrier();
    const bool ok = *flag == 0;
    lds_barrier();
    if (threadIdx.x == 0) *flag = 0;
    return ok;
}

// The thread's share of the places whose key's bits from H on are those of the
// place before (ties), and << 32 of all places out of (key, index) order. Rows of
// one key are ties, but in order: input with many rows a key is done without its
// lower bits.
template <int NT, int KI, typename KA, typename IA>
__device__ __forceinline__ uint64_t count_ties(KA lds_key, IA lds_idx, uint32_t n, int H)
{
    uint64_t ties = 0;
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = threadIdx.x + r * NT;
        if (q > 0 && q < n) {
            const auto k0 = lds_key[q - 1], k1 = lds_key[q];
            const bool out = k0 > k1 || (k0 == k1 && lds_idx[q - 1] > lds_idx[q]);
            ties += ((k0 >> H) == (k1 >> H) ? 1u : 0u) + (out ? 1ull << 32 : 0ull);
        }
    }
    return ties;
}

// Puts runs of ties in (key, index) order, one thread a run (insertion sort).
// Ends with a barrier.
template <typename KW, int NT, int KI, typename KA, typename IA>
__device__ __forceinline__ void sort_ties(KA lds_key, IA lds_idx, uint32_t n, int H)
{
#pragma unroll 1
    for (int r = 0; r < KI; r++) {
        const uint32_t q = threadIdx.x + r * NT;
        const bool head = q + 1 < n && (lds_key[q] >> H) == (lds_key[q + 1] >> H) &&
                          (q == 0 || (lds_key[q] >> H) != (lds_key[q - 1] >> H));
        if (!head) continue;
        uint32_t e = q + 1;
        while (e < n && (lds_key[e] >> H) == (lds_key[q] >> H)) e++;
        for (uint32_t i = q + 1; i < e; i++) {
            const KW kv = lds_key[i];
            const uint16_t iv = lds_idx[i];
            uint32_t j = i;
            while (j > q && (lds_key[j - 1] > kv || (lds_key[j - 1] == kv && lds_idx[j - 1] > iv))) {
                lds_key[j] = lds_key[j - 1];
                lds_idx[j] = lds_idx[j - 1];
                j--;
            }
            lds_key[j] = kv;
            lds_idx[j] = iv;
        }
    }
    lds_barrier();
}

// Stable sort of a leaf block's items (see block_bin_sort for their layout) into
// lds_key / lds_idx: one counting pass, or digit passes when a bin is too full.
// reload() gives the items their keys and indices again.
template <typename KW, int NT, int KI, int NBB, typename KA, typename IA, class Reload>
__device__ __forceinline__ void block_sort(KW (&key)[KI], uint16_t (&idx)[KI], int bits, uint32_t n, KA lds_key,
                                           IA lds_idx, uint32_t* cnt, uint32_t* tmp, uint64_t* tmp64, Reload&& reload)
{
    if (bits > 0 &&
        block_bin_sort<KW, NT, KI, NBB>(key, bits, n, lds_key, lds_idx, cnt, tmp)) {
        // sorted in one counting pass
    } else if (sizeof(KW) == 8 && bits > 32) {
        // Wide keys: sort by the top 32 bits of the relative key only (4 digit
        // passes instead of up to 8). The order is final unless two rows share
        // those 32 bits; short runs of such ties are then put in order by one
        // thread each (insertion sort on the full key, which keeps equal keys in
        // input order); many ties fall back to the full sort.
        const int H = bits - 32;
        block_lsd_sort<KW, NT, KI>(key, idx, 32, lds_key, lds_idx, cnt, tmp, H);
        const uint64_t c = block_sum64<NT>(count_ties<NT, KI>(lds_key, lds_idx, n, H), tmp64);
        const uint32_t ties = c >> 32 ? (uint32_t)c : 0u;
        if (ties > 0 && ties <= 256) {
            sort_ties<KW, NT, KI>(lds_key, lds_idx, n, H);
        } else if (ties > 256) {
            reload();
            block_lsd_sort<KW, NT, KI>(key, idx, bits, lds_key, lds_idx, cnt, tmp);
        }
    } else {
        block_lsd_sort<KW, NT, KI>(key, idx, bits, lds_key, lds_idx, cnt, tmp);
    }
}

// Leaves up to which each has a CU of its own, and may use all of its registers
// (beyond, two blocks a CU pay: see k_leaf_sort).
constexpr uint32_t DENSE_LEAVES = 256;

// Shape of a sort leaf: 1024 threads x 8 rows within 64 VGPRs and half of a
// CU's LDS, so that two blocks share a CU.
template <typename KW> struct SortLeaf {
    static constexpr int NT = 1024, KI = LEAF_CAP / NT, NBB = 13, NBIN = 1 << NBB;
    static constexpr int WORDS = LEAF_CAP * sizeof(KW);  // words in bins, then sorted keys
    static constexpr int HIST = NBIN * 2;                // bin counters, or indices (digit passes)
    static constexpr int BYTES = sizeof(KW) == 8 ? WORDS + HIST : 2 * WORDS;
    static_assert(BYTES <= 81920 && LEAF_CAP * 2 <= HIST && KI * NT == LEAF_CAP, "two blocks a CU");
};

// The sort of one leaf by digit passes, for leaves with too many rows in one bin.
template <typename K, typename KW>
__device__ __forceinline__ void leaf_sort_passes(char* pool, uint32_t n, uint64_t base, int bits,
                                                 const K* __restrict__ src_k, const int32_t* __restrict__ src_r,
                                                 K* __restrict__ out_k, int32_t* __restrict__ out_r)
{
    using SL = SortLeaf<KW>;
    constexpr int NT = SL::NT, KI = SL::KI;
    const LdsPad<KW, KI, 0> lds_key{(KW*)pool};
    const LdsPad<uint16_t, KI, 0> lds_idx{(uint16_t*)(pool + SL::WORDS)};
    uint32_t* const cnt = (uint32_t*)pool;
    uint32_t* const tmp = cnt + NT / 64 * LSTRIDE;
    uint64_t* const tmp64 = (uint64_t*)(pool + SL::WORDS);
    const uint32_t w = threadIdx.x / 64, l = threadIdx.x & 63;
    KW key[KI];
    uint16_t idx[KI];
    auto load_items = [&]() {
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const uint32_t q = (w * KI + r) * 64 + l;
            const K v = ld_clamp(src_k, q, n);
            key[r] = q < n ? (KW)(ord_of(v) - base) : (KW)~(KW)0;
            idx[r] = (uint16_t)q;
        }
    };
    lds_barrier();
    load_items();
    // Wide keys: by the top 32 bits of the relative key first (4 digit passes
    // instead of up to 8). That order is final unless rows share those bits and
    // differ below; few such ties are put in order by one thread a run, more take
    // the passes over all bits.
    for (int H = bits > 32 ? bits - 32 : 0;; H = 0) {
        block_lsd_sort<KW, NT, KI, false, true>(key, idx, bits - H, lds_key, lds_idx, cnt, tmp, H);
        if (H == 0) break;
        uint64_t c = count_ties<NT, KI>(lds_key, lds_idx, n, H);
        lds_barrier();
        c = uniform(block_sum64<NT>(c, tmp64));
#pragma unroll
        for (int r = 0; r < KI; r++) lds_idx[(w * KI + r) * 64 + l] = idx[r];
        lds_barrier();
        if (c >> 32 == 0) break;
        if ((uint32_t)c <= 256) {
            sort_ties<KW, NT, KI>(lds_key, lds_idx, n, H);
            break;
        }
        load_items();
    }
    // Keys go out first. The bucket may be sorted in place (its rows already
    // sit in the output columns), so its row ids are all read (coalesced, into
    // the now free key array) before any of them is overwritten.
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = (w * KI + r) * 64 + l;
        if (q < n) out_k[q] = key_of<K>(base + (uint64_t)lds_key[q]);
    }
    lds_barrier();
    int32_t* const lds_rid = (int32_t*)pool;
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = threadIdx.x + r * NT;
        if (q < n) lds_rid[q] = src_r[q];
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = (w * KI + r) * 64 + l;
        if (q < n) out_r[q] = lds_rid[lds_idx[q]];
    }
}

// The sort of one leaf. Each row is one word [key below its bin's bits | row] in
// its bin of 2^13 (one to two rows a bin on average where keys are even), so that
// one comparison of words decides the order (key, row) inside a bin whatever order
// the bins were filled in. A row's key and row id stay with its thread, which
// puts them in their places in LDS, from where they leave coalesced.
// Bound by the memory traffic of its rows once two blocks share a CU: 2^29 rows
// of 64-bit keys, 2.8 ms (4.6 TB/s; a copy reaches 4.7) from 4.3 ms with one block
// of 148 KiB a CU, whose loads, LDS steps and stores followed one another.
// DENSE: two blocks a CU, which leaves 64 VGPRs; a leaf with too many rows in one
// bin is marked, for k_leaf_sort_passes (as a call from here the passes would make
// this way spill). Otherwise, with a CU for every leaf, the leaf is sorted that way
// at once: 100k rows, 14 us from 29; 1M Zipf rows, 92 us from 131.
template <typename K, typename KW, bool DENSE>
__global__ __launch_bounds__(SortLeaf<KW>::NT)
__attribute__((amdgpu_waves_per_eu(DENSE ? 8 : 4))) void k_leaf_sort(LeafDesc* __restrict__ leaves, BufSet bufs,
                                                                     K* __restrict__ out_k,
                                                                     int32_t* __restrict__ out_r)
{
    using SL = SortLeaf<KW>;
    constexpr int NT = SL::NT, KI = SL::KI;
    __shared__ __align__(16) char pool[SL::BYTES];
    KW* const word = (KW*)pool;
    uint16_t* const start = (uint16_t*)(pool + SL::WORDS);  // rows of a bin, then its first place
    uint32_t* const tmp = (uint32_t*)pool;

    const LeafDesc L = leaves[blockIdx.x];
    const uint32_t n = L.rn;
    if (n == 0) return;
    const K* __restrict__ src_k = (const K*)bufs.key[L.buf][0] + L.kr0;
    const int32_t* __restrict__ src_r = bufs.rid[L.buf][0] + L.r0;
    const uint32_t w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.x / 64) * (KI * 64);
    const uint32_t t = threadIdx.x;
    uint32_t l = t & 63;
    auto row = [&](int r) { return w0 + r * 64 + l; };
    auto fresh = [&]() { asm volatile("" : "+v"(l)); };
    // rows beyond n take no part: nothing of theirs is stored in LDS
    KW key[KI];
    uint32_t info[KI];
    {
        K v[KI];
#pragma unroll
        for (int r = 0; r < KI; r++) v[r] = ld_now(src_k, min(row(r), n - 1));
#pragma unroll
        for (int r = 0; r < KI; r++) key[r] = (KW)(ord_of(v[r]) - L.base);
    }
    const int sh = (int)L.bits > SL::NBB ? (int)L.bits - SL::NBB : 0;
    static_assert(SL::HIST == NT * 16, "16 bytes of counters a thread");
    ((uint4*)start)[t] = uint4{0, 0, 0, 0};
    lds_barrier();
    fresh();
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t b = (uint32_t)(key[r] >> sh) & (SL::NBIN - 1u);
        uint32_t slot = 0;
        if (row(r) < n) slot = atomicAdd((uint32_t*)start + b / 2, 1u << (b & 1) * 16) >> (b & 1) * 16;
        info[r] = b | slot << 16;
    }
    lds_barrier();
    {
        uint4 x = ((const uint4*)start)[t];
        uint32_t c[4] = {x.x, x.y, x.z, x.w}, sum = 0, mx = 0, all;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t a = c[i] & 0xffffu, b = c[i] >> 16;
            sum += a + b;
            mx = max(mx, max(a, b));
        }
        if (uniform(block_max<NT>(mx, tmp)) > BIN_MAXC) {
            if constexpr (DENSE) {
                if (t == 0) leaves[blockIdx.x].flags = L.flags | LEAF_CROWDED;
            } else {
                leaf_sort_passes<K, KW>(pool, n, L.base, (int)L.bits, src_k, src_r, out_k + L.out, out_r + L.out);
            }
            return;
        }
        uint32_t ex = block_excl_scan<NT>(sum, tmp, &all);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t a = c[i] & 0xffffu, b = c[i] >> 16;
            c[i] = ex | (ex + a) << 16;
            ex += a + b;
        }
        ((uint4*)start)[t] = uint4{c[0], c[1], c[2], c[3]};
    }
    lds_barrier();
    fresh();
    uint32_t cbmax = 0;
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t b = info[r] & 0xffffu, slot = info[r] >> 16;
        const uint32_t s0 = start[b], e0 = b + 1 < (uint32_t)SL::NBIN ? start[b + 1] : n, cb = e0 - s0;
        const bool valid = row(r) < n;
        key[r] = (key[r] & (((KW)1 << sh) - 1)) << 13 | (KW)row(r);
        if (valid) word[s0 + slot] = key[r];
        info[r] = valid ? s0 | cb << 13 | b << 19 : 0u;  // first place, rows and number of its bin
        cbmax = valid && cb > 1 && cb > cbmax ? cb : cbmax;
    }
#pragma unroll
    for (int r = 0; r < KI; r++) asm volatile("" : "+v"(info[r]));  // (packed, see k_leaf_join)
    lds_barrier();
    // The thread's rows walk their bins in step (past a shorter bin's end, still
    // in the pool: ignored).
    uint32_t rank[KI];
#pragma unroll
    for (int r = 0; r < KI; r++) rank[r] = 0;
#pragma unroll 1
    for (uint32_t j = 0; j < cbmax; j++) {
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const KW x = word[(info[r] & 0x1fffu) + j];
            rank[r] += j < (info[r] >> 13 & 63u) && x < key[r] ? 1u : 0u;
        }
    }
    // (row ids: on their way while the keys leave)
    fresh();
    int32_t rid[KI];
#pragma unroll
    for (int r = 0; r < KI; r++) rid[r] = ld_now(src_r, min(row(r), n - 1));
#pragma unroll
    for (int r = 0; r < KI; r++) rank[r] += info[r] & 0x1fffu;
    lds_barrier();
    int32_t* const lds_rid = (int32_t*)(sizeof(KW) == 8 ? pool : pool + SL::WORDS);
    const bool together = sizeof(KW) == 4;
#pragma unroll
    for (int r = 0; r < KI; r++) {
        if (info[r]) {
            word[rank[r]] = (KW)(info[r] >> 19) << sh | key[r] >> 13;
            if (together) lds_rid[rank[r]] = rid[r];
        }
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = t + r * NT;
        if (q < n) out_k[L.out + q] = key_of<K>(L.base + (uint64_t)word[q]);
    }
    if (!together) {
        lds_barrier();
#pragma unroll
        for (int r = 0; r < KI; r++)
            if (info[r]) lds_rid[rank[r]] = rid[r];
        lds_barrier();
    }
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = t + r * NT;
        if (q < n) out_r[L.out + q] = lds_rid[q];
    }
}

// The wide leaves that k_leaf_sort has marked, by digit passes: one block a CU,
// each with every 256th leaf (crowded leaves are often neighbours).
template <typename K, typename KW>
__global__ __launch_bounds__(SortLeaf<KW>::NT)
__attribute__((amdgpu_waves_per_eu(4))) void k_leaf_sort_passes(const LeafDesc* __restrict__ leaves, uint32_t count,
                                                                BufSet bufs, K* __restrict__ out_k,
                                                                int32_t* __restrict__ out_r)
{
    __shared__ __align__(16) char pool[SortLeaf<KW>::BYTES];
    for (uint32_t i0 = blockIdx.x; i0 < count; i0 += DENSE_LEAVES * 64) {
        const uint32_t i = i0 + (threadIdx.x & 63) * DENSE_LEAVES;
        uint64_t marked = ballot(i < count && (leaves[min(i, count - 1)].flags & LEAF_CROWDED));
        while (marked) {
            const LeafDesc L = leaves[i0 + (uint32_t)(__ffsll((unsigned long long)marked) - 1) * DENSE_LEAVES];
            marked &= marked - 1;
            leaf_sort_passes<K, KW>(pool, L.rn, L.base, (int)L.bits, (const K*)bufs.key[L.buf][0] + L.kr0,
                                    bufs.rid[L.buf][0] + L.r0, out_k + L.out, out_r + L.out);
        }
    }
}

// The sort of many leaves of 32-bit keys: one block does both ways, a counting
// pass, or digit passes for crowded leaves. Narrow keys are often few with many
// rows each, and a marked leaf has been read in vain: 2^28 rows of 2^20 keys take
// 1.8 ms here, 2^27 rows with 64 a key 1.5; with k_leaf_sort and
// k_leaf_sort_passes the latter took 2.5 (even keys would gain: 2^27 uniform ones
// 2.7 ms the whole sort there, 3.1 here).
template <typename K>
__global__ __launch_bounds__(LeafShape<uint32_t>::NT)
__attribute__((amdgpu_waves_per_eu(4))) void k_leaf_sort_narrow(const LeafDesc* __restrict__ leaves,
                                                            BufSet bufs, K* __restrict__ out_k,
                                                            int32_t* __restrict__ out_r)
{
    using KW = uint32_t;
    constexpr int NT = LeafShape<KW>::NT, KI = LeafShape<KW>::KI, NW = LeafShape<KW>::NW, C = LEAF_CAP;
    __shared__ KW lds_key_raw[C];
    __shared__ __align__(16) uint16_t lds_idx_raw[C];
    const KeyPlain<KW> lds_key{lds_key_raw};
    const IdxPlain<KW> lds_idx{lds_idx_raw};
    __shared__ uint32_t cnt[LeafShape<KW>::CNT_WORDS];
    __shared__ uint32_t tmp[NW];
    __shared__ uint64_t tmp64[NW];

    const LeafDesc L = leaves[blockIdx.x];
    if (L.rn == 0) return;
    const K* __restrict__ src_k = (const K*)bufs.key[L.buf][0] + L.kr0;
    const int32_t* __restrict__ src_r = bufs.rid[L.buf][0] + L.r0;
    const uint32_t w = threadIdx.x / 64, l = threadIdx.x & 63;
    KW key[KI];
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = (w * KI + r) * 64 + l;
        const K v = ld_clamp(src_k, q, L.rn);
        key[r] = q < L.rn ? (KW)(ord_of(v) - L.base) : (KW)~(KW)0;
    }
    uint16_t idx[KI];
#pragma unroll
    for (int r = 0; r < KI; r++) idx[r] = (uint16_t)((w * KI + r) * 64 + l);
    block_sort<KW, NT, KI, LeafShape<KW>::NBB>(key, idx, (int)L.bits, L.rn, lds_key, lds_idx, cnt, tmp, tmp64, [&]() {
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const uint32_t q = (w * KI + r) * 64 + l;
            const K v = ld_clamp(src_k, q, L.rn);
            key[r] = q < L.rn ? (KW)(ord_of(v) - L.base) : (KW)~(KW)0;
            idx[r] = (uint16_t)q;
        }
    });
    // Keys go out first. The bucket may be sorted in place (its rows already
    // sit in the output columns), so its row ids are all read (coalesced, into
    // the now free key array) before any of them is overwritten.
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = (w * KI + r) * 64 + l;
        if (q < L.rn) out_k[L.out + q] = key_of<K>(L.base + (uint64_t)lds_key[q]);
    }
    int32_t* lds_rid = (int32_t*)lds_key_raw;
    lds_barrier();
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = threadIdx.x + r * NT;
        const int32_t v = ld_clamp(src_r, q, L.rn);
        if (q < L.rn) lds_rid[q] = v;
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = (w * KI + r) * 64 + l;
        if (q < L.rn) out_r[L.out + q] = lds_rid[lds_idx[q]];
    }
}

hipError_t launch_leaf_sort(int key_bytes, bool wide, LeafDesc* leaves, uint32_t n,
                            BufSet bufs, void* out_k, int32_t* out_r, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    const dim3 grid(n), block(SortLeaf<uint64_t>::NT), narrow(LeafShape<uint32_t>::NT);
#define TJ_LS(K)                                                                                                   \
    do {                                                                                                           \
        if (n <= DENSE_LEAVES && wide) {                                                                           \
            hipLaunchKernelGGL((k_leaf_sort<K, uint64_t, false>), grid, block, 0, st, leaves, bufs, (K*)out_k, out_r); \
        } else if (n <= DENSE_LEAVES) {                                                                            \
            hipLaunchKernelGGL((k_leaf_sort<K, uint32_t, false>), grid, block, 0, st, leaves, bufs, (K*)out_k, out_r); \
        } else if (wide) {                                                                                         \
            hipLaunchKernelGGL((k_leaf_sort<K, uint64_t, true>), grid, block, 0, st, leaves, bufs, (K*)out_k, out_r); \
            hipLaunchKernelGGL((k_leaf_sort_passes<K, uint64_t>), dim3(DENSE_LEAVES), block, 0, st, leaves, n, bufs, \
                               (K*)out_k, out_r);                                                                  \
        } else {                                                                                                   \
            hipLaunchKernelGGL((k_leaf_sort_narrow<K>), grid, narrow, 0, st, leaves, bufs, (K*)out_k, out_r);      \
        }                                                                                                          \
    } while (0)
    if (key_bytes == 4) TJ_LS(int32_t);
    else TJ_LS(int64_t);
#undef TJ_LS
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// sort of an input that fits one block: the key range, the sort and the output
// in one launch, so that the call waits once. The time is the block's own
// chain of latencies (two loads, about a dozen barriers) and hardly depends on
// the rows, so the block has few rows a thread and all its loads go out at once.
// A call of 1000 int32 rows: 65 us with two fills, a probe, its read-back and a
// 512 x 16 leaf, 24 us with this (about 6 us of them in the kernel).
// ---------------------------------------------------------------------------
template <typename K, int C>
__global__ __launch_bounds__((LeafShape<typename std::make_unsigned<K>::type, C>::NT)) void k_small_sort(
    const K* __restrict__ src_k, const int32_t* __restrict__ src_r, uint32_t n, K* __restrict__ out_k,
    int32_t* __restrict__ out_r)
{
    using KW = typename std::make_unsigned<K>::type;
    using SH = LeafShape<KW, C>;
    constexpr int NT = SH::NT, KI = SH::KI, NW = SH::NW;
    __shared__ KW lds_key_raw[C];
    __shared__ __align__(16) uint16_t lds_idx_raw[C];
    __shared__ int32_t lds_rid[C];
    __shared__ uint32_t cnt[SH::CNT_WORDS];
    __shared__ uint32_t tmp[NW];
    __shared__ uint64_t tmp64[NW];
    const KeyPlain<KW, C> lds_key{lds_key_raw};
    const IdxPlain<KW, C> lds_idx{lds_idx_raw};
    const uint32_t w = threadIdx.x / 64, l = threadIdx.x & 63;
    K v[KI];
    int32_t rid[KI];
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = (w * KI + r) * 64 + l;
        v[r] = ld_clamp(src_k, q, n);
        rid[r] = ld_clamp(src_r, q, n);
    }
    uint64_t lo = ~0ull, hi = 0;  // clamped loads repeat a real row
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint64_t o = ord_of(v[r]);
        lo = o < lo ? o : lo;
        hi = o > hi ? o : hi;
    }
    block_minmax64<NT>(lo, hi, tmp64);
    const uint64_t span = hi - lo;
    const int bits = span ? 64 - (int)__clzll((long long)span) : 0;
    KW key[KI];
    uint16_t idx[KI];
    auto load_items = [&]() {
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const uint32_t q = (w * KI + r) * 64 + l;
            key[r] = q < n ? (KW)(ord_of(v[r]) - lo) : (KW)~(KW)0;
            idx[r] = (uint16_t)q;
        }
    };
    load_items();
#pragma unroll
    for (int r = 0; r < KI; r++) lds_rid[(w * KI + r) * 64 + l] = rid[r];
    block_sort<KW, NT, KI, SH::NBB>(key, idx, bits, n, lds_key, lds_idx, cnt, tmp, tmp64, load_items);
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t q = (w * KI + r) * 64 + l;
        if (q < n) {
            out_k[q] = key_of<K>(lo + (uint64_t)lds_key[q]);
            out_r[q] = lds_rid[lds_idx[q]];
        }
    }
}

hipError_t launch_small_sort(int key_bytes, const void* keys, const int32_t* rids, uint32_t n, void* out_k,
                             int32_t* out_r, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    if (n > (uint32_t)LEAF_CAP) return hipErrorInvalidValue;
#define TJ_SS(K, C)                                                                                              \
    hipLaunchKernelGGL((k_small_sort<K, C>), dim3(1), dim3(LeafShape<typename std::make_unsigned<K>::type, C>::NT), \
                       0, st, (const K*)keys, rids, n, (K*)out_k, out_r)
    if (key_bytes == 4) {
        if (n <= 1024) TJ_SS(int32_t, 1024);
        else if (n <= 4096) TJ_SS(int32_t, 4096);
        else TJ_SS(int32_t, LEAF_CAP);
    } else {
        if (n <= 1024) TJ_SS(int64_t, 1024);
        else if (n <= 4096) TJ_SS(int64_t, 4096);
        else TJ_SS(int64_t, LEAF_CAP);
    }
#undef TJ_SS
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// per-bucket join of one block: R's rows and S's rows of its co-partition. The
// rows of one key form a run; a run with a R rows and b S rows contributes a*b
// pairs, and R row i of the run owns the b consecutive output slots of its
// pairs, so the output is key-ascending, R-major, S in input order. k_leaf_join
// sorts the side of fewer rows and looks the other side's rows up in it;
// join_sorted sorts both together, stably, by key (R's rows at positions
// 0..rn-1, S's at rn..rn+sn-1), which makes every run
// [R rows in input order][S rows in input order].
//
// Count mode adds the block's pair count to *total. Materialise mode takes a
// ticket (so blocks handle buckets in key order), publishes its pair count,
// and finds its output offset by decoupled look-back over the published
// counts of the buckets before it; status[0] holds the offset carried in, and
// the last bucket stores the pairs so far to *total. (*total and *err are then
// pinned host memory, so that the call reads them when the stream is done.)
// Pairs at or beyond `capacity` are not written.
// ---------------------------------------------------------------------------
constexpr uint64_t ST_AGG = 1ull << 62, ST_INC = 2ull << 62, ST_VAL = (1ull << 62) - 1;
constexpr uint64_t LOOKBACK_SPIN_LIMIT = 1ull << 22;
constexpr uint32_t COOP_PAIRS = 16;  // R rows with more pairs are written by their whole wave

// A status word carries its whole message (flag and value in one 64-bit word)
// and no other data is published through it, so relaxed device-scope atomics
// suffice: release/acquire would make every block wait for its earlier
// memory operations and write back or invalidate its L2 (each XCD has its
// own) on the way.
__device__ __forceinline__ void status_store(uint64_t* p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t status_load(const uint64_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Exclusive prefix of bucket `slot - 1` (slot >= 1), computed by one whole
// wave: lane i reads status[hi - i] for a window of 64 predecessors. The window
// is summed from its newest entry down to the nearest inclusive prefix; if the
// window holds only aggregates it is summed whole and the walk moves 64 slots
// back. A window is re-read while any entry it needs is unpublished. Every
// predecessor already holds its ticket, so it is running or done and will
// publish; the spin is bounded all the same, and on expiry *err is set and 0
// returned. status[0] is always an inclusive prefix, so the walk ends.
__device__ uint64_t look_back(uint64_t* status, uint32_t slot, uint32_t* err)
{
    const uint32_t l = lane_id();
    uint64_t sum = 0, spins = 0;
    int64_t hi = (int64_t)slot - 1;
    while (true) {
        const int64_t j = hi - (int64_t)l;
        const uint64_t s = j >= 0 ? status_load(&status[j]) : 0;
        const uint64_t f = s & ~ST_VAL;
        const uint64_t inc = ballot(j >= 0 && f == ST_INC);
        const uint64_t pending = ballot(j >= 0 && f == 0);
        const int first = inc ? __ffsll((unsigned long long)inc) - 1 : 64;
        const uint64_t need = first >= 63 ? ~0ull : ((2ull << first) - 1);
        if (pending & need) {
            if (++spins > LOOKBACK_SPIN_LIMIT) {
                if (l == 0) *err = 1u;
                return 0;
            }
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        sum += wave_sum64(((need >> l) & 1ull) && j >= 0 ? (s & ST_VAL) : 0ull);
        if (first < 64) return sum;
        hi -= 64;
    }
}

// Rows of a run ranked by looking at all of them; larger runs are ranked by
// counters at a fixed cost, about that of looking at 30 rows.
constexpr uint32_t RUN_SCAN = 32;

// LDS of a join block: one pool, laid out by each of its two ways.
template <typename KW, bool MAT, int C> struct JoinLds {
    using SH = LeafShape<KW, C, true>;
    // (padded for the count; the materialising block keeps the plain layout:
    // the padding's address arithmetic costs it registers it does not have)
    using KA = typename std::conditional<MAT, LdsPad<KW, SH::KI, 0>, LdsPad<KW, SH::KI, 1>>::type;
    using IA = typename std::conditional<MAT, LdsPad<uint16_t, SH::KI, 0>, LdsPad<uint16_t, SH::KI, 2>>::type;
    // sorted way: keys, indices, digit counters, scan scratch, offset, flag
    static constexpr int KEYS = KA::size(C) * sizeof(KW), IDX = IA::size(C) * 2, CNT = SH::NW * LSTRIDE * 4;
    static constexpr int TMP64 = (KEYS + IDX + CNT + 15) / 16 * 16, TMP = TMP64 + SH::NW * 8, BASE = TMP + SH::NW * 4,
                         FLAG = BASE + 8, SORTED = FLAG + 16;
    // bins of the table's keys
    static constexpr int NBB = C == 1024 ? 10 : 12, BINS = 1 << NBB, HIST = (BINS * 2 + 2 + 15) / 16 * 16;
    // binned way, for tn rows of the table and pn probing ones: the table's row ids
    // (MAT), bins' ends, its keys in order and PAD largest ones, its keys in bins
    // (later its runs), its rows in bins (later the probing rows in runs and
    // RUN_SCAN more words, MAT). Grows with tn where tn + pn is given: halves need most.
    static constexpr uint32_t PAD = BIN_MAXC + 8;
    static constexpr uint32_t need(uint32_t tn, uint32_t pn)
    {
        const uint32_t k = sizeof(KW), ti = 2 * tn, pi = MAT ? 4 * pn + 4 * RUN_SCAN : 0u;
        return HIST + (tn + PAD) * k + tn * (k + (MAT ? 4u : 0u)) + (ti > pi ? ti : pi) + 64;
    }
    static constexpr int ALL = need(C / 2, C / 2);
    // 32-bit keys: half of a CU's 160 KiB with the block's other words, so that two blocks fit
    static constexpr int HALF = 81920 - 512;
    static constexpr int MOST = sizeof(KW) == 4 && C == LEAF_CAP ? HALF : ALL;
    static_assert(MOST >= ALL, "any two sides of one block fit");
    static constexpr int BYTES = ((MOST > SORTED ? MOST : SORTED) + 15) / 16 * 16;
};

// The argument `bits` of join_sorted, from a block of either key width (ANY) whose keys have 4 bytes.
constexpr int ANY_FOUR = 256;

template <typename K> struct JoinIn {
    const K *rk, *sk;
    const int32_t *rr, *sr;
};

// The join of one block by sorting R's and S's rows together (see above), for
// leaves that the binned way does not take. Not inlined: its registers would
// weigh on the other way's.
template <typename K, typename KW, bool MAT, bool SELF, int C, bool ANY>
static __device__ __noinline__ void join_sorted(__attribute__((address_space(3))) char* pool3, uint32_t rn, uint32_t n,
                                                uint64_t leaf_base, uint64_t out, int bits, bool reorder, uint32_t li,
                                                const K* rk_, const K* sk_, const int32_t* rr_, const int32_t* sr_,
                                                uint64_t* __restrict__ status,
                                                uint64_t* __restrict__ total, uint32_t* __restrict__ err,
                                                int32_t* out_r_, int32_t* out_s_,
                                                uint64_t capacity)
{
    using JL = JoinLds<KW, MAT, C>;
    using KA = typename JL::KA;
    using IA = typename JL::IA;
    constexpr int NT = JL::SH::NT, KI = JL::SH::KI;
    char* const pool = (char*)pool3;
    // (as arguments of a call they would be taken for any address space's)
    typedef __attribute__((address_space(1))) K GK;
    typedef __attribute__((address_space(1))) int32_t G32;
    const GK *const rk = (const GK*)rk_, *const sk = (const GK*)sk_;
    const G32 *const rr = (const G32*)rr_, *const sr = (const G32*)sr_;
    G32 *const out_r = (G32*)out_r_, *const out_s = (G32*)out_s_;
    const bool four = ANY && bits >= ANY_FOUR;
    if (ANY) bits &= ANY_FOUR - 1;
    KW* const lds_key_raw = (KW*)pool;
    uint16_t* const lds_idx_raw = (uint16_t*)(pool + JL::KEYS);
    const KA lds_key{lds_key_raw};
    const IA lds_idx{lds_idx_raw};
    uint32_t* const cnt = (uint32_t*)(pool + JL::KEYS + JL::IDX);
    uint32_t* const tmp = (uint32_t*)(pool + JL::TMP);
    uint64_t* const tmp64 = (uint64_t*)(pool + JL::TMP64);
    uint64_t& s_base = *(uint64_t*)(pool + JL::BASE);
    uint32_t& s_unordered = *(uint32_t*)(pool + JL::FLAG);
    const uint32_t w = threadIdx.x / 64, l = threadIdx.x & 63;
    lds_barrier();
    if (threadIdx.x == 0) s_unordered = 0;
    KW key[KI];
    uint16_t idx[KI];
    auto load_items = [&]() {
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const uint32_t q = (w * KI + r) * 64 + l;
            key[r] = (KW)~(KW)0;
            idx[r] = (uint16_t)q;
        }
        if (n > 0) {
#pragma unroll
            for (int r = 0; r < KI; r++) {
                const uint32_t q = (w * KI + r) * 64 + l;
                const uint32_t qc = q < n ? q : n - 1;  // every lane loads a real row
                uint64_t o;
                if (ANY && four) o = ord_of((int32_t)(qc < rn ? ((const G32*)rk)[qc] : ((const G32*)sk)[qc - rn]));
                else o = ord_of((K)(qc < rn ? rk[qc] : sk[qc - rn]));
                if (q < n) key[r] = (KW)(o - leaf_base);
            }
        }
    };
    // (LSD rather than block_bin_sort: a key here usually has several rows, one
    // of R and its S matches, which makes the bins too full for the exact
    // in-bin ranking to pay.) Ranked by atomics, then checked; sorted again
    // with ballot ranking if the order is not exact.
    load_items();
    block_lsd_sort<KW, NT, KI, true>(key, idx, bits, lds_key, lds_idx, cnt, tmp);
    if (!block_check_order<KW, NT, KI>(lds_key, lds_idx, n, &s_unordered) || reorder) {
        load_items();
        block_lsd_sort<KW, NT, KI, false>(key, idx, bits, lds_key, lds_idx, cnt, tmp);
    }

    // Run analysis on blocked positions p = tid*KI + i. A run is a maximal
    // stretch of equal keys: [rs, s0) holds its a R items, [s0, re) its b S
    // items. rs comes from a block-wide max-scan of run starts; s0 and re are
    // written, indexed by rs, by the run's last R item (or its first item when
    // the run has no R item) and by its last item.
    const uint32_t p0 = threadIdx.x * KI;
    KW kk[KI];
    uint32_t id[KI];
    lds_idx.blk_all(threadIdx.x, id);
#pragma unroll
    for (int i = 0; i < KI; i++) kk[i] = lds_key.blk(threadIdx.x, i);
    const KW kprev = p0 ? lds_key.blk(threadIdx.x - 1, KI - 1) : (KW)0;
    const KW knext = p0 + KI < C ? lds_key.blk(threadIdx.x + 1, 0) : (KW)0;
    const uint32_t inext = p0 + KI < C ? lds_idx.blk(threadIdx.x + 1, 0) : 0xffffu;
    uint32_t rs[KI];
    uint32_t run_start = 0;
#pragma unroll
    for (int i = 0; i < KI; i++) {
        const uint32_t p = p0 + i;
        const bool start = p == 0 || p >= n || kk[i] != (i ? kk[i - 1] : kprev);
        run_start = start ? p : run_start;
        rs[i] = run_start;
    }
    {
        const uint32_t carry = block_excl_max<NT>(run_start, tmp);  // barriers: keys all read
#pragma unroll
        for (int i = 0; i < KI; i++) rs[i] = max(rs[i], carry);
    }
    uint16_t* run_s0 = (uint16_t*)lds_key_raw;   // the key array is free from here on
    uint16_t* run_end = run_s0 + C;
#pragma unroll
    for (int i = 0; i < KI; i++) {
        const uint32_t p = p0 + i;
        if (p >= n) continue;
        const bool last = p == n - 1 || (i + 1 < KI ? kk[i + 1] : knext) != kk[i];
        const uint32_t idn = i + 1 < KI ? id[i + 1] : inext;
        const bool isr = id[i] < rn;
        if (last) run_end[rs[i]] = (uint16_t)(p + 1);
        if (isr && (last || idn >= rn)) run_s0[rs[i]] = (uint16_t)(p + 1);   // last R item
        if (!isr && p == rs[i]) run_s0[rs[i]] = (uint16_t)p;                  // run without R items
    }
    lds_barrier();
    // per item, packed: [is R:1][a:14][b:14], a = R items and b = S items of its
    // run (0 for padding); kv = position of the item inside the run's S part
    uint32_t abv[KI], kv[KI];
    uint32_t local = 0;
#pragma unroll
    for (int i = 0; i < KI; i++) {
        abv[i] = 0;
        kv[i] = 0;
        if (p0 + i < n) {
            const uint32_t s0 = run_s0[rs[i]], re = run_end[rs[i]];
            const uint32_t a = s0 - rs[i], b = re - s0;
            const bool isr = id[i] < rn;
            abv[i] = (isr ? 0x80000000u : 0u) | (a << 14) | b;
            kv[i] = p0 + i - s0;
            if (isr) local += b;  // an R item owns b pairs
        }
    }
    if (!MAT) {
        const uint64_t c = block_sum64<NT>((uint64_t)local, tmp64);
        if (SELF && threadIdx.x == 0) *total = c;
        if (!SELF && threadIdx.x == 0 && c) atomicAdd((unsigned long long*)total, (unsigned long long)c);
        return;
    }
    uint32_t ltot;
    uint32_t ex = block_excl_scan<NT>(local, tmp, &ltot);  // barriers: run tables all read
    if (SELF && threadIdx.x == 0) *total = ltot;
    if (!SELF && threadIdx.x == 0) status_store(&status[li + 1], ST_AGG | (uint64_t)ltot);
    // Row ids: one coalesced load of the block's rows (R then S) into the free
    // key array, then every item picks its own from LDS.
    int32_t* lds_w = (int32_t*)lds_key_raw;
    {
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const uint32_t q = threadIdx.x + r * NT;
            const uint32_t qc = q < n ? q : n - 1;
            const int32_t v = qc < rn ? rr[qc] : sr[qc - rn];
            if (q < n) lds_w[q] = v;
        }
    }
    if (!SELF && threadIdx.x < 64) {
        const uint64_t excl = look_back(status, li + 1, err);
        if (threadIdx.x == 0) {
            status_store(&status[li + 1], ST_INC | (excl + ltot));
            if (li == gridDim.x - 1) *total = excl + ltot;
            s_base = excl + out;
        }
    }
    lds_barrier();
    const uint64_t base = SELF ? 0 : s_base;
    // Pairs are written R item by R item: its b slots are consecutive, and so are
    // their S items (kv: minus the R item's distance to its run's S part). A lane
    // writes an item of few slots, a wave one of many, and these go round the
    // block's waves through LDS: the R items of one key sit with one wave. Both
    // columns leave in stretches. 2^21 x 2^21 rows of 21000 keys, 32-bit, 209
    // million pairs in 1.2 ms, from 3.6 with S items writing their slots b apart;
    // one block of 490 x 5089 rows of one key: 0.26 ms, from 3.1 with one wave at work.
    struct Shared { uint32_t e, sb; };  // first slot; first S position << 13 | slots
    static_assert(NT * 8 <= JL::IDX + JL::CNT && C <= 8192, "sorting is over: its memory is free");
    Shared* const shared = (Shared*)lds_idx_raw;
    bool many = false;
#pragma unroll
    for (int i = 0; i < KI; i++) many = many || ((abv[i] >> 31) && (abv[i] & 0x3fffu) > COOP_PAIRS);
    if (threadIdx.x == 0) s_unordered = 0;
    int32_t rid[KI];
#pragma unroll
    for (int i = 0; i < KI; i++) rid[i] = p0 + i < n ? lds_w[id[i]] : 0;
    lds_barrier();
    int32_t* const sid = lds_w;  // row ids by sorted position
#pragma unroll
    for (int i = 0; i < KI; i++)
        if (p0 + i < n) sid[p0 + i] = rid[i];
    if (many) s_unordered = 1;
    lds_barrier();
    const bool some_many = uniform(s_unordered) != 0;
#pragma unroll
    for (int i = 0; i < KI; i++) {
        const uint32_t b = (abv[i] >> 31) ? abv[i] & 0x3fffu : 0u;
        const uint32_t s0 = p0 + i - kv[i], e = ex;
        ex += b;
        if (b <= COOP_PAIRS) {
#pragma unroll 1
            for (uint32_t j = 0; j < b; j++) {
                const uint64_t o = base + e + j;
                if (o < capacity) {
                    out_r[o] = sid[p0 + i];
                    out_s[o] = sid[s0 + j];
                }
            }
        }
        if (!some_many) continue;
        shared[threadIdx.x] = Shared{e, b > COOP_PAIRS ? s0 << 13 | b : 0u};
        lds_barrier();
        const uint32_t from = w + (NT / 64) * l;
        const Shared it = shared[from];
        uint64_t m = ballot(it.sb != 0);
        while (m) {
            const int src = __ffsll((unsigned long long)m) - 1;
            m &= m - 1;
            const uint32_t sb = (uint32_t)__builtin_amdgcn_readlane((int)it.sb, src);
            const uint32_t cb = sb & 0x1fffu, cs = sb >> 13;
            const uint64_t ce = base + (uint32_t)__builtin_amdgcn_readlane((int)it.e, src);
            const int32_t cr = sid[(uint32_t)__builtin_amdgcn_readlane((int)from, src) * KI + i];
#pragma unroll 1
            for (uint32_t j = l; j < cb; j += 64) {
                if (ce + j < capacity) {
                    out_r[ce + j] = cr;
                    out_s[ce + j] = sid[cs + j];
                }
            }
        }
        lds_barrier();
    }
}

// Pairs a probing row, on average over the block, beyond which its runs are
// written as they come (write_runs) instead of in stretches staged in LDS, where
// each stretch looks at all pairs of its rows. Joins of 2^18 rows with `a` a key
// and up to 2^22 with `b`, in stretches and as they come: a = b = 6, 108 and 122
// us; a = b = 8, 127 and 126; a = 8, b = 128, 440 and 367; a = b = 16, 220 and
// 142; a = b = 47, 820 and 174.
constexpr uint32_t DIRECT_PAIRS = 6;

// The pairs of a join block, straight from the row ids in run order: each wave
// takes an equal share of the slots and writes 64 at a time. run[p] (at the
// first table position of a run): slots << 13 | probing rows before it; `all`
// the same for the whole block. trid, prid: the table's and the probing rows'
// ids in run order; the probing rows are the outer loop of a run if `swap`.
template <int NW>
__device__ __forceinline__ void write_runs(const uint32_t* run, uint32_t all, uint32_t tn, uint32_t slots, bool swap,
                                           uint64_t base, uint64_t capacity, const int32_t* trid, const int32_t* prid,
                                           int32_t* __restrict__ out_t, int32_t* __restrict__ out_p)
{
    const uint32_t l = threadIdx.x & 63, w = uniform(threadIdx.x / 64);
    const uint32_t share = (slots / NW + 64) & ~63u;
    const uint32_t end = min((w + 1) * share, slots);
    uint32_t x = w * share;
    // the run of slot x: the last position whose runs before it end at or before x
    // (a run's other positions, and runs without probing rows, end where they start)
    auto find = [&]() {
        uint32_t lo = 0, hi = tn;
        while (hi - lo > 1) {
            const uint32_t m = (lo + hi) / 2;
            if (uniform(run[m]) >> 13 <= x) lo = m;
            else hi = m;
        }
        return lo;
    };
    if (x >= end) return;
    uint32_t p = find();
    while (x < end) {
        const uint32_t here = uniform(run[p]), next = p + 1 < tn ? uniform(run[p + 1]) : all;
        const uint32_t e0 = here >> 13, e1 = next >> 13;
        if (e1 <= x) {  // (behind the last run: table rows without a match)
            p = find();
            continue;
        }
        const uint32_t g = here & 0x1fffu, b = (next & 0x1fffu) - g, a = (e1 - e0) / b;
        const uint32_t m = swap ? a : b, dq = 64 / m, dr = 64 % m;
        const uint32_t stop = min(e1, end);
        uint32_t y = x + l, outer = (y - e0) / m, inner = y - e0 - outer * m;
        for (; y < stop; y += 64) {
            const uint64_t o = base + y;
            if (o < capacity) {
                out_t[o] = trid[p + (swap ? inner : outer)];
                out_p[o] = prid[g + (swap ? outer : inner)];
            }
            outer += dq;
            inner += dr;
            if (inner >= m) {
                inner -= m;
                outer++;
            }
        }
        x = stop;
        p += a;
    }
}

// The join of one block. The side of fewer rows is the table: its keys are
// binned by their top bits (a quarter to one row a bin where keys are even),
// placed, and ranked exactly inside their bin, so that it is in (key, position)
// order; every row of the other side, which probes, then finds its table rows by
// looking through one bin. Probing rows of one key (a run of the table) are
// collected run by run and ranked by position within the run, so nothing depends
// on the order of atomics. Pairs: R item i of a run and S item k have slot
// E + i * b + k, with E the pairs before the run and b its S items; the probing
// rows write both columns into LDS, from where they leave coalesced (blocks of
// many pairs a row: see write_runs).
// What bounds the block is its LDS work and its waits, not memory. Only the
// table's rows are sorted, which are the fewer, where sorting both sides together
// took three to five digit passes over all rows and a check of the order; and with
// 32-bit keys two blocks of 64 VGPRs and half of the LDS share a CU, so that one
// works while the other waits. 2^27 x 2^29 rows, 32-bit keys: 4.2 ms (2.1 TB/s)
// from 9.0; counting 2^28 of Zipf keys: 0.92 ms from 3.9. With the plain sides'
// roles (R always the table) blocks of many R rows fell to the sorted way: 2^24 x
// 2^18 rows, 1.59 ms for the whole join and now 0.82.
// Blocks whose table rows crowd one bin (over BIN_MAXC of them, so both sides
// have many rows a key there) are sorted (join_sorted).
// SELF (a whole input that fits one block): the leaf is `self`, whose key
// range the block finds itself; its pairs start at 0 and their number is
// stored to *total (in either mode). One launch then serves the whole call.
// ANY (K of 8 bytes): leaves of either key width, which each leaf tells. A level
// whose segments narrow their keys only in part leaves widths that alternate in
// key order, and a launch (and a wait) for every stretch of one width: 2^24 x 2^26
// rows of exponential keys, 12.0 ms in 258 launches and 4.7 in one; 2^26 x 2^28 of
// normal ones took 350 ms in 3663.
template <typename K, typename KW, bool MAT, bool SELF = false, int C = LEAF_CAP, bool ANY = false>
__global__ __launch_bounds__((JoinLds<KW, MAT, C>::SH::NT))
__attribute__((amdgpu_waves_per_eu(sizeof(KW) == 4 && !SELF ? 8 : 4))) void k_leaf_join(const LeafDesc* __restrict__ leaves,
                                                            BufSet bufs, uint64_t* __restrict__ status,
                                                            uint32_t* __restrict__ ticket,
                                                            uint64_t* __restrict__ total,
                                                            uint32_t* __restrict__ err,
                                                            int32_t* __restrict__ out_r,
                                                            int32_t* __restrict__ out_s,
                                                            uint64_t capacity, LeafDesc self)
{
    using JL = JoinLds<KW, MAT, C>;
    constexpr int NT = JL::SH::NT, KI = JL::SH::KI, NW = JL::SH::NW;
    __shared__ __align__(16) char pool[JL::BYTES];
    __shared__ uint32_t tmp[NW];
    __shared__ uint64_t tmp64[NW];
    __shared__ uint32_t s_leaf, s_all;
    __shared__ uint32_t s_spare[64];  // a counter per lane for rows that take no part
    __shared__ uint64_t s_base;

    uint32_t li = blockIdx.x;
    if (MAT && !SELF) {
        if (threadIdx.x == 0) s_leaf = atomicAdd(ticket, 1u);
        lds_barrier();
        li = s_leaf;
    }
    LeafDesc L;
    if constexpr (SELF) L = self;
    else L = leaves[li];
    JoinIn<K> in;
    bool four = false;
    if constexpr (ANY) four = uniform((uint32_t)L.kb) == 4;
    in.rk = (const K*)bufs.key[L.buf][0] + L.kr0;
    in.sk = (const K*)bufs.key[L.buf][1] + L.ks0;
    if (ANY && four) {
        in.rk = (const K*)((const int32_t*)bufs.key[L.buf][0] + L.kr0);
        in.sk = (const K*)((const int32_t*)bufs.key[L.buf][1] + L.ks0);
    }
    in.rr = MAT ? bufs.rid[L.buf][0] + L.r0 : nullptr;
    in.sr = MAT ? bufs.rid[L.buf][1] + L.s0 : nullptr;
    // the table: the side of fewer rows (R, if alike)
    const bool swap = L.rn > L.sn;
    const uint32_t tn = swap ? L.sn : L.rn, pn = swap ? L.rn : L.sn;
    // (every load below is made without a branch, so that all are in flight at
    // once; an empty side reads the other's first row, an empty leaf its record)
    const K* const pk = !pn ? (const K*)leaves : swap ? in.rk : in.sk;
    const K* const tk = !tn ? pk : swap ? in.sk : in.rk;
    const int32_t* const pr = !pn ? (const int32_t*)leaves : swap ? in.rr : in.sr;
    const int32_t* const tr = !tn ? pr : swap ? in.sr : in.rr;
    const uint32_t w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.x / 64) * (KI * 64);
    uint32_t l = threadIdx.x & 63, t = threadIdx.x;
    // row r of the thread, formed anew in each step (kept over the steps, the
    // rows' numbers and what is compared with them take registers twice over)
    auto row = [&](int r) { return w0 + r * 64 + l; };
    auto fresh = [&]() { asm volatile("" : "+v"(l), "+v"(t)); };
    // packed words stay packed (their parts would be kept beside them: 64 VGPRs
    // are all that two blocks a CU leave, and spills made the block 1.7 times slower)
    auto packed = [](uint32_t(&w)[KI]) {
#pragma unroll
        for (int r = 0; r < KI; r++) asm volatile("" : "+v"(w[r]));
    };

    // The probing rows stay in registers (row r of the thread: row(r)); the
    // table's are loaded with them (row t + i * NT).
    constexpr int TI = C / 2 / NT;
    const uint32_t tlast = tn ? tn - 1 : 0u, plast = pn ? pn - 1 : 0u;
    K tv[TI];
    KW key[KI];
    {
        K v[KI];
        if (ANY && four) {  // as keys of K with the same ordinals
#pragma unroll
            for (int i = 0; i < TI; i++) tv[i] = key_of<K>(ord_of(ld_now((const int32_t*)tk, min(t + i * NT, tlast))));
#pragma unroll
            for (int r = 0; r < KI; r++) v[r] = key_of<K>(ord_of(ld_now((const int32_t*)pk, min(row(r), plast))));
        } else {
#pragma unroll
            for (int i = 0; i < TI; i++) tv[i] = ld_now(tk, min(t + i * NT, tlast));
#pragma unroll
            for (int r = 0; r < KI; r++) v[r] = ld_now(pk, min(row(r), plast));
        }
        if constexpr (SELF) {
            uint64_t lo = ~0ull, hi = 0;
#pragma unroll
            for (int r = 0; r < KI; r++) {
                const uint64_t o = ord_of(v[r]);
                lo = o < lo ? o : lo;
                hi = o > hi ? o : hi;
            }
#pragma unroll
            for (int i = 0; i < TI; i++) {
                const uint64_t o = ord_of(tv[i]);
                lo = o < lo ? o : lo;
                hi = o > hi ? o : hi;
            }
            block_minmax64<NT>(lo, hi, tmp64);
            L.base = lo;
            L.bits = (uint16_t)(hi > lo ? 64 - (int)__clzll((long long)(hi - lo)) : 0);
        }
#pragma unroll
        for (int r = 0; r < KI; r++) key[r] = (KW)(ord_of(v[r]) - L.base);
    }
    const uint32_t tn4 = (tn + 3) & ~3u;
    int32_t* const trid = (int32_t*)pool;                            // the table's places by row, then its row ids in key order
    uint16_t* const bend = (uint16_t*)(pool + (MAT ? tn4 * 4 : 0));  // end of each bin in the table's order
    KW* const tkey = (KW*)((char*)bend + JL::HIST);                  // the table's keys in order
    KW* const bkey = tkey + tn4 + JL::PAD;                           // its keys in their bins, in any order
    uint16_t* const bidx = (uint16_t*)(bkey + tn4);                  // their rows
    const int sh = (int)L.bits > JL::NBB ? (int)L.bits - JL::NBB : 0;
    auto bin_of = [&](KW k) { return (uint32_t)(k >> sh) & (JL::BINS - 1u); };
    auto bin_add = [&](uint32_t b) { return atomicAdd((uint32_t*)bend + b / 2, 1u << (b & 1) * 16) >> (b & 1) * 16 & 0xffffu; };

    bool fast = !(L.flags & LEAF_FORCE_REORDER);
    if (fast) {
        for (uint32_t i = t; i < JL::BINS / 2; i += NT) ((uint32_t*)bend)[i] = 0;
        lds_barrier();
#pragma unroll
        for (int i = 0; i < TI; i++) {
            if (i * NT >= (int)tn) break;
            const uint32_t q = t + i * NT;
            const KW k = (KW)(ord_of(tv[i]) - L.base);
            if (q < tn) {
                tkey[q] = k;  // (in row order so far)
                bin_add(bin_of(k));
            }
        }
        lds_barrier();
        constexpr int BPT = JL::BINS / NT;
        uint32_t c[BPT], sum = 0, mx = 0;
#pragma unroll
        for (int i = 0; i < BPT; i += 2) {
            const uint32_t x = ((const uint32_t*)bend)[(t * BPT + i) / 2];
            c[i] = x & 0xffffu;
            c[i + 1] = x >> 16;
        }
#pragma unroll
        for (int i = 0; i < BPT; i++) {
            sum += c[i];
            mx = c[i] > mx ? c[i] : mx;
        }
        fast = block_max<NT>(mx, tmp) <= BIN_MAXC;
        if (fast) {
            uint32_t all;
            uint32_t ex = block_excl_scan<NT>(sum, tmp, &all);
#pragma unroll
            for (int i = 0; i < BPT; i += 2) {
                ((uint32_t*)bend)[(t * BPT + i) / 2] = ex | (ex + c[i]) << 16;
                ex += c[i] + c[i + 1];
            }
        }
    }
    if (!fast) {
        join_sorted<K, KW, MAT, SELF, C, ANY>((__attribute__((address_space(3))) char*)pool, L.rn, L.rn + L.sn, L.base, L.out,
                                         (int)L.bits + (four ? ANY_FOUR : 0), L.flags & LEAF_FORCE_REORDER, li, in.rk, in.sk, in.rr, in.sr,
                                         status, total, err, out_r, out_s, capacity);
        return;
    }
    lds_barrier();
    for (uint32_t q = t; q < tn; q += NT) {
        const KW k = tkey[q];
        const uint32_t p = bin_add(bin_of(k));  // bend[b] moves from the bin's start to its end
        bkey[p] = k;
        bidx[p] = (uint16_t)q;
    }
    lds_barrier();
    auto bin_start = [&](uint32_t b) { return b ? (uint32_t)bend[b - 1] : 0u; };
    for (uint32_t p = t; p < tn; p += NT) {
        const KW k = bkey[p];
        const uint32_t q = bidx[p], b = bin_of(k), s0 = bin_start(b), e0 = bend[b];
        uint32_t at = s0;
        for (uint32_t j = s0; j < e0; j++) {
            const KW kj = bkey[j];
            at += kj < k || (kj == k && bidx[j] < q) ? 1u : 0u;
        }
        tkey[at] = k;
        if constexpr (MAT) trid[q] = (int32_t)at;
    }
    if (t < JL::PAD) tkey[tn + t] = (KW)~(KW)0;
    lds_barrier();
    // the table's row ids, on their way during the search
    int32_t tid[MAT ? TI : 1] = {};
    uint32_t tat[MAT ? TI : 1] = {};
    if constexpr (MAT) {
#pragma unroll
        for (int i = 0; i < TI; i++) {
            tat[i] = (uint32_t)trid[min(t + i * NT, tlast)];
            tid[i] = ld_now(tr, min(t + i * NT, tlast));
        }
    }
    // Every probing row looks through the table's keys from its bin's start on,
    // all rows of the thread in step: keys smaller than its own are counted (they
    // end where the bin does at the latest), and equal ones.
    fresh();
    uint32_t info[KI], seen[KI], cbmax = 0;
#pragma unroll
    for (int r = 0; r < KI; r++) {
        const uint32_t b = bin_of(key[r]), s0 = bin_start(b), cb = bend[b] - s0;
        info[r] = s0;
        seen[r] = 0;  // smaller | same << 8
        cbmax = cb > cbmax ? cb : cbmax;
    }
#pragma unroll 1
    for (uint32_t j = 0; j < cbmax; j += 2) {
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const KW* const at = tkey + info[r] + j;
            const KW k0 = at[0], k1 = at[1];
            seen[r] += (k0 < key[r] ? 1u : 0u) + (k1 < key[r] ? 1u : 0u);
            seen[r] += (k0 == key[r] ? 0x100u : 0u) + (k1 == key[r] ? 0x100u : 0u);
        }
    }
    if ((int)L.bits == (int)sizeof(KW) * 8) {
        // the largest key of all also met the padding
        const uint32_t it = (cbmax + 1) / 2 * 2;
#pragma unroll
        for (int r = 0; r < KI; r++)
            if (key[r] == (KW)~(KW)0 && info[r] + it > tn) seen[r] -= (info[r] + it - tn) << 8;
    }
    fresh();
#pragma unroll
    for (int r = 0; r < KI; r++)  // first table position of the row's run, table rows there (0: no match)
        info[r] = (info[r] + (seen[r] & 0xffu)) | (row(r) < pn ? seen[r] >> 8 << 13 : 0u);
    packed(info);
    if constexpr (!MAT) {
        uint32_t local = 0;
#pragma unroll
        for (int r = 0; r < KI; r++) local += info[r] >> 13;
        const uint64_t c = block_sum64<NT>((uint64_t)local, tmp64);
        if (SELF && t == 0) *total = c;
        if (!SELF && t == 0 && c) atomicAdd((unsigned long long*)total, (unsigned long long)c);
        return;
    } else {
        // run[p]: probing rows found so far | table rows << 16 at a run's first position, 0 at its others
        uint32_t* const run = (uint32_t*)bkey;
        uint32_t* const prow = (uint32_t*)(bkey + tn4);  // run << 13 | probing row, by run
        for (uint32_t p = t; p < tn; p += NT) {
            const KW k = tkey[p];
            uint32_t a = 0;
            if (p == 0 || tkey[p - 1] != k)
                do a++; while (p + a < tn && tkey[p + a] == k);
            run[p] = a << 16;
        }
        lds_barrier();
#pragma unroll
        for (int i = 0; i < TI; i++)
            if (i * NT < (int)tn && t + i * NT < tn) trid[tat[i]] = tid[i];
        fresh();
        uint32_t at[KI];
#pragma unroll
        for (int r = 0; r < KI; r++)
            at[r] = atomicAdd(info[r] >> 13 ? &run[info[r] & 0x1fffu] : &s_spare[l], 1u) & 0xffffu;
        packed(info);
        lds_barrier();
        // exclusive prefix over table positions of pairs << 13 | probing rows (at
        // most 48 * 8191 pairs: 19 bits)
        uint32_t ltot, maxb = 0;
        {
            const uint32_t ppt = (tn + NT - 1) / NT, p0 = t * ppt;
            uint32_t sum = 0;
            for (uint32_t i = 0; i < ppt; i++) {
                const uint32_t x = p0 + i < tn ? run[p0 + i] : 0u, b = x & 0xffffu;
                sum += ((x >> 16) * b << 13) + b;
                maxb = b > maxb ? b : maxb;
            }
            uint32_t all;
            uint32_t ex = block_excl_scan<NT>(sum, tmp, &all);
            for (uint32_t i = 0; i < ppt && p0 + i < tn; i++) {
                const uint32_t x = run[p0 + i], b = x & 0xffffu;
                run[p0 + i] = ex;
                ex += ((x >> 16) * b << 13) + b;
            }
            ltot = all >> 13;
            maxb = block_max<NT>(maxb, tmp);
            // (the word after the last position: read for the last run's size)
            if (t == 0) s_all = all;
            // a row looks past its run's end: the words after the last run's
            if (t < RUN_SCAN) prow[(all & 0x1fffu) + t] = ~0u;
        }
        if (SELF && t == 0) *total = ltot;
        if (!SELF && t == 0) status_store(&status[li + 1], ST_AGG | (uint64_t)ltot);
        lds_barrier();
        // the run's probing rows together, in any order
        fresh();
        uint32_t bmax = 0;
#pragma unroll
        for (int r = 0; r < KI; r++) {
            const uint32_t rs = info[r] & 0x1fffu;
            const bool m = info[r] >> 13;
            const uint32_t x = run[m ? rs : 0u], y = *(m && rs + 1 < tn ? &run[rs + 1] : &s_all);
            const uint32_t g = x & 0x1fffu, b = m ? (y & 0x1fffu) - g : 0u;
            if (m) prow[g + at[r]] = rs << 13 | row(r);
            at[r] = g | b << 13;  // the run's first place, its probing rows
            bmax = b <= RUN_SCAN && b > bmax ? b : bmax;
        }
        packed(info);
        packed(at);
        lds_barrier();
        int32_t rid[KI];
#pragma unroll
        for (int r = 0; r < KI; r++) rid[r] = ld_now(pr, min(row(r), plast));
        // (the row ids are loaded during the ranking; wave 0 waits for the look-back's answer while the others rank)
        if (!SELF && t < 64) {
            const uint64_t excl = look_back(status, li + 1, err);
            if (t == 0) {
                status_store(&status[li + 1], ST_INC | (excl + ltot));
                if (li == gridDim.x - 1) *total = excl + ltot;
                s_base = excl + L.out;
            }
        }
        // a row's place in its run: the run's rows before its own (words of later
        // runs are larger)
        uint32_t rank[KI];
#pragma unroll
        for (int r = 0; r < KI; r++) rank[r] = 0;
#pragma unroll 1
        for (uint32_t j = 0; j < bmax; j += 2) {
            fresh();
#pragma unroll
            for (int r = 0; r < KI; r++) {
                const uint32_t* const x = prow + (at[r] & 0x1fffu) + j;
                const uint32_t mine = (info[r] & 0x1fffu) << 13 | row(r);
                rank[r] += (x[0] < mine ? 1u : 0u) + (x[1] < mine ? 1u : 0u);
            }
        }
        if (maxb > RUN_SCAN) {
            // Runs of more rows: a counter per run and wave, numbered by the run's
            // first place (runs of over RUN_SCAN rows start in different stretches
            // of RUN_SCAN places); a row comes after its run's rows of earlier waves,
            // of the wave's earlier rows and of earlier lanes.
            constexpr uint32_t NRUN = C / RUN_SCAN;
            constexpr int RBITS = 31 - __builtin_clz(NRUN);
            static_assert(NRUN == 1u << RBITS && NRUN * NW * 2 <= JL::HIST, "the counters fit the bins' place");
            static_assert(NRUN <= NT, "a run a thread");
            uint16_t* const cnt = bend;
            const uint32_t w = w0 / (KI * 64);
            for (uint32_t i = t; i < NRUN * NW / 2; i += NT) ((uint32_t*)cnt)[i] = 0;
            lds_barrier();
            fresh();
#pragma unroll
            for (int r = 0; r < KI; r++) {
                const bool big = at[r] >> 13 > RUN_SCAN;
                const uint32_t id = (at[r] & 0x1fffu) / RUN_SCAN;
                uint64_t same = ballot(big);
#pragma unroll
                for (int i = 0; i < RBITS; i++) {
                    const uint64_t on = ballot(id >> i & 1u);
                    same &= (id >> i & 1u) ? on : ~on;
                }
                if (big) {
                    const uint32_t c = cnt[id * NW + w];
                    rank[r] = c + (uint32_t)__popcll(same & ((1ull << l) - 1));
                    if ((same & ((1ull << l) - 1)) == 0) cnt[id * NW + w] = (uint16_t)(c + (uint32_t)__popcll(same));
                }
            }
            lds_barrier();
            if (t < NRUN) {
                uint32_t sum = 0;
#pragma unroll 1
                for (int i = 0; i < NW; i++) {
                    const uint32_t c = cnt[t * NW + i];
                    cnt[t * NW + i] = (uint16_t)sum;
                    sum += c;
                }
            }
            lds_barrier();
#pragma unroll
            for (int r = 0; r < KI; r++)
                if (at[r] >> 13 > RUN_SCAN) rank[r] += cnt[(at[r] & 0x1fffu) / RUN_SCAN * NW + w];
        }
        fresh();
        int32_t* const out_t = swap ? out_s : out_r;
        int32_t* const out_p = swap ? out_r : out_s;
        // many pairs a row: their runs are written as they come, from the row ids in order
        const bool direct = uniform(ltot) > DIRECT_PAIRS * pn;
        if (direct) {
#pragma unroll
            for (int r = 0; r < KI; r++) at[r] = (at[r] & 0x1fffu) + rank[r];  // the row's place
        } else {
#pragma unroll
            for (int r = 0; r < KI; r++)  // first slot, stride
                at[r] = ((run[info[r] >> 13 ? info[r] & 0x1fffu : 0u] >> 13) + rank[r] * (swap ? info[r] >> 13 : 1u)) |
                        (swap ? 1u : at[r] >> 13) << 19;
        }
        lds_barrier();
        if (direct) {
            int32_t* const prid = (int32_t*)prow;
#pragma unroll
            for (int r = 0; r < KI; r++)
                if (info[r] >> 13) prid[at[r]] = rid[r];
            lds_barrier();
            write_runs<NW>(run, uniform(s_all), tn, uniform(ltot), swap, SELF ? 0 : s_base, capacity, trid, prid, out_t, out_p);
            return;
        }
        const uint64_t base = SELF ? 0 : s_base;
        // all but the table's row ids is free: a stretch of both output columns at a time
        const uint32_t slots = (JL::BYTES - tn4 * 4) / 8;
        int32_t* const col_t = (int32_t*)(pool + tn4 * 4);
        int32_t* const col_p = col_t + slots;
        for (uint32_t c0 = 0; c0 < ltot; c0 += slots) {
            const uint32_t cn = ltot - c0 < slots ? ltot - c0 : slots;
#pragma unroll
            for (int r = 0; r < KI; r++) {
                asm volatile("" : "+v"(info[r]), "+v"(at[r]));  // (unpacked here, not kept unpacked over the loop)
                const uint32_t a = info[r] >> 13, rs = info[r] & 0x1fffu, b = at[r] >> 19;
                uint32_t x = (at[r] & 0x7ffffu) - c0;
                if (a && x < cn) {
                    col_t[x] = trid[rs];
                    col_p[x] = rid[r];
                }
                if (ballot(a > 1)) {
#pragma unroll 1
                    for (uint32_t i = 1; i < a; i++) {
                        x += b;
                        if (x < cn) {
                            col_t[x] = trid[rs + i];
                            col_p[x] = rid[r];
                        }
                    }
                }
            }
            lds_barrier();
            for (uint32_t x = t; x < cn; x += NT) {
                const uint64_t o = base + c0 + x;
                if (o < capacity) {
                    out_t[o] = col_t[x];
                    out_p[o] = col_p[x];
                }
            }
            lds_barrier();
        }
    }
}

hipError_t launch_leaf_join(int key_bytes, bool wide, bool materialize, const LeafDesc* leaves,
                            uint32_t n, BufSet bufs, uint64_t* status, uint32_t* ticket,
                            uint64_t* total, uint32_t* err, int32_t* out_r, int32_t* out_s,
                            uint64_t capacity, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    const dim3 grid(n), block(LeafShape<uint32_t, LEAF_CAP, true>::NT);
#define TJ_LJ(K, KW, M)                                                                              \
    hipLaunchKernelGGL((k_leaf_join<K, KW, M>), grid, block, 0, st, leaves, bufs, status, ticket,    \
                       total, err, out_r, out_s, capacity, LeafDesc{})
    if (key_bytes == 0) {
        if (!materialize) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_leaf_join<int64_t, uint64_t, true, false, LEAF_CAP, true>), grid, block, 0, st, leaves, bufs,
                           status, ticket, total, err, out_r, out_s, capacity, LeafDesc{});
    } else if (key_bytes == 4) {
        if (wide) { if (materialize) TJ_LJ(int32_t, uint64_t, true); else TJ_LJ(int32_t, uint64_t, false); }
        else      { if (materialize) TJ_LJ(int32_t, uint32_t, true); else TJ_LJ(int32_t, uint32_t, false); }
    } else {
        if (wide) { if (materialize) TJ_LJ(int64_t, uint64_t, true); else TJ_LJ(int64_t, uint64_t, false); }
        else      { if (materialize) TJ_LJ(int64_t, uint32_t, true); else TJ_LJ(int64_t, uint32_t, false); }
    }
#undef TJ_LJ
    return hipGetLastError();
}

hipError_t launch_small_join(int key_bytes, bool materialize, uint32_t rn, uint32_t sn, uint16_t flags, BufSet bufs,
                             uint64_t* total, int32_t* out_r, int32_t* out_s, uint64_t capacity, hipStream_t st)
{
    const uint32_t n = rn + sn;
    if (n == 0 || rn > (uint32_t)LEAF_CAP || n > (uint32_t)LEAF_CAP) return hipErrorInvalidValue;
    LeafDesc self{};
    self.rn = rn;
    self.sn = sn;
    self.buf = BUF_IN;
    self.flags = flags;
#define TJ_SJ(K, M, C)                                                                                              \
    hipLaunchKernelGGL((k_leaf_join<K, typename std::make_unsigned<K>::type, M, true, C>), dim3(1),                 \
                       dim3(LeafShape<typename std::make_unsigned<K>::type, C, true>::NT), 0, st, nullptr, bufs, nullptr, \
                       nullptr, total, nullptr, out_r, out_s, capacity, self)
#define TJ_SJC(K, M)                     \
    do {                                 \
        if (n <= 1024) TJ_SJ(K, M, 1024); \
        else if (n <= 4096) TJ_SJ(K, M, 4096); \
        else TJ_SJ(K, M, LEAF_CAP);      \
    } while (0)
    if (key_bytes == 4) {
        if (materialize) TJ_SJC(int32_t, true); else TJ_SJC(int32_t, false);
    } else {
        if (materialize) TJ_SJC(int64_t, true); else TJ_SJC(int64_t, false);
    }
#undef TJ_SJC
#undef TJ_SJ
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// single-key buckets of the join: pair t of a unit with a R rows and b S rows
// is (R row t / b, S row t mod b); consecutive t are written by consecutive
// threads (coalesced). Units are flattened into one sequence of pairs and
// each block takes a fixed stretch of it. A unit's output offset is the
// inclusive pair prefix of the per-bucket joins before it (status, after the
// materialising leaf launch) plus the pairs of earlier single-key units.
// ---------------------------------------------------------------------------
constexpr int CROSS_THREADS = 256;
constexpr uint64_t CROSS_PER_BLOCK = 256 * 64;

// Pairs (rows of a copy) of a block: as many as leave every CU eight blocks, in
// whole steps of a block's loads, up to CROSS_PER_BLOCK (more blocks would only
// repeat the search for their first unit).
inline uint32_t cross_rows(uint64_t total, uint64_t step)
{
    const uint64_t even = (total / (256 * 8) + step - 1) / step * step;
    return (uint32_t)std::min(std::max(even, step), CROSS_PER_BLOCK);
}

__device__ __forceinline__ uint32_t find_unit(const uint64_t* pfx_base, size_t stride_words,
                                              uint32_t n, uint64_t t)
{
    // last unit u with pfx(u) <= t
    uint32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const uint32_t m = (lo + hi) >> 1;
        if (pfx_base[(size_t)m * stride_words] <= t) lo = m; else hi = m;
    }
    return lo;
}

__global__ __launch_bounds__(CROSS_THREADS) void k_cross(const CrossDesc* __restrict__ units,
                                                         uint32_t n, uint64_t total, uint32_t per, BufSet bufs,
                                                         const uint64_t* __restrict__ status,
                                                         int32_t* __restrict__ out_r,
                                                         int32_t* __restrict__ out_s,
                                                         uint64_t capacity)
{
    const uint64_t t0 = blockIdx.x * (uint64_t)per;
    uint64_t t1 = t0 + per;
    if (t1 > total) t1 = total;
    const size_t stride = sizeof(CrossDesc) / 8;
    const uint64_t* pfx = &units[0].pfx;
    uint64_t t = t0 + threadIdx.x;
    if (t >= t1) return;
    uint32_t u = find_unit(pfx, stride, n, t);
    CrossDesc U;
    uint64_t base = 0, end = 0, i = 0, j = 0;
    uint32_t qi = 0, qj = 0;  // a step of CROSS_THREADS pairs moves (i, j) by (qi, qj), then carries
    // pair loc = t - pfx of the unit is (R row i, S row j) with loc = i*b + j;
    // only a thread's first pair of a unit divides, later pairs step
    auto enter = [&]() {
        U = units[u];
        base = U.out + (status[U.leaf_before] & ST_VAL);
        end = U.pfx + U.a * U.b;
        const uint64_t loc = t - U.pfx;
        i = (uint64_t)((double)loc / (double)U.b);
        while (i * U.b > loc) i--;
        while ((i + 1) * U.b <= loc) i++;
        j = loc - i * U.b;
        qi = U.b > CROSS_THREADS ? 0u : (uint32_t)(CROSS_THREADS / U.b);
        qj = (uint32_t)(CROSS_THREADS - (uint64_t)qi * U.b);
    };
    auto step = [&](uint64_t& si, uint64_t& sj) {
        si += qi;
        sj += qj;
        if (sj >= U.b) {
            sj -= U.b;
            si++;
        }
    };
    constexpr int UNR = 4;  // pairs per thread whose row-id loads are issued together
    enter();
    while (t < t1) {
        if (t >= end) {
            do ++u; while (t >= units[u].pfx + units[u].a * units[u].b);
            enter();
        }
        const int32_t* __restrict__ rr = bufs.rid[U.buf][0] + U.r0;
        const int32_t* __restrict__ sr = bufs.rid[U.buf][1] + U.s0;
        const uint64_t last = t + (UNR - 1) * (uint64_t)CROSS_THREADS;
        if (last < end && last < t1) {
            uint64_t ii[UNR], jj[UNR];
            ii[0] = i;
            jj[0] = j;
#pragma unroll
            for (int k = 1; k < UNR; k++) {
                ii[k] = ii[k - 1];
                jj[k] = jj[k - 1];
                step(ii[k], jj[k]);
            }
            int32_t vr[UNR], vs[UNR];
#pragma unroll
            for (int k = 0; k < UNR; k++) {
                vr[k] = rr[ii[k]];
                vs[k] = sr[jj[k]];
            }
#pragma unroll
            for (int k = 0; k < UNR; k++) {
                const uint64_t o = base + (t + k * (uint64_t)CROSS_THREADS - U.pfx);
                if (o < capacity) {
                    out_r[o] = vr[k];
                    out_s[o] = vs[k];
                }
            }
            i = ii[UNR - 1];
            j = jj[UNR - 1];
            step(i, j);
            t += UNR * (uint64_t)CROSS_THREADS;
        } else {
            const uint64_t o = base + (t - U.pfx);
            if (o < capacity) {
                out_r[o] = rr[i];
                out_s[o] = sr[j];
            }
            step(i, j);
            t += CROSS_THREADS;
        }
    }
}

hipError_t launch_cross(const CrossDesc* units, uint32_t n, uint64_t total, BufSet bufs,
                        const uint64_t* status, int32_t* out_r, int32_t* out_s, uint64_t capacity,
                        hipStream_t st)
{
    if (n == 0 || total == 0) return hipSuccess;
    const uint32_t per = cross_rows(total, CROSS_THREADS * 4);
    const uint64_t blocks = (total + per - 1) / per;
    hipLaunchKernelGGL(k_cross, dim3((uint32_t)blocks), dim3(CROSS_THREADS), 0, st, units, n, total, per,
                       bufs, status, out_r, out_s, capacity);
    return hipGetLastError();
}

// single-key buckets of the sort that are not yet in the output columns. A
// thread has eight rows in flight: 90k rows of a 1M Zipf sort took 43 us with one
// row in flight in 6 blocks, 8 in 44 blocks so; 2^27 rows' hot keys 147 -> 99 us.
constexpr int COPY_UNROLL = 8;

template <typename K>
__global__ __launch_bounds__(CROSS_THREADS) void k_copy(const CopyDesc* __restrict__ units,
                                                        uint32_t n, uint64_t total, uint32_t per, BufSet bufs,
                                                        K* __restrict__ out_k,
                                                        int32_t* __restrict__ out_r)
{
    const uint64_t t0 = blockIdx.x * (uint64_t)per;
    uint64_t t1 = t0 + per;
    if (t1 > total) t1 = total;
    const size_t stride = sizeof(CopyDesc) / 8;
    const uint64_t* pfx = &units[0].pfx;
    uint64_t t = t0 + threadIdx.x;
    if (t >= t1) return;
    uint32_t u = find_unit(pfx, stride, n, t);
    CopyDesc U = units[u];
    while (t < t1) {
        while (t >= U.pfx + U.len) U = units[++u];
        const uint64_t loc = t - U.pfx;
        const uint64_t end = U.pfx + U.len < t1 ? U.pfx + U.len : t1;  // the thread's rows of this unit
        const uint32_t rows = (uint32_t)((end - t + CROSS_THREADS - 1) / CROSS_THREADS);
        const uint32_t m = rows < (uint32_t)COPY_UNROLL ? rows : (uint32_t)COPY_UNROLL;
        const K* const src_k = (const K*)bufs.key[U.buf][0] + U.start + loc;
        const int32_t* const src_r = bufs.rid[U.buf][0] + U.start + loc;
        K k[COPY_UNROLL];
        int32_t r[COPY_UNROLL];
#pragma unroll
        for (int i = 0; i < COPY_UNROLL; i++) {
            k[i] = ld_now(src_k, min((uint32_t)i, m - 1) * CROSS_THREADS);
            r[i] = ld_now(src_r, min((uint32_t)i, m - 1) * CROSS_THREADS);
        }
#pragma unroll
        for (int i = 0; i < COPY_UNROLL; i++) {
            if ((uint32_t)i < m) {
                out_k[U.out + loc + i * CROSS_THREADS] = k[i];
                out_r[U.out + loc + i * CROSS_THREADS] = r[i];
            }
        }
        t += m * CROSS_THREADS;
    }
}

hipError_t launch_copy(int key_bytes, const CopyDesc* units, uint32_t n, uint64_t total,
                       BufSet bufs, void* out_k, int32_t* out_r, hipStream_t st)
{
    if (n == 0 || total == 0) return hipSuccess;
    const uint32_t per = cross_rows(total, CROSS_THREADS * COPY_UNROLL);
    const uint64_t blocks = (total + per - 1) / per;
    if (key_bytes == 4)
        hipLaunchKernelGGL(k_copy<int32_t>, dim3((uint32_t)blocks), dim3(CROSS_THREADS), 0, st, units, n,
                           total, per, bufs, (int32_t*)out_k, out_r);
    else
        hipLaunchKernelGGL(k_copy<int64_t>, dim3((uint32_t)blocks), dim3(CROSS_THREADS), 0, st, units, n,
                           total, per, bufs, (int64_t*)out_k, out_r);
    return hipGetLastError();
}

}  // namespace tj
