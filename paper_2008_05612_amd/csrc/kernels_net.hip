// Genotype-network kernels of libhpmap: single-point-mutation counts (the
// numerators of phi_pq, robustness and phi_del of Eq. 2) and neutral-network
// components by union-find on the N-cube of sequences.
//
// All of them stream the uint16 phenotype map and gather the mutants' vectors
// from it; besides these gathers they wait for atomics on the classes' counters
// (neighbours), on the dense matrix (phi) and for chains of parents (union-find).
#include <hip/hip_runtime.h>

#include "hp_internal.h"
#include "kernels.h"

namespace hpmap {

namespace {

unsigned grid_for(uint64_t n, unsigned block)
{
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;   // a grid-size hint only
    const uint64_t want = (n + block - 1) / block;
    const uint64_t cap = uint64_t(cus) * 16;
    return unsigned(std::max<uint64_t>(1, std::min(want, cap)));
}

}  // namespace

// For each designing genotype g (phenotype q) and each one-bit mutant p:
// neutral / deleterious / other counts of q, and the phi row of phi_q.
__global__ __launch_bounds__(256) void k_neighbors(const uint16_t *__restrict__ map, int N,
                                                   uint64_t total, int n_class,
                                                   unsigned long long *neutral,
                                                   unsigned long long *deleterious,
                                                   unsigned long long *other, int phi_q,
                                                   unsigned long long *phi_row)
{
    for (uint64_t g = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; g < total;
         g += uint64_t(gridDim.x) * blockDim.x) {
        const uint16_t q = map[g];
        if (q == HP_NONE || int(q) >= n_class)   // ids beyond n_class are not phenotypes
            continue;
        unsigned a = 0, d = 0, o = 0;
        for (int i = 0; i < N; ++i) {
            const uint16_t p = map[g ^ (uint64_t(1) << i)];
            a += p == q;
            d += p == HP_NONE;
            o += (p != q) & (p != HP_NONE);
            if (phi_row && int(q) == phi_q)
                atomicAdd(&phi_row[(p == HP_NONE || int(p) >= n_class) ? n_class : int(p)], 1ull);
        }
        if (neutral && a)
            atomicAdd(&neutral[q], (unsigned long long)a);
        if (deleterious && d)
            atomicAdd(&deleterious[q], (unsigned long long)d);
        if (other && o)
            atomicAdd(&other[q], (unsigned long long)o);
    }
}

// ---------------------------------------------------------------------------
// Eight genotypes per lane.  The map is read as 16-byte vectors holding the
// genotypes 8k .. 8k+7: the mutants of bits 0..2 lie in the same vector, and
// the mutants of bit i >= 3 of all eight are the eight entries of vector
// k ^ 2^(i-3).  One 16-byte load then replaces eight 2-byte loads, so a wave
// issues an eighth of the load instructions.  These kernels serve 16-byte
// aligned maps with N >= 3; the one-genotype kernels cover the rest.
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t geno8(const uint4 &v, int r)
{
    const uint32_t w = r < 2 ? v.x : (r < 4 ? v.y : (r < 6 ? v.z : v.w));
    return (w >> (16 * (r & 1))) & 0xffffu;
}

__device__ __forceinline__ void unpack8(const uint4 &v, uint32_t q[8])
{
#pragma unroll
    for (int r = 0; r < 8; ++r)
        q[r] = geno8(v, r);
}

// Orders a wave's LDS accesses between its lanes (which run in step).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

static bool use_geno8(const uint16_t *map, int N)
{
    return N >= 3 && (reinterpret_cast<uintptr_t>(map) & 15u) == 0;
}

// Counts a and d of a vector's genotypes, added up over genotypes of one
// phenotype at the first of them (0 at the others); the number of genotypes goes
// to the upper 16 bits of a.  Neighbours are often of one phenotype, and the
// atomics on the classes' counters follow (3x3x3: k_neighbors8 1.10 -> 0.99 ms,
// k_phi_counts8 1.55 -> 1.44 ms).
__device__ __forceinline__ void merge8(const uint32_t q[8], uint32_t a[8], uint32_t d[8])
{
#pragma unroll
    for (int r = 0; r < 8; ++r)
        a[r] += 1u << 16;
#pragma unroll
    for (int i = 0; i < 7; ++i)
#pragma unroll
        for (int j = i + 1; j < 8; ++j) {
            const bool same = q[j] == q[i];
            a[i] += same ? a[j] : 0u;
            d[i] += same ? d[j] : 0u;
            a[j] = same ? 0u : a[j];
            d[j] = same ? 0u : d[j];
        }
}

// Calls f(k, on) for the vectors k < n8 that hold a phenotype below n_class
// (ANY: any id but HP_NONE), 64 at a time: each wave collects such vectors in a
// list of its own in LDS and hands them on once it has a wave full.  About
// one vector in five holds one on the 3x3x3 map, so the loops over mutants run
// with all lanes busy instead of a fifth of them (3x3x3: k_phi_counts8 2.0 ->
// 1.5 ms, k_neighbors8 1.16 -> 1.10 ms; k_uf_hook8 with its edge list 3.0 ->
// 1.05 ms).  `on` is false in the lanes beyond the end of the last, partial wave
// full.
template <bool ANY, class F>
__device__ __forceinline__ void for_active8(const uint4 *__restrict__ m4, uint64_t n8, int n_class,
                                            uint64_t *list, F f)
{
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1;
    const uint64_t step = uint64_t(gridDim.x) * blockDim.x;
    int n = 0;
    for (uint64_t base = uint64_t(blockIdx.x) * blockDim.x + (threadIdx.x & ~63u); base < n8;
         base += step) {
        const uint64_t k = base + lane;
        bool act = false;
        if (k < n8) {
            uint32_t q[8];
            unpack8(m4[k], q);
#pragma unroll
            for (int r = 0; r < 8; ++r)
                act |= ANY ? q[r] != HP_NONE : int(q[r]) < n_class;
        }
        const unsigned long long m = __ballot(act);
        if (act)
            list[n + __popcll(m & below)] = k;
        n += __popcll(m);
        if (n >= 64) {
            wave_sync();
            const uint64_t full = list[lane], rest = list[64 + lane];
            f(full, true);
            wave_sync();
            list[lane] = rest;   // meaningful below n - 64
            n -= 64;
        }
    }
    wave_sync();
    if (n > 0)
        f(lane < n ? list[lane] : 0, lane < n);
}

__global__ __launch_bounds__(256) void k_neighbors8(const uint4 *__restrict__ m4, int N, uint64_t n8,
                                                    int n_class, unsigned long long *neutral,
                                                    unsigned long long *deleterious,
                                                    unsigned long long *other, int phi_q,
                                                    unsigned long long *phi_row)
{
    __shared__ uint64_t lists[4][128];
    const uint16_t *__restrict__ map = reinterpret_cast<const uint16_t *>(m4);
    for_active8<false>(m4, n8, n_class, lists[threadIdx.x >> 6], [&](uint64_t k, bool on) {
        if (!on)
            return;
        uint32_t q[8];
        unpack8(m4[k], q);
        // a: neutral mutants, d: deleterious ones; the other N - a - d change the phenotype
        uint32_t a[8], d[8];
#pragma unroll
        for (int r = 0; r < 8; ++r)
            a[r] = d[r] = 0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const uint32_t p = q[r ^ (1 << i)];
                a[r] += p == q[r] ? 1u : 0u;
                d[r] += p == HP_NONE ? 1u : 0u;
            }
#pragma unroll 4
        for (int i = 3; i < N; ++i) {
            const uint4 nv = m4[k ^ (uint64_t(1) << (i - 3))];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const uint32_t p = geno8(nv, r);
                a[r] += p == q[r] ? 1u : 0u;
                d[r] += p == HP_NONE ? 1u : 0u;
            }
        }
        merge8(q, a, d);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (int(q[r]) >= n_class)
                continue;
            const uint32_t o = uint32_t(N) * (a[r] >> 16) - (a[r] & 0xffffu) - d[r];
            if (neutral && (a[r] & 0xffffu))
                atomicAdd(&neutral[q[r]], (unsigned long long)(a[r] & 0xffffu));
            if (deleterious && d[r])
                atomicAdd(&deleterious[q[r]], (unsigned long long)d[r]);
            if (other && o)
                atomicAdd(&other[q[r]], (unsigned long long)o);
            if (phi_row && int(q[r]) == phi_q) {
                const uint64_t g = 8 * k + uint64_t(r);
                for (int i = 0; i < N; ++i) {
                    const uint16_t p = map[g ^ (uint64_t(1) << i)];
                    atomicAdd(&phi_row[(p == HP_NONE || int(p) >= n_class) ? n_class : int(p)],
                              1ull);
                }
            }
        }
    });
}

hipError_t launch_neighbors(const uint16_t *map, int N, int n_class, unsigned long long *neutral,
                            unsigned long long *deleterious, unsigned long long *other, int phi_q,
                            unsigned long long *phi_row, hipStream_t st)
{
    const uint64_t total = uint64_t(1) << N;
    if (use_geno8(map, N)) {
        const uint64_t n8 = total / 8;
        hipLaunchKernelGGL(k_neighbors8, dim3(grid_for(n8, 256)), dim3(256), 0, st,
                           reinterpret_cast<const uint4 *>(map), N, n8, n_class, neutral,
                           deleterious, other, phi_q, phi_row);
    } else {
        hipLaunchKernelGGL(k_neighbors, dim3(grid_for(total, 256)), dim3(256), 0, st, map, N,
                           total, n_class, neutral, deleterious, other, phi_q, phi_row);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The whole phi_pq matrix (Eq. 2) as dense counts: row q (phenotype of the
// genotype, q < n_class), column p (phenotype of its single-point mutant,
// column n_class for deleterious ids).  Neutral and deleterious mutants of
// a genotype are summed in registers and added once; each mutant into
// another phenotype adds one at (q, p).
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_phi_counts(const uint16_t *__restrict__ map, int N,
                                                    uint64_t total, int n_class,
                                                    unsigned long long *counts)
{
    const uint64_t ld = uint64_t(n_class) + 1;
    for (uint64_t g = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; g < total;
         g += uint64_t(gridDim.x) * blockDim.x) {
        const int q = map[g];
        if (q >= n_class)   // 0xFFFF and ids beyond n_class have no row
            continue;
        unsigned long long *row = counts + uint64_t(q) * ld;
        unsigned neutral = 0, del = 0;
        for (int i = 0; i < N; ++i) {
            const int p = map[g ^ (uint64_t(1) << i)];
            if (p == q)
                ++neutral;
            else if (p >= n_class)
                ++del;
            else
                atomicAdd(&row[p], 1ull);
        }
        if (neutral)
            atomicAdd(&row[q], (unsigned long long)neutral);
        if (del)
            atomicAdd(&row[n_class], (unsigned long long)del);
    }
}

// Eight genotypes per lane (the vector layout of k_neighbors8).
__global__ __launch_bounds__(256) void k_phi_counts8(const uint4 *__restrict__ m4, int N,
                                                     uint64_t n8, int n_class,
                                                     unsigned long long *counts)
{
    __shared__ uint64_t lists[4][128];
    const uint64_t ld = uint64_t(n_class) + 1;
    for_active8<false>(m4, n8, n_class, lists[threadIdx.x >> 6], [&](uint64_t k, bool on) {
        if (!on)
            return;
        uint32_t q[8];
        unpack8(m4[k], q);
        uint32_t neutral[8], del[8];
#pragma unroll
        for (int r = 0; r < 8; ++r)
            neutral[r] = del[r] = 0;
        // one mutant p of genotype r: neutral and deleterious ones are
        // counted in registers, one into another phenotype adds at (q, p)
        auto take = [&](int r, uint32_t p) {
            const bool row = int(q[r]) < n_class;
            neutral[r] += row && p == q[r] ? 1u : 0u;
            del[r] += row && p != q[r] && int(p) >= n_class ? 1u : 0u;
            if (row && p != q[r] && int(p) < n_class)
                atomicAdd(&counts[uint64_t(q[r]) * ld + p], 1ull);
        };
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int r = 0; r < 8; ++r)
                take(r, q[r ^ (1 << i)]);
        for (int i = 3; i < N; ++i) {
            const uint4 nv = m4[k ^ (uint64_t(1) << (i - 3))];
#pragma unroll
            for (int r = 0; r < 8; ++r)
                take(r, geno8(nv, r));
        }
        merge8(q, neutral, del);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (int(q[r]) >= n_class)
                continue;
            unsigned long long *row = counts + uint64_t(q[r]) * ld;
            if (neutral[r] & 0xffffu)
                atomicAdd(&row[q[r]], (unsigned long long)(neutral[r] & 0xffffu));
            if (del[r])
                atomicAdd(&row[n_class], (unsigned long long)del[r]);
        }
    });
}

// Sparse rows (CSR, columns ascending).  Both passes stream the dense
// matrix once (HBM-bound) as 16-byte vectors; each thread keeps kPhiUnroll
// loads in flight, a workgroup covers kPhiChunk consecutive vectors per
// iteration.  Rows are odd numbers of entries as often as not, so a row
// starts with the one entry before its first 16-byte boundary, if there is one
// (the second half of its vector 0), and may end in half a vector.  Measured
// on the 21.4 GB matrix of 3x3x3: counting 3.40 ms, 6.3 TB/s (8-byte loads
// 3.74 ms, 5.7 TB/s); compaction, which also writes the entries, 3.82 ms (3.89).
constexpr int kPhiUnroll = 4;
constexpr int kPhiChunk = 256 * kPhiUnroll;

struct PhiRow {
    const ulonglong2 *v;   // 16-byte aligned: entries 2 i - shift, 2 i - shift + 1
    uint64_t n;            // vectors that hold an entry of the row
    uint64_t ld;
    uint32_t shift;        // 1: the row starts in the second half of v[0]
};

__device__ __forceinline__ PhiRow phi_row_of(const unsigned long long *counts, uint64_t ld,
                                             uint64_t row)
{
    const unsigned long long *r = counts + row * ld;
    const uint32_t shift = (reinterpret_cast<uintptr_t>(r) >> 3) & 1u;
    return {reinterpret_cast<const ulonglong2 *>(r - shift), (ld + shift + 1) / 2, ld, shift};
}

// Entries 2 i - shift (x) and 2 i + 1 - shift (y) of the row, 0 beyond its ends;
// the halves that lie outside the row are not read.
__device__ __forceinline__ ulonglong2 phi_load(const PhiRow &r, uint64_t i)
{
    if (i >= r.n)
        return ulonglong2{0, 0};
    const bool lead = i == 0 && r.shift, tail = 2 * i + 1 - r.shift >= r.ld;
    if (lead | tail) {
        const auto *e = reinterpret_cast<const unsigned long long *>(r.v + i);
        return ulonglong2{lead ? 0 : e[0], tail ? 0 : e[1]};
    }
    return r.v[i];
}

// k_phi_row_nnz: one workgroup per row writes its number of non-zero
// entries to row_ptr[q].
__global__ __launch_bounds__(256) void k_phi_row_nnz(const unsigned long long *__restrict__ counts,
                                                     int n_class, uint64_t *row_ptr)
{
    __shared__ unsigned part[4];
    const PhiRow row = phi_row_of(counts, uint64_t(n_class) + 1, blockIdx.x);
    unsigned c = 0;
    for (uint64_t base = 0; base < row.n; base += kPhiChunk) {
        ulonglong2 v[kPhiUnroll];
#pragma unroll
        for (int k = 0; k < kPhiUnroll; ++k)
            v[k] = phi_load(row, base + k * 256 + threadIdx.x);
#pragma unroll
        for (int k = 0; k < kPhiUnroll; ++k)
            c += (v[k].x != 0) + (v[k].y != 0);
    }
    for (int o = 32; o; o >>= 1)
        c += __shfl_xor(c, o);
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0)
        row_ptr[blockIdx.x] = uint64_t(part[0]) + part[1] + part[2] + part[3];
}

// In-place exclusive scan of row_ptr[0 .. n) with the total written to
// row_ptr[n]: one workgroup walks tiles of 8192 rows, 8 per thread; the loads
// of the next tile are in flight while a tile is scanned (51704 rows: 0.05 ms; a
// contiguous chunk per thread, read twice, 0.13 ms).
__global__ __launch_bounds__(1024) void k_phi_scan(uint64_t *row_ptr, int n)
{
    constexpr int kPer = 8;
    __shared__ uint64_t sums[2][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t v[kPer], run = 0;
    auto load = [&](int lo) {
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            v[i] = lo + i < n ? row_ptr[lo + i] : 0;
    };
    load(threadIdx.x * kPer);
    for (int base = 0, t = 0; base < n; base += 1024 * kPer, t ^= 1) {
        const int lo = base + int(threadIdx.x) * kPer;
        uint64_t cur[kPer], own = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            cur[i] = own;   // of this thread's earlier rows
            own += v[i];
        }
        load(lo + 1024 * kPer);
        uint64_t upto = own;   // inclusive over the wave
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint64_t below = __shfl_up((unsigned long long)upto, o);
            upto += lane >= o ? below : 0;
        }
        if (lane == 63)
            sums[t][wave] = upto;
        __syncthreads();   // the other half of sums serves the next tile
        uint64_t before = run + upto - own;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const uint64_t s = sums[t][w];
            before += w < wave ? s : 0;
            run += s;
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (lo + i < n)
                row_ptr[lo + i] = before + cur[i];
    }
    if (threadIdx.x == 0)
        row_ptr[n] = run;
}

// One workgroup per row: the non-zero entries in column order, from
// row_ptr[q] onwards.  Sub-chunk k of a chunk holds the vectors base + 256 k ..
// base + 256 k + 255 (thread t reads vector base + 256 k + t); an entry's
// slot is the count of non-zeros in earlier sub-chunks, earlier waves of its
// sub-chunk (per-wave counts in LDS) and earlier lanes of its wave (ballots).
__global__ __launch_bounds__(256) void k_phi_compact(const unsigned long long *__restrict__ counts,
                                                     int n_class, const uint64_t *__restrict__ row_ptr,
                                                     uint32_t *cols, uint64_t *vals)
{
    __shared__ unsigned wave_n[2][kPhiUnroll][4];
    const PhiRow row = phi_row_of(counts, uint64_t(n_class) + 1, blockIdx.x);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long below = (1ull << lane) - 1;
    uint64_t at = row_ptr[blockIdx.x];
    ulonglong2 next[kPhiUnroll];
#pragma unroll
    for (int k = 0; k < kPhiUnroll; ++k)
        next[k] = phi_load(row, k * 256 + threadIdx.x);
    int t = 0;
    for (uint64_t base = 0; base < row.n; base += kPhiChunk, t ^= 1) {
        ulonglong2 v[kPhiUnroll];
        unsigned before[kPhiUnroll];
#pragma unroll
        for (int k = 0; k < kPhiUnroll; ++k) {
            v[k] = next[k];
            next[k] = phi_load(row, base + kPhiChunk + k * 256 + threadIdx.x);
        }
#pragma unroll
        for (int k = 0; k < kPhiUnroll; ++k) {
            const unsigned long long mx = __ballot(v[k].x != 0), my = __ballot(v[k].y != 0);
            before[k] = __popcll(mx & below) + __popcll(my & below);
            if (lane == 0)
                wave_n[t][k][wave] = __popcll(mx) + __popcll(my);
        }
        __syncthreads();   // the other half of wave_n serves the next chunk
        unsigned run = 0;
#pragma unroll
        for (int k = 0; k < kPhiUnroll; ++k) {
            unsigned off = run + before[k];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const unsigned c = wave_n[t][k][w];
                off += w < wave ? c : 0;
                run += c;
            }
            const uint32_t col = uint32_t(2 * (base + k * 256 + threadIdx.x) - row.shift);
            uint64_t slot = at + off;
            if (v[k].x) {
                cols[slot] = col;
                vals[slot++] = v[k].x;
            }
            if (v[k].y) {
                cols[slot] = col + 1;
                vals[slot] = v[k].y;
            }
        }
        at += run;
    }
}

hipError_t launch_phi_counts(const uint16_t *map, int N, int n_class, unsigned long long *counts,
                             hipStream_t st)
{
    const uint64_t total = uint64_t(1) << N;
    if (use_geno8(map, N)) {
        const uint64_t n8 = total / 8;
        hipLaunchKernelGGL(k_phi_counts8, dim3(grid_for(n8, 256)), dim3(256), 0, st,
                           reinterpret_cast<const uint4 *>(map), N, n8, n_class, counts);
    } else {
        hipLaunchKernelGGL(k_phi_counts, dim3(grid_for(total, 256)), dim3(256), 0, st, map, N,
                           total, n_class, counts);
    }
    return hipGetLastError();
}

hipError_t launch_phi_row_ptr(const unsigned long long *counts, int n_class, uint64_t *row_ptr,
                              hipStream_t st)
{
    hipLaunchKernelGGL(k_phi_row_nnz, dim3(n_class), dim3(256), 0, st, counts, n_class, row_ptr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_phi_scan, dim3(1), dim3(1024), 0, st, row_ptr, n_class);
    return hipGetLastError();
}

hipError_t launch_phi_compact(const unsigned long long *counts, int n_class,
                              const uint64_t *row_ptr, uint32_t *cols, uint64_t *vals,
                              hipStream_t st)
{
    hipLaunchKernelGGL(k_phi_compact, dim3(n_class), dim3(256), 0, st, counts, n_class, row_ptr,
                       cols, vals);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Union-find.  parent[x] <= x always holds and roots satisfy parent[x] == x;
// two roots are joined by pointing the larger at the smaller with a CAS, so
// the root of every tree is its smallest member and the final labels do not
// depend on the schedule.  Path halving writes only ancestors, so concurrent
// readers always see a valid (older or newer) ancestor.
// ---------------------------------------------------------------------------

constexpr uint32_t kNoLabel = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t uf_root(uint32_t *parent, uint32_t x)
{
    uint32_t p = parent[x];
    while (p != x) {
        const uint32_t gp = parent[p];
        if (gp != p)
            parent[x] = gp;
        x = p;
        p = gp;
    }
    return x;
}

__device__ __forceinline__ void uf_unite(uint32_t *parent, uint32_t a, uint32_t b)
{
    uint32_t ra = uf_root(parent, a), rb = uf_root(parent, b);
    while (ra != rb) {
        const uint32_t hi = max(ra, rb), lo = min(ra, rb);
        const uint32_t old = atomicCAS(&parent[hi], hi, lo);
        if (old == hi)
            break;
        ra = uf_root(parent, old);
        rb = uf_root(parent, lo);
    }
}

__global__ __launch_bounds__(256) void k_uf_init(const uint16_t *__restrict__ map, uint32_t *parent,
                                                 uint32_t *compsize, uint64_t total)
{
    for (uint64_t g = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; g < total;
         g += uint64_t(gridDim.x) * blockDim.x) {
        parent[g] = map[g] == HP_NONE ? kNoLabel : uint32_t(g);
        compsize[g] = 0;
    }
}

// Edge g -- g|bit for every clear bit of g between equal designing phenotypes.
__global__ __launch_bounds__(256) void k_uf_hook(const uint16_t *__restrict__ map, int N,
                                                 uint32_t *parent, uint64_t total)
{
    for (uint64_t g = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; g < total;
         g += uint64_t(gridDim.x) * blockDim.x) {
        const uint16_t q = map[g];
        if (q == HP_NONE)
            continue;
        for (int i = 0; i < N; ++i) {
            const uint64_t u = g | (uint64_t(1) << i);
            if (u != g && map[u] == q)
                uf_unite(parent, uint32_t(g), uint32_t(u));
        }
    }
}

// Eight genotypes per lane (the vector layout of k_neighbors8): the edges
// g -- g|bit of the genotypes 8k .. 8k+7.  Few lanes find an edge at the same
// mutant, and a union is a chain of dependent reads of the parents, so the
// edges are collected in LDS and united a wave full at a time.  An edge between
// the vectors k and k | bit is left out where it closes a square: genotype r
// has a set bit j < 3, r ^ j has the same edge and both vectors join r and r ^
// j.
// Per wave: what a flush may leave (255) and the most that is pushed before the
// next one, 4 edges of each bit j < 3 for 64 lanes (768), fit.
constexpr int kEdges = 1024;
constexpr int kEdgesFlush = 256;
static_assert(kEdgesFlush - 1 + 64 * 12 <= kEdges, "edge list");

__global__ __launch_bounds__(256) void k_uf_hook8(const uint4 *__restrict__ m4, int N,
                                                  uint32_t *parent, uint64_t n8)
{
    __shared__ uint64_t lists[4][128];
    __shared__ uint2 edges[4][kEdges];
    __shared__ int n_edges[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint2 *const edge = edges[wave];
    int *const count = &n_edges[wave];
    if (lane == 0)
        *count = 0;
    wave_sync();
    auto flush = [&](int least) {
        wave_sync();
        const int c = *count;
        if (c < least)
            return;
        for (int e = lane; e < c; e += 64)
            uf_unite(parent, edge[e].x, edge[e].y);
        wave_sync();
        if (lane == 0)
            *count = 0;
        wave_sync();
    };
    for_active8<true>(m4, n8, 0, lists[wave], [&](uint64_t k, bool on) {
        uint32_t q[8];
        unpack8(m4[k], q);
        // genotypes with a phenotype; same[j]: those with bit j set joined to r ^ j
        uint32_t has = 0, same[3] = {0, 0, 0};
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            has |= q[r] != HP_NONE ? 1u << r : 0u;
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (r & (1 << j))
                    same[j] |= q[r] == q[r ^ (1 << j)] ? 1u << r : 0u;
        }
        has = on ? has : 0u;
        const uint32_t g0 = uint32_t(8 * k);
        auto push = [&](uint32_t e, uint32_t bit) {   // edges g0 + r -- g0 + r | bit
            if (e) {
                int at = atomicAdd(count, __popc(e));
                do {
                    const uint32_t g = g0 + uint32_t(__ffs(e) - 1);
                    edge[at++] = uint2{g, g | bit};
                    e &= e - 1;
                } while (e);
            }
        };
#pragma unroll
        for (int j = 0; j < 3; ++j)
            push((same[j] & has) >> (1 << j), 1u << j);
        flush(kEdgesFlush);
        for (int i = 3; i < N; i += 4) {
            uint4 nv[4];
            bool up[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint64_t u = k | (uint64_t(1) << (i + j - 3));
                up[j] = i + j < N && u != k && has;
                nv[j] = up[j] ? m4[u] : uint4{0, 0, 0, 0};
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t e = 0;
#pragma unroll
                for (int r = 0; r < 8; ++r)
                    e |= geno8(nv[j], r) == q[r] ? 1u << r : 0u;
                e &= up[j] ? has : 0u;
                e &= ~(((e << 1) & same[0]) | ((e << 2) & same[1]) | ((e << 4) & same[2]));
                push(e, 1u << (i + j));
                flush(kEdgesFlush);
            }
        }
    });
    flush(1);
}

__global__ __launch_bounds__(256) void k_uf_compress(const uint16_t *__restrict__ map,
                                                     uint32_t *parent, uint32_t *compsize,
                                                     uint64_t total)
{
    for (uint64_t g = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; g < total;
         g += uint64_t(gridDim.x) * blockDim.x) {
        if (map[g] == HP_NONE)
            continue;
        uint32_t r = uint32_t(g);
        while (parent[r] != r)
            r = parent[r];
        parent[g] = r;
        atomicAdd(&compsize[r], 1u);
    }
}

// Eight genotypes per lane.  Genotypes of one vector are often of one
// component: their sizes are added up first, one atomic per root and vector
// (3x3x3: 0.41 ms, one genotype per lane 0.63 ms).
__global__ __launch_bounds__(256) void k_uf_compress8(const uint4 *__restrict__ m4,
                                                      uint32_t *parent, uint32_t *compsize,
                                                      uint64_t n8)
{
    __shared__ uint64_t lists[4][128];
    uint4 *parent4 = reinterpret_cast<uint4 *>(parent);
    for_active8<true>(m4, n8, 0, lists[threadIdx.x >> 6], [&](uint64_t k, bool on) {
        if (!on)
            return;
        const uint4 a = parent4[2 * k], b = parent4[2 * k + 1];
        uint32_t r[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        uint32_t up[8];   // the parents one step further; kNoLabel stays
        bool more = false;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            up[i] = r[i] == kNoLabel ? kNoLabel : parent[r[i]];
            more |= up[i] != r[i];
        }
        while (more) {
            more = false;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (up[i] != r[i]) {
                    r[i] = up[i];
                    up[i] = parent[r[i]];
                    more |= up[i] != r[i];
                }
            }
        }
        parent4[2 * k] = uint4{r[0], r[1], r[2], r[3]};
        parent4[2 * k + 1] = uint4{r[4], r[5], r[6], r[7]};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            uint32_t c = 1;
            bool first = r[i] != kNoLabel;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                c += j > i && r[j] == r[i] ? 1u : 0u;
                first &= !(j < i && r[j] == r[i]);
            }
            if (first)
                atomicAdd(&compsize[r[i]], c);
        }
    });
}

__global__ __launch_bounds__(256) void k_uf_count(const uint16_t *__restrict__ map,
                                                  const uint32_t *__restrict__ labels,
                                                  const uint32_t *__restrict__ compsize,
                                                  uint32_t *ncomp, uint32_t *largest,
                                                  int n_class, uint64_t total)
{
    for (uint64_t g = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; g < total;
         g += uint64_t(gridDim.x) * blockDim.x) {
        const uint16_t q = map[g];
        if (q == HP_NONE || int(q) >= n_class || labels[g] != uint32_t(g))
            continue;
        if (ncomp)
            atomicAdd(&ncomp[q], 1u);
        if (largest)
            atomicMax(&largest[q], compsize[g]);
    }
}

// Eight genotypes per lane (map and labels read as vectors).
__global__ __launch_bounds__(256) void k_uf_count8(const uint4 *__restrict__ m4,
                                                   const uint4 *__restrict__ labels4,
                                                   const uint32_t *__restrict__ compsize,
                                                   uint32_t *ncomp, uint32_t *largest,
                                                   int n_class, uint64_t n8)
{
    for (uint64_t k = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; k < n8;
         k += uint64_t(gridDim.x) * blockDim.x) {
        uint32_t q[8];
        unpack8(m4[k], q);
        bool any = false;
#pragma unroll
        for (int r = 0; r < 8; ++r)
            any |= int(q[r]) < n_class;
        if (!any)
            continue;
        const uint4 la = labels4[2 * k], lb = labels4[2 * k + 1];
        const uint32_t lab[8] = {la.x, la.y, la.z, la.w, lb.x, lb.y, lb.z, lb.w};
        const uint32_t g0 = uint32_t(8 * k);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (int(q[r]) >= n_class || lab[r] != g0 + uint32_t(r))
                continue;
            if (ncomp)
                atomicAdd(&ncomp[q[r]], 1u);
            if (largest)
                atomicMax(&largest[q[r]], compsize[g0 + r]);
        }
    }
}

hipError_t launch_components(const uint16_t *map, int N, uint32_t *labels, uint32_t *compsize,
                             uint32_t *ncomp, uint32_t *largest, int n_class, hipStream_t st)
{
    const uint64_t total = uint64_t(1) << N;
    const dim3 grid(grid_for(total, 256)), block(256);
    hipError_t e;
    if (ncomp && (e = launch_fill_u32(ncomp, 0u, uint64_t(n_class), st)) != hipSuccess)
        return e;
    if (largest && (e = launch_fill_u32(largest, 0u, uint64_t(n_class), st)) != hipSuccess)
        return e;
    // eight genotypes per lane where the map (and, for the count, the labels)
    // are 16-byte vectors; one genotype per lane otherwise.  The init pass
    // stays one genotype per lane: its 4-byte stores are contiguous per wave
    // (measured 0.30 ms against 0.36 ms for 8 per lane on the 3x3x3 map).
    const bool v8 = use_geno8(map, N) && (reinterpret_cast<uintptr_t>(labels) & 15u) == 0;
    const uint64_t n8 = total / 8;
    const dim3 grid8(grid_for(n8, 256));
    const uint4 *m4 = reinterpret_cast<const uint4 *>(map);
    hipLaunchKernelGGL(k_uf_init, grid, block, 0, st, map, labels, compsize, total);
    if (use_geno8(map, N))
        hipLaunchKernelGGL(k_uf_hook8, grid8, block, 0, st, m4, N, labels, n8);
    else
        hipLaunchKernelGGL(k_uf_hook, grid, block, 0, st, map, N, labels, total);
    if (v8)
        hipLaunchKernelGGL(k_uf_compress8, grid8, block, 0, st, m4, labels, compsize, n8);
    else
        hipLaunchKernelGGL(k_uf_compress, grid, block, 0, st, map, labels, compsize, total);
    if (v8)
        hipLaunchKernelGGL(k_uf_count8, grid8, block, 0, st, m4,
                           reinterpret_cast<const uint4 *>(labels), compsize, ncomp, largest,
                           n_class, n8);
    else
        hipLaunchKernelGGL(k_uf_count, grid, block, 0, st, map, labels, compsize, ncomp, largest,
                           n_class, total);
    return hipGetLastError();
}

}  // namespace hpmap
