// Stands in for the HIP runtime when a kernel body is compiled for the CPU
// (host test only): the lanes of one workgroup are coroutines, switched at
// every operation that a wave or the workgroup does together, in an order
// drawn from a seed.  Between two such operations each lane reads and writes
// LDS on its own, so whatever order the hardware serves the lanes of different
// waves in, some seed has an order that is no better.
#pragma once

#include <algorithm>
#include <array>
#include <cstdint>
#include <cstdlib>
#include <functional>

#define __device__
#define __host__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define hipLaunchKernelGGL(...) ((void)0)
// the only assembly with operands is the median of (a, b, c) into m
#define asm(...) (m = std::max(std::min(a, b), std::min(std::max(a, b), c)))

typedef int hipError_t;
typedef void *hipStream_t;
constexpr hipError_t hipSuccess = 0, hipErrorInvalidValue = 1;
inline hipError_t hipGetLastError() { return hipSuccess; }
struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

namespace emu {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned v6u __attribute__((ext_vector_type(6)));
typedef float v16f __attribute__((ext_vector_type(16)));

extern unsigned lane_id;          // thread index of the running lane
extern dim3 block_dim, block_idx, grid_dim;
struct Lane {
    unsigned x;
};
inline Lane lane() { return {lane_id}; }

void workgroup_barrier();
uint64_t ballot(bool on);
uint64_t exchange(uint64_t own, unsigned from);   // `own` of the wave's lane `from`
v16f mfma_scale(const v8i &a, const v8i &b, const v16f &c, int fmt_a, int fmt_b, int scale_a,
                int scale_b);
v16i mfma_i8(const v4i &a, const v4i &b, const v16i &c);
v6u to_fp6(const v16f &even, const v16f &odd, float scale);   // values in turn, divided by scale
unsigned byte_permute(unsigned upper, unsigned lower, unsigned select);

// Runs `body` on every lane of a workgroup of `threads`, in the order of `seed`.
void run(unsigned threads, uint64_t seed, const std::function<void()> &body);

}  // namespace emu

#define threadIdx emu::lane()
#define blockDim emu::block_dim
#define blockIdx emu::block_idx
#define gridDim emu::grid_dim

inline void __syncthreads() { emu::workgroup_barrier(); }
inline uint64_t __ballot(bool on) { return emu::ballot(on); }
inline int __any(bool on) { return emu::ballot(on) != 0; }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline int __popc(uint32_t x) { return __builtin_popcount(x); }
inline int __shfl(int v, int from) { return int(emu::exchange(uint32_t(v), unsigned(from) & 63u)); }
inline int __shfl_xor(int v, int mask)
{
    return int(emu::exchange(uint32_t(v), ((emu::lane_id & 63u) ^ unsigned(mask)) & 63u));
}
inline float __uint_as_float(unsigned x) { return __builtin_bit_cast(float, x); }

struct int2 {
    int x, y;
};
struct uint2 {
    unsigned x, y;
};
struct uint4 {
    unsigned x, y, z, w;
};

inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }
inline unsigned min(unsigned a, unsigned b) { return a < b ? a : b; }
inline unsigned max(unsigned a, unsigned b) { return a > b ? a : b; }

template <class T>
inline T atomicAdd(T *p, T v)
{
    const T old = *p;
    *p = old + v;
    return old;
}
inline unsigned atomicMax(unsigned *p, unsigned v)
{
    const unsigned old = *p;
    *p = max(old, v);
    return old;
}

// [0]: half 0's value in both halves of the wave, [1]: half 1's (both operands alike)
inline std::array<unsigned, 2> __builtin_amdgcn_permlane32_swap(unsigned a, unsigned, bool, bool)
{
    const unsigned col = emu::lane_id & 31u;
    const unsigned lower = unsigned(emu::exchange(a, col));
    return {lower, unsigned(emu::exchange(a, col + 32))};
}
inline int __builtin_amdgcn_readfirstlane(int v) { return int(emu::exchange(uint32_t(v), 0)); }
inline void __builtin_amdgcn_s_waitcnt(int) {}
inline void __builtin_amdgcn_s_setprio(int) {}
inline void __builtin_amdgcn_sched_group_barrier(int, int, int) {}
inline void __builtin_amdgcn_sched_barrier(int) {}
inline void __builtin_amdgcn_wave_barrier() {}
#define __builtin_amdgcn_perm emu::byte_permute
#define __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32 emu::to_fp6
#define __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, x, y, z) emu::mfma_i8(a, b, c)
#define __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, fa, fb, oa, sa, ob, sb) \
    emu::mfma_scale(a, b, c, fa, fb, sa, sb)
