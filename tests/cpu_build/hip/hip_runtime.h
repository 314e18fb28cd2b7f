// Stand-in for <hip/hip_runtime.h> with which the library's sources compile for the host CPU, for tests that must see an
// access out of bounds before a GPU does. A launch runs its workgroups one after the other; the threads of a workgroup are
// fibers that change places where lanes exchange values and at barriers (emulator.cpp). Only what the sources under test use.
#ifndef CPU_BUILD_HIP_RUNTIME_H_
#define CPU_BUILD_HIP_RUNTIME_H_

#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <functional>

#define __host__
#define __device__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __asm(name) __asm__("emu." name)  // compiler intrinsics declared by their names: emulator.cpp defines them
#define __align__(n) __attribute__((aligned(n)))

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct float2 { float x, y; };
struct int2 { int x, y; };
struct alignas(16) int4 { int x, y, z, w; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };
inline float2 make_float2(float x, float y) { return {x, y}; }
inline int2 make_int2(int x, int y) { return {x, y}; }
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }

typedef void *hipStream_t;
enum hipError_t { hipSuccess = 0, hipErrorInvalidDevice, hipErrorInvalidSymbol };
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int *dev) { *dev = 0; return hipSuccess; }
template <class T> hipError_t hipGetSymbolAddress(void **p, T &symbol) { *p = &symbol; return hipSuccess; }
#define HIP_SYMBOL(x) x

namespace emu {
extern dim3 thread_idx, block_idx, block_dim, grid_dim;
void launch(dim3 grid, dim3 block, const std::function<void()> &body);
void barrier();
int lane();
// Every live lane of the wave puts `bytes` (at most 64) down and gets the array of all 64 lanes' values (zeros for lanes
// that have returned), valid until its next exchange.
const void *exchange(const void *value, size_t bytes);
uint64_t live();  // lanes of the wave that have not returned
template <class T> T from(T x, int src) {
  T out;
  memcpy(&out, static_cast<const char *>(exchange(&x, sizeof x)) + 64 * (src & 63), sizeof out);
  return out;
}
struct Pair {
  uint32_t v[2];
  uint32_t operator[](int i) const { return v[i]; }
};
Pair swap_halves(uint32_t x, uint32_t y, int width);
int update_dpp(int old, int src, int ctrl, int row_mask);
void mfma_16x16x32_bf16(const void *x, const void *y, const float *c, float *d);
}  // namespace emu

#define threadIdx emu::thread_idx
#define blockIdx emu::block_idx
#define blockDim emu::block_dim
#define gridDim emu::grid_dim
#define __syncthreads() emu::barrier()
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) emu::launch(grid, block, [=] { kernel(__VA_ARGS__); })

template <class T> T min(T a, T b) { return b < a ? b : a; }
template <class T> T max(T a, T b) { return a < b ? b : a; }
inline int __float_as_int(float x) { return __builtin_bit_cast(int, x); }
inline uint32_t __float_as_uint(float x) { return __builtin_bit_cast(uint32_t, x); }
inline float __int_as_float(int x) { return __builtin_bit_cast(float, x); }
inline float __uint_as_float(uint32_t x) { return __builtin_bit_cast(float, x); }
inline int __popc(unsigned x) { return __builtin_popcount(x); }
inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
inline int __ffsll(long long x) { return __builtin_ffsll(x); }
inline int __clz(int x) { return x ? __builtin_clz((unsigned)x) : 32; }
inline int atomicAdd(int *p, int v) { const int old = *p; *p = old + v; return old; }
template <class T> T __shfl(T x, int src) { return emu::from(x, src); }
template <class T> T __shfl_xor(T x, int mask) { return emu::from(x, emu::lane() ^ mask); }
template <class T> T __shfl_up(T x, int n) { return emu::from(x, emu::lane() < n ? emu::lane() : emu::lane() - n); }
inline unsigned long long __ballot(int p) {
  const char *all = static_cast<const char *>(emu::exchange(&p, sizeof p));
  unsigned long long mask = 0;
  for (int i = 0; i < 64; ++i) {
    int q;
    memcpy(&q, all + 64 * i, sizeof q);
    if (q) mask |= 1ull << i;
  }
  return mask & emu::live();
}
inline int __any(int p) { return __ballot(p) != 0; }

#define __builtin_amdgcn_update_dpp(old, src, ctrl, rows, banks, bound) emu::update_dpp(old, src, ctrl, rows)
#define __builtin_amdgcn_readlane(x, l) emu::from((int)(x), l)
#define __builtin_amdgcn_readfirstlane(x) emu::from((int)(x), __builtin_ctzll(emu::live()))
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_permlane16_swap(x, y, a, b) emu::swap_halves(x, y, 16)
#define __builtin_amdgcn_permlane32_swap(x, y, a, b) emu::swap_halves(x, y, 32)
inline uint32_t __builtin_amdgcn_mbcnt_lo(uint32_t mask, uint32_t c) {
  return c + __builtin_popcount(emu::lane() < 32 ? mask & ((1u << emu::lane()) - 1u) : mask);
}
inline uint32_t __builtin_amdgcn_mbcnt_hi(uint32_t mask, uint32_t c) {
  return c + (emu::lane() < 32 ? 0 : __builtin_popcount(mask & ((1u << (emu::lane() - 32)) - 1u)));
}
inline uint32_t __builtin_amdgcn_perm(uint32_t hi, uint32_t lo, uint32_t sel) {
  const uint64_t both = (uint64_t)hi << 32 | lo;
  uint32_t out = 0;
  for (int i = 0; i < 4; ++i) out |= (uint32_t)(both >> (8 * ((sel >> (8 * i)) & 7)) & 0xff) << (8 * i);
  return out;
}
template <class V, class F> F mfma_16x16x32(const V &x, const V &y, F acc) {
  F out;
  emu::mfma_16x16x32_bf16(&x, &y, reinterpret_cast<const float *>(&acc), reinterpret_cast<float *>(&out));
  return out;
}
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, acc, a, b, c) mfma_16x16x32(x, y, acc)

#endif
