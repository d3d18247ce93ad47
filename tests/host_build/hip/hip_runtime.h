// What the kernels' sources need of the HIP language and runtime, for a build that runs them on the host: the threads of a
// workgroup are fibers of one thread, barriers and wave operations are their meeting points, LDS is an array that ends at a page
// nobody may touch, and a buffer descriptor is a base and a length.  Matrix instructions return their accumulator: this build
// checks which memory the kernels touch, not what they compute.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define __align__(n) __attribute__((aligned(n)))
#define __expf(x) expf(x)

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct alignas(8) float2 { float x, y; };
struct alignas(16) float4 { float x, y, z, w; };
struct alignas(8) int2 { int x, y; };
struct alignas(8) uint2 { unsigned x, y; };
struct alignas(16) uint4 { unsigned x, y, z, w; };
static inline float4 make_float4(float a, float b, float c, float d) { return {a, b, c, d}; }
static inline float2 make_float2(float a, float b) { return {a, b}; }
static inline int2 make_int2(int a, int b) { return {a, b}; }
static inline uint2 make_uint2(unsigned a, unsigned b) { return {a, b}; }
static inline uint4 make_uint4(unsigned a, unsigned b, unsigned c, unsigned d) { return {a, b, c, d}; }
using std::max;
using std::min;
static inline unsigned __float_as_uint(float f) { unsigned u; memcpy(&u, &f, 4); return u; }
static inline float __uint_as_float(unsigned u) { float f; memcpy(&f, &u, 4); return f; }
static inline int __float_as_int(float v) { int u; memcpy(&u, &v, 4); return u; }
static inline float __int_as_float(int u) { float v; memcpy(&v, &u, 4); return v; }
static inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
static inline int __popc(unsigned v) { return __builtin_popcount(v); }
static inline unsigned __umulhi(unsigned a, unsigned b) { return (unsigned)(((unsigned long long)a * b) >> 32); }

namespace host {
struct Fiber {
  void* sp;
  int state, lane;
  dim3 tid;
  int kind, arg;           // wave operation the fiber waits in
  uint64_t value, result;
};
extern Fiber* current;
extern dim3 block, grid, block_size;
extern unsigned char* lds;  // dynamic LDS of the launch
void barrier();
enum { BALLOT, XOR, UP, FROM };
uint64_t wave_op(int kind, uint64_t value, int arg);
template <typename T>
T shuffle(int kind, T v, int arg) {
  uint64_t u = 0;
  memcpy(&u, &v, sizeof(T));
  u = wave_op(kind, u, arg);
  memcpy(&v, &u, sizeof(T));
  return v;
}
void request_lds(const void* function, int bytes);
void launch(dim3 grid, dim3 block, size_t lds_bytes, const char* kernel, const void* function, const std::function<void()>& body);

struct Rsrc { const char* base; unsigned bytes; };
typedef unsigned Chunk __attribute__((ext_vector_type(4)));
unsigned load_dword(const Rsrc& r, unsigned voff, unsigned soff);  // zero past the descriptor's end
uint8_t load_byte(const Rsrc& r, unsigned voff, unsigned soff);
Chunk load_chunk(const Rsrc& r, unsigned voff, unsigned soff);
void store_chunk(const Chunk& c, const Rsrc& r, unsigned voff, unsigned soff);  // dropped past the descriptor's end
void load_to_lds(const Rsrc& r, unsigned voff, unsigned soff, unsigned lds_base);
void load_dword_to_lds(const Rsrc& r, unsigned voff, unsigned soff, unsigned lds_base);
struct Pair {
  unsigned v[2];
  unsigned operator[](int i) const { return v[i]; }
};
static inline int lanes_below(unsigned mask, int first) {  // set bits of 32 lanes from `first` on, below the calling lane
  const int n = std::min(std::max(current->lane - first, 0), 32);
  return __builtin_popcount(n < 32 ? mask & ((1u << n) - 1) : mask);
}
}  // namespace host

#define threadIdx (host::current->tid)
#define blockIdx (host::block)
#define gridDim (host::grid)
#define blockDim (host::block_size)
#define __syncthreads() host::barrier()
#define __ballot(p) ((unsigned long long)host::wave_op(host::BALLOT, (p) ? 1 : 0, 0))
#define __shfl_xor(v, o, w) host::shuffle(host::XOR, v, o)
#define __shfl_up(v, o, w) host::shuffle(host::UP, v, o)
#define __shfl(v, l, w) host::shuffle(host::FROM, v, l)
// (rotations of the rows of sixteen lanes only)
#define __builtin_amdgcn_mov_dpp(v, c, r, b, z) host::shuffle(host::FROM, v, (host::current->lane & 48) | ((host::current->lane - ((c) - 0x120)) & 15))
#define __amdgpu_buffer_rsrc_t host::Rsrc
#define __builtin_amdgcn_make_buffer_rsrc(p, stride, bytes, flags) (host::Rsrc{(const char*)(p), (unsigned)(bytes)})
#define __builtin_amdgcn_raw_buffer_load_b128(r, v, s, a) host::load_chunk(r, v, s)
#define __builtin_amdgcn_raw_buffer_store_b128(c, r, v, s, a) host::store_chunk(c, r, v, s)
#define __builtin_amdgcn_raw_buffer_load_b8(r, v, s, a) host::load_byte(r, v, s)
#define __builtin_amdgcn_raw_buffer_load_b32(r, v, s, a) host::load_dword(r, v, s)
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_permlane32_swap(a, b, c, d) (host::Pair{{a, b}})
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sched_barrier(x)
#define __builtin_amdgcn_s_setprio(x)
#define __builtin_amdgcn_mbcnt_lo(m, v) ((v) + host::lanes_below(m, 0))
#define __builtin_amdgcn_mbcnt_hi(m, v) ((v) + host::lanes_below(m, 32))

typedef void* hipStream_t;
typedef void* hipEvent_t;
enum { hipSuccess = 0, hipFuncAttributeMaxDynamicSharedMemorySize, hipDeviceAttributeMultiprocessorCount };
static inline int hipGetDevice(int* d) { *d = 0; return 0; }
static inline int hipFuncSetAttribute(const void* f, int, int v) { host::request_lds(f, v); return 0; }
static inline int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
static inline int hipGetLastError() { return 0; }
static inline int hipEventCreate(hipEvent_t* e) { *e = nullptr; return 0; }
static inline int hipEventRecord(hipEvent_t, hipStream_t) { return 0; }
static inline int hipEventSynchronize(hipEvent_t) { return 0; }
static inline int hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return 0; }
static inline int hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return 0; }
#define HIP_SYMBOL(x) ((const void*)&x)
#define hipLaunchKernelGGL(k, g, b, bytes, stream, ...) host::launch(g, b, bytes, #k, reinterpret_cast<const void*>(k), [=] { (k)(__VA_ARGS__); })
