// Stand-in for the HIP runtime header that lets the resident kernels' headers
// compile for the host: a workgroup's lanes run as fibers, one wave at a time.
//
// The waves of a workgroup run one after the other between two barriers, in an
// order that the caller chooses (sim::order).  Two waves that touch the same LDS word
// between the same two barriers therefore give another result in one of the
// orders, where the GPU's timing may hide it.  Buffer accesses are checked
// against the resource's range (as the hardware does) and against the tensors
// that the caller named (sim::allow).
#pragma once

#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <utility>
#include <vector>

#define __device__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define __restrict__ __restrict
#define asm(...)

struct float2 { float x, y; };
struct float4 { float x, y, z, w; };
struct uint2 { unsigned x, y; };
struct uint4 { unsigned x, y, z, w; };
inline float2 make_float2(float a, float b) { return {a, b}; }
inline float4 make_float4(float a, float b, float c, float d) { return {a, b, c, d}; }
inline uint2 make_uint2(unsigned a, unsigned b) { return {a, b}; }
inline uint4 make_uint4(unsigned a, unsigned b, unsigned c, unsigned d) { return {a, b, c, d}; }
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
using std::max;
using std::min;

typedef void* hipStream_t;
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorInvalidConfiguration = 9 };
enum { hipFuncAttributeMaxDynamicSharedMemorySize = 8 };
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount };
template <typename... A>
hipError_t hipFuncSetAttribute(A...) { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }

namespace sim {

constexpr int kLdsBytes = 160 * 1024, kGuard = 4096;
constexpr size_t kStack = 512 * 1024;

[[noreturn]] inline void fail(const char* what) {
  std::fprintf(stderr, "wave model: %s\n", what);
  std::abort();
}

// ---- memory ---------------------------------------------------------------
struct Range { const char *lo, *hi; };
inline std::vector<Range> allowed;
inline void allow(const void* p, size_t bytes) {
  if (p) allowed.push_back({(const char*)p, (const char*)p + bytes});
}
struct Rsrc {
  char* base;
  uint32_t bytes;
  // the address of `size` bytes at the offsets, null where out of range
  char* at(int voff, int soff, int size) const {
    const uint64_t o = (uint64_t)(uint32_t)voff + (uint32_t)soff;
    if (o + size > bytes) return nullptr;
    for (const Range& r : allowed)
      if (base + o >= r.lo && base + o + size <= r.hi) return base + o;
    fail("access outside the tensors");
  }
};
template <typename W>
W load(const Rsrc& r, int voff, int soff) {
  W v{};
  if (const char* p = r.at(voff, soff, sizeof(W))) std::memcpy(&v, p, sizeof(W));
  return v;
}
template <typename W>
void store(W v, const Rsrc& r, int voff, int soff) {
  if (char* p = r.at(voff, soff, sizeof(W))) std::memcpy(p, &v, sizeof(W));
}

// ---- lanes and waves ------------------------------------------------------
enum Stop { kShift, kBarrier, kEnd };
struct Lane {
  ucontext_t ctx;
  Stop stop;
  int shifts;
};
inline std::vector<Lane> lanes;
inline ucontext_t home;
inline int cur;                       // the running lane
inline int waves;
inline std::vector<int> order;        // waves in the order in which they run between barriers
inline uint32_t slots[16][2][64];     // values of the lanes of a wave, for the shifts
inline const std::function<void()>* body;
inline std::vector<uint64_t> grids;   // work items of every launch
inline hipError_t last_error = hipSuccess;
inline bool dry;                      // record launches, run nothing

inline void stop_at(Stop s) {
  lanes[cur].stop = s;
  swapcontext(&lanes[cur].ctx, &home);
}
inline uint32_t shifted(uint32_t v, uint32_t none, int ctrl) {
  Lane& l = lanes[cur];
  uint32_t(&s)[64] = slots[cur >> 6][l.shifts++ & 1];
  s[cur & 63] = v;
  stop_at(kShift);
  const int from = (cur & 63) + (ctrl == 0x138 ? -1 : 1);
  return from < 0 || from > 63 ? none : s[from];
}
inline void barrier() { stop_at(kBarrier); }
inline void entry() {
  (*body)();
  stop_at(kEnd);
}

}  // namespace sim

struct SimIdx { unsigned x; };
inline SimIdx threadIdx, blockIdx;
inline dim3 blockDim, gridDim;
namespace gspn {
extern float lds[(sim::kLdsBytes + sim::kGuard) / 4];
}

namespace sim {

// Runs a wave until its lanes stop at a barrier or end.
inline Stop run_wave(int w) {
  for (;;) {
    for (int l = 64 * w; l < 64 * w + 64; ++l) {
      cur = l;
      threadIdx.x = (unsigned)l;
      swapcontext(&home, &lanes[l].ctx);
      if (lanes[l].stop != lanes[64 * w].stop) fail("lanes of a wave diverge at a shift or barrier");
    }
    if (lanes[64 * w].stop != kShift) return lanes[64 * w].stop;
  }
}

inline void run_block(int threads, size_t lds_bytes) {
  static std::vector<char> stacks;
  waves = threads / 64;
  lanes.resize(threads);
  stacks.resize(kStack * threads);
  for (size_t i = 0; i < sizeof(gspn::lds) / 4; ++i) gspn::lds[i] = i * 4 < lds_bytes ? NAN : 1.25f;
  for (int l = 0; l < threads; ++l) {
    getcontext(&lanes[l].ctx);
    lanes[l].ctx.uc_stack.ss_sp = stacks.data() + kStack * l;
    lanes[l].ctx.uc_stack.ss_size = kStack;
    lanes[l].ctx.uc_link = nullptr;
    lanes[l].shifts = 0;
    makecontext(&lanes[l].ctx, entry, 0);
  }
  std::vector<Stop> st(waves, kBarrier);
  for (int live = waves; live > 0;) {
    for (int w : order)
      if (w < waves && st[w] != kEnd && (st[w] = run_wave(w)) == kEnd) --live;
  }
  for (size_t i = (lds_bytes + 3) / 4; i < sizeof(gspn::lds) / 4; ++i)
    if (gspn::lds[i] != 1.25f) fail("store past the end of LDS");
}

inline void launch(dim3 grid, dim3 block, size_t lds_bytes, const std::function<void()>& f) {
  grids.push_back((uint64_t)grid.x * block.x);
  // a dimension's work items are counted in 32 bits (the GPU runs fewer without an error)
  if (grids.back() > 0xffffffffull || grid.x == 0) {
    last_error = hipErrorInvalidConfiguration;
    return;
  }
  if (lds_bytes > kLdsBytes) {
    last_error = hipErrorInvalidValue;
    return;
  }
  if (dry) return;
  body = &f;
  blockDim = block;
  gridDim = grid;
  for (unsigned b = 0; b < grid.x; ++b) {
    blockIdx.x = b;
    run_block((int)block.x, lds_bytes);
  }
}

}  // namespace sim

inline hipError_t hipGetLastError() { return std::exchange(sim::last_error, hipSuccess); }
#define hipLaunchKernelGGL(k, g, b, l, s, ...) sim::launch((g), (b), (size_t)(l), [&] { (k)(__VA_ARGS__); })

// ---- device functions -----------------------------------------------------
typedef unsigned sim_u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned sim_u32x4 __attribute__((ext_vector_type(4)));
typedef sim::Rsrc __amdgpu_buffer_rsrc_t;
inline sim::Rsrc sim_rsrc(void* p, short, int bytes, int) { return {(char*)p, (uint32_t)bytes}; }
#define __builtin_amdgcn_make_buffer_rsrc sim_rsrc
#define __builtin_amdgcn_raw_buffer_load_b16(r, v, s, a) sim::load<unsigned short>(r, v, s)
#define __builtin_amdgcn_raw_buffer_load_b32(r, v, s, a) sim::load<unsigned>(r, v, s)
#define __builtin_amdgcn_raw_buffer_load_b64(r, v, s, a) sim::load<sim_u32x2>(r, v, s)
#define __builtin_amdgcn_raw_buffer_load_b128(r, v, s, a) sim::load<sim_u32x4>(r, v, s)
#define __builtin_amdgcn_raw_buffer_store_b16(d, r, v, s, a) sim::store<unsigned short>(d, r, v, s)
#define __builtin_amdgcn_raw_buffer_store_b32(d, r, v, s, a) sim::store<unsigned>(d, r, v, s)
#define __builtin_amdgcn_raw_buffer_store_b64(d, r, v, s, a) sim::store<sim_u32x2>(d, r, v, s)
#define __builtin_amdgcn_raw_buffer_store_b128(d, r, v, s, a) sim::store<sim_u32x4>(d, r, v, s)
#define __builtin_amdgcn_mov_dpp(v, c, rm, bm, bc) (int)sim::shifted((uint32_t)(v), 0, c)
#define __builtin_amdgcn_update_dpp(o, v, c, rm, bm, bc) (int)sim::shifted((uint32_t)(v), (uint32_t)(o), c)
#define __builtin_amdgcn_readfirstlane(v) (int)(v)
#define __builtin_amdgcn_sched_barrier(m) (void)0
#define __builtin_amdgcn_alignbit(h, l, n) (uint32_t)((((uint64_t)(h) << 32) | (l)) >> (n))
#define __builtin_amdgcn_rcpf(v) (1.f / (v))
inline float __expf(float v) { return std::exp(v); }
inline float __uint_as_float(uint32_t v) { return __builtin_bit_cast(float, v); }
inline uint32_t __float_as_uint(float v) { return __builtin_bit_cast(uint32_t, v); }
inline void __syncthreads() { sim::barrier(); }
