// Small helpers shared by the SpMM kernels (device code only).
#pragma once
#include "spmm_internal.h"

namespace spmm {

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float2_t __attribute__((ext_vector_type(2)));

constexpr int kWavesPerBlock = 4;
constexpr int kXcds = 8;     // accelerator complex dies of an MI355X, each with its own L2

template <int V> struct Vec;
template <> struct Vec<1> { typedef float type; };
template <> struct Vec<2> { typedef float2_t type; };
template <> struct Vec<4> { typedef float4_t type; };

template <int V>
__device__ inline void load_vec(const float* __restrict__ p, float (&out)[V]) {
  typedef typename Vec<V>::type vt;
  const vt v = *reinterpret_cast<const vt*>(p);
  if constexpr (V == 1) out[0] = v;
  else {
#pragma unroll
    for (int w = 0; w < V; ++w) out[w] = v[w];
  }
}

template <int V>
__device__ inline void store_vec(float* __restrict__ p, const float (&in)[V]) {
  typedef typename Vec<V>::type vt;
  vt v;
  if constexpr (V == 1) v = in[0];
  else {
#pragma unroll
    for (int w = 0; w < V; ++w) v[w] = in[w];
  }
  *reinterpret_cast<vt*>(p) = v;
}

// V consecutive floats at a 4-byte aligned address, V = 1..4: one global load or store of V dwords,
// which gfx950 does at any dword address (V = 3 through a struct: a three-element vector type
// would be widened to four elements and touch memory behind the last one).
template <int V> struct AnyVec { typedef float type __attribute__((ext_vector_type(V), aligned(4))); };
template <> struct AnyVec<1> { typedef float type; };

template <int V>
__device__ inline void load_any(const char* __restrict__ p, float* out) {
  if constexpr (V == 3) {
    struct F3 { float x, y, z; };
    const F3 t = *reinterpret_cast<const F3*>(p);
    out[0] = t.x; out[1] = t.y; out[2] = t.z;
  } else {
    const typename AnyVec<V>::type t = *reinterpret_cast<const typename AnyVec<V>::type*>(p);
    if constexpr (V == 1) out[0] = t;
    else {
#pragma unroll
      for (int w = 0; w < V; ++w) out[w] = t[w];
    }
  }
}

template <int V>
__device__ inline void store_any_nt(float* __restrict__ p, const float* in) {
  if constexpr (V == 3) {
#pragma unroll
    for (int w = 0; w < 3; ++w) __builtin_nontemporal_store(in[w], p + w);
  } else {
    typename AnyVec<V>::type t;
    if constexpr (V == 1) t = in[0];
    else {
#pragma unroll
      for (int w = 0; w < V; ++w) t[w] = in[w];
    }
    __builtin_nontemporal_store(t, reinterpret_cast<typename AnyVec<V>::type*>(p));
  }
}

// Work item `id` of a list, or, without one (every panel whole, in order), panel `id` itself: its
// bricks come from panel_ptr, 8 bytes instead of 16, and no list has to be built, copied and kept.
// With a list and without, 262,144 rows: plan, product (N = 128) and destruction 351 and 284 us, the
// first product of a new width (N = 124) 203 and 151; a 4096-row band, N = 32, without allocation 11.5
// and 8.4.
__device__ inline WorkItem work_item(const WorkItem* __restrict__ items,
                                     const uint32_t* __restrict__ panel_ptr, int64_t id) {
  if (items) return items[id];
  return WorkItem{(uint32_t)id, panel_ptr[id], panel_ptr[id + 1], kNoSlot};
}

// Workgroups are handed to the 8 XCDs round-robin, and each XCD has its own L2.  This maps a
// workgroup to a "virtual" index such that each XCD works through a contiguous range of work
// items: neighbouring panels -- which share most of their B rows in banded matrices -- then
// meet in one L2 instead of every XCD fetching every B row.  gridDim.x is a multiple of 8.
__device__ inline uint32_t xcd_contiguous_block() {
  const uint32_t per_xcd = gridDim.x / kXcds;
  return (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
}

inline bool ptr_aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace spmm
