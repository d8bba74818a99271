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

// One of the floats behind `base`, at `index` (per lane) behind byte `at` (uniform): a buffer load of stride four,
// which scales the index itself.  With a global load the shift is a vector instruction a brick, which costs tiles of up
// to 64 columns, whose loop has few others (see values_by_index).  The wider tiles gain nothing, and a graph at N = 128
// lost 8 %.
typedef int int4_t __attribute__((ext_vector_type(4)));
extern "C" __device__ float spmm_load_indexed(int4_t buffer, int index, int offset, int at, int aux) __asm(
    "llvm.amdgcn.struct.buffer.load.f32");
__device__ inline int4_t float_buffer(const float* base) {
  const uint64_t a = (uint64_t)base;
  return int4_t{(int)(uint32_t)a, (int)((uint32_t)(a >> 32) | 4u << 16), -1 /* indexes */, 0x00027000};
}

// Workgroups are handed to the 8 XCDs round-robin, and each XCD has its own L2.  This maps a
// workgroup to a "virtual" index such that each XCD works through a contiguous range of work
// items: neighbouring panels -- which share most of their B rows in banded matrices -- then
// meet in one L2 instead of every XCD fetching every B row.  gridDim.x is a multiple of 8.
__device__ inline uint32_t xcd_contiguous_block() {
  const uint32_t per_xcd = gridDim.x / kXcds;
  return (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
}

// A WorkSource as the kernels take it.  The items are mapped to the XCDs as xcd_contiguous_block does; the
// parts of split panels come behind them, dealt to the XCDs in turn: they fill the time in which the last
// panels end (a graph of 20,360 panels of which 184 are split, N = 128: parts in their panels' places
// 117.2 us, in front 118.1, behind 115.6).
struct ItemMap {
  uint32_t n_items, per_xcd;        // items, and their workgroups on each XCD
  uint32_t n_parts, split_bricks;
  const WorkItem *items, *parts;
};

template <int kPer>
inline uint32_t xcd_rounds(uint32_t n) { return ((n + kPer - 1) / kPer + kXcds - 1) / kXcds; }

template <int kPer>
inline unsigned item_blocks(const WorkSource& w) {
  return (xcd_rounds<kPer>(w.n_items) + xcd_rounds<kPer>(w.n_parts)) * kXcds;
}

// As kernel parameters: scalars and not the struct, and in front, because a wavefront waits for these first
// and the build has the leading ones in registers when it starts (-amdgpu-kernarg-preload-count).  Read
// from memory they are a round trip before panel_ptr: 6250 panels of 40 bricks 31.2 -> 31.5 us.
#define SPMM_ITEM_PARAMS                                                                        \
  uint32_t n_items, uint32_t per_xcd, uint32_t n_parts, uint32_t split_bricks,                  \
      const WorkItem *__restrict__ items, const WorkItem *__restrict__ parts
#define SPMM_ITEM_MAP \
  ItemMap { n_items, per_xcd, n_parts, split_bricks, items, parts }
#define SPMM_ITEM_ARGS(PER, w) \
  (w).n_items, xcd_rounds<PER>((w).n_items), (w).n_parts, (w).split_bricks, (w).items, (w).parts

// The item of wavefront (or workgroup, kPer = 1) `wave` of this workgroup; false: none.  Without a list
// a panel's bricks come from panel_ptr, 8 bytes instead of 16, and no list has to be built, copied and
// kept (262,144 rows: plan, product at N = 128 and destruction 351 us with a list, 284 without; a graph
// of 20,360 panels of which 184 are split 332 with a list of all items, 286 with one of the parts).
template <int kPer>
__device__ inline bool work_item(const ItemMap& m, const uint32_t* panel_ptr, uint32_t wave, WorkItem* it) {
  const uint32_t whole = m.per_xcd * kXcds;   // workgroups of the items
  const bool part = blockIdx.x >= whole;
  const uint32_t block = part ? blockIdx.x - whole : (blockIdx.x % kXcds) * m.per_xcd + blockIdx.x / kXcds;
  const uint32_t id = block * kPer + wave;
  if (__builtin_expect(id >= (part ? m.n_parts : m.n_items), 0)) return false;
  const WorkItem* list = part ? m.parts : m.items;
  // (the loads of begin and end stand behind the branch, and the test for a split panel is no branch, so
  // that nothing which follows waits for them: a split panel has nothing to multiply and, as a panel behind
  // the last row, nothing to store)
  const uint32_t *begin = panel_ptr + id, *end = begin + 1;
  uint32_t panel = id, slot = kNoSlot, split = m.split_bricks;
  if (list) {
    begin = &list[id].brick_begin;
    end = &list[id].brick_end;
    panel = list[id].panel;
    slot = list[id].slot;
    split = kNoSplit;
  }
  const uint32_t b = *begin, e = *end;
  const bool is_whole = e - b < split;
  *it = WorkItem{is_whole ? panel : kNoPanel, b, is_whole ? e : b, slot};
  return true;
}

// Whether values are loaded by index (spmm_load_indexed).  It saves an instruction a brick, but a wavefront's first
// bricks arrive later, so panels have to have as many bricks as each width wants, and SIMDs at least 3.5 wavefronts, of
// which others hide it.  us, shift / index; matrices of even panels, 12 entries a brick, the columns in a band or anywhere:
//   16 columns: from 64 bricks a panel, and from 44 with more than 5 wavefronts a SIMD.  4 a SIMD, band, 44 bricks 8.03 / 8.19, 64
//     10.51 / 10.51, 80 12.56 / 12.47; 5 a SIMD, 44 bricks 9.13 / 9.26; 5.5, 10.39 / 10.40, anywhere 12.18 / 11.96; 8, 13.91 / 13.52,
//     160 bricks 49.8 / 47.4; 24 a SIMD, 44 bricks 37.2 / 36.0, anywhere 51.2 / 51.1.
//   32 columns: from 20 bricks.  Blocks of 15 bricks, 8 a SIMD 8.93 / 9.10, of 22, 16 a SIMD 21.69 / 21.61, of 29 26.92 / 26.44;
//     64 bricks, 4 a SIMD 14.63 / 14.28, anywhere 16.50 / 16.31; 12 a SIMD 40.05 / 39.00, anywhere 62.2 / 61.9.
//   48 columns: from 64 bricks.  Blocks of 32, 8 a SIMD 21.72 / 21.85, 44 bricks, 10 a SIMD 30.05 / 30.87; 64 bricks, 4 a SIMD 18.23 /
//     17.91, 8 34.02 / 33.64, anywhere 54.1 / 54.5; 16 a SIMD 62.6 / 61.3; 80 bricks, 8 a SIMD, anywhere 66.2 / 65.0.
//   64 columns: from 64 bricks, as long as all wavefronts are resident: the kernel with the index takes 60 vector registers and
//     a SIMD holds six, the other 62 and five.  64 bricks, 4 a SIMD 21.82 / 21.84, anywhere 26.8 / 25.0; 5.5 32.2 / 30.9, 46.5 / 45.2; 6.0
//     32.6 / 31.2, 50.5 / 48.1; 6.05 35.8 / 36.9, 53.0 / 53.1; 8 41.1 / 43.5, 71.3 / 72.7; 12 64.0 / 63.8, 118.2 / 119.2.
//     With several tiles of 64 a panel beyond that, too (anywhere, 10 to 16 a SIMD, N = 128 to 256: 64 bricks 0.95 to 1.02 of
//     the time, 120 0.95 to 1.00; 3500 panels of 120, N = 160 120.6 / 115.3).
// Fewer wavefronts a SIMD (cells of 75 bricks): 1, N = 16 9.06 / 9.34, N = 32 9.94 / 10.2; 2 of 64 columns 12.3 / 12.7; 3, N = 16
// 12.1 / 12.2, N = 64 22.5 / 23.0.
inline bool values_by_index(const WorkSource& w, int tile, int64_t tiles) {
  const int64_t waves = tiles * ((int64_t)w.n_items + w.n_parts);
  const int64_t least = tile == 32 ? 20 : tile == 16 && waves > 5 * (int64_t)w.simds ? 44 : 64;
  return w.mean_bricks() >= least && 2 * waves >= 7 * (int64_t)w.simds && (tile != 64 || tiles > 1 || waves <= 6 * (int64_t)w.simds);
}

constexpr int64_t kNarrowLargeB = int64_t(64) << 20;

// Workgroups of one wavefront, for graphs (scattered, one panel in 512 and more of them split) where B is large: their
// panels differ so much that the slots of a workgroup's first wavefronts stay empty until the last one ends.  us, four /
// one, each product with a B of its own: graphs of 326 k and 800 k rows, N = 64 60.5 / 58.7 and 143.5 / 138.2, N = 96 88.6 / 86.8 and
// 212 / 208, N = 112 109 / 106 and 260 / 255, N = 128 113.8 / 109.8 and 273 / 262, N = 256 216 / 213 and 558 / 535; narrower ones of
// 400 k and 1.05 M rows, N = 32 45.0 / 43.7 and 101.8 / 96.3, N = 16 (the latter) 80.7 / 80.4; 60 k rows, N = 384 66.2 / 63.7.  With
// one B for all products, from the Infinity Cache where it fits, four wavefronts are 1 to 5 % ahead there (326 k rows, N = 64
// 53.4 / 55.2, N = 128 102.1 / 105.0), and behind as ever beyond (N = 384 323 / 311).
// Tiles of 48 and 80 columns keep four, new B / one B: 326 k rows, N = 80 83.7 / 83.0 and 78.1 / 78.9; 500 k, N = 48 83.1 / 83.1
// and 78.4 / 79.0; 1.05 M, N = 48 163.6 / 165.7 and 154 / 159, N = 80 261.9 / 261.3 and 259.7 / 258.8.
// Even panels keep four, whether some are long or not: 400 k rows of blocks, N = 128 181 / 184, with one full row 270 / 272,
// with two 285 / 293, with 200 of 3000 entries 255 / 264, 800 k rows, N = 32 and one full row 187 / 191; only where the
// long rows are a quarter of the matrix and more either may win by far (350 k rows, 16 full ones, N = 128 541 / 602, N = 256
// 1143 / 922).  Cells of 600 k rows with one long row 209 / 212, with 30 215 / 220, with 300 278 / 268.
inline bool single_waves(const WorkSource& w, int tile, int64_t N, int64_t K) {
  return tile != 48 && tile != 80 && w.scattered && w.n_split > 0 && 512 * w.n_split >= w.panels && K * N * 4 >= kNarrowLargeB;
}

inline bool ptr_aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

}  // namespace spmm
