// Brick kernel for tiles of 16 and 32 columns: T = 1 or 2 MFMAs a brick, work item and decode as in
// k_spmm_mfma_fast, another way to read B.
//
// A CU's L1 takes a load four lanes a clock, whatever a lane asks for: 16 clocks for a wave's dword, eight
// or sixteen bytes alike.  With T columns a lane (four or eight bytes) a brick of these tiles cost it as much as one
// of four times the width, and that, not bytes or MFMAs, bounded them.  Here a lane loads sixteen bytes always: 4T
// lanes hold a row of the tile, so one load holds the rows of G = 4/T bricks, and lane groups and registers then
// change places (T = 2: eight lanes; T = 1: eight, then four) until register (brick, column) holds the four rows
// of one brick in the MFMA's layout.  Column u of lane l's MFMA is then column 4*j + T*s + u of the tile, where
// l % 16 = 4T*s + j.  923,136 rows of blocks, N = 32, products one after another: accesses to L1 85 M -> 52 M,
// 213.7 -> 180.4 us (the first hundred after an idle time take 195 to 290, so traces of short runs show more); L1
// now takes accesses for 0.47 of the time and waits for lines from L2 for 0.48.  There is room for 8 wavefronts a
// SIMD (50 vector, 98 scalar registers); a launch bound that asks for 8 makes the compiler keep to 80 scalar
// registers and spill as many again: 184.9.  At most 5 wavefronts 185.9; fetching half a chunk at an item's end
// (more code, spilled scalars) 181.8.
//
// Wider C of few panels takes several such tiles (mfma_run_tile): MANY, as a first column that is not known cost short
// panels of one tile 1 % (310,036 rows, 3 a row, N = 17 16.3 / 16.5 us).
//
// A chunk of eight bricks is in flight while it is multiplied load by load, and each load's registers take
// the next chunk's.  The last chunk is fetched behind tests for what is left, so that items of ten bricks do not
// read eight more.
#include "exec_common.h"

#include <type_traits>

namespace spmm {
namespace {

constexpr int kNarrowChunk = 8;   // bricks in flight per wavefront

// lanes 8..15 of every 16 of `a` change places with lanes 0..7 of `c`
__device__ inline void swap_eights(float& a, float& c) {
  const int x = __builtin_bit_cast(int, a), y = __builtin_bit_cast(int, c);
  a = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, y, 0x128 /* row_ror:8 */, 0xF, 0xC, false));
  c = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(y, x, 0x128, 0xF, 0x3, false));
}
// lanes 4..7 of every 8 of `a` change places with lanes 0..3 of `c`
__device__ inline void swap_fours(float& a, float& c) {
  const int x = __builtin_bit_cast(int, a), y = __builtin_bit_cast(int, c);
  a = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, y, 0x114 /* row_shr:4 */, 0xF, 0xA, false));
  c = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(y, x, 0x104 /* row_shl:4 */, 0xF, 0x5, false));
}

template <int T, bool IDX, bool MANY, int WPB>
__global__ __launch_bounds__(64 * WPB, T == 2 ? 4 : 1) void k_spmm_mfma_narrow(
    SPMM_ITEM_PARAMS, const uint32_t* __restrict__ panel_ptr, const uint32_t* __restrict__ brick_cols,
    const uint64_t* __restrict__ brick_mask, const uint32_t* __restrict__ brick_valptr,
    const float* __restrict__ vals, const float* __restrict__ B, float* __restrict__ C,
    float* __restrict__ partial, int64_t M, int64_t N, uint32_t k_last) {
  constexpr int CH = kNarrowChunk;
  constexpr int G = 4 / T;          // bricks of a load
  constexpr int NG = CH / G;        // loads of a chunk
  const int lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  WorkItem it;
  if (!work_item<WPB>(SPMM_ITEM_MAP, panel_ptr, wave, &it))
    return;  // whole wavefront leaves together
  const uint32_t panel = it.panel, b_begin = it.brick_begin, b_end = it.brick_end, slot = it.slot;

  const int kq = lane >> 4;
  const uint32_t j = lane & (4 * T - 1);             // vector of a B row
  const uint32_t in_load = (lane & 15) / (4 * T);    // brick of a load
  const uint32_t perm_transpose = 4u * (uint32_t)(4 * (lane & 15) + kq);
  const uint32_t perm_base = 4u * (4u * in_load + kq);
  const uint32_t row_bytes = (uint32_t)N * 4u;
  const uint32_t col0 = (MANY ? blockIdx.y * (16u * T) : 0u) + 4u * j;
  const uint32_t at = min(col0, (uint32_t)N - 4u);
  const uint32_t lane_off = at * 4u;

  float4_t acc[T];
#pragma unroll
  for (int u = 0; u < T; ++u) acc[u] = float4_t{0.f, 0.f, 0.f, 0.f};

  if (b_begin < b_end) {
    const uint32_t nbricks = b_end - b_begin;
    const char* Bbytes = reinterpret_cast<const char*>(B);
    [[maybe_unused]] const int4_t vals_at = float_buffer(vals);
    struct Meta { uint64_t mask[CH]; uint32_t off[CH]; };
    auto load_meta = [&](uint32_t base) {
      const uint64_t* __restrict__ mp = brick_mask + base;
      const uint32_t* __restrict__ op = brick_valptr + base;
      Meta m;
#pragma unroll
      for (int i = 0; i < CH; ++i) { m.mask[i] = mp[i]; m.off[i] = op[i]; }
      return m;
    };
    auto load_col = [&](uint32_t base) {
      const uint32_t s = (uint32_t)lane & (CH * kBrickK - 1);
      const uint32_t idx = min(base * kBrickK + s, (b_end - 1) * kBrickK + (s & (kBrickK - 1)));
      return brick_cols[idx];
    };
    auto row_offset = [&](uint32_t col) { return min(col, k_last) * row_bytes; };

    uint64_t st_mask[CH];
    float st_a[CH];
    float st_b[NG][4];
    auto issue_value = [&](uint64_t mask, uint32_t off, int i) {
      st_mask[i] = mask;
      const uint32_t cnt = __builtin_amdgcn_mbcnt_hi(
          (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
      if constexpr (IDX) st_a[i] = spmm_load_indexed(vals_at, (int)cnt, 0, (int)(off * 4u), 0);
      else
        st_a[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(vals) + (off * 4u + cnt * 4u));
    };
    auto rows_of = [&](uint32_t ro, int q) {
      return (uint32_t)__builtin_amdgcn_ds_bpermute(perm_base + 16u * G * q, ro);
    };
    auto issue_rows = [&](uint32_t ro, int q) {
      load_any<4>(Bbytes + (ro + lane_off), st_b[q]);
    };
    auto operand = [&](int i) {
      float in_bit_order;
      asm("v_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(in_bit_order) : "v"(st_a[i]), "s"(st_mask[i]));
      return __builtin_bit_cast(
          float, __builtin_amdgcn_ds_bpermute(perm_transpose, __builtin_bit_cast(int, in_bit_order)));
    };
    // register w of a load: B[row of brick `in_load`][at + w] -> register of (brick, column)
    auto turn = [&](int q) {
      swap_eights(st_b[q][0], st_b[q][2]);
      swap_eights(st_b[q][1], st_b[q][3]);
      if constexpr (T == 1) {
        swap_fours(st_b[q][0], st_b[q][1]);
        swap_fours(st_b[q][2], st_b[q][3]);
      }
    };
    auto multiply = [&](float a, int q, int s) {
#pragma unroll
      for (int u = 0; u < T; ++u)
        acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, st_b[q][T * s + u], acc[u], 0, 0, 0);
    };

    Meta nxt = load_meta(b_begin);
    const uint32_t col_first = load_col(b_begin), col_second = load_col(b_begin + CH);
    Meta second = load_meta(b_begin + CH);   // (what it reads behind a short item is not used)
    uint32_t ro = row_offset(col_first);
    const uint32_t off_last = brick_valptr[b_end - 1];
    // One chunk: multiplies what is in flight (kCompute; kPartial: `live` bricks of it) and fetches the next
    // (kFetch 1: all of it, 2: `left` bricks; those of a load that are none take a pattern of zeros).
    auto chunk = [&](auto compute, auto fetch, uint32_t live, uint32_t left) {
      constexpr bool kCompute = decltype(compute)::value != 0, kPartial = decltype(compute)::value == 2;
      constexpr int kFetch = decltype(fetch)::value;
      float a = 0.f;
      if constexpr (kCompute) a = operand(0);
      uint32_t ro_ahead = 0;
      if constexpr (kFetch != 0) ro_ahead = rows_of(ro, 0);
#pragma unroll
      for (int q = 0; q < NG; ++q) {
        if constexpr (kCompute) {
          if (!kPartial || (uint32_t)(G * q) < live) {
            turn(q);
#pragma unroll
            for (int s = 0; s < G; ++s) {
              const float now = a;
              if (G * q + s + 1 < CH) a = operand(G * q + s + 1);
              // (zeros times the rows that stand in for no brick are NaN where those are infinite)
              if (!kPartial || (uint32_t)(G * q + s) < live) multiply(now, q, s);
            }
          }
        }
        if constexpr (kFetch != 0) {
          if (kFetch == 1 || (uint32_t)(G * q) < left) {
            const uint32_t r = ro_ahead;
            if (q + 1 < NG) ro_ahead = rows_of(ro, q + 1);
#pragma unroll
            for (int s = 0; s < G; ++s) {
              const int i = G * q + s;
              const bool on = kFetch == 1 || (uint32_t)i < left;
              issue_value(on ? nxt.mask[i] : 0ull, on ? nxt.off[i] : off_last, i);
            }
            issue_rows(r, q);
          } else {
#pragma unroll
            for (int s = 0; s < G; ++s) st_mask[G * q + s] = 0;
          }
        }
        if constexpr (kCompute && kFetch == 1) __builtin_amdgcn_sched_barrier(0);
      }
    };
    typedef std::integral_constant<int, 0> None;
    typedef std::integral_constant<int, 1> Whole;
    typedef std::integral_constant<int, 2> Part;
#pragma unroll
    for (int i = 0; i < CH; ++i) { st_a[i] = 0.f; st_mask[i] = 0; }
#pragma unroll
    for (int q = 0; q < NG; ++q)
#pragma unroll
      for (int w = 0; w < 4; ++w) st_b[q][w] = 0.f;
    if (nbricks >= (uint32_t)CH) chunk(None{}, Whole{}, 0, CH);
    else chunk(None{}, Part{}, 0, nbricks);
    uint32_t c = 0;   // first brick in flight
    if (nbricks > (uint32_t)CH) {
      nxt = second;
      ro = row_offset(col_second);
      asm volatile("" : "+v"(ro));
#pragma unroll
      for (int i = 0; i < CH; ++i) asm volatile("" : "+s"(nxt.mask[i]), "+s"(nxt.off[i]));
      for (; c + 2 * CH <= nbricks; c += CH) {
        const Meta fol = load_meta(b_begin + c + 2 * CH);
        const uint32_t col_fol = load_col(b_begin + c + 2 * CH);
        chunk(Whole{}, Whole{}, CH, CH);
        nxt = fol;
        ro = row_offset(col_fol);
      }
      if (c + CH < nbricks) {
        chunk(Whole{}, Part{}, CH, nbricks - c - CH);
        c += CH;
      }
    }
    chunk(Part{}, None{}, nbricks - c, 0);
  }

  float* out;
  int64_t rows_left;
  if (slot == kNoSlot) {
    const int64_t row0 = (int64_t)panel * kPanel + 4 * kq;
    out = C + row0 * N;
    rows_left = M - row0;
  } else {
    out = partial + ((int64_t)slot * kPanel + 4 * kq) * N;
    rows_left = 4;
  }
  if (col0 < (uint32_t)N) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (v < rows_left) {
        float t[T];
#pragma unroll
        for (int u = 0; u < T; ++u) t[u] = acc[u][v];
        store_any_nt<T>(out + v * N + at + T * in_load, t);
      }
    }
  }
}

}  // namespace

hipError_t launch_spmm_mfma_narrow(const BrickFormat& f, const WorkSource& w, int tile, const float* B, float* C,
                                   float* partial, int64_t M, int64_t N, int64_t K, hipStream_t s) {
  const unsigned gy = (unsigned)((N + tile - 1) / tile);
  const uint32_t k_last = (uint32_t)(K - 1);
#define SPMM_LAUNCH_WAVES(TT, II, MM, W)                                                        \
  hipLaunchKernelGGL((k_spmm_mfma_narrow<TT, II, MM, W>), dim3(item_blocks<W>(w), gy), dim3(64 * W), 0, s, \
                     SPMM_ITEM_ARGS(W, w), f.panel_ptr, f.brick_cols,                           \
                     f.brick_mask, f.brick_valptr, f.vals, B, C, partial, M, N, k_last)
#define SPMM_LAUNCH_NARROW(TT)                                                                  \
  do {                                                                                          \
    if (gy > 1) SPMM_LAUNCH_WAVES(TT, false, true, kWavesPerBlock);   /* too few for an index */ \
    else if (single_waves(w, tile, N, K))                                                             \
      { if (by_index) SPMM_LAUNCH_WAVES(TT, true, false, 1); else SPMM_LAUNCH_WAVES(TT, false, false, 1); } \
    else if (by_index) SPMM_LAUNCH_WAVES(TT, true, false, kWavesPerBlock);                      \
    else SPMM_LAUNCH_WAVES(TT, false, false, kWavesPerBlock);                                   \
  } while (0)
  const bool by_index = values_by_index(w, tile, gy);
  if (tile == 16) SPMM_LAUNCH_NARROW(1); else SPMM_LAUNCH_NARROW(2);
#undef SPMM_LAUNCH_NARROW
#undef SPMM_LAUNCH_WAVES
  return hipGetLastError();
}

}  // namespace spmm
