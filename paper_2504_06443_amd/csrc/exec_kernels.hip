// SpMM kernels for gfx950 (paper Section 3.3 / Algorithm 1, re-designed for
// wave64 and v_mfma_f32_16x16x4_f32).
//
// MFMA brick kernel.  One wavefront owns one work item: the bricks
// [brick_begin, brick_end) of one 16-row panel and a tile of n_tile = 16*T
// columns of C.  A 16x4 brick is exactly the A operand of the 16x16x4 MFMA:
//   A operand (1 VGPR): lane l holds A[row l%16][k = l/16]
//   B operand (1 VGPR): lane l holds B[k = l/16][col l%16]
//   D (4 VGPRs):        lane l, register v holds D[row 4*(l/16)+v][col l%16]
// so lane l expands pattern bit 4*(l%16) + l/16 (the paper numbers brick
// elements row-major): value index = popcount of the pattern below that bit,
// which is the prefix-count decode of Algorithm 1 done per lane on a
// wave-uniform mask.  Which column of the C tile an MFMA "column" stands for is
// free, so lane l loads T consecutive floats of B row brick_cols[4b + l/16]
// (dwordx4 loads, 256 contiguous bytes per 16 lanes) and feeds element u to
// MFMA u; its accumulators then hold T consecutive columns of 4 rows of C and
// are stored as dwordx4.  B therefore goes HBM/L2 -> registers directly; no
// LDS staging is needed because a B row of a panel is used by exactly one
// brick when panels are 16 rows high.
//
// Loads are software-pipelined through a ring of register stages: while the
// MFMAs of brick b issue, the values and B rows of the next kStages bricks are
// in flight; brick metadata is fetched 16 bricks at a time with coalesced loads
// and distributed by cross-lane reads.
//
// Vector-ALU CSR kernels (the paper's "scalar core" path): one B-row load and one FMA per
// stored entry, no zero filling and no reuse of B rows inside a panel.  Rows are processed
// side by side in a wavefront (k_spmm_valu_rows), very long rows by a workgroup each
// (k_spmm_valu_long); k_spmm_valu (one wavefront per row) serves widths that are not a
// multiple of four.  Used for the panels that the routing sends to the CSR path.
#include "exec_common.h"

#include <algorithm>
#include <type_traits>

namespace spmm {

int long_row_threshold() { return 256; }

int mfma_tile_for(int64_t N) { return N <= 16 ? 16 : (N <= 32 ? 32 : (N <= 64 ? 64 : 128)); }

namespace {

constexpr int kStages = 4;   // bricks whose loads are in flight per wavefront (MFMA kernel)
constexpr int kChunk = 16;   // bricks per coalesced metadata fetch
static_assert(kChunk % kStages == 0 && kChunk == 16, "stage and lane mapping assume this");

// T floats of one B row for this lane: NV vectors of V floats.
// ALIGNED: N % V == 0 and 16-byte aligned base, so a vector is entirely inside
// or entirely outside [0, N).  Columns at or beyond N are read from a clamped,
// valid address instead of being zeroed: column j of the product depends only
// on column j of B, and columns >= N of the tile are never stored.
template <int T, bool ALIGNED>
__device__ inline void load_b(const float* __restrict__ brow, int64_t N, int64_t ncol0,
                              float (&bv)[T]) {
  constexpr int V = T < 4 ? T : 4;
  constexpr int NV = T / V;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const int64_t n = ncol0 + q * 16 * V;
    if constexpr (ALIGNED) {
      float tmp[V];
      load_vec<V>(brow + min(n, N - V), tmp);
#pragma unroll
      for (int w = 0; w < V; ++w) bv[q * V + w] = tmp[w];
    } else {
#pragma unroll
      for (int w = 0; w < V; ++w) bv[q * V + w] = brow[min(n + w, N - 1)];
    }
  }
}

template <int T, bool ALIGNED>
__global__ __launch_bounds__(64 * kWavesPerBlock) void k_spmm_mfma(
    SPMM_ITEM_PARAMS, BrickFormat f, const float* __restrict__ B, float* __restrict__ C, float* __restrict__ partial, int64_t M,
    int64_t N) {
  constexpr int V = T < 4 ? T : 4;
  constexpr int NV = T / V;
  const int lane = threadIdx.x & 63;
  WorkItem it;
  if (!work_item<kWavesPerBlock>(SPMM_ITEM_MAP, f.panel_ptr, threadIdx.x >> 6, &it))
    return;  // whole wavefront leaves together
  const uint32_t panel = __builtin_amdgcn_readfirstlane(it.panel);
  const uint32_t b_begin = __builtin_amdgcn_readfirstlane(it.brick_begin);
  const uint32_t b_end = __builtin_amdgcn_readfirstlane(it.brick_end);
  const uint32_t slot = __builtin_amdgcn_readfirstlane(it.slot);

  const int j = lane & 15;   // MFMA column / brick row
  const int kq = lane >> 4;  // MFMA k / brick column
  const int bit = 4 * j + kq;
  const uint64_t below = (1ull << bit) - 1ull;
  const int64_t ncol0 = (int64_t)blockIdx.y * (16 * T) + V * j;  // first C column of this lane

  float4_t acc[T];
#pragma unroll
  for (int u = 0; u < T; ++u) acc[u] = float4_t{0.f, 0.f, 0.f, 0.f};

  if (b_begin < b_end) {
    const uint32_t last = b_end - 1;
    const uint32_t nbricks = b_end - b_begin;
    constexpr int R = kStages;   // bricks in flight per wavefront
    constexpr int CH = kChunk;   // bricks per metadata chunk

    // Metadata of CH consecutive bricks, fetched with three coalesced loads and
    // handed out per brick by cross-lane reads (no memory latency per brick):
    //   cols: lane l holds brick_cols[4*(base + l/4) + l%4]
    //   mask, off: lane l holds brick_mask / brick_valptr of brick base + l%16
    struct Chunk { uint32_t cols; uint32_t mask_lo, mask_hi; uint32_t off; };
    auto load_chunk = [&](uint32_t base) {
      const uint32_t bc = min(base + (uint32_t)(lane >> 2), last);
      const uint32_t bm = min(base + (uint32_t)(lane & (CH - 1)), last);
      const uint64_t m = f.brick_mask[bm];
      return Chunk{f.brick_cols[(int64_t)bc * kBrickK + (lane & 3)], (uint32_t)m,
                   (uint32_t)(m >> 32), f.brick_valptr[bm]};
    };

    // R register stages; stage s holds the loads of one brick in flight.
    uint64_t st_mask[R];
    float st_a[R];
    float st_b[R][T];

    // Issue the loads of brick i of the chunk into stage s.  The value index is
    // the number of pattern bits below this lane's bit; lanes whose bit is clear
    // read a neighbouring value (vals has one pad element) that is discarded.
    auto issue = [&](const Chunk& ch, uint32_t i, int s) {
      const uint32_t mlo = __builtin_amdgcn_readlane(ch.mask_lo, i);
      const uint32_t mhi = __builtin_amdgcn_readlane(ch.mask_hi, i);
      const uint32_t off = __builtin_amdgcn_readlane(ch.off, i);
      const uint64_t mask = ((uint64_t)mhi << 32) | mlo;
      const uint32_t col = __builtin_amdgcn_ds_bpermute(4 * (4 * i + kq), ch.cols);
      st_mask[s] = mask;
      st_a[s] = f.vals[(int64_t)off + __popcll(mask & below)];
      load_b<T, ALIGNED>(B + (int64_t)(col == kPadCol ? 0u : col) * N, N, ncol0, st_b[s]);
    };
    auto compute = [&](int s) {
      const float a = ((st_mask[s] >> bit) & 1ull) ? st_a[s] : 0.f;
#pragma unroll
      for (int u = 0; u < T; ++u)
        acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, st_b[s][u], acc[u], 0, 0, 0);
    };

    // The first chunk passes through an empty asm statement so that it is not a
    // plain load: otherwise the compiler merges it with the in-loop chunk load
    // into one load at the top of the loop, serialising that latency.
    Chunk cur = load_chunk(b_begin);
    asm volatile("" : "+v"(cur.cols), "+v"(cur.mask_lo), "+v"(cur.mask_hi), "+v"(cur.off));

    // Step g computes brick g-R from stage g%R and then refills that stage with
    // brick g, so R bricks' loads are in flight while the MFMAs issue.  Refills
    // are unconditional (past the end they re-read the last brick, which is
    // harmless and keeps the compiler's count of outstanding loads exact); only
    // the MFMAs are skipped for steps that hold no brick.
    const uint32_t total = nbricks + R;
    for (uint32_t c = 0; c < total; c += CH) {
      const Chunk nxt = load_chunk(b_begin + c + CH);
#pragma unroll 1
      for (uint32_t i0 = 0; i0 < (uint32_t)CH; i0 += R) {
        if (c + i0 >= total) break;
#pragma unroll
        for (int s = 0; s < R; ++s) {
          const uint32_t g = c + i0 + s;
          if (g >= (uint32_t)R && g - R < nbricks) compute(s);
          issue(cur, i0 + s, s);
        }
      }
      cur = nxt;
    }
  }

  // acc[q*V + w][v] = C[row 4*kq + v][ncol0 + q*16*V + w]
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
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    if (v < rows_left) {
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const int64_t n = ncol0 + q * 16 * V;
        float tmp[V];
#pragma unroll
        for (int w = 0; w < V; ++w) tmp[w] = acc[q * V + w][v];
        if constexpr (ALIGNED) {
          if (n < N) store_vec<V>(out + v * N + n, tmp);
        } else {
#pragma unroll
          for (int w = 0; w < V; ++w)
            if (n + w < N) out[v * N + n + w] = tmp[w];
        }
      }
    }
  }
}

// ------------------------------------------------------------------ MFMA, fast path
// Same lane mapping as above for B smaller than 4 GiB (32-bit byte offsets), any N and any
// dword-aligned B and C, on tiles of 16*T columns, T = 1..8 (T = 1 and 2 where launch_spmm_mfma does not
// choose exec_narrow.hip).  A lane owns one vector of W0 =
// min(T, 4) columns and, for T > 4, a second one of W1 = T - 4.  Loads and stores need no more
// than dword alignment, so rows of an odd N are read with the same vectors as rows of a whole
// one.  A vector that reaches past column N is moved back to end at N, for the load and for the
// store: its lane then holds some columns that its neighbour holds too, with the same bits, and
// both store them.
//
// Vector-ALU instructions overlap only partly with MFMAs on a SIMD (measured:
// about 2 cycles of MFMA time lost per extra VALU instruction), so the per-brick
// VALU work is kept small:
//   * pattern and value offset of each brick come through the scalar cache into
//     SGPRs (8 bricks per fetch), not through vector loads and cross-lane reads;
//   * the B-row byte offsets of 8 bricks are computed once per 8 bricks (one
//     lane per brick column) and handed out with ds_bpermute, which issues on
//     the LDS port;
//   * loads use a scalar base plus a 32-bit lane offset.
// The arrays behind BrickFormat carry kFormatPad spare bricks at the end, so
// patterns and value offsets are fetched 8 bricks at a time without clamping.
// The loads issued for the few steps past a work item's last brick repeat that
// brick's B rows and values (cache hits, data never used): with short panels (ten
// bricks, say) four steps of the next panel's rows would otherwise add 40 % to
// the traffic from memory.
constexpr int kFastChunk = 8;

template <int T, bool FULL, bool IDX, int WPB>
__global__ __launch_bounds__(64 * WPB) void k_spmm_mfma_fast(
    SPMM_ITEM_PARAMS, const uint32_t* __restrict__ panel_ptr, const uint32_t* __restrict__ brick_cols,
    const uint64_t* __restrict__ brick_mask, const uint32_t* __restrict__ brick_valptr,
    const float* __restrict__ vals,
    const float* __restrict__ B, float* __restrict__ C, float* __restrict__ partial, int64_t M,
    int64_t N, uint32_t k_last) {
  // (the format arrays are separate __restrict__ parameters, not a struct, so that
  // the compiler knows they are read-only here and may use the scalar cache)
  constexpr int W0 = T < 4 ? T : 4, W1 = T - W0;   // columns of the lane's first, second vector
  constexpr int R = kStages;
  constexpr int CH = kFastChunk;
  static_assert(CH % R == 0 && CH * kBrickK <= 64, "stage and lane mapping assume this");

  const int lane = threadIdx.x & 63;
  // the wavefront's index as a scalar, so that its work item comes through the scalar cache
  // (one round trip less through the vector-memory path before the first brick)
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  WorkItem it;
  if (!work_item<WPB>(SPMM_ITEM_MAP, panel_ptr, wave, &it))
    return;  // whole wavefront leaves together
  const uint32_t panel = it.panel;
  const uint32_t b_begin = it.brick_begin;
  const uint32_t b_end = it.brick_end;
  const uint32_t slot = it.slot;

  const int j = lane & 15;
  const int kq = lane >> 4;
  const uint32_t perm_transpose = 4u * (uint32_t)(4 * j + kq);  // ds_bpermute: read lane 4j + kq
  const uint32_t row_bytes = (uint32_t)N * 4u;
  // first columns of this lane's vectors and their byte offsets inside a B row (a vector that
  // would reach past N ends at N; N >= W0 and, where there is a second vector, N > 64)
  const uint32_t ncol0 = blockIdx.y * (16u * T) + W0 * j;
  const uint32_t ncol1 = blockIdx.y * (16u * T) + 64u + W1 * j;
  const uint32_t at0 = min(ncol0, (uint32_t)N - W0), at1 = min(ncol1, (uint32_t)N - W1);
  const uint32_t lane_off0 = at0 * 4u, lane_off1 = at1 * 4u;
  const uint32_t perm_base = 4u * (uint32_t)kq;  // ds_bpermute byte address of lane kq

  float4_t acc[T];
#pragma unroll
  for (int u = 0; u < T; ++u) acc[u] = float4_t{0.f, 0.f, 0.f, 0.f};

  if (b_begin < b_end) {
    const uint32_t nbricks = b_end - b_begin;
    const char* Bbytes = reinterpret_cast<const char*>(B);
    [[maybe_unused]] const int4_t vals_at = float_buffer(vals);

    struct Meta { uint64_t mask[CH]; uint32_t off[CH]; };
    auto load_meta = [&](uint32_t base) {   // uniform addresses: scalar loads
      // one pointer per array, constant offsets: lets the loads merge into wide scalar loads
      const uint64_t* __restrict__ mp = brick_mask + base;
      const uint32_t* __restrict__ op = brick_valptr + base;
      Meta m;
#pragma unroll
      for (int i = 0; i < CH; ++i) { m.mask[i] = mp[i]; m.off[i] = op[i]; }
      return m;
    };
    // lane 4*i + c: byte offset of B row brick_cols[4*(base+i) + c]; pad columns
    // (0xFFFFFFFF) clamp to the last row, which is harmless since A is 0 there
    auto load_col = [&](uint32_t base) {
      // steps past the work item's last brick re-read that brick's rows (cache hits) instead
      // of pulling the next panel's B rows through the memory system for nothing
      const uint32_t slot = (uint32_t)lane & (CH * kBrickK - 1);
      const uint32_t idx = min(base * kBrickK + slot, (b_end - 1) * kBrickK + (slot & (kBrickK - 1)));
      return brick_cols[idx];
    };
    auto row_offset = [&](uint32_t col) { return min(col, k_last) * row_bytes; };

    uint64_t st_mask[R];
    float st_a[R];
    float st_b[R][T];
    // Decode (the prefix-count decode of Algorithm 1) in pattern-bit order, then transpose:
    // lane l first acts for pattern bit l.  Its value index is the number of pattern bits
    // below bit l, which is what v_mbcnt computes from the wave-uniform pattern in two
    // instructions; the gather that fetches it has addresses that never decrease from lane
    // to lane, which the vector-memory pipe handles as cheaply as a contiguous load (a gather
    // in MFMA lane order costs it as much as a dwordx4 load).  Lanes whose bit is clear are
    // zeroed with the pattern itself as the select mask.  One ds_bpermute (LDS port, no
    // vector-ALU slot) then moves element (row r, column c) from lane 4r + c to the lane the
    // MFMA wants it in, 16c + r.
    auto issue = [&](uint64_t mask, uint32_t off, uint32_t ro, int s) {
      st_mask[s] = mask;
      const uint32_t cnt = __builtin_amdgcn_mbcnt_hi(
          (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
      // scalar base + 32-bit byte offset (the launcher checks that the values fit 4 GiB)
      if constexpr (IDX) st_a[s] = spmm_load_indexed(vals_at, (int)cnt, 0, (int)(off * 4u), 0);
      else
        st_a[s] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(vals) + (off * 4u + cnt * 4u));
      const char* brow = Bbytes + (ro + lane_off0);
      load_any<W0>(brow, &st_b[s][0]);
      // whole 128-column tiles: the second vector lies a constant distance behind the first
      if constexpr (W1 > 0) load_any<W1>(FULL ? brow + 256 : Bbytes + (ro + lane_off1), &st_b[s][W0]);
    };
    // the A operand of the brick in stage s: zero fill, then the transposition
    auto operand = [&](int s) {
      float in_bit_order;
      asm("v_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(in_bit_order) : "v"(st_a[s]), "s"(st_mask[s]));
      return __builtin_bit_cast(
          float, __builtin_amdgcn_ds_bpermute(perm_transpose, __builtin_bit_cast(int, in_bit_order)));
    };
    auto multiply = [&](float a, int s) {
#pragma unroll
      for (int u = 0; u < T; ++u)
        acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, st_b[s][u], acc[u], 0, 0, 0);
    };
    auto compute = [&](int s) { multiply(operand(s), s); };
    float a_ahead = 0.f;   // steady chunks: the next step's A operand, made one step early

    Meta cur = load_meta(b_begin);
    uint32_t ro_cur = row_offset(load_col(b_begin));
    const uint32_t off_last = brick_valptr[b_end - 1];
    // keep the first fetch from being merged with the in-loop fetch into one
    // load at the top of the loop (which would expose its latency every chunk)
    asm volatile("" : "+v"(ro_cur));
#pragma unroll
    for (int i = 0; i < CH; ++i) asm volatile("" : "+s"(cur.mask[i]), "+s"(cur.off[i]));

    // Step g computes brick g-R from stage g%R and then refills that stage with
    // brick g, so R bricks' loads are in flight while the MFMAs issue.  Refills
    // are unconditional up to the next multiple of R past the end (keeps the
    // compiler's count of outstanding loads exact); only MFMAs are skipped for
    // steps that hold no brick.
    const uint32_t total = nbricks + R;
    uint32_t ro_next = __builtin_amdgcn_ds_bpermute(perm_base, ro_cur);
    // `steady`: the chunk lies entirely inside the work item and behind its first R steps, so
    // every step has a brick to compute and a brick to fetch and needs none of the checks
    // col_following: the next chunk's columns as loaded at the start of this chunk; they are
    // turned into row offsets in the chunk's last step, so that nothing waits for that load
    // while the ring's loads are younger than it
    uint32_t ro_following = 0;
    auto step = [&](auto steady, auto ordered, int i, uint32_t g, const Meta& m, uint32_t ro_this,
                    uint32_t col_following) {
      constexpr bool kSteady = decltype(steady)::value;
      if constexpr (kSteady) {
        // the cross-lane move of the next brick's operand runs under this brick's MFMAs
        const float a = a_ahead;
        a_ahead = operand((i + 1) % R);
        multiply(a, i % R);
      } else {
        if (g >= (uint32_t)R && g - R < nbricks) compute(i % R);
      }
      // this lane's row offset was fetched across lanes one step ago (its LDS-port latency
      // hides behind the MFMAs above); fetch the next brick's now
      const uint32_t ro = ro_next;
      if (i + 1 < CH) {
        ro_next = __builtin_amdgcn_ds_bpermute(perm_base + 16u * (i + 1), ro_this);
      } else {
        ro_following = row_offset(col_following);
        ro_next = __builtin_amdgcn_ds_bpermute(perm_base, ro_following);
      }
      const bool live = kSteady || g < nbricks;   // uniform: scalar selects
      issue(live ? m.mask[i] : 0ull, live ? m.off[i] : off_last, ro, i % R);
      // without the branches of the checked variant the steps of a chunk are one basic block;
      // `ordered` keeps the scheduler from sinking a step's loads down to their use R steps later
      if constexpr (decltype(ordered)::value) __builtin_amdgcn_sched_barrier(0);
    };
    // Whole chunks run in loops whose only exit is at their top; the last, partial chunk is
    // straight-line code after them.  With an exit in the middle of a loop body the compiler
    // must assume, at the loop head, that the steps after that exit issued no loads (it
    // cannot see that the loop ends on that path), and it then waits for all but the newest
    // load at the start of every chunk, which empties the ring every CH bricks.
    // Three phases: the first chunk (its first R steps have nothing to compute), the chunks
    // that lie entirely inside the work item (no checks), and the one or two chunks around its
    // end.  Every chunk issues the same loads in the same order, so the count of loads in
    // flight is the same on every path into a loop head.
    uint32_t c = 0;
    auto chunk = [&](auto steady, auto ordered) {
      const Meta nxt = load_meta(b_begin + c + CH);
      const uint32_t col_nxt = load_col(b_begin + c + CH);
#pragma unroll
      for (int i = 0; i < CH; ++i) step(steady, ordered, i, c + i, cur, ro_cur, col_nxt);
      cur = nxt;
      ro_cur = ro_following;
    };
    // (ordered in the narrowest tile, whose steps hold so little else that their loads changed places: the
    // check-free loop behind then began with a wait for younger ones.  512 panels of 160 scattered bricks,
    // N = 16: 21.6 us, in order 20.3; panels of 39 the same.  In order in every chunk the kernel takes more
    // scalar registers: 28 wavefronts a CU instead of 32, and Eq. 7 splits differently.)
    if (c + CH <= total) {
      chunk(std::false_type{}, std::bool_constant<T == 1>{});
      c += CH;
    }
    if (c + CH <= nbricks) a_ahead = operand(0);   // c is a multiple of CH, so stage 0 is next
    for (; c + CH <= nbricks; c += CH) chunk(std::true_type{}, std::true_type{});
    for (; c + CH <= total; c += CH) chunk(std::false_type{}, std::false_type{});
    if (c < total) {
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        if (i % R == 0 && i > 0 && c + i >= total) break;
        // (its last step fetches nothing real)
        step(std::false_type{}, std::false_type{}, i, c + i, cur, ro_cur, 0u);
      }
    }
  }

  // acc[w][v] = C[row 4*kq + v][at0 + w], acc[W0 + w][v] = C[row 4*kq + v][at1 + w]
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
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    if (v < rows_left) {
      float t[T];
#pragma unroll
      for (int w = 0; w < T; ++w) t[w] = acc[w][v];
      // C is written once and not read again here: stream it past the caches
      if (ncol0 < (uint32_t)N) store_any_nt<W0>(out + v * N + at0, t);
      if constexpr (W1 > 0) {
        if (ncol1 < (uint32_t)N) store_any_nt<W1>(out + v * N + at1, t + W0);
      }
    }
  }
}

// ------------------------------------------------------------------ VALU CSR
template <int V, bool ALIGNED>
__global__ __launch_bounds__(64 * kWavesPerBlock) void k_spmm_valu(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind,
    const float* __restrict__ vals, const uint32_t* __restrict__ panels, int64_t n_panels,
    const float* __restrict__ B, float* __restrict__ C, int64_t M, int64_t N) {
  const int lane = threadIdx.x & 63;
  const int64_t wid = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int64_t pslot = wid / kPanel;
  if (pslot >= n_panels) return;
  const uint32_t panel = __builtin_amdgcn_readfirstlane(panels[pslot]);
  const int64_t row = (int64_t)panel * kPanel + (wid % kPanel);
  if (row >= M) return;
  const int32_t s = __builtin_amdgcn_readfirstlane(rowptr[row]);
  const int32_t t = __builtin_amdgcn_readfirstlane(rowptr[row + 1]);
  const int64_t n = (int64_t)blockIdx.y * (64 * V) + V * lane;

  float acc[V];
#pragma unroll
  for (int w = 0; w < V; ++w) acc[w] = 0.f;

  // columns >= N are read from a clamped address and never stored
  const int64_t n_ld = ALIGNED ? min(n, N - V) : n;
  auto load_row = [&](int32_t col, float (&bv)[V]) {
    const float* brow = B + (int64_t)col * N;
    if constexpr (ALIGNED) load_vec<V>(brow + n_ld, bv);
    else {
#pragma unroll
      for (int w = 0; w < V; ++w) bv[w] = brow[min(n + w, N - 1)];
    }
  };

  int32_t e = s;
  for (; e + 4 <= t; e += 4) {
    int32_t c[4];
    float a[4];
    float bv[4][V];
#pragma unroll
    for (int x = 0; x < 4; ++x) { c[x] = colind[e + x]; a[x] = vals[e + x]; }
#pragma unroll
    for (int x = 0; x < 4; ++x) load_row(c[x], bv[x]);
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int w = 0; w < V; ++w) acc[w] = fmaf(a[x], bv[x][w], acc[w]);
  }
  for (; e < t; ++e) {
    float bv[V];
    load_row(colind[e], bv);
    const float a = vals[e];
#pragma unroll
    for (int w = 0; w < V; ++w) acc[w] = fmaf(a, bv[w], acc[w]);
  }

  float* out = C + row * N;
  if constexpr (ALIGNED) {
    if (n < N) store_vec<V>(out + n, acc);
  } else {
#pragma unroll
    for (int w = 0; w < V; ++w)
      if (n + w < N) out[n + w] = acc[w];
  }
}

// ------------------------------------------------------------------ VALU CSR, rows side by side
// Several rows per wavefront: a group of LPR lanes owns one row and covers 4*LPR columns of C
// (one dwordx4 per lane and stored entry), so a wavefront works on 64/LPR rows at once: two rows
// at N = 128, eight at N = 32, a whole panel at N = 16.  Column index and value of an entry are
// fetched LPR at a time with coalesced loads and handed out across the group's lanes.
// Four entries are in flight per group and iteration; past the end of a row the last entry is
// re-read with a zero multiplier.  Rows longer than kLongRow entries are left to
// k_spmm_valu_long, which spreads one row over a whole workgroup.
constexpr int kLongRow = 256;   // == long_row_threshold()

template <int LPR>
__global__ __launch_bounds__(64 * kWavesPerBlock) void k_spmm_valu_rows(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind,
    const float* __restrict__ vals, const uint32_t* __restrict__ panels, int64_t n_panels,
    const float* __restrict__ B, float* __restrict__ C, int64_t M, int64_t N) {
  constexpr int R = 64 / LPR;              // rows per wavefront
  constexpr int WPP = kPanel / R;          // wavefronts per panel (R <= 16)
  const int lane = threadIdx.x & 63;
  const int64_t wid = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int64_t pslot = wid / WPP;
  if (pslot >= n_panels) return;
  const uint32_t panel = __builtin_amdgcn_readfirstlane(panels[pslot]);
  const int64_t row = (int64_t)panel * kPanel + (wid % WPP) * R + lane / LPR;
  const int64_t n = (int64_t)blockIdx.y * (4 * LPR) + 4 * (lane % LPR);
  if (row >= M) return;                    // the whole group leaves together
  // Lanes whose columns lie past N (N is a multiple of 4: whole vectors only) stay: they hold
  // entries that the other lanes of the group fetch from them.  They read a clamped address
  // and store nothing.
  const bool in_range = n < N;
  const int32_t s = rowptr[row], t = rowptr[row + 1];
  if (t - s > kLongRow) return;
  const float* __restrict__ Bn = B + (in_range ? n : N - 4);
  float4_t acc = {0.f, 0.f, 0.f, 0.f};
  // The group fetches LPR entries of its row with one coalesced load each for column and
  // value (lane i of the group takes entry i) and hands them out across lanes, four at a
  // time: one B-row load per entry is then the only traffic through the vector-memory pipe.
  const int gl = lane % LPR;               // lane inside the group
  const int g0 = lane - gl;                // first lane of the group
  for (int32_t e0 = s; e0 < t; e0 += LPR) {
    const int32_t me = min(e0 + gl, t - 1);
    const int32_t cv = colind[me];                      // past the end: the last entry again,
    const float av = e0 + gl < t ? vals[me] : 0.f;      // with a zero multiplier
    const int cnt = min(LPR, t - e0);
    for (int x0 = 0; x0 < cnt; x0 += 4) {
      float4_t b[4];
      float a[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int src = g0 + min(x0 + x, LPR - 1);
        const int32_t c = __shfl(cv, src, 64);
        a[x] = __shfl(av, src, 64);
        b[x] = *reinterpret_cast<const float4_t*>(Bn + (int64_t)c * N);
      }
#pragma unroll
      for (int x = 0; x < 4; ++x) {
#pragma unroll
        for (int w = 0; w < 4; ++w) acc[w] = fmaf(a[x], b[x][w], acc[w]);
      }
    }
  }
  if (in_range) __builtin_nontemporal_store(acc, reinterpret_cast<float4_t*>(C + row * N + n));
}

// One workgroup of kLongWaves wavefronts per long row: its kLongWaves * (64/LPR) lane groups
// take the row's entries in turn, four at a time, with the next four columns and values
// fetched while the current B rows are in flight; the partial sums are added in group order
// through LDS (deterministic).  `long_rows` lists every row of the matrix with more than
// kLongRow entries; rows whose panel is not in the sorted list `panels` belong to the brick
// kernel and are skipped.
constexpr int kLongWaves = 16;

template <int LPR>
__global__ __launch_bounds__(64 * kLongWaves) void k_spmm_valu_long(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind,
    const float* __restrict__ vals, const uint32_t* __restrict__ long_rows,
    const uint32_t* __restrict__ panels, int64_t n_panels, const float* __restrict__ B,
    float* __restrict__ C, int64_t N) {
  constexpr int R = 64 / LPR;
  constexpr int G = R * kLongWaves;        // lane groups of the workgroup
  __shared__ float4_t part[G][LPR];
  const int64_t row = long_rows[blockIdx.x];
  const uint32_t panel = (uint32_t)(row / kPanel);
  {   // is the row's panel routed here?  (uniform binary search in the sorted panel list)
    int64_t lo = 0, hi = n_panels;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (panels[mid] < panel) lo = mid + 1; else hi = mid;
    }
    if (lo >= n_panels || panels[lo] != panel) return;
  }
  const int lane = threadIdx.x & 63;
  const int grp = (threadIdx.x >> 6) * R + lane / LPR;
  const int gl = lane % LPR;
  const int64_t n = (int64_t)blockIdx.y * (4 * LPR) + 4 * gl;
  const bool active = n < N;
  const int32_t s = rowptr[row], t = rowptr[row + 1];
  const float* __restrict__ Bn = B + (active ? n : 0);
  float4_t acc = {0.f, 0.f, 0.f, 0.f};
  int32_t c[4];
  float a[4];
  auto fetch = [&](int32_t e, int32_t (&cc)[4], float (&aa)[4]) {
#pragma unroll
    for (int x = 0; x < 4; ++x) {   // past the end: the last entry again, with a zero multiplier
      const int32_t ex = min(e + x, t - 1);
      cc[x] = colind[ex];
      aa[x] = e + x < t ? vals[ex] : 0.f;
    }
  };
  int32_t e = s + 4 * grp;
  if (e < t) fetch(e, c, a);
  for (; e < t; e += 4 * G) {
    float4_t b[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) b[x] = *reinterpret_cast<const float4_t*>(Bn + (int64_t)c[x] * N);
    int32_t cn[4];
    float an[4];
    fetch(e + 4 * G, cn, an);
#pragma unroll
    for (int x = 0; x < 4; ++x) {
#pragma unroll
      for (int w = 0; w < 4; ++w) acc[w] = fmaf(a[x], b[x][w], acc[w]);
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) { c[x] = cn[x]; a[x] = an[x]; }
  }
  part[grp][gl] = acc;
  __syncthreads();
  if (grp == 0 && active) {
    float4_t sum = part[0][gl];
    for (int q = 1; q < G; ++q) sum += part[q][gl];
    __builtin_nontemporal_store(sum, reinterpret_cast<float4_t*>(C + row * N + n));
  }
}

// ------------------------------------------------------------------ merge (a8)
// Sum the partial 16 x N tiles of a split panel in part order and store to C.
// A thread owns four floats and reads kMergeAhead parts at a time.  The sum runs in part order; the parts
// of a round are added by selects, not behind a branch each, which would make the compiler load them one
// after the other.  The workgroups of a panel share its 16 * N floats.  Bound by the latency of the rounds
// (a part was written through another L2).  One load at a time, eight and sixteen in flight, us: 3750
// panels of which one has 151 parts, N = 1 39.6 / 12.9 / 10.5, N = 128 65.9 / 17.3 / 17.0; 6250 panels, up
// to 47 parts, N = 16 21.0 / 6.1 / 4.5, N = 128 12.9 / 6.0 / 6.8.  Thirty-two are behind at narrow widths
// (N = 16 6.3).
constexpr int kMergeAhead = 16, kMergeThreads = 256;

__global__ __launch_bounds__(kMergeThreads) void k_merge(const MergeItem* __restrict__ items,
                                                         const float* __restrict__ partial,
                                                         float* __restrict__ C, int64_t M, int64_t N) {
  const MergeItem it = items[blockIdx.x];
  const int64_t row0 = (int64_t)it.panel * kPanel;
  const int64_t rows = min<int64_t>(kPanel, M - row0);
  const int64_t tile = (int64_t)kPanel * N;
  const float* src = partial + (int64_t)it.slot_begin * tile;
  float* dst = C + row0 * N;
  auto merge = [&](auto width, int64_t x) {
    constexpr int V = decltype(width)::value;
    float s[V];
    load_any<V>(reinterpret_cast<const char*>(src + x), s);
    for (uint32_t q = 1; q < it.nparts; q += kMergeAhead) {
      float t[kMergeAhead][V];
#pragma unroll
      for (int k = 0; k < kMergeAhead; ++k)   // past the last part: the last again, not added
        load_any<V>(reinterpret_cast<const char*>(src + (int64_t)min(q + k, it.nparts - 1) * tile + x), t[k]);
#pragma unroll
      for (int k = 0; k < kMergeAhead; ++k) {
        const bool is = q + k < it.nparts;
#pragma unroll
        for (int w = 0; w < V; ++w) s[w] = is ? s[w] + t[k][w] : s[w];
      }
    }
    store_any_nt<V>(dst + x, s);
  };
  const int64_t whole = rows * N & ~(int64_t)3;   // the last panel of a ragged M may end off a vector
  const int64_t first = (int64_t)blockIdx.y * kMergeThreads + threadIdx.x;
  for (int64_t x = first * 4; x < whole; x += (int64_t)gridDim.y * kMergeThreads * 4)
    merge(std::integral_constant<int, 4>{}, x);
  if (whole + first < rows * N) merge(std::integral_constant<int, 1>{}, whole + first);
}

template <int T, bool ALIGNED>
hipError_t launch_mfma_t(const BrickFormat& f, const WorkSource& w, const float* B, float* C,
                         float* partial, int64_t M, int64_t N, hipStream_t s) {
  const unsigned gx = item_blocks<kWavesPerBlock>(w);
  const unsigned gy = (unsigned)((N + 16 * T - 1) / (16 * T));
  hipLaunchKernelGGL((k_spmm_mfma<T, ALIGNED>), dim3(gx, gy), dim3(64 * kWavesPerBlock), 0, s, SPMM_ITEM_ARGS(kWavesPerBlock, w), f,
                     B, C, partial, M, N);
  return hipGetLastError();
}

template <int T, bool ALIGNED>
int occupancy_t() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_spmm_mfma<T, ALIGNED>,
                                                   64 * kWavesPerBlock, 0) != hipSuccess || nb < 1)
    nb = 1;
  return nb * kWavesPerBlock;
}

template <int T>
int occupancy_fast_t() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_spmm_mfma_fast<T, false, false, kWavesPerBlock>, 64 * kWavesPerBlock,
                                                   0) != hipSuccess || nb < 1)
    nb = 1;
  return nb * kWavesPerBlock;
}

}  // namespace

// tiles of 16, 32, 64 or 128 columns: N a multiple of the vector width, B below 4 GiB
bool mfma_fast_shape(int64_t N, int64_t K) {
  const int tile = mfma_tile_for(N);
  const int V = tile >= 64 ? 4 : tile / 16;
  return N % V == 0 && mfma_32bit_shape(N, K);
}

// what the fast FP32 kernel serves: B rows reachable by 32-bit byte offsets, and the packed values
// with their 64 spare floats
bool mfma_32bit_shape(int64_t N, int64_t K) {
  return K > 0 && (double)K * (double)N * 4.0 < 4294967296.0;
}
bool mfma_32bit_values(int64_t nnz) { return nnz + 64 < (int64_t(1) << 30); }

// Columns of C per wavefront of the FP32 kernel that serves (N, K, nnz).  The fast kernel takes as few
// tiles of at most 128 columns as N needs, all of the same width, in steps of 16 columns: N = 77
// is one tile of 80 (five MFMAs a brick), not one of 128 (eight), and N = 144 two of 80, not two
// of 128.  Measured on 131,072 rows of 3x3 blocks (322 k bricks), against tiles of 16, 32, 64 and
// 128 with a scalar-load kernel for odd N: N = 48 30.2 -> 26.5 us, 80 50.9 -> 35.3, 144 96.2 ->
// 64.1, 33 61.5 -> 26.4, 77 139.6 -> 35.8, 511 729 -> 250; N = 16, 32, 64, 128 as before.
// Where rows start on 128-byte lines (N a multiple of 32), several tiles also end on them (a
// multiple of 32 columns): a line shared by two tiles is fetched twice.  843 k scattered bricks,
// tiles of 80 against 96 columns at N = 160: 384 / 328 us; of 112 against 128 at N = 224: 515 /
// 458.  Other N have no such lines to keep, and there the narrower tile is ahead (N = 144 on the
// blocks: 137 / 152).
int mfma_fp32_tile(int64_t N, int64_t K, int64_t nnz) {
  if (!mfma_32bit_shape(N, K) || !mfma_32bit_values(nnz)) return mfma_tile_for(N);
  const int64_t tiles = std::max<int64_t>(1, (N + 127) / 128);
  const int t = (int)std::max<int64_t>(1, ((N + 15) / 16 + tiles - 1) / tiles);
  return 16 * (tiles > 1 && N % 32 == 0 ? (t + 1) / 2 * 2 : t);
}

// Columns per wavefront that run.  Few panels on the tiles above leave SIMDs idle, or one with twice the
// wavefronts of another, and a single wavefront is a chain of latencies; on tiles of half the width they are
// twice as many.  Times in us, wide / narrower, of 3x3 blocks (ten a block row) and of cells of fill 0.1:
//   128 -> 64 columns at up to 2.5 wavefronts a SIMD: 640 panels, N = 128 10.5 / 9.7 and 14.7 / 12.5; 2500 panels
//     21.1 / 19.3 and 31.9 / 27.8; at 2.9 a SIMD blocks lose (21.6 / 24.0).  Less far where the narrower are not twice
//     as many (N = 300, 5 tiles for 3: at 3.6 a SIMD 21.3 / 18.3, at 4 a band 13.9 / 14.5), or rows of B are not
//     aligned (N = 339, at 4.1 a SIMD 23.1 / 21.3, at 4.95 22.0 / 23.0).  Beyond that, as long as B stays in the Infinity
//     Cache (a graph of 12,288 panels, B of 100 MB, 73.6 / 75.1):
//     - graphs: scattered panels of few bricks, bound by memory and not by MFMAs, one in 40 and more of them split (4096
//       panels 30.3 / 26.6; not of many: 2500 panels of 120 bricks, N = 64 in tiles of 32 34.7 / 40.5, of 51 19.9 / 21.7, of 27 14.6 /
//       15.5, of 18 12.7 / 13.2; graphs have 12 to 15);
//     - scattered panels of many bricks (cells of 8192 panels 112.5 / 107.1; N = 128, 6000 panels of 25 bricks 46.7 / 44.1, of
//       6 21.2 / 21.8; 4000 of 25, 7.8 a SIMD, 32.2 / 33.0; N = 256, 2800 of 25 44.5 / 41.8);
//     - any matrix with split panels whose wide wavefronts are more than the device holds (4 a SIMD, 5 of 96 columns), where
//       the long ones of a second round end alone: blocks and one row of 1000 entries, 3750 panels 29.6 / 32.9, 4100 39.1 /
//       35.8, 4500 40.1 / 37.9, 5300 44.6 / 42.9, 6100 45.3 / 48.1, 7100 51.1 / 52.7; so beyond 11/8 rounds only scattered ones
//       (cells and four long rows, 6100 46.3 / 44.7) and those with one brick in 128 in split panels (blocks and 30 rows of 2000
//       entries, 6100 56.1 / 52.6, 7100 61.8 / 58.5; one full row, 6250 78.6 / 78.7), of several wide tiles up to 7/4 rounds
//       (N = 256, 3300 panels and 30 rows 62.0 / 60.0, 3750 62.4 / 65.3).
//     Not where the SIMD with most has as many columns as before (blocks of 1977 panels, N = 128 20.7 / 21.0; 463, N = 160,
//     three tiles for two 8.4 / 8.55).
//   64 -> 32 and 32 -> 16 where the wider one gives at most 1.5 a SIMD, in 16-byte loads (exec_narrow.hip): 256
//     panels, N = 64 6.8 / 5.3 / 4.7 and 8.5 / 6.5 / 5.6; 1250 panels, N = 64 10.0 / 9.0 / 9.2; 1530, N = 64 11.4 / 10.1 and
//     18.3 / 15.4; 1024 panels, N = 128 10.4 / 11.0 / 13.4.  Where the wide tile is 32 itself, only as long as each of the
//     narrower ones has a SIMD to itself: blocks of 30 bricks, 440 panels 4.58 / 4.32, 560 4.71 / 4.96, 850 4.69 / 5.08; of 117
//     bricks, 390 panels 11.5 / 9.8, 520 11.7 / 11.7, 880 11.9 / 12.2; with split panels 100 11.6 / 9.7, 1087 27.6 / 30.0.
//     Cells of 3000 panels lose (22.5 /
//     24.7); graphs gain further (of 2500 panels, N = 64 14.9 / 14.2, N = 96 18.2 / 16.8; of 4000, N = 64 18.4 /
//     17.9), up to twelve of the narrower a SIMD (of 10,000 31.5 / 31.9).  Matrices with a few long rows, which as graphs
//     would lose (blocks and one of 1000 entries, 3750 panels, N = 64 19.0 / 20.9; cells and one of 2000, 4000 panels
//     15.8 / 17.0), gain as far as twelve where the wide tiles multiply columns behind N and these do not (N = 160, 96 / 32:
//     cells of 850 panels and three rows of 2000 11.7 / 9.9; 1670 of a band and three of 700 11.2 / 9.5; at 2.5 and more a SIMD of 96
//     0.87 to 0.91; with one panel in 40 and more split up to seven, 0.82 to 0.98, and 1.05 beyond), and any with split panels up to 1.5 wide ones a SIMD where there are no
//     tiles of 64 between (N = 96, 96 / 32: 0.92 to 1.00 at 0.75 to 1.5 a SIMD, 1.02 beyond).
// Not where the narrower tiles multiply many columns more than there are: N = 80 as two of 48, 930 panels, 9.1 / 9.7.
// Work lists and Eq. 7 go by the wide tiles, so which panels are split does not depend on this.
int mfma_run_tile(const WorkSource& w, int64_t N, int64_t K, int64_t nnz) {
  const int whole = mfma_fp32_tile(N, K, nnz);
  if (!mfma_32bit_shape(N, K) || !mfma_32bit_values(nnz) || N < 20 || (N > 32 && N < 48)) return whole;
  const int64_t items = (int64_t)w.n_items + w.n_parts;
  auto tiles = [&](int64_t width) { return (N + width - 1) / width; };
  const bool whole_lines = N % 32 == 0 && K * N * 4 < kNarrowLargeB;
  const bool graph = w.scattered && 40 * w.n_split >= w.panels && w.mean_bricks() <= 16;
  const int64_t wide = items * tiles(whole);
  const int64_t round = (whole > 96 ? 4 : 5) * (int64_t)w.simds;
  const bool second_round = w.n_split > 0 && wide > round &&
                            (w.scattered || 8 * wide <= 11 * round ||
                             (128 * w.part_bricks >= w.bricks && (tiles(whole) == 1 || 4 * wide <= 7 * round)));
  int tile = whole;
  for (int width = 64; width >= 16; width /= 2) {
    const int64_t k = tiles(width), t = ((N + 15) / 16 + k - 1) / k;
    const int64_t narrower = 16 * (t > 1 && N % 32 == 0 ? (t + 1) / 2 * 2 : t);
    const int64_t columns = k * narrower, least = tiles(whole) * whole;   // multiplied, with those behind N
    const int64_t waves = items * tiles(2 * width);
    if (narrower >= tile || (whole == 32 && 2 * items > w.simds)) continue;
    const int64_t most = k < 2 * tiles(whole) ? 8 : (N % 4 ? 9 : 10);   // narrower wavefronts for two SIMDs
    // columns of the SIMD with most: no gain where that stays, but for wavefronts that were alone
    const int64_t then = (items * k + w.simds - 1) / w.simds * narrower;
    const bool less = then < (wide + w.simds - 1) / w.simds * whole + (wide <= w.simds ? 1 : 0);
    const int64_t most_32 = graph ? 12 : w.n_split == 0 || columns >= least ? 0 : 40 * w.n_split < w.panels ? 12 : 7;
    if (width == 64 ? 10 * columns <= 11 * least &&
                          ((less && 2 * items * k <= most * w.simds) ||
                           (whole_lines && (graph || second_round ||
                                            (w.scattered && w.mean_bricks() >= 16 && items * k >= 10 * w.simds))))
                    : 4 * columns < 5 * least &&
                          ((less && 2 * waves <= 3 * w.simds) ||
                           (width == 32 && whole_lines &&
                            (items * k <= most_32 * w.simds || (w.n_split > 0 && tile == whole && 2 * wide <= 3 * w.simds)))))
      tile = (int)narrower;
  }
  return tile;
}

// The "thread blocks per SM" of Eq. 7: wavefronts of the MFMA kernel that fit on one CU at a time,
// taken at the power-of-two tile of N (the fast kernel's where N is a multiple of its vector width,
// else the general kernel's), not at the narrower tile that runs.  The narrower tiles hold up to
// half as many wavefronts more (5 x 16 columns: 24 a CU, 8 x 16: 16), and Eq. 7 then splits more
// panels: more partial tiles, and calls of spmm_exec_noalloc that no longer fit the static scratch.
int mfma_resident_waves_per_cu(int64_t N, int64_t K) {
  const int tile = mfma_tile_for(N);
  if (mfma_fast_shape(N, K)) {
    switch (tile) {
      case 16: return occupancy_fast_t<1>();
      case 32: return occupancy_fast_t<2>();
      case 64: return occupancy_fast_t<4>();
      default: return occupancy_fast_t<8>();
    }
  }
  const bool aligned = N % (tile >= 64 ? 4 : tile / 16) == 0;
  switch (tile) {
    case 16: return occupancy_t<1, true>();
    case 32: return aligned ? occupancy_t<2, true>() : occupancy_t<2, false>();
    case 64: return aligned ? occupancy_t<4, true>() : occupancy_t<4, false>();
    default: return aligned ? occupancy_t<8, true>() : occupancy_t<8, false>();
  }
}

hipError_t launch_spmm_mfma(const BrickFormat& f, const WorkSource& w, const float* B, float* C,
                            float* partial, int64_t M, int64_t N, int64_t K, int64_t nnz, hipStream_t s) {
  if (w.n_items == 0 || N == 0) return hipSuccess;
  if (mfma_32bit_shape(N, K) && mfma_32bit_values(nnz)) {
    // Tiles of 16 and 32 columns in 16-byte loads (exec_narrow.hip).  Not where panels are split, as in
    // power-law graphs, and B is not large: short panels of scattered rows, each a miss, gain nothing from fewer
    // accesses and lose 1 to 3 % to the larger chunk (graphs of 283 k and 450 k rows, us: N = 14 26.7 / 27.5 and 40.1 /
    // 41.5, N = 32 28.4 / 28.8 and 41.8 / 42.6; 600 k and 900 k rows, B of 77 and 115 MB: 63.6 / 60.5 and
    // 95.7 / 82.6; N = 8 at 283 k 22.5 / 21.3).  Without split panels, N = 14 to 32, bands, cells and blocks of
    // 25 k to 400 k rows: 2 to 12 % ahead or the same.  The tiles of few panels at wider N are ahead or the same, split
    // or not (graph of 640 panels, N = 64 9.7 / 9.2).
    const int tile = mfma_run_tile(w, N, K, nnz);
    if (N >= 4 && tile <= 32 && (N > 32 || w.n_split == 0 || N <= 8 || K * N * 4 >= kNarrowLargeB))
      return launch_spmm_mfma_narrow(f, w, tile, B, C, partial, M, N, K, s);
    const unsigned gy = (unsigned)((N + tile - 1) / tile);
    const uint32_t k_last = (uint32_t)(K - 1);
    const bool single = single_waves(w, tile, N, K);
#define SPMM_LAUNCH_WAVES(TT, FF, II, W)                                                        \
  hipLaunchKernelGGL((k_spmm_mfma_fast<TT, FF, II, W>), dim3(item_blocks<W>(w), gy), dim3(64 * W), 0, s, \
                     SPMM_ITEM_ARGS(W, w), f.panel_ptr, f.brick_cols,                           \
                     f.brick_mask, f.brick_valptr, f.vals, B, C, partial, M, N, k_last)
// (single_waves: no tiles of 48 and 80; those of 32 are for a B below its bound)
#define SPMM_LAUNCH_FAST(TT, FF, II)                                                            \
  do {                                                                                          \
    if (single) SPMM_LAUNCH_WAVES(TT, FF, II, 1); else SPMM_LAUNCH_WAVES(TT, FF, II, kWavesPerBlock); \
  } while (0)
    switch (tile / 16) {
      case 1: SPMM_LAUNCH_FAST(1, false, false); break;   // (split panels: short ones mostly)
      case 2: SPMM_LAUNCH_WAVES(2, false, false, kWavesPerBlock); break;
      case 3:
        if (values_by_index(w, tile, gy)) SPMM_LAUNCH_WAVES(3, false, true, kWavesPerBlock);
        else SPMM_LAUNCH_WAVES(3, false, false, kWavesPerBlock);
        break;
      case 4: if (values_by_index(w, tile, gy)) SPMM_LAUNCH_FAST(4, false, true); else SPMM_LAUNCH_FAST(4, false, false); break;
      case 5: SPMM_LAUNCH_WAVES(5, false, false, kWavesPerBlock); break;
      case 6: SPMM_LAUNCH_FAST(6, false, false); break;
      case 7: SPMM_LAUNCH_FAST(7, false, false); break;
      default:   // whole 128-column tiles: the second vector of a B row at a constant offset
        if (N % 128 == 0) SPMM_LAUNCH_FAST(8, true, false); else SPMM_LAUNCH_FAST(8, false, false);
        break;
    }
#undef SPMM_LAUNCH_WAVES
#undef SPMM_LAUNCH_FAST
    return hipGetLastError();
  }
  const int tile = mfma_tile_for(N);
  const int V = tile >= 64 ? 4 : tile / 16;
  const bool al = (N % V == 0) && ptr_aligned16(B) && ptr_aligned16(C) &&
                  (partial == nullptr || ptr_aligned16(partial));
  switch (tile) {
    case 16: return launch_mfma_t<1, true>(f, w, B, C, partial, M, N, s);
    case 32: return al ? launch_mfma_t<2, true>(f, w, B, C, partial, M, N, s)
                       : launch_mfma_t<2, false>(f, w, B, C, partial, M, N, s);
    case 64: return al ? launch_mfma_t<4, true>(f, w, B, C, partial, M, N, s)
                       : launch_mfma_t<4, false>(f, w, B, C, partial, M, N, s);
    default: return al ? launch_mfma_t<8, true>(f, w, B, C, partial, M, N, s)
                       : launch_mfma_t<8, false>(f, w, B, C, partial, M, N, s);
  }
}

hipError_t launch_spmm_valu(const int32_t* rowptr, const int32_t* colind, const float* vals,
                            const uint32_t* panels, int64_t n_panels, const uint32_t* long_rows,
                            int64_t n_long_rows, const float* B, float* C, int64_t M, int64_t N,
                            hipStream_t s) {
  if (n_panels == 0 || N == 0) return hipSuccess;
  const bool a16 = ptr_aligned16(B) && ptr_aligned16(C);
  if (a16 && N % 4 == 0) {
    // lanes per row: the smallest power of two that covers N in vectors of four, at most 64
    int lpr = 4;
    while (lpr < 64 && 4 * lpr < N) lpr *= 2;
    const unsigned gy = (unsigned)((N + 4 * lpr - 1) / (4 * lpr));
    const int wpp = kPanel / (64 / lpr);
    const unsigned gx = (unsigned)((n_panels * wpp + kWavesPerBlock - 1) / kWavesPerBlock);
#define SPMM_LAUNCH_ROWS(L)                                                                     \
  do {                                                                                          \
    hipLaunchKernelGGL(k_spmm_valu_rows<L>, dim3(gx, gy), dim3(64 * kWavesPerBlock), 0, s,      \
                       rowptr, colind, vals, panels, n_panels, B, C, M, N);                     \
    if (n_long_rows > 0)                                                                        \
      hipLaunchKernelGGL(k_spmm_valu_long<L>, dim3((unsigned)n_long_rows, gy),                  \
                         dim3(64 * kLongWaves), 0, s, rowptr, colind, vals, long_rows,          \
                         panels, n_panels, B, C, N);                                            \
  } while (0)
    switch (lpr) {
      case 4: SPMM_LAUNCH_ROWS(4); break;
      case 8: SPMM_LAUNCH_ROWS(8); break;
      case 16: SPMM_LAUNCH_ROWS(16); break;
      case 32: SPMM_LAUNCH_ROWS(32); break;
      default: SPMM_LAUNCH_ROWS(64); break;
    }
#undef SPMM_LAUNCH_ROWS
    return hipGetLastError();
  }
  // any N, any alignment: one wavefront per row
  const unsigned gx = (unsigned)((n_panels * kPanel + kWavesPerBlock - 1) / kWavesPerBlock);
  const unsigned gy = (unsigned)((N + 63) / 64);
  hipLaunchKernelGGL((k_spmm_valu<1, true>), dim3(gx, gy), dim3(64 * kWavesPerBlock), 0, s, rowptr,
                     colind, vals, panels, n_panels, B, C, M, N);
  return hipGetLastError();
}

hipError_t launch_merge(const MergeItem* items, int64_t n_items, const float* partial, float* C,
                        int64_t M, int64_t N, hipStream_t s) {
  if (n_items == 0 || N == 0) return hipSuccess;
  const unsigned gy = (unsigned)std::min<int64_t>((kPanel * N + 4 * kMergeThreads - 1) / (4 * kMergeThreads), 64);
  hipLaunchKernelGGL(k_merge, dim3((unsigned)n_items, gy), dim3(kMergeThreads), 0, s, items, partial,
                     C, M, N);
  return hipGetLastError();
}

}  // namespace spmm
