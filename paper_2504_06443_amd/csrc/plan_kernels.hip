// CSR -> brick format on the GPU (paper Section 3.2: active-column compaction,
// bricks of 4 columns, 64-bit pattern per brick, values packed row-major).
//
// No kernel waits on another workgroup; the only atomics are integer OR / ADD / MAX,
// so every output is reproducible bit for bit.
//
// Three ways to find a panel's active columns and their ranks:
//  * bitmap (matrices whose panels span few columns compared with their entries): one
//    wavefront per panel keeps a bitmap of the panel's column span in LDS; see the section
//    "per-panel path" below.
//  * sort (every other matrix whose panels are small enough): a panel's entries sorted by
//    column in registers, by class of panel size.
//  * search (what is left): the rows of a panel are already sorted, so "is this the
//    first row of the panel that holds column j" and "how many distinct columns of the
//    panel are smaller than j" are answered by binary searches in the (at most 16) rows of
//    the panel plus one exclusive scan of the first-occurrence flags over the whole entry
//    array.  The second question is only asked once per active column (the
//    first-occurrence entries, compacted into a list); the other entries of that column
//    follow a link to it.  One thread per entry (or per row / panel / brick).
#include "panel_layout.h"
#include "spmm_internal.h"

#include <algorithm>

namespace spmm {

namespace {

constexpr int kThreads = 256;

inline unsigned grid_for(int64_t n, int64_t threads = kThreads) {
  int64_t g = (n + threads - 1) / threads;
  return (unsigned)(g > 0 ? g : 1);
}

// first index in [lo, hi) whose column is >= j
__device__ inline int64_t lower_bound_col(const int32_t* __restrict__ colind, int64_t lo,
                                          int64_t hi, int32_t j) {
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (colind[mid] < j) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// reductions across the wavefront (every lane takes part; all get the result)
template <typename T> __device__ inline T wave_sum(T v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}
template <typename T> __device__ inline T wave_max(T v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v = max(v, __shfl_xor(v, d, 64));
  return v;
}
template <typename T> __device__ inline T wave_or(T v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v |= __shfl_xor(v, d, 64);
  return v;
}
// raises *p to v; the plain look first spares the atomic that would change nothing
__device__ inline void raise_to(uint32_t* p, uint32_t v) {
  if (v > __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(p, v);
}

// Requires a valid rowptr.  Also records the row of every entry.
__global__ void k_validate_cols(const int32_t* __restrict__ rowptr,
                                const int32_t* __restrict__ colind, int64_t M, int64_t K,
                                int64_t nnz, uint32_t* __restrict__ ent_row, uint32_t* err) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  int64_t lo = 0, hi = M;  // rowptr[lo] <= e < rowptr[hi]
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (rowptr[mid] <= e) lo = mid; else hi = mid;
  }
  ent_row[e] = (uint32_t)lo;
  const int64_t j = colind[e];
  uint32_t bad = 0;
  if (j < 0 || j >= K) bad |= kErrColRange;
  if (e > rowptr[lo] && colind[e - 1] >= j) bad |= kErrColOrder;
  if (bad) atomicOr(err, bad);
}

// ---------------------------------------------------------------- a1 census
// first[e] = 1 iff no earlier row of the same panel stores column colind[e].
// link[e] = the entry of that first row that stores the same column (e itself if first).
__global__ void k_first_in_panel(const int32_t* __restrict__ rowptr,
                                 const int32_t* __restrict__ colind,
                                 const uint32_t* __restrict__ ent_row, int64_t nnz,
                                 uint8_t* __restrict__ first, uint32_t* __restrict__ link) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  const int64_t i = ent_row[e];
  const int32_t j = colind[e];
  const int64_t r0 = i & ~(int64_t)(kPanel - 1);
  uint8_t f = 1;
  int64_t where = e;
  for (int64_t r = r0; r < i; ++r) {  // rows in ascending order: the first hit is the first occurrence
    const int64_t s = rowptr[r], t = rowptr[r + 1];
    const int64_t pos = lower_bound_col(colind, s, t, j);
    if (pos < t && colind[pos] == j) { f = 0; where = pos; break; }
  }
  first[e] = f;
  link[e] = (uint32_t)where;
}

// first_list[k] = the k-th first-occurrence entry (k = exclusive scan of the flags)
__global__ void k_compact_first(const uint8_t* __restrict__ first,
                                const uint32_t* __restrict__ first_scan, int64_t nnz,
                                uint32_t* __restrict__ first_list) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < nnz && first[e]) first_list[first_scan[e]] = (uint32_t)e;
}

// a2: active columns of each panel.
__global__ void k_panel_counts(const int32_t* __restrict__ rowptr,
                               const uint32_t* __restrict__ first_scan, int64_t M, int64_t P,
                               uint32_t* __restrict__ ncols_p) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P) return;
  const int64_t r0 = p * kPanel, r1 = min(r0 + kPanel, M);
  ncols_p[p] = first_scan[rowptr[r1]] - first_scan[rowptr[r0]];
}

template <typename T>
__global__ void k_fill(T* __restrict__ p, int64_t n, T v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// a2: one thread per active column (= per first-occurrence entry): its rank among the
// panel's active columns = number of first-occurrence entries of the panel with a smaller
// column, counted row by row with one binary search and two reads of the scanned flags.
__global__ void k_rank_first(const int32_t* __restrict__ rowptr,
                             const int32_t* __restrict__ colind,
                             const uint32_t* __restrict__ ent_row,
                             const uint32_t* __restrict__ first_list,
                             const uint32_t* __restrict__ first_scan,
                             const uint32_t* __restrict__ panel_ptr, int64_t M, int64_t n_active,
                             uint32_t* __restrict__ ent_rank, uint32_t* __restrict__ brick_cols) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_active) return;
  const int64_t e = first_list[k];
  const int64_t i = ent_row[e];
  const int32_t j = colind[e];
  const int64_t p = i / kPanel;
  const int64_t r0 = p * kPanel, r1 = min(r0 + kPanel, M);
  uint32_t rank = 0;
  for (int64_t r = r0; r < r1; ++r) {
    const int64_t s = rowptr[r], t = rowptr[r + 1];
    const int64_t pos = (r == i) ? e : lower_bound_col(colind, s, t, j);
    rank += first_scan[pos] - first_scan[s];
  }
  ent_rank[e] = rank;
  brick_cols[(int64_t)panel_ptr[p] * kBrickK + rank] = (uint32_t)j;
}

// a3: every entry takes the rank of its column's first occurrence, which gives its brick,
// its brick column and its pattern bit 4*row + column.
__global__ void k_scatter_bits(const int32_t* __restrict__ colind,
                               const uint32_t* __restrict__ ent_row,
                               const uint32_t* __restrict__ link,
                               const uint32_t* __restrict__ ent_rank,
                               const uint32_t* __restrict__ panel_ptr, int64_t nnz,
                               uint64_t* brick_mask, uint32_t* __restrict__ ent_brick,
                               uint8_t* __restrict__ ent_bit, uint8_t* __restrict__ col_seen) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  const int64_t i = ent_row[e];
  const uint32_t rank = ent_rank[link[e]];
  const uint32_t b = panel_ptr[i / kPanel] + rank / kBrickK;
  const uint32_t c = rank % kBrickK;
  const uint32_t bit = (uint32_t)(i % kPanel) * kBrickK + c;
  atomicOr((unsigned long long*)&brick_mask[b], 1ull << bit);
  ent_brick[e] = b;
  ent_bit[e] = (uint8_t)bit;
  col_seen[colind[e]] = 1;
}

// a4: position of a value = start of its brick + set bits below its own bit.
__global__ void k_pack_values(const float* __restrict__ vals,
                              const uint32_t* __restrict__ ent_brick,
                              const uint8_t* __restrict__ ent_bit,
                              const uint64_t* __restrict__ brick_mask,
                              const uint32_t* __restrict__ brick_valptr, int64_t nnz,
                              float* __restrict__ packed, uint32_t* __restrict__ src) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  const uint32_t b = ent_brick[e];
  const uint64_t below = brick_mask[b] & ((1ull << ent_bit[e]) - 1ull);
  const uint32_t pos = brick_valptr[b] + (uint32_t)__popcll(below);
  packed[pos] = vals[e];
  src[pos] = (uint32_t)e;
}

// entries(p): the CSR entry of packed value p; of four consecutive ones from a multiple of four
struct EntrySource {
  const uint32_t* p;
  __device__ uint32_t operator()(int64_t i) const { return p[i]; }
  __device__ uint4 four(int64_t i) const { return *reinterpret_cast<const uint4*>(p + i); }
};
struct StepSource {
  const int16_t* p;
  __device__ uint32_t operator()(int64_t i) const { return (uint32_t)(i + p[i]); }
  __device__ uint4 four(int64_t i) const {
    const short4 d = *reinterpret_cast<const short4*>(p + i);
    return uint4{(uint32_t)(i + d.x), (uint32_t)(i + 1 + d.y), (uint32_t)(i + 2 + d.z), (uint32_t)(i + 3 + d.w)};
  }
};

// New values for an unchanged pattern: packed position p takes the CSR entry that was recorded when
// the plan was built.  Bound by memory: 4 bytes each of values and packed values per entry, and 4 or 2 of
// where it comes from.  Gathering by packed position keeps the stores whole (the entries of a panel are 2 KB or
// so, and their reads hit a cache); four positions a thread.  CSR: the plan also keeps the values in CSR order, for the
// vector-ALU kernels.  7.86 M entries, one update behind another: from the entries 17.3 us, 94 MB; from steps 14.3, 79 MB.
// Eight positions a thread took 13.5 there, but longer where there are fewer (1.1 M entries, update and product at N =
// 16 15.7 / 16.7 us; 3.75 M of cells 19.9 / 21.3).
constexpr int64_t kUpdateBlock = (int64_t)kThreads * 4;   // positions a workgroup

template <typename Source, bool CSR>
__global__ __launch_bounds__(kThreads) void k_update_values(
    const float* __restrict__ vals, Source src, int64_t nnz,
    float* __restrict__ packed, float* __restrict__ csr_vals) {
  const int64_t first = blockIdx.x * kUpdateBlock + 4 * threadIdx.x;
  if ((blockIdx.x + 1) * kUpdateBlock <= nnz) {
    const uint4 e = src.four(first);
    float4 v;
    v.x = vals[e.x]; v.y = vals[e.y]; v.z = vals[e.z]; v.w = vals[e.w];
    *reinterpret_cast<float4*>(packed + first) = v;
    if constexpr (CSR) {
#pragma unroll
      for (int k = 0; k < 4; ++k) csr_vals[first + k] = vals[first + k];
    }
  } else {
    for (int64_t p = blockIdx.x * kUpdateBlock + threadIdx.x; p < nnz; p += kThreads) {
      packed[p] = vals[src(p)];
      if constexpr (CSR) csr_vals[p] = vals[p];
    }
  }
}

// Columns and values in CSR order again, from the bricks: a wavefront takes a brick at a time, lane l
// the element of pattern bit l.  At most kRestoreBlocks workgroups walk the bricks: a plan holds up to
// 2^30 of them, a launch fewer than kMaxLaunchThreads threads.
constexpr int kRestoreBlocks = 1 << 16;

template <typename Source>
__global__ __launch_bounds__(kThreads) void k_restore_csr(
    const uint32_t* __restrict__ brick_cols, const uint64_t* __restrict__ brick_mask,
    const uint32_t* __restrict__ brick_valptr, const float* __restrict__ packed,
    Source src, int64_t nb, int32_t* __restrict__ colind,
    float* __restrict__ csr_vals) {
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * (kThreads / 64);
  for (int64_t b = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); b < nb; b += stride) {
    const uint64_t mask = brick_mask[b];
    if (!((mask >> lane) & 1ull)) continue;
    const uint32_t pos = brick_valptr[b] + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
    const uint32_t e = src(pos);
    colind[e] = (int32_t)brick_cols[b * kBrickK + (lane & (kBrickK - 1))];
    csr_vals[e] = packed[pos];
  }
}

__device__ inline void wave_stores_done() {   // the wavefront's own stores and atomics have arrived
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// a5: per-panel class (Table 1, integer compare) and class totals, histogram of bricks by stored
// elements, columns that occur.  Few, large workgroups: each adds its totals to the counters once,
// and same-address atomics of many workgroups were what the separate kernels for these three spent
// their time on (630 k bricks of 16,384 panels: 55 us in three launches, 8 us in
// this one).
// The first workgroup also writes the spare entries behind the brick arrays (see BrickFormat).  The last one to
// end puts the counters into pinned memory, flag last, for the host that looks for it, and all copy panel_ptr there
// where the host wants it: two copies and the wait for the stream took 10 to 20 us more.  Everything a
// workgroup has written is visible to the device and the host before it counts itself as ended: every
// wavefront waits for its own stores and atomics (a barrier does not, and a release only for those of the
// wavefront that makes it) before the thread that counts the workgroup releases.
constexpr int kStatThreads = 1024;
constexpr int kStatBlocks = 128;

__global__ __launch_bounds__(kStatThreads) void k_plan_stats(
    const uint32_t* __restrict__ panel_ptr, const uint32_t* __restrict__ panel_nnzptr, int64_t P,
    uint32_t* __restrict__ brick_cols, uint64_t* __restrict__ brick_mask,
    uint32_t* __restrict__ brick_valptr, float* __restrict__ vals, int64_t nb, int64_t nnz,
    const uint8_t* __restrict__ col_seen, int64_t K, PlanControl* ctl, PlanControl* pinned,
    uint32_t* pinned_ptr, int64_t n_ptr, uint32_t* flag) {
  unsigned long long* counters = ctl->counters;
  static_assert(kFormatPad * kBrickK <= kStatThreads && kFormatPad < 64, "one workgroup writes the pads");
  if (blockIdx.x == 0) {
    const int t = threadIdx.x;
    if (t < kFormatPad * kBrickK) brick_cols[nb * kBrickK + t] = 0;
    if (t < kFormatPad) brick_mask[nb + t] = 0;
    if (t < kFormatPad + 1) brick_valptr[nb + t] = (uint32_t)nnz;
    if (t < 64) vals[nnz + t] = 0.f;
  }
  constexpr int kWaves = kStatThreads / 64;
  __shared__ uint32_t hist[kWaves][65];          // a histogram per wavefront: fewer collisions
  __shared__ unsigned long long acc[kCntPopHist];
  for (int t = threadIdx.x; t < kWaves * 65; t += kStatThreads) (&hist[0][0])[t] = 0;
  if (threadIdx.x < kCntPopHist) acc[threadIdx.x] = 0;
  __syncthreads();
  const int64_t first = (int64_t)blockIdx.x * kStatThreads + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * kStatThreads;

  uint32_t* mine = hist[threadIdx.x >> 6];
  int64_t b = first;
  for (; b + 3 * stride < nb; b += 4 * stride) {   // four loads in flight
    uint64_t m[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) m[k] = brick_mask[b + k * stride];
#pragma unroll
    for (int k = 0; k < 4; ++k) atomicAdd(&mine[__popcll(m[k])], 1u);
  }
  for (; b < nb; b += stride) atomicAdd(&mine[__popcll(brick_mask[b])], 1u);

  // class totals in registers: bricks and entries of a thread's panels
  unsigned long long panels[3] = {0, 0, 0}, bricks[3] = {0, 0, 0}, entries[3] = {0, 0, 0};
  for (int64_t p = first; p < P; p += stride) {
    const unsigned long long n = panel_ptr[p + 1] - panel_ptr[p];
    const unsigned long long nz = panel_nnzptr[p + 1] - panel_nnzptr[p];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const bool is = n && (nz < 8 * n ? 0 : (nz < 16 * n ? 1 : 2)) == c;
      panels[c] += is;
      bricks[c] += is ? n : 0;
      entries[c] += is ? nz : 0;
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    panels[c] = wave_sum(panels[c]);
    if (!panels[c]) continue;   // (the same in every lane)
    bricks[c] = wave_sum(bricks[c]);
    entries[c] = wave_sum(entries[c]);
    if ((threadIdx.x & 63) == 0) {
      atomicAdd(&acc[kCntPanelsByClass + c], panels[c]);
      atomicAdd(&acc[kCntBricksByClass + c], bricks[c]);
      atomicAdd(&acc[kCntNnzByClass + c], entries[c]);
      atomicAdd(&acc[kCntNonEmptyPanels], panels[c]);
    }
  }

  // flags of 0 or 1, sixteen at a time (the array is 256-byte aligned)
  uint32_t seen = 0;
  const int64_t vecs = K / 16;
  for (int64_t v = first; v < vecs; v += stride) {
    const uint4 f = reinterpret_cast<const uint4*>(col_seen)[v];
    seen += __popc(f.x) + __popc(f.y) + __popc(f.z) + __popc(f.w);
  }
  if (first < K - vecs * 16) seen += col_seen[vecs * 16 + first];
  seen = wave_sum(seen);
  if (seen && (threadIdx.x & 63) == 0) atomicAdd(&acc[kCntDistinctCols], (unsigned long long)seen);

  __syncthreads();
  if (threadIdx.x < kCntPopHist && acc[threadIdx.x])
    atomicAdd(&counters[threadIdx.x], acc[threadIdx.x]);
  if (threadIdx.x < 65) {
    unsigned long long h = 0;
    for (int w = 0; w < kWaves; ++w) h += hist[w][threadIdx.x];
    if (h) atomicAdd(&counters[kCntPopHist + threadIdx.x], h);
  }
  if (!pinned) return;
  if (pinned_ptr)
    for (int64_t p = first; p < n_ptr; p += stride)
      __hip_atomic_store(&pinned_ptr[p], panel_ptr[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  // (one release a workgroup, by the thread that counts it: one by every wavefront took 25 us)
  __shared__ uint32_t s_last;
  wave_stores_done();
  __syncthreads();
  if (threadIdx.x == 0)
    s_last = __hip_atomic_fetch_add(&ctl->ended, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  __syncthreads();
  if (!s_last) return;
  if (threadIdx.x < kNumCounters)
    __hip_atomic_store(&pinned->counters[threadIdx.x],
                       __hip_atomic_load(&counters[threadIdx.x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  wave_stores_done();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(flag, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// the control block into pinned memory, flag last; one wavefront, whose release covers every lane's stores
__global__ __launch_bounds__(64) void k_publish(const uint32_t* __restrict__ ctl, uint32_t n_words,
                                                uint32_t* pinned, uint32_t* flag) {
  for (uint32_t i = threadIdx.x; i < n_words; i += 64)
    __hip_atomic_store(&pinned[i], ctl[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  if (threadIdx.x == 0) __hip_atomic_store(flag, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Rows with more than `threshold` entries, compacted in any order (the CSR kernel gives each of
// them a workgroup of its own).  The list has room for nnz / threshold + 1 rows.
__global__ void k_find_long_rows(const int32_t* __restrict__ rowptr, int64_t M, int threshold,
                                 uint32_t* __restrict__ list, unsigned long long* counter) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M) return;
  if (rowptr[i + 1] - rowptr[i] > threshold) list[atomicAdd(counter, 1ull)] = (uint32_t)i;
}

// ---------------------------------------------------------------- scan
// Three-pass exclusive scan (block sums, scan of block sums, rescan + offset).
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;

struct LoadU8 { const uint8_t* p; __device__ uint32_t operator()(int64_t i) const { return p[i]; } };
struct LoadU32 { const uint32_t* p; __device__ uint32_t operator()(int64_t i) const { return p[i]; } };
struct LoadPopc { const uint64_t* p; __device__ uint32_t operator()(int64_t i) const { return __popcll(p[i]); } };
struct LoadNonZero { const uint64_t* p; __device__ uint32_t operator()(int64_t i) const { return p[i] != 0 ? 1u : 0u; } };

// exclusive scan of one value per thread across the block; returns the block total
__device__ inline uint32_t block_exclusive(uint32_t v, uint32_t* total_out) {
  __shared__ uint32_t wave_sum[kScanThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(incl, d, 64);
    if (lane >= d) incl += up;
  }
  __syncthreads();  // protect wave_sum from the previous use
  if (lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  uint32_t base = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) {
    if (w < wave) base += wave_sum[w];
    total += wave_sum[w];
  }
  *total_out = total;
  return base + incl - v;
}

template <typename Load>
__global__ void k_scan_block_sums(Load load, int64_t n, uint32_t* __restrict__ block_sums) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k)
    if (base + k < n) s += load(base + k);
  uint32_t total;
  block_exclusive(s, &total);
  if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

// single block: in-place exclusive scan of block_sums[0..nblocks), total to *grand
__global__ void k_scan_of_sums(uint32_t* __restrict__ block_sums, int64_t nblocks,
                               uint32_t* __restrict__ grand) {
  uint32_t carry = 0;
  for (int64_t base = 0; base < nblocks; base += kScanThreads) {
    const int64_t i = base + threadIdx.x;
    const uint32_t v = i < nblocks ? block_sums[i] : 0;
    uint32_t total;
    const uint32_t ex = block_exclusive(v, &total);
    if (i < nblocks) block_sums[i] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) *grand = carry;
}

template <typename Load>
__global__ void k_scan_final(Load load, int64_t n, const uint32_t* __restrict__ block_offsets,
                             uint32_t* __restrict__ out) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = base + k < n ? load(base + k) : 0;
    s += v[k];
  }
  uint32_t total;
  uint32_t run = block_offsets[blockIdx.x] + block_exclusive(s, &total);
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) out[base + k] = run;
    run += v[k];
  }
}

template <typename Load>
hipError_t scan_impl(Load load, int64_t n, uint32_t* out, uint32_t* tmp, hipStream_t s) {
  // out[n] receives the total even when n == 0
  const int64_t nblocks = (n + kScanTile - 1) / kScanTile;
  if (nblocks > 0)
    hipLaunchKernelGGL(k_scan_block_sums<Load>, dim3((unsigned)nblocks), dim3(kScanThreads), 0, s,
                       load, n, tmp);
  hipLaunchKernelGGL(k_scan_of_sums, dim3(1), dim3(kScanThreads), 0, s, tmp, nblocks, out + n);
  if (nblocks > 0)
    hipLaunchKernelGGL(k_scan_final<Load>, dim3((unsigned)nblocks), dim3(kScanThreads), 0, s, load,
                       n, tmp, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- panel_ptr
// Bricks of each panel (a quarter of its active columns, rounded up), scanned; two launches of at
// most kPanelScanBlocks workgroups, each thread a run of `run` panels.  The first also totals the
// active columns and finds the largest column count; in the second every workgroup adds up the
// sums before its own, which saves the launch that would scan them.
constexpr int kPanelScanBlocks = 1024;

inline int64_t panel_scan_run(int64_t P) {
  return std::max<int64_t>(4, (P + (int64_t)kPanelScanBlocks * kScanThreads - 1) /
                                  ((int64_t)kPanelScanBlocks * kScanThreads));
}

__global__ __launch_bounds__(kScanThreads) void k_panel_sums(const uint32_t* __restrict__ ncols_p,
                                                             int64_t P, int64_t run,
                                                             uint32_t* __restrict__ block_sums,
                                                             PlanControl* ctl) {
  __shared__ unsigned long long s_cols, s_blocks;
  __shared__ uint32_t s_max;
  if (threadIdx.x == 0) { s_cols = 0; s_blocks = 0; s_max = 0; }
  const int64_t p0 = min(((int64_t)blockIdx.x * kScanThreads + threadIdx.x) * run, P);
  const int64_t p1 = min(p0 + run, P);
  uint32_t bricks = 0, most = 0;
  unsigned long long cols = 0, blocks = 0;
  for (int64_t p = p0; p < p1; ++p) {
    const uint32_t n = ncols_p[p];
    bricks += (n + kBrickK - 1) / kBrickK;
    blocks += ((n + kBrickK - 1) / kBrickK + kBrickK - 1) / kBrickK;
    cols += n;
    most = max(most, n);
  }
  uint32_t total;
  block_exclusive(bricks, &total);   // (its barriers also cover the zeroing above)
  cols = wave_sum(cols);
  blocks = wave_sum(blocks);
  most = wave_max(most);
  if (cols && (threadIdx.x & 63) == 0) {
    atomicAdd(&s_cols, cols);
    atomicAdd(&s_blocks, blocks);
    atomicMax(&s_max, most);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    block_sums[blockIdx.x] = total;
    if (s_cols) {
      atomicAdd(&ctl->n_active, s_cols);
      atomicAdd(&ctl->n_blocks, s_blocks);
      raise_to(&ctl->max_cols, s_max);
    }
  }
}

__global__ __launch_bounds__(kScanThreads) void k_panel_scan(const uint32_t* __restrict__ ncols_p,
                                                             int64_t P, int64_t run,
                                                             const uint32_t* __restrict__ block_sums,
                                                             uint32_t* __restrict__ panel_ptr,
                                                             PlanControl* ctl) {
  uint32_t before = 0;
  for (uint32_t b = threadIdx.x; b < blockIdx.x; b += kScanThreads) before += block_sums[b];
  uint32_t base;
  block_exclusive(before, &base);
  const int64_t p0 = min(((int64_t)blockIdx.x * kScanThreads + threadIdx.x) * run, P);
  const int64_t p1 = min(p0 + run, P);
  uint32_t bricks = 0;
  for (int64_t p = p0; p < p1; ++p) bricks += (ncols_p[p] + kBrickK - 1) / kBrickK;
  uint32_t total;
  uint32_t at = base + block_exclusive(bricks, &total);
  for (int64_t p = p0; p < p1; ++p) {
    panel_ptr[p] = at;
    at += (ncols_p[p] + kBrickK - 1) / kBrickK;
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    panel_ptr[P] = base + total;
    ctl->nb = base + total;
  }
}

// The same in one launch, for as many panels as a workgroup adds up while it could wait for another launch:
// each adds up the bricks of all panels before its own, the last one everything.  20,360 panels: 5.0 + 5.0 us and the
// gap between -> 7.6; 62,500: 6.0 + 5.0 -> 10.6.
constexpr int kOneScanThreads = 1024;
constexpr int64_t kOneScanPanels = 1 << 16;

__global__ __launch_bounds__(kOneScanThreads) void k_panel_scan_one(const uint32_t* __restrict__ ncols_p, int64_t P,
                                                                    uint32_t* __restrict__ panel_ptr, PlanControl* ctl) {
  constexpr int kWaves = kOneScanThreads / 64, kOwn = 4;
  struct Sums { uint32_t bricks, blocks, most; unsigned long long cols; };
  __shared__ Sums s_before[kWaves], s_own[kWaves];
  auto add = [](Sums& t, uint32_t n) {
    const uint32_t b = (n + kBrickK - 1) / kBrickK;
    t.bricks += b;
    t.blocks += (b + kBrickK - 1) / kBrickK;
    t.most = max(t.most, n);
    t.cols += n;
  };
  auto over_wave = [](Sums t) {
    return Sums{wave_sum(t.bricks), wave_sum(t.blocks), wave_max(t.most), wave_sum(t.cols)};
  };
  const int64_t first = (int64_t)blockIdx.x * kOneScanThreads * kOwn;
  Sums before{};
  for (int64_t p = 4 * threadIdx.x; p < first; p += 4 * kOneScanThreads) {   // (first is a multiple of the step)
    const uint4 n = *reinterpret_cast<const uint4*>(ncols_p + p);
    add(before, n.x); add(before, n.y); add(before, n.z); add(before, n.w);
  }
  const int64_t p0 = first + kOwn * threadIdx.x;
  uint32_t nb[kOwn];
  Sums own{};
#pragma unroll
  for (int k = 0; k < kOwn; ++k) {
    const uint32_t n = p0 + k < P ? ncols_p[p0 + k] : 0u;
    nb[k] = (n + kBrickK - 1) / kBrickK;
    add(own, n);
  }
  const int wave = threadIdx.x >> 6;
  const uint32_t mine = own.bricks;
  uint32_t in_wave = mine;   // exclusive scan across the wavefront
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(in_wave, d, 64);
    if ((int)(threadIdx.x & 63) >= d) in_wave += up;
  }
  in_wave -= mine;
  before = over_wave(before);
  own = over_wave(own);
  if ((threadIdx.x & 63) == 0) { s_before[wave] = before; s_own[wave] = own; }
  __syncthreads();
  uint32_t at = in_wave;
  for (int w = 0; w < kWaves; ++w) at += s_before[w].bricks + (w < wave ? s_own[w].bricks : 0u);
#pragma unroll
  for (int k = 0; k < kOwn; ++k) {
    if (p0 + k < P) panel_ptr[p0 + k] = at;
    at += nb[k];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    Sums t{};
    for (int w = 0; w < kWaves; ++w) {
      t.bricks += s_before[w].bricks + s_own[w].bricks;
      t.blocks += s_before[w].blocks + s_own[w].blocks;
      t.most = max(t.most, max(s_before[w].most, s_own[w].most));
      t.cols += s_before[w].cols + s_own[w].cols;
    }
    panel_ptr[P] = t.bricks;
    ctl->nb = t.bricks;
    ctl->n_active = t.cols;
    ctl->n_blocks = t.blocks;
    ctl->max_cols = t.most;
  }
}

// ---------------------------------------------------------------- per-panel path
// One wavefront (a 64-thread workgroup) per panel, the panel's active columns as a bitmap in
// LDS over the panel's column span [cmin, cmax]: setting a bit per entry is the census (a1),
// the number of set bits below a column is its rank (a2), and from the rank follow brick,
// brick column and pattern bit (a3, patterns accumulated in LDS) and, after a scan of the
// panel's pattern popcounts, the value positions (a4; a panel's values are contiguous, so
// brick_valptr needs no scan across panels).  Used when the widest panel span and the largest
// brick count of a panel fit in LDS; other matrices take the search-based kernels above.

struct PanelExtent {
  int64_t e0, e1;        // entries of the panel
  int32_t cmin, cmax;    // column span (valid if e0 < e1)
};

// exclusive scan of one value per lane across the wavefront; returns the total in *total_out
__device__ inline uint32_t wave_exclusive(uint32_t v, uint32_t* total_out) {
  const int lane = threadIdx.x & 63;
  uint32_t incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(incl, d, 64);
    if (lane >= d) incl += up;
  }
  *total_out = __shfl(incl, 63, 64);
  return incl - v;
}

// rows of panel p -> rp[0..16] (entry offsets, repeated past the last row), span of columns
__device__ inline PanelExtent panel_extent(const int32_t* __restrict__ rowptr,
                                           const int32_t* __restrict__ colind, int64_t M,
                                           int64_t p, int32_t* rp /* LDS [17] */) {
  const int64_t r0 = p * kPanel;
  if (threadIdx.x <= kPanel) rp[threadIdx.x] = rowptr[min(r0 + (int64_t)threadIdx.x, M)];
  __syncthreads();
  int32_t lo = 0x7FFFFFFF, hi = -1;
  if (threadIdx.x < kPanel) {
    const int32_t s = rp[threadIdx.x], t = rp[threadIdx.x + 1];
    if (s < t) {   // sorted rows: first and last entry bound the row's columns
      lo = colind[s];
      hi = colind[t - 1];
    }
  }
#pragma unroll
  for (int d = 8; d > 0; d >>= 1) {   // rows sit in lanes 0..15
    lo = min(lo, __shfl_xor(lo, d, 64));
    hi = max(hi, __shfl_xor(hi, d, 64));
  }
  lo = __shfl(lo, 0, 64);
  hi = __shfl(hi, 0, 64);
  return PanelExtent{rp[0], rp[kPanel], lo, hi};
}

// row (0..15) of entry e inside the panel whose row offsets are rp[0..16]
__device__ inline int row_in_panel(const int32_t* rp, int64_t e) {
  int r = 0;
#pragma unroll
  for (int d = 8; d > 0; d >>= 1)
    if (rp[r + d] <= e) r += d;
  return r;
}

// sets the panel's bitmap; checks the columns on the way (range, order, inside the span)
__device__ inline void panel_bitmap(const int32_t* __restrict__ colind, const PanelExtent& x,
                                    const int32_t* rp, int64_t K, uint32_t words, uint32_t* bm,
                                    uint32_t* err) {
  for (uint32_t w = threadIdx.x; w < words; w += kPanelThreads) bm[w] = 0;
  __syncthreads();
  uint32_t bad = 0;
  for (int64_t e = x.e0 + threadIdx.x; e < x.e1; e += kPanelThreads) {
    const int32_t j = colind[e];
    if (j < 0 || j >= K) bad |= kErrColRange;
    if (e > rp[row_in_panel(rp, e)] && colind[e - 1] >= j) bad |= kErrColOrder;
    if (j >= x.cmin && j <= x.cmax) {
      const uint32_t d = (uint32_t)(j - x.cmin);
      atomicOr(&bm[d >> 5], 1u << (d & 31));
    } else {
      bad |= kErrColOrder;   // outside the span its sorted row promised
    }
  }
  if (bad) atomicOr(err, bad);
  __syncthreads();
}

// a1/a2 (counting half): active columns of each panel; validates colind.  Requires a valid rowptr (the
// host has seen k_rows_census' verdict).  Dynamic LDS: the bitmap.
__global__ __launch_bounds__(kPanelThreads) void k_panel_census(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind, int64_t M, int64_t K,
    int64_t P, uint32_t words_cap, uint32_t* err, uint32_t* __restrict__ ncols_p) {
  extern __shared__ uint32_t lds[];
  __shared__ int32_t rp[kPanel + 1];
  const int64_t p = blockIdx.x;
  const PanelExtent x = panel_extent(rowptr, colind, M, p, rp);
  if (x.e0 >= x.e1 || x.cmax < x.cmin) {
    // Entries but an inverted span (the last column of every row lies below the first column
    // of some row): a row is stored in descending order, or a column is negative.  No bitmap
    // can hold that, so the per-entry checks below would never see it.
    if (threadIdx.x == 0) {
      if (x.e0 < x.e1) atomicOr(err, (uint32_t)kErrColOrder);
      ncols_p[p] = 0;
    }
    return;
  }
  const uint32_t words = (uint32_t)(x.cmax - x.cmin) / 32u + 1u;
  if (words > words_cap) {   // cannot happen for sorted rows (the cap comes from k_rows_census)
    if (threadIdx.x == 0) { atomicOr(err, (uint32_t)kErrColOrder); ncols_p[p] = 0; }
    return;
  }
  panel_bitmap(colind, x, rp, K, words, lds, err);
  uint32_t cnt = 0;
  for (uint32_t w = threadIdx.x; w < words; w += kPanelThreads) cnt += __popc(lds[w]);
  uint32_t total;
  wave_exclusive(cnt, &total);
  if (threadIdx.x == 0) ncols_p[p] = total;
}

// ---- rows and, for band-like matrices, the census in the same pass
// The first launch of every plan.  A wavefront takes a panel: checks its rowptr, copies it into the plan,
// writes the panel's entry offset, finds its column span and entry count (from which the plan chooses how to
// build), and, where a bitmap over that span is short, counts the panel's active columns as k_panel_census
// does.  A row's columns are bounded by its first and last entry; they are read only where the row's own
// offsets are in order and inside [0, nnz].  A panel with entries and an inverted span (the last column of
// every row below the first column of some row) is not sorted or has a negative column.
// A workgroup takes a run of panels and leaves its totals in `totals`, so nothing is added to a common
// counter and the scan that follows needs no pass of its own over the counts.  Entries are read four a lane,
// neighbours, whose columns mostly share a bitmap word and then cost one LDS atomic; only an entry that does
// not lie above the one before it looks up whether it begins a row.
// Bound by the latency of dependent loads, so the next panel's rows and the first rounds of entries are on their way
// early; it also clears the control block and the flags of columns, which takes a launch before it and its gap
// (2 us; 4096 rows: plan, product and destruction 54.6 -> 52.5 us).  262,144 rows, 7.86 M entries: a pass over the rows,
// a wait for their span and the census took 12 + 15 + 20 us, one pass 18.7, three workgroups a CU so 18.4, four 17.1; the
// rows of a graph of 20,360 panels 12.2 -> 9.6.
constexpr int kFirstThreads = 512, kFirstWaves = kFirstThreads / 64;
constexpr int kFirstBlocks = 1024;                  // four a CU
constexpr uint32_t kFirstWords = 512;               // bitmap words a wavefront: 16,384 columns
constexpr size_t kClearEach = 8;                    // vectors a thread clears at most

constexpr uint32_t kSortSmall = 512, kSortMid = 2048, kSortBig = 8192;   // entries; see the path that sorts

// of a workgroup's panels: two vectors, and every workgroup of the scan reads all at once (three of them, one after another:
// 16,384 panels 4.8 -> 5.1 us, now 4.45)
struct PanelTotals {
  uint32_t bricks, blocks, cols;
  uint32_t span, max_nnz;                 // the largest
  uint32_t err;                           // and kNotCounted
  float spans;                            // the sum
  uint16_t max_cols, listed;              // most of a panel; panels of more than kSortSmall entries, or 65,535
  __device__ void add(const PanelTotals& o) {
    bricks += o.bricks; blocks += o.blocks; cols += o.cols;
    span = max(span, o.span); max_nnz = max(max_nnz, o.max_nnz);
    err |= o.err;
    spans += o.spans;
    max_cols = max(max_cols, o.max_cols);
    listed = (uint16_t)min((uint32_t)listed + o.listed, 65535u);
  }
};
constexpr uint32_t kNotCounted = 1u << 31;            // a panel has no count
static_assert(kFirstWords * 32 <= 65535, "a panel's columns fit 16 bits");

typedef int32_t Int4Any __attribute__((ext_vector_type(4), aligned(4)));   // at any dword address

__device__ inline void wave_lds_fence() {   // LDS writes of the wavefront's lanes, seen by its other lanes
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(kFirstThreads, 8) void k_rows_census(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind, int64_t M, int64_t K,
    int64_t P, int64_t nnz, int64_t run, int32_t* __restrict__ rowptr_copy,
    uint32_t* __restrict__ panel_nnzptr, uint32_t* __restrict__ ncols_p,
    PanelTotals* __restrict__ totals, uint4* __restrict__ clear, uint32_t n_clear) {
  __shared__ uint32_t s_bm[kFirstWaves][kFirstWords];
  __shared__ int32_t s_rp[kFirstWaves][kPanel + 1];
  __shared__ PanelTotals s_tot[kFirstWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t* bm = s_bm[wave];
  int32_t* rp = s_rp[wave];
  PanelTotals t{};
  const int64_t p_end = min((int64_t)(blockIdx.x + 1) * run, P), p_first = (int64_t)blockIdx.x * run + wave;
  int32_t a_next = rowptr[min(p_first * kPanel + lane, M)];
  for (uint32_t i = blockIdx.x * kFirstThreads + threadIdx.x; i < n_clear; i += gridDim.x * kFirstThreads)
    clear[i] = uint4{0, 0, 0, 0};
  for (int64_t p = p_first; p < p_end; p += kFirstWaves) {
    const int64_t i = p * kPanel + lane;
    const int32_t a = a_next;
    a_next = rowptr[min(i + kFirstWaves * kPanel, M)];
    const int32_t b = __shfl_down(a, 1, 64);   // (row M's own offset past the last row)
    int32_t lo = 0x7FFFFFFF, hi = -1;
    uint32_t cnt = 0, err = 0;
    if (lane <= kPanel) rp[lane] = a;
    const bool row = lane < kPanel && i < M;
    const bool in_order = row && a >= 0 && a <= nnz && b >= a;
    const bool has = in_order && a < b && b <= nnz;
    if (row) {
      rowptr_copy[i] = a;
      if (i == 0 && a != 0) err |= kErrRowptrEnds;
      if (!in_order) err |= kErrRowptrOrder;
      if (has) cnt = (uint32_t)(b - a);
    }
    if (i == M && lane <= kPanel) {            // the end of the last row
      rowptr_copy[M] = a;
      panel_nnzptr[P] = (uint32_t)a;
      if (a != nnz) err |= kErrRowptrEnds;
      if (a < 0 || a > nnz) err |= kErrRowptrOrder;
    }
    if (lane == 0) panel_nnzptr[p] = (uint32_t)a;
    err = wave_or(err);
#pragma unroll
    for (int d = 8; d > 0; d >>= 1) cnt += __shfl_xor(cnt, d, 64);   // rows sit in lanes 0..15
    const uint32_t n = __builtin_amdgcn_readfirstlane(cnt);
    // The first two rounds of entries come with the rows' ends: with the rows in order, as they are without `err`
    // (but for the matrix's very end, which is another panel's), they are the n from the first row's offset on.
    const int32_t* __restrict__ col = colind + __builtin_amdgcn_readfirstlane(a);
    auto four = [&](uint32_t e, int32_t (&j)[4]) {
      if (e + 4 <= n) {
        const Int4Any v = *reinterpret_cast<const Int4Any*>(col + e);
        j[0] = v.x; j[1] = v.y; j[2] = v.z; j[3] = v.w;
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) j[k] = col[min(e + k, n - 1)];
      }
    };
    int32_t ahead[2][4] = {};
    if (has) {
      lo = colind[a];
      hi = colind[b - 1];
    }
    if (n && !err) {
      four(4 * lane, ahead[0]);
      if (n > 256) four(256 + 4 * lane, ahead[1]);
    }
#pragma unroll
    for (int d = 8; d > 0; d >>= 1) {
      lo = min(lo, __shfl_xor(lo, d, 64));
      hi = max(hi, __shfl_xor(hi, d, 64));
    }
    const int32_t cmin = __builtin_amdgcn_readfirstlane(lo), cmax = __builtin_amdgcn_readfirstlane(hi);
    t.max_nnz = max(t.max_nnz, n);
    t.listed = (uint16_t)min((uint32_t)t.listed + (n > kSortSmall), 65535u);
    if (cmax < cmin) {
      t.err |= err | (n ? (uint32_t)kErrColOrder : 0u);
      if (lane == 0) ncols_p[p] = 0;
      continue;
    }
    if (cmin < 0 || cmax >= K) err |= kErrColRange;   // (the span of such a panel may not fit 32 bits)
    const uint32_t span = (uint32_t)((int64_t)cmax - cmin + 1);
    const uint32_t words = (span + 31) / 32;
    t.span = max(t.span, span);
    t.spans += (float)span;
    t.err |= err;
    if (err || words > kFirstWords || words > 4 * n + 64) {
      t.err |= kNotCounted;
      continue;
    }

    // census
    for (uint32_t w = lane; w < words; w += 64) bm[w] = 0;
    wave_lds_fence();
    uint32_t bad = 0;
    int32_t last = -1;                         // the column before this round's first
    for (uint32_t base = 0; base < n; base += 256) {
      const uint32_t e = base + 4 * lane;
      int32_t j[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) { j[k] = ahead[0][k]; ahead[0][k] = ahead[1][k]; }
      if (base + 512 < n) four(e + 512, ahead[1]);
      int32_t before = __shfl_up(j[3], 1, 64);
      if (lane == 0) before = last;
      last = __shfl(j[3], 63, 64);
      uint32_t word = 0xFFFFFFFFu, bits = 0, unsure = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (e + k < n) {
          if (j[k] < 0 || j[k] >= K) bad |= kErrColRange;
          if ((k ? j[k > 0 ? k - 1 : 0] : before) >= j[k]) unsure |= 1u << k;
          if (j[k] >= cmin && j[k] <= cmax) {
            const uint32_t d = (uint32_t)(j[k] - cmin);
            if (d / 32 != word) {
              if (bits) atomicOr(&bm[word], bits);
              word = d / 32;
              bits = 0;
            }
            bits |= 1u << (d & 31);
          } else {
            bad |= kErrColOrder;   // outside the span its sorted row promised
          }
        }
      }
      if (bits) atomicOr(&bm[word], bits);
      while (unsure) {             // above its predecessor, or the first of a row
        const int64_t at = (int64_t)rp[0] + e + (uint32_t)__builtin_ctz(unsure);
        if (at > rp[row_in_panel(rp, at)]) bad |= kErrColOrder;
        unsure &= unsure - 1;
      }
    }
    wave_lds_fence();
    uint32_t cols = 0;
    for (uint32_t w = lane; w < words; w += 64) cols += __popc(bm[w]);
    cols = __builtin_amdgcn_readfirstlane(wave_sum(cols));
    t.err |= wave_or(bad);
    if (lane == 0) ncols_p[p] = cols;
    const uint32_t bricks = (cols + kBrickK - 1) / kBrickK;
    t.bricks += bricks;
    t.blocks += (bricks + kBrickK - 1) / kBrickK;
    t.cols += cols;
    t.max_cols = max(t.max_cols, (uint16_t)cols);
    wave_lds_fence();              // (bm and rp are the next panel's from here on)
  }
  if (P == 0 && threadIdx.x == 0) {
    const int32_t a = rowptr[0];
    rowptr_copy[0] = a;
    panel_nnzptr[0] = (uint32_t)a;
    if (a != 0 || a != nnz) t.err |= kErrRowptrEnds;
    if (a < 0 || a > nnz) t.err |= kErrRowptrOrder;
  }
  if (lane == 0) s_tot[wave] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < kFirstWaves; ++w) t.add(s_tot[w]);
    totals[blockIdx.x] = t;
  }
}

// panel_ptr from the counts and totals of k_rows_census (n_totals workgroups of `run` panels each); a
// workgroup here takes `group` of those runs.  Without every panel's count there is nothing to scan.  The
// first workgroup puts the matrix's totals into the control block and, for the host that waits for them,
// into pinned memory, flag last (a copy behind the kernels takes 4 us, and the wait for the stream more).
// Where the panels will be sorted, those of more than kSortSmall and of more than kSortMid entries are listed, in any
// order (a launch of its own: 2.9 us and the gap before it).
__global__ __launch_bounds__(kScanThreads) void k_census_scan(
    const uint32_t* __restrict__ ncols_p, int64_t P, int64_t run, const PanelTotals* __restrict__ totals,
    uint32_t n_totals, uint32_t group, uint32_t* __restrict__ panel_ptr, PlanControl* ctl,
    PlanControl* pinned, uint32_t* flag, int64_t nnz, const uint32_t* __restrict__ panel_nnzptr,
    uint32_t* __restrict__ mid_list, uint32_t* __restrict__ big_list) {
  __shared__ PanelTotals s_tot[kScanThreads / 64];
  __shared__ uint32_t s_before[kScanThreads / 64];
  PanelTotals t{};
  uint32_t before = 0;
  PanelTotals of[kFirstBlocks / kScanThreads];   // (all loads at once)
#pragma unroll
  for (int k = 0; k < kFirstBlocks / kScanThreads; ++k) of[k] = totals[min(k * kScanThreads + threadIdx.x, n_totals - 1)];
#pragma unroll
  for (int k = 0; k < kFirstBlocks / kScanThreads; ++k) {
    const uint32_t b = k * kScanThreads + threadIdx.x;
    if (b >= n_totals) break;
    if (b < blockIdx.x * group) before += of[k].bricks;
    t.add(of[k]);
  }
  t = PanelTotals{wave_sum(t.bricks), wave_sum(t.blocks), wave_sum(t.cols), wave_max(t.span), wave_max(t.max_nnz),
                  wave_or(t.err), wave_sum(t.spans), (uint16_t)wave_max((uint32_t)t.max_cols),
                  (uint16_t)min(wave_sum((uint32_t)t.listed), 65535u)};
  before = wave_sum(before);
  if ((threadIdx.x & 63) == 0) { s_tot[threadIdx.x >> 6] = t; s_before[threadIdx.x >> 6] = before; }
  __syncthreads();
  t = s_tot[0];
  uint32_t at = s_before[0];
#pragma unroll
  for (int w = 1; w < kScanThreads / 64; ++w) {
    const PanelTotals o = s_tot[w];
    t.add(o);
    at += s_before[w];
  }
  const bool counted = !t.err;
  t.err &= ~kNotCounted;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    PlanControl c;                 // (its counters stay as they are)
    c.err = t.err; c.span = t.span; c.max_nnz = t.max_nnz; c.counted = counted; c.spans = t.spans;
    c.n_listed = t.listed;
    c.max_cols = counted ? t.max_cols : 0;
    c.nb = counted ? t.bricks : 0;
    c.n_active = counted ? t.cols : 0;
    c.n_blocks = counted ? t.blocks : 0;
    for (PlanControl* to : {ctl, pinned}) {
      if (!to) continue;
      to->err = c.err; to->span = c.span; to->max_nnz = c.max_nnz; to->counted = c.counted; to->spans = c.spans;
      to->n_listed = c.n_listed;
      to->max_cols = c.max_cols; to->nb = c.nb; to->n_active = c.n_active; to->n_blocks = c.n_blocks;
    }
    if (counted) panel_ptr[P] = t.bricks;
    if (flag) __hip_atomic_store(flag, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  const int64_t p_end = min((int64_t)(blockIdx.x + 1) * group * run, P);
  const uint32_t words = panel_bitmap_words(t.span, P);
  const bool band = words != 0 && (int64_t)words * P <= kBandWords * nnz;   // (as the host chooses)
  if (!t.err && !band && t.max_nnz > kSortSmall) {   // (rowptr is in order: the lists have room)
    __shared__ uint32_t s_count[2], s_base[2];
    for (int64_t p0 = (int64_t)blockIdx.x * group * run; p0 < p_end; p0 += kScanThreads) {
      __syncthreads();
      if (threadIdx.x < 2) s_count[threadIdx.x] = 0;
      __syncthreads();
      const int64_t p = p0 + threadIdx.x;
      const uint32_t n = p < p_end ? panel_nnzptr[p + 1] - panel_nnzptr[p] : 0;
      const int which = n > kSortMid ? 1 : (n > kSortSmall ? 0 : -1);
      uint32_t in_block = 0;
      if (which >= 0) in_block = atomicAdd(&s_count[which], 1u);
      __syncthreads();
      if (threadIdx.x < 2 && s_count[threadIdx.x])
        s_base[threadIdx.x] = atomicAdd(threadIdx.x ? &ctl->n_big : &ctl->n_mid, s_count[threadIdx.x]);
      __syncthreads();
      if (which >= 0) (which ? big_list : mid_list)[s_base[which] + in_block] = (uint32_t)p;
    }
  }
  if (!counted) return;
  for (int64_t p0 = (int64_t)blockIdx.x * group * run; p0 < p_end; p0 += 4 * kScanThreads) {
    const int64_t p = p0 + 4 * threadIdx.x;
    uint32_t nb[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) nb[k] = p + k < p_end ? (ncols_p[p + k] + kBrickK - 1) / kBrickK : 0u;
    uint32_t total;
    uint32_t to = at + block_exclusive(nb[0] + nb[1] + nb[2] + nb[3], &total);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (p + k < p_end) panel_ptr[p + k] = to;
      to += nb[k];
    }
    at += total;
  }
}

// ---- per-panel path for scattered matrices: sort instead of a bitmap
// A panel's entries are sorted by (column, entry): equal columns end up next to each other, and the
// number of column changes before an entry is the rank of its column, whatever the width of the
// panel's column span.  Panels come in three classes of size, so that a few heavy panels cost the many light
// ones neither registers nor LDS: up to 512 entries a wavefront each, up to 2048 a
// workgroup of 256, up to 8192 one of 1024.  All sort in registers, up to eight keys a lane: a
// compare-exchange inside a lane is a min and a max, across lanes one cross-lane read a key, and only
// steps across wavefronts go through LDS (a sort all through LDS moved four words a pair and step).
// The columns of the largest class, and of few panels of the middle one beside it, are ranked by a bitmap of all columns
// instead, where that fits (k_panel_bitmap_census).
// The census leaves the entries, rank << 16 | index inside the panel, for the build, sorted or as they are stored.
// 20,360 panels of 46 entries, the largest 3000: the search-based kernels 167 us, sorting all classes 84.
// 18,750 panels of 430: a sort through LDS by one wavefront 163 + 101 us (census, build), now 84 + 67.
constexpr int kMidThreads = 256, kBigThreads = 1024;
static_assert(kMidThreads * 8 == kSortMid && kBigThreads * 8 == kSortBig, "eight keys a lane");

// A key is column << B | index.  In 32 bits, half the moves of a 64-bit one: B = 11 for panels of up to
// kSortMid entries and fewer than 2^21 columns (fewer, so that no key is all ones, which pads).  In 64 bits: B = 32.
constexpr int kMidBits = 11;
static_assert(kSortMid <= 1u << kMidBits, "indexes fit");
template <typename KT, int B> struct SortKey {
  static __device__ KT make(uint32_t col, uint32_t idx) { return ((KT)col << B) | idx; }
  static __device__ uint32_t col(KT k) { return (uint32_t)(k >> B); }
  static __device__ uint32_t idx(KT k) { return (uint32_t)(k & (((KT)1 << B) - 1)); }
};

// entries and row starts of panel p, as scalars (uniform addresses)
struct PanelRows {
  int64_t e0;
  uint32_t n;
  uint32_t start[kPanel];   // first entry of each row, relative to e0
  __device__ PanelRows(const int32_t* __restrict__ rowptr, int64_t M, int64_t p) {
    const int64_t r0 = p * kPanel;
    e0 = rowptr[r0];
    n = (uint32_t)(rowptr[min(r0 + kPanel, M)] - rowptr[r0]);
#pragma unroll
    for (int r = 0; r < kPanel; ++r) start[r] = (uint32_t)(rowptr[min(r0 + r, M)] - rowptr[r0]);
  }
  __device__ uint32_t row_of(uint32_t i) const {   // last row that starts at or before entry i
    uint32_t r = 0;
#pragma unroll
    for (int k = 1; k < kPanel; ++k) r += i >= start[k] ? 1u : 0u;
    return r;
  }
  __device__ bool starts_row(uint32_t i) const {
    bool is = false;
#pragma unroll
    for (int k = 0; k < kPanel; ++k) is |= i == start[k];
    return is;
  }
  // range and order of entry i's column
  __device__ uint32_t check(const int32_t* __restrict__ colind, int64_t K, uint32_t i, int32_t j) const {
    uint32_t bad = (j < 0 || j >= K) ? kErrColRange : 0u;
    if (!starts_row(i) && colind[e0 + i - 1] >= j) bad |= kErrColOrder;
    return bad;
  }
};

// exclusive scan of one value per thread across a workgroup of T threads (T = 64: across the
// wavefront); the total in *total_out.  `sums` is LDS for a word per wavefront
template <int T>
__device__ inline uint32_t group_exclusive(uint32_t v, uint32_t* total_out, uint32_t* sums) {
  uint32_t mine;
  const uint32_t ex = wave_exclusive(v, &mine);
  if constexpr (T == 64) {
    *total_out = mine;
    return ex;
  } else {
    __syncthreads();   // (the previous use has been read)
    if ((threadIdx.x & 63) == 0) sums[threadIdx.x >> 6] = mine;
    __syncthreads();
    uint32_t base = 0, total = 0;
#pragma unroll
    for (uint32_t w = 0; w < T / 64; ++w) {
      base += w < (threadIdx.x >> 6) ? sums[w] : 0;
      total += sums[w];
    }
    *total_out = total;
    return base + ex;
  }
}

// Bitonic sort of T * R keys, ascending in t * R + r for thread t of T (T = 64: for the lanes of a
// wavefront).  In the halves that a step sorts downwards the keys are held complemented, so every
// exchange puts the smaller key first.  `lds` holds T * R keys (T = 64: unused).
template <int T, int R, typename KT>
__device__ inline void group_sort(KT (&k)[R], KT* lds) {
  const uint32_t t = threadIdx.x & (T - 1);
  auto exchange = [&](int a, int b) {
    const KT lo = min(k[a], k[b]), hi = max(k[a], k[b]);
    k[a] = lo;
    k[b] = hi;
  };
  auto complement = [&](KT mask) {
#pragma unroll
    for (int r = 0; r < R; ++r) k[r] ^= mask;
  };
  // inside the lane: sizes 2 .. R (R itself upwards or downwards by lane)
#pragma unroll
  for (int size = 2; size <= R; size *= 2) {
    if (size == R) complement((t & 1) ? ~(KT)0 : (KT)0);
#pragma unroll
    for (int j = size / 2; j > 0; j /= 2) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r & j) continue;
        if (size < R && (r & size)) exchange(r | j, r);
        else exchange(r, r | j);
      }
    }
    if (size == R) complement((t & 1) ? ~(KT)0 : (KT)0);
  }
  // across lanes: sizes 2R .. T * R, that is 2 .. T lanes
#pragma unroll 1
  for (uint32_t lanes = 2; lanes <= (uint32_t)T; lanes *= 2) {
    const KT flip = (t & lanes) ? ~(KT)0 : (KT)0;   // (none at T: the whole is ascending)
    complement(flip);
#pragma unroll 1
    for (uint32_t m = lanes / 2; m > 0; m /= 2) {
      const bool keep_small = !(t & m);
      KT other[R];
      if (T > 64 && m >= 64) {
#pragma unroll
        for (int r = 0; r < R; ++r) lds[r * T + t] = k[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) other[r] = lds[r * T + (t ^ m)];
        __syncthreads();
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) other[r] = __shfl_xor(k[r], (int)m, 64);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) k[r] = (other[r] < k[r]) == keep_small ? other[r] : k[r];
    }
#pragma unroll
    for (int j = R / 2; j > 0; j /= 2)
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (!(r & j)) exchange(r, r | j);
    complement(flip);
  }
}

// one panel of at most T * R entries: sort, count the columns, leave the order; returns the count
template <int T, int R, int B, typename KT>
__device__ inline uint32_t group_census(const int32_t* __restrict__ colind, const PanelRows& x,
                                        int64_t K, uint32_t* err, uint32_t* __restrict__ order,
                                        KT* lds, uint32_t* sums) {
  const uint32_t t = threadIdx.x & (T - 1);
  KT k[R];
  uint32_t bad = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = r * T + t;
    k[r] = ~(KT)0;
    if (i < x.n) {
      const int32_t j = colind[x.e0 + i];
      bad |= x.check(colind, K, i, j);
      k[r] = SortKey<KT, B>::make((uint32_t)j, i);
    }
  }
  if (bad) atomicOr(err, bad);
  group_sort<T, R, KT>(k, lds);
  // changes of column: against the key before, the previous thread's last for the first of a thread
  KT before = __shfl_up(k[R - 1], 1, 64);
  if constexpr (T > 64) {
    lds[t] = k[R - 1];
    __syncthreads();
    if (t > 0) before = lds[t - 1];
  }
  uint32_t first = 0;   // bit r: a column begins at element t * R + r
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool is = r == 0 ? t == 0 || SortKey<KT, B>::col(k[0]) != SortKey<KT, B>::col(before)
                           : SortKey<KT, B>::col(k[r]) != SortKey<KT, B>::col(k[r > 0 ? r - 1 : 0]);
    first |= (is && t * R + r < x.n ? 1u : 0u) << r;
  }
  uint32_t total;
  uint32_t rank = group_exclusive<T>((uint32_t)__popc(first), &total, sums) - 1u;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    rank += (first >> r) & 1u;
    if (t * R + r < x.n) order[x.e0 + t * R + r] = rank << 16 | SortKey<KT, B>::idx(k[r]);
  }
  return total;
}

// Census of the panels of at most kSortMid entries; rowptr is valid, as above.  Those above kSortSmall,
// which are listed, take the first mid_blocks workgroups, one each (the host does not know their count
// yet); a wavefront takes each of the others.  One launch: the few hundred listed panels of a graph are
// a chain of latencies that hides among the many small ones (20,360 panels, 159 of them listed: 24 + 16
// us as two launches, 27 so).
template <typename KT, int B, bool MID>
__global__ __launch_bounds__(kMidThreads) void k_panel_sort_census(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind, int64_t M, int64_t K,
    int64_t P, const uint32_t* __restrict__ mid_list, const uint32_t* __restrict__ n_mid,
    uint32_t mid_blocks, uint32_t* err, uint32_t* __restrict__ ncols_p, uint32_t* __restrict__ order) {
  if constexpr (MID) {
    if (blockIdx.x < mid_blocks) {
      __shared__ KT lds[kSortMid];
      __shared__ uint32_t sums[kMidThreads / 64];
      if (blockIdx.x >= *n_mid) return;
      const int64_t p = mid_list[blockIdx.x];
      const PanelRows x(rowptr, M, p);
      uint32_t cols = 0;
      if (x.n <= kMidThreads * 4) cols = group_census<kMidThreads, 4, B, KT>(colind, x, K, err, order, lds, sums);
      else if (x.n <= kSortMid) cols = group_census<kMidThreads, 8, B, KT>(colind, x, K, err, order, lds, sums);
      if (threadIdx.x == 0) ncols_p[p] = cols;
      return;
    }
  }
  const int64_t p = (int64_t)(blockIdx.x - mid_blocks) * (kMidThreads / 64) +
                    __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (p >= P) return;
  const PanelRows x(rowptr, M, p);
  if (x.n > kSortSmall) return;
  uint32_t cols = 0;
  KT* none = nullptr;
  if (x.n == 0) cols = 0;
  else if (x.n <= 64) cols = group_census<64, 1, B, KT>(colind, x, K, err, order, none, nullptr);
  else if (x.n <= 128) cols = group_census<64, 2, B, KT>(colind, x, K, err, order, none, nullptr);
  else if (x.n <= 256) cols = group_census<64, 4, B, KT>(colind, x, K, err, order, none, nullptr);
  else cols = group_census<64, 8, B, KT>(colind, x, K, err, order, none, nullptr);
  if ((threadIdx.x & 63) == 0) ncols_p[p] = cols;
}

// census of the listed panels of at most kSortBig entries, a workgroup each (columns beyond the bitmaps, so keys of 64
// bits)
__global__ __launch_bounds__(kBigThreads) void k_panel_sort_census_big(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind, int64_t M, int64_t K,
    const uint32_t* __restrict__ list, const uint32_t* __restrict__ listed, uint32_t* err,
    uint32_t* __restrict__ ncols_p, uint32_t* __restrict__ order) {
  __shared__ unsigned long long lds[kSortBig];
  __shared__ uint32_t sums[kBigThreads / 64];
  if (blockIdx.x >= *listed) return;   // (the host does not know the count yet)
  const int64_t p = list[blockIdx.x];
  const PanelRows x(rowptr, M, p);
  uint32_t cols = 0;
  if (x.n <= kBigThreads * 4)
    cols = group_census<kBigThreads, 4, 32, unsigned long long>(colind, x, K, err, order, lds, sums);
  else if (x.n <= kSortBig)
    cols = group_census<kBigThreads, 8, 32, unsigned long long>(colind, x, K, err, order, lds, sums);
  if (threadIdx.x == 0) ncols_p[p] = cols;
}

// Census of listed panels by a bitmap of all columns, a workgroup each: no order, so no sort, and a rank from a
// table of the bits set before every eighth word.  `order` keeps the entries as they are stored.
// Bound by latency, so all loads of a thread are in flight at once.  A workgroup clears and counts the whole bitmap,
// however few entries it has, so which panels come here goes by how many they are.  us, census of all classes, sorted
// / the largest class by bitmap / the middle one, too (in brackets: panels of the largest, of the middle class):
//   graphs of 30,000 rows (4, 11) 32.0 / 20.8 / 15.8; of 326,000 (32, 156) 44.3 / 34.6 / 32.6; of 460,000 (53, 219) 50.7 / 43.0 / 44.3
//   65,536 columns, 4000 and 600 entries, (1, 450) 29.3 / 19.2 / 15.1; 8000 entries, (16, 1000) 50.9 / 24.8 / 23.5
//   262,144 columns, 4000 and 600 entries, (1, 0) 33.0 / 23.8; (16, 450) 37.9 / 28.4 / 26.2; (16, 1000) 41.7 / 32.9 / 33.4; (64, 3000)
//     56.7 / 47.1 / 59.3; (700, 450) 64.2 / 40.3 / 42.0
//   524,288 columns, (16, 450) 59.1 / 41.9 / 41.9; (16, 1000) 62.8 / 45.8 / 54.1; (64, 3000) 77.4 / 60.1 / 99.1; (700, 0) 99.3 / 56.6;
//     2100 entries, (1500, 0) 156 / 73
// The largest class is ahead everywhere: it is spared a launch and the longest sorts.  The middle class alone, whose
// sorts run beside those of the small panels, is behind (65,536 columns, 16 panels of 600 10.1 / 12.3; 524,288, 4096 of
// them 53.7 / 114.7), and with the largest ahead as long as all are one round of workgroups, two a CU.
// Bitmaps of a million columns leave a CU one workgroup: 640 listed panels 65 us, sorted 40.
constexpr int kListedThreads = 1024;
constexpr uint32_t kListedMaxWords = 16384;          // 512 Ki columns: 72 KiB of LDS with the table
constexpr uint32_t kListedRound = 512;

__global__ __launch_bounds__(kListedThreads) void k_panel_bitmap_census(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind, int64_t M, int64_t K,
    const uint32_t* __restrict__ mid_list, const uint32_t* __restrict__ big_list, const PlanControl* ctl,
    bool with_mid, uint32_t words, uint32_t* err, uint32_t* __restrict__ ncols_p, uint32_t* __restrict__ order) {
  extern __shared__ uint32_t lds[];
  __shared__ uint32_t sums[kListedThreads / 64];
  uint32_t *bm = lds, *pre = lds + words;   // [words], [words / kGroupWords, rounded up]
  const uint32_t n_big = ctl->n_big, n_mid = with_mid ? ctl->n_mid : 0u;   // (the host does not know them yet)
  if (blockIdx.x >= n_big + n_mid) return;
  const int64_t p = blockIdx.x < n_big ? big_list[blockIdx.x] : mid_list[blockIdx.x - n_big];
  const PanelRows x(rowptr, M, p);
  constexpr int R = kSortBig / kListedThreads;
  int32_t j[R], before[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = r * kListedThreads + threadIdx.x;
    j[r] = i < x.n ? colind[x.e0 + i] : -1;
    before[r] = i < x.n && i > 0 ? colind[x.e0 + i - 1] : -1;
  }
  for (uint32_t w = threadIdx.x; w < words; w += kListedThreads) bm[w] = 0;
  __syncthreads();
  uint32_t bad = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = r * kListedThreads + threadIdx.x;
    if (i < x.n) {
      if (before[r] >= j[r] && !x.starts_row(i)) bad |= kErrColOrder;
      if (j[r] < 0 || j[r] >= K) bad |= kErrColRange;
      else atomicOr(&bm[(uint32_t)j[r] >> 5], 1u << (j[r] & 31));
    }
  }
  if (bad) atomicOr(err, bad);
  __syncthreads();
  const uint32_t groups = (words + kGroupWords - 1) / kGroupWords;
  const uint32_t per = (groups + kListedThreads - 1) / kListedThreads;
  const uint32_t g0 = min(threadIdx.x * per, groups), g1 = min(g0 + per, groups);
  uint32_t mine = 0;
  for (uint32_t g = g0; g < g1; ++g) {
    uint32_t c = 0;
    for (uint32_t w = g * kGroupWords; w < min((g + 1) * kGroupWords, words); ++w) c += __popc(bm[w]);
    pre[g] = c;
    mine += c;
  }
  uint32_t total;
  uint32_t run = group_exclusive<kListedThreads>(mine, &total, sums);
  for (uint32_t g = g0; g < g1; ++g) {
    const uint32_t c = pre[g];
    pre[g] = run;
    run += c;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = r * kListedThreads + threadIdx.x;
    if (i >= x.n || j[r] < 0 || j[r] >= K) continue;   // (with the latter the plan is refused)
    const uint32_t w = (uint32_t)j[r] >> 5;
    uint32_t rank = pre[w / kGroupWords] + __popc(bm[w] & ((1u << (j[r] & 31)) - 1u));
    for (uint32_t v = w & ~(kGroupWords - 1); v < w; ++v) rank += __popc(bm[v]);
    order[x.e0 + i] = rank << 16 | i;
  }
  if (threadIdx.x == 0) ncols_p[p] = total;
}

// a2 (placing half), a3 and a4 of the listed panels (n_first of `list`, then those of `rest`; no list:
// of all) of at most n_cap entries, from what the census left in `src` (which this kernel then overwrites with
// the entry of each packed value).  T threads a panel.  Dynamic LDS: patterns (nb_cap x u64), ranks and indexes
// (n_cap words), value offsets (nb_cap words), the order of the packed values (n_cap x two bytes),
// through which they leave in order, whole lines at a time.
template <int T>
__global__ __launch_bounds__(T) void k_panel_sort_build(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind,
    const float* __restrict__ vals, int64_t M, const uint32_t* __restrict__ list,
    const uint32_t* __restrict__ rest, uint32_t n_first, uint32_t n_cap, uint32_t nb_cap,
    const uint32_t* __restrict__ panel_ptr, const uint32_t* __restrict__ ncols_p, uint32_t* __restrict__ brick_cols,
    uint64_t* __restrict__ brick_mask, uint32_t* __restrict__ brick_valptr,
    float* __restrict__ packed, uint32_t* src, uint8_t* __restrict__ col_seen) {
  extern __shared__ unsigned long long lds64[];
  __shared__ uint32_t sums[T / 64];
  unsigned long long* pat = lds64;                                   // [nb_cap]
  uint32_t* ent = reinterpret_cast<uint32_t*>(pat + nb_cap);         // [n_cap]: rank << 16 | index
  uint32_t* vptr = ent + n_cap;                                      // [nb_cap]
  uint16_t* at = reinterpret_cast<uint16_t*>(vptr + nb_cap);         // [n_cap]
  const int64_t p = !list ? blockIdx.x : blockIdx.x < n_first ? list[blockIdx.x] : rest[blockIdx.x - n_first];
  const PanelRows x(rowptr, M, p);
  if (x.n == 0 || x.n > n_cap) return;
  const uint32_t n = x.n;
  const uint32_t pp = panel_ptr[p];
  const uint32_t nb = panel_ptr[p + 1] - pp;
  if (nb == 0 || nb > nb_cap) return;   // (cannot happen: the cap is a maximum)
  for (uint32_t k = threadIdx.x; k < nb; k += T) pat[k] = 0;
  for (uint32_t i = threadIdx.x; i < n; i += T) ent[i] = src[x.e0 + i];
  __syncthreads();

  // columns, from the first entry of each (entries that are not sorted may write one several times, all the same); the
  // tail of the last brick padded.  Pattern bits.
  const uint32_t ncols = ncols_p[p];
  auto rank_of = [&](uint32_t w) { return min(w >> 16, nb * kBrickK - 1); };
  auto index_of = [&](uint32_t w) { return min(w & 0xFFFFu, n - 1); };
  auto bit_of = [&](uint32_t w) { return x.row_of(index_of(w)) * kBrickK + rank_of(w) % kBrickK; };
  for (uint32_t i = threadIdx.x; i < n; i += T) {
    const uint32_t w = ent[i], rank = rank_of(w);
    if (i == 0 || (ent[i - 1] >> 16) != (w >> 16)) {
      const uint32_t col = (uint32_t)colind[x.e0 + index_of(w)];
      brick_cols[(int64_t)pp * kBrickK + rank] = col;
      col_seen[col] = 1;
    }
    atomicOr(&pat[rank / kBrickK], 1ull << bit_of(w));
  }
  for (uint32_t k = ncols + threadIdx.x; k < nb * kBrickK; k += T)
    brick_cols[(int64_t)pp * kBrickK + k] = kPadCol;
  __syncthreads();

  // a4: value offsets = entries before the panel + popcounts of the panel's earlier bricks
  uint32_t off = 0;
  for (uint32_t base = 0; base < nb; base += T) {
    const uint32_t k = base + threadIdx.x;
    uint32_t c = 0;
    if (k < nb) {
      const unsigned long long m = pat[k];
      brick_mask[pp + k] = m;
      c = (uint32_t)__popcll(m);
    }
    uint32_t total;
    const uint32_t ex = group_exclusive<T>(c, &total, sums);
    if (k < nb) {
      vptr[k] = off + ex;
      brick_valptr[pp + k] = (uint32_t)x.e0 + off + ex;
    }
    off += total;
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < n; i += T) {
    const uint32_t w = ent[i], k = rank_of(w) / kBrickK;
    const uint32_t pos = vptr[k] + (uint32_t)__popcll(pat[k] & ((1ull << bit_of(w)) - 1ull));
    if (pos < n) at[pos] = (uint16_t)index_of(w);   // (always, for a census and a build that agree)
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < n; i += T) {
    const uint32_t e = (uint32_t)x.e0 + min((uint32_t)at[i], n - 1);
    packed[x.e0 + i] = vals[e];
    src[x.e0 + i] = e;
  }
}

// a2 (placing half), a3 and a4 for one panel.  Dynamic LDS: patterns of the panel's bricks (nb_cap x
// u64), the bitmap (words_cap words), the rank table (words_cap / G + 1 words: set bits before every
// G-th word), value offsets of the panel's bricks (nb_cap words), and for panels of at most
// stage_cap entries a word per entry and their order (two bytes per entry).
// Bound by the latency of what one wavefront does in turn, so the columns are read once, four loads
// in flight, and an entry's row and rank are worked out once and kept in LDS; the packed values and
// their sources leave in order, whole lines at a time.  Panels above stage_cap go through the same
// steps without the staging: they read the columns again and scatter their values.
// 7.86 M entries in 16,384 panels: 71 us unstaged and walking groups of bitmap words, 49 us staged, 46.6 with
// four neighbouring columns a lane (one LDS atomic a bitmap word) and an entry's row from bit counts (18.5 M -> 14.3 M
// vector instructions), 44.3 with 16-bit steps for sources; 41 M entries in 57,696 panels 434 -> 250 us staged (0.76 GB).
template <int G>
__global__ __launch_bounds__(kPanelThreads) void k_panel_build(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind,
    const float* __restrict__ vals, int64_t M, int64_t K, uint32_t words_cap, uint32_t nb_cap,
    uint32_t stage_cap, const uint32_t* __restrict__ panel_ptr, uint32_t* __restrict__ brick_cols,
    uint64_t* __restrict__ brick_mask, uint32_t* __restrict__ brick_valptr,
    float* __restrict__ packed, ValueSources src, uint8_t* __restrict__ col_seen) {
  extern __shared__ unsigned long long lds64[];
  __shared__ int32_t rp[kPanel + 1];
  // staged panels: bit i of `starts` is set where a row with entries begins at entry i + 1, and rows[k] is the
  // k-th such row: an entry's row from two bit counts and a look into the table, not from a comparison with every
  // row's start
  __shared__ unsigned long long starts[kPanelStageMax / 64];
  __shared__ uint32_t rows[kPanel];
  unsigned long long* pat = lds64;                                   // [nb_cap]
  uint32_t* bm = reinterpret_cast<uint32_t*>(lds64 + nb_cap);        // [words_cap]
  uint32_t* pre = bm + words_cap;     // [words_cap / G + 1]; pre[g] = set bits in words [0, G*g)
  uint32_t* vptr = pre + words_cap / G + 1;                          // [nb_cap]
  uint32_t* key = vptr + nb_cap;                                     // [stage_cap]
  uint16_t* at = reinterpret_cast<uint16_t*>(key + stage_cap);       // [stage_cap]
  const int64_t p = blockIdx.x;
  const uint32_t pp = panel_ptr[p];
  const uint32_t nb = panel_ptr[p + 1] - pp;
  const PanelExtent x = panel_extent(rowptr, colind, M, p, rp);
  if (nb == 0) return;
  const uint32_t words = (uint32_t)(x.cmax - x.cmin) / 32u + 1u;
  if (words > words_cap || nb > nb_cap) return;   // (cannot happen: both caps are maxima)
  const uint32_t n = (uint32_t)(x.e1 - x.e0);
  const bool staged = n <= stage_cap;
  // row starts as scalars, relative to the panel's first entry
  uint32_t row_start[kPanel];
#pragma unroll
  for (int r = 0; r < kPanel; ++r)
    row_start[r] = __builtin_amdgcn_readfirstlane((uint32_t)(rp[r] - rp[0]));
  auto row_of = [&](uint32_t i) {   // last row that starts at or before entry i
    uint32_t r = 0;
#pragma unroll
    for (int k = 1; k < kPanel; ++k) r += i >= row_start[k] ? 1u : 0u;
    return r;
  };

  for (uint32_t k = threadIdx.x; k < nb; k += kPanelThreads) pat[k] = 0;
  for (uint32_t w = threadIdx.x; w < words; w += kPanelThreads) bm[w] = 0;
  static_assert(kPanelStageMax / 64 <= kPanelThreads, "a lane clears a word");
  if (threadIdx.x < kPanelStageMax / 64) starts[threadIdx.x] = 0;
  __syncthreads();
  if (staged) {
    const uint32_t r = min(threadIdx.x, (uint32_t)kPanel - 1);
    const uint32_t begin = (uint32_t)(rp[r] - rp[0]), end = (uint32_t)(rp[r + 1] - rp[0]);
    const bool has = threadIdx.x < kPanel && begin < end;
    const uint64_t which = __ballot(has);
    if (has) {
      rows[__popcll(which & ((1ull << threadIdx.x) - 1ull))] = r;
      if (begin > 0) atomicOr(&starts[(begin - 1) / 64], 1ull << ((begin - 1) % 64));
    }
  }
  for (uint32_t i0 = 4 * threadIdx.x; i0 < n; i0 += 4 * kPanelThreads) {
    uint32_t d[4];
    if (i0 + 4 <= n) {
      const Int4Any v = *reinterpret_cast<const Int4Any*>(colind + x.e0 + i0);
      d[0] = (uint32_t)(v.x - x.cmin); d[1] = (uint32_t)(v.y - x.cmin);
      d[2] = (uint32_t)(v.z - x.cmin); d[3] = (uint32_t)(v.w - x.cmin);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)   // past the end: the last entry again
        d[u] = (uint32_t)(colind[x.e0 + min(i0 + u, n - 1)] - x.cmin);
    }
    uint32_t word = d[0] >> 5, bits = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (d[u] >> 5 != word) {
        if (word < words) atomicOr(&bm[word], bits);
        word = d[u] >> 5;
        bits = 0;
      }
      bits |= 1u << (d[u] & 31);
      if (i0 + u < n && staged) key[i0 + u] = d[u];
    }
    if (word < words) atomicOr(&bm[word], bits);
  }
  __syncthreads();

  // rank table: exclusive scan over groups of G words, a contiguous run per lane
  const uint32_t ngroups = (words + G - 1) / G;
  const uint32_t per = (ngroups + kPanelThreads - 1) / kPanelThreads;
  const uint32_t g0 = min(threadIdx.x * per, ngroups), g1 = min(g0 + per, ngroups);
  uint32_t mine = 0;
  for (uint32_t g = g0; g < g1; ++g) {
    uint32_t s = 0;
    for (uint32_t w = g * G; w < min((g + 1) * G, words); ++w) s += __popc(bm[w]);
    pre[g] = s;
    mine += s;
  }
  uint32_t ncols;
  uint32_t run = wave_exclusive(mine, &ncols);
  for (uint32_t g = g0; g < g1; ++g) {
    const uint32_t s = pre[g];
    pre[g] = run;
    run += s;
  }
  __syncthreads();
  auto rank_of = [&](uint32_t d) {   // set bits before bit d
    const uint32_t w = d >> 5;
    uint32_t r = pre[w / G] + __popc(bm[w] & ((1u << (d & 31)) - 1u));
    if constexpr (G > 1)
      for (uint32_t v = w & ~(uint32_t)(G - 1); v < w; ++v) r += __popc(bm[v]);
    return r;
  };

  // a2: active columns in ascending order, four per brick, the tail padded; a lane takes the
  // columns of eight bits at a time
  for (uint32_t q = threadIdx.x; q < 4 * words; q += kPanelThreads) {
    uint32_t bits = (bm[q >> 2] >> (8 * (q & 3))) & 0xFFu;
    if (!bits) continue;
    uint32_t r = rank_of(8 * q);
    do {
      const uint32_t col = (uint32_t)x.cmin + 8u * q + (uint32_t)__builtin_ctz(bits);
      brick_cols[(int64_t)pp * kBrickK + r++] = col;
      col_seen[col] = 1;
      bits &= bits - 1;
    } while (bits);
  }
  for (uint32_t k = ncols + threadIdx.x; k < nb * kBrickK; k += kPanelThreads)
    brick_cols[(int64_t)pp * kBrickK + k] = kPadCol;

  // a3: pattern bits, accumulated in LDS; a staged entry keeps rank and row, 16 * rank + row
  auto entry_key = [&](uint32_t row, uint32_t d) { return min(rank_of(d), nb * kBrickK - 1) * kPanel + row; };
  auto unstaged_key = [&](uint32_t i) {
    return entry_key(row_of(i), (uint32_t)(colind[x.e0 + i] - x.cmin));
  };
  auto brick_of = [](uint32_t k) { return k / (kPanel * kBrickK); };
  auto bit_of = [](uint32_t k) { return k % kPanel * kBrickK + k / kPanel % kBrickK; };
  if (staged) {
    uint32_t before = 0;   // rows that begin in the entries before these 64, the first not counted
    for (uint32_t i0 = 0; i0 < n; i0 += kPanelThreads) {
      const unsigned long long m = starts[i0 / 64];
      const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)m), hi = __builtin_amdgcn_readfirstlane((uint32_t)(m >> 32));
      const uint32_t i = i0 + threadIdx.x;
      if (i < n) {
        const uint32_t nth = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, before));
        const uint32_t k = entry_key(rows[min(nth, (uint32_t)kPanel - 1)], key[i]);
        key[i] = k;
        atomicOr(&pat[brick_of(k)], 1ull << bit_of(k));
      }
      before += __popc(lo) + __popc(hi);
    }
  } else {
    for (uint32_t i = threadIdx.x; i < n; i += kPanelThreads) {
      const uint32_t k = unstaged_key(i);
      atomicOr(&pat[brick_of(k)], 1ull << bit_of(k));
    }
  }
  __syncthreads();

  // a4: value offsets = entries before the panel + popcounts of the panel's earlier bricks
  uint32_t carry = 0;
  for (uint32_t base = 0; base < nb; base += kPanelThreads) {
    const uint32_t k = base + threadIdx.x;
    uint32_t c = 0;
    if (k < nb) {
      const unsigned long long m = pat[k];
      brick_mask[pp + k] = m;
      c = (uint32_t)__popcll(m);
    }
    uint32_t total;
    const uint32_t ex = wave_exclusive(c, &total);
    if (k < nb) {
      vptr[k] = carry + ex;
      brick_valptr[pp + k] = (uint32_t)x.e0 + carry + ex;
    }
    carry += total;
  }
  __syncthreads();
  auto put_source = [&](uint32_t to, uint32_t from) {   // inside the panel
    if (src.steps) src.steps[x.e0 + to] = (int16_t)((int32_t)from - (int32_t)to);
    else src.entries[x.e0 + to] = (uint32_t)x.e0 + from;
  };
  auto place_of = [&](uint32_t k) {   // inside the panel's values
    return vptr[brick_of(k)] + (uint32_t)__popcll(pat[brick_of(k)] & ((1ull << bit_of(k)) - 1ull));
  };
  if (staged) {
    for (uint32_t i = threadIdx.x; i < n; i += kPanelThreads) {
      const uint32_t pos = place_of(key[i]);
      if (pos < n) at[pos] = (uint16_t)i;   // (always, for a census and a build that agree)
    }
    __syncthreads();
    for (uint32_t i0 = threadIdx.x; i0 < n; i0 += 4 * kPanelThreads) {
      uint32_t from[4];
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        from[u] = min((uint32_t)at[min(i0 + u * kPanelThreads, n - 1)], n - 1);
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = vals[x.e0 + from[u]];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t i = i0 + u * kPanelThreads;
        if (i < n) {
          packed[x.e0 + i] = v[u];
          put_source(i, from[u]);
        }
      }
    }
  } else {
    for (uint32_t i = threadIdx.x; i < n; i += kPanelThreads) {
      const uint32_t pos = place_of(unstaged_key(i));
      if (pos < n) {
        packed[x.e0 + pos] = vals[x.e0 + i];
        put_source(pos, i);
      }
    }
  }
}

}  // namespace

size_t scan_tmp_elems(int64_t n) { return (size_t)((n + kScanTile - 1) / kScanTile) + 1; }

hipError_t launch_scan_u8(const uint8_t* in, int64_t n, uint32_t* out, uint32_t* tmp, hipStream_t s) {
  return scan_impl(LoadU8{in}, n, out, tmp, s);
}
hipError_t launch_scan_u32(const uint32_t* in, int64_t n, uint32_t* out, uint32_t* tmp,
                           hipStream_t s) {
  return scan_impl(LoadU32{in}, n, out, tmp, s);
}
hipError_t launch_scan_popc64(const uint64_t* in, int64_t n, uint32_t* out, uint32_t* tmp,
                              hipStream_t s) {
  return scan_impl(LoadPopc{in}, n, out, tmp, s);
}

hipError_t launch_scan_nonzero64(const uint64_t* in, int64_t n, uint32_t* out, uint32_t* tmp,
                                 hipStream_t s) {
  return scan_impl(LoadNonZero{in}, n, out, tmp, s);
}

hipError_t launch_rows_census(const int32_t* rowptr, const int32_t* colind, int64_t M, int64_t K,
                              int64_t P, int64_t nnz, int32_t* rowptr_copy, uint32_t* panel_nnzptr,
                              uint32_t* ncols_p, uint32_t* panel_ptr, uint32_t* tmp, PlanControl* ctl,
                              PlanControl* pinned, uint32_t* flag, uint32_t* mid_list, uint32_t* big_list,
                              void* clear, size_t clear_bytes, hipStream_t s) {
  static_assert(sizeof(PanelTotals) == 32, "eight words of `tmp` each");
  PanelTotals* totals = reinterpret_cast<PanelTotals*>(tmp);
  const int64_t want = std::max<int64_t>(1, std::min<int64_t>((P + kFirstWaves - 1) / kFirstWaves, kFirstBlocks));
  const int64_t run = std::max<int64_t>(1, (P + want - 1) / want);
  const unsigned n = (unsigned)std::max<int64_t>(1, (P + run - 1) / run);
  // Few panels and many columns: more to clear than these workgroups should
  uint32_t n_clear = (uint32_t)(clear_bytes / sizeof(uint4));
  if (clear_bytes / sizeof(uint4) > kClearEach * kFirstThreads * n) {
    const hipError_t e = hipMemsetAsync(clear, 0, clear_bytes, s);
    if (e != hipSuccess) return e;
    n_clear = 0;
  }
  hipLaunchKernelGGL(k_rows_census, dim3(n), dim3(kFirstThreads), 0, s, rowptr, colind, M, K, P, nnz, run,
                     rowptr_copy, panel_nnzptr, ncols_p, totals, static_cast<uint4*>(clear), n_clear);
  const unsigned group = (unsigned)std::max<int64_t>(1, 4 * kScanThreads / run);
  hipLaunchKernelGGL(k_census_scan, dim3((n + group - 1) / group), dim3(kScanThreads), 0, s, ncols_p, P, run,
                     totals, n, group, panel_ptr, ctl, pinned, flag, nnz, panel_nnzptr, mid_list, big_list);
  return hipGetLastError();
}

size_t panel_scan_tmp_elems() {
  return std::max<size_t>(kPanelScanBlocks, kFirstBlocks * sizeof(PanelTotals) / sizeof(uint32_t));
}

hipError_t launch_panel_scan(const uint32_t* ncols_p, int64_t P, uint32_t* panel_ptr, uint32_t* tmp,
                             PlanControl* ctl, hipStream_t s) {
  if (P <= kOneScanPanels) {
    hipLaunchKernelGGL(k_panel_scan_one, dim3(grid_for(P, 4 * kOneScanThreads)), dim3(kOneScanThreads), 0, s,
                       ncols_p, P, panel_ptr, ctl);
    return hipGetLastError();
  }
  const int64_t run = panel_scan_run(P);
  const dim3 grid(grid_for((P + run - 1) / run, kScanThreads)), block(kScanThreads);
  hipLaunchKernelGGL(k_panel_sums, grid, block, 0, s, ncols_p, P, run, tmp, ctl);
  hipLaunchKernelGGL(k_panel_scan, grid, block, 0, s, ncols_p, P, run, tmp, panel_ptr, ctl);
  return hipGetLastError();
}

hipError_t launch_validate_cols(const int32_t* rowptr, const int32_t* colind, int64_t M, int64_t K,
                                int64_t nnz, uint32_t* ent_row, uint32_t* err, hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  hipLaunchKernelGGL(k_validate_cols, dim3(grid_for(nnz)), dim3(kThreads), 0, s, rowptr, colind, M,
                     K, nnz, ent_row, err);
  return hipGetLastError();
}

hipError_t launch_first_in_panel(const int32_t* rowptr, const int32_t* colind,
                                 const uint32_t* ent_row, int64_t nnz, uint8_t* first,
                                 uint32_t* link, hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  hipLaunchKernelGGL(k_first_in_panel, dim3(grid_for(nnz)), dim3(kThreads), 0, s, rowptr, colind,
                     ent_row, nnz, first, link);
  return hipGetLastError();
}

hipError_t launch_compact_first(const uint8_t* first, const uint32_t* first_scan, int64_t nnz,
                                uint32_t* first_list, hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  hipLaunchKernelGGL(k_compact_first, dim3(grid_for(nnz)), dim3(kThreads), 0, s, first, first_scan,
                     nnz, first_list);
  return hipGetLastError();
}

hipError_t launch_panel_counts(const int32_t* rowptr, const uint32_t* first_scan, int64_t M,
                               int64_t P, uint32_t* ncols_p, hipStream_t s) {
  if (P == 0) return hipSuccess;
  hipLaunchKernelGGL(k_panel_counts, dim3(grid_for(P)), dim3(kThreads), 0, s, rowptr, first_scan, M,
                     P, ncols_p);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill<uint32_t>, dim3(grid_for(n)), dim3(kThreads), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_fill_u64(uint64_t* p, int64_t n, uint64_t v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill<uint64_t>, dim3(grid_for(n)), dim3(kThreads), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_rank_first(const int32_t* rowptr, const int32_t* colind, const uint32_t* ent_row,
                             const uint32_t* first_list, const uint32_t* first_scan,
                             const uint32_t* panel_ptr, int64_t M, int64_t n_active,
                             uint32_t* ent_rank, uint32_t* brick_cols, hipStream_t s) {
  if (n_active == 0) return hipSuccess;
  hipLaunchKernelGGL(k_rank_first, dim3(grid_for(n_active)), dim3(kThreads), 0, s, rowptr, colind,
                     ent_row, first_list, first_scan, panel_ptr, M, n_active, ent_rank, brick_cols);
  return hipGetLastError();
}

hipError_t launch_scatter_bits(const int32_t* colind, const uint32_t* ent_row, const uint32_t* link,
                               const uint32_t* ent_rank, const uint32_t* panel_ptr, int64_t nnz,
                               uint64_t* brick_mask, uint32_t* ent_brick, uint8_t* ent_bit,
                               uint8_t* col_seen, hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter_bits, dim3(grid_for(nnz)), dim3(kThreads), 0, s, colind, ent_row,
                     link, ent_rank, panel_ptr, nnz, brick_mask, ent_brick, ent_bit, col_seen);
  return hipGetLastError();
}

hipError_t launch_pack_values(const float* vals, const uint32_t* ent_brick, const uint8_t* ent_bit,
                              const uint64_t* brick_mask, const uint32_t* brick_valptr,
                              int64_t nnz, float* packed, uint32_t* src, hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  hipLaunchKernelGGL(k_pack_values, dim3(grid_for(nnz)), dim3(kThreads), 0, s, vals, ent_brick,
                     ent_bit, brick_mask, brick_valptr, nnz, packed, src);
  return hipGetLastError();
}

template <typename Source>
static hipError_t update_values(const float* vals, Source src, int64_t nnz, float* packed, float* csr_vals,
                                hipStream_t s) {
  const dim3 grid(grid_for(nnz, kUpdateBlock)), block(kThreads);
  if (csr_vals)
    hipLaunchKernelGGL((k_update_values<Source, true>), grid, block, 0, s, vals, src, nnz, packed, csr_vals);
  else
    hipLaunchKernelGGL((k_update_values<Source, false>), grid, block, 0, s, vals, src, nnz, packed, csr_vals);
  return hipGetLastError();
}

hipError_t launch_update_values(const float* vals, const ValueSources& src, int64_t nnz, float* packed,
                                float* csr_vals, hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  return src.steps ? update_values(vals, StepSource{src.steps}, nnz, packed, csr_vals, s)
                   : update_values(vals, EntrySource{src.entries}, nnz, packed, csr_vals, s);
}

template <typename Source>
static hipError_t restore_csr(const BrickFormat& f, Source src, int64_t nb, int32_t* colind, float* csr_vals,
                              hipStream_t s) {
  const unsigned g = (unsigned)std::min<int64_t>(grid_for(nb, kThreads / 64), kRestoreBlocks);
  hipLaunchKernelGGL(k_restore_csr<Source>, dim3(g), dim3(kThreads), 0, s, f.brick_cols, f.brick_mask,
                     f.brick_valptr, f.vals, src, nb, colind, csr_vals);
  return hipGetLastError();
}

hipError_t launch_restore_csr(const BrickFormat& f, const ValueSources& src, int64_t nb, int32_t* colind,
                              float* csr_vals, hipStream_t s) {
  if (nb == 0) return hipSuccess;
  return src.steps ? restore_csr(f, StepSource{src.steps}, nb, colind, csr_vals, s)
                   : restore_csr(f, EntrySource{src.entries}, nb, colind, csr_vals, s);
}

hipError_t launch_publish(const PlanControl* ctl, PlanControl* pinned, uint32_t* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, reinterpret_cast<const uint32_t*>(ctl),
                     (uint32_t)(sizeof(PlanControl) / sizeof(uint32_t)), reinterpret_cast<uint32_t*>(pinned), flag);
  return hipGetLastError();
}

hipError_t launch_plan_stats(const uint32_t* panel_ptr, const uint32_t* panel_nnzptr, int64_t P,
                             uint32_t* brick_cols, uint64_t* brick_mask, uint32_t* brick_valptr,
                             float* vals, int64_t nb, int64_t nnz, const uint8_t* col_seen, int64_t K,
                             PlanControl* ctl, PlanControl* pinned, uint32_t* pinned_ptr,
                             uint32_t* flag, hipStream_t s) {
  const int64_t most = std::max(std::max(nb, P), K / 16 + 16);
  const unsigned g = nb == 0 ? 1u   // no brick: every count is zero
                             : (unsigned)std::min<int64_t>(grid_for(most, kStatThreads), kStatBlocks);
  hipLaunchKernelGGL(k_plan_stats, dim3(g), dim3(kStatThreads), 0, s, panel_ptr, panel_nnzptr,
                     nb == 0 ? 0 : P, brick_cols, brick_mask, brick_valptr, vals, nb, nnz, col_seen,
                     nb == 0 ? 0 : K, ctl, pinned, pinned_ptr, P + 1, flag);
  return hipGetLastError();
}

hipError_t launch_find_long_rows(const int32_t* rowptr, int64_t M, int threshold, uint32_t* list,
                                 unsigned long long* counter, hipStream_t s) {
  if (M == 0) return hipSuccess;
  hipLaunchKernelGGL(k_find_long_rows, dim3(grid_for(M)), dim3(kThreads), 0, s, rowptr, M,
                     threshold, list, counter);
  return hipGetLastError();
}

// ---- sort-based per-panel path
// (the census is the largest launch: a wavefront a panel and, of 256 threads, a workgroup for each
// 512 entries; a launch has fewer than 2^32 threads, which M from 2^30 on would take)
bool panel_sort_fits(int64_t P, int64_t nnz, uint32_t max_nnz) {
  return max_nnz <= kSortBig &&
         64 * (P + kMidThreads / 64) + kMidThreads * panel_mid_list_elems(nnz) < kMaxLaunchThreads;
}
int64_t panel_mid_list_elems(int64_t nnz) { return nnz / kSortSmall; }
int64_t panel_big_list_elems(int64_t nnz) { return nnz / kSortMid; }

hipError_t launch_panel_sort_census(const int32_t* rowptr, const int32_t* colind, int64_t M,
                                    int64_t K, int64_t P, int64_t nnz, uint32_t max_nnz, uint32_t n_listed,
                                    const uint32_t* mid_list, const uint32_t* big_list, PlanControl* ctl,
                                    uint32_t* ncols_p, uint32_t* order, hipStream_t s) {
  if (P == 0) return hipSuccess;
  const bool narrow = K < (int64_t(1) << (32 - kMidBits));
  const int64_t words = (K + 31) / 32;
  const bool bitmap = max_nnz > kSortMid && words <= kListedMaxWords;   // (see the kernel)
  const bool with_mid = bitmap && n_listed <= kListedRound;
  if (bitmap) {
    const size_t lds = (size_t)(words + (words + kGroupWords - 1) / kGroupWords) * 4;
    if (lds > 48 * 1024) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_panel_bitmap_census),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    const int64_t at_most = with_mid ? n_listed : std::min(P, panel_big_list_elems(nnz));
    hipLaunchKernelGGL(k_panel_bitmap_census, dim3((unsigned)at_most), dim3(kListedThreads), lds, s, rowptr, colind, M, K, mid_list, big_list, ctl, with_mid,
                       (uint32_t)words, &ctl->err, ncols_p, order);
  }
  const bool mid = max_nnz > kSortSmall && !with_mid;
  const unsigned mid_blocks = mid ? (unsigned)std::min(P, panel_mid_list_elems(nnz)) : 0u;
  const dim3 grid(mid_blocks + grid_for(P, kMidThreads / 64)), block(kMidThreads);
#define SPMM_LAUNCH_CENSUS(KT, BITS, MID)                                                         \
  hipLaunchKernelGGL((k_panel_sort_census<KT, BITS, MID>), grid, block, 0, s, rowptr, colind, M, K, \
                     P, mid_list, &ctl->n_mid, mid_blocks, &ctl->err, ncols_p, order)
  if (narrow) {
    if (mid) SPMM_LAUNCH_CENSUS(uint32_t, kMidBits, true);
    else SPMM_LAUNCH_CENSUS(uint32_t, kMidBits, false);
  } else {
    if (mid) SPMM_LAUNCH_CENSUS(unsigned long long, 32, true);
    else SPMM_LAUNCH_CENSUS(unsigned long long, 32, false);
  }
#undef SPMM_LAUNCH_CENSUS
  if (max_nnz > kSortMid && !bitmap) {
    const dim3 at_most((unsigned)std::min(P, panel_big_list_elems(nnz))), big(kBigThreads);
    hipLaunchKernelGGL(k_panel_sort_census_big, at_most, big, 0, s, rowptr, colind, M, K, big_list, &ctl->n_big,
                       &ctl->err, ncols_p, order);
  }
  return hipGetLastError();
}

constexpr uint32_t kSortBuildRound = 256;   // a workgroup per CU

template <int T>
static hipError_t sort_build(const int32_t* rowptr, const int32_t* colind, const float* vals,
                             int64_t M, const uint32_t* list, const uint32_t* rest,
                             uint32_t n_first, int64_t n_panels, uint32_t n_cap, uint32_t nb_cap,
                             const uint32_t* panel_ptr, const uint32_t* ncols_p, uint32_t* brick_cols,
                             uint64_t* brick_mask, uint32_t* brick_valptr, float* packed, uint32_t* src,
                             uint8_t* col_seen, hipStream_t s) {
  if (n_panels == 0) return hipSuccess;
  n_cap = (n_cap + 1) & ~1u;
  // All bricks of a panel but the last have four columns, so four entries at least.  With room for a
  // brick per entry the small class took 9 KiB a wavefront, 17 on a CU; with 4.6 KiB a CU is full
  // (20,360 panels 31 -> 25 us; spmm_plan of a million-row graph 302 -> 283).
  nb_cap = std::min(nb_cap, (n_cap + kBrickK - 1) / kBrickK);
  const size_t lds = (size_t)nb_cap * 12 + (size_t)n_cap * 6;   // at most 9 bytes x kSortBig
  if (lds > 48 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_panel_sort_build<T>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_panel_sort_build<T>, dim3((unsigned)n_panels), dim3(T), lds, s, rowptr, colind, vals, M, list,
                     rest, n_first, n_cap, nb_cap, panel_ptr, ncols_p, brick_cols,
                     brick_mask, brick_valptr, packed, src, col_seen);
  return hipGetLastError();
}

hipError_t launch_panel_sort_build(const int32_t* rowptr, const int32_t* colind, const float* vals,
                                   int64_t M, int64_t P, const PanelLists& l, uint32_t max_nnz,
                                   uint32_t max_bricks, const uint32_t* panel_ptr, const uint32_t* ncols_p,
                                   uint32_t* brick_cols, uint64_t* brick_mask,
                                   uint32_t* brick_valptr, float* packed, uint32_t* src,
                                   uint8_t* col_seen, hipStream_t s) {
  hipError_t e = sort_build<64>(rowptr, colind, vals, M, nullptr, nullptr, 0, P, std::min(max_nnz, kSortSmall),
                                   max_bricks, panel_ptr, ncols_p, brick_cols, brick_mask, brick_valptr, packed,
                                   src, col_seen, s);
  // Few listed panels are one round of workgroups: together, in the time of the largest (48 panels
  // above 2048 entries and 159 above 512: 15 + 10 us as two launches, 10 as one).  Many are
  // ahead with the smaller workgroups and the LDS that the smaller ones need.
  const bool together = l.n_big > 0 && l.n_big + l.n_mid <= kSortBuildRound;
  if (e == hipSuccess && !together)
    e = sort_build<kMidThreads>(rowptr, colind, vals, M, l.mid, nullptr, l.n_mid, l.n_mid,
                                   std::min(max_nnz, kSortMid), max_bricks, panel_ptr, ncols_p, brick_cols,
                                   brick_mask, brick_valptr, packed, src, col_seen, s);
  if (e == hipSuccess)
    e = sort_build<kBigThreads>(rowptr, colind, vals, M, l.big, l.mid, l.n_big,
                                   together ? l.n_big + l.n_mid : l.n_big, max_nnz, max_bricks, panel_ptr, ncols_p,
                                   brick_cols, brick_mask, brick_valptr, packed, src, col_seen, s);
  return e;
}

bool panel_build_fits(uint32_t words_cap, uint32_t nb_cap) {
  return panel_build_layout(words_cap, nb_cap, 0).bytes != 0;
}

hipError_t launch_panel_census(const int32_t* rowptr, const int32_t* colind, int64_t M, int64_t K,
                               int64_t P, uint32_t words_cap, uint32_t* err, uint32_t* ncols_p,
                               hipStream_t s) {
  if (P == 0) return hipSuccess;
  const size_t lds = (size_t)words_cap * 4;
  if (lds > 48 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_panel_census),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_panel_census, dim3((unsigned)P), dim3(kPanelThreads), lds, s, rowptr, colind,
                     M, K, P, words_cap, err, ncols_p);
  return hipGetLastError();
}

hipError_t launch_panel_build(const int32_t* rowptr, const int32_t* colind, const float* vals,
                              int64_t M, int64_t K, int64_t P, uint32_t words_cap, uint32_t nb_cap,
                              uint32_t max_nnz, const uint32_t* panel_ptr, uint32_t* brick_cols,
                              uint64_t* brick_mask, uint32_t* brick_valptr, float* packed,
                              const ValueSources& src, uint8_t* col_seen, hipStream_t s) {
  if (P == 0) return hipSuccess;
  const PanelBuildLayout layout = panel_build_layout(words_cap, nb_cap, max_nnz);
  if (layout.bytes == 0) return hipErrorInvalidValue;   // (the caller asked panel_build_fits)
  const bool fine = layout.group == 1;
  const uint32_t stage_cap = layout.stage_cap;
  const size_t lds = layout.bytes;
  const void* fn = fine ? reinterpret_cast<const void*>(k_panel_build<1>)
                        : reinterpret_cast<const void*>(k_panel_build<kGroupWords>);
  if (lds > 48 * 1024) {
    const hipError_t e =
        hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const dim3 grid((unsigned)P), block(kPanelThreads);
  if (fine)
    hipLaunchKernelGGL(k_panel_build<1>, grid, block, lds, s, rowptr, colind, vals, M, K, words_cap,
                       nb_cap, stage_cap, panel_ptr, brick_cols, brick_mask, brick_valptr, packed,
                       src, col_seen);
  else
    hipLaunchKernelGGL(k_panel_build<kGroupWords>, grid, block, lds, s, rowptr, colind, vals, M, K,
                       words_cap, nb_cap, stage_cap, panel_ptr, brick_cols, brick_mask, brick_valptr,
                       packed, src, col_seen);
  return hipGetLastError();
}

}  // namespace spmm
