// Kernels of one DPD time step with phase-field bounce-back on gfx950.
//
// Per-particle state lives in float4 arrays (16-byte loads and stores):
//   pos4 = (x, y, z, gid bits)   vel4 = (v, last event code bits)
//   frc4 = (f, 0)                vt4  = (predicted velocity, event code bits)
// Fluid particles are kept in cell-sorted order: the force kernel writes the
// state of slot s (the s-th particle of the cell list) to slot s of the next
// buffers, so each step's integrate kernel streams a nearly sorted array and
// the force kernel's gathers of neighbour cells hit consecutive addresses.
// Frozen wall particles are sorted by cell once, at create, and stored after
// the fluid in the position and predicted-velocity arrays (index nf + w, with
// zero predicted velocity), so that one merged list per cell (walls first,
// then fluid) serves the neighbour search without a fluid/wall branch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device.h"
#include "kernels.h"

namespace dpd {

namespace {

constexpr int kBlock = 256;

inline unsigned grid_for(int64_t n, int block = kBlock) {
  return (unsigned)((n + block - 1) / block);
}

// ---------------------------------------------------------------------------
// Upload and bookkeeping
// ---------------------------------------------------------------------------
__global__ void k_pack(int64_t n, const float *__restrict__ pos, const float *__restrict__ vel,
                       const uint32_t *__restrict__ gid, const int64_t *__restrict__ rows,
                       float4 *pos4, float4 *vel4, float4 *vt4, float4 *frc4) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const int64_t r = rows[p];
  const uint32_t g = gid ? gid[r] : (uint32_t)r;
  pos4[p] = make_float4(pos[3 * r], pos[3 * r + 1], pos[3 * r + 2], __uint_as_float(g));
  if (vel4) {
    const float4 v = make_float4(vel[3 * r], vel[3 * r + 1], vel[3 * r + 2], 0.0f);
    vel4[p] = v;
    if (vt4) vt4[p] = v;
  }
  if (frc4) frc4[p] = make_float4(0.f, 0.f, 0.f, 0.f);
}

__global__ void k_fill_zero(uint32_t *p, size_t nwords) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < nwords; i += stride) p[i] = 0u;
}

// Plain streaming copy, 16 bytes per thread per iteration (the traffic
// reference for hardware byte counters).
__global__ void k_copy16(float4 *__restrict__ dst, const float4 *__restrict__ src, size_t n16) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n16; i += stride) dst[i] = src[i];
}

// VALU calibration: every thread runs `iters` x 64 VALU instructions of one
// kind on 8 independent register chains (inline assembly, so the count is
// exact), then stores one value so that nothing is dead.  Kinds: 0
// v_fmac_f32, 1 v_mad_u64_u32 (the 32 x 32 -> 64-bit multiply of Philox),
// 2 v_xor_b32, 3 v_log_f32 (a transcendental).
#define DPD_PROBE8(INS) INS(0) INS(1) INS(2) INS(3) INS(4) INS(5) INS(6) INS(7)
template <int KIND>
__global__ __launch_bounds__(256) void k_valu_probe(int iters, float *out) {
  const uint32_t t = threadIdx.x + blockIdx.x * blockDim.x;
  float f[8];
  uint32_t u[8];
  uint64_t w[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    f[k] = (float)(t + k) * 1e-3f + 1.0f;
    u[k] = t * 2654435761u + (uint32_t)k;
    w[k] = (uint64_t)u[k] << 7;
  }
  const float fb = 1.0000001f, fc = 1e-7f;
  const uint32_t ub = 0x9E3779B9u;
  uint64_t cy = 0;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int rep = 0; rep < 8; ++rep) {
      if (KIND == 0) {
#define DPD_FMA(k) asm volatile("v_fmac_f32 %0, %1, %2" : "+v"(f[k]) : "v"(fb), "v"(fc));
        DPD_PROBE8(DPD_FMA)
#undef DPD_FMA
      } else if (KIND == 1) {
#define DPD_MAD(k) asm volatile("v_mad_u64_u32 %0, %1, %2, %3, %0" : "+v"(w[k]), "=s"(cy) : "v"(u[k]), "v"(ub));
        DPD_PROBE8(DPD_MAD)
#undef DPD_MAD
      } else if (KIND == 2) {
#define DPD_XOR(k) asm volatile("v_xor_b32 %0, %1, %0" : "+v"(u[k]) : "v"(ub));
        DPD_PROBE8(DPD_XOR)
#undef DPD_XOR
      } else {
#define DPD_LOG(k) asm volatile("v_log_f32 %0, %0" : "+v"(f[k]));
        DPD_PROBE8(DPD_LOG)
#undef DPD_LOG
      }
    }
  }
  float acc = 0.f;
#pragma unroll
  for (int k = 0; k < 8; ++k) acc += f[k] + (float)u[k] + (float)(uint32_t)w[k];
  out[t] = acc + (float)(uint32_t)cy;
}
#undef DPD_PROBE8

__global__ void k_copy1(uint8_t *__restrict__ dst, const uint8_t *__restrict__ src, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

// ---------------------------------------------------------------------------
// Counting sort into cells
// ---------------------------------------------------------------------------
// Run structure of equal cells across a wavefront (cell < 0: inactive lane).
struct RunInfo {
  unsigned long long heads;
  int len;     // run length, for head lanes
  bool head;
};

__device__ __forceinline__ RunInfo wave_runs(int cell) {
  const int lane = (int)__lane_id();
  const int prev = __shfl_up(cell, 1, 64);
  RunInfo r;
  r.head = lane == 0 || prev != cell;
  r.heads = __ballot(r.head);
  const unsigned long long after = lane == 63 ? 0ull : (r.heads >> (lane + 1));
  r.len = after ? __ffsll((long long)after) : 64 - lane;
  return r;
}

__device__ __forceinline__ int wave_rank(const RunInfo &r, int base) {
  const int lane = (int)__lane_id();
  const unsigned long long upto = lane == 63 ? r.heads : (r.heads & ((2ull << lane) - 1ull));
  const int h = 63 - __clzll((long long)upto);
  return __shfl(base, h, 64) + (lane - h);
}

// Rank of a lane's particle among the particles of its cell c (c < 0: none,
// the result unused), called by every lane of the wavefront: the lanes that
// share a cell (consecutive, as the particles arrive cell-sorted from the
// previous step) take their ranks with one atomic per run of equal cells.
// Ranks come in any order; the per-cell sort orders the cells' runs by
// storage index afterwards.
__device__ __forceinline__ int rank_in_cell(int c, int32_t *__restrict__ count) {
  const RunInfo r = wave_runs(c);
  int base = r.len;
  if (r.head && c >= 0) base = atomicAdd(&count[c], r.len);
  return wave_rank(r, base);
}

// Cell of each of n particles and its rank in that cell.
__global__ void k_bin(const KGeom G, int64_t cell_off, int64_t n, const float4 *__restrict__ pos4,
                      int32_t *__restrict__ cell_of, int32_t *__restrict__ rank_of,
                      int32_t *__restrict__ count) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int c = -1;
  if (p < n) {
    const float4 x = pos4[p];
    int cx, cy, cz;
    c = (int)cell_off + cell_index(G, x.x, x.y, x.z, cx, cy, cz);
    cell_of[p] = c;
  }
  const int k = rank_in_cell(c, count);
  if (p < n) rank_of[p] = k;
}

// Exclusive scan over the block's threads (kScanThreads, four wavefronts), and total.
template <typename V>
__device__ __forceinline__ V block_exclusive_scan(V v, V *lds, V &total) {
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  V incl = v;
  for (int d = 1; d < 64; d <<= 1) {
    const V o = __shfl_up(incl, d, 64);
    if (lane >= d) incl += o;
  }
  if (lane == 63) lds[wave] = incl;
  __syncthreads();
  V before = 0;
  total = 0;
  for (int w = 0; w < kScanThreads / 64; ++w) {
    if (w < wave) before += lds[w];
    total += lds[w];
  }
  __syncthreads();
  return before + incl - v;
}

// Sum of v over the block (kScanThreads threads, four wavefronts).
template <typename V>
__device__ __forceinline__ V block_sum(V v, V *lds) {
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  V t = 0;
  for (int w = 0; w < kScanThreads / 64; ++w) t += lds[w];
  __syncthreads();
  return t;
}

// Sum of count over the chunk [base, min(base + ITEMS kScanThreads, n)) into *out.
template <int ITEMS>
__device__ __forceinline__ void scan_reduce_chunk(int64_t base, int64_t n,
                                                  const int32_t *__restrict__ count,
                                                  int32_t *__restrict__ out, int *lds) {
  int acc = 0;
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int64_t i = base + (int64_t)k * kScanThreads + threadIdx.x;
    if (i < n) acc += count[i];
  }
  acc = block_sum(acc, lds);
  if (threadIdx.x == 0) *out = acc;
}

// With gridDim.y = 2 of the walls' counts too.
template <int ITEMS>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(int64_t n,
                                                              const int32_t *__restrict__ count,
                                                              int32_t *__restrict__ bsum,
                                                              const int32_t *__restrict__ wcount,
                                                              int32_t *__restrict__ wsum) {
  __shared__ int lds[kScanThreads / 64];
  scan_reduce_chunk<ITEMS>((int64_t)blockIdx.x * ITEMS * kScanThreads, n,
                           blockIdx.y ? wcount : count, (blockIdx.y ? wsum : bsum) + blockIdx.x,
                           lds);
}

// Each thread owns ITEMS consecutive cells; the block's cells are read
// through LDS so that global loads and stores stay coalesced.  The block's
// offset is the sum of the block sums bsum[0 .. blockIdx) of k_scan_reduce, added up
// (prior) while the counts are on their way.  With wall
// offsets wstart (exclusive scan of the static wall counts) it also writes
// the merged runs: start_all[c] = start[c] + wstart[c] begins cell c's run of
// walls then fluid, fluid_off[c] = start_all[c] + (walls in c) its fluid part.
// The chunk [base, min(base + ITEMS kScanThreads, n)) of the exclusive scan, offset
// by the sum of everything before it; the last chunk (last) also writes the
// entry n after the end.  count is cleared for the next step.
// BOTH: the walls' counts too, scanned into wstart in the upper halves of 64-bit
// sums.
template <int ITEMS, bool BOTH, typename V, typename Prior>
__device__ __forceinline__ void scan_down_chunk(int64_t base, int64_t n, bool last, Prior &&prior,
                                                int32_t *__restrict__ count,
                                                int32_t *__restrict__ wcount,
                                                int32_t *__restrict__ start,
                                                std::conditional_t<BOTH, int32_t, const int32_t>
                                                    *__restrict__ wstart,
                                                int32_t *__restrict__ start_all,
                                                int32_t *__restrict__ fluid_off, V *tile, V *lds) {
  V own[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int64_t i = base + k * kScanThreads + (int)threadIdx.x;
    own[k] = 0;
    if (i < n) {
      own[k] = count[i];
      if constexpr (BOTH) own[k] += (V)wcount[i] << 32;
    }
  }
  const V offset = prior();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int local = k * kScanThreads + (int)threadIdx.x;
    const int64_t i = base + local;
    if (i < n) {
      count[i] = 0;
      if constexpr (BOTH) wcount[i] = 0;
    }
    tile[local + local / 32] = own[k];
  }
  __syncthreads();
  V run = 0;
  const int first = (int)threadIdx.x * ITEMS;
  for (int k = 0; k < ITEMS; ++k) {
    const int local = first + k;
    run += tile[local + local / 32];
  }
  V total;
  V ex = block_exclusive_scan(run, lds, total) + offset;
  for (int k = 0; k < ITEMS; ++k) {
    const int local = first + k;
    const V v = tile[local + local / 32];
    tile[local + local / 32] = ex;
    ex += v;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int local = k * kScanThreads + (int)threadIdx.x;
    const int64_t i = base + local;
    if (i < n) {
      const V at = tile[local + local / 32];
      const int st = (int)at;
      start[i] = st;
      if constexpr (BOTH) {
        const int w0 = (int)(at >> 32);
        wstart[i] = w0;
        start_all[i] = st + w0;
        fluid_off[i] = st + w0 + (int)(own[k] >> 32);
      } else if (wstart) {
        const int w0 = wstart[i], w1 = wstart[i + 1];
        start_all[i] = st + w0;
        fluid_off[i] = st + w1;
      }
    }
  }
  if (last && threadIdx.x == kScanThreads - 1) {
    const V end = offset + total;
    start[n] = (int)end;
    if constexpr (BOTH) {
      wstart[n] = (int)(end >> 32);
      start_all[n] = (int)end + (int)(end >> 32);
    } else if (wstart) {
      start_all[n] = (int)end + wstart[n];
    }
  }
  __syncthreads();
}

template <int ITEMS>
__global__ __launch_bounds__(kScanThreads) void k_scan_down(
    int64_t n, int32_t *__restrict__ count, int32_t *__restrict__ start,
    const int32_t *__restrict__ bsum, const int32_t *__restrict__ wstart,
    int32_t *__restrict__ start_all, int32_t *__restrict__ fluid_off) {
  constexpr int chunk = ITEMS * kScanThreads;
  __shared__ int tile[chunk + chunk / 32];
  __shared__ int lds[kScanThreads / 64];
  scan_down_chunk<ITEMS, false>(
      (int64_t)blockIdx.x * chunk, n, blockIdx.x == gridDim.x - 1,
      [&] {
        int before = 0;
        for (int j = (int)threadIdx.x; j < (int)blockIdx.x; j += kScanThreads) before += bsum[j];
        return block_sum(before, lds);
      },
      count, nullptr, start, wstart, start_all, fluid_off, tile, lds);
}

// Moving walls: the walls' counts scanned into wstart in the same pass.
//
// After k_wall_move_bin (one launch per box with walls) five launches list fluid and
// moving walls together: k_scan_reduce, this one, k_scatter_both, k_sort_both and
// k_permute, and k_quant_runs writes the codes of large contexts.  The five take the
// place of nine of 5 to 8 us each, most of it the launch: a step of 746,000 fluid and
// 304,000 wall particles 178 to 167 us.  (With 16 cells a thread, from 2^20 cells on, the
// 64-bit sums take this kernel to 238 VGPRs, one wavefront per SIMD.)
template <int ITEMS>
__global__ __launch_bounds__(kScanThreads) void k_scan_down_both(
    int64_t n, int32_t *__restrict__ count, int32_t *__restrict__ start,
    const int32_t *__restrict__ bsum, int32_t *__restrict__ wcount, int32_t *__restrict__ wstart,
    const int32_t *__restrict__ wsum, int32_t *__restrict__ start_all,
    int32_t *__restrict__ fluid_off) {
  constexpr int chunk = ITEMS * kScanThreads;
  __shared__ long long tile[chunk + chunk / 32];
  __shared__ long long lds[kScanThreads / 64];
  scan_down_chunk<ITEMS, true>(
      (int64_t)blockIdx.x * chunk, n, blockIdx.x == gridDim.x - 1,
      [&] {
        long long before = 0;
        for (int j = (int)threadIdx.x; j < (int)blockIdx.x; j += kScanThreads)
          before += (long long)bsum[j] + ((long long)wsum[j] << 32);
        return block_sum(before, lds);
      },
      count, wcount, start, wstart, start_all, fluid_off, tile, lds);
}

// idx[start[cell_of[p]] + rank_of[p]] = p for the n entries.  Threads n ..
// n + nw - 1 write the wall part of the merged runs (wall w, cell-sorted in
// cell wcell[w], is index n + w of the position arrays), and with dk the
// first thread advances the force evaluation index, so that one launch does
// the work of three.
__device__ __forceinline__ void scatter_one(int64_t p, int64_t n, const int32_t *__restrict__ cell_of,
                                            const int32_t *__restrict__ rank_of,
                                            const int32_t *__restrict__ start,
                                            int32_t *__restrict__ idx, int64_t nw,
                                            const int32_t *__restrict__ wcell,
                                            const int32_t *__restrict__ wstart,
                                            const int32_t *__restrict__ start_all,
                                            int32_t *__restrict__ idx_all) {
  if (p < n) {
    idx[start[cell_of[p]] + rank_of[p]] = (int32_t)p;
    return;
  }
  const int64_t w = p - n;
  if (w >= nw) return;
  const int c = wcell[w];
  idx_all[start_all[c] + ((int)w - wstart[c])] = (int32_t)(n + w);
}

__global__ void k_scatter(int64_t n, const int32_t *__restrict__ cell_of,
                          const int32_t *__restrict__ rank_of, const int32_t *__restrict__ start,
                          int32_t *__restrict__ idx, int64_t nw, const int32_t *__restrict__ wcell,
                          const int32_t *__restrict__ wstart,
                          const int32_t *__restrict__ start_all, int32_t *__restrict__ idx_all,
                          unsigned long long *__restrict__ dk) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (dk && p == 0) *dk += 1ull;
  scatter_one(p, n, cell_of, rank_of, start, idx, nw, wcell, wstart, start_all, idx_all);
}

// The same for n fluid particles and nw walls, each in an index array of its own.
__global__ void k_scatter_both(int64_t n, const int32_t *__restrict__ cell_of,
                               const int32_t *__restrict__ rank_of,
                               const int32_t *__restrict__ start, int32_t *__restrict__ idx,
                               int64_t nw, const int32_t *__restrict__ wcell_of,
                               const int32_t *__restrict__ wrank_of,
                               const int32_t *__restrict__ wstart, int32_t *__restrict__ widx,
                               unsigned long long *__restrict__ dk) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (dk && p == 0) *dk += 1ull;
  if (p < n)
    idx[start[cell_of[p]] + rank_of[p]] = (int32_t)p;
  else if (p - n < nw)
    widx[wstart[wcell_of[p - n]] + wrank_of[p - n]] = (int32_t)(p - n);
}

// Insertion network of compare-exchanges over K registers.
template <int K>
__device__ __forceinline__ void sort_network(uint32_t (&v)[K]) {
#pragma unroll
  for (int i = 1; i < K; ++i)
#pragma unroll
    for (int j = i; j > 0; --j) {
      const uint32_t lo = min(v[j - 1], v[j]), hi = max(v[j - 1], v[j]);
      v[j - 1] = lo;
      v[j] = hi;
    }
}

// A cell's run of up to K storage indices (the common case: about four per
// cell at density 4), loaded into registers with independent loads and sorted by a
// fixed insertion network of compare-exchanges, the slots past the run padded
// with a key above every index; written back to idx and, if out, to out.
template <int K>
__device__ __forceinline__ void sort_run_regs(int32_t *__restrict__ idx, int a, int n,
                                              int32_t *__restrict__ out) {
  uint32_t v[K];
#pragma unroll
  for (int i = 0; i < K; ++i) v[i] = i < n ? (uint32_t)idx[a + i] : 0xffffffffu;
  sort_network<K>(v);
#pragma unroll
  for (int i = 0; i < K; ++i)
    if (i < n) {
      idx[a + i] = (int32_t)v[i];
      if (out) out[i] = (int32_t)v[i];
    }
}

// A cell's run idx[a .. b) sorted by storage index and, if out, copied to out:
// in registers up to 16, by an insertion sort in memory above.
__device__ __forceinline__ void sort_run(int32_t *__restrict__ idx, int a, int b,
                                         int32_t *__restrict__ out) {
  if (b - a <= 4) {
    sort_run_regs<4>(idx, a, b - a, out);
  } else if (b - a <= 8) {
    sort_run_regs<8>(idx, a, b - a, out);
  } else if (b - a <= 16) {
    sort_run_regs<16>(idx, a, b - a, out);
  } else {
    for (int i = a + 1; i < b; ++i) {
      const int v = idx[i];
      int j = i - 1;
      while (j >= a && idx[j] > v) {
        idx[j + 1] = idx[j];
        --j;
      }
      idx[j + 1] = v;
    }
    if (out)
      for (int i = a; i < b; ++i) out[i - a] = idx[i];
  }
}

// Atomic ranks arrive in any order: sort each cell's run by storage index so
// that the cell list, and every sum over it, is deterministic.  With key4 the
// run is sorted by the gid bits of key4[i].w instead, which makes the order
// independent of how the particles were stored before (used when a state is
// loaded from outside).  With idx_all the sorted run is also written to the
// fluid part of the merged run.
// Runs of up to 16 are sorted in registers (sort_run_regs); longer runs, and
// the gid order, by an insertion sort in memory.
template <bool BY_GID>
__device__ __forceinline__ void sort_cell(int64_t c, const int32_t *__restrict__ start,
                                          int32_t *__restrict__ idx,
                                          const float4 *__restrict__ key4,
                                          const int32_t *__restrict__ fluid_off,
                                          int32_t *__restrict__ idx_all) {
  const int a = start[c], b = start[c + 1];
  if (!BY_GID) {
    sort_run(idx, a, b, idx_all ? idx_all + fluid_off[c] : nullptr);
    return;
  }
  for (int i = a + 1; i < b; ++i) {
    const int v = idx[i];
    const uint32_t kv = __float_as_uint(key4[v].w);
    int j = i - 1;
    while (j >= a && __float_as_uint(key4[idx[j]].w) > kv) {
      idx[j + 1] = idx[j];
      --j;
    }
    idx[j + 1] = v;
  }
  if (idx_all) {
    const int o = fluid_off[c];
    for (int i = a; i < b; ++i) idx_all[o + (i - a)] = idx[i];
  }
}

template <bool BY_GID>
__global__ void k_sort_cells(int64_t ncell, const int32_t *__restrict__ start,
                             int32_t *__restrict__ idx, const float4 *__restrict__ key4,
                             const int32_t *__restrict__ fluid_off,
                             int32_t *__restrict__ idx_all) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncell) return;
  sort_cell<BY_GID>(c, start, idx, key4, fluid_off, idx_all);
}

// The walls' per-cell sort (by storage index, as sort_cell), which also
// writes the cell of every sorted position: cell_out[i] = c for i in
// [start[c], start[c + 1]).
__global__ void k_sort_wall_cells(int64_t ncell, const int32_t *__restrict__ start,
                                  int32_t *__restrict__ idx, int32_t *__restrict__ cell_out) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncell) return;
  sort_cell<false>(c, start, idx, nullptr, nullptr, nullptr);
  const int a = start[c], b = start[c + 1];
  for (int i = a; i < b; ++i) cell_out[i] = (int32_t)c;
}

// Fluid and moving walls: each cell's runs sorted by storage index, its merged run
// written, and the cell of each sorted wall.  The first half of the threads take the
// cells' fluid, the second (whole blocks) their walls.  (Moving the walls' records in
// the same launch held a thread for two more dependent loads per wall: 20 us instead of
// 8 and a launch of k_permute, 6.)
__global__ __launch_bounds__(kBlock) void k_sort_both(
    int64_t ncell, int64_t n, const int32_t *__restrict__ start, int32_t *__restrict__ idx,
    const int32_t *__restrict__ wstart, int32_t *__restrict__ widx,
    const int32_t *__restrict__ start_all, const int32_t *__restrict__ fluid_off,
    int32_t *__restrict__ idx_all, int32_t *__restrict__ wcell) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncell) return;
  if (blockIdx.y == 0) {
    sort_run(idx, start[c], start[c + 1], idx_all + fluid_off[c]);
    return;
  }
  const int a = wstart[c], b = wstart[c + 1], out = start_all[c] - a;
  sort_run(widx, a, b, nullptr);
  for (int w = a; w < b; ++w) {
    wcell[w] = (int32_t)c;
    idx_all[out + w] = (int32_t)(n + w);
  }
}

// The whole cell list of small boxes in one launch: the exclusive scan of a
// box's cell counts, the scatter of its fluid and walls and the per-cell sort, in
// LDS as 16-bit numbers within the box.  The four separate launches
// (scan_reduce, scan_down, scatter, sort_cells) take 4 to 5 us each, most of it
// the launch.  Every list has one entry order (cells in order, each sorted by
// storage index), so the result is theirs exactly (cstart and fluid_off, which
// only those launches and the brick kernel read, are not written).
//
// gridDim.y blocks share a box, each for an equal part of its cells: it adds up
// the counts before its part, scans the part, and takes the particles whose cell
// lies there from the whole box.  With one block per box the sort and the LDS
// traffic of one CU bound it (20 us at 16,000 particles); with 16 it is the chain
// of phases (8 us).  A single block clears the counts for the next step; blocks that
// share a box must not (others may still read), so the pair force after them does.
constexpr int kBoxThreads = 1024;

// The 19-exchange network over 8 keys.
__device__ __forceinline__ void sort8(uint32_t (&v)[8]) {
  constexpr int net[19][2] = {{0, 2}, {1, 3}, {4, 6}, {5, 7}, {0, 4}, {1, 5}, {2, 6},
                              {3, 7}, {0, 1}, {2, 3}, {4, 5}, {6, 7}, {2, 4}, {3, 5},
                              {1, 4}, {3, 6}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
  for (int q = 0; q < 19; ++q) {
    const uint32_t x = v[net[q][0]], y = v[net[q][1]];
    v[net[q][0]] = min(x, y);
    v[net[q][1]] = max(x, y);
  }
}

__global__ __launch_bounds__(kBoxThreads) void k_cells_box(
    const Box *__restrict__ boxes, int64_t NF, const int32_t *__restrict__ cell_of,
    const int32_t *__restrict__ rank_of, int32_t *__restrict__ count,
    const int32_t *__restrict__ wcstart, int32_t *__restrict__ start_all,
    int32_t *__restrict__ idx, int32_t *__restrict__ idx_all, const int32_t *__restrict__ wcell,
    const float4 *__restrict__ pos4, uint32_t *__restrict__ cq,
    unsigned long long *__restrict__ dk) {
  __shared__ uint16_t start[kBoxCells + 1];
  __shared__ uint16_t slot[kBoxFluid], cell[kBoxFluid];   // of each slot: particle and its cell
  __shared__ int wave_sum[kBoxThreads / 64], wave_before[kBoxThreads / 64];
  const int t = (int)threadIdx.x, parts = (int)gridDim.y, part = (int)blockIdx.y;
  const Box &B = boxes[blockIdx.x];
  const int co = (int)B.co, nc = (int)B.ncell, fo = (int)B.fo, nf = (int)B.nf;
  const int lo = (int)((int64_t)nc * part / parts), n = (int)((int64_t)nc * (part + 1) / parts) - lo;
  if (dk && blockIdx.x == 0 && part == 0 && t == 0) *dk += 1ull;
  int before = 0;   // particles in the cells before the part
#pragma unroll 4
  for (int c = t; c < lo; c += kBoxThreads) before += count[co + c];
#pragma unroll 4
  for (int c = t; c < n; c += kBoxThreads) {
    start[c] = (uint16_t)count[co + lo + c];
    if (parts == 1) count[co + c] = 0;
  }
  for (int m = 32; m > 0; m >>= 1) before += __shfl_xor(before, m, 64);
  if ((t & 63) == 0) wave_before[t >> 6] = before;
  __syncthreads();
  // each thread's run of cells (an odd number, against bank conflicts), after
  // those of the threads before it
  const int per = ((n + kBoxThreads - 1) / kBoxThreads) | 1;
  const int c0 = min(t * per, n), c1 = min(c0 + per, n);
  int sum = 0;
  for (int c = c0; c < c1; ++c) sum += start[c];
  int incl = sum;
  for (int d = 1; d < 64; d <<= 1) {
    const int v = __shfl_up(incl, d, 64);
    if ((t & 63) >= d) incl += v;
  }
  if ((t & 63) == 63) wave_sum[t >> 6] = incl;
  __syncthreads();
  int run = incl - sum, own = 0;
  before = 0;
  for (int w = 0; w < kBoxThreads / 64; ++w) {
    if (w < (t >> 6)) run += wave_sum[w];
    own += wave_sum[w];
    before += wave_before[w];
  }
  for (int c = c0; c < c1; ++c) {
    const int k = start[c];
    start[c] = (uint16_t)run;
    run += k;
  }
  if (t == 0) start[n] = (uint16_t)own;
  __syncthreads();
  const int first = fo + before;   // the part's first slot
  // eight rounds of the box's particles at a time (past the end: the last one
  // again), so that one round trip to memory serves eight
  for (int p0 = t; p0 < nf; p0 += 8 * kBoxThreads) {
    int c[8], r[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int p = fo + min(p0 + u * kBoxThreads, nf - 1);
      c[u] = cell_of[p] - co - lo;
      r[u] = rank_of[p];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int p = p0 + u * kBoxThreads;
      if (p < nf && c[u] >= 0 && c[u] < n) {
        const int s = start[c[u]] + r[u];
        slot[s] = (uint16_t)p;
        cell[s] = (uint16_t)c[u];
      }
    }
  }
  const int w1 = wcstart[co + lo + n];
#pragma unroll 4
  for (int w = wcstart[co + lo] + t; w < w1; w += kBoxThreads) {
    // entry start_all[c] + (w - wcstart[c]) of the merged runs
    const int e = first + start[wcell[w] - co - lo] + w;
    idx_all[e] = (int)NF + w;
    if (cq) {
      const float4 x = pos4[NF + w];
      cq[e] = qcode3(x.x, x.y, x.z);
    }
  }
#pragma unroll 4
  for (int c = t; c < n; c += kBoxThreads)
    start_all[co + lo + c] = first + start[c] + wcstart[co + lo + c];
  if (blockIdx.x == gridDim.x - 1 && part == parts - 1 && t == 0)
    start_all[co + nc] = fo + nf + wcstart[co + nc];
  __syncthreads();
  for (int c = t; c < n; c += kBoxThreads) {
    const int a = start[c], k = start[c + 1] - a;
    if (k < 2) continue;
    if (k <= 8) {
      uint32_t v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = i < k ? (uint32_t)slot[a + i] : 0xffffu;
      sort8(v);
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (i < k) slot[a + i] = (uint16_t)v[i];
    } else {
      for (int i = a + 1; i < a + k; ++i) {
        const uint16_t v = slot[i];
        int j = i - 1;
        while (j >= a && slot[j] > v) {
          slot[j + 1] = slot[j];
          --j;
        }
        slot[j + 1] = v;
      }
    }
  }
  __syncthreads();
#pragma unroll 4
  for (int s = t; s < own; s += kBoxThreads) {
    const int i = fo + slot[s], e = first + s + wcstart[co + lo + cell[s] + 1];
    idx[first + s] = i;
    idx_all[e] = i;
    if (cq) {
      const float4 x = pos4[i];
      cq[e] = qcode3(x.x, x.y, x.z);
    }
  }
}

// Coarse codes of the merged runs, cq[t] = qcode3(pos4[idx_all[t]]): one
// thread per entry, so that the index reads and code writes coalesce.
__global__ void k_quant_runs(int64_t n, const int32_t *__restrict__ idx_all,
                             const float4 *__restrict__ pos4, uint32_t *__restrict__ cq) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const float4 x = pos4[idx_all[t]];
  cq[t] = qcode3(x.x, x.y, x.z);
}

// The pad entry after fluid and walls: a position far outside the box, so
// that it never tests as a neighbour; the spare run-array entries after the
// last run name it.
__global__ void k_set_pad(float4 *pos4, float4 *vt4, int32_t *slack, int32_t pad) {
  *pos4 = make_float4(1e30f, 1e30f, 1e30f, __uint_as_float(0xFFFFFFFFu));
  if (vt4) *vt4 = make_float4(0.f, 0.f, 0.f, 0.f);
  if (slack)
    for (int u = 0; u < kIdxSlack; ++u) slack[u] = pad;
}

__global__ void k_cells(const KGeom G, int64_t cell_off, int64_t n,
                        const float4 *__restrict__ pos4, int32_t *__restrict__ cell) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const float4 x = pos4[p];
  int cx, cy, cz;
  cell[p] = (int)cell_off + cell_index(G, x.x, x.y, x.z, cx, cy, cz);
}

__global__ void k_permute(int64_t n, const int32_t *__restrict__ idx, const float4 *a_in,
                          float4 *a_out, const float4 *b_in, float4 *b_out, const float4 *c_in,
                          float4 *c_out, const float4 *d_in, float4 *d_out) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const int i = idx[s];
  if (a_in) a_out[s] = a_in[i];
  if (b_in) b_out[s] = b_in[i];
  if (c_in) c_out[s] = c_in[i];
  if (d_in) d_out[s] = d_in[i];
}

// ---------------------------------------------------------------------------
// Phase field: near-interface mask and create-time check
// ---------------------------------------------------------------------------
// One bit per grid cube (the cube with lower corner node (i, j, k)): set if
// any of its 8 corner nodes is negative.  A trilinear value inside a cube
// whose corners are all >= 0 is >= 0 in the rounding of the decision form
// (each lerp of non-negative values is non-negative), so particles in
// unflagged cubes cannot have phi < 0 and skip the interpolation.
// One thread per cube, so that the node reads coalesce (a thread per word of 32
// cubes read nodes 128 B apart: 4.8 ms for 672^3, 31 us for 80^3); a wavefront
// writes two words.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_cube_mask(const KGeom G, const T *__restrict__ grid,
                                                      int64_t nwords,
                                                      uint32_t *__restrict__ bits) {
  const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t nx = G.ng[0], ny = G.ng[1], nz = G.ng[2];
  bool neg = false;
  if (q < nx * ny * nz) {
    const int64_t r = q / nx;
    const int i = (int)(q - r * nx), j = (int)(r % ny), k = (int)(r / ny);
    const int i1 = i + 1 == nx ? 0 : i + 1;
    const int j1 = j + 1 == ny ? 0 : j + 1;
    const int k1 = k + 1 == nz ? 0 : k + 1;
    for (int dk = 0; dk < 2; ++dk)
      for (int dj = 0; dj < 2; ++dj) {
        const T *row = grid + ((dk ? k1 : k) * ny + (dj ? j1 : j)) * nx;
        neg |= row[i] < (T)0;
        neg |= row[i1] < (T)0;
      }
  }
  const unsigned long long m = __ballot(neg);
  const int lane = (int)__lane_id();
  const int64_t w = (q - lane) / 32 + (lane >> 5);
  if ((lane & 31) == 0 && w < nwords) bits[w] = (uint32_t)(m >> lane);
}

// The face layout of the phase field (PhiQuad): node (i, j, k) gets
// (phi(i, j, k), phi(i+1, j, k), phi(i, j+1, k), phi(i+1, j+1, k)).
template <typename T>
__global__ void k_build_quad(const KGeom G, const T *__restrict__ grid, int64_t nodes,
                             typename PhiQuad<T>::type *__restrict__ quad) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nodes) return;
  const int nx = G.ng[0], ny = G.ng[1];
  const int i = (int)(q % nx);
  const int64_t r = q / nx;
  const int j = (int)(r % ny);
  const int64_t k = r / ny;
  const int i1 = i + 1 == nx ? 0 : i + 1;
  const int j1 = j + 1 == ny ? 0 : j + 1;
  const T *row0 = grid + ((size_t)k * ny + j) * nx;
  const T *row1 = grid + ((size_t)k * ny + j1) * nx;
  typename PhiQuad<T>::type v;
  v.x = row0[i];
  v.y = row0[i1];
  v.z = row1[i];
  v.w = row1[i1];
  quad[q] = v;
}

__device__ __forceinline__ bool cube_flagged(const uint32_t *__restrict__ bits, size_t q) {
  return (bits[q >> 5] >> (q & 31)) & 1u;
}

template <typename T>
__global__ void k_check_grid(const T *__restrict__ grid, int64_t count, Status *st) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  unsigned long long bad = 0;
  for (; i < count; i += stride)
    if (!isfinite(grid[i])) ++bad;
  if (bad) atomicAdd(&st->bad_grid, bad);
}

template <typename T>
__global__ void k_check_phi(const KGeom G, const T *__restrict__ grid, int64_t n,
                            const float4 *__restrict__ pos4, Status *st) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const float4 x = pos4[p];
  if (phi_at(grid, G, x.x, x.y, x.z) < (T)0) atomicAdd(&st->bad_phi, 1ull);
}

// ---------------------------------------------------------------------------
// Integrate + reflect + bin (Groot-Warren drift, Sec. II.C bounce-back)
//
// Each thread advances PPT particles (p, p + kBlock, ... of a tile of PPT kBlock),
// so that their loads and atomics are in flight together.  Ranks within a
// cell come from one atomic per run of equal cells in a wavefront: the
// particles arrive sorted by their previous cell and most keep it, so runs
// are the common case.
// ---------------------------------------------------------------------------
struct Moved {
  float4 pos;  // new position, gid bits in w
  float4 vt;   // predicted velocity, event code bits in w
  int cell;
};

// Velocity of the solid at each reflection of a wavefront (the lanes with `here`, at
// their (x, y, z); called by every lane): that of the wall
// particle nearest to the point among the walls of the 27 cells around its
// cell, nearness by the FP32 pair-decision r2 (with the neighbour cell's
// image shift), ties to the smaller gid; zero where there is none.  Walls
// are at their start-of-step positions: entry NF + w of pos4 and vt4, wall
// runs wcstart over the global cells (box offset co).  The minimum of
// (r2, gid) does not depend on the visiting order, so 16 lanes take a
// reflection, nine of them a row of its neighbourhood each (the three cells of a
// row are one run, two where it wraps in x), four independent loads at a time, and
// four reflections are searched together.  With the reflecting lane going through
// its nine rows alone, and its wavefront waiting, the launch took 42 us at 746,000
// particles between walls, against 27.
__device__ __forceinline__ float4 wall_velocity(const KGeom &G, int co, int64_t NF, bool here,
                                                float x, float y, float z,
                                                const int32_t *__restrict__ wcstart,
                                                const float4 *__restrict__ pos4,
                                                const float4 *__restrict__ vt4) {
  const float4 *walls = pos4 + NF;
  const int lane = (int)__lane_id(), row = lane & 15;
  const int nx = G.nc[0], ny = G.nc[1], nz = G.nc[2];
  int mine = -1;   // the nearest wall of this lane's own reflection
  unsigned long long left = __ballot(here);
  while (left) {
    // the lowest four lanes still to serve, one for each 16 lanes
    unsigned long long rest = left;
    int src = -1;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (lane >> 4 == g && rest) src = __ffsll((long long)rest) - 1;
      rest &= rest - 1ull;   // 0 stays 0
    }
    const int from = max(src, 0);
    const float px = __shfl(x, from, 64), py = __shfl(y, from, 64), pz = __shfl(z, from, 64);
    float best = INFINITY;
    uint32_t best_gid = 0;
    int best_w = -1;
    if (src >= 0 && row < 9) {
      int cx, cy, cz;
      cell_index(G, px, py, pz, cx, cy, cz);
      int qy = cy + row % 3 - 1, qz = cz + row / 3 - 1;
      float sy = 0.f, sz = 0.f;
      if (qy < 0) { qy += ny; sy = -G.L[1]; }
      else if (qy >= ny) { qy -= ny; sy = G.L[1]; }
      if (qz < 0) { qz += nz; sz = -G.L[2]; }
      else if (qz >= nz) { qz -= nz; sz = G.L[2]; }
      const float ay = sub_nc(py, sy), az = sub_nc(pz, sz);
      auto search = [&](int t, int te, float ax) {
        for (int w = t; w < te; w += 4) {
          float4 q[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) q[u] = walls[min(w + u, te - 1)];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float r2 = pair_r2(sub_nc(ax, q[u].x), sub_nc(ay, q[u].y), sub_nc(az, q[u].z));
            const uint32_t g = __float_as_uint(q[u].w);
            if (w + u < te && (r2 < best || (r2 == best && g < best_gid))) {
              best = r2;
              best_gid = g;
              best_w = w + u;
            }
          }
        }
      };
      // run A, and run B where the row wraps: the last cell seen across the left
      // edge and cells 0 and 1, or the last two and cell 0 seen across the right
      const int32_t *at = wcstart + co + (qz * ny + qy) * nx;
      const bool left_edge = cx == 0, right_edge = cx == nx - 1;
      const int first = left_edge ? nx - 1 : (right_edge ? nx - 2 : cx - 1);
      const int t = at[first], te = at[left_edge || right_edge ? nx : cx + 2];
      int tb = 0, tbe = 0;
      if (left_edge || right_edge) {
        tb = at[0];
        tbe = at[left_edge ? 2 : 1];
      }
      search(t, te, sub_nc(px, left_edge ? -G.L[0] : 0.f));
      search(tb, tbe, sub_nc(px, right_edge ? G.L[0] : 0.f));
    }
    for (int m = 8; m > 0; m >>= 1) {
      const float r2 = __shfl_xor(best, m, 64);
      const uint32_t g = (uint32_t)__shfl_xor((int)best_gid, m, 64);
      const int w = __shfl_xor(best_w, m, 64);
      if (w >= 0 && (best_w < 0 || r2 < best || (r2 == best && g < best_gid))) {
        best = r2;
        best_gid = g;
        best_w = w;
      }
    }
    const int turn = (int)__popcll(left & ((1ull << lane) - 1ull));
    const int found = __shfl(best_w, 16 * (turn & 3), 64);
    if (((left >> lane) & 1ull) && turn < 4) mine = found;
    left = rest;
  }
  if (mine < 0) return make_float4(0.f, 0.f, 0.f, 0.f);
  return vt4[NF + mine];
}

// REFLECT: compiled with the moving-wall and specular forms (the other
// instances keep the register budget of plain bounce-back off resting walls); they are
// called by every lane, act telling which have a particle.
template <typename T, bool REFLECT>
__device__ __forceinline__ Moved integrate_one(const KGeom &G, const KParams &P, bool act,
                                               float4 x, float4 v, float4 f,
                                               const uint32_t *__restrict__ bits, int use_mask,
                                               const typename PhiQuad<T>::type *__restrict__ quad,
                                               Status *st, int co,
                                               int64_t NF, const int32_t *__restrict__ wcstart,
                                               const float4 *__restrict__ pos4,
                                               const float4 *__restrict__ vt4) {
  float xs = drift1(x.x, v.x, f.x, P.hdt, P.dt, G.L[0]);
  float ys = drift1(x.y, v.y, f.y, P.hdt, P.dt, G.L[1]);
  float zs = drift1(x.z, v.z, f.z, P.hdt, P.dt, G.L[2]);
  float4 vt = make_float4(v.x + P.lamdt * f.x, v.y + P.lamdt * f.y, v.z + P.lamdt * f.z, 0.f);
  {
    const float dx = P.dt * (v.x + P.hdt * f.x), dy = P.dt * (v.y + P.hdt * f.y),
                dz = P.dt * (v.z + P.hdt * f.z);
    const float d2 = dx * dx + dy * dy + dz * dz;
    if (!(d2 <= P.max_disp2)) {
      if (act) atomicAdd(d2 != d2 || isinf(d2) ? &st->nonfinite : &st->unstable, 1ull);
      // keep indices in range for the rest of the step
      if (!(xs >= 0.f && xs <= G.L[0])) xs = x.x;
      if (!(ys >= 0.f && ys <= G.L[1])) ys = x.y;
      if (!(zs >= 0.f && zs <= G.L[2])) zs = x.z;
    }
  }
  int event = 0;
  const GridLoc<T> loc = grid_locate<T>(G, xs, ys, zs);
  T phis = (T)0;
  if (!use_mask || cube_flagged(bits, cube_index(G, loc)))
    phis = phi_interp_quad<T>(quad, G, loc);
  float4 vw = make_float4(0.f, 0.f, 0.f, 0.f);
  if (REFLECT && (P.reflect & kReflectMoving))
    vw = wall_velocity(G, co, NF, act && phis < (T)0, xs, ys, zs, wcstart, pos4, vt4);
  if (phis < (T)0) {
    // Eq. 16-17: distances beyond and before the interface from atanh(phi)
    const T phit = phi_at_quad<T>(quad, G, x.x, x.y, x.z);
    const T lim = (T)1 - (T)0x1p-20;
    const T a1 = fmin(fmax(-phis, (T)0), lim);
    const T a0 = fmin(fmax(phit, (T)0), lim);
    const T c1 = atanh(a1), c0 = atanh(a0);
    const T sfrac = c1 > (T)0 ? c1 / (c0 + c1) : (T)0;
    const float k2 = (float)((T)2 * sfrac * (T)P.dt);
    // the reversed part u of the velocity relative to the wall: all of it
    // (bounce-back) or its component along the normal (specular)
    float ux = v.x - vw.x, uy = v.y - vw.y, uz = v.z - vw.z;
    if (REFLECT && (P.reflect & kReflectSpecular)) {
      T gx, gy, gz;
      phi_grad_quad<T>(quad, G, loc, gx, gy, gz);
      const T gn = sqrt(gx * gx + gy * gy + gz * gz);
      if (gn > (T)0) {
        const T nx = gx / gn, ny = gy / gn, nz = gz / gn;
        const T un = (T)ux * nx + (T)uy * ny + (T)uz * nz;
        ux = (float)(un * nx);
        uy = (float)(un * ny);
        uz = (float)(un * nz);
      }
    }
    float bx = wrap1(xs - k2 * ux, G.L[0]);
    float by = wrap1(ys - k2 * uy, G.L[1]);
    float bz = wrap1(zs - k2 * uz, G.L[2]);
    if (phi_at_quad<T>(quad, G, bx, by, bz) < (T)0) {
      bx = x.x;
      by = x.y;
      bz = x.z;
      event = 2;
    } else {
      event = 1;
    }
    xs = bx;
    ys = by;
    zs = bz;
    vt = make_float4(v.x - 2.f * ux, v.y - 2.f * uy, v.z - 2.f * uz, 0.f);
  }
  vt.w = __int_as_float(event);
  Moved m;
  m.pos = make_float4(xs, ys, zs, x.w);
  m.vt = vt;
  int cx, cy, cz;
  m.cell = cell_index(G, xs, ys, zs, cx, cy, cz);
  return m;
}

// Tile tid of up to PPT x kBlock particles of one box, by one block of
// kBlock threads; each thread advances PPT particles (pos_out may be pos4: a
// thread reads its own particles before it writes them).
template <typename T, int PPT, bool REFLECT>
__device__ __forceinline__ void integrate_tile(
    int tid, const Box *__restrict__ boxes, const Tile *__restrict__ tiles,
    const float4 *pos4, float4 *pos_out, const float4 *__restrict__ vel4,
    const float4 *__restrict__ frc4, float4 *__restrict__ vt4,
    int32_t *__restrict__ cell_of, int32_t *__restrict__ rank_of,
    int32_t *__restrict__ count, const uint32_t *__restrict__ bits_base, int use_mask,
    const typename PhiQuad<T>::type *__restrict__ quad_base, Status *st, int64_t NF,
    const int32_t *__restrict__ wcstart) {
  const Tile tile = tiles[tid];
  const Box &B = boxes[tile.box];
  const KGeom G = B.G;
  const KParams P = B.P;
  const typename PhiQuad<T>::type *quad = quad_base + B.go;
  const uint32_t *bits = bits_base + B.bo;
  const int co = (int)B.co;
  int64_t p[PPT];
  bool a[PPT];
  float4 x[PPT], v[PPT], f[PPT];
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    const int local = u * kBlock + (int)threadIdx.x;
    a[u] = local < tile.count;
    p[u] = (int64_t)tile.first + local;
    x[u] = v[u] = f[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a[u]) {
      x[u] = load_stream(&pos4[p[u]]);
      v[u] = load_stream(&vel4[p[u]]);
      f[u] = load_stream(&frc4[p[u]]);
    }
  }
  Moved m[PPT];
  RunInfo r[PPT];
  int b[PPT];
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    m[u].cell = -1;
    if (REFLECT || a[u]) {
      m[u] = integrate_one<T, REFLECT>(G, P, a[u], x[u], v[u], f[u], bits, use_mask, quad, st, co,
                                       NF, wcstart, pos4, vt4);
      m[u].cell = a[u] ? m[u].cell + co : -1;
    }
    r[u] = wave_runs(m[u].cell);
    b[u] = 0;
  }
#pragma unroll
  for (int u = 0; u < PPT; ++u)
    if (r[u].head && m[u].cell >= 0) b[u] = atomicAdd(&count[m[u].cell], r[u].len);
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    const int k = wave_rank(r[u], b[u]);
    if (a[u]) {
      store_stream(&pos_out[p[u]], m[u].pos);
      store_stream(&vt4[p[u]], m[u].vt);
      store_stream(&cell_of[p[u]], m[u].cell);
      store_stream(&rank_of[p[u]], k);
    }
  }
  // event counts: one atomic per wavefront, after the stores (a per-lane
  // atomic put its latency into the step's chain), on the tile's line of 64
  int nbounce = 0, nfall = 0;
#pragma unroll
  for (int u = 0; u < PPT; ++u) {
    const int ev = a[u] ? __float_as_int(m[u].vt.w) : 0;
    nbounce += __popcll(__ballot(ev == 1));
    nfall += __popcll(__ballot(ev == 2));
  }
  if (__lane_id() == 0) {
    StatusBlock::Line &at = ((StatusBlock *)st)->lines[tid & 63];
    if (nbounce) atomicAdd(&at.bounce, (unsigned long long)nbounce);
    if (nfall) atomicAdd(&at.fallback, (unsigned long long)nfall);
  }
}

template <typename T, int PPT, bool REFLECT>
__global__ __launch_bounds__(kBlock) void k_integrate(
    const Box *__restrict__ boxes, const Tile *__restrict__ tiles, int ntiles,
    const float4 *pos4, float4 *pos_out, const float4 *__restrict__ vel4,
    const float4 *__restrict__ frc4, float4 *__restrict__ vt4, int32_t *__restrict__ cell_of,
    int32_t *__restrict__ rank_of,
    int32_t *__restrict__ count, const uint32_t *__restrict__ bits_base, int use_mask,
    const typename PhiQuad<T>::type *__restrict__ quad_base, Status *st, int64_t NF,
    const int32_t *__restrict__ wcstart) {
  const int tid = xcd_block();
  if (tid >= ntiles) return;
  integrate_tile<T, PPT, REFLECT>(tid, boxes, tiles, pos4, pos_out, vel4, frc4, vt4, cell_of, rank_of, count,
                                  bits_base, use_mask, quad_base, st, NF, wcstart);
}

// Walls of one box re-binned: each is advanced by dt v with move (its solid
// translates: x += dt v per axis in the decision form of the fluid drift
// with zero force, then the single-edge wrap) or kept, written to walls_out
// with its velocity to vt_out, and binned (cell and rank in cell, as k_bin).
__global__ void k_wall_move_bin(const KGeom G, float hdt, float dt, int move, int64_t cell_off,
                                int64_t nw, const float4 *__restrict__ walls_in,
                                const float4 *__restrict__ vt_in, float4 *__restrict__ walls_out,
                                float4 *__restrict__ vt_out, int32_t *__restrict__ cell_of,
                                int32_t *__restrict__ rank_of, int32_t *__restrict__ count) {
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int c = -1;
  if (w < nw) {
    float4 x = walls_in[w];
    const float4 v = vt_in[w];
    if (move)
      x = make_float4(drift1(x.x, v.x, 0.f, hdt, dt, G.L[0]), drift1(x.y, v.y, 0.f, hdt, dt, G.L[1]),
                      drift1(x.z, v.z, 0.f, hdt, dt, G.L[2]), x.w);
    walls_out[w] = x;
    vt_out[w] = v;
    int cx, cy, cz;
    c = (int)cell_off + cell_index(G, x.x, x.y, x.z, cx, cy, cz);
    cell_of[w] = c;
  }
  const int k = rank_in_cell(c, count);
  if (w < nw) rank_of[w] = k;
}

// Wall positions from gid-ordered rows (gid in pos4[w].w).
__global__ void k_import_walls(int64_t nw, float4 *__restrict__ walls, const float *__restrict__ pos) {
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= nw) return;
  const float4 x = walls[w];
  const size_t g = (size_t)__float_as_uint(x.w);
  walls[w] = make_float4(pos[3 * g], pos[3 * g + 1], pos[3 * g + 2], x.w);
}

// Number of fluid particles whose grid cube is flagged (the particles that
// interpolate phi in a step), one atomic per block.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_count_flagged(const KGeom G, int64_t nf,
                                                          const float4 *__restrict__ pos4,
                                                          const uint32_t *__restrict__ bits,
                                                          unsigned long long *out) {
  __shared__ int lds[kBlock];
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int v = 0;
  if (p < nf) {
    const float4 x = pos4[p];
    v = cube_flagged(bits, cube_index(G, grid_locate<T>(G, x.x, x.y, x.z))) ? 1 : 0;
  }
  lds[threadIdx.x] = v;
  __syncthreads();
  for (int off = kBlock / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) lds[threadIdx.x] += lds[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0 && lds[0]) atomicAdd(out, (unsigned long long)lds[0]);
}

// ---------------------------------------------------------------------------
// Pair force (Eq. 3-10), body force, velocity update
//
// One thread per fluid particle i, in cell-sorted slot order; a wavefront is
// 64 consecutive particles.  Phase A: the wavefront visits the 9 rows of the
// 27-cell neighbourhood together (the x-neighbours of a row are consecutive
// cells, so a row is one run of merged entries, walls then fluid, or two
// where it wraps in x) and walks each row in lockstep, four run entries per
// lane and pass so that their loads overlap, testing the entries' coarse
// position codes against a bound that keeps every pair of the FP32 cutoff
// decision; kept candidates go to the lane's column of an LDS list
// (slot-major, so the wavefront's appends fall in different banks).  Phase
// B: each lane takes the exact FP32 decision on its listed candidates; the
// random-number and force arithmetic runs only for pairs inside the
// cutoff.  The wavefront runs phase B on the first kDrain listed of every lane
// when any lane's list could overflow in the next pass, and on all at the end.  Lanes
// never branch apart inside a pass, so the wavefront pays for the longest
// run of each row, not for every lane's row switches.  Sums run in
// candidate order, so runs are deterministic.
// ---------------------------------------------------------------------------
// 26 entries per lane: with 256-thread blocks at six wavefronts per SIMD,
// six blocks' lists (26 KB each) fill a CU's 160 KB of LDS, and most lanes'
// pairs (about 16 plus the pre-test's extras) fit.
constexpr int kListCap = 26;
constexpr int kBatch = 4;   // = the width of one run-array load
// Pairs a lane evaluates when a list could overflow: fewer than nearly every lane
// has listed by then, so that few lanes idle; the rest stays listed.  Emptying the
// lists costs the longest list's pairs twice: by a count over random boxes 42
// evaluations a wavefront for the 20 candidates a lane lists at 4 particles per
// unit volume (27 for 15 at 3), against 30 (23) with 10, 31 (23) with 12 and 34
// (24) with 16.  Measured: 16 cylinder cells 43.1 to 40.3 us, SPH in 1.17 million
// particles 182 to 175; the 168^3 porous box (6.3 million), which the line accesses
// of the gathers bound, 845 before and after; 8 and 13 as 10.
constexpr int kDrain = 10;

struct Acc {
  float x, y, z;
};

// One pair's force on i: mag along the unit vector (ex, ey, ez).
struct PairTerm {
  float mag, ex, ey, ez;
};

// SPH: compiled with the conservative force of Eq. 22-24 for boxes that use
// it (wall: j is a wall particle, selecting the fluid-wall strengths).  Each
// operation is written out (fused where it says so), so that every kernel that
// evaluates a pair gets the same bits.
template <bool SPH>
__device__ __forceinline__ PairTerm pair_term(float dx, float dy, float dz, float r2, float dvx,
                                              float dvy, float dvz, bool wall, const KParams &P,
                                              uint32_t gi, uint32_t gj, uint32_t klo,
                                              uint32_t khi) {
#pragma clang fp contract(off)
  const float rinv = rsqrtf(r2);
  const float r = r2 * rinv;
  const float w = fmaxf(__builtin_fmaf(-r, P.inv_rc, 1.0f), 0.0f);
  PairTerm t;
  t.ex = dx * rinv;
  t.ey = dy * rinv;
  t.ez = dz * rinv;
  const float edv = __builtin_fmaf(t.ez, dvz, __builtin_fmaf(t.ex, dvx, t.ey * dvy));
  const float xi = pair_gauss(gi, gj, klo, khi, P.key0, P.key1);
  const float gw = P.gamma * w;
  if (SPH && P.sph) {
    const float cr = wall ? P.cr_fw : P.cr_ff, ca = wall ? P.ca_fw : P.ca_ff;
    const float fc = __builtin_fmaf(ca, spline_dp(r * P.inv_ha), -(cr * spline_dp(r * P.inv_hr)));
    t.mag = __builtin_fmaf(w, __builtin_fmaf(P.sigma_rdt, xi, -(gw * edv)), fc);
  } else {
    const float a = wall ? P.a_fw : P.a_ff;
    t.mag = w * __builtin_fmaf(P.sigma_rdt, xi, __builtin_fmaf(-edv, gw, a));
  }
  return t;
}

// Velocity and carried force of particle i after its pair sum (acc) is
// complete, written with its position to slot s of the next buffers.
struct Finished {
  float4 vel, frc;
};

template <bool INIT>
__device__ __forceinline__ Finished finish_particle(const KParams &P, const Acc &acc, int i,
                                                          const float4 &vti,
                                                          const float4 *__restrict__ vel4,
                                                          const float4 *__restrict__ frc4) {
#pragma clang fp contract(off)
  Finished r;
  const float fx = acc.x + P.g[0], fy = acc.y + P.g[1], fz = acc.z + P.g[2];
  r.frc = make_float4(fx, fy, fz, 0.f);
  const float4 vo = load_stream(&vel4[i]);
  if (INIT) {
    r.vel = make_float4(vo.x, vo.y, vo.z, __int_as_float(0));
    return r;
  }
  const int event = __float_as_int(vti.w);
  if (event) {
    r.vel = make_float4(vti.x, vti.y, vti.z, __int_as_float(event));
  } else {
    const float4 fo = load_stream(&frc4[i]);
    r.vel = make_float4(__builtin_fmaf(P.hdt, fo.x + fx, vo.x),
                        __builtin_fmaf(P.hdt, fo.y + fy, vo.y),
                        __builtin_fmaf(P.hdt, fo.z + fz, vo.z), __int_as_float(0));
  }
  return r;
}

// Tile tid by one block of BS threads; list: kListCap x BS words of LDS.
// The walk tests candidates on their coarse codes (cq, one word per
// merged-run entry, in run order) and lists every candidate the bound
// keeps; the pair pass then takes the exact FP32 decision, so the pairs
// summed and their order are those of an exact walk over the same runs.
// T (the grid's type, or void): the particles go on to the drift and the binning of the
// next step (integrate_one, as k_integrate) into next.  That spares a launch and 64 of
// the 136 B a particle that drift and binning move apart; the registers are free by then
// (77 VGPRs).  A step of steps in a row, us: 16 cylinder cells 58.1 to 50.2, 64 uneven
// boxes 106 to 93.4, 330,000 particles in a cylinder 76.1 to 71.4, porous SPH with
// 1.17 million 227 to 214, the 168^3 porous box (6.3 million) 1,129 to 1,097.
// REFLECT: integrate_one's moving walls and specular reflection.  SPLIT: the pair pass
// is compiled apart for interior wavefronts and for the end of the walk (1 % of a step); as a
// callee, whose registers are fewer, the function spills then (a persistent step of 200
// boxes with 1.56 million particles: 1,139 us against 1,054).
template <bool INIT, int BS, bool SPH, typename T, bool REFLECT, bool SPLIT = true>
__device__ __forceinline__ void force_tile(
    int tid, uint32_t *list, const Box *__restrict__ boxes, const Tile *__restrict__ tiles,
    int64_t NF, int32_t pad, int32_t ncell_all, const float4 *__restrict__ pos4,
    const float4 *__restrict__ vt4, const float4 *__restrict__ vel4,
    const float4 *__restrict__ frc4, const int32_t *__restrict__ idx,
    const int32_t *__restrict__ idx_all, const int32_t *__restrict__ start_all,
    const uint32_t *__restrict__ cq,
    float4 *__restrict__ pos_out, float4 *__restrict__ vel_out, float4 *__restrict__ frc_out,
    const unsigned long long *__restrict__ dk, Status *st,
    const NextStep &next) {
  const Tile tile = tiles[tid];
  if (((int)threadIdx.x & ~63) >= tile.count) return;
  const bool act = (int)threadIdx.x < tile.count;   // the others follow the last particle
  const Box &B = boxes[tile.box];
  const KGeom G = B.G;
  const KParams P = B.P;
  const int co = (int)B.co;
  // force evaluation index k, kept on the device so that a captured step
  // draws new random numbers on every replay
  const unsigned long long kk = *dk;
  const uint32_t klo = (uint32_t)kk;
  const uint32_t khi = ((uint32_t)(kk >> 32) & 0xFFFFu) | (P.replica << 16);
  const int64_t s = (int64_t)tile.first + min((int)threadIdx.x, tile.count - 1);
  const int i = idx[s];
  const float4 pi = pos4[i];
  const float4 vti = vt4[i];
  const uint32_t gi = __float_as_uint(pi.w);
  int cx, cy, cz;
  cell_index(G, pi.x, pi.y, pi.z, cx, cy, cz);
  // pos4 and vt4 hold NF + NW + 1 records (the pad last); the run array and
  // the codes hold NF + NW entries and kIdxSlack spare ones (the run's read
  // as the pad); the run starts hold ncell_all + 1 entries and kStartSlack
  // spare ones
  const Records16 posr(pos4, pad + 1), vtr(vt4, pad + 1);
  const Ints4 runs(idx_all, pad + kIdxSlack);
  const Ints4 codes((const int32_t *)cq, pad + kIdxSlack);
  const Ints4 starts(start_all, ncell_all + 1 + kStartSlack);
  // (as a scalar, so that its two cases are not tested per candidate)
  const uint32_t qth = __builtin_amdgcn_readfirstlane(qthresh(P.rc2));
  // this lane's list column as LDS byte offsets: entry q at lane0 + q * BS * 4
  char *const lds = (char *)list;
  const uint32_t lane0 = threadIdx.x * 4u;
  const uint32_t full = lane0 + (uint32_t)((kListCap - kBatch) * BS * 4);
  uint32_t tail = lane0;   // next free entry
  const int nf32 = (int)NF;
  // wave-uniform: some lane sees neighbour cells across an edge of the box (or
  // the axis is so short that half of it is within two cells)
  const bool edge = wave_any(cx == 0 || cy == 0 || cz == 0 || cx == G.nc[0] - 1 ||
                             cy == G.nc[1] - 1 || cz == G.nc[2] - 1 || G.nc[0] < 5 ||
                             G.nc[1] < 5 || G.nc[2] < 5);
  Acc acc = {0.f, 0.f, 0.f};
  // phase B: the listed candidates of this lane, in list (= candidate)
  // order, with the exact decision; the next candidate's data is fetched
  // while the current one is evaluated.  Where no lane's cell is at an edge of
  // the box the separation needs no image (sep's value in that case): 21 of
  // about 150 instructions a pair.
  auto pairs_of_list = [&](auto at_edge, uint32_t upto) {
    if (tail == lane0) return;
    const uint32_t last = min(tail, upto) - BS * 4u;
    uint32_t q = lane0;
    auto evaluate = [&](int j, const float4 &pj, const float4 &vtj) {
      const float dx = at_edge.value ? sep(pi.x, pj.x, G.L[0]) : sub_nc(pi.x, pj.x);
      const float dy = at_edge.value ? sep(pi.y, pj.y, G.L[1]) : sub_nc(pi.y, pj.y);
      const float dz = at_edge.value ? sep(pi.z, pj.z, G.L[2]) : sub_nc(pi.z, pj.z);
      // the pair decision (r2 > 0 also drops coincident particles, whose
      // force is 0)
      const float r2 = pair_r2(dx, dy, dz);
      if (r2 < P.rc2 && r2 > 0.0f) {
        const PairTerm t = pair_term<SPH>(dx, dy, dz, r2, vti.x - vtj.x, vti.y - vtj.y,
                                          vti.z - vtj.z, j >= nf32, P, gi,
                                          __float_as_uint(pj.w), klo, khi);
        acc.x = __builtin_fmaf(t.ex, t.mag, acc.x);
        acc.y = __builtin_fmaf(t.ey, t.mag, acc.y);
        acc.z = __builtin_fmaf(t.ez, t.mag, acc.z);
      }
    };
    // two sets of registers in turn, so that the fetched pair need not be
    // copied (8 of 122 vector instructions a pair)
    int j = *(const int *)(lds + lane0);
    float4 pj = posr[j], vtj = vtr[j];
    for (;;) {
      const int j2 = *(const int *)(lds + min(q + BS * 4u, last));
      const float4 pj2 = posr[j2], vtj2 = vtr[j2];
      evaluate(j, pj, vtj);
      q += BS * 4u;
      if (q > last) break;
      j = *(const int *)(lds + min(q + BS * 4u, last));
      pj = posr[j];
      vtj = vtr[j];
      evaluate(j2, pj2, vtj2);
      q += BS * 4u;
      if (q > last) break;
    }
  };
  // the first `count` entries of every lane's list
  auto drain = [&](int count) {
    const uint32_t upto = lane0 + (uint32_t)(count * BS * 4);
    if (!SPLIT || edge)
      pairs_of_list(std::true_type{}, upto);
    else
      pairs_of_list(std::false_type{}, upto);
  };
  // Phase A: the wavefront goes through the nine neighbour rows together and
  // walks the lane's runs of each in lockstep, kBatch run entries per lane and
  // pass (run A [t, t_end), then run B [tb, tb_end) where the row wraps; a lane
  // moves to B on its own), with qa / qb the lane's code shifted by the image of
  // run A / B.  Entries past the lane's run are read (other cells' entries, or the
  // pad) but never listed; neither is the lane's own particle.  Phase B runs when
  // a lane's list could overflow in the next pass, and after the last row; rows
  // and passes are one loop.
  const int nx = G.nc[0], ny = G.nc[1], nz = G.nc[2];
  int t = 0, t_end = 0, tb = 0, tb_end = 0;
  uint32_t qa = 0, qb = 0;
  int row = -1;   // of the nine, z outermost
  for (;;) {
    if (!wave_any(t < t_end)) {
      if (++row == 9) {
        if constexpr (SPLIT) {
          drain(kListCap);
          break;
        }
      } else {
        const int oz = row / 3 - 1, oy = row % 3 - 1;
        int qz = cz + oz, qy = cy + oy;
        float sz = 0.f, sy = 0.f;
        if (qz < 0) { qz += nz; sz = -G.L[2]; }
        else if (qz >= nz) { qz -= nz; sz = G.L[2]; }
        if (qy < 0) { qy += ny; sy = -G.L[1]; }
        else if (qy >= ny) { qy -= ny; sy = G.L[1]; }
        const uint32_t cyz_code = (qshift(pi.y, sy) << 11) | (qshift(pi.z, sz) << 22);
        // the row's x-neighbours [cx-1, cx+1] as run A, plus run B where the
        // row wraps (cell nx-1 seen across the left edge, then cells 0 and 1;
        // or cells nx-2 and nx-1, then cell 0 seen across the right edge)
        const int base = co + (qz * ny + qy) * nx;
        const bool left = cx == 0, right = cx == nx - 1;
        const int a0 = left ? base + nx - 1 : (right ? base + nx - 2 : base + cx - 1);
        int v[4];
        starts.load(a0, v);
        t = v[0];
        t_end = left ? v[1] : (right ? v[2] : v[3]);
        tb = 0;
        tb_end = 0;
        if (wave_any(left || right)) {
          int w[4];
          starts.load(base, w);
          tb = (left || right) ? w[0] : 0;
          tb_end = left ? w[2] : (right ? w[1] : 0);
        }
        qa = qshift(pi.x, left ? -G.L[0] : 0.f) | cyz_code;
        qb = qshift(pi.x, right ? G.L[0] : 0.f) | cyz_code;
        const bool sw = t >= t_end;
        t = sw ? tb : t;
        t_end = sw ? tb_end : t_end;
        tb = sw ? tb_end : tb;
        qa = sw ? qb : qa;
        continue;
      }
    }
    if ((!SPLIT && row == 9) || wave_any(tail > full)) {
      drain(!SPLIT && row == 9 ? kListCap : kDrain);
      if (!SPLIT && row == 9) break;
      // the entries that are left, to the list's front
      int *const column = (int *)(lds + lane0);
#pragma unroll
      for (int e = 0; e + kDrain < kListCap; ++e) column[e * BS] = column[(e + kDrain) * BS];
      tail = max(tail, lane0 + (uint32_t)(kDrain * BS * 4)) - (uint32_t)(kDrain * BS * 4);
    }
    const int rem = t_end - t;
    int jb[kBatch], w[kBatch];
    runs.load(t, jb);
    codes.load(t, w);
    // the conditions are joined as masks, by the scalar unit; the particle
    // itself is met in the home row alone
    unsigned long long self[kBatch] = {};
    if (row == 4) {
#pragma unroll
      for (int u = 0; u < kBatch; ++u) self[u] = __ballot(jb[u] == i);
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const unsigned long long keep =
          __ballot(qdist2((uint32_t)w[u], qa) <= qth) & __ballot(u < rem) & ~self[u];
      *(int *)(lds + tail) = jb[u];
      tail += __builtin_amdgcn_inverse_ballot_w64(keep) ? (uint32_t)(BS * 4) : 0u;
    }
    t = rem > 0 ? t + kBatch : t;
    const bool sw = t >= t_end && tb < tb_end;
    t = sw ? tb : t;
    t_end = sw ? tb_end : t_end;
    tb = sw ? tb_end : tb;
    qa = sw ? qb : qa;
  }
  const Finished fin = finish_particle<INIT>(P, acc, i, vti, vel4, frc4);
  if (act) {
    if (!(isfinite(fin.frc.x) && isfinite(fin.frc.y) && isfinite(fin.frc.z)))
      atomicAdd(&st->nonfinite, 1ull);
    if (std::is_void_v<T> || next.pos != pos_out) store_stream(&pos_out[s], pi);
    store_stream(&vel_out[s], fin.vel);
    store_stream(&frc_out[s], fin.frc);
  }
  if constexpr (!std::is_void_v<T>) {
    const Moved m = integrate_one<T, REFLECT>(
        G, P, act, pi, fin.vel, fin.frc, next.bits + B.bo, next.use_mask,
        (const typename PhiQuad<T>::type *)next.quad + B.go, st, co, NF, next.wcstart, pos4, vt4);
    const int cell = act ? co + m.cell : -1;
    const int rank = rank_in_cell(cell, next.count);
    if (act) {
      store_stream(&next.pos[s], m.pos);
      store_stream(&next.vt[s], m.vt);
      store_stream(&next.cell_of[s], cell);
      store_stream(&next.rank_of[s], rank);
    }
    const int ev = act ? __float_as_int(m.vt.w) : 0;
    const int nbounce = (int)__popcll(__ballot(ev == 1)), nfall = (int)__popcll(__ballot(ev == 2));
    if (__lane_id() == 0) {
      StatusBlock::Line &at = ((StatusBlock *)st)->lines[tid & 63];
      if (nbounce) atomicAdd(&at.bounce, (unsigned long long)nbounce);
      if (nfall) atomicAdd(&at.fallback, (unsigned long long)nfall);
    }
  }
}

// The cell counts cleared for the next step's binning, by the blocks of a pair
// force that follows a cell list whose blocks could not (clear: null where they did).
__device__ __forceinline__ void clear_counts(int32_t *__restrict__ clear, int n) {
  if (!clear) return;
  for (int c = (int)(blockIdx.x * blockDim.x + threadIdx.x); c < n;
       c += (int)(gridDim.x * blockDim.x))
    clear[c] = 0;
}

// Six wavefronts per SIMD: at most 80 VGPRs, so the walk and the pair pass
// run without register spills, and six blocks' lists fit in LDS.
template <bool INIT, int BS, bool SPH, typename T, bool REFLECT>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(6))) void k_force(
    const Box *__restrict__ boxes, const Tile *__restrict__ tiles, int ntiles, int64_t NF,
    int32_t pad, int32_t ncell_all, const float4 *__restrict__ pos4,
    const float4 *__restrict__ vt4, const float4 *__restrict__ vel4,
    const float4 *__restrict__ frc4, const int32_t *__restrict__ idx,
    const int32_t *__restrict__ idx_all, const int32_t *__restrict__ start_all,
    const uint32_t *__restrict__ cq,
    float4 *__restrict__ pos_out, float4 *__restrict__ vel_out, float4 *__restrict__ frc_out,
    const unsigned long long *__restrict__ dk, Status *st, int32_t *__restrict__ clear,
    const NextStep next) {
  __shared__ uint32_t list[kListCap * BS];
  clear_counts(clear, ncell_all);
  const int tid = xcd_block();
  if (tid >= ntiles) return;
  force_tile<INIT, BS, SPH, T, REFLECT>(tid, list, boxes, tiles, NF, pad, ncell_all, pos4, vt4, vel4, frc4,
                            idx, idx_all, start_all, cq, pos_out, vel_out, frc_out, dk, st, next);
}

// ---------------------------------------------------------------------------
// Pair force of small contexts: 16 lanes per particle.
//
// With one lane per particle a context of a few thousand particles fills a
// few wavefronts, each walking nine neighbour rows in sequence: 27 us for 2,100
// particles and 26 us for 16,000, whatever the arithmetic.  Here the candidates of a particle's
// nine rows are numbered through (row by row, as the walk visits them) and
// taken 16 lanes x 8 at a time, so their indices are one level of loads and
// their positions another; the pairs found are listed in candidate order, the
// 16 lanes evaluate 16 of them at a time, and three lanes add the terms up
// in list order.  The terms and their order are those of force_tile, so the
// results are too, bit for bit, and a box gives the same in a context of any size.
//
// T (the grid's type, or void): the particle goes on to the drift and the binning of
// the next step (integrate_one, as k_integrate), so that steps that follow one another in a
// call are two launches instead of three: 19.6 to 16.2 us a step at 2,400 particles,
// 24.1 to 21.9 at 16,500.  Five wavefronts per SIMD (96 VGPRs, of which the drifting
// instances spill one to four, 8 to 20 B of scratch a lane): with four the blocks of
// 16,500 particles took a second round, 24.4 us.
// ---------------------------------------------------------------------------
template <bool INIT, bool SPH, typename T, bool REFLECT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(5))) void k_force_wide(
    const Box *__restrict__ boxes, const Tile *__restrict__ tiles, int ntiles, int64_t NF,
    const float4 *__restrict__ pos4, const float4 *__restrict__ vt4,
    const float4 *__restrict__ vel4, const float4 *__restrict__ frc4,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ idx_all,
    const int32_t *__restrict__ start_all, float4 *__restrict__ pos_out,
    float4 *__restrict__ vel_out, float4 *__restrict__ frc_out,
    const unsigned long long *__restrict__ dk, Status *st, int32_t *__restrict__ clear,
    int ncell_all, const NextStep next) {
  clear_counts(clear, ncell_all);
  // padded so that the four groups of a wavefront use different banks
  __shared__ int ring[kWideParts][kWideRing + 8];
  __shared__ float4 term[kWideParts][kWideLanes + 1];
  __shared__ int4 rows_lds[kWideParts][9];
  const int tid = xcd_block();
  if (tid >= ntiles) return;
  const Tile tile = tiles[tid];
  const int grp = (int)threadIdx.x / kWideLanes, g = (int)threadIdx.x % kWideLanes;
  if (grp >= tile.count) return;   // whole groups
  const Box &B = boxes[tile.box];
  const KGeom G = B.G;
  const KParams P = B.P;
  const unsigned long long kk = *dk;
  const uint32_t klo = (uint32_t)kk;
  const uint32_t khi = ((uint32_t)(kk >> 32) & 0xFFFFu) | (P.replica << 16);
  const int64_t s = (int64_t)tile.first + grp;
  const int i = idx[s];
  const float4 pi = pos4[i];
  const float4 vti = vt4[i];
  const uint32_t gi = __float_as_uint(pi.w);
  int cx, cy, cz;
  cell_index(G, pi.x, pi.y, pi.z, cx, cy, cz);
  WideRows rows;
  rows.init(G, (int)B.co, cx, cy, cz, g, start_all, rows_lds[grp]);
  int *const list = ring[grp];
  float4 *const terms = term[grp];
  const int shift = ((int)__lane_id() / kWideLanes) * kWideLanes;   // the group's bits of a ballot
  int listed = 0, done = 0;
  float acc = 0.f;   // lanes 0, 1, 2: the sum of component x, y, z
  // the next 16 listed pairs (the last call: fewer), one per lane, then their
  // terms added up in list order
  auto evaluate = [&]() {
    const int e = done + g;
    PairTerm t = {0.f, 0.f, 0.f, 0.f};
    if (e < listed) {
      const int j = list[e & (kWideRing - 1)];
      const float4 pj = pos4[j], vtj = vt4[j];
      const float dx = sep(pi.x, pj.x, G.L[0]), dy = sep(pi.y, pj.y, G.L[1]),
                  dz = sep(pi.z, pj.z, G.L[2]);
      t = pair_term<SPH>(dx, dy, dz, pair_r2(dx, dy, dz), vti.x - vtj.x, vti.y - vtj.y,
                         vti.z - vtj.z, (int64_t)j >= NF, P, gi, __float_as_uint(pj.w), klo, khi);
    }
    terms[g] = make_float4(t.mag, t.ex, t.ey, t.ez);
    wave_lds_sync();
    if (g < 3) {
      const float *m = (const float *)terms;
#pragma unroll
      for (int q = 0; q < kWideLanes; ++q) acc = __builtin_fmaf(m[4 * q + 1 + g], m[4 * q], acc);
    }
    wave_lds_sync();
    done += kWideLanes;
  };
  for (int c0 = 0; c0 < rows.total; c0 += kWideBatch * kWideLanes) {
    int j[kWideBatch];
    float4 pj[kWideBatch];
#pragma unroll
    for (int k = 0; k < kWideBatch; ++k)
      j[k] = idx_all[rows.entry(min(c0 + k * kWideLanes + g, rows.total - 1))];
#pragma unroll
    for (int k = 0; k < kWideBatch; ++k) pj[k] = pos4[j[k]];
#pragma unroll
    for (int k = 0; k < kWideBatch; ++k) {
      const float r2 = pair_r2(sep(pi.x, pj[k].x, G.L[0]), sep(pi.y, pj[k].y, G.L[1]),
                               sep(pi.z, pj[k].z, G.L[2]));
      // the pair decision (r2 > 0 drops the particle itself and coincident
      // ones, whose force is 0)
      const bool hit = r2 < P.rc2 && r2 > 0.0f && c0 + k * kWideLanes + g < rows.total;
      const uint32_t m = (uint32_t)(__ballot(hit) >> shift) & 0xFFFFu;
      if (hit) list[(listed + __popc(m & ((1u << g) - 1u))) & (kWideRing - 1)] = j[k];
      listed += __popc(m);
    }
    wave_lds_sync();
    while (listed - done >= kWideLanes) evaluate();
  }
  if (done < listed) evaluate();
  const Acc sum = {__shfl(acc, 0, kWideLanes), __shfl(acc, 1, kWideLanes),
                   __shfl(acc, 2, kWideLanes)};
  const Finished fin = finish_particle<INIT>(P, sum, i, vti, vel4, frc4);
  if (g == 0) {
    if (!(isfinite(fin.frc.x) && isfinite(fin.frc.y) && isfinite(fin.frc.z)))
      atomicAdd(&st->nonfinite, 1ull);
    vel_out[s] = fin.vel;
    frc_out[s] = fin.frc;
    if (std::is_void_v<T> || next.pos != pos_out) pos_out[s] = pi;
  }
  if constexpr (!std::is_void_v<T>) {
    // one lane's work; with REFLECT by all lanes, which search a reflection's wall
    // together (groups leave from the last on, and there are no more reflections than
    // groups)
    if (REFLECT || g == 0) {
      const int co = (int)B.co;
      const Moved m = integrate_one<T, REFLECT>(
          G, P, g == 0, pi, fin.vel, fin.frc, next.bits + B.bo, next.use_mask,
          (const typename PhiQuad<T>::type *)next.quad + B.go, st, co, NF, next.wcstart, pos4,
          vt4);
      if (g == 0) {
        const int cell = co + m.cell;
        const int rank = atomicAdd(&next.count[cell], 1);
        next.pos[s] = m.pos;
        next.vt[s] = m.vt;
        next.cell_of[s] = cell;
        next.rank_of[s] = rank;
        const int ev = __float_as_int(m.vt.w);
        StatusBlock::Line &at = ((StatusBlock *)st)->lines[tid & 63];
        if (ev == 1) atomicAdd(&at.bounce, 1ull);
        if (ev == 2) atomicAdd(&at.fallback, 1ull);
      }
    }
  }
}

// Interacting pairs with the same decision as the force kernel.  Each thread
// counts its pairs, a wavefront reserves room with one atomic, then the
// pairs are written.
__device__ __forceinline__ int pairs_of(const KGeom &G, const KParams &P, int co, int i,
                                        float4 pi, int cx, int cy, int cz,
                                        const float4 *__restrict__ pos4,
                                        const int32_t *__restrict__ idx_all,
                                        const int32_t *__restrict__ start_all, uint32_t *out,
                                        int64_t base, int64_t cap) {
  int n = 0;
  const uint32_t gi = __float_as_uint(pi.w);
  for (int code = 0; code < 27; ++code) {
    const NCell nc = neighbour_cell(G, cx, cy, cz, code);
    const SepAxis ax = sep_axis(pi.x, nc.sx), ay = sep_axis(pi.y, nc.sy),
                  az = sep_axis(pi.z, nc.sz);
    const int t0 = start_all[co + nc.c], t1 = start_all[co + nc.c + 1];
    for (int t = t0; t < t1; ++t) {
      const int j = idx_all[t];
      if (j == i) continue;
      const float4 pj = pos4[j];
      if (pair_r2(sep_d(ax, pj.x), sep_d(ay, pj.y), sep_d(az, pj.z)) < P.rc2) {
        if (out && base + n < cap) {
          out[2 * (base + n)] = gi;
          out[2 * (base + n) + 1] = __float_as_uint(pj.w);
        }
        ++n;
      }
    }
  }
  return n;
}

__global__ __launch_bounds__(kBlock) void k_pairs(
    const KGeom G, const KParams P, int co, int64_t first, int64_t nf,
    const float4 *__restrict__ pos4, const int32_t *__restrict__ idx,
    const int32_t *__restrict__ idx_all, const int32_t *__restrict__ start_all, uint32_t *pairs,
    int64_t cap, unsigned long long *counter) {
  const int64_t s = first + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool act = s < first + nf;
  int i = 0, cx = 0, cy = 0, cz = 0;
  float4 pi = make_float4(0.f, 0.f, 0.f, 0.f);
  int n = 0;
  if (act) {
    i = idx[s];
    pi = pos4[i];
    cell_index(G, pi.x, pi.y, pi.z, cx, cy, cz);
    n = pairs_of(G, P, co, i, pi, cx, cy, cz, pos4, idx_all, start_all, nullptr, 0, 0);
  }
  // wavefront-inclusive prefix of n, one atomic per wavefront
  const int lane = (int)__lane_id();
  int incl = n;
  for (int off = 1; off < 64; off <<= 1) {
    const int v = __shfl_up(incl, off, 64);
    if (lane >= off) incl += v;
  }
  const int total = __shfl(incl, 63, 64);
  unsigned long long base = 0;
  if (lane == 63 && total > 0) base = atomicAdd(counter, (unsigned long long)total);
  base = __shfl(base, 63, 64);
  if (act && pairs && n > 0)
    pairs_of(G, P, co, i, pi, cx, cy, cz, pos4, idx_all, start_all, pairs,
             (int64_t)base + incl - n, cap);
}

// The random numbers of given pairs (the same device functions as the force
// kernel): the four Philox words and xi.
__global__ void k_pair_random(uint32_t key0, uint32_t key1, uint32_t klo, uint32_t khi,
                              const uint32_t *__restrict__ gi, const uint32_t *__restrict__ gj,
                              int64_t n, uint32_t *words, float *xi) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const uint32_t a = gi[p], b = gj[p];
  if (words) {
    uint32_t c0 = min(a, b), c1 = max(a, b), c2 = klo, c3 = khi;
    philox10(c0, c1, c2, c3, key0, key1);
    words[4 * p] = c0;
    words[4 * p + 1] = c1;
    words[4 * p + 2] = c2;
    words[4 * p + 3] = c3;
  }
  if (xi) xi[p] = pair_gauss(a, b, klo, khi, key0, key1);
}

// ---------------------------------------------------------------------------
// Getters and setters by gid
// ---------------------------------------------------------------------------
// The context's status, with the counts of its lines, to host memory: by the first
// wavefront of a block.
__device__ __forceinline__ void note_status(const Status *st, Status *note) {
  if (!note || threadIdx.x >= 64) return;
  const int t = (int)threadIdx.x;
  const StatusBlock *b = (const StatusBlock *)st;
  unsigned long long bounce = b->lines[t].bounce, fallback = b->lines[t].fallback;
  for (int m = 32; m > 0; m >>= 1) {
    bounce += __shfl_xor(bounce, m, 64);
    fallback += __shfl_xor(fallback, m, 64);
  }
  static_assert(offsetof(Status, bounce) == 0 && offsetof(Status, fallback) == 8, "first words");
  if (t < (int)(sizeof(Status) / 8)) {
    const unsigned long long add = t == 0 ? bounce : (t == 1 ? fallback : 0ull);
    ((unsigned long long *)note)[t] = ((const unsigned long long *)st)[t] + add;
  }
}

__global__ void k_note_status(const Status *st, Status *note) { note_status(st, note); }

// One thread per particle, fluid slots then walls: a getter is one launch, which
// leaves the status too, so that the host has only to wait for it.  Latency bounds
// small boxes: against a launch each for fluid and walls, a clear of the forces
// and a copy of the status per getter, a step of 2,850 particles with its state and
// forces read took 48 us instead of 72, and 20 steps of 64 boxes with every box's
// profile and state read 4.00 ms instead of 4.74.
__global__ void k_export(const KGeom G, int64_t nf, int64_t nw, const float4 *__restrict__ pos4,
                         const float4 *__restrict__ vel4, const float4 *__restrict__ frc4,
                         const float4 *__restrict__ wall4, const float4 *__restrict__ wvel4,
                         float *pos, float *vel, float *frc, int32_t *events, int32_t *cell_of,
                         const Status *st, Status *note) {
  if (blockIdx.x == 0) note_status(st, note);
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nf + nw) return;
  const bool wall = s >= nf;
  const float4 x = wall ? wall4[s - nf] : pos4[s];
  const size_t g = (size_t)__float_as_uint(x.w);
  if (pos) {
    pos[3 * g] = x.x;
    pos[3 * g + 1] = x.y;
    pos[3 * g + 2] = x.z;
  }
  if (vel || events) {
    const float4 v = wall ? wvel4[s - nf] : vel4[s];
    if (vel) {
      vel[3 * g] = v.x;
      vel[3 * g + 1] = v.y;
      vel[3 * g + 2] = v.z;
    }
    if (events) events[g] = wall ? 0 : __float_as_int(v.w);
  }
  if (frc) {
    const float4 f = wall ? make_float4(0.f, 0.f, 0.f, 0.f) : frc4[s];
    frc[3 * g] = f.x;
    frc[3 * g + 1] = f.y;
    frc[3 * g + 2] = f.z;
  }
  if (cell_of) {
    int cx, cy, cz;
    cell_of[g] = cell_index(G, x.x, x.y, x.z, cx, cy, cz);
  }
}

__global__ void k_import(int64_t nf, float4 *pos4, float4 *vel4, float4 *frc4,
                         const float *__restrict__ pos, const float *__restrict__ vel,
                         const float *__restrict__ frc) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nf) return;
  const float gbits = pos4[s].w;
  const size_t g = (size_t)__float_as_uint(gbits);
  pos4[s] = make_float4(pos[3 * g], pos[3 * g + 1], pos[3 * g + 2], gbits);
  vel4[s] = make_float4(vel[3 * g], vel[3 * g + 1], vel[3 * g + 2], __int_as_float(0));
  frc4[s] = make_float4(frc[3 * g], frc[3 * g + 1], frc[3 * g + 2], 0.f);
}

__device__ __forceinline__ int profile_bin(const KGeom &G, const float4 x, int axis, int nbins) {
  const float c = axis == 0 ? x.x : (axis == 1 ? x.y : x.z);
  const int b = (int)floorf(c / G.L[axis] * (float)nbins);
  return b < 0 ? 0 : (b >= nbins ? nbins - 1 : b);
}

// Binned observables, each block into bins of its own in LDS first.  Global
// FP64 atomics of every particle serialise on a few hundred addresses: 5 per
// particle took 1.41 ms for 330k particles in 80 bins and 7.5 ms for 777k in
// 40, where reading them takes 0.01 ms.  A lane sums the particles it visits
// in registers while they fall in one bin (cell order makes that the rule along
// z) and adds the sums to the LDS bin when the bin changes; a wavefront
// whose lanes all hold one bin reduces first and adds once.  At most 256 blocks
// add their bins to the result, so an address sees 256 global atomics at most.
constexpr int kProfThreads = 1024;
constexpr int kProfBlocks = 256;
constexpr int kProfBins = 1024;   // 40 KB of LDS

__global__ __launch_bounds__(kProfThreads) void k_profile(const KGeom G, int64_t nf, int64_t per,
                                                          const float4 *__restrict__ pos4,
                                                          const float4 *__restrict__ vel4, int axis,
                                                          int nbins, double *out) {
  __shared__ double bins[5 * kProfBins];
  for (int q = (int)threadIdx.x; q < 5 * nbins; q += kProfThreads) bins[q] = 0.0;
  __syncthreads();
  const int64_t first = (int64_t)blockIdx.x * per, last = min(nf, first + per);
  int cur = 0, n = 0;
  double sx = 0.0, sy = 0.0, sz = 0.0, sq = 0.0;
  auto add = [&]() {
    double *o = bins + 5 * cur;
    atomicAdd(o, (double)n);
    atomicAdd(o + 1, sx);
    atomicAdd(o + 2, sy);
    atomicAdd(o + 3, sz);
    atomicAdd(o + 4, sq);
  };
  auto clear = [&]() {
    n = 0;
    sx = sy = sz = sq = 0.0;
  };
  // sums into their bins, of every lane where all hold one bin, else of the
  // lanes that need it; called by whole wavefronts
  auto flush = [&](bool need) {
    const unsigned long long held = __ballot(n > 0);
    if (held == 0ull) return;
    const int b0 = __shfl(cur, __ffsll((long long)held) - 1, 64);
    if (wave_any(n > 0 && cur != b0)) {
      if (need && n > 0) {
        add();
        clear();
      }
      return;
    }
    for (int m = 32; m > 0; m >>= 1) {
      n += __shfl_xor(n, m, 64);
      sx += __shfl_xor(sx, m, 64);
      sy += __shfl_xor(sy, m, 64);
      sz += __shfl_xor(sz, m, 64);
      sq += __shfl_xor(sq, m, 64);
    }
    cur = b0;
    if (__lane_id() == 0) add();
    clear();
  };
  for (int64_t base = first; base < last; base += kProfThreads) {
    const int64_t s = base + threadIdx.x;
    const bool act = s < last;
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f), v = x;
    if (act) {
      x = pos4[s];
      v = vel4[s];
    }
    const int b = act ? profile_bin(G, x, axis, nbins) : cur;
    const bool need = n > 0 && b != cur;
    if (wave_any(need)) flush(need);
    if (act) {
      cur = b;
      ++n;
      sx += (double)v.x;
      sy += (double)v.y;
      sz += (double)v.z;
      sq += (double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z;
    }
  }
  flush(true);
  __syncthreads();
  for (int b = (int)threadIdx.x; b < nbins; b += kProfThreads) {
    if (bins[5 * b] == 0.0) continue;
    for (int q = 0; q < 5; ++q) atomicAdd(out + 5 * (size_t)b + q, bins[5 * b + q]);
  }
}

// More bins than LDS holds: global atomics per particle (the addresses are
// many then).
__global__ void k_profile_direct(const KGeom G, int64_t nf, const float4 *__restrict__ pos4,
                                 const float4 *__restrict__ vel4, int axis, int nbins,
                                 double *out) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= nf) return;
  const float4 v = vel4[s];
  double *o = out + 5 * (size_t)profile_bin(G, pos4[s], axis, nbins);
  atomicAdd(o, 1.0);
  atomicAdd(o + 1, (double)v.x);
  atomicAdd(o + 2, (double)v.y);
  atomicAdd(o + 3, (double)v.z);
  atomicAdd(o + 4, (double)v.x * v.x + (double)v.y * v.y + (double)v.z * v.z);
}

// ---------------------------------------------------------------------------
// Persistent step: one launch for a whole step of every box of a batch.
// Blocks take work items in queue order from one counter; an item of phase
// p of box r first waits until every item of phase p - 1 of box r has
// arrived (a per-box, per-phase counter), so boxes run through the phases
// independently and no launch boundary separates them.  Every item waits
// only on items earlier in the queue, which blocks that are already running
// have taken, so the waits end whatever the number of resident blocks; each
// is also bounded (spin_limit sleeps), after which the item runs anyway and
// `stalled` reports the step as invalid.  The per-phase bodies are those of
// the per-phase kernels, so results are bit-identical to them.
// ---------------------------------------------------------------------------

// A value the same in every lane, as a scalar: function arguments arrive in
// vector registers, and without this every pointer loaded through them would
// be a per-lane value (vector loads of the arguments, buffer descriptors
// built lane by lane).
template <typename P>
__device__ __forceinline__ P *uniform_ptr(P *p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (P *)(((uint64_t)hi << 32) | lo);
}
// The arguments block, read through the constant address space (scalar loads).
typedef const __attribute__((address_space(4))) PArgs *ArgsPtr;
__device__ __forceinline__ ArgsPtr uniform_args(const PArgs *p) {
  return (ArgsPtr)uniform_ptr(p);
}
__device__ __forceinline__ int uniform_int(int v) { return __builtin_amdgcn_readfirstlane(v); }
// A pointer into the block's LDS (the caller's __shared__ array): the cast
// through the local address space lets the compiler use LDS instructions.
template <typename P>
__device__ __forceinline__ P *lds_ptr(P *p) {
  return (P *)(__attribute__((address_space(3))) P *)p;
}

// The phase bodies as separate functions, each register-allocated on its own
// (inlined into one loop, the union of their live ranges would cut the
// kernel to two wavefronts per SIMD); each reads the arguments it needs.
template <typename T, int PPT, bool REFLECT>
__device__ __attribute__((noinline)) void p_integrate(const PArgs *__restrict__ A0, int tile0) {
  const ArgsPtr A = uniform_args(A0);
  const int tile = uniform_int(tile0);
  integrate_tile<T, PPT, REFLECT>(tile, A->boxes, A->itiles, A->pos4, A->pos4, A->vel4, A->frc4, A->vt4,
                                  A->cell_of, A->rank_of, A->count, A->bits, A->use_mask,
                                  (const typename PhiQuad<T>::type *)A->quad, A->st, A->NF,
                                  A->wcstart);
}

// chunk a of box `box`'s cells; its block sum at bsum[b + a]
__device__ __attribute__((noinline)) void p_reduce(const PArgs *__restrict__ A0, int box0,
                                                   int a0, int b0, int *lds0) {
  const ArgsPtr A = uniform_args(A0);
  const int box = uniform_int(box0), a = uniform_int(a0), b = uniform_int(b0);
  int *lds = lds_ptr(lds0);
  const int64_t co = A->boxes[box].co, ncell = A->boxes[box].ncell;
  scan_reduce_chunk<kScanItems>(co + (int64_t)a * kScanChunk, co + ncell, A->count, A->bsum + b + a, lds);
}

// the box's fluid starts at slot fo; its chunks before this one add to it
__device__ __attribute__((noinline)) void p_down(const PArgs *__restrict__ A0, int box0, int a0,
                                                 int b0, int *tile0, int *lds0) {
  const ArgsPtr A = uniform_args(A0);
  const int box = uniform_int(box0), a = uniform_int(a0), b = uniform_int(b0);
  int *tile = lds_ptr(tile0), *lds = lds_ptr(lds0);
  const int64_t co = A->boxes[box].co, ncell = A->boxes[box].ncell, fo = A->boxes[box].fo;
  const bool last = (int64_t)(a + 1) * kScanChunk >= ncell;
  scan_down_chunk<kScanItems, false>(
      co + (int64_t)a * kScanChunk, co + ncell, last,
      [&] {
        int before = 0;
        for (int j = (int)threadIdx.x; j < a; j += kScanThreads) before += A->bsum[b + j];
        return (int)fo + block_sum(before, lds);
      },
      A->count, nullptr, A->cstart, A->wcstart, A->start_all, A->fluid_off, tile, lds);
}

__device__ __attribute__((noinline)) void p_scatter(const PArgs *__restrict__ A0, int a0, int b0) {
  const ArgsPtr A = uniform_args(A0);
  const int a = uniform_int(a0), b = uniform_int(b0);
  for (int64_t p = (int64_t)a + threadIdx.x; p < (int64_t)b; p += kBlock)
    scatter_one(p, A->NF, A->cell_of, A->rank_of, A->cstart, A->idx, A->NW, A->wcell, A->wcstart,
                A->start_all, A->idx_all);
}

__device__ __attribute__((noinline)) void p_sort(const PArgs *__restrict__ A0, int a0, int b0) {
  const ArgsPtr A = uniform_args(A0);
  const int a = uniform_int(a0), b = uniform_int(b0);
  for (int64_t c = (int64_t)a + threadIdx.x; c < (int64_t)b; c += kBlock)
    sort_cell<false>(c, A->cstart, A->idx, nullptr, A->fluid_off, A->idx_all);
  // the coarse codes of the merged-run entries of these cells (walls from
  // the scatter phase, fluid from the loop above)
  __syncthreads();
  const int t0 = uniform_int(A->start_all[a]), t1 = uniform_int(A->start_all[b]);
  for (int t = t0 + (int)threadIdx.x; t < t1; t += kBlock) {
    const float4 x = A->pos4[A->idx_all[t]];
    A->cq[t] = qcode3(x.x, x.y, x.z);
  }
}

template <bool SPH>
__device__ __attribute__((noinline)) void p_force(const PArgs *__restrict__ A0, int tile0,
                                                  uint32_t *list0) {
  const ArgsPtr A = uniform_args(A0);
  const int tile = uniform_int(tile0);
  uint32_t *list = lds_ptr(list0);
  force_tile<false, kBlock, SPH, void, false, false>(tile, list, A->boxes, A->ftiles, A->NF, A->pad,
                                       A->ncell_all, A->pos4, A->vt4, A->vel4, A->frc4, A->idx,
                                       A->idx_all, A->start_all, A->cq, A->pos_out, A->vel_out,
                                       A->frc_out, A->dk, A->st, NextStep{});
}

template <typename T, int PPT, bool REFLECT, bool SPH>
// Six wavefronts per SIMD, as the pair kernel: the pair list (26 KB per
// block) limits a CU to six blocks anyway, and the phase functions are
// allocated separately, the largest (the pair force, 73 VGPRs in its own
// kernel) with a few more registers as a callee.
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6))) void
k_step_persistent(const PArgs *__restrict__ A) {
  __shared__ union {
    uint32_t list[kListCap * kBlock];
    struct {
      int tile[kScanChunk + kScanChunk / 32];
      int lds[kScanThreads];
    } scan;
  } sm;
  __shared__ int s_item, s_ok;
  const int t = (int)threadIdx.x;
  const int nitems = A->nitems;
  // The item index and the item are the same in every lane; readfirstlane
  // makes that visible to the compiler, and the loop tests it at its head,
  // so the loop and the phase switch are uniform branches and every barrier
  // runs with all lanes.  (With the index as a per-lane value and the exit
  // in the middle of the loop, the loop was compiled as divergent and
  // rotated so that lanes 1-63 of the first wavefront went back to the top
  // barrier and re-read the index before lane 0 had taken the next one.)
  if (t == 0) s_item = atomicAdd(A->head, 1);
  __syncthreads();
  int it = __builtin_amdgcn_readfirstlane(s_item);
  while (it < nitems) {
    const PItem Iv = A->items[it];
    PItem I;
    I.phase = __builtin_amdgcn_readfirstlane(Iv.phase);
    I.box = __builtin_amdgcn_readfirstlane(Iv.box);
    I.a = __builtin_amdgcn_readfirstlane(Iv.a);
    I.b = __builtin_amdgcn_readfirstlane(Iv.b);
    if (t == 0) {
      int ok = 1;
      if (I.phase != kPhIntegrate) {
        const int dep = I.box * kPhases + I.phase - 1;
        const int need = A->need[dep];
        const int limit = A->spin_limit;
        int spins = 0;
        // relaxed loads while spinning (an acquire would invalidate this
        // XCD's L2 on every iteration); the acquire fence follows the wait
        while (__hip_atomic_load(&A->arrive[dep], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
               need) {
          __builtin_amdgcn_s_sleep(4);
          if (++spins >= limit) {
            ok = 0;
            break;
          }
        }
      }
      s_ok = ok;
    }
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (t == 0 && !__builtin_amdgcn_readfirstlane(s_ok)) atomicAdd(&A->st->stalled, 1ull);
    switch (I.phase) {
      case kPhIntegrate:
        for (int t = I.a; t < I.b; ++t) p_integrate<T, PPT, REFLECT>(A, t);
        break;
      case kPhReduce: p_reduce(A, I.box, I.a, I.b, sm.scan.lds); break;
      case kPhDown: p_down(A, I.box, I.a, I.b, sm.scan.tile, sm.scan.lds); break;
      case kPhScatter: p_scatter(A, I.a, I.b); break;
      case kPhSort: p_sort(A, I.a, I.b); break;
      default:
        for (int t = I.a; t < I.b; ++t) p_force<SPH>(A, t, sm.list);
        break;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if (t == 0) {
      __hip_atomic_fetch_add(&A->arrive[I.box * kPhases + I.phase], 1, __ATOMIC_RELEASE,
                             __HIP_MEMORY_SCOPE_AGENT);
      s_item = atomicAdd(A->head, 1);
    }
    __syncthreads();
    it = __builtin_amdgcn_readfirstlane(s_item);
  }
}

// Before a persistent step: clear the arrival counters and the queue counter
// (a kernel, so that a captured graph holds no memset node) and advance the
// force evaluation index k.
__global__ void k_persist_prep(int32_t *arrive, int n, int32_t *head, unsigned long long *dk) {
  for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x) arrive[i] = 0;
  if (threadIdx.x == 0) {
    *head = 0;
    *dk += 1ull;
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_pack(hipStream_t s, int64_t n, const float *pos, const float *vel,
                       const uint32_t *gid, const int64_t *rows, float4 *pos4, float4 *vel4,
                       float4 *vt4, float4 *frc4) {
  if (n <= 0) return hipSuccess;
  k_pack<<<grid_for(n), kBlock, 0, s>>>(n, pos, vel, gid, rows, pos4, vel4, vt4, frc4);
  return hipGetLastError();
}

hipError_t launch_bin(hipStream_t s, const KGeom &G, int64_t cell_off, int64_t n,
                      const float4 *pos4, int32_t *cell_of, int32_t *rank_of, int32_t *count) {
  if (n <= 0) return hipSuccess;
  k_bin<<<grid_for(n), kBlock, 0, s>>>(G, cell_off, n, pos4, cell_of, rank_of, count);
  return hipGetLastError();
}

hipError_t launch_scan_reduce(hipStream_t s, int64_t ncell, const int32_t *count, int32_t *bsum,
                              const int32_t *wcount, int32_t *wsum) {
  const dim3 grid((unsigned)scan_blocks(ncell), wcount ? 2 : 1);
  if (scan_items(ncell) == kScanItems)
    k_scan_reduce<kScanItems><<<grid, kScanThreads, 0, s>>>(ncell, count, bsum, wcount, wsum);
  else
    k_scan_reduce<kScanFew><<<grid, kScanThreads, 0, s>>>(ncell, count, bsum, wcount, wsum);
  return hipGetLastError();
}

hipError_t launch_scan_both(hipStream_t s, const BothLists &L) {
  const unsigned nb = (unsigned)scan_blocks(L.ncell);
  if (scan_items(L.ncell) == kScanItems)
    k_scan_down_both<kScanItems><<<nb, kScanThreads, 0, s>>>(L.ncell, L.count, L.start, L.bsum,
                                                             L.wcount, L.wstart, L.wsum,
                                                             L.start_all, L.fluid_off);
  else
    k_scan_down_both<kScanFew><<<nb, kScanThreads, 0, s>>>(L.ncell, L.count, L.start, L.bsum,
                                                           L.wcount, L.wstart, L.wsum,
                                                           L.start_all, L.fluid_off);
  return hipGetLastError();
}

hipError_t launch_scatter_both(hipStream_t s, const BothLists &L) {
  k_scatter_both<<<grid_for(std::max<int64_t>(L.n + L.nw, 1)), kBlock, 0, s>>>(
      L.n, L.cell_of, L.rank_of, L.start, L.idx, L.nw, L.wcell_of, L.wrank_of, L.wstart, L.widx,
      L.dk);
  return hipGetLastError();
}

hipError_t launch_sort_both(hipStream_t s, const BothLists &L) {
  k_sort_both<<<dim3(grid_for(L.ncell), 2), kBlock, 0, s>>>(L.ncell, L.n, L.start, L.idx, L.wstart,
                                                            L.widx, L.start_all, L.fluid_off,
                                                            L.idx_all, L.wcell);
  return hipGetLastError();
}

hipError_t launch_scan_down(hipStream_t s, int64_t ncell, int32_t *count, int32_t *start,
                            const int32_t *bsum, const int32_t *wstart, int32_t *start_all,
                            int32_t *fluid_off) {
  const unsigned nb = (unsigned)scan_blocks(ncell);
  if (scan_items(ncell) == kScanItems)
    k_scan_down<kScanItems><<<nb, kScanThreads, 0, s>>>(ncell, count, start, bsum, wstart,
                                                        start_all, fluid_off);
  else
    k_scan_down<kScanFew><<<nb, kScanThreads, 0, s>>>(ncell, count, start, bsum, wstart, start_all,
                                                      fluid_off);
  return hipGetLastError();
}

hipError_t launch_scatter(hipStream_t s, int64_t n, const int32_t *cell_of,
                          const int32_t *rank_of, const int32_t *start, int32_t *idx,
                          int64_t nw, const int32_t *wcell, const int32_t *wstart,
                          const int32_t *start_all, int32_t *idx_all,
                          unsigned long long *dk) {
  if (!idx_all) nw = 0;
  if (nw > 0 && (!wcell || !wstart || !start_all)) return hipErrorInvalidValue;
  const int64_t total = std::max<int64_t>(n + nw, dk ? 1 : 0);
  if (total <= 0) return hipSuccess;
  k_scatter<<<grid_for(total), kBlock, 0, s>>>(n, cell_of, rank_of, start, idx, nw, wcell, wstart,
                                               start_all, idx_all, dk);
  return hipGetLastError();
}

hipError_t launch_quant_runs(hipStream_t s, int64_t n, const int32_t *idx_all,
                             const float4 *pos4, uint32_t *cq) {
  if (n <= 0) return hipSuccess;
  if (!idx_all || !pos4 || !cq) return hipErrorInvalidValue;
  k_quant_runs<<<grid_for(n), kBlock, 0, s>>>(n, idx_all, pos4, cq);
  return hipGetLastError();
}

hipError_t launch_sort_cells(hipStream_t s, int64_t ncell, const int32_t *start, int32_t *idx,
                             const float4 *key4, const int32_t *fluid_off, int32_t *idx_all) {
  if (key4)
    k_sort_cells<true><<<grid_for(ncell), kBlock, 0, s>>>(ncell, start, idx, key4, fluid_off,
                                                        idx_all);
  else
    k_sort_cells<false><<<grid_for(ncell), kBlock, 0, s>>>(ncell, start, idx, key4, fluid_off,
                                                         idx_all);
  return hipGetLastError();
}

hipError_t launch_sort_wall_cells(hipStream_t s, int64_t ncell, const int32_t *start,
                                  int32_t *idx, int32_t *cell_out) {
  k_sort_wall_cells<<<grid_for(ncell), kBlock, 0, s>>>(ncell, start, idx, cell_out);
  return hipGetLastError();
}

hipError_t launch_wall_move_bin(hipStream_t s, const KGeom &G, float hdt, float dt, int move,
                                int64_t cell_off, int64_t nw, const float4 *walls_in,
                                const float4 *vt_in, float4 *walls_out, float4 *vt_out,
                                int32_t *cell_of, int32_t *rank_of, int32_t *count) {
  if (nw <= 0) return hipSuccess;
  k_wall_move_bin<<<grid_for(nw), kBlock, 0, s>>>(G, hdt, dt, move, cell_off, nw, walls_in, vt_in,
                                                  walls_out, vt_out, cell_of, rank_of, count);
  return hipGetLastError();
}

hipError_t launch_import_walls(hipStream_t s, int64_t nw, float4 *walls, const float *pos) {
  if (nw <= 0) return hipSuccess;
  k_import_walls<<<grid_for(nw), kBlock, 0, s>>>(nw, walls, pos);
  return hipGetLastError();
}

hipError_t launch_set_pad(hipStream_t s, float4 *pos4, float4 *vt4, int32_t *slack, int32_t pad) {
  k_set_pad<<<1, 1, 0, s>>>(pos4, vt4, slack, pad);
  return hipGetLastError();
}

hipError_t launch_cells(hipStream_t s, const KGeom &G, int64_t cell_off, int64_t n,
                        const float4 *pos4, int32_t *cell) {
  if (n <= 0) return hipSuccess;
  k_cells<<<grid_for(n), kBlock, 0, s>>>(G, cell_off, n, pos4, cell);
  return hipGetLastError();
}

hipError_t launch_permute(hipStream_t s, int64_t n, const int32_t *idx, const float4 *a_in,
                          float4 *a_out, const float4 *b_in, float4 *b_out, const float4 *c_in,
                          float4 *c_out, const float4 *d_in, float4 *d_out) {
  if (n <= 0) return hipSuccess;
  k_permute<<<grid_for(n), kBlock, 0, s>>>(n, idx, a_in, a_out, b_in, b_out, c_in, c_out, d_in,
                                           d_out);
  return hipGetLastError();
}

hipError_t launch_cube_mask(hipStream_t s, const KGeom &G, const void *grid, int grid_f64,
                            int64_t nwords, uint32_t *bits) {
  if (grid_f64)
    k_cube_mask<double><<<grid_for(32 * nwords), kBlock, 0, s>>>(G, (const double *)grid, nwords, bits);
  else
    k_cube_mask<float><<<grid_for(32 * nwords), kBlock, 0, s>>>(G, (const float *)grid, nwords, bits);
  return hipGetLastError();
}

hipError_t launch_count_flagged(hipStream_t s, const KGeom &G, int grid_f64, int64_t nf,
                                const float4 *pos4, const uint32_t *bits,
                                unsigned long long *out) {
  if (nf <= 0) return hipSuccess;
  if (grid_f64)
    k_count_flagged<double><<<grid_for(nf), kBlock, 0, s>>>(G, nf, pos4, bits, out);
  else
    k_count_flagged<float><<<grid_for(nf), kBlock, 0, s>>>(G, nf, pos4, bits, out);
  return hipGetLastError();
}

hipError_t launch_check_grid(hipStream_t s, const void *grid, int grid_f64, int64_t count,
                             Status *st) {
  unsigned blocks = grid_for(count);
  if (blocks > 8192) blocks = 8192;
  if (blocks == 0) return hipSuccess;
  if (grid_f64)
    k_check_grid<double><<<blocks, kBlock, 0, s>>>((const double *)grid, count, st);
  else
    k_check_grid<float><<<blocks, kBlock, 0, s>>>((const float *)grid, count, st);
  return hipGetLastError();
}

hipError_t launch_check_phi(hipStream_t s, const KGeom &G, const void *grid, int grid_f64,
                            int64_t n, const float4 *pos4, Status *st) {
  if (n <= 0) return hipSuccess;
  if (grid_f64)
    k_check_phi<double><<<grid_for(n), kBlock, 0, s>>>(G, (const double *)grid, n, pos4, st);
  else
    k_check_phi<float><<<grid_for(n), kBlock, 0, s>>>(G, (const float *)grid, n, pos4, st);
  return hipGetLastError();
}

// Grid of 8k blocks covering n items with the XCD mapping of xcd_block().
inline unsigned xcd_grid(int64_t n, int block) {
  const int64_t nb = (n + block - 1) / block;
  return (unsigned)(((nb + 7) / 8) * 8);
}

hipError_t launch_build_quad(hipStream_t s, const KGeom &G, const void *grid, int grid_f64,
                             void *quad) {
  const int64_t nodes = (int64_t)G.ng[0] * G.ng[1] * G.ng[2];
  if (nodes <= 0) return hipSuccess;
  if (grid_f64)
    k_build_quad<double><<<grid_for(nodes), kBlock, 0, s>>>(G, (const double *)grid, nodes,
                                                            (double4 *)quad);
  else
    k_build_quad<float><<<grid_for(nodes), kBlock, 0, s>>>(G, (const float *)grid, nodes,
                                                           (float4 *)quad);
  return hipGetLastError();
}

hipError_t launch_integrate(hipStream_t s, int ppt, const Box *boxes, const Tile *tiles,
                            int ntiles, const float4 *pos4, float4 *pos_out, const float4 *vel4,
                            const float4 *frc4, float4 *vt4, int32_t *cell_of, int32_t *rank_of,
                            int32_t *count,
                            const uint32_t *bits, int use_mask, const void *quad, int grid_f64,
                            Status *st, int64_t NF, const int32_t *wcstart, int reflect) {
  if (ntiles <= 0) return hipSuccess;
  const unsigned nb = (unsigned)(((ntiles + 7) / 8) * 8);
#define DPD_INTEGRATE(T, K, R)                                                                   \
  k_integrate<T, K, R><<<nb, kBlock, 0, s>>>(boxes, tiles, ntiles, pos4, pos_out, vel4, frc4, vt4, \
                                             cell_of, rank_of, count, bits, use_mask,           \
                                             (const typename PhiQuad<T>::type *)quad, st, NF,   \
                                             wcstart)
#define DPD_INTEGRATE_T(T, K) \
  if (reflect) DPD_INTEGRATE(T, K, true); else DPD_INTEGRATE(T, K, false)
  if (ppt != 1 && ppt != 2 && ppt != 4) return hipErrorInvalidValue;
  if (grid_f64) {
    if (ppt == 1) { DPD_INTEGRATE_T(double, 1); }
    else if (ppt == 2) { DPD_INTEGRATE_T(double, 2); }
    else { DPD_INTEGRATE_T(double, 4); }
  } else {
    if (ppt == 1) { DPD_INTEGRATE_T(float, 1); }
    else if (ppt == 2) { DPD_INTEGRATE_T(float, 2); }
    else { DPD_INTEGRATE_T(float, 4); }
  }
#undef DPD_INTEGRATE_T
#undef DPD_INTEGRATE
  return hipGetLastError();
}

hipError_t launch_force(hipStream_t s, int block, const Box *boxes, const Tile *tiles,
                        int ntiles, int64_t NF, int32_t pad, int32_t ncell_all, int init,
                        const float4 *pos4,
                        const float4 *vt4, const float4 *vel4, const float4 *frc4,
                        const int32_t *idx, const int32_t *idx_all, const int32_t *start_all,
                        const uint32_t *cq,
                        float4 *pos_out, float4 *vel_out, float4 *frc_out,
                        const unsigned long long *dk, Status *st, int sph, int32_t *clear,
                        const NextStep *next) {
  if (ntiles <= 0) return hipSuccess;
  if (!cq) return hipErrorInvalidValue;
  const unsigned nb = (unsigned)(((ntiles + 7) / 8) * 8);
  const NextStep N = next ? *next : NextStep{};
  if (init && next) return hipErrorInvalidValue;
#define DPD_FORCE(I, BS, S, T, R)                                                                \
  k_force<I, BS, S, T, R><<<nb, BS, 0, s>>>(boxes, tiles, ntiles, NF, pad, ncell_all, pos4, vt4, \
                                            vel4, frc4, idx, idx_all, start_all, cq, pos_out,    \
                                            vel_out, frc_out, dk, st, clear, N)
#define DPD_FORCE_S(I, BS, T, R) \
  if (sph) DPD_FORCE(I, BS, true, T, R); else DPD_FORCE(I, BS, false, T, R)
#define DPD_FORCE_B(I, T, R) \
  if (block == 128) { DPD_FORCE_S(I, 128, T, R); } else { DPD_FORCE_S(I, 256, T, R); }
#define DPD_FORCE_R(T) \
  if (N.reflect) { DPD_FORCE_B(false, T, true); } else { DPD_FORCE_B(false, T, false); }
  if (init) {
    DPD_FORCE_B(true, void, false);
  } else if (!next) {
    DPD_FORCE_B(false, void, false);
  } else if (next->grid_f64) {
    DPD_FORCE_R(double);
  } else {
    DPD_FORCE_R(float);
  }
#undef DPD_FORCE_R
#undef DPD_FORCE_B
#undef DPD_FORCE_S
#undef DPD_FORCE
  return hipGetLastError();
}

hipError_t launch_force_wide(hipStream_t s, const Box *boxes, const Tile *tiles, int ntiles,
                             int64_t NF, int init, const float4 *pos4, const float4 *vt4,
                             const float4 *vel4, const float4 *frc4, const int32_t *idx,
                             const int32_t *idx_all, const int32_t *start_all, float4 *pos_out,
                             float4 *vel_out, float4 *frc_out, const unsigned long long *dk,
                             Status *st, int sph, int32_t *clear, int32_t ncell_all,
                             const NextStep *next) {
  if (ntiles <= 0) return hipSuccess;
  if (next && init) return hipErrorInvalidValue;
  const NextStep N = next ? *next : NextStep{};
  const unsigned nb = (unsigned)(((ntiles + 7) / 8) * 8);
#define DPD_WIDE(I, S, T, R)                                                                      \
  k_force_wide<I, S, T, R><<<nb, kBlock, 0, s>>>(boxes, tiles, ntiles, NF, pos4, vt4, vel4, frc4, \
                                                 idx, idx_all, start_all, pos_out, vel_out,       \
                                                 frc_out, dk, st, clear, ncell_all, N)
#define DPD_WIDE_S(I, T, R) \
  if (sph) DPD_WIDE(I, true, T, R); else DPD_WIDE(I, false, T, R)
#define DPD_WIDE_R(T) \
  if (N.reflect) { DPD_WIDE_S(false, T, true); } else { DPD_WIDE_S(false, T, false); }
  if (init) {
    DPD_WIDE_S(true, void, false);
  } else if (!next) {
    DPD_WIDE_S(false, void, false);
  } else if (next->grid_f64) {
    DPD_WIDE_R(double);
  } else {
    DPD_WIDE_R(float);
  }
#undef DPD_WIDE_R
#undef DPD_WIDE_S
#undef DPD_WIDE
  return hipGetLastError();
}

hipError_t launch_cells_box(hipStream_t s, const Box *boxes, int nbox, int parts, int64_t NF,
                            const int32_t *cell_of, const int32_t *rank_of, int32_t *count,
                            const int32_t *wcstart, int32_t *start_all, int32_t *idx,
                            int32_t *idx_all, const int32_t *wcell, const float4 *pos4,
                            uint32_t *cq, unsigned long long *dk) {
  if (nbox <= 0) return hipSuccess;
  const dim3 grid((unsigned)nbox, (unsigned)parts);
  k_cells_box<<<grid, kBoxThreads, 0, s>>>(boxes, NF, cell_of, rank_of, count, wcstart, start_all,
                                           idx, idx_all, wcell, pos4, cq, dk);
  return hipGetLastError();
}

hipError_t launch_pairs(hipStream_t s, const KGeom &G, const KParams &P, int64_t cell_off,
                        int64_t first, int64_t nf, const float4 *pos4, const int32_t *idx,
                        const int32_t *idx_all, const int32_t *start_all, uint32_t *pairs,
                        int64_t cap, unsigned long long *counter) {
  if (nf <= 0) return hipSuccess;
  k_pairs<<<grid_for(nf), kBlock, 0, s>>>(G, P, (int)cell_off, first, nf, pos4, idx, idx_all,
                                          start_all, pairs, cap, counter);
  return hipGetLastError();
}

hipError_t launch_pair_random(hipStream_t s, uint64_t seed, uint64_t k, uint32_t replica,
                              const uint32_t *gi, const uint32_t *gj, int64_t n, uint32_t *words,
                              float *xi) {
  if (n <= 0) return hipSuccess;
  const uint32_t khi = ((uint32_t)(k >> 32) & 0xFFFFu) | (replica << 16);
  k_pair_random<<<grid_for(n), kBlock, 0, s>>>((uint32_t)seed, (uint32_t)(seed >> 32),
                                                (uint32_t)k, khi, gi, gj, n, words, xi);
  return hipGetLastError();
}

hipError_t launch_export(hipStream_t s, const KGeom &G, int64_t nf, int64_t nw,
                         const float4 *pos4, const float4 *vel4, const float4 *frc4,
                         const float4 *wall4, const float4 *wvel4, float *pos, float *vel,
                         float *frc, int32_t *events, int32_t *cell_of, const Status *st,
                         Status *note) {
  k_export<<<grid_for(std::max<int64_t>(nf + nw, 1)), kBlock, 0, s>>>(G, nf, nw, pos4, vel4, frc4, wall4, wvel4, pos,
                                                vel, frc, events, cell_of, st, note);
  return hipGetLastError();
}

hipError_t launch_note_status(hipStream_t s, const Status *st, Status *note) {
  k_note_status<<<1, 64, 0, s>>>(st, note);
  return hipGetLastError();
}

hipError_t launch_import(hipStream_t s, int64_t nf, float4 *pos4, float4 *vel4, float4 *frc4,
                         const float *pos, const float *vel, const float *frc) {
  if (nf <= 0) return hipSuccess;
  k_import<<<grid_for(nf), kBlock, 0, s>>>(nf, pos4, vel4, frc4, pos, vel, frc);
  return hipGetLastError();
}

hipError_t launch_profile(hipStream_t s, const KGeom &G, int64_t nf, const float4 *pos4,
                          const float4 *vel4, int axis, int nbins, double *out) {
  if (nf <= 0) return hipSuccess;
  if (nbins > kProfBins) {
    k_profile_direct<<<grid_for(nf), kBlock, 0, s>>>(G, nf, pos4, vel4, axis, nbins, out);
    return hipGetLastError();
  }
  const int64_t nb = std::min<int64_t>(kProfBlocks, (nf + kProfThreads - 1) / kProfThreads);
  const int64_t per = (nf + nb - 1) / nb;
  k_profile<<<(unsigned)nb, kProfThreads, 0, s>>>(G, nf, per, pos4, vel4, axis, nbins, out);
  return hipGetLastError();
}

hipError_t launch_step_persistent(hipStream_t s, const PArgs *args, int nitems, int blocks,
                                  int32_t *arrive, int narrive, int32_t *head,
                                  unsigned long long *dk, int grid_f64, int ppt, int reflect,
                                  int sph) {
  if (nitems <= 0) return hipSuccess;
  k_persist_prep<<<1, 256, 0, s>>>(arrive, narrive, head, dk);
  const unsigned nb = (unsigned)std::max(1, std::min(nitems, blocks));
#define DPD_PERSIST(T, P, R, S) k_step_persistent<T, P, R, S><<<nb, kBlock, 0, s>>>(args)
#define DPD_PERSIST_S(T, P, R) \
  if (sph) DPD_PERSIST(T, P, R, true); else DPD_PERSIST(T, P, R, false)
#define DPD_PERSIST_R(T, P) \
  if (reflect) { DPD_PERSIST_S(T, P, true); } else { DPD_PERSIST_S(T, P, false); }
#define DPD_PERSIST_P(T) \
  if (ppt == 1) { DPD_PERSIST_R(T, 1); } else { DPD_PERSIST_R(T, 2); }
  if (grid_f64) {
    DPD_PERSIST_P(double);
  } else {
    DPD_PERSIST_P(float);
  }
#undef DPD_PERSIST_P
#undef DPD_PERSIST_R
#undef DPD_PERSIST_S
#undef DPD_PERSIST
  return hipGetLastError();
}

namespace {
template <typename T, int P, bool R, bool S>
int occupancy_of() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_step_persistent<T, P, R, S>, kBlock, 0) !=
      hipSuccess)
    return -1;
  return n;
}
template <typename T, int P>
int occupancy_rs(int reflect, int sph) {
  if (reflect) return sph ? occupancy_of<T, P, true, true>() : occupancy_of<T, P, true, false>();
  return sph ? occupancy_of<T, P, false, true>() : occupancy_of<T, P, false, false>();
}
}  // namespace

int persistent_blocks_per_cu(int ppt, int grid_f64, int reflect, int sph) {
  if (grid_f64)
    return ppt == 1 ? occupancy_rs<double, 1>(reflect, sph) : occupancy_rs<double, 2>(reflect, sph);
  return ppt == 1 ? occupancy_rs<float, 1>(reflect, sph) : occupancy_rs<float, 2>(reflect, sph);
}

hipError_t launch_fill_zero(hipStream_t s, void *p, size_t bytes) {
  if (bytes == 0) return hipSuccess;
  const size_t words = (bytes + 3) / 4;
  unsigned blocks = (unsigned)((words + kBlock - 1) / kBlock);
  if (blocks > 4096) blocks = 4096;
  k_fill_zero<<<blocks, kBlock, 0, s>>>((uint32_t *)p, words);
  return hipGetLastError();
}

hipError_t launch_valu_probe(hipStream_t s, int kind, int64_t waves, int iters, float *out) {
  const unsigned blocks = (unsigned)((waves * 64 + 255) / 256);
  if (kind == 0) k_valu_probe<0><<<blocks, 256, 0, s>>>(iters, out);
  else if (kind == 1) k_valu_probe<1><<<blocks, 256, 0, s>>>(iters, out);
  else if (kind == 2) k_valu_probe<2><<<blocks, 256, 0, s>>>(iters, out);
  else k_valu_probe<3><<<blocks, 256, 0, s>>>(iters, out);
  return hipGetLastError();
}

hipError_t launch_copy(hipStream_t s, void *dst, const void *src, size_t bytes) {
  if (bytes == 0) return hipSuccess;
  if ((bytes % 16) == 0 && ((uintptr_t)dst % 16) == 0 && ((uintptr_t)src % 16) == 0) {
    const size_t n16 = bytes / 16;
    unsigned blocks = (unsigned)((n16 + kBlock - 1) / kBlock);
    if (blocks > 8192) blocks = 8192;
    k_copy16<<<blocks, kBlock, 0, s>>>((float4 *)dst, (const float4 *)src, n16);
  } else {
    k_copy1<<<grid_for((int64_t)bytes), kBlock, 0, s>>>((uint8_t *)dst, (const uint8_t *)src,
                                                       bytes);
  }
  return hipGetLastError();
}

}  // namespace dpd
