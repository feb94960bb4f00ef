// Adjoint of the DPD step: vector-Jacobian products of the pair force
// (Eq. 3-10), the Groot-Warren update and the phase-field bounce-back
// (Eq. 16-17) with the bounce-back events held at their recorded values,
// plus the window observable (mean v_x per bin) and its adjoint seed.
//
// Notation of one step t (fluid particle i, h = dt/2):
//   w = v + h f,  r* = r + dt w,  vt = v + lambda dt f
//   event 0: r' = r*                      v' = w + h f'
//   event 1: r' = r* - 2 s dt v, s(phi(r*), phi(r))   vt = -v, v' = -v
//   event 2: r' = r                                   vt = -v, v' = -v
//   f'_i = sum_j F_ij(r'_i - r'_j, vt_i - vt_j) + g
// The backward sweep of step t takes the adjoints of (r', v', f') in the
// slot order of step t + 1 and returns the adjoints of (r, v, f) in the
// order of step t, which is the slot order of step t - 1.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"

namespace dpd {
namespace {

constexpr int kBlockA = 256;
constexpr int kListCapA = 24;
constexpr int kBatchA = 4;

inline unsigned grid_a(int64_t n) { return (unsigned)((n + kBlockA - 1) / kBlockA); }

// Profile bin in decision form: clamp(floor(fl(x * scale)), 0, nbins - 1).
__device__ __forceinline__ int bin_of(float x, float scale, int nbins) {
#pragma clang fp contract(off)
  const float g = floorf(x * scale);
  return g >= 0.0f ? (g > (float)(nbins - 1) ? nbins - 1 : (int)g) : 0;
}

// Coordinate `axis` of a position held in registers.  The argument is a
// value on purpose: selecting through a reference to global memory lets the
// compiler turn the choice into a choice of load address, which the gfx950
// backend lowers incorrectly for the z case (a load through an address
// register that the z path never writes).
__device__ __forceinline__ float axis_of(const float4 x, int axis) {
  return axis == 0 ? x.x : (axis == 1 ? x.y : x.z);
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// Block sum of three values added to slot[0..2] by thread 0 (a fixed
// summation order: the partial of a block is the same in every run).  Every
// thread of the block must call it.
template <int BS>
__device__ __forceinline__ void block_add3(double a, double b, double c, double *slot) {
  __shared__ double red[3][BS / 64];
  a = wave_sum(a);
  b = wave_sum(b);
  c = wave_sum(c);
  const int lane = (int)__lane_id(), wv = (int)threadIdx.x >> 6;
  if (lane == 0) {
    red[0][wv] = a;
    red[1][wv] = b;
    red[2][wv] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int q = 0; q < BS / 64; ++q) {
      s0 += red[0][q];
      s1 += red[1][q];
      s2 += red[2][q];
    }
    slot[0] += s0;
    slot[1] += s1;
    slot[2] += s2;
  }
}

// ---------------------------------------------------------------------------
// Window observable
// ---------------------------------------------------------------------------
// The states of a window, `per` entries of (state, particle) per block: the
// blocks' bins meet in global memory once per block, so few blocks with many
// entries each.
__global__ __launch_bounds__(kBlockA) void k_obs(int64_t nf, int64_t total, int64_t per,
                                                 int64_t stride, const float4 *__restrict__ pos4,
                                                 const float4 *__restrict__ vel4, int axis,
                                                 int nbins, float scale, double *sums,
                                                 unsigned long long *counts) {
  __shared__ double s_sum[kMaxBins];
  __shared__ unsigned s_cnt[kMaxBins];
  for (int b = threadIdx.x; b < nbins; b += blockDim.x) {
    s_sum[b] = 0.0;
    s_cnt[b] = 0u;
  }
  __syncthreads();
  const int64_t first = (int64_t)blockIdx.x * per, last = min(total, first + per);
  int64_t at = first + threadIdx.x, state = at / nf, p = at - state * nf;
  for (; at < last; at += kBlockA, p += kBlockA) {
    while (p >= nf) {
      p -= nf;
      ++state;
    }
    const float4 x = pos4[state * stride + p];
    const int b = bin_of(axis_of(x, axis), scale, nbins);
    atomicAdd(&s_sum[b], (double)vel4[state * stride + p].x);
    atomicAdd(&s_cnt[b], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nbins; b += blockDim.x) {
    if (s_cnt[b]) {
      atomicAdd(&sums[b], s_sum[b]);
      atomicAdd(&counts[b], (unsigned long long)s_cnt[b]);
    }
  }
}

__global__ __launch_bounds__(kBlockA) void k_store_walls(int64_t nrec, int nsteps, int64_t stride,
                                                         const float4 *__restrict__ pos,
                                                         const float4 *__restrict__ vt,
                                                         float4 *pos_out, float4 *vt_out,
                                                         int64_t run_stride, int32_t *slack,
                                                         int32_t pad) {
  const int64_t w = (int64_t)blockIdx.x * kBlockA + threadIdx.x;
  float4 x, v;
  if (w < nrec) {
    x = pos[w];
    v = vt[w];
  }
  for (int64_t t = blockIdx.y; t < nsteps; t += gridDim.y) {
    if (w < kIdxSlack) slack[t * run_stride + w] = pad;
    if (w < nrec) {
      pos_out[t * stride + w] = x;
      vt_out[t * stride + w] = v;
    }
  }
}

__global__ void k_obs_final(int nbins, const double *__restrict__ sums,
                            const unsigned long long *__restrict__ counts, double *profile,
                            int64_t *counts_out) {
  const int b = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (b >= nbins) return;
  const unsigned long long c = counts[b];
  if (profile) profile[b] = c ? sums[b] / (double)c : 0.0;
  if (counts_out) counts_out[b] = (int64_t)c;
}

// Adjoint seed: d(mean v_x in bin b)/d(v_x of a term in b) = 1 / N_b.
__global__ void k_loss_weights(int nbins, const double *__restrict__ dldp,
                               const unsigned long long *__restrict__ counts, float *lw) {
  const int b = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (b >= nbins) return;
  const unsigned long long c = counts[b];
  lw[b] = c ? (float)(dldp[b] / (double)c) : 0.0f;
}

__global__ void k_vt_from_v(int64_t nf, const float4 *__restrict__ vel4, float4 *vt4) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nf) return;
  const float4 v = vel4[p];
  vt4[p] = make_float4(v.x, v.y, v.z, __int_as_float(0));
}

__global__ void k_set_u64(unsigned long long *p, unsigned long long v) { *p = v; }

// ---------------------------------------------------------------------------
// Step seed: the adjoint of f' (with the loss term of v' added) moved from
// the slot order of step t + 1 to the order of step t.  In a window kept whole the
// integrator's VJP of step t + 1 does it (k_integrate_vjp with NEXT).
//   Fbar_i = fbar'_i + h vbar'_i   (event 0: v' = w + h f')
//   Fbar_i = fbar'_i               (events 1, 2: v' = -v)
// initial = 1: the refreshed starting force f0 = F(r0, v0) + g, whose
// adjoint is already in index order (no permutation, no loss term).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void prep_one(const KParams &P, const AdjPrep &N, int64_t s, float4 rb,
                                         float4 vb, float4 &F) {
  const int i = N.idx[s];
  const int ev = __float_as_int(N.vt4[i].w);
  const float4 xi = N.pos4[i];
  vb.x += N.lw[bin_of(axis_of(xi, N.axis), N.scale, N.nbins)];
  if (ev == 0) {
    F.x += P.hdt * vb.x;
    F.y += P.hdt * vb.y;
    F.z += P.hdt * vb.z;
  }
  N.fbar[i] = F;
  N.rn[i] = rb;
  N.vn[i] = vb;
}

__global__ __launch_bounds__(kBlockA) void k_adj_prep(
    const Box *__restrict__ boxes, int64_t nf, int initial, const float4 *__restrict__ rb_s,
    const float4 *__restrict__ vb_s, const float4 *__restrict__ fb_s, const AdjPrep N) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  float4 F = make_float4(0.f, 0.f, 0.f, 0.f);
  if (s < nf) {
    F = fb_s[s];
    if (initial)
      N.fbar[s] = F;
    else
      prep_one(boxes[0].P, N, s, rb_s[s], vb_s[s], F);
  }
  block_add3<kBlockA>(F.x, F.y, F.z, N.part_g + 3 * (size_t)blockIdx.x);
}

// ---------------------------------------------------------------------------
// Pair-force VJP.  With d = r_i - r_j, r = |d|, e = d / r, w = 1 - r/rc,
// u = e . (vt_i - vt_j), s = sigma xi / sqrt(dt) and
// F_ij = c e, c = w (a - gamma w u + s), the adjoint mu_ij = Fbar_i - Fbar_j
// (Fbar_j = 0 for a wall: its force is never used) gives
//   rbar_i  += (dc/dd) (e . mu) + c (mu - e (e . mu)) / r
//              dc/dd = -(a - 2 gamma w u + s) e / rc - gamma w^2 (dv - u e) / r
//   vtbar_i += -gamma w^2 e (e . mu)
// gathered per particle over its full neighbour shell (F_ji = -F_ij, and the
// Jacobian is even in d, so both terms of a pair land on i this way), and
// the parameter terms of f_i, with eF = e . Fbar_i:
//   abar    += w eF            (a_ff for a fluid j, a_fw for a wall)
//   gammabar += (-w^2 u + w xi dsigma/dgamma / sqrt(dt)) eF
// Pairs are found with the force kernel's decision at the same positions,
// so the set is the forward's.
// ---------------------------------------------------------------------------
struct VjpSums {
  float rx, ry, rz;           // rbar_i
  float vx, vy, vz;           // vtbar_i
  double aff, afw, gam;       // parameter terms
};

__device__ __forceinline__ void vjp_pair(VjpSums &S, const KGeom &G, const KParams &P,
                                         const float4 &pi, const float4 &vti, const float4 &Fi,
                                         const float4 &pj, const float4 &vtj, const float4 &Fj,
                                         bool fluid_j, uint32_t klo, uint32_t khi) {
  const float dx = sep(pi.x, pj.x, G.L[0]);
  const float dy = sep(pi.y, pj.y, G.L[1]);
  const float dz = sep(pi.z, pj.z, G.L[2]);
  const float r2 = dx * dx + dy * dy + dz * dz;
  const float rinv = rsqrtf(r2);
  const float r = r2 * rinv;
  const float w = 1.0f - r * P.inv_rc;
  if (!(w > 0.0f)) return;   // the forward's force is zero there
  const float ex = dx * rinv, ey = dy * rinv, ez = dz * rinv;
  const float dvx = vti.x - vtj.x, dvy = vti.y - vtj.y, dvz = vti.z - vtj.z;
  const float u = ex * dvx + ey * dvy + ez * dvz;
  const float xi = pair_gauss(__float_as_uint(pi.w), __float_as_uint(pj.w), klo, khi, P.key0,
                              P.key1);
  const float sr = P.sigma_rdt * xi;
  const float a = fluid_j ? P.a_ff : P.a_fw;
  const float c = w * (a - P.gamma * w * u + sr);
  const float mx = Fi.x - Fj.x, my = Fi.y - Fj.y, mz = Fi.z - Fj.z;
  const float em = ex * mx + ey * my + ez * mz;
  const float gw = -(a - 2.0f * P.gamma * w * u + sr) * P.inv_rc * em;
  const float gwu = -P.gamma * w * w;
  const float gu = gwu * rinv * em;
  const float cr = c * rinv;
  S.rx += gw * ex + gu * (dvx - u * ex) + cr * (mx - ex * em);
  S.ry += gw * ey + gu * (dvy - u * ey) + cr * (my - ey * em);
  S.rz += gw * ez + gu * (dvz - u * ez) + cr * (mz - ez * em);
  S.vx += gwu * em * ex;
  S.vy += gwu * em * ey;
  S.vz += gwu * em * ez;
  const float eF = ex * Fi.x + ey * Fi.y + ez * Fi.z;
  if (fluid_j)
    S.aff += (double)(w * eF);
  else
    S.afw += (double)(w * eF);
  S.gam += (double)((-w * w * u + P.dsig_rdt * w * xi) * eF);
}

template <int BS>
__global__ __launch_bounds__(BS) void k_force_vjp(
    const Box *__restrict__ boxes, const Tile *__restrict__ tiles, int ntiles, int64_t NF,
    int32_t pad, const float4 *__restrict__ pos4, const float4 *__restrict__ vt4,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ idx_all,
    const int32_t *__restrict__ start_all, const float4 *__restrict__ fbar,
    const float4 *__restrict__ rn, float4 *__restrict__ rt_out, float4 *__restrict__ vt_out,
    const unsigned long long *__restrict__ dk0, unsigned long long koff, double *part) {
  __shared__ uint32_t list[kListCapA * BS];
  const int tid = xcd_block();
  bool act = tid < ntiles;
  Tile tile{0, 0, 0, 0};
  if (act) {
    tile = tiles[tid];
    act = (int)threadIdx.x < tile.count;
  }
  VjpSums S = {};
  if (act) {
    const Box &B = boxes[tile.box];
    const KGeom G = B.G;
    const KParams P = B.P;
    const int co = (int)B.co;
    const unsigned long long kk = *dk0 + koff;
    const uint32_t klo = (uint32_t)kk;
    const uint32_t khi = ((uint32_t)(kk >> 32) & 0xFFFFu) | (P.replica << 16);
    const int64_t s = (int64_t)tile.first + threadIdx.x;
    const int i = idx[s];
    const float4 pi = pos4[i];
    const float4 vti = vt4[i];
    const float4 Fi = fbar[i];
    const uint32_t gi = __float_as_uint(pi.w);
    int cx, cy, cz;
    cell_index(G, pi.x, pi.y, pi.z, cx, cy, cz);
    uint32_t *mine = list + threadIdx.x;
    NeighbourRows rows;
    rows.init(cx, cy, cz);
    int t = 0, t_end = 0;
    SepAxis ax = sep_axis(pi.x, 0.f), ay = sep_axis(pi.y, 0.f), az = sep_axis(pi.z, 0.f);
    bool done = false;
    while (!done) {
      int cnt = 0;
      while (cnt <= kListCapA - kBatchA) {
        if (t >= t_end) {
          float sx, sy, sz;
          if (!rows.next(G, start_all, co, t, t_end, sx, sy, sz)) {
            done = true;
            break;
          }
          ax = sep_axis(pi.x, sx);
          ay = sep_axis(pi.y, sy);
          az = sep_axis(pi.z, sz);
          continue;
        }
        int jb[kBatchA];
#pragma unroll
        for (int u = 0; u < kBatchA; ++u) jb[u] = t + u < t_end ? idx_all[t + u] : pad;
        float4 pb[kBatchA];
#pragma unroll
        for (int u = 0; u < kBatchA; ++u) pb[u] = pos4[jb[u]];
#pragma unroll
        for (int u = 0; u < kBatchA; ++u) {
          const float r2 = pair_r2(sep_d(ax, pb[u].x), sep_d(ay, pb[u].y), sep_d(az, pb[u].z));
          if (r2 < P.rc2 && r2 > 0.0f) {
            mine[cnt * BS] = (uint32_t)jb[u];
            ++cnt;
          }
        }
        t += kBatchA;
      }
      for (int q = 0; q < cnt; ++q) {
        const uint32_t j = mine[q * BS];
        const float4 pj = pos4[j];
        const float4 vtj = vt4[j];
        const bool fluid_j = (int64_t)j < NF;
        const float4 Fj = fluid_j ? fbar[j] : make_float4(0.f, 0.f, 0.f, 0.f);
        vjp_pair(S, G, P, pi, vti, Fi, pj, vtj, Fj, fluid_j, klo, khi);
      }
    }
    if (rn) {
      const float4 b = rn[i];
      S.rx += b.x;
      S.ry += b.y;
      S.rz += b.z;
    }
    rt_out[i] = make_float4(S.rx, S.ry, S.rz, 0.f);
    vt_out[i] = make_float4(S.vx, S.vy, S.vz, 0.f);
  }
  block_add3<BS>(S.aff, S.afw, S.gam, part + 3 * (size_t)tid);
}

// The same with 16 lanes per particle, for small contexts (see WideRows): the
// lanes sum every sixteenth pair and their sums meet in a fixed order at the end.
// One lane per particle took 54 us for 15,000 particles, 12 us of it arithmetic.
__global__ __launch_bounds__(kBlockA) void k_force_vjp_wide(
    const Box *__restrict__ boxes, const Tile *__restrict__ tiles, int ntiles, int64_t NF,
    const float4 *__restrict__ pos4, const float4 *__restrict__ vt4,
    const int32_t *__restrict__ idx, const int32_t *__restrict__ idx_all,
    const int32_t *__restrict__ start_all, const float4 *__restrict__ fbar,
    const float4 *__restrict__ rn, float4 *__restrict__ rt_out, float4 *__restrict__ vt_out,
    const unsigned long long *__restrict__ dk0, unsigned long long koff, double *part) {
  __shared__ int ring[kWideParts][kWideRing + 8];
  __shared__ int4 rows_lds[kWideParts][9];
  const int tid = xcd_block();
  const int grp = (int)threadIdx.x / kWideLanes, g = (int)threadIdx.x % kWideLanes;
  bool act = tid < ntiles;
  Tile tile{0, 0, 0, 0};
  if (act) {
    tile = tiles[tid];
    act = grp < tile.count;   // whole groups
  }
  VjpSums S = {};
  if (act) {
    const Box &B = boxes[tile.box];
    const KGeom G = B.G;
    const KParams P = B.P;
    const unsigned long long kk = *dk0 + koff;
    const uint32_t klo = (uint32_t)kk;
    const uint32_t khi = ((uint32_t)(kk >> 32) & 0xFFFFu) | (P.replica << 16);
    const int i = idx[(int64_t)tile.first + grp];
    const float4 pi = pos4[i], vti = vt4[i], Fi = fbar[i];
    int cx, cy, cz;
    cell_index(G, pi.x, pi.y, pi.z, cx, cy, cz);
    WideRows rows;
    rows.init(G, (int)B.co, cx, cy, cz, g, start_all, rows_lds[grp]);
    int *const list = ring[grp];
    const int shift = ((int)__lane_id() / kWideLanes) * kWideLanes;
    int listed = 0, done = 0;
    auto evaluate = [&]() {
      const int e = done + g;
      if (e < listed) {
        const int j = list[e & (kWideRing - 1)];
        const bool fluid_j = (int64_t)j < NF;
        const float4 pj = pos4[j], vtj = vt4[j];
        const float4 Fj = fluid_j ? fbar[j] : make_float4(0.f, 0.f, 0.f, 0.f);
        vjp_pair(S, G, P, pi, vti, Fi, pj, vtj, Fj, fluid_j, klo, khi);
      }
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
        const bool hit = r2 < P.rc2 && r2 > 0.0f && c0 + k * kWideLanes + g < rows.total;
        const uint32_t m = (uint32_t)(__ballot(hit) >> shift) & 0xFFFFu;
        if (hit) list[(listed + __popc(m & ((1u << g) - 1u))) & (kWideRing - 1)] = j[k];
        listed += __popc(m);
      }
      wave_lds_sync();
      while (listed - done >= kWideLanes) evaluate();
      wave_lds_sync();
    }
    if (done < listed) evaluate();
#pragma unroll
    for (int d = kWideLanes / 2; d > 0; d >>= 1) {
      S.rx += __shfl_xor(S.rx, d, kWideLanes);
      S.ry += __shfl_xor(S.ry, d, kWideLanes);
      S.rz += __shfl_xor(S.rz, d, kWideLanes);
      S.vx += __shfl_xor(S.vx, d, kWideLanes);
      S.vy += __shfl_xor(S.vy, d, kWideLanes);
      S.vz += __shfl_xor(S.vz, d, kWideLanes);
    }
    if (g == 0) {
      const float4 b = rn ? rn[i] : make_float4(0.f, 0.f, 0.f, 0.f);
      rt_out[i] = make_float4(S.rx + b.x, S.ry + b.y, S.rz + b.z, 0.f);
      vt_out[i] = make_float4(S.vx, S.vy, S.vz, 0.f);
    }
  }
  block_add3<kBlockA>(S.aff, S.afw, S.gam, part + 3 * (size_t)tid);
}

// Gradient of the trilinear interpolant at a located point (per unit
// length), and bar * (corner weight) added to each of the 8 corner nodes.
template <typename T>
__device__ __forceinline__ void phi_grad_scatter(const T *__restrict__ grid, const KGeom &G,
                                                 const GridLoc<T> &L, T bar, double *dphi,
                                                 T g[3]) {
  const size_t nx = (size_t)G.ng[0], nxy = nx * (size_t)G.ng[1];
  T gx = 0, gy = 0, gz = 0;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const T wz = c ? L.t[2] : (T)1 - L.t[2], dwz = c ? (T)1 : (T)-1;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const T wy = b ? L.t[1] : (T)1 - L.t[1], dwy = b ? (T)1 : (T)-1;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const T wx = a ? L.t[0] : (T)1 - L.t[0], dwx = a ? (T)1 : (T)-1;
        const size_t node = (size_t)(c ? L.i1[2] : L.i0[2]) * nxy +
                            (size_t)(b ? L.i1[1] : L.i0[1]) * nx + (size_t)(a ? L.i1[0] : L.i0[0]);
        const T p = grid[node];
        gx += p * dwx * wy * wz;
        gy += p * wx * dwy * wz;
        gz += p * wx * wy * dwz;
        if (dphi && bar != (T)0) atomicAdd(&dphi[node], (double)(bar * wx * wy * wz));
      }
    }
  }
  g[0] = gx * GridScale<T>::inv_h(G, 0);
  g[1] = gy * GridScale<T>::inv_h(G, 1);
  g[2] = gz * GridScale<T>::inv_h(G, 2);
}

// ---------------------------------------------------------------------------
// Integrate + bounce-back VJP with the step's events held fixed: from the
// adjoints of r' (rt, pair part included), of vt (vtb) and of v' (vn, loss
// term included) to those of (r, v, f) of step t.  Event 1 differentiates
// Eq. 17's s = c1 / (c0 + c1), c1 = atanh(-phi(r*)), c0 = atanh(phi(r)),
// through the interpolated phi at both points (gradient and node values).
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void integrate_vjp_one(
    const Box &B, int64_t i, const float4 *__restrict__ pos_t, const float4 *__restrict__ vel_t,
    const float4 *__restrict__ frc_t, const float4 *__restrict__ vt4,
    const float4 *__restrict__ rt, const float4 *__restrict__ vtb, const float4 *__restrict__ vn,
    const T *__restrict__ grid_base, double *dphi_base, float rb[3], float vb[3], float fb[3]) {
  const KGeom G = B.G;
  const KParams P = B.P;
  const int ev = __float_as_int(vt4[i].w);
  const float4 R = rt[i], V = vtb[i], W = vn[i];
  if (ev == 0) {
    const float wb[3] = {P.dt * R.x + W.x, P.dt * R.y + W.y, P.dt * R.z + W.z};
    const float vv[3] = {V.x, V.y, V.z};
    const float rr[3] = {R.x, R.y, R.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      rb[a] = rr[a];
      vb[a] = wb[a] + vv[a];
      fb[a] = P.hdt * wb[a] + P.lamdt * vv[a];
    }
  } else if (ev == 2) {
    rb[0] = R.x;
    rb[1] = R.y;
    rb[2] = R.z;
    vb[0] = -V.x - W.x;
    vb[1] = -V.y - W.y;
    vb[2] = -V.z - W.z;
    fb[0] = fb[1] = fb[2] = 0.f;
  } else {
    const T *grid = grid_base + B.go;
    double *dphi = dphi_base ? dphi_base + B.go : nullptr;
    const float4 x = pos_t[i], v = vel_t[i], f = frc_t[i];
    const float xs = drift1(x.x, v.x, f.x, P.hdt, P.dt, G.L[0]);
    const float ys = drift1(x.y, v.y, f.y, P.hdt, P.dt, G.L[1]);
    const float zs = drift1(x.z, v.z, f.z, P.hdt, P.dt, G.L[2]);
    const GridLoc<T> ls = grid_locate<T>(G, xs, ys, zs);
    const GridLoc<T> lt = grid_locate<T>(G, x.x, x.y, x.z);
    const T phis = phi_interp(grid, G, ls);
    const T phit = phi_interp(grid, G, lt);
    const T lim = (T)1 - (T)0x1p-20;
    const T a1 = fmin(fmax(-phis, (T)0), lim);
    const T a0 = fmin(fmax(phit, (T)0), lim);
    const T c1 = atanh(a1), c0 = atanh(a0);
    const T sfrac = c1 > (T)0 ? c1 / (c0 + c1) : (T)0;
    const float rr[3] = {R.x, R.y, R.z};
    const float vv[3] = {v.x, v.y, v.z};
    // r' = r* - 2 s dt v
    const T sbar = (T)(-2.0f * P.dt) * (T)(vv[0] * rr[0] + vv[1] * rr[1] + vv[2] * rr[2]);
    const float k2 = (float)((T)2 * sfrac * (T)P.dt);
    float rsb[3] = {rr[0], rr[1], rr[2]};
    float rtb[3] = {0.f, 0.f, 0.f};
    if (c1 > (T)0) {
      const T den = c0 + c1;
      const T ds1 = c0 / (den * den), ds0 = -c1 / (den * den);
      const T dp1 = (-phis > (T)0 && -phis < lim) ? (T)-1 / ((T)1 - a1 * a1) : (T)0;
      const T dp0 = (phit > (T)0 && phit < lim) ? (T)1 / ((T)1 - a0 * a0) : (T)0;
      const T pbs = sbar * ds1 * dp1, pbt = sbar * ds0 * dp0;
      T gs[3], gt[3];
      phi_grad_scatter<T>(grid, G, ls, pbs, dphi, gs);
      phi_grad_scatter<T>(grid, G, lt, pbt, dphi, gt);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        rsb[a] += (float)(pbs * gs[a]);
        rtb[a] = (float)(pbt * gt[a]);
      }
    }
    const float vtv[3] = {V.x, V.y, V.z}, vnv[3] = {W.x, W.y, W.z};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      // r* = r + dt w, w = v + h f; vt = -v; v' = -v
      const float wb = P.dt * rsb[a];
      rb[a] = rsb[a] + rtb[a];
      vb[a] = -k2 * rr[a] + wb - vtv[a] - vnv[a];
      fb[a] = P.hdt * wb;
    }
  }
}

// NEXT: the particle goes on to the step before (prep_one of its slot) instead of leaving
// its adjoints; vn and next.vn differ then.  One launch less per step: a window of 24
// steps of 16,000 particles and its backward sweep 1,620 to 1,480 us.
template <typename T, bool NEXT>
__global__ __launch_bounds__(kBlockA) void k_integrate_vjp(
    const Box *__restrict__ boxes, int64_t nf, const float4 *__restrict__ pos_t,
    const float4 *__restrict__ vel_t, const float4 *__restrict__ frc_t,
    const float4 *__restrict__ vt4, const float4 *__restrict__ rt,
    const float4 *__restrict__ vtb, const float4 *__restrict__ vn, const T *__restrict__ grid_base,
    double *dphi_base, float4 *__restrict__ rb_out, float4 *__restrict__ vb_out,
    float4 *__restrict__ fb_out, const AdjPrep next) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  float rb[3], vb[3], fb[3] = {0.f, 0.f, 0.f};
  if (i < nf) {
    integrate_vjp_one<T>(boxes[0], i, pos_t, vel_t, frc_t, vt4, rt, vtb, vn, grid_base, dphi_base,
                         rb, vb, fb);
    const float4 R = make_float4(rb[0], rb[1], rb[2], 0.f);
    const float4 V = make_float4(vb[0], vb[1], vb[2], 0.f);
    float4 F = make_float4(fb[0], fb[1], fb[2], 0.f);
    if (NEXT) {
      prep_one(boxes[0].P, next, i, R, V, F);
      fb[0] = F.x;
      fb[1] = F.y;
      fb[2] = F.z;
    } else {
      rb_out[i] = R;
      vb_out[i] = V;
      fb_out[i] = F;
    }
  }
  if (NEXT) block_add3<kBlockA>(fb[0], fb[1], fb[2], next.part_g + 3 * (size_t)blockIdx.x);
}

// Fixed-order final sums of the per-block partials:
// out = {a_ff, a_fw, gamma} from the pair VJP and {g_x, g_y, g_z}.
// (one wavefront per sum, each lane every 64th block)
__global__ __launch_bounds__(6 * 64) void k_reduce_partials(int nb_f,
                                                            const double *__restrict__ part_f,
                                                            int nb_g,
                                                            const double *__restrict__ part_g,
                                                            double *out) {
  const int k = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
  const double *p = k < 3 ? part_f + k : part_g + (k - 3);
  const int nb = k < 3 ? nb_f : nb_g;
  double s = 0.0;
  for (int b = lane; b < nb; b += 64) s += p[3 * (size_t)b];
  s = wave_sum(s);
  if (lane == 0) out[k] = s;
}

}  // namespace

hipError_t launch_obs(hipStream_t s, int64_t nf, int nstates, int64_t stride, const float4 *pos4,
                      const float4 *vel4, int axis, int nbins, float scale, double *sums,
                      unsigned long long *counts) {
  if (nf <= 0 || nstates <= 0) return hipSuccess;
  // a block per 1,024 entries, at most 512 blocks
  const int64_t total = nf * nstates;
  const int64_t nb = std::min<int64_t>(512, (total + 1023) / 1024);
  k_obs<<<(unsigned)nb, kBlockA, 0, s>>>(nf, total, (total + nb - 1) / nb, stride, pos4, vel4,
                                         axis, nbins, scale, sums, counts);
  return hipGetLastError();
}

hipError_t launch_store_walls(hipStream_t s, int64_t nrec, int nsteps, int64_t stride,
                              const float4 *pos, const float4 *vt, float4 *pos_out,
                              float4 *vt_out, int64_t run_stride, int32_t *slack, int32_t pad) {
  if (nsteps <= 0) return hipSuccess;
  const dim3 grid(grid_a(std::max<int64_t>(nrec, kIdxSlack)), (unsigned)std::min(nsteps, 64));
  k_store_walls<<<grid, kBlockA, 0, s>>>(nrec, nsteps, stride, pos, vt, pos_out, vt_out, run_stride,
                                         slack, pad);
  return hipGetLastError();
}

hipError_t launch_obs_final(hipStream_t s, int nbins, const double *sums,
                            const unsigned long long *counts, double *profile,
                            int64_t *counts_out) {
  k_obs_final<<<(nbins + 255) / 256, 256, 0, s>>>(nbins, sums, counts, profile, counts_out);
  return hipGetLastError();
}

hipError_t launch_loss_weights(hipStream_t s, int nbins, const double *dldp,
                               const unsigned long long *counts, float *lw) {
  k_loss_weights<<<(nbins + 255) / 256, 256, 0, s>>>(nbins, dldp, counts, lw);
  return hipGetLastError();
}

hipError_t launch_vt_from_v(hipStream_t s, int64_t nf, const float4 *vel4, float4 *vt4) {
  if (nf <= 0) return hipSuccess;
  k_vt_from_v<<<grid_a(nf), kBlockA, 0, s>>>(nf, vel4, vt4);
  return hipGetLastError();
}

hipError_t launch_set_u64(hipStream_t s, unsigned long long *p, unsigned long long v) {
  k_set_u64<<<1, 1, 0, s>>>(p, v);
  return hipGetLastError();
}

int adj_prep_blocks(int64_t nf) { return nf > 0 ? (int)grid_a(nf) : 0; }

hipError_t launch_adj_prep(hipStream_t s, const Box *boxes, int64_t nf, int initial,
                           const float4 *rb_s, const float4 *vb_s, const float4 *fb_s,
                           const AdjPrep &N) {
  if (nf <= 0) return hipSuccess;
  k_adj_prep<<<grid_a(nf), kBlockA, 0, s>>>(boxes, nf, initial, rb_s, vb_s, fb_s, N);
  return hipGetLastError();
}

int force_vjp_blocks(int ntiles) { return ((ntiles + 7) / 8) * 8; }

hipError_t launch_force_vjp(hipStream_t s, int block, const Box *boxes, const Tile *tiles,
                            int ntiles, int64_t NF, int32_t pad, const float4 *pos4,
                            const float4 *vt4, const int32_t *idx, const int32_t *idx_all,
                            const int32_t *start_all, const float4 *fbar, const float4 *rn,
                            float4 *rt_out, float4 *vt_out, const unsigned long long *dk0,
                            unsigned long long koff, double *part) {
  if (ntiles <= 0) return hipSuccess;
  const unsigned nb = (unsigned)force_vjp_blocks(ntiles);
  if (block == 0)
    k_force_vjp_wide<<<nb, kBlockA, 0, s>>>(boxes, tiles, ntiles, NF, pos4, vt4, idx, idx_all,
                                            start_all, fbar, rn, rt_out, vt_out, dk0, koff, part);
  else if (block == 128)
    k_force_vjp<128><<<nb, 128, 0, s>>>(boxes, tiles, ntiles, NF, pad, pos4, vt4, idx, idx_all,
                                        start_all, fbar, rn, rt_out, vt_out, dk0, koff, part);
  else
    k_force_vjp<256><<<nb, 256, 0, s>>>(boxes, tiles, ntiles, NF, pad, pos4, vt4, idx, idx_all,
                                        start_all, fbar, rn, rt_out, vt_out, dk0, koff, part);
  return hipGetLastError();
}

hipError_t launch_integrate_vjp(hipStream_t s, const Box *boxes, int64_t nf, const float4 *pos_t,
                                const float4 *vel_t, const float4 *frc_t, const float4 *vt4,
                                const float4 *rt, const float4 *vtb, const float4 *vn,
                                const void *grid, int grid_f64, double *dphi, float4 *rb_out,
                                float4 *vb_out, float4 *fb_out, const AdjPrep *next) {
  if (nf <= 0) return hipSuccess;
  const AdjPrep N = next ? *next : AdjPrep{};
#define DPD_IVJP(T, NEXT)                                                                        \
  k_integrate_vjp<T, NEXT><<<grid_a(nf), kBlockA, 0, s>>>(boxes, nf, pos_t, vel_t, frc_t, vt4, rt, \
                                                          vtb, vn, (const T *)grid, dphi, rb_out, \
                                                          vb_out, fb_out, N)
  if (grid_f64) {
    if (next) DPD_IVJP(double, true); else DPD_IVJP(double, false);
  } else {
    if (next) DPD_IVJP(float, true); else DPD_IVJP(float, false);
  }
#undef DPD_IVJP
  return hipGetLastError();
}

hipError_t launch_reduce_partials(hipStream_t s, int nb_f, const double *part_f, int nb_g,
                                  const double *part_g, double *out) {
  k_reduce_partials<<<1, 6 * 64, 0, s>>>(nb_f, part_f, nb_g, part_g, out);
  return hipGetLastError();
}

}  // namespace dpd
