// The kernels of density_gradient_on_grid: the density and its gradient from
// one real coefficient part C on the stored pairs (a scalar density matrix of
// one component: the forward density update of Eq. 39 with the gradient a
// GGA needs).  Per batch with functions phi_1..phi_n at its points,
//   n = sum over stored elements C_ij phi_i phi_j = phi^T M phi,
//   grad n = 2 grad phi^T M phi,
// with M the symmetric n x n matrix of the batch (half of each stored
// off-diagonal element on both sides, the symmetric part of a self pair's
// block).  So per batch one product Y = M Phi (2 P n^2 flops, on FP64 MFMA)
// and lane-local dot products of Y with phi and grad phi.
//   k_grad_cdense  M of every batch of a pass, dense (np x np, zero padding);
//   k_grad_gemm    one wave per (batch, point chunk, function chunk i) of at
//                  most 64 x 64: Y_i(pt) = sum_j phi_j(pt) M_ji, then n and
//                  grad n partials over its functions;
//   k_grad_points  the partials of a point over the function chunks, in order.
// (Gathering the M slices from the store inside the product instead of
// materialising M was slower: two dependent memory round trips per 16
// functions do not hide behind 16 MFMAs.)
// The panel tabulation and the launches around these are in q4c_kernels.hip.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "q4c_internal.h"
#include "q4c_device.h"

namespace q4c {
namespace {

constexpr int GT = 64;  // most points and functions of an item


// packed slot data of a batch function: slot, the slot's first function and
// its function count
__device__ __forceinline__ int fslot(int64_t v) { return (int)(v & 0xFFFFF); }
__device__ __forceinline__ int ffirst(int64_t v) { return (int)((v >> 20) & 0xFFFFF); }
__device__ __forceinline__ int fcount(int64_t v) { return (int)(v >> 40); }

constexpr int CD_T = 64;       // M tile edge
constexpr int CD_PO = 256;     // entries of the (row slot, column slot) pair-offset table of a tile in LDS

// One upper-triangle tile (rt <= ct) of M of one batch: M_rc for the tile's
// rows r and columns c, and by symmetry the mirrored tile M_cr.  Slots
// (relevant atoms) ascend with the batch's functions and with the atom
// index, so slot lo < hi is the stored pair (atom(lo), atom(hi)) with rows =
// lo's functions; above the diagonal (r < c) the row slot never exceeds the
// column slot and the store is read in its own orientation, coalesced along
// c (a self pair also takes its transposed element).  The tile goes through
// LDS so that both it and its mirror are written along rows.
__global__ __launch_bounds__(256) void k_grad_cdense(DevPlan d, const int32_t *items, int64_t it0,
                                                     const int64_t *cd_off, const int64_t *fninfo,
                                                     const double *coef, double *cd) {
  __shared__ double s_t[CD_T][CD_T + 1];
  __shared__ int64_t s_ri[CD_T], s_ci[CD_T];
  __shared__ int64_t s_po[CD_PO];
  const int64_t it = it0 + blockIdx.x;
  const int b = items[3 * it], rt = items[3 * it + 1], ct = items[3 * it + 2];
  const int f0 = d.batch_fn_off[b], n = d.batch_fn_off[b + 1] - f0, np = (int)pad16(n);
  const int sbase = d.batch_slot_off[b], ns = d.batch_slot_off[b + 1] - sbase;
  const int64_t spb = d.batch_sp_off[b];
  double *M = cd + cd_off[b];
  const int r0 = CD_T * rt, c0 = CD_T * ct;  // both below n (tiles start below np - 15)
  const int nr = min(CD_T, np - r0), nc = min(CD_T, np - c0);
  auto stored_po = [&](int rs, int cs) -> int64_t {
    const int lo = min(rs, cs), hi = max(rs, cs);
    const int q = d.sp_pair[spb + (int64_t)lo * ns - (int64_t)lo * (lo - 1) / 2 + (hi - lo)];
    return q >= 0 ? d.pair_off[q] : (int64_t)-1;
  };
  if (threadIdx.x < CD_T) s_ri[threadIdx.x] = fninfo[f0 + min(r0 + (int)threadIdx.x, n - 1)];
  else if (threadIdx.x < 2 * CD_T) s_ci[threadIdx.x - CD_T] = fninfo[f0 + min(c0 + (int)threadIdx.x - CD_T, n - 1)];
  __syncthreads();  // slot data visible
  const int rs0 = fslot(s_ri[0]), rs1 = fslot(s_ri[min(CD_T, n - r0) - 1]);
  const int cs0 = fslot(s_ci[0]), cs1 = fslot(s_ci[min(CD_T, n - c0) - 1]);
  const int nrs = rs1 - rs0 + 1, ncs = cs1 - cs0 + 1;
  const bool po_lds = nrs * ncs <= CD_PO;  // workgroup-uniform
  if (po_lds)
    for (int t = threadIdx.x; t < nrs * ncs; t += blockDim.x) s_po[t] = stored_po(rs0 + t / ncs, cs0 + t % ncs);
  __syncthreads();  // pair offsets visible
  // Lane l holds column c0 + l, wave w takes rows w, w + 4, .. of the tile, so
  // the row's data are wave-uniform and an element costs a table lookup, one
  // multiply-add and its load.  Eight rows at a time, loads unconditional
  // (element 0 of the store stands in for an absent one) and in flight
  // together; elements below the diagonal come from their mirror.
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = c0 + lane;
  const int64_t ci = s_ci[lane];
  const int cs = fslot(ci), ic = c - ffirst(ci), cn = fcount(ci);
  const bool self_tile = rs1 >= cs0;  // workgroup-uniform: some row and column of one atom
  for (int i0 = 0; i0 < CD_T / 4; i0 += 8) {
    int64_t a1[8], a2[8];
    bool live[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int rl = 4 * (i0 + u) + wave, r = r0 + rl;
      const int64_t ri = uniform_i64(s_ri[rl]);
      const int rs = fslot(ri), ir = r - ffirst(ri);
      const bool in = r < n && c < n && r <= c;
      const int64_t po = !in ? -1 : (po_lds ? s_po[(rs - rs0) * ncs + cs - cs0] : stored_po(rs, cs));
      live[u] = po >= 0;
      a1[u] = live[u] ? po + (uint32_t)(ir * cn + ic) : 0;              // rs <= cs here
      a2[u] = live[u] && rs == cs ? po + (uint32_t)(ic * cn + ir) : -1;  // the self pair's transposed element
    }
    double v1[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v1[u] = coef[a1[u]];
    if (self_tile) {
      double v2[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v2[u] = coef[a2[u] >= 0 ? a2[u] : 0];
#pragma unroll
      for (int u = 0; u < 8; ++u) v1[u] += a2[u] >= 0 ? v2[u] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int rl = 4 * (i0 + u) + wave;
      const double v = live[u] ? 0.5 * v1[u] : 0.0;
      s_t[rl][lane] = v;
      if (rl < nr && lane < nc && (rt != ct || rl <= lane)) M[(int64_t)(r0 + rl) * np + c] = v;
    }
  }
  __syncthreads();  // the tile is in LDS
  // its mirror, along rows (on the diagonal tile the part below the diagonal)
  for (int rl = wave; rl < nc; rl += 4)
    if (lane < nr && (rt != ct || rl > lane)) M[(int64_t)(c0 + rl) * np + r0 + lane] = s_t[lane][rl];
}

// One wave's item: Y = M phi for F <= 4 blocks of 16 functions and Q <= 4
// blocks of 16 points, then its products with phi, 2 d_x phi, 2 d_y phi and
// 2 d_z phi summed over the item's functions, written as 4 x 16 Q partials.
// FP64 MFMA 16x16x4 with A = M [function i][j] (M is symmetric, so its row j
// is read along i) and B = phi [j][point].  Two blocks are read at a time, 16
// bytes per lane: lane l16 holds functions (or points) 2 l16 and 2 l16 + 1 of
// the 32, one of either block, so a K step of 4 functions is at most four
// loads for 16 MFMAs, with no vector instruction beside them; an odd last
// block takes 8-byte loads.  No LDS, no barriers: operands go to registers
// three K steps ahead, and the waves of a workgroup (items of one batch) share
// them in L1 and L2.
//
// Bound: the matrix pipe 63% of the time, and L2 misses (66% of its reads): an item reads
// 512 n bytes each of M and phi per 64 x 64 outputs, and a batch's M (0.9 MB at
// n = 335) leaves an XCD's L2 between the waves that share it.  40 atoms, both
// components (155 and 335 functions per batch on average) 4.17 -> 3.29 ms
// against 64 x 64 tiles in LDS with a barrier every 16 functions; the MFMAs
// alone take 1.7 ms at their peak rate.  Chunks of at most 48 points with
// three waves per SIMD took the same time.
template <int F, int Q>
__device__ __forceinline__ void grad_item(int np, int Pp, int i0, int q0, const double *M, const double *pb,
                                          double *part) {
  constexpr int FP = F / 2, QP = Q / 2, NS = 4;  // block pairs; operand sets
  const int lane = threadIdx.x & 63, l16 = lane & 15, lk = lane >> 4;
  const int64_t plane = (int64_t)Pp * np;
  // lane offsets (bytes) of the operands: M row lk, function; quad, function lk, point of the quad
  const uint32_t am = (uint32_t)lk * np * 8u + 16u * l16, am1 = (uint32_t)lk * np * 8u + 8u * (16 * (F - 1) + l16);
  uint32_t bp[QP + 1];
#pragma unroll
  for (int q = 0; q < QP; ++q) bp[q] = ((uint32_t)(8 * q + (l16 >> 1)) * np + lk) * 32u + 16u * (l16 & 1);
  bp[QP] = ((uint32_t)(4 * (Q - 1) + (l16 >> 2)) * np + lk) * 32u + 8u * (l16 & 3);
  const double *Mi = M + i0, *pq = pb + (int64_t)q0 * np;  // q0: the item's first point (np doubles per point)
  struct Set {
    double a[F], b[Q];
  } st[NS];
  // past the last function an empty buffer: nothing is read, and no branch
  // makes the waits of the next K steps count for both of its sides
  auto load = [&](Set &s, int j) {
    const int nr = j < np ? 0x7ffffff0 : 0;
    const __amdgpu_buffer_rsrc_t ra =
        __builtin_amdgcn_make_buffer_rsrc((void *)(Mi + (int64_t)j * np), (short)0, nr, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb =
        __builtin_amdgcn_make_buffer_rsrc((void *)(pq + 4 * (int64_t)j), (short)0, nr, 0x00020000);
#pragma unroll
    for (int f = 0; f < FP; ++f) {
      const dbl2 v = __builtin_bit_cast(dbl2, __builtin_amdgcn_raw_buffer_load_b128(ra, am + 256 * f, 0, 0));
      s.a[2 * f] = v[0];
      s.a[2 * f + 1] = v[1];
    }
    if (F & 1) s.a[F - 1] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(ra, am1, 0, 0));
#pragma unroll
    for (int q = 0; q < QP; ++q) {
      const dbl2 v = __builtin_bit_cast(dbl2, __builtin_amdgcn_raw_buffer_load_b128(rb, bp[q], 0, 0));
      s.b[2 * q] = v[0];
      s.b[2 * q + 1] = v[1];
    }
    if (Q & 1) s.b[Q - 1] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rb, bp[QP], 0, 0));
  };
  dbl4 acc[F][Q];
#pragma unroll
  for (int f = 0; f < F; ++f)
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[f][q] = dbl4{0.0, 0.0, 0.0, 0.0};
  load(st[0], 0);
  load(st[1], 4);
  load(st[2], 8);
  for (int j = 0; j < np; j += 16) {  // np is a multiple of 16
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      load(st[(u + 3) % NS], j + 4 * u + 12);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int f = 0; f < F; ++f)
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[f][q] = mfma64(st[u].a[f], st[u].b[q], acc[f][q]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // register r of block (f, q): Y at row R = lk + 4 r, i.e. function 2 R + f % 2
  // of the block pair (R of an odd last block), and the point of column l16
  double s[Q][4];
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int c = 0; c < 4; ++c) s[q][c] = 0.0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(pq + c * plane + 4 * (int64_t)i0), (short)0, 0x7ffffff0, 0x00020000);
#pragma unroll
    for (int f = 0; f < F; ++f) {
      double t[Q];  // this block's rows first: shorter chains round less
#pragma unroll
      for (int q = 0; q < Q; ++q) t[q] = 0.0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool pair = f < 2 * FP;
        // bytes from function lk of the quad to the row's function
        const uint32_t fo = (pair ? (uint32_t)(32 * (f >> 1) + 8 * r + (f & 1)) + lk : (uint32_t)(16 * f + 4 * r)) * 32u;
#pragma unroll
        for (int q = 0; q < QP; ++q) {
          const dbl2 e = __builtin_bit_cast(dbl2, __builtin_amdgcn_raw_buffer_load_b128(rs, bp[q] + fo, 0, 0));
          t[2 * q] += acc[f][2 * q][r] * e[0];
          t[2 * q + 1] += acc[f][2 * q + 1][r] * e[1];
        }
        if (Q & 1) {
          const double e = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, bp[QP] + fo, 0, 0));
          t[Q - 1] += acc[f][Q - 1][r] * e;
        }
      }
#pragma unroll
      for (int q = 0; q < Q; ++q) s[q][c] += t[q];
    }
    __builtin_amdgcn_sched_barrier(0);  // one component's loads at a time
  }
  // over the rows of the four lane groups; group lk writes component lk
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    double mine = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      double v = s[q][c];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (lk == c) mine = c ? 2.0 * v : v;
    }
    const int pt = q < 2 * QP ? 32 * (q >> 1) + 2 * l16 + (q & 1) : 16 * q + l16;
    part[(int64_t)lk * Pp + q0 + pt] = mine;
  }
}

// Four independent waves per workgroup, one item each: items (batch, point
// chunk, function chunk) where the batch's 16-blocks are divided evenly into as
// many chunks of at most four as they need (no padding beyond the blocks).
__global__ __launch_bounds__(256, 2) void k_grad_gemm(DevPlan d, const int32_t *items, int64_t it0, int64_t nit,
                                                      const int64_t *cd_off, const int64_t *part_off,
                                                      const double *cd, const double *panel, double *part) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t pos = 4 * xcd_map_runs(blockIdx.x, (nit + 3) / 4, 16) + wave;
  if (pos >= nit) return;
  const int64_t it = it0 + pos;
  const int b = __builtin_amdgcn_readfirstlane(items[3 * it]), tp = __builtin_amdgcn_readfirstlane(items[3 * it + 1]),
            ti = __builtin_amdgcn_readfirstlane(items[3 * it + 2]);
  const int P = d.batch_pt_off[b + 1] - d.batch_pt_off[b], n = d.batch_fn_off[b + 1] - d.batch_fn_off[b];
  const int Pp = (int)pad16(P), np = (int)pad16(n);
  const int mf = np >> 4, mq = Pp >> 4, nf = (mf + 3) >> 2, nq = (mq + 3) >> 2;
  const int fb = (int)((int64_t)ti * mf / nf), qb = (int)((int64_t)tp * mq / nq);
  const int F = (int)((int64_t)(ti + 1) * mf / nf) - fb, Q = (int)((int64_t)(tp + 1) * mq / nq) - qb;
  const double *pb = panel + d.panel_off[b], *M = cd + cd_off[b];
  double *pt = part + part_off[b] + (int64_t)ti * 4 * Pp;
  auto go = [&](auto f, auto q) { grad_item<decltype(f)::value, decltype(q)::value>(np, Pp, 16 * fb, 16 * qb, M, pb, pt); };
  auto with_q = [&](auto f) {
    switch (Q) {
      case 1: go(f, std::integral_constant<int, 1>{}); break;
      case 2: go(f, std::integral_constant<int, 2>{}); break;
      case 3: go(f, std::integral_constant<int, 3>{}); break;
      default: go(f, std::integral_constant<int, 4>{}); break;
    }
  };
  switch (F) {
    case 1: with_q(std::integral_constant<int, 1>{}); break;
    case 2: with_q(std::integral_constant<int, 2>{}); break;
    case 3: with_q(std::integral_constant<int, 3>{}); break;
    default: with_q(std::integral_constant<int, 4>{}); break;
  }
}

// The partials of a point summed over the batch's function tiles in tile
// order: out is [4][n_points] (n, d_x n, d_y n, d_z n) in user point order.
__global__ void k_grad_points(DevPlan d, int64_t b0, const int64_t *part_off, const double *part, double *out) {
  const int64_t b = b0 + blockIdx.x;
  const int g0 = d.batch_pt_off[b], P = d.batch_pt_off[b + 1] - g0;
  const int n = d.batch_fn_off[b + 1] - d.batch_fn_off[b];
  const int Pp = (int)pad16(P), nti = ((int)pad16(n) + GT - 1) / GT;
  const double *pp = part + part_off[b];
  for (int e = threadIdx.x; e < 4 * P; e += blockDim.x) {
    const int c = e / P, g = e - c * P;
    double s = 0.0;
    for (int t = 0; t < nti; ++t) s += pp[((int64_t)t * 4 + c) * Pp + g];
    out[(int64_t)c * d.n_points + d.perm[g0 + g]] = s;
  }
}

}  // namespace

int launch_grad_pass(const q4c_plan *p, size_t ip, const double *coef, const double *panel, double *out,
                     hipStream_t s) {
  const Pass &ps = p->passes[ip];
  const int64_t c0 = p->gr_cd_item_off[ip], nc = p->gr_cd_item_off[ip + 1] - c0;
  const int64_t w0 = p->gr_item_off[ip], nw = p->gr_item_off[ip + 1] - w0;
  if (nc > 0) {
    {
      TimedLaunch tl_(p, Q4C_TIMER_OTHER, s);
      hipLaunchKernelGGL(k_grad_cdense, dim3((unsigned)nc), dim3(256), 0, s, p->dp, p->d_gr_cditems, c0,
                         p->d_gr_cd_off, p->d_gr_fninfo, coef, p->d_gr_cd);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_grad_cdense");
  }
  if (nw > 0) {
    {
      TimedLaunch tl_(p, Q4C_TIMER_DENSITY_TILES, s);
      hipLaunchKernelGGL(k_grad_gemm, dim3((unsigned)((nw + 3) / 4)), dim3(256), 0, s, p->dp, p->d_gr_items, w0, nw,
                         p->d_gr_cd_off, p->d_gr_part_off, (const double *)p->d_gr_cd, panel, p->d_gr_part);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_grad_gemm");
  }
  const int64_t nbt = ps.b1 - ps.b0;
  if (nbt > 0) {
    {
      TimedLaunch tl_(p, Q4C_TIMER_DENSITY_POINTS, s);
      hipLaunchKernelGGL(k_grad_points, dim3((unsigned)nbt), dim3(256), 0, s, p->dp, ps.b0, p->d_gr_part_off,
                         (const double *)p->d_gr_part, out);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_grad_points");
  }
  return Q4C_OK;
}

}  // namespace q4c
