// The FP64 contraction of q4c_integrate_H: the five parts of every batch's
// upper block triangle, from the batch's FP64 panel (phi, d/dx, d/dy, d/dz).
// The panel tabulation, batch sums and launches around it are in
// q4c_kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "q4c_internal.h"
#include "q4c_device.h"

namespace q4c {
namespace {

// The operands of one K pair (8 points) of one 16-function block: component q
// at points 2 lk and 2 lk + 1 of the 8, of function l16 of the block.
struct Operand {
  dbl2 v[4];
};

constexpr int kJoin = 32;  // points between two joins of the D and M sums (see forward_item)

// One wave's item: the 16 x 16 blocks (rb, cb .. cb + NB - 1) of a batch, all
// its points.  With a = grad phi_i (rows, weighted by w v) and b = grad phi_j
// (columns), the nine products of grad phi_i and grad phi_j that W needs come
// from six:
//   D_m = a_m b_m,   M_x = (a_y - a_z)(b_y + b_z) and cyclic,
//   Ws = D_x + D_y + D_z,
//   Wso_x = a_y b_z - a_z b_y = M_x - (D_y - D_z) and cyclic
// (a_y b_y and a_z b_z are already there), so with V seven FP64 MFMAs per K
// step instead of ten, for three subtractions per row block and three
// additions per column block.  FP64 vector instructions and FP64 MFMA share
// one pipe on this chip (measured: 4.5 cycles against 64), so the row operand,
// of which there is one, takes the weight.
//
// No LDS and no barriers: every lane reads its operands straight from the
// panel, 16 bytes (two points) each, one K pair ahead in a second register
// set.  A wave reads (1 + NB) KB x 4 per 14 NB MFMAs; four waves of a
// workgroup take consecutive row blocks of one column pair and share its
// lines in L1 (70% of the reads hit there, 76% of the rest in L2 on the cluster
// below, 84% on the slab).  Waves never wait for each other.
//
// Wso is the difference of sums that grow with the products of D, so these run
// over kJoin points only and then join the running Ws and Wso.  RMS error of Wso
// against 80-bit sums relative to its own products, in units of that of the
// nine products summed by MFMA over a whole batch, same panels: without joins
// 1.19 (3 atoms), 1.24 (60 atoms), 2.65 (points within 0.1 bohr of the axis of
// two atoms, where D outweighs Wso most); joined every 64 points 1.06, 0.96,
// 1.14; every 32 points 1.01, 0.91, 1.04.  With the distances of k_panel, which
// all parts profit from, 0.59, 0.66, 0.30 of what it was.  The joins cost 2%
// (cluster) and 3.6% (slab below); every 64 points 0.7 and 1.9%.
//
// Bound: FP64 matrix pipe.  120-atom cluster (1.9M points, 171 functions per
// batch on average) 14.5 -> 9.4 ms, dense 300-atom slab (319 per batch) 43.3
// -> 29.0 ms against ten products from 64 x 64 tiles in LDS with a barrier
// every 8 points; the seven MFMAs alone take 6.7 and 21.3 ms at their peak
// rate (the matrix pipe is busy for 76 and 78% of the active cycles).
template <int NB>
__device__ __forceinline__ void forward_item(const DevPlan &d, int f0, int n, int g0, int P, const double *pb, int rb,
                                             int cb, const double *om, double *staging) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lk = lane >> 4;
  const int Pp = (int)pad16(P), np = (int)pad16(n);
  const int64_t plane = (int64_t)Pp * np;
  // lane offsets (bytes) within a K pair's two point quads: quad lk / 2, then
  // the function's 32 bytes, then its point pair lk % 2
  uint32_t off[1 + NB];
  off[0] = ((uint32_t)(lk >> 1) * np + 16 * rb + l16) * 32u + 16u * (lk & 1);
#pragma unroll
  for (int c = 0; c < NB; ++c) off[1 + c] = ((uint32_t)(lk >> 1) * np + 16 * (cb + c) + l16) * 32u + 16u * (lk & 1);
  // past the last point an empty buffer: nothing is read, and no branch makes
  // the waits of the next K pairs count for both of its sides (with one, every
  // other K pair waited for loads just issued: 9.52 instead of 9.15 ms)
  auto load = [&](int k, Operand (&o)[1 + NB], dbl2 &w) {
    const int nr = k < Pp ? np * 64 : 0;
    // w v from point k on; past the batch's points 0: the buffer ends there and
    // the lanes' offsets alone are checked against it (no scalar offset)
    const __amdgpu_buffer_rsrc_t ro =
        __builtin_amdgcn_make_buffer_rsrc((void *)(om + g0 + k), (short)0, k < P ? (P - k) * 8 : 0, 0x00020000);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // the K pair's two point quads of component q: a wave-uniform base, so
      // that no vector instruction computes an address
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void *)(pb + (int64_t)q * plane + (int64_t)(k >> 2) * np * 4), (short)0, nr, 0x00020000);
#pragma unroll
      for (int x = 0; x < 1 + NB; ++x)
        o[x].v[q] = __builtin_bit_cast(dbl2, __builtin_amdgcn_raw_buffer_load_b128(rs, off[x], 0, 0));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
      w[h] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(ro, 16 * lk + 8 * h, 0, 0));
  };
  dbl4 acc[NB][7];
#pragma unroll
  for (int c = 0; c < NB; ++c)
#pragma unroll
    for (int q = 0; q < 7; ++q) acc[c][q] = dbl4{0.0, 0.0, 0.0, 0.0};
  // first: the D sums start from zero here
  auto multiply = [&](const Operand (&o)[1 + NB], const dbl2 &w, auto first) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double a0 = o[0].v[0][h] * w[h], ax = o[0].v[1][h] * w[h], ay = o[0].v[2][h] * w[h],
                   az = o[0].v[3][h] * w[h];
      const double ayz = ay - az, azx = az - ax, axy = ax - ay;
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        const double b0 = o[1 + c].v[0][h], bx = o[1 + c].v[1][h], by = o[1 + c].v[2][h], bz = o[1 + c].v[3][h];
        acc[c][0] = mfma64(a0, b0, acc[c][0]);
        const bool z = decltype(first)::value && h == 0;
        const dbl4 z4 = dbl4{0.0, 0.0, 0.0, 0.0};
        acc[c][1] = mfma64(ax, bx, z ? z4 : acc[c][1]);
        acc[c][2] = mfma64(ay, by, z ? z4 : acc[c][2]);
        acc[c][3] = mfma64(az, bz, z ? z4 : acc[c][3]);
        acc[c][4] = mfma64(ayz, by + bz, acc[c][4]);
        acc[c][5] = mfma64(azx, bz + bx, acc[c][5]);
        acc[c][6] = mfma64(axy, bx + by, acc[c][6]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  dbl4 ws[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) ws[c] = dbl4{0.0, 0.0, 0.0, 0.0};
  Operand oa[1 + NB], ob[1 + NB];
  dbl2 wa, wb;
  load(0, oa, wa);
  auto turn = [&](int k, auto first) {  // two K pairs (Pp is a multiple of 16)
    load(k + 8, ob, wb);
    __builtin_amdgcn_sched_barrier(0);
    multiply(oa, wa, first);
    __builtin_amdgcn_sched_barrier(0);
    load(k + 16, oa, wa);
    __builtin_amdgcn_sched_barrier(0);
    multiply(ob, wb, std::false_type{});
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int k0 = 0; k0 < Pp; k0 += kJoin) {
    turn(k0, std::true_type{});
    for (int k = k0 + 16; k < min(Pp, k0 + kJoin); k += 16) turn(k, std::false_type{});
    // Ws and Wso of these points join the running sums (Wso in M's registers)
#pragma unroll
    for (int c = 0; c < NB; ++c) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double dx = acc[c][1][r], dy = acc[c][2][r], dz = acc[c][3][r];
        ws[c][r] += (dx + dy) + dz;
        acc[c][4][r] -= dy - dz;
        acc[c][5][r] -= dz - dx;
        acc[c][6][r] -= dx - dy;
      }
    }
  }
  // write the blocks to the staged atom-pair blocks
  const double cp = d.cprime;
  const StageRows sr = stage_rows(d, f0, n, rb, lk, staging);
#pragma unroll
  for (int c = 0; c < NB; ++c)
    stage_block<0, 5>(sr, d, f0, n, rb, cb + c, l16, [&](int r, int q) {
      return q == 0 ? acc[c][0][r] : cp * (q == 1 ? ws[c][r] : acc[c][q + 2][r]);
    });
}

// A workgroup is four independent waves with one item each (item 4 x + wave
// of the pass, consecutive workgroups of an XCD in batch order).  tickets !=
// NULL: a persistent launch, every wave draws items until none is left.
template <bool PERSIST>
__global__ __launch_bounds__(256, 2) void k_forward(DevPlan d, const BlockItem *items, int64_t ni, int global_queue,
                                                    const double *om, const double *panel, double *staging,
                                                    unsigned *tickets) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool gq = global_queue != 0;
  auto draw = [&]() -> int64_t {
    int64_t p = 0;
    if ((threadIdx.x & 63) == 0) p = ticket_pos(tickets, ni, gq, draw_ticket(tickets, gq));
    return uniform_i64(p);
  };
  int64_t pos = PERSIST ? draw()
                        : 4 * (gq ? (int64_t)blockIdx.x : xcd_map_runs(blockIdx.x, (ni + 3) / 4, 128)) + wave;
  while (pos < ni) {
    const BlockItem it = items[pos];
    const int b = it.batch;
    const int g0 = d.batch_pt_off[b], P = d.batch_pt_off[b + 1] - g0;
    const int f0 = d.batch_fn_off[b], n = d.batch_fn_off[b + 1] - f0;
    const double *pb = panel + d.panel_off[b];
    if (it.wide)
      forward_item<2>(d, f0, n, g0, P, pb, it.rb, it.cb, om, staging);
    else
      forward_item<1>(d, f0, n, g0, P, pb, it.rb, it.cb, om, staging);
    if (!PERSIST) return;
    pos = draw();
  }
}

}  // namespace

int launch_forward(const q4c_plan *p, const Pass &ps, const double *panel, unsigned *tickets, hipStream_t s) {
  const LaunchCfg cfg = p->cfg_contract;
  const BlockItem *items = (cfg.order ? p->d_blocks_cost : p->d_blocks) + ps.bi0;
  const int64_t ni = ps.bi1 - ps.bi0;
  if (ni <= 0) return Q4C_OK;
  const int64_t groups = (ni + 3) / 4;
  if (tickets)
    hipLaunchKernelGGL(k_forward<true>, dim3((unsigned)std::min<int64_t>(cfg.persistent, groups)), dim3(256), 0, s,
                       p->dp, items, ni, (int)cfg.order, (const double *)p->d_om, panel, p->d_staging, tickets);
  else
    hipLaunchKernelGGL(k_forward<false>, dim3((unsigned)groups), dim3(256), 0, s, p->dp, items, ni, (int)cfg.order,
                       (const double *)p->d_om, panel, p->d_staging, tickets);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "k_forward");
  return Q4C_OK;
}

}  // namespace q4c
