// The contraction of q4c_integrate_HS: H and S of one component, the Q4C
// integrand of Eq. 19 in the scalar form of Eq. 29, symmetrised.  The panel
// tabulation, batch sums and launches around it are in q4c_kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "q4c_internal.h"
#include "q4c_device.h"

namespace q4c {
namespace {

// phi and psi of one 16-function block at one K pair (8 points): points 2 lk
// and 2 lk + 1 of the 8, function l16 of the block.
struct OperandHS {
  dbl2 v[2];
};

// H and S of one component (the Q4C integrand of Eq. 19 in the scalar form
// of Eq. 29, symmetrised), from panels of phi and psi = u phi / 2:
//   H = Phi^T diag(w) (v Phi + Psi) + Psi^T diag(w) Phi,   S = Phi^T diag(w) Phi
// i.e. per 16 x 16 block and K step of 4 points three FP64 MFMAs: the row
// operands w phi_i and w v phi_i + w psi_i, formed once for the item's
// columns, against phi_j and psi_j.  The wave's item, loads and epilogue are
// those of the FP64 forward contraction: blocks (rb, cb .. cb + NB - 1), no
// LDS, no barriers, operands read from the panel a K pair ahead.
//
// Bound: FP64 matrix pipe.  60 atoms, both components (163 and 353 functions
// per batch on average) 8.6 -> 7.1 ms against 64 x 64 tiles in LDS with a
// barrier every 16 points; the MFMAs alone take 4.7 ms at their peak rate, 5.3
// at the clock of this kernel (74% of the active cycles; the other vector
// instructions, 1.4 per MFMA, 8% more).
template <int NB>
__device__ __forceinline__ void hs_item(const DevPlan &d, int f0, int n, int g0, int P, const double *pb, int rb, int cb,
                                        const double *om, double *staging) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, lk = lane >> 4;
  const int Pp = (int)pad16(P), np = (int)pad16(n);
  const int64_t plane = (int64_t)Pp * np;
  uint32_t off[1 + NB];
  off[0] = ((uint32_t)(lk >> 1) * np + 16 * rb + l16) * 32u + 16u * (lk & 1);
#pragma unroll
  for (int c = 0; c < NB; ++c) off[1 + c] = ((uint32_t)(lk >> 1) * np + 16 * (cb + c) + l16) * 32u + 16u * (lk & 1);
  // past the last point an empty buffer: nothing is read, and no branch makes
  // the waits of the next K pairs count for both of its sides
  auto load = [&](int k, OperandHS (&o)[1 + NB], dbl2 &wv, dbl2 &w) {
    const int nr = k < Pp ? np * 64 : 0;
    // w v and w from point k on, 0 past the batch's points (as in k_forward)
    const int nw = k < P ? (P - k) * 8 : 0;
    const __amdgpu_buffer_rsrc_t ro =
        __builtin_amdgcn_make_buffer_rsrc((void *)(om + g0 + k), (short)0, nw, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc((void *)(d.pw + g0 + k), (short)0, nw, 0x00020000);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void *)(pb + (int64_t)q * plane + (int64_t)(k >> 2) * np * 4), (short)0, nr, 0x00020000);
#pragma unroll
      for (int x = 0; x < 1 + NB; ++x)
        o[x].v[q] = __builtin_bit_cast(dbl2, __builtin_amdgcn_raw_buffer_load_b128(rs, off[x], 0, 0));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      wv[h] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(ro, 16 * lk + 8 * h, 0, 0));
      w[h] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rw, 16 * lk + 8 * h, 0, 0));
    }
  };
  dbl4 acc[NB][3];  // H (w v phi + w psi, phi), S, H (w phi, psi)
#pragma unroll
  for (int c = 0; c < NB; ++c)
#pragma unroll
    for (int q = 0; q < 3; ++q) acc[c][q] = dbl4{0.0, 0.0, 0.0, 0.0};
  auto multiply = [&](const OperandHS (&o)[1 + NB], const dbl2 &wv, const dbl2 &w) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double as = w[h] * o[0].v[0][h];                               // w phi_i
      const double ah = fma(wv[h], o[0].v[0][h], w[h] * o[0].v[1][h]);     // w v phi_i + w psi_i
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        acc[c][0] = mfma64(ah, o[1 + c].v[0][h], acc[c][0]);
        acc[c][1] = mfma64(as, o[1 + c].v[0][h], acc[c][1]);
        acc[c][2] = mfma64(as, o[1 + c].v[1][h], acc[c][2]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  OperandHS oa[1 + NB], ob[1 + NB];
  dbl2 va, vb, wa, wb;
  load(0, oa, va, wa);
  for (int k = 0; k < Pp; k += 16) {  // Pp is a multiple of 16: two K pairs per turn
    load(k + 8, ob, vb, wb);
    __builtin_amdgcn_sched_barrier(0);
    multiply(oa, va, wa);
    __builtin_amdgcn_sched_barrier(0);
    load(k + 16, oa, va, wa);
    __builtin_amdgcn_sched_barrier(0);
    multiply(ob, vb, wb);
    __builtin_amdgcn_sched_barrier(0);
  }
  // write the blocks (H, S) to the staged atom-pair blocks
  const StageRows sr = stage_rows(d, f0, n, rb, lk, staging);
#pragma unroll
  for (int c = 0; c < NB; ++c)
    stage_block<0, 2>(sr, d, f0, n, rb, cb + c, l16,
                   [&](int r, int q) { return q ? acc[c][1][r] : acc[c][0][r] + acc[c][2][r]; });
}

// Four independent waves per workgroup, one item each (as k_forward).
// tickets != NULL: a persistent launch, every wave draws items until none is
// left.
template <bool PERSIST>
__global__ __launch_bounds__(256, 3) void k_contract_hs(DevPlan d, const BlockItem *items, int64_t ni, int global_queue,
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
      hs_item<2>(d, f0, n, g0, P, pb, it.rb, it.cb, om, staging);
    else
      hs_item<1>(d, f0, n, g0, P, pb, it.rb, it.cb, om, staging);
    if (!PERSIST) return;
    pos = draw();
  }
}

}  // namespace

int launch_contract_hs(const q4c_plan *p, const Pass &ps, const double *panel, unsigned *tickets, hipStream_t s) {
  const LaunchCfg cfg = p->cfg_hs;
  const BlockItem *items = (cfg.order ? p->d_blocks_cost : p->d_blocks) + ps.bi0;
  const int64_t ni = ps.bi1 - ps.bi0;
  if (ni <= 0) return Q4C_OK;
  const int64_t groups = (ni + 3) / 4;
  if (tickets)
    hipLaunchKernelGGL(k_contract_hs<true>, dim3((unsigned)std::min<int64_t>(cfg.persistent, groups)), dim3(256), 0, s,
                       p->dp, items, ni, (int)cfg.order, (const double *)p->d_om, panel, p->d_staging, tickets);
  else
    hipLaunchKernelGGL(k_contract_hs<false>, dim3((unsigned)groups), dim3(256), 0, s, p->dp, items, ni, (int)cfg.order,
                       (const double *)p->d_om, panel, p->d_staging, tickets);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "k_contract_hs");
  return Q4C_OK;
}

}  // namespace q4c
