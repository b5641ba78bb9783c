// HIP kernels of libq4c for CDNA4 (gfx950).
//
//  k_tabulate[_few]  nao_tabulate: phi and grad phi of a batch's relevant
//                    functions at its points (Eq. 12a, App. B), as the
//                    panels compute them; FP64 or FP32 hi + lo output.
//  k_om              w_g v_g per active point (the weighting of Eq. 29).
//  k_panel           per (batch, function tile, 64 points): phi and grad phi
//                    into the batch's operand panel (HBM).
//  k_contract_*      per (batch, tile ti <= tj) work item, or smaller items of
//                    it: the weighted products
//                        V  = Phi^T diag(w v) Phi
//                        Gs = sum_a dPhi_a^T diag(w v) dPhi_a
//                        Gm = dPhi_b^T diag(w v) dPhi_c - dPhi_c^T diag(w v) dPhi_b
//                    accumulate on MFMA (Eq. 29 restricted to the batch,
//                    Eq. 31): the reduced precisions, V alone and the vector
//                    ALU baseline here, FP64 in q4c_forward_kernels.hip.  The
//                    lower atom-block triangle follows from (anti)symmetry.
//                    Results go to a staging buffer laid out per (batch, atom
//                    pair).
//  k_reduce          deterministic batch-to-global sum: every stored atom
//                    pair adds its staged blocks in batch order (FP64).
//  k_spinor          2x2-spinor assembly of the W and V blocks.
// The adjoint (density_on_grid) is in q4c_density_kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "q4c_internal.h"
#include "q4c_device.h"

namespace q4c {
namespace {


// ---------------------------------------------------------------------------
// Basis functions
// ---------------------------------------------------------------------------

// A function's value is the same to the bit in every kernel that forms it:
// products and sums are fused within an expression only, not as the code
// around them happens to allow.
#pragma clang fp contract(on)

// Real solid harmonics S_lm = s^l Y_lm (App. B convention, Condon-Shortley
// phase as written there: Y_1,1 = -sqrt(3/4pi) x/s) and their gradients,
// l <= 4, indexed by lm = l^2 + l + m.
__device__ __forceinline__ void solid_harmonic(int lm, double x, double y, double z, double &S, double &gx,
                                               double &gy, double &gz) {
  constexpr double C00 = 0.28209479177387814, C1 = 0.4886025119029199, C2a = 1.0925484305920792,
                   C20 = 0.31539156525252005, C22 = 0.5462742152960396, C33 = 0.5900435899266435,
                   C32b = 2.8906114426405543, C31 = 0.4570457994644657, C30 = 0.3731763325901154,
                   C32a = 1.4453057213202771;
  // l = 4: K_4^0 / 8 and sqrt2 K_4^|m| times the integer factors of the polynomials
  constexpr double C40 = 0.10578554691520431, C41 = 0.6690465435572891, C42 = 0.47308734787878,
                   C43 = 1.7701307697799304, C44 = 0.6258357354491761;
  switch (lm) {
    case 0: S = C00; gx = gy = gz = 0.0; break;
    case 1: S = -C1 * y; gx = 0.0; gy = -C1; gz = 0.0; break;
    case 2: S = C1 * z; gx = 0.0; gy = 0.0; gz = C1; break;
    case 3: S = -C1 * x; gx = -C1; gy = 0.0; gz = 0.0; break;
    case 4: S = C2a * x * y; gx = C2a * y; gy = C2a * x; gz = 0.0; break;
    case 5: S = -C2a * y * z; gx = 0.0; gy = -C2a * z; gz = -C2a * y; break;
    case 6: S = C20 * (2.0 * z * z - x * x - y * y); gx = -2.0 * C20 * x; gy = -2.0 * C20 * y; gz = 4.0 * C20 * z; break;
    case 7: S = -C2a * x * z; gx = -C2a * z; gy = 0.0; gz = -C2a * x; break;
    case 8: S = C22 * (x * x - y * y); gx = 2.0 * C22 * x; gy = -2.0 * C22 * y; gz = 0.0; break;
    case 9: S = -C33 * y * (3.0 * x * x - y * y); gx = -6.0 * C33 * x * y; gy = -3.0 * C33 * (x * x - y * y); gz = 0.0; break;
    case 10: S = C32b * x * y * z; gx = C32b * y * z; gy = C32b * x * z; gz = C32b * x * y; break;
    case 11: {
      double q = 4.0 * z * z - x * x - y * y;
      S = -C31 * y * q; gx = 2.0 * C31 * x * y; gy = -C31 * (q - 2.0 * y * y); gz = -8.0 * C31 * y * z;
    } break;
    case 12: S = C30 * z * (2.0 * z * z - 3.0 * x * x - 3.0 * y * y); gx = -6.0 * C30 * x * z; gy = -6.0 * C30 * y * z;
      gz = C30 * (6.0 * z * z - 3.0 * x * x - 3.0 * y * y); break;
    case 13: {
      double q = 4.0 * z * z - x * x - y * y;
      S = -C31 * x * q; gx = -C31 * (q - 2.0 * x * x); gy = 2.0 * C31 * x * y; gz = -8.0 * C31 * x * z;
    } break;
    case 14: S = C32a * z * (x * x - y * y); gx = 2.0 * C32a * x * z; gy = -2.0 * C32a * y * z; gz = C32a * (x * x - y * y); break;
    case 15: S = -C33 * x * (x * x - 3.0 * y * y); gx = -3.0 * C33 * (x * x - y * y); gy = 6.0 * C33 * x * y; gz = 0.0; break;
    // l = 4 (the small-component partners of f shells), rho = x^2 + y^2 + z^2
    case 16: S = 4.0 * C44 * (x * x * x * y - x * y * y * y); gx = 4.0 * C44 * (3.0 * x * x * y - y * y * y);
      gy = 4.0 * C44 * (x * x * x - 3.0 * x * y * y); gz = 0.0; break;
    case 17: S = -C43 * z * (3.0 * x * x * y - y * y * y); gx = -6.0 * C43 * x * y * z;
      gy = -3.0 * C43 * z * (x * x - y * y); gz = -C43 * (3.0 * x * x * y - y * y * y); break;
    case 18: {
      const double t = 6.0 * z * z - x * x - y * y;  // 7 z^2 - rho
      S = 2.0 * C42 * x * y * t; gx = 2.0 * C42 * y * (t - 2.0 * x * x); gy = 2.0 * C42 * x * (t - 2.0 * y * y);
      gz = 24.0 * C42 * x * y * z;
    } break;
    case 19: {
      const double q = 4.0 * z * z - 3.0 * x * x - 3.0 * y * y;  // 7 z^2 - 3 rho
      S = -C41 * y * z * q; gx = 6.0 * C41 * x * y * z; gy = -C41 * z * (q - 6.0 * y * y); gz = -C41 * y * (q + 8.0 * z * z);
    } break;
    case 20: {
      const double rho = x * x + y * y + z * z, z2 = z * z;
      S = C40 * (35.0 * z2 * z2 - 30.0 * z2 * rho + 3.0 * rho * rho); gx = C40 * x * (12.0 * rho - 60.0 * z2);
      gy = C40 * y * (12.0 * rho - 60.0 * z2); gz = C40 * z * (80.0 * z2 - 48.0 * rho);
    } break;
    case 21: {
      const double q = 4.0 * z * z - 3.0 * x * x - 3.0 * y * y;
      S = -C41 * x * z * q; gx = -C41 * z * (q - 6.0 * x * x); gy = 6.0 * C41 * x * y * z; gz = -C41 * x * (q + 8.0 * z * z);
    } break;
    case 22: {
      const double t = 6.0 * z * z - x * x - y * y;
      S = C42 * (x * x - y * y) * t; gx = 2.0 * C42 * x * (t - x * x + y * y); gy = -2.0 * C42 * y * (t + x * x - y * y);
      gz = 12.0 * C42 * (x * x - y * y) * z;
    } break;
    case 23: S = -C43 * z * (x * x * x - 3.0 * x * y * y); gx = -3.0 * C43 * z * (x * x - y * y);
      gy = 6.0 * C43 * x * y * z; gz = -C43 * (x * x * x - 3.0 * x * y * y); break;
    default: S = C44 * (x * x * x * x - 6.0 * x * x * y * y + y * y * y * y); gx = 4.0 * C44 * (x * x * x - 3.0 * x * y * y);
      gy = 4.0 * C44 * (y * y * y - 3.0 * x * x * y); gz = 0.0; break;
  }
}

// ---------------------------------------------------------------------------
// Tabulation: one wave walks the shells of up to 64 functions at 64 points.
// ---------------------------------------------------------------------------

// Radial interval of a shell (cutoff > s) at distance s: index j and s - r_j.
// The index comes from an approximate square root corrected against the exact
// knots r_j = j^2 k2; s - r_j is rounded once.
__device__ __forceinline__ int radial_interval(double s, int n, double k1, double k2, double &dd) {
  const double u = s * k1;
  int j = u > 0.0 ? (int)(u * __builtin_amdgcn_rsq(u)) : 0;
  j = j < 0 ? 0 : (j > n - 1 ? n - 1 : j);
  double rj = (double)j * (double)j * k2;
  if (s < rj && j > 0) {
    --j;
    rj = (double)j * (double)j * k2;
  } else if (j < n - 1 && s >= (double)(j + 1) * (double)(j + 1) * k2) {
    ++j;
    rj = (double)j * (double)j * k2;
  }
  dd = fma(-(double)j * (double)j, k2, s);
  return j;
}

// 1 / s and s of a squared distance s2 (0 for 0), s to its last bit: the steep
// radials of tight functions carry its error 10 times and more into phi (V,
// relative to its terms: RMS error 1.2e-15 -> 2.8e-16 on 60 atoms).
__device__ __forceinline__ void distance(double s2, double &rinv, double &s) {
  rinv = s = 0.0;
  if (s2 > 0.0) {
    rinv = __builtin_amdgcn_rsq(s2);
    rinv = rinv * (1.5 - 0.5 * s2 * rinv * rinv);
    s = s2 * rinv;
    s = fma(fma(-s, s, s2), 0.5 * rinv, s);
  }
}

// lane k's value of a vector register as a scalar
__device__ __forceinline__ int64_t lane_i64(int64_t v, int k) {
  const uint32_t lo = __builtin_amdgcn_readlane((int)v, k), hi = __builtin_amdgcn_readlane((int)(v >> 32), k);
  return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double lane_f64(double v, int k) {
  return __builtin_bit_cast(double, lane_i64(__builtin_bit_cast(int64_t, v), k));
}

// The data of up to 64 functions of a batch: lane k holds function r0 + k.
struct FnData {
  int atom, l, nint;
  int i_first;  // the first function of function r0's shell, which may begin before r0 (wave-uniform)
  double ax, ay, az, rc, k1, k2;
  int64_t coef, u;
};
template <bool HS>
__device__ __forceinline__ FnData fn_data(const DevPlan &d, int f0, int n, int r0) {
  const int lane = threadIdx.x & 63;
  const int mine = r0 + lane < n ? r0 + lane : n - 1;
  const int fn = d.loc_fn[f0 + mine], shlm = d.fn_shlm[fn], sh = shlm >> 5, lm = shlm & 31;
  FnData m;
  m.atom = d.fn_atom[fn];
  m.l = (lm >= 1) + (lm >= 4) + (lm >= 9) + (lm >= 16);
  m.ax = d.R[3 * m.atom];
  m.ay = d.R[3 * m.atom + 1];
  m.az = d.R[3 * m.atom + 2];
  m.rc = d.shell_rcut[sh];
  m.k1 = d.shell_knot[2 * sh];
  m.k2 = d.shell_knot[2 * sh + 1];
  m.nint = d.shell_nint[sh];
  m.coef = d.shell_coef_off[sh];
  m.u = HS ? d.shell_u_off[sh] : 0;
  m.i_first = r0 - __builtin_amdgcn_readlane(lm - m.l * m.l, 0);
  return m;
}

// Functions r0 .. rn - 1 (at most 64) of a batch at this lane's point, by
// shells: put(i, phi, d/dx, d/dy, d/dz) or (HS) put(i, phi, psi = u phi / 2, 0,
// 0) for every function of every shell that has one in the range, in order (so
// a first or last shell's functions outside the range too).  All lanes work on
// the same function; lanes that are not live get zeros.
template <bool HS, typename Put>
__device__ __forceinline__ void walk_shells(const DevPlan &d, const FnData &m, int r0, int rn, double px, double py,
                                            double pz, bool live, Put put) {
  // the distance to an atom and a shell's table entry, fetched a shell ahead
  struct { double dx, dy, dz, s2, rinv, s; } geo = {};
  struct { dbl4 c, e; double dd; } rad;
  int atom = -1;
  auto fetch = [&](int k) {
    const int at = __builtin_amdgcn_readlane(m.atom, k);
    if (at != atom) {
      atom = at;
      geo.dx = px - lane_f64(m.ax, k);
      geo.dy = py - lane_f64(m.ay, k);
      geo.dz = pz - lane_f64(m.az, k);
      const double s2 = geo.s2 = geo.dx * geo.dx + geo.dy * geo.dy + geo.dz * geo.dz;
      distance(s2, geo.rinv, geo.s);
    }
    const double rc = lane_f64(m.rc, k);
    rad.c = rad.e = dbl4{0.0, 0.0, 0.0, 0.0};
    rad.dd = 0.0;
    if (live && geo.s2 < rc * rc) {
      const int j = radial_interval(geo.s, __builtin_amdgcn_readlane(m.nint, k), lane_f64(m.k1, k), lane_f64(m.k2, k),
                                    rad.dd);
      rad.c = *reinterpret_cast<const dbl4 *>(d.coef + lane_i64(m.coef, k) + 4 * (int64_t)j);
      if (HS) rad.e = *reinterpret_cast<const dbl4 *>(d.ucoef + lane_i64(m.u, k) + 4 * (int64_t)j);
    }
  };
  if (rn > r0) fetch(0);
  for (int i = m.i_first; i < rn;) {  // the shells (wave-uniform)
    const int ls = __builtin_amdgcn_readlane(m.l, i > r0 ? i - r0 : 0);
    const double dx = geo.dx, dy = geo.dy, dz = geo.dz, rinv = geo.rinv, dd = rad.dd;
    const dbl4 c = rad.c, e = rad.e;
    if (i + 2 * ls + 1 < rn) fetch(i + 2 * ls + 1 - r0);
    // Rt and Rt' / s, or (H/S) Rt and u / 2
    const double R = ((c[3] * dd + c[2]) * dd + c[1]) * dd + c[0];
    const double q = HS ? 0.5 * (((e[3] * dd + e[2]) * dd + e[1]) * dd + e[0])
                                   : ((3.0 * c[3] * dd + 2.0 * c[2]) * dd + c[1]) * rinv;
    auto shell = [&](auto lc) {
      constexpr int l = decltype(lc)::value;
      // an opaque copy: the harmonics of every l would otherwise be hoisted
      // out of the loop over the shells and held in registers
      double x = dx, y = dy, z = dz;
      asm volatile("" : "+v"(x), "+v"(y), "+v"(z));
      static_for<0, 2 * l + 1>([&](auto mc) {
        constexpr int mm = decltype(mc)::value;
        double S, gx, gy, gz;
        solid_harmonic(l * l + mm, x, y, z, S, gx, gy, gz);
        const double f = R * S;
        if (HS)
          put(i + mm, f, q * f, 0.0, 0.0);
        else
          put(i + mm, f, q * x * S + R * gx, q * y * S + R * gy, q * z * S + R * gz);
      });
      i += 2 * l + 1;
    };
    switch (ls) {
      case 0: shell(std::integral_constant<int, 0>{}); break;
      case 1: shell(std::integral_constant<int, 1>{}); break;
      case 2: shell(std::integral_constant<int, 2>{}); break;
      case 3: shell(std::integral_constant<int, 3>{}); break;
      default: shell(std::integral_constant<int, 4>{}); break;
    }
  }
}

#pragma clang fp contract(fast)

// ---------------------------------------------------------------------------
// nao_tabulate: out is [ncomp][P][n] per batch (FP64), or [ncomp][2][P][n]
// floats with the hi and lo planes (F32_HILO).  One workgroup per (batch,
// 64-function tile, 64 points): each wave walks the shells of 8 functions, two
// components at a time (67 KB of LDS, so that two workgroups share a CU), and
// the values leave as runs of the tile's 64 functions per point.
//
// Bound: the latency of the shells' table reads, with four waves per SIMD to
// cover it (0.16 ms of stores alone, 0.25 ms without the stores).  30 atoms
// (0.79 GB, 0.12 ms at the rate of a fill) 0.31 ms with every function looked
// up on its own by one workgroup per tile, 0.28 ms with that split over the
// points, 0.26 ms so; 16 functions per wave 0.30 ms; one wave per 64 functions
// with runs of 16, as the panels, 0.37 ms (lines shared by two runs).
// ---------------------------------------------------------------------------

template <bool HILO>
__global__ __launch_bounds__(512, 4) void k_tabulate(DevPlan d, const WorkItem *tiles, int64_t t0, int64_t wg0, int npb,
                                                     int64_t b0, int deriv, void *out) {
  constexpr int SR = T + 1;
  __shared__ double st[2][64 * SR];
  const int64_t bid = wg0 + xcd_map(blockIdx.x, gridDim.x);  // as in k_panel
  const WorkItem it = tiles[t0 + bid / npb];
  const int b = it.batch;
  const int g0 = d.batch_pt_off[b], P = d.batch_pt_off[b + 1] - g0;
  const int f0 = d.batch_fn_off[b], n = d.batch_fn_off[b + 1] - f0;
  const int r0 = it.ti * T;
  const int nrow = n - r0 < T ? n - r0 : T;
  const int64_t plane = (int64_t)P * n;
  const int64_t base = (deriv ? 4 : 1) * (d.tab_off[b] - d.tab_off[b0]);  // values before this batch
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int p0 = 64 * (int)(bid % npb);
  if (p0 >= P) return;  // workgroup-uniform
  const int w0 = r0 + 8 * wave, wn = w0 + 8 < n ? w0 + 8 : n;  // this wave's functions
  const FnData fd = fn_data<false>(d, f0, n, w0 < n ? w0 : n - 1);
  const int npt = P - p0 < 64 ? P - p0 : 64;
  const bool live = lane < npt;
  const int g = g0 + p0 + (live ? lane : 0);
  const double px = d.px[g], py = d.py[g], pz = d.pz[g];
  auto pass = [&](auto qc) {  // components q and q + 1
    constexpr int q = decltype(qc)::value;
    if (w0 < n)
      walk_shells<false>(d, fd, w0, wn, px, py, pz, live, [&](int i, double f, double fx, double fy, double fz) {
        if (i < w0 || i >= wn) return;  // of a shell that another wave shares
        st[0][lane * SR + i - r0] = q ? fy : f;
        st[1][lane * SR + i - r0] = q ? fz : fx;
      });
    __syncthreads();  // staged
    if (lane < nrow)
      for (int c = 0; c < (deriv ? 2 : 1); ++c)
#pragma unroll 8
        for (int pt = wave; pt < npt; pt += 8) {
          const double x = st[c][pt * SR + lane];
          const int64_t o = (int64_t)(p0 + pt) * n + r0 + lane;
          if (HILO) {
            float *of = static_cast<float *>(out) + 2 * (base + (q + c) * plane);
            const float hi = (float)x;
            of[o] = hi;
            of[plane + o] = (float)(x - (double)hi);
          } else {
            static_cast<double *>(out)[base + (q + c) * plane + o] = x;
          }
        }
    __syncthreads();  // read
  };
  pass(std::integral_constant<int, 0>{});
  if (deriv) pass(std::integral_constant<int, 2>{});
}

// nao_tabulate where batches leave many of k_tabulate's lanes without a point
// (launch_tabulate): one workgroup per (batch, 64-function tile), 8 points at a
// time, every (function, point) on a lane of its own, the functions in the order
// of lm.
struct TileMeta {
  double ax[T], ay[T], az[T];  // centres
  double rc[T];                // cutoffs (0 for padding)
  double k1[T], k2[T];         // nint^2 / rcut, rcut / nint^2
  int64_t coef[T];             // offset of the shell's table
  int nint[T], lm[T];
  int order[T];                // tile functions sorted by lm
};

// Stage metadata of the tile's functions (threads 0 .. T-1) and an ordering
// by lm, so that lanes working on neighbouring items mostly take the same
// solid-harmonic branch.
__device__ __forceinline__ void load_tile_meta(const DevPlan &d, TileMeta &M, int f0, int n, int r0) {
  const int tid = threadIdx.x;
  if (tid < T) {
    const int lf = r0 + tid;
    if (lf < n) {
      const int fn = d.loc_fn[f0 + lf];
      const int a = d.fn_atom[fn], shlm = d.fn_shlm[fn], sh = shlm >> 5;
      M.ax[tid] = d.R[3 * a];
      M.ay[tid] = d.R[3 * a + 1];
      M.az[tid] = d.R[3 * a + 2];
      M.rc[tid] = d.shell_rcut[sh];
      M.k1[tid] = d.shell_knot[2 * sh];
      M.k2[tid] = d.shell_knot[2 * sh + 1];
      M.coef[tid] = d.shell_coef_off[sh];
      M.nint[tid] = d.shell_nint[sh];
      M.lm[tid] = shlm & 31;
    } else {
      M.ax[tid] = M.ay[tid] = M.az[tid] = 0.0;
      M.rc[tid] = 0.0;
      M.k1[tid] = M.k2[tid] = 0.0;
      M.coef[tid] = 0;
      M.nint[tid] = 0;
      M.lm[tid] = 32;  // padding sorts last
    }
  }
  __syncthreads();
  if (tid < T) {
    const int mine = M.lm[tid];
    int rank = 0;
    for (int o = 0; o < T; ++o) rank += (M.lm[o] < mine) || (M.lm[o] == mine && o < tid);
    M.order[rank] = tid;
  }
}

#pragma clang fp contract(on)
// phi and grad phi of tile function m at point (px, py, pz), as walk_shells.
__device__ __forceinline__ void tab_meta(const DevPlan &d, const TileMeta &M, int m, double px, double py, double pz,
                                         double &f, double &fx, double &fy, double &fz) {
  const double dx = px - M.ax[m], dy = py - M.ay[m], dz = pz - M.az[m];
  const double s2 = dx * dx + dy * dy + dz * dz, rc = M.rc[m];
  if (!(s2 < rc * rc)) {
    f = fx = fy = fz = 0.0;
    return;
  }
  double rinv, s, dd;
  distance(s2, rinv, s);
  const int j = radial_interval(s, M.nint[m], M.k1[m], M.k2[m], dd);
  const dbl4 c = *reinterpret_cast<const dbl4 *>(d.coef + M.coef[m] + 4 * (int64_t)j);
  const double R = ((c[3] * dd + c[2]) * dd + c[1]) * dd + c[0];
  const double q = ((3.0 * c[3] * dd + 2.0 * c[2]) * dd + c[1]) * rinv;  // Rt'(s) / s
  double S, gx, gy, gz;
  solid_harmonic(M.lm[m], dx, dy, dz, S, gx, gy, gz);
  f = R * S;
  fx = q * dx * S + R * gx;
  fy = q * dy * S + R * gy;
  fz = q * dz * S + R * gz;
}

#pragma clang fp contract(fast)

template <bool HILO>
__global__ __launch_bounds__(256) void k_tabulate_few(DevPlan d, const WorkItem *tiles, int64_t t0, int64_t b0,
                                                      int deriv, void *out) {
  constexpr int CP = 8;
  constexpr int SR = T + 1;
  __shared__ TileMeta M;
  __shared__ double st[4 * CP * SR];
  const WorkItem it = tiles[t0 + blockIdx.x];
  const int b = it.batch;
  const int g0 = d.batch_pt_off[b], P = d.batch_pt_off[b + 1] - g0;
  const int f0 = d.batch_fn_off[b], n = d.batch_fn_off[b + 1] - f0;
  const int r0 = it.ti * T;
  const int nrow = n - r0 < T ? n - r0 : T;
  const int nq = deriv ? 4 : 1;
  const int64_t plane = (int64_t)P * n;
  const int64_t base = (int64_t)nq * (d.tab_off[b] - d.tab_off[b0]);  // values before this batch
  load_tile_meta(d, M, f0, n, r0);
  __syncthreads();
  for (int g8 = 0; g8 < P; g8 += CP) {
    for (int e = threadIdx.x; e < T * CP; e += 256) {
      const int k = e / CP, pt = e % CP;
      const int fl = M.order[k];
      double f = 0.0, fx = 0.0, fy = 0.0, fz = 0.0;
      const int g = g8 + pt;
      if (M.nint[fl] > 0 && g < P) tab_meta(d, M, fl, d.px[g0 + g], d.py[g0 + g], d.pz[g0 + g], f, fx, fy, fz);
      st[(0 * CP + pt) * SR + fl] = f;
      st[(1 * CP + pt) * SR + fl] = fx;
      st[(2 * CP + pt) * SR + fl] = fy;
      st[(3 * CP + pt) * SR + fl] = fz;
    }
    __syncthreads();
    // (component, point) rows of the tile's functions: 256 threads = 4 rows x 64 functions
    for (int e = threadIdx.x; e < nq * CP * T; e += 256) {
      const int fl = e % T, row = e / T;
      const int q = row / CP, pt = row % CP;
      const int g = g8 + pt;
      if (fl < nrow && g < P) {
        const double x = st[(q * CP + pt) * SR + fl];
        const int64_t o = (int64_t)g * n + r0 + fl;
        if (HILO) {
          float *of = static_cast<float *>(out) + 2 * (base + q * plane);
          const float hi = (float)x;
          of[o] = hi;
          of[plane + o] = (float)(x - (double)hi);
        } else {
          static_cast<double *>(out)[base + q * plane + o] = x;
        }
      }
    }
    __syncthreads();  // st consumed
  }
}

// ---------------------------------------------------------------------------
// Operand panels.  Batch b's panel holds phi, d/dx, d/dy, d/dz of its
// functions at its points, padded to Pp = pad16(P) points and np = pad16(n)
// functions (zeros in the padding), in a 4-point-interleaved layout:
//     element (q, pt, i) at ((q * Pp/4 + pt/4) * np + i) * 4 + pt % 4.
// A 64-lane MFMA operand slice (16 functions x 4 points) is then one
// contiguous 512-byte run, for the forward (functions as rows) and, in
// 128-byte runs, for the adjoint (points as rows).
// ---------------------------------------------------------------------------

__global__ void k_zero_u32(unsigned *p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

// w_g v_g for every active point (batch order).
__global__ void k_om(DevPlan d, const double *v, double *om) {
  const int64_t n = d.n_active;
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n; g += (int64_t)gridDim.x * blockDim.x)
    om[g] = d.pw[g] * v[d.perm[g]];
}

// Panel kinds:
//   PK_F64:   phi, d/dx, d/dy, d/dz in FP64 (4 planes of Pp np doubles)
//   PK_HS:    phi and psi = u phi / 2 in FP64 (2 planes)
//   PK_F32:   phi in FP64 (1 plane), then sqrt|w v| times d/dx, d/dy, d/dz
//             (formed in FP64) as FP32 planes (Pp np floats each) after it
//   PK_SPLIT: phi in FP64, then d/dx, d/dy, d/dz as FP32 hi planes fl32(x)
//             and the three lo planes fl32(x - hi)
//   PK_BF16:  phi in FP64 (1 plane), then the BF16 region: for component q
//             and split part t of sqrt|w v| times the gradient (formed in
//             FP64), plane 3 q + t of (Pp / 8) point octets x np functions x
//             8 points (16 bytes per function and octet)
// The FP64 and FP32 planes use the 4-point interleave above (FP32 planes
// counted in floats).
enum { PK_F64 = 0, PK_HS = 1, PK_F32 = 2, PK_SPLIT = 3, PK_BF16 = 4 };

// BF16 (8 significant bits) three-way split of two values a, b at once:
// each is rounded to FP32, and each part is the BF16 nearest (ties to even)
// to what the previous parts leave; the remainders are exact in FP32, so
// |x - x1 - x2 - x3| <= (2^-24 + 2^-24) |x|.  Part k of both values comes
// as one word wk (a in the low half, b in the high half), from one packed
// conversion per part.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ void split3_bf16x2(double a, double b, uint32_t &w1, uint32_t &w2, uint32_t &w3) {
  const float fa = (float)a, fb = (float)b;
  w1 = pack_bf16(fa, fb);
  const float ra = fa - __uint_as_float(w1 << 16), rb = fb - __uint_as_float(w1 & 0xffff0000u);
  w2 = pack_bf16(ra, rb);
  w3 = pack_bf16(ra - __uint_as_float(w2 << 16), rb - __uint_as_float(w2 & 0xffff0000u));
}

// LDS accesses of a wave's lanes before this are ordered before those after it,
// for the compiler (the hardware runs a wave's LDS accesses in order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave (a workgroup of its own: nothing is shared) per (batch, T / sub
// functions, 64 points), one point per lane.  All lanes work on the same
// function, so a shell's interval search, table read and cubic are done once
// for its 2 l + 1 functions, no branch diverges and the functions' data come
// from scalar registers (lane k holds the wave's function k); the table entry
// of the next shell is fetched while this one's rows are formed.  The values
// of neighbouring panel rows are staged in LDS and written out as whole
// 128-byte lines: four rows of an FP64 plane, eight of an FP32 or BF16 plane.
// Bound by the writes: 10.9 GB of FP64 panels (120 atoms, 2.2 M points) take
// 2.05 ms, 5.3 TB/s (a fill reaches 6.6), 0.9 ms without the stores; tiles of 64
// functions staged by a workgroup, every function on its own, took 2.43 ms.
// The FP32 kind 1.07 -> 0.85 ms (48 atoms), BF16 2.51 -> 1.68 ms, H/S 1.93 ->
// 1.16 ms.  What did not reach this: 32-byte stores straight from the lanes
// (4.9 ms: 16 requests to L2 each), rows cut at the atoms (2.85 ms: a line
// that two workgroups write is written twice), 64-byte runs of the BF16 planes
// (2.85 ms).
// Points P .. Pp - 1 and rows n .. np - 1 are written as zeros.
// the staged bytes are written and read as different types
typedef double stage_f64 __attribute__((may_alias));
typedef float stage_f32 __attribute__((may_alias));
typedef uint16_t stage_u16 __attribute__((may_alias));
typedef u32x4 stage_u32x4 __attribute__((may_alias));
constexpr int PR8 = 576, PR4 = 272, PR2 = 144;  // bytes of a staged row: 64 values and a pad against bank conflicts
constexpr int panel_stage(int kind) {           // staged bytes per wave: four rows of the FP64 planes, eight of the others
  return kind == PK_F64   ? 16 * PR8
         : kind == PK_HS  ? 8 * PR8
         : kind == PK_F32 ? 4 * PR8 + 24 * PR4
         : kind == PK_SPLIT ? 4 * PR8 + 48 * PR4
                            : 4 * PR8 + 72 * PR2;
}
template <int KIND>
__global__ __launch_bounds__(64, 3) void k_panel(DevPlan d, const WorkItem *tiles, int64_t t0, int64_t wg0, int sub,
                                              int npb, double *panel, const double *om) {
  __shared__ __attribute__((aligned(16))) unsigned char st[panel_stage(KIND)];
  // neighbouring waves (of one batch) on one XCD
  const int64_t bid = wg0 + xcd_map(blockIdx.x, gridDim.x), pos = bid / npb;
  const int p0 = 64 * (int)(bid % npb);
  const WorkItem it = tiles[t0 + pos / sub];
  const int b = it.batch, rows = T / sub;
  const int g0 = d.batch_pt_off[b], P = d.batch_pt_off[b + 1] - g0;
  const int f0 = d.batch_fn_off[b], n = d.batch_fn_off[b + 1] - f0;
  const int r0 = it.ti * T + (int)(pos % sub) * rows;
  const int Pp = (int)pad16(P), np = (int)pad16(n);
  if (r0 >= np || p0 >= Pp) return;
  const int r1 = r0 + rows < np ? r0 + rows : np, rn = r1 < n ? r1 : n;  // rows written; of functions
  const int lane = threadIdx.x;
  double *pb = panel + d.panel_off[b];
  const int64_t plane = (int64_t)Pp * np;
  constexpr int NQ = KIND == PK_HS ? 2 : KIND == PK_F64 ? 4 : 1;  // FP64 planes
  const FnData fd = fn_data<KIND == PK_HS>(d, f0, n, r0);
  const int pt = p0 + lane;
  const bool live = pt < P;
  const int g = g0 + (live ? pt : 0);
  const double px = d.px[g], py = d.py[g], pz = d.pz[g];
  double sw = 0.0;
  if (KIND == PK_F32 || KIND == PK_BF16) sw = live ? sqrt(fabs(om[g])) : 0.0;
  constexpr int S4 = 4 * NQ * PR8, N4 = KIND == PK_F32 ? 3 : KIND == PK_SPLIT ? 6 : 0;  // FP32 planes staged from S4 on
  constexpr int S2 = 4 * NQ * PR8, N2 = KIND == PK_BF16 ? 9 : 0;                         // BF16 planes from S2 on
  // writes the staged group of four (panel rows 4 r4 .. 4 r4 + 3), by global
  // stores: 16-byte buffer stores with the offset in a scalar register have
  // written registers that the next instructions had already reused
  auto flush = [&](int r4) {
    // every lane has staged its values: the barrier (no instruction) also
    // keeps the compiler from running lanes with different radial branches
    // through here apart
    wave_sync();
    {
      // FP64 planes: 8 quads of four rows per store, 16 bytes per lane
      const int row = (lane >> 1) & 3, qd = lane >> 3;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t vo = ((uint32_t)(8 * h + qd) * np + row) * 32u + 16u * (lane & 1);
        if (p0 + 32 * h + 4 * qd < Pp) {
#pragma unroll
          for (int q = 0; q < NQ; ++q)
            *reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(pb + q * plane + (int64_t)p0 * np + r4 * 16) + vo) =
                *reinterpret_cast<const stage_u32x4 *>(st + (4 * q + row) * PR8 + (8 * h + qd) * 32 + 16 * (lane & 1));
        }
      }
    }
    if (N4 > 0 && (r4 & 1)) {
      // FP32 planes: 8 quads of eight rows per store
      const int row = lane & 7, qd = lane >> 3;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t vo = ((uint32_t)(8 * h + qd) * np + row) * 16u;
        if (p0 + 32 * h + 4 * qd < Pp) {
#pragma unroll
          for (int q = 0; q < N4; ++q)
            *reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(reinterpret_cast<float *>(pb + plane) + q * plane +
                                                                (int64_t)p0 * np + (r4 >> 1) * 32) + vo) =
                *reinterpret_cast<const stage_u32x4 *>(st + S4 + (8 * q + row) * PR4 + (8 * h + qd) * 16);
        }
      }
    }
    if (N2 > 0 && (r4 & 1)) {
      // BF16 planes: 8 octets of eight rows per store
      const int row = lane & 7, oc = lane >> 3;
      const uint32_t vo = ((uint32_t)oc * np + row) * 16u;
      if (p0 + 8 * oc < Pp) {
#pragma unroll
        for (int q = 0; q < N2; ++q)
          *reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(reinterpret_cast<uint16_t *>(pb + plane) + q * plane +
                                                              (int64_t)p0 * np + (r4 >> 1) * 64) + vo) =
              *reinterpret_cast<const stage_u32x4 *>(st + S2 + (8 * q + row) * PR2 + oc * 16);
      }
    }
    wave_sync();  // the rows are read
  };
  // stages the values of panel row i: phi, then psi (H/S) or the gradient
  auto put = [&](int i, double f, double fx, double fy, double fz) {
    if (i < r0 || i >= r1) return;  // of a shell that another wave shares
    const double x[4] = {f, fx, fy, fz};
    const int row = i & 3, row8 = i & 7;
#pragma unroll
    for (int q = 0; q < NQ; ++q) *reinterpret_cast<stage_f64 *>(st + (4 * q + row) * PR8 + 8 * lane) = x[q];
    if (KIND == PK_F32 || KIND == PK_SPLIT) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const float hi = KIND == PK_F32 ? (float)(sw * x[q + 1]) : (float)x[q + 1];
        *reinterpret_cast<stage_f32 *>(st + S4 + (8 * q + row8) * PR4 + 4 * lane) = hi;
        if (KIND == PK_SPLIT)
          *reinterpret_cast<stage_f32 *>(st + S4 + (8 * (3 + q) + row8) * PR4 + 4 * lane) =
              (float)(x[q + 1] - (double)hi);
      }
    }
    if (KIND == PK_BF16) {
      uint32_t w[2][3];
      split3_bf16x2(sw * fx, sw * fy, w[0][0], w[0][1], w[0][2]);
      split3_bf16x2(sw * fz, 0.0, w[1][0], w[1][1], w[1][2]);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        *reinterpret_cast<stage_u16 *>(st + S2 + (8 * k + row8) * PR2 + 2 * lane) = (uint16_t)w[0][k];
        *reinterpret_cast<stage_u16 *>(st + S2 + (8 * (3 + k) + row8) * PR2 + 2 * lane) = (uint16_t)(w[0][k] >> 16);
        *reinterpret_cast<stage_u16 *>(st + S2 + (8 * (6 + k) + row8) * PR2 + 2 * lane) = (uint16_t)w[1][k];
      }
    }
    if (row == 3) flush(i >> 2);  // wave-uniform
  };
  walk_shells<KIND == PK_HS>(d, fd, r0, rn, px, py, pz, live, put);
  for (int i = rn; i < r1; ++i) put(i, 0.0, 0.0, 0.0, 0.0);
}

// V alone (the V part of F32 and SPLIT_F32, and V-only calls): one MFMA per
// row and column value, too little work per chunk to hide the next chunk's
// loads at two workgroups per CU: its 16-point chunks (33 KB of LDS) and 110
// VGPRs let four share a CU.
// Work item positions 0..nw-1 of a pass map to work items w0 + order[w0 + pos]
// (order != NULL: cost-sorted) or w0 + pos.  tickets == NULL: one workgroup
// per position; otherwise a persistent loop (next_item).
template <bool FAR, bool PERSIST>
__global__ __launch_bounds__(NT, 4) void k_contract_v(
    DevPlan d, const WorkItem *work, const int32_t *order, int64_t w0, int64_t nw, const double *om,
    const double *panel, double *staging, unsigned *tickets) {
  // Chunks of CH points in two LDS buffers, the next chunk's DMA in flight
  // while this one is multiplied (one barrier per chunk)
  constexpr int CH = 16;
  constexpr int RPQ = CH / 2;              // LDS rows: point pairs
  constexpr int BUFD = RPQ * DROW;         // doubles per chunk image
  __shared__ double sa[2 * BUFD], sb[2 * BUFD];
  __shared__ int64_t s_pos;
  int64_t pos = PERSIST ? next_item(tickets, nw, order != nullptr, &s_pos)
                        : (order ? (int64_t)blockIdx.x : xcd_map_runs(blockIdx.x, nw, 64));
  while (!PERSIST || pos < nw) {
  const int64_t wi = w0 + (order ? order[w0 + pos] : pos);
  const WorkItem it = work[wi];
  const int b = it.batch;
  const int g0 = d.batch_pt_off[b], P = d.batch_pt_off[b + 1] - g0;
  const int f0 = d.batch_fn_off[b], n = d.batch_fn_off[b + 1] - f0;
  const int r0 = it.ti * T, c0 = it.tj * T;
  const int Pp = (int)pad16(P), np = (int)pad16(n);
  const double *pb = panel + d.panel_off[b];
  const int64_t plane = (int64_t)Pp * np;
  const int tid = threadIdx.x;
  // wave index as a scalar: conditions derived from it stay uniform
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li16 = lane & 15, lk = lane >> 4;
  int brow[4], bcol[4];
  bool act[4];
  wave_blocks(r0, c0, n, wave, brow, bcol, act);

  dbl4 acc[4];
#pragma unroll
  for (int sl = 0; sl < 4; ++sl) acc[sl] = dbl4{0.0, 0.0, 0.0, 0.0};
  // K steps go in pairs over 8 points: K index lk of the first step of the
  // pair is point 2 lk of the 8, of the second point 2 lk + 1 (one 16-byte
  // LDS read per operand gives a lane both).  w v at the points this lane's
  // K index visits in the next chunk, loaded a chunk ahead with the next
  // image's DMA, so that nothing consumed between the barrier and the last
  // MFMA of a chunk waits on loads in flight
  double omn[CH / 4];
  auto load_om = [&](int k) {
#pragma unroll
    for (int ks = 0; ks < CH / 4; ++ks) {
      const int pt = k + 8 * (ks >> 1) + 2 * lk + (ks & 1);
      omn[ks] = pt < P ? om[g0 + pt] : 0.0;
    }
  };
  load_om(0);
  dma_chunk<NT, CH, T, DROW, 1>(pb, plane, np, r0, 0, sa);
  dma_chunk<NT, CH, T, DROW, 1>(pb, plane, np, c0, 0, sb);
  for (int k0 = 0; k0 < Pp; k0 += CH) {
    const int bo = ((k0 / CH) & 1) * BUFD;  // this chunk's buffer
    __builtin_amdgcn_s_waitcnt(0);  // this thread's loads of this chunk have landed
    __syncthreads();                // ... everyone's; the previous chunk is consumed
    double omv[CH / 4];
#pragma unroll
    for (int ks = 0; ks < CH / 4; ++ks) omv[ks] = omn[ks];
    if (k0 + CH < Pp) {
      const int nbo = BUFD - bo;
      load_om(k0 + CH);
      dma_chunk<NT, CH, T, DROW, 1>(pb, plane, np, r0, (k0 + CH) >> 2, sa + nbo);
      dma_chunk<NT, CH, T, DROW, 1>(pb, plane, np, c0, (k0 + CH) >> 2, sb + nbo);
    }
    const double *ca = sa + bo, *cb = sb + bo;
#pragma unroll
    for (int kp = 0; kp < CH / 8; ++kp) {
      // image row 4 kp + lk holds points 8 kp + 2 lk and 8 kp + 2 lk + 1 of
      // the chunk; the row operand takes the weight w v there, as in k_forward
      const int row = 4 * kp + lk;
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) {
        if (!act[sl]) continue;  // wave-uniform
        const dbl2 ap = *reinterpret_cast<const dbl2 *>(&ca[row * DROW + 2 * (brow[sl] + li16)]);
        const dbl2 bp = *reinterpret_cast<const dbl2 *>(&cb[row * DROW + 2 * (bcol[sl] + li16)]);
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[sl] = mfma64(ap[h] * omv[2 * kp + h], bp[h], acc[sl]);
      }
    }
  }
  // write the computed blocks to the staged atom-pair blocks
#pragma unroll
  for (int sl = 0; sl < 4; ++sl) {
    if (!act[sl]) continue;  // wave-uniform
    const int rb = (r0 + brow[sl]) >> 4;
    stage_block<0, 1, FAR>(stage_rows(d, f0, n, rb, lk, staging), d, f0, n, rb, (c0 + bcol[sl]) >> 4, li16,
                      [&](int r, int) { return acc[sl][r]; });
  }
  if (!PERSIST) break;
  pos = next_item(tickets, nw, order != nullptr, &s_pos);
  }
}

// The plain FP64 baseline (precision F64_VALU): the five parts of a work
// item on the vector ALU, no matrix cores.  Same work items, FP64 panels,
// chunk DMA and staging as the other contractions; each thread owns a 4 x 4
// patch of the 64 x 64 tile (rows 4 (t / 16), columns 4 (t % 16)) and adds
// every point's ten products to its 80 FP64 sums with fused multiply-adds,
// point after point.  Patches in blocks no work item computes (below the
// diagonal, beyond n) skip the arithmetic.
__global__ __launch_bounds__(NT, 1) void k_contract_valu(DevPlan d, const WorkItem *work, const int32_t *order,
                                                         int64_t w0, int64_t nw, const double *om,
                                                         const double *panel, double *staging, unsigned *tickets) {
  (void)tickets;
  constexpr int NQ = 4, CH = 8, RPQ = CH / 2;
  constexpr int BUFD = NQ * RPQ * DROW;  // doubles per chunk image
  __shared__ double sa[2 * BUFD], sb[2 * BUFD];
  __shared__ double s_om[2][CH];
  // slot data of the tile's 64 rows and 64 columns for the epilogue, loaded
  // when the work item starts (slot -1: beyond n)
  __shared__ int s_fslot[2 * T], s_ffn[2 * T], s_fnf[2 * T];
  __shared__ int64_t s_frow[2 * T];
  const int64_t pos = order ? (int64_t)blockIdx.x : xcd_map(blockIdx.x, nw);
  const int64_t wi = w0 + (order ? order[w0 + pos] : pos);
  const WorkItem it = work[wi];
  const int b = it.batch;
  const int g0 = d.batch_pt_off[b], P = d.batch_pt_off[b + 1] - g0;
  const int f0 = d.batch_fn_off[b], n = d.batch_fn_off[b + 1] - f0;
  const int r0 = it.ti * T, c0 = it.tj * T;
  const int Pp = (int)pad16(P), np = (int)pad16(n);
  const double *pb = panel + d.panel_off[b];
  const int64_t plane = (int64_t)Pp * np;
  const int tid = threadIdx.x;
  const int pr = 4 * (tid >> 4), pc = 4 * (tid & 15);  // the thread's patch (tile-local)
  const int rb = pr & ~15, cb = pc & ~15;
  const bool live = block_active(r0 + rb, c0 + cb, n);
  double acc[5][4][4];
#pragma unroll
  for (int q = 0; q < 5; ++q)
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[q][a][c] = 0.0;
  double omr = tid < CH && tid < P ? om[g0 + tid] : 0.0;  // 0 past the batch's points
  dma_chunk<NT, CH, T, DROW, NQ>(pb, plane, np, r0, 0, sa);
  dma_chunk<NT, CH, T, DROW, NQ>(pb, plane, np, c0, 0, sb);
  if (tid < 2 * T) {  // visible from the first chunk's barrier on
    const int lf = tid < T ? r0 + tid : c0 + tid - T;
    int64_t v = 0, ro = 0;
    if (lf < n) {
      v = d.loc_info[f0 + lf];
      ro = d.loc_rowoff[f0 + lf];
    }
    s_fslot[tid] = lf < n ? (int)(v & 0xFFFFF) : -1;
    s_ffn[tid] = (int)((v >> 20) & 0xFFFFF);
    s_fnf[tid] = (int)(v >> 40);
    s_frow[tid] = ro;
  }
  __builtin_amdgcn_s_waitcnt(0);
  if (tid < CH) s_om[0][tid] = omr;
  for (int k0 = 0; k0 < Pp; k0 += CH) {
    const int bi = (k0 / CH) & 1;
    __syncthreads();  // this chunk visible; the previous one consumed
    if (k0 + CH < Pp) {
      omr = tid < CH && k0 + CH + tid < P ? om[g0 + k0 + CH + tid] : 0.0;
      dma_chunk<NT, CH, T, DROW, NQ>(pb, plane, np, r0, (k0 + CH) >> 2, sa + (bi ^ 1) * BUFD);
      dma_chunk<NT, CH, T, DROW, NQ>(pb, plane, np, c0, (k0 + CH) >> 2, sb + (bi ^ 1) * BUFD);
    }
    if (live) {
      const double *ca = sa + bi * BUFD, *cbp = sb + bi * BUFD;
      for (int u = 0; u < RPQ; ++u) {  // point pairs of the chunk
        // component q of functions pr + a (rows) and pc + c (columns) at
        // points 2u, 2u + 1 (16 bytes each)
        dbl2 av[NQ][4], bv[NQ][4];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            av[q][a] = *reinterpret_cast<const dbl2 *>(&ca[(q * RPQ + u) * DROW + 2 * (pr + a)]);
            bv[q][a] = *reinterpret_cast<const dbl2 *>(&cbp[(q * RPQ + u) * DROW + 2 * (pc + a)]);
          }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const double w = s_om[bi][2 * u + h];
#pragma unroll
          for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const double x0 = av[0][a][h], x1 = av[1][a][h], x2 = av[2][a][h], x3 = av[3][a][h];
              const double y0 = w * bv[0][c][h], y1 = w * bv[1][c][h], y2 = w * bv[2][c][h], y3 = w * bv[3][c][h];
              acc[0][a][c] = fma(x0, y0, acc[0][a][c]);
              acc[1][a][c] = fma(x1, y1, fma(x2, y2, fma(x3, y3, acc[1][a][c])));
              acc[2][a][c] = fma(x2, y3, fma(-x3, y2, acc[2][a][c]));
              acc[3][a][c] = fma(x3, y1, fma(-x1, y3, acc[3][a][c]));
              acc[4][a][c] = fma(x1, y2, fma(-x2, y1, acc[4][a][c]));
            }
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0);  // the next chunk's images and w v have landed
    if (k0 + CH < Pp && tid < CH) s_om[bi ^ 1][tid] = omr;
  }
  if (!live) return;
  const double cp = d.cprime;
  const bool upper = r0 + rb < c0 + cb;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int lj = c0 + pc + c;
    if (lj >= n) continue;
    const int cj = lj - c0 + T;
    const SlotInfo sj{s_fslot[cj], s_ffn[cj], s_fnf[cj], s_frow[cj]};
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const int li = r0 + pr + a;
      if (li >= n) continue;
      const int ri = li - r0;
      const SlotInfo si{s_fslot[ri], s_ffn[ri], s_fnf[ri], s_frow[ri]};
      double vals[5];
      vals[0] = acc[0][a][c];
#pragma unroll
      for (int q = 1; q < 5; ++q) vals[q] = cp * acc[q][a][c];
      stage_store<0, 5>(staging, si, sj, li, lj, upper, vals);
    }
  }
}

// The four W parts on FP32 MFMA (precisions F32 and SPLIT_F32), from the FP32
// gradient planes of a PK_F32 / PK_SPLIT panel; V runs beside it on FP64
// (k_contract_v).  Same work items, wave blocks and staging as
// k_contract_v.  F32: both operands are sqrt|w v| times the gradient (formed in
// FP64, rounded to FP32 once in the panel), the row operand with the sign of
// w v.  Per 16 points, every element's FP32 partial sum (of at most 48
// products: 16 points x 3) is converted to FP64 and added to an FP64 running
// sum, then restarted from zero, so FP32 rounding never accumulates beyond
// one 16-point chunk: with unit roundoff u = 2^-24 each element's error is at
// most gamma_52 = 52 u / (1 - 52 u) times the sum over all points of the
// magnitudes of its terms (two operands rounded to FP32, 48 products and
// additions), plus FP64 rounding and the loss of relative precision of values
// below FP32's normal range (the far tails of tight functions).  SPLIT: each
// operand x enters as hi = fl32(x) and lo = fl32(x - hi) (the column operand
// w v x formed in FP64 and split again), and every product as
// hi hi + hi lo + lo hi (three FP32 MFMAs): the operands' rounding drops to
// about 2^-48, and a 16-point partial sum holds up to 144 products
// (gamma_150).
template <bool SPLIT, bool FAR, bool PERSIST>
__global__ __launch_bounds__(NT, 2) void k_contract_w(DevPlan d, const WorkItem *work, const int32_t *order,
                                                      int64_t w0, int64_t nw, const double *om,
                                                      const double *panel, double *staging, unsigned *tickets) {
  // Chunks of CH points; an image row is one point quad of 64 functions
  // (1 KB of floats, in the panel's own order: element (pt, f) of the quad at
  // 4 f + pt % 4), rows (component q, quad) for q = 0..2 (d/dx, d/dy, d/dz),
  // then, for SPLIT, the same rows of the lo planes.
  constexpr int CH = SPLIT ? 8 : 16;
  constexpr int NQR = CH / 4;                  // quads per chunk
  constexpr int NPL = SPLIT ? 6 : 3;           // FP32 planes read
  constexpr int ROWF = 4 * T;                  // floats per image row
  constexpr int BUFF = NPL * NQR * ROWF;       // floats per chunk image
  constexpr int FLUSH = 16;                    // points per FP32 partial sum
  __shared__ __attribute__((aligned(16))) float fa[2 * BUFF], fb[2 * BUFF];
  __shared__ int64_t s_pos;
  int64_t pos = PERSIST ? next_item(tickets, nw, order != nullptr, &s_pos)
                        : (order ? (int64_t)blockIdx.x : xcd_map_runs(blockIdx.x, nw, 64));
  while (!PERSIST || pos < nw) {
  const int64_t wi = w0 + (order ? order[w0 + pos] : pos);
  const WorkItem it = work[wi];
  const int b = it.batch;
  const int g0 = d.batch_pt_off[b], P = d.batch_pt_off[b + 1] - g0;
  const int f0 = d.batch_fn_off[b], n = d.batch_fn_off[b + 1] - f0;
  const int r0 = it.ti * T, c0 = it.tj * T;
  const int Pp = (int)pad16(P), np = (int)pad16(n);
  const int64_t fplane = (int64_t)Pp * np;
  const float *pf = reinterpret_cast<const float *>(panel + d.panel_off[b] + fplane);
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li16 = lane & 15, lk = lane >> 4;
  int brow[4], bcol[4];
  bool act[4];
  wave_blocks(r0, c0, n, wave, brow, bcol, act);

  flt4 accf[4][4];   // FP32 partial sums of the current 16 points
  dbl4 accw[4][4];   // FP64 running sums
#pragma unroll
  for (int sl = 0; sl < 4; ++sl)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      accf[sl][q] = flt4{0.f, 0.f, 0.f, 0.f};
      accw[sl][q] = dbl4{0.0, 0.0, 0.0, 0.0};
    }
  // LDS DMA of one chunk of 64 functions from row0 (a tile): image row r =
  // (plane pl, quad qd) is the 1 KB run of plane pl (hi d/dx, d/dy, d/dz,
  // then the lo planes) at point quad quad0 + qd, 16 bytes (4 points of one
  // function) per lane.  Functions at or beyond np are not loaded (their
  // blocks are never multiplied).
  auto dma = [&](int row0, int quad0, float *dst) {
    const bool ok = row0 + lane < np;
#pragma unroll
    for (int k = 0; k < NPL * NQR / 4; ++k) {
      const int r = wave + 4 * k;
      const int pl = r / NQR, qd = r % NQR;
      if (ok)
        __builtin_amdgcn_global_load_lds(
            (const void *)(pf + (int64_t)pl * fplane + ((int64_t)(quad0 + qd) * np + row0 + lane) * 4),
            (lds_void *)(dst + r * ROWF), 16, 0, 0);
    }
  };
  // w v at the points this lane's K index visits in the next chunk: points
  // 4 ks + lk (SPLIT), or the four points of quad lk (otherwise)
  double omn[CH / 4];
  auto load_om = [&](int k) {
#pragma unroll
    for (int ks = 0; ks < CH / 4; ++ks) {
      const int pt = SPLIT ? k + 4 * ks + lk : k + 4 * lk + ks;
      omn[ks] = pt < P ? om[g0 + pt] : 0.0;
    }
  };
  load_om(0);
  dma(r0, 0, fa);
  dma(c0, 0, fb);
  for (int k0 = 0; k0 < Pp; k0 += CH) {
    const int bo = ((k0 / CH) & 1) * BUFF;
    __builtin_amdgcn_s_waitcnt(0);  // this thread's loads of this chunk have landed
    __syncthreads();                // ... everyone's; the previous chunk is consumed
    double omv[CH / 4];
#pragma unroll
    for (int ks = 0; ks < CH / 4; ++ks) omv[ks] = omn[ks];
    if (k0 + CH < Pp) {
      load_om(k0 + CH);
      dma(r0, (k0 + CH) >> 2, fa + BUFF - bo);
      dma(c0, (k0 + CH) >> 2, fb + BUFF - bo);
    }
    const float *ca = fa + bo, *cb = fb + bo;
    if constexpr (!SPLIT) {
      // The panel holds sqrt|w v| times the gradient, so each product is
      // w v times two gradient components once the row operand takes the
      // sign of w v.  MFMA m of the chunk sums over points 4 lk + m (K index
      // lk): one 16-byte LDS read per operand gives a lane all four.
      uint32_t sgn[4];
#pragma unroll
      for (int m = 0; m < 4; ++m)
        sgn[m] = (uint32_t)((uint64_t)__double_as_longlong(omv[m]) >> 32) & 0x80000000u;
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) {
        if (!act[sl]) continue;  // wave-uniform
        flt4 a4[3], b4[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          a4[q] = *reinterpret_cast<const flt4 *>(&ca[(q * NQR + lk) * ROWF + 4 * (brow[sl] + li16)]);
          b4[q] = *reinterpret_cast<const flt4 *>(&cb[(q * NQR + lk) * ROWF + 4 * (bcol[sl] + li16)]);
#pragma unroll
          for (int m = 0; m < 4; ++m) a4[q][m] = __uint_as_float(__float_as_uint(a4[q][m]) ^ sgn[m]);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          // parts: Ws = dx dx + dy dy + dz dz; Wso_x = dy dz - dz dy;
          // Wso_y = dz dx - dx dz; Wso_z = dx dy - dy dx (row x column)
          accf[sl][0] = mfma32(a4[0][m], b4[0][m], accf[sl][0]);
          accf[sl][1] = mfma32(a4[1][m], b4[2][m], accf[sl][1]);
          accf[sl][2] = mfma32(a4[2][m], b4[0][m], accf[sl][2]);
          accf[sl][3] = mfma32(a4[0][m], b4[1][m], accf[sl][3]);
          accf[sl][0] = mfma32(a4[1][m], b4[1][m], accf[sl][0]);
          accf[sl][1] = mfma32(-a4[2][m], b4[1][m], accf[sl][1]);
          accf[sl][2] = mfma32(-a4[0][m], b4[2][m], accf[sl][2]);
          accf[sl][3] = mfma32(-a4[1][m], b4[0][m], accf[sl][3]);
          accf[sl][0] = mfma32(a4[2][m], b4[2][m], accf[sl][0]);
        }
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < CH / 4; ++ks) {
        const double omk = omv[ks];
#pragma unroll
        for (int sl = 0; sl < 4; ++sl) {
          if (!act[sl]) continue;  // wave-uniform
          // A[i][k] = component q of row function brow + i at point 4 ks + k
          // (hi and lo); B[k][j] = w v times component q of column function
          // bcol + j there, formed in FP64 from hi + lo and split again
          float ah[3], bh[3], al[3], bl[3];
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            ah[q] = ca[(q * NQR + ks) * ROWF + 4 * (brow[sl] + li16) + lk];
            const float bx = cb[(q * NQR + ks) * ROWF + 4 * (bcol[sl] + li16) + lk];
            al[q] = ca[((3 + q) * NQR + ks) * ROWF + 4 * (brow[sl] + li16) + lk];
            const float bxl = cb[((3 + q) * NQR + ks) * ROWF + 4 * (bcol[sl] + li16) + lk];
            const double x = omk * ((double)bx + (double)bxl);
            bh[q] = (float)x;
            bl[q] = (float)(x - (double)bh[q]);
          }
          // the same products, each as hi hi + hi lo + lo hi
#define W32(ACC, AI, BI, SG)              \
  ACC = mfma32(SG ah[AI], bh[BI], ACC);   \
  ACC = mfma32(SG ah[AI], bl[BI], ACC);   \
  ACC = mfma32(SG al[AI], bh[BI], ACC);
          W32(accf[sl][0], 0, 0, +)
          W32(accf[sl][1], 1, 2, +)
          W32(accf[sl][2], 2, 0, +)
          W32(accf[sl][3], 0, 1, +)
          W32(accf[sl][0], 1, 1, +)
          W32(accf[sl][1], 2, 1, -)
          W32(accf[sl][2], 0, 2, -)
          W32(accf[sl][3], 1, 0, -)
          W32(accf[sl][0], 2, 2, +)
#undef W32
        }
      }
    }
    if (((k0 + CH) % FLUSH) == 0 || k0 + CH >= Pp) {
      // the 16-point FP32 partial sums join the FP64 running sums
#pragma unroll
      for (int sl = 0; sl < 4; ++sl) {
        if (!act[sl]) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
          for (int r = 0; r < 4; ++r) accw[sl][q][r] += (double)accf[sl][q][r];
          accf[sl][q] = flt4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
  }
  const double cp = d.cprime;
#pragma unroll
  for (int sl = 0; sl < 4; ++sl) {
    if (!act[sl]) continue;  // wave-uniform
    const int rb = (r0 + brow[sl]) >> 4;
    stage_block<1, 5, FAR>(stage_rows<true>(d, f0, n, rb, lk, staging), d, f0, n, rb, (c0 + bcol[sl]) >> 4, li16,
                      [&](int r, int q) { return cp * accw[sl][q - 1][r]; });
  }
  if (!PERSIST) break;
  pos = next_item(tickets, nw, order != nullptr, &s_pos);
  }
}

// BF16X3 precision: V on FP64 MFMA and the four W parts on BF16 MFMA with
// three-way split operands (PK_BF16 panels), in one kernel.  One workgroup
// per column half (32 columns) of a work item's 64 x 64 tile; wave w takes
// the 16-row block w against the half's two 16-column blocks, so each A
// operand it reads serves both.  Per 16-point chunk the four images (FP64 phi
// and the BF16 parts of sqrt|w v| times the gradient, of rows and of
// columns) arrive by LDS DMA, double-buffered, with w v of the chunk's
// points.  The row operand takes the sign of w v (its BF16 sign bits
// flipped), so each product is w v times the two gradient components.
// W products: a b ~ a1 b1 + a2 b1 + a1 b2 + a1 b3 + a2 b2 + a3 b1 (the terms
// of order 2^-16 and above), three MFMAs of K = 32 per component pair: the
// K index runs over two slots of the chunk's 16 points, slot 0 (lanes with
// lk < 2) holding one part and slot 1 another ([a1|a2] x [b1|b1],
// [a1|a1] x [b2|b3], [a2|a3] x [b2|b1]).  Dropped terms and split remainders
// are below 3 2^-23 |a b|.  The spin-orbit parts keep their positive and
// negative products in separate FP32 sums (no operand is negated).  Each
// chunk's FP32 sums start from zero and are added into FP64 running sums
// (the spin-orbit pair as their FP32 difference).
//
// Bound: LDS, 33 KB of operand reads per wave and chunk for 62 MFMAs (1.0 of
// their 1.4 thousand cycles, the barrier aside): 120 atoms 8.6 ms, the MFMAs
// alone 2.6.  Results staged in LDS for coalesced stores took 1700 vector
// instructions per item, 9.2 ms.  Row operands straight to registers, with
// half of the LDS reads, were no faster at two waves per SIMD (8.6 ms,
// prefetched, 8.8 not): latency takes over.
template <bool PERSIST>
__global__ __launch_bounds__(NT, 2) void k_contract_b3(DevPlan d, const WorkItem *work, const int32_t *order,
                                                       int64_t w0, int64_t nw, const double *om,
                                                       const double *panel, double *staging, unsigned *tickets) {
  constexpr int CH = 16;            // points per chunk
  constexpr int RBF = 18 * 64;      // 16-byte items of the row BF16 image: 18 rows (plane, octet) x 64 functions
  constexpr int CBF = 18 * 32;      // ... of the column image (32 functions)
  constexpr int RD = 8 * DROW;      // doubles of the row phi image: 8 point pairs x 64 functions x 2
  constexpr int CDW = 2 * 32;       // doubles per row of the column phi image
  constexpr int CD = 8 * CDW;
  // chunk images (double-buffered)
  constexpr int IMG_BYTES = 2 * 16 * (RBF + CBF) + 2 * 8 * (RD + CD);
  __shared__ __attribute__((aligned(16))) unsigned char smem[IMG_BYTES];
  u32x4(*sr)[RBF] = reinterpret_cast<u32x4(*)[RBF]>(smem);
  u32x4(*sc)[CBF] = reinterpret_cast<u32x4(*)[CBF]>(smem + 2 * 16 * RBF);
  double(*dr)[RD] = reinterpret_cast<double(*)[RD]>(smem + 2 * 16 * (RBF + CBF));
  double(*dc)[CD] = reinterpret_cast<double(*)[CD]>(smem + 2 * 16 * (RBF + CBF) + 2 * 8 * RD);
  __shared__ double som[2][CH];
  __shared__ int64_t s_pos;
  const int64_t npos = 2 * nw;
  int64_t pos = PERSIST ? next_item(tickets, npos, order != nullptr, &s_pos)
                        : (order ? (int64_t)blockIdx.x : xcd_map_runs(blockIdx.x, npos, 64));
  while (!PERSIST || pos < npos) {
  const int half = (int)(pos & 1);
  const int64_t wi = w0 + (order ? order[w0 + (pos >> 1)] : (pos >> 1));
  const WorkItem it = work[wi];
  const int b = it.batch;
  const int f0 = d.batch_fn_off[b], n = d.batch_fn_off[b + 1] - f0;
  if (it.tj * T + 32 * half < n) {  // workgroup-uniform: the half has columns
  const int g0 = d.batch_pt_off[b], P = d.batch_pt_off[b + 1] - g0;
  const int r0 = it.ti * T, c0 = it.tj * T + 32 * half;
  const int Pp = (int)pad16(P), np = (int)pad16(n);
  const double *pb = panel + d.panel_off[b];
  const int64_t fplane = (int64_t)Pp * np, noct = Pp >> 3;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lk = lane >> 4;
  const int rb = 16 * wave;  // this wave's row block (tile-local)
  bool act[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) act[c] = block_active(r0 + rb, c0 + 16 * c, n);

  // the chunk of 16 points from k0 into buffer bf, by buffer loads straight
  // into LDS: the batch's panel is one buffer, each lane's offset is fixed for
  // the work item and the chunk and image row go into the scalar offset.
  // Lanes whose function lies at or beyond np load nothing.
  const __amdgpu_buffer_rsrc_t prs =
      __builtin_amdgcn_make_buffer_rsrc((void *)pb, (short)0, (int)(26 * fplane), 0x00020000);
  // lanes whose function lies at or beyond np take an offset past the
  // buffer's range: the load is issued by every lane and reads nothing there
  const bool okr = r0 + lane < np, okc = c0 + (lane & 31) < np;
  constexpr uint32_t OOB = 0x80000000u;
  const uint32_t vrow = okr ? lane * 16u : OOB;
  const uint32_t vcol = okc ? (lane & 31) * 16u + (lane >> 5) * (uint32_t)np * 16u : OOB;
  const uint32_t vprow = okr ? lane * 32u : OOB, vpcol = okc ? (lane & 31) * 32u + (lane >> 5) * 16u : OOB;
  auto dma = [&](int k0, int bf) {
    const int og = k0 >> 3;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
      const int k = wave + 4 * i;  // wave-uniform
      if (k < 18) {  // row image row (plane k / 2, octet k % 2), 64 functions
        const uint32_t so = 8u * (uint32_t)fplane + (uint32_t)((((k >> 1) * noct + og + (k & 1)) * np + r0) * 16);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(prs, (lds_void *)(&sr[bf][k * 64]), 16, vrow, so, 0, 0);
      } else if (k < 27) {  // column image rows (plane, octet 0) and (plane, octet 1), 32 functions each
        const int pl = k - 18;
        const uint32_t so = 8u * (uint32_t)fplane + (uint32_t)(((pl * noct + og) * np + c0) * 16);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(prs, (lds_void *)(&sc[bf][pl * 64]), 16, vcol, so, 0, 0);
      }
    }
    // FP64 phi: image row u = point pair u of the chunk (16 bytes per function)
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // rows: two point pairs per wave
      const int u = wave + 4 * h;
      const uint32_t so = (uint32_t)(((((k0 >> 2) + (u >> 1)) * np + r0) * 4 + 2 * (u & 1)) * 8);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(prs, (lds_void *)(&dr[bf][u * DROW]), 16, vprow, so, 0, 0);
    }
    {  // columns: point pairs 2 w and 2 w + 1 (one quad) per wave
      const uint32_t so = (uint32_t)(((((k0 >> 2) + wave) * np + c0) * 4) * 8);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(prs, (lds_void *)(&dc[bf][2 * wave * CDW]), 16, vpcol, so, 0, 0);
    }
  };

  dbl4 accw[2][4];   // FP64 running sums of Ws, Wso_x, Wso_y, Wso_z
  dbl4 accv[2];      // V
#pragma unroll
  for (int c = 0; c < 2; ++c) {
#pragma unroll
    for (int q = 0; q < 4; ++q) accw[c][q] = dbl4{0.0, 0.0, 0.0, 0.0};
    accv[c] = dbl4{0.0, 0.0, 0.0, 0.0};
  }
  double omr = tid < CH && tid < P ? om[g0 + tid] : 0.0;  // 0 past the batch's points
  dma(0, 0);
  __builtin_amdgcn_s_waitcnt(0);
  if (tid < CH) som[0][tid] = omr;
  const int slot = lk >> 1, oc = lk & 1;
  // split parts of the A and B operands of MFMA s for this lane's slot
  const int ta0 = slot ? 1 : 0, ta2 = slot ? 2 : 1;  // A: s = 0 [1|2], s = 1 [1|1], s = 2 [2|3]
  const int tb1 = slot ? 2 : 1, tb2 = slot ? 0 : 1;  // B: s = 0 [1|1], s = 1 [2|3], s = 2 [2|1]
  for (int k0 = 0; k0 < Pp; k0 += CH) {
    const int bi = (k0 / CH) & 1;
    __syncthreads();  // this chunk's images and w v visible; the previous chunk is consumed
    if (k0 + CH < Pp) {
      omr = tid < CH && k0 + CH + tid < P ? om[g0 + k0 + CH + tid] : 0.0;
      dma(k0 + CH, bi ^ 1);
    }
    // the chunk's products for the active column blocks (a compile-time set:
    // both, or one on diagonal and edge tiles), as straight-line code
    auto chunk = [&](auto a0c, auto a1c) {
      constexpr bool ACT[2] = {decltype(a0c)::value, decltype(a1c)::value};
      // V: four K steps of 4 points on FP64 MFMA, in pairs over 8 points as
      // in the FP64 path (the same order)
#pragma unroll
      for (int kp = 0; kp < 2; ++kp) {
        const int row = 4 * kp + lk;
        const dbl2 ap = *reinterpret_cast<const dbl2 *>(&dr[bi][row * DROW + 2 * (rb + l16)]);
        dbl2 bp[2];
#pragma unroll
        for (int c = 0; c < 2; ++c)
          if (ACT[c]) bp[c] = *reinterpret_cast<const dbl2 *>(&dc[bi][row * CDW + 2 * (16 * c + l16)]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const double apw = ap[h] * som[bi][8 * kp + 2 * lk + h];
#pragma unroll
          for (int c = 0; c < 2; ++c)
            if (ACT[c]) accv[c] = mfma64(apw, bp[c][h], accv[c]);
        }
      }
      // W: this chunk's FP32 sums, Ws then (+, -) of Wso_x, Wso_y, Wso_z
      flt4 accf[2][7];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < 7; ++q) accf[c][q] = flt4{0.f, 0.f, 0.f, 0.f};
      // the sign of w v at this lane's 8 points (octet oc), on the BF16 sign
      // bits of the row operand
      u32x4 sgn;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const uint64_t ua = (uint64_t)__double_as_longlong(som[bi][8 * oc + 2 * m]);
        const uint64_t ub = (uint64_t)__double_as_longlong(som[bi][8 * oc + 2 * m + 1]);
        sgn[m] = ((uint32_t)(ua >> 48) & 0x8000u) | ((uint32_t)(ub >> 32) & 0x80000000u);
      }
      // A operands of the row block, all components and split pairs
      u32x4 fa[3][3];
#pragma unroll
      for (int qa = 0; qa < 3; ++qa) {
        const int base = rb + l16;
        fa[qa][0] = sr[bi][((3 * qa + ta0) * 2 + oc) * 64 + base] ^ sgn;
        fa[qa][1] = sr[bi][((3 * qa + 0) * 2 + oc) * 64 + base] ^ sgn;
        fa[qa][2] = sr[bi][((3 * qa + ta2) * 2 + oc) * 64 + base] ^ sgn;
      }
#pragma unroll
      for (int qb = 0; qb < 3; ++qb) {
        u32x4 gb[2][3];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          if (!ACT[c]) continue;
          const int base = 16 * c + l16;
          gb[c][0] = sc[bi][((3 * qb + 0) * 2 + oc) * 32 + base];
          gb[c][1] = sc[bi][((3 * qb + tb1) * 2 + oc) * 32 + base];
          gb[c][2] = sc[bi][((3 * qb + tb2) * 2 + oc) * 32 + base];
        }
        // FP32 sum of (row component qa, column component qb): Ws on the
        // diagonal; y z -> 1, z y -> 2, z x -> 3, x z -> 4, x y -> 5, y x -> 6
#pragma unroll
        for (int sp = 0; sp < 3; ++sp)
#pragma unroll
          for (int qa = 0; qa < 3; ++qa) {
            constexpr int MAP[3][3] = {{0, 5, 4}, {6, 0, 1}, {3, 2, 0}};
            const int t = MAP[qa][qb];
#pragma unroll
            for (int c = 0; c < 2; ++c)
              if (ACT[c]) accf[c][t] = mfma_bf16(fa[qa][sp], gb[c][sp], accf[c][t]);
          }
      }
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        if (!ACT[c]) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          accw[c][0][r] += (double)accf[c][0][r];
#pragma unroll
          for (int m = 0; m < 3; ++m) accw[c][1 + m][r] += (double)(accf[c][1 + 2 * m][r] - accf[c][2 + 2 * m][r]);
        }
      }
    };
    if (act[0] && act[1])
      chunk(std::true_type{}, std::true_type{});
    else if (act[0])
      chunk(std::true_type{}, std::false_type{});
    else if (act[1])
      chunk(std::false_type{}, std::true_type{});
    __builtin_amdgcn_s_waitcnt(0);  // the next chunk's images and w v have landed
    if (k0 + CH < Pp && tid < CH) som[bi ^ 1][tid] = omr;
  }
  // write the computed blocks to the staged atom-pair blocks
  if (act[0] || act[1]) {
    const double cp = d.cprime;
    const int rbk = (r0 + rb) >> 4;
    const StageRows s8 = stage_rows(d, f0, n, rbk, lk, staging), s4 = stage_rows<true>(d, f0, n, rbk, lk, staging);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if (!act[c]) continue;
      const int cbk = (c0 >> 4) + c;
      stage_block<0, 1>(s8, d, f0, n, rbk, cbk, l16, [&](int r, int) { return accv[c][r]; });
      stage_block<1, 5>(s4, d, f0, n, rbk, cbk, l16, [&](int r, int q) { return cp * accw[c][q - 1][r]; });
    }
  }
  }  // the half has columns
  if (!PERSIST) break;
  pos = next_item(tickets, npos, order != nullptr, &s_pos);
  }
}

// Batch-to-global sum for one pass: reduction entry r adds the staged blocks
// of pair red_pair[r] in batch order, one after another onto the running
// value (zero, or the stored value when a previous pass or ACCUMULATE left
// one).  The sum is a single sequential chain in batch order, so results
// repeat bit for bit and do not depend on how batches are split into passes.
// Workgroup (x, y) takes elements y NTR .. y NTR + NTR - 1 of entry x, one per
// thread (gridDim.y covers the largest entry), so the heavy atom pairs are
// spread over many workgroups instead of setting the kernel's tail; the
// loads of 32 incidences are issued together, those of the last ones 16 at a
// time.  Bound by those loads' latency on small plans and by HBM reads on large
// ones: against eight at a time 16.3 -> 13.1 us (3 atoms, 128 batches),
// 1.22 -> 1.20 ms (120 atoms), 1.09 -> 1.05 ms (H/S, 60 atoms).
constexpr int NTR = 256;  // threads of a k_reduce workgroup
__global__ __launch_bounds__(NTR) void k_reduce(DevPlan d, int64_t r0, const int32_t *red_pair,
                                                const uint8_t *red_first, const int64_t *red_inc_off,
                                                const int64_t *inc_src, const double *staging, double *store,
                                                int accumulate, int nq, unsigned part_mask) {
  __shared__ int64_t s_src[NTR];
  const int64_t r = r0 + blockIdx.x;
  const int p = red_pair[r];
  const int blk = d.pair_na[p] * d.pair_nb[p];
  const int m = nq * blk;  // parts 0 .. nq-1 of the staged blocks (the first nq of five)
  if ((int)blockIdx.y * NTR >= m) return;  // workgroup-uniform: past this entry's elements
  const int64_t k0 = red_inc_off[r], k1 = red_inc_off[r + 1];
  const bool add = accumulate || !red_first[r];
  const int64_t po = d.pair_off[p];
  const int e = blockIdx.y * NTR + threadIdx.x;
  const int q = e / blk;
  const bool own = e < m && ((part_mask >> q) & 1);
  double sum = own && add ? store[q * d.store_len + po + (e - q * blk)] : 0.0;
  for (int64_t kb = k0; kb < k1; kb += NTR) {
    const int nk = (int)(k1 - kb < NTR ? k1 - kb : NTR);
    __syncthreads();  // previous offsets consumed
    if (threadIdx.x < nk) s_src[threadIdx.x] = inc_src[kb + threadIdx.x];
    __syncthreads();
    int k = 0;
    for (; k + 32 <= nk; k += 32) {
      double a[32];
#pragma unroll
      for (int u = 0; u < 32; ++u) a[u] = e < m ? staging[s_src[k + u] + e] : 0.0;
#pragma unroll
      for (int u = 0; u < 32; ++u) sum += a[u];
    }
    for (; k < nk; k += 16) {  // the rest, also in flight together
      double a[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) a[u] = e < m && k + u < nk ? staging[s_src[k + u] + e] : 0.0;
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (k + u < nk) sum += a[u];  // workgroup-uniform
    }
  }
  if (own) store[q * d.store_len + po + (e - q * blk)] = sum;
}

// Pairs no batch touches are zero unless accumulating (selected parts).
__global__ void k_zero_pairs(DevPlan d, const int32_t *pairs, double *store, int nq, unsigned part_mask) {
  const int p = pairs[blockIdx.x];
  const int64_t blk = (int64_t)d.pair_na[p] * d.pair_nb[p];
  for (int64_t e = threadIdx.x; e < nq * blk; e += blockDim.x) {
    const int q = (int)(e / blk);
    if ((part_mask >> q) & 1) store[q * d.store_len + d.pair_off[p] + (e - q * blk)] = 0.0;
  }
}

// W_sp = Ws (x) I2 + i sum_m Wso_m (x) sigma_m and V_sp = V (x) I2, per pair a
// (2 nA) x (2 nB) complex block, spin-major rows and columns.
__global__ void k_spinor(DevPlan d, const double *store, double *spin_w, double *spin_v) {
  const int p = blockIdx.x;
  const int na = d.pair_na[p], nb = d.pair_nb[p];
  const int64_t blk = (int64_t)na * nb;
  const int64_t po = d.pair_off[p];
  const int64_t L = d.store_len;
  const int64_t cb = 8 * po;           // doubles: complex offset 4 po
  const int64_t rs = 2 * (int64_t)nb;  // complex row stride
  for (int64_t e = threadIdx.x; e < blk; e += blockDim.x) {
    const int i = (int)(e / nb), j = (int)(e - (int64_t)i * nb);
    const int64_t uu = 2 * ((int64_t)i * rs + j), ud = 2 * ((int64_t)i * rs + nb + j);
    const int64_t du = 2 * ((int64_t)(na + i) * rs + j), dd = 2 * ((int64_t)(na + i) * rs + nb + j);
    if (spin_w) {
      const double ws = store[L + po + e], wx = store[2 * L + po + e], wy = store[3 * L + po + e],
                   wz = store[4 * L + po + e];
      double *o = spin_w + cb;
      o[uu] = ws; o[uu + 1] = wz;
      o[ud] = wy; o[ud + 1] = wx;
      o[du] = -wy; o[du + 1] = wx;
      o[dd] = ws; o[dd + 1] = -wz;
    }
    if (spin_v) {
      const double vv = store[po + e];
      double *o = spin_v + cb;
      o[uu] = vv; o[uu + 1] = 0.0;
      o[ud] = 0.0; o[ud + 1] = 0.0;
      o[du] = 0.0; o[du + 1] = 0.0;
      o[dd] = vv; o[dd + 1] = 0.0;
    }
  }
}

__global__ void k_fill(double *p, int64_t n, double v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// Coefficients from spinor blocks D_AB (see q4c_coef_from_spinor).
__global__ void k_coef_from_spinor(DevPlan d, const double *spin, double *coef) {
  const int p = blockIdx.x;
  const int na = d.pair_na[p], nb = d.pair_nb[p];
  const int64_t blk = (int64_t)na * nb;
  const int64_t po = d.pair_off[p];
  const int64_t L = d.store_len;
  const int64_t rs = 2 * (int64_t)nb;
  const double f = d.pair_a[p] == d.pair_b[p] ? 1.0 : 2.0;
  const double *D = spin + 8 * po;
  for (int64_t e = threadIdx.x; e < blk; e += blockDim.x) {
    const int i = (int)(e / nb), j = (int)(e - (int64_t)i * nb);
    const double *uu = D + 2 * ((int64_t)i * rs + j), *ud = D + 2 * ((int64_t)i * rs + nb + j);
    const double *du = D + 2 * ((int64_t)(na + i) * rs + j), *dd = D + 2 * ((int64_t)(na + i) * rs + nb + j);
    const double dsum = f * (uu[0] + dd[0]);
    coef[po + e] = dsum;
    coef[L + po + e] = dsum;
    coef[2 * L + po + e] = f * (ud[1] + du[1]);
    coef[3 * L + po + e] = f * (ud[0] - du[0]);
    coef[4 * L + po + e] = f * (uu[1] - dd[1]);
  }
}

__global__ void k_check_finite(const double *v, int64_t n, int32_t *flag) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    if (!isfinite(v[i])) flag[0] = 1;
}

}  // namespace

static int check_launch(const char *what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, what);
  return Q4C_OK;
}

// Waves per 64-function tile: quarter tiles while whole ones would not even give
// each of the 1024 SIMDs a wave: 256 waves (3 atoms) take 22 us whole and 16 us
// in quarters, 6100 (17 atoms) 100 and 115 us (a shell cut by a tile's edge is
// looked up twice).
static int panel_sub(int64_t waves) { return waves <= 1024 ? 4 : 1; }

// Whether k_tabulate_few is the faster one: batches of few points, where a share
// of k_tabulate's lanes has no point (the values are the same).  24 atoms, with
// gradients, k_tabulate / k_tabulate_few: 8 points per batch 94 / 29 us, 32 120 /
// 76, 48 148 / 128, 64 46 / 52 (a quarter of the batches), 80 80 / 63, 96 81 / 75,
// 112 82 / 90, 144 103 / 113; values alone 50 / 23, 64 / 60, 69 / 82, 25 / 40, 41
// / 48 up to 80 points.
static bool tabulate_few(const q4c_plan *p, int deriv) {
  return p->max_batch_points <= 128 && p->tab_fill < (deriv ? 0.8 : 0.6);
}

int launch_tabulate(const q4c_plan *p, int64_t b0, int64_t b1, int deriv, int dtype, void *out, hipStream_t s) {
  const int64_t t0 = p->batch_tile_off[b0], nt = p->batch_tile_off[b1] - t0;
  if (nt <= 0) return Q4C_OK;
  int pmax = 0;
  for (int64_t b = b0; b < b1; ++b) pmax = std::max(pmax, (int)(p->batch_pt_off[b + 1] - p->batch_pt_off[b]));
  const int npb = (pmax + 63) / 64;
  if (tabulate_few(p, deriv)) {
    {
      TimedLaunch tl_(p, Q4C_TIMER_TABULATE, s);
      hipLaunchKernelGGL(dtype == Q4C_DTYPE_F32_HILO ? k_tabulate_few<true> : k_tabulate_few<false>, dim3((unsigned)nt),
                         dim3(256), 0, s, p->dp, p->d_ptile, t0, b0, deriv, out);
    }
    return check_launch("k_tabulate_few");
  }
  {
    TimedLaunch tl_(p, Q4C_TIMER_TABULATE, s);
    for_grids(nt * npb, [&](int64_t wg0, unsigned grid) {
      hipLaunchKernelGGL(dtype == Q4C_DTYPE_F32_HILO ? k_tabulate<true> : k_tabulate<false>, dim3(grid), dim3(512), 0, s,
                         p->dp, p->d_ptile, t0, wg0, npb, b0, deriv, out);
    });
  }
  return check_launch("k_tabulate");
}

// Launch one contraction kernel over work positions [w0, w0 + nw) of a pass,
// persistent (tickets) or one workgroup per position.
template <typename K>
static void launch_work(K kernel_p, K kernel_1, unsigned grid, bool persistent, hipStream_t s, const DevPlan &dp,
                        const WorkItem *work, const int32_t *order, int64_t w0, int64_t nw, const double *om,
                        const double *panel, double *staging, unsigned *tickets) {
  if (persistent)
    hipLaunchKernelGGL(kernel_p, dim3(grid), dim3(NT), 0, s, dp, work, order, w0, nw, om, panel, staging, tickets);
  else
    hipLaunchKernelGGL(kernel_1, dim3(grid), dim3(NT), 0, s, dp, work, order, w0, nw, om, panel, staging, tickets);
}

// The panels of a pass: one wave per (tile or quarter tile, 64 points).
template <typename K>
static void launch_panel(K kernel, const q4c_plan *p, const Pass &ps, double *panel, hipStream_t s) {
  const int64_t nt = ps.t1 - ps.t0;
  const int npb = (ps.p_max + 63) / 64;
  const int sub = panel_sub(nt * npb);
  for_grids(nt * sub * npb, [&](int64_t wg0, unsigned grid) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64), 0, s, p->dp, p->d_ptile, ps.t0, wg0, sub, npb, panel,
                       (const double *)p->d_om);
  });
}

int launch_integrate(const q4c_plan *p, const double *v, int precision, uint32_t parts, uint32_t flags,
                     double *store, double *spin_w, double *spin_v, hipStream_t s) {
  const int accumulate = (flags & Q4C_ACCUMULATE) ? 1 : 0;
  const bool wantV = parts & Q4C_PART_V, wantW = parts & (Q4C_PART_WS | Q4C_PART_WSO);
  // store parts written: 0 V, 1 Ws, 2..4 Wso
  const unsigned pmask = (wantV ? 1u : 0u) | ((parts & Q4C_PART_WS) ? 2u : 0u) | ((parts & Q4C_PART_WSO) ? 28u : 0u);
  // FP64 with W parts: one kernel for all five (PK_F64 panels); otherwise V
  // on FP64 from phi alone and the W parts on FP32 (PK_F32 / PK_SPLIT panels)
  // BF16X3 with W parts: one kernel for all five (PK_BF16 panels)
  const bool full64 = (precision == Q4C_PREC_F64 || precision == Q4C_PREC_F64_VALU) && wantW;
  const bool fused_b3 = precision == Q4C_PREC_BF16X3 && wantW;
  const int kind = (full64 || precision == Q4C_PREC_F64_VALU) ? PK_F64
                   : fused_b3 ? PK_BF16
                              : (precision == Q4C_PREC_SPLIT_F32 && wantW ? PK_SPLIT : PK_F32);
  int rc;
  {
    TimedLaunch tl_(p, Q4C_TIMER_OTHER, s);
    const unsigned nb = (unsigned)std::max<int64_t>(1, std::min<int64_t>((p->n_active + 255) / 256, 65535));
    hipLaunchKernelGGL(k_om, dim3(nb), dim3(256), 0, s, p->dp, v, p->d_om);
  }
  if ((rc = check_launch("k_om")) != Q4C_OK) return rc;
  const LaunchCfg cfg = p->cfg_contract;
  const int32_t *order = cfg.order ? p->d_order : nullptr;
  const int64_t np_ = (int64_t)p->passes.size();
  if (cfg.persistent > 0) {
    // ticket queues: [V or all-parts kernel][W kernel] x passes
    hipLaunchKernelGGL(k_zero_u32, dim3(8), dim3(256), 0, s, p->d_tickets, 2 * np_ * kTicketsPerLaunch);
    if ((rc = check_launch("k_zero_u32")) != Q4C_OK) return rc;
  }
  for (size_t ip = 0; ip < p->passes.size(); ++ip) {
    const Pass &ps = p->passes[ip];
    const int64_t nw = ps.w1 - ps.w0, nt = ps.t1 - ps.t0, nr = ps.r1 - ps.r0;
    const bool pers = cfg.persistent > 0;
    unsigned *tick_a = pers ? p->d_tickets + ip * kTicketsPerLaunch : nullptr;
    unsigned *tick_w = pers ? p->d_tickets + (np_ + ip) * kTicketsPerLaunch : nullptr;
    const unsigned grid = (unsigned)(pers ? std::min<int64_t>(cfg.persistent, nw) : nw);
    double *panel = p->d_staging + ps.staging_len + ps.partial_len;
    if (nt > 0) {
      {
        TimedLaunch tl_(p, Q4C_TIMER_TABULATE, s);
        if (kind == PK_F64)
          launch_panel(k_panel<PK_F64>, p, ps, panel, s);
        else if (kind == PK_BF16)
          launch_panel(k_panel<PK_BF16>, p, ps, panel, s);
        else if (kind == PK_SPLIT)
          launch_panel(k_panel<PK_SPLIT>, p, ps, panel, s);
        else
          launch_panel(k_panel<PK_F32>, p, ps, panel, s);
      }
      if ((rc = check_launch("k_panel")) != Q4C_OK) return rc;
    }
    if (nw > 0) {
      TimedLaunch tl_(p, Q4C_TIMER_CONTRACT, s);
      if (precision == Q4C_PREC_F64_VALU) {
        // the plain FP64 baseline: one workgroup per work item, every part
        hipLaunchKernelGGL(k_contract_valu, dim3((unsigned)nw), dim3(NT), 0, s, p->dp, p->d_work, order, ps.w0, nw,
                           p->d_om, panel, p->d_staging, (unsigned *)nullptr);
      } else if (full64) {
        if ((rc = launch_forward(p, ps, panel, tick_a, s)) != Q4C_OK) return rc;
      } else if (fused_b3) {
        // one workgroup per column half of each work item
        const unsigned grid2 = (unsigned)(pers ? std::min<int64_t>(cfg.persistent, 2 * nw) : 2 * nw);
        launch_work(k_contract_b3<true>, k_contract_b3<false>, grid2, pers, s, p->dp, p->d_work, order, ps.w0, nw,
                    p->d_om, panel, p->d_staging, tick_a);
      } else {
        if (wantV) {
          // four V-only workgroups fit on a CU, twice the other contraction
          // kernels' two: twice the persistent workgroups
          const unsigned grid_v = (unsigned)(pers ? std::min<int64_t>(2 * (int64_t)cfg.persistent, nw) : nw);
          auto go = [&](auto kernel_p, auto kernel_1) {
            launch_work(kernel_p, kernel_1, grid_v, pers, s, p->dp, p->d_work, order, ps.w0, nw, p->d_om, panel,
                        p->d_staging, tick_a);
          };
          p->stage_far ? go(k_contract_v<true, true>, k_contract_v<true, false>)
                       : go(k_contract_v<false, true>, k_contract_v<false, false>);
        }
        if (wantW) {
          auto go = [&](auto kernel_p, auto kernel_1) {
            launch_work(kernel_p, kernel_1, grid, pers, s, p->dp, p->d_work, order, ps.w0, nw, p->d_om, panel,
                        p->d_staging, tick_w);
          };
          if (precision == Q4C_PREC_SPLIT_F32)
            p->stage_far ? go(k_contract_w<true, true, true>, k_contract_w<true, true, false>)
                         : go(k_contract_w<true, false, true>, k_contract_w<true, false, false>);
          else
            p->stage_far ? go(k_contract_w<false, true, true>, k_contract_w<false, true, false>)
                         : go(k_contract_w<false, false, true>, k_contract_w<false, false, false>);
        }
      }
    }
    if (nw > 0 && (rc = check_launch("k_contract")) != Q4C_OK) return rc;
    if (nr > 0) {
      {
        TimedLaunch tl_(p, Q4C_TIMER_REDUCE, s);
        hipLaunchKernelGGL(k_reduce, dim3((unsigned)nr, (unsigned)((5 * p->max_pair_block + NTR - 1) / NTR)), dim3(NTR),
                           0, s, p->dp, ps.r0, p->d_red_pair, p->d_red_first, p->d_red_inc_off, p->d_inc_src,
                           p->d_staging, store, accumulate, 5, pmask);
      }
      if ((rc = check_launch("k_reduce")) != Q4C_OK) return rc;
    }
  }
  if (!accumulate && !p->untouched_pairs.empty()) {
    {
      TimedLaunch tl_(p, Q4C_TIMER_OTHER, s);
      hipLaunchKernelGGL(k_zero_pairs, dim3((unsigned)p->untouched_pairs.size()), dim3(256), 0, s, p->dp,
                         p->d_untouched, store, 5, pmask);
    }
    if ((rc = check_launch("k_zero_pairs")) != Q4C_OK) return rc;
  }
  if ((flags & (Q4C_ASSEMBLE_W | Q4C_ASSEMBLE_V)) && p->n_pairs > 0) {
    {
      TimedLaunch tl_(p, Q4C_TIMER_SPINOR, s);
      hipLaunchKernelGGL(k_spinor, dim3((unsigned)p->n_pairs), dim3(256), 0, s, p->dp, store,
                         (flags & Q4C_ASSEMBLE_W) ? spin_w : nullptr, (flags & Q4C_ASSEMBLE_V) ? spin_v : nullptr);
    }
    if ((rc = check_launch("k_spinor")) != Q4C_OK) return rc;
  }
  return Q4C_OK;
}

int launch_integrate_hs(const q4c_plan *p, const double *v, uint32_t flags, double *hs, hipStream_t s) {
  const int accumulate = (flags & Q4C_ACCUMULATE) ? 1 : 0;
  int rc;
  {
    TimedLaunch tl_(p, Q4C_TIMER_OTHER, s);
    const unsigned nb = (unsigned)std::max<int64_t>(1, std::min<int64_t>((p->n_active + 255) / 256, 65535));
    hipLaunchKernelGGL(k_om, dim3(nb), dim3(256), 0, s, p->dp, v, p->d_om);
  }
  if ((rc = check_launch("k_om")) != Q4C_OK) return rc;
  const LaunchCfg cfg = p->cfg_hs;
  if (cfg.persistent > 0) {
    hipLaunchKernelGGL(k_zero_u32, dim3(8), dim3(256), 0, s, p->d_tickets,
                       (int64_t)p->passes.size() * kTicketsPerLaunch);
    if ((rc = check_launch("k_zero_u32")) != Q4C_OK) return rc;
  }
  for (size_t ip = 0; ip < p->passes.size(); ++ip) {
    const Pass &ps = p->passes[ip];
    const int64_t nw = ps.w1 - ps.w0, nt = ps.t1 - ps.t0, nr = ps.r1 - ps.r0;
    unsigned *tickets = cfg.persistent > 0 ? p->d_tickets + ip * kTicketsPerLaunch : nullptr;
    double *panel = p->d_staging + ps.staging_len + ps.partial_len;
    if (nt > 0) {
      {
        TimedLaunch tl_(p, Q4C_TIMER_TABULATE, s);
        launch_panel(k_panel<PK_HS>, p, ps, panel, s);
      }
      if ((rc = check_launch("k_panel<hs>")) != Q4C_OK) return rc;
    }
    if (nw > 0) {
      {
        TimedLaunch tl_(p, Q4C_TIMER_CONTRACT, s);
        rc = launch_contract_hs(p, ps, panel, tickets, s);
      }
      if (rc != Q4C_OK) return rc;
    }
    if (nr > 0) {
      {
        TimedLaunch tl_(p, Q4C_TIMER_REDUCE, s);
        hipLaunchKernelGGL(k_reduce, dim3((unsigned)nr, (unsigned)((2 * p->max_pair_block + NTR - 1) / NTR)), dim3(NTR),
                           0, s, p->dp, ps.r0, p->d_red_pair, p->d_red_first, p->d_red_inc_off, p->d_inc_src,
                           p->d_staging, hs, accumulate, 2, 3u);
      }
      if ((rc = check_launch("k_reduce")) != Q4C_OK) return rc;
    }
  }
  if (!accumulate && !p->untouched_pairs.empty()) {
    {
      TimedLaunch tl_(p, Q4C_TIMER_OTHER, s);
      hipLaunchKernelGGL(k_zero_pairs, dim3((unsigned)p->untouched_pairs.size()), dim3(256), 0, s, p->dp,
                         p->d_untouched, hs, 2, 3u);
    }
    if ((rc = check_launch("k_zero_pairs")) != Q4C_OK) return rc;
  }
  return Q4C_OK;
}

int launch_density(const q4c_plan *p, const double *coef, uint32_t terms, int precision, int weight_mode,
                   double *out, int64_t resident_pass, hipStream_t s) {
  int rc;
  if (p->n_points > 0) {
    {
      TimedLaunch tl_(p, Q4C_TIMER_OTHER, s);
      const unsigned nb = (unsigned)std::min<int64_t>((p->n_points + 255) / 256, 65535);
      hipLaunchKernelGGL(k_fill, dim3(nb), dim3(256), 0, s, out, p->n_points, 0.0);
    }
    if ((rc = check_launch("k_fill")) != Q4C_OK) return rc;
  }
  if ((rc = launch_density_fold(p, coef, terms, precision, s)) != Q4C_OK) return rc;
  const LaunchCfg cfg = p->cfg_density;
  unsigned *tick0 = p->d_tickets + p->passes.size() * kTicketsPerLaunch;
  if (cfg.persistent > 0) {
    hipLaunchKernelGGL(k_zero_u32, dim3(8), dim3(256), 0, s, tick0, (int64_t)p->passes.size() * kTicketsPerLaunch);
    if ((rc = check_launch("k_zero_u32")) != Q4C_OK) return rc;
  }
  // passes from the last one down: the first one may find its panels resident
  // (the forward call ends with its last pass); each point's partials lie in
  // one pass, so the order of the passes does not change any result
  for (size_t ipr = p->passes.size(); ipr-- > 0;) {
    const size_t ip = ipr;
    const Pass &ps = p->passes[ip];
    const int64_t nt = (int64_t)ip == resident_pass ? 0 : ps.t1 - ps.t0;
    unsigned *tickets = cfg.persistent > 0 ? tick0 + ip * kTicketsPerLaunch : nullptr;
    double *partial = p->d_staging + ps.staging_len;
    double *panel = partial + ps.partial_len;
    if (nt > 0) {
      {
        TimedLaunch tl_(p, Q4C_TIMER_TABULATE, s);
        launch_panel(k_panel<PK_F64>, p, ps, panel, s);
      }
      if ((rc = check_launch("k_panel")) != Q4C_OK) return rc;
    }
    if ((rc = launch_density_pass(p, ps, terms, precision, weight_mode, panel, partial, tickets, out, s)) != Q4C_OK) return rc;
  }
  return Q4C_OK;
}

int launch_density_grad(const q4c_plan *p, const double *coef, double *out, hipStream_t s) {
  int rc;
  if (p->n_points > 0) {
    {
      TimedLaunch tl_(p, Q4C_TIMER_OTHER, s);
      const unsigned nb = (unsigned)std::min<int64_t>((4 * p->n_points + 255) / 256, 65535);
      hipLaunchKernelGGL(k_fill, dim3(nb), dim3(256), 0, s, out, 4 * p->n_points, 0.0);
    }
    if ((rc = check_launch("k_fill")) != Q4C_OK) return rc;
  }
  for (size_t ip = 0; ip < p->passes.size(); ++ip) {
    const Pass &ps = p->passes[ip];
    const int64_t nt = ps.t1 - ps.t0;
    double *panel = p->d_staging + ps.staging_len + ps.partial_len;
    if (nt > 0) {
      {
        TimedLaunch tl_(p, Q4C_TIMER_TABULATE, s);
        launch_panel(k_panel<PK_F64>, p, ps, panel, s);
      }
      if ((rc = check_launch("k_panel")) != Q4C_OK) return rc;
    }
    if ((rc = launch_grad_pass(p, ip, coef, panel, out, s)) != Q4C_OK) return rc;
  }
  return Q4C_OK;
}

int launch_coef_from_spinor(const q4c_plan *p, const double *spin_d, double *coef_out, hipStream_t s) {
  if (p->n_pairs == 0) return Q4C_OK;
  {
    TimedLaunch tl_(p, Q4C_TIMER_OTHER, s);
    hipLaunchKernelGGL(k_coef_from_spinor, dim3((unsigned)p->n_pairs), dim3(256), 0, s, p->dp, spin_d, coef_out);
  }
  return check_launch("k_coef_from_spinor");
}

int launch_check_finite(const q4c_plan *p, const double *v, hipStream_t s, bool *finite) {
  hipError_t e = hipMemsetAsync(p->d_flag, 0, sizeof(int32_t), s);
  if (e != hipSuccess) return hip_fail(e, "hipMemsetAsync");
  if (p->n_points > 0) {
    unsigned nb = (unsigned)std::min<int64_t>((p->n_points + 255) / 256, 65535);
    hipLaunchKernelGGL(k_check_finite, dim3(nb), dim3(256), 0, s, v, p->n_points, p->d_flag);
    int rc = check_launch("k_check_finite");
    if (rc != Q4C_OK) return rc;
  }
  int32_t h = 0;
  e = hipMemcpyAsync(&h, p->d_flag, sizeof(int32_t), hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
  *finite = (h == 0);
  return Q4C_OK;
}

}  // namespace q4c
