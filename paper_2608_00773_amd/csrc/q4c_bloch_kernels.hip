// Bloch sums of unit-cell integrals (paper Sec. II C, Eq. 27 with the
// restricted sum of Eq. 28): for a plan whose atoms are a reference cell's
// atoms and their periodic images (q4c_plan_set_cells), every element of
// every cell pair block (a <= b) at every k-point is
//   O_ab(k)[i][j] = sum over contributions (stored pair, orientation, T)
//                   exp(i k.T) O_pair[i][j]   (or s_q O_pair[j][i] transposed),
// s_q = -1 for the spin-orbit parts (q >= 2) of a five-part store.
//
// Two kernels per chunk of at most KB k-points:
//   k_bloch_phase  exp(i k.T) once per (contribution, k-point), [t][k] layout;
//   k_bloch_sum    one workgroup per (cell pair, part, group of k-points):
//                  contributions' offsets and phases are staged in LDS, each
//                  thread keeps a few elements x KC k-points of complex sums
//                  in registers, and the stored blocks are read in their own
//                  order, the transposed ones' sums turned once at the end.
// The reverse direction (q4c_bloch_density, the periodic density matrix of
// the same section) reuses k_bloch_phase with k-point weights, per stored
// pair; k_bloch_density runs one workgroup per group of stored pairs that
// share a cell pair.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <optional>

#include "q4c_internal.h"
#include "q4c_device.h"

// Fixed device scratch of q4c_bloch_sum_noalloc (the phase table of one
// k-point chunk), for callers that cannot allocate.  Each device the library
// runs on holds its own copy until the process ends; every call on a device
// shares it.  Host code must not pass this name to a kernel (it is a host
// stand-in there): it uses the device address from hipGetSymbolAddress.
static __device__ __align__(256) double scratch[q4c::kNoAllocScratchDoubles];

namespace q4c {
namespace {

constexpr int KB = kBlochKChunk;  // k-points per phase-table chunk

// ph[t][k] = w_k exp(i k.T_t) (w_k = 1 without weights)
__global__ __launch_bounds__(256) void k_bloch_phase(int n_k, int64_t n_ct, const double *kpts, const double *kw,
                                                     const double *ct_T, double *ph) {
  const int64_t total = (int64_t)n_k * n_ct;
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < total; g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = g / n_k;
    const int ik = (int)(g - t * n_k);
    double sn, cs;
    sincos(kpts[3 * ik] * ct_T[3 * t] + kpts[3 * ik + 1] * ct_T[3 * t + 1] + kpts[3 * ik + 2] * ct_T[3 * t + 2], &sn,
           &cs);
    const double w = kw ? kw[ik] : 1.0;
    ph[2 * g] = w * cs;
    ph[2 * g + 1] = w * sn;
  }
}

constexpr int BS_EPT = 3;  // cell elements per thread: blocks of up to 27 x 28 functions in one go
constexpr int BS_EL = 256 * BS_EPT;
constexpr int BS_TB = 64;  // contributions staged in LDS at a time
constexpr int BS_PF = 4;   // contributions whose values are loaded together

// One workgroup per (cell pair c, part q) and group of kper <= KC k-points.
// The contributions' store offsets and phases are staged in LDS (BS_TB
// contributions at a time) and read as broadcasts; each thread holds BS_EPT
// elements x KC k-points of complex sums, so that one staged phase serves
// BS_EPT elements.  A cell pair's contributions come transposed ones first:
// both kinds are read in the stored order (contiguous), the sums of the
// transposed ones are turned through LDS and the direct ones added on.
// Bound: HBM, the store read once (the groups of k-points of a cell pair run
// side by side and share its L2), and the latency of those reads, hence the
// values of the next contributions in flight while these are added.  2 x 2 x 1
// cell (9.5M elements, 5 parts, 18 k-points, 494 MB): 414 -> 155 us (3.2 TB/s)
// against 8 k-points at a time one launch row after the other, transposed
// blocks read by column and two elements per thread; 301 us without the loads
// ahead and with the groups apart.
// Blocks of more than BS_EL elements take several rounds over the contributions and
// read the transposed ones by column; 3,228 pairs of 28 x 28 functions 0.73 -> 0.26
// ms (4 k-points), 2.1 -> 0.38 (18), of 54 x 54 3.0 -> 1.1 and 7.7 -> 1.2.
// ph: [n_ct][n_k] complex phases of this chunk; out: [n_k][n_parts][clen] complex.
template <int KC>
__global__ __launch_bounds__(256, 2) void k_bloch_sum(DevPlan d, int n_parts, int64_t ncp, const int64_t *cp_off,
                                                      const int64_t *ct_off, const int32_t *ct_pair,
                                                      const int32_t *ct_flag, int64_t wg0, int n_k, int n_grp,
                                                      int kper, const double *ph,
                                                      const double *__restrict__ store, double *__restrict__ out) {
  __shared__ int64_t s_off[BS_TB];
  __shared__ dbl2 s_ph[BS_TB][KC];
  __shared__ dbl2 s_turn[BS_EL];
  // the k-point groups of one (cell pair, part) next to each other on one XCD:
  // they read the same blocks
  const int64_t wg = wg0 + xcd_map(blockIdx.x, gridDim.x), cq = wg / n_grp;
  const int64_t c = cq / n_parts;
  const int q = (int)(cq - c * n_parts);
  const int k0 = (int)(wg - cq * n_grp) * kper, nk = min(kper, n_k - k0);
  const int64_t clen = cp_off[ncp];
  const int64_t e0 = cp_off[c], blk = cp_off[c + 1] - e0;
  const int64_t t0 = ct_off[2 * c], tm = ct_off[2 * c + 1], t1 = ct_off[2 * c + 2];
  const double sq = (n_parts == 5 && q >= 2) ? -1.0 : 1.0;
  const int64_t L = d.store_len;
  // columns of the cell-pair block: those of the stored block (direct) or
  // its rows (transposed), the same for every contribution of the cell pair
  const int64_t p0 = ct_pair[t0];
  const int ncol = ct_flag[t0] ? d.pair_na[p0] : d.pair_nb[p0];
  const int64_t nrow = blk / ncol;
  const int tid = threadIdx.x;
  const bool whole = blk <= BS_EL;  // workgroup-uniform: the transposed sums can be turned
  for (int64_t eb = 0; eb < blk; eb += BS_EL) {
    double re[BS_EPT][KC], im[BS_EPT][KC];
#pragma unroll
    for (int x = 0; x < BS_EPT; ++x)
#pragma unroll
      for (int kk = 0; kk < KC; ++kk) re[x][kk] = im[x][kk] = 0.0;
    // adds contributions [ta, tz), element le + 256 x at at[x] of the stored block
    auto add = [&](int64_t ta, int64_t tz, const int64_t (&at)[BS_EPT], double sign) {
      for (int64_t tb = ta; tb < tz; tb += BS_TB) {
        const int nb = (int)min<int64_t>(BS_TB, tz - tb);
        __syncthreads();  // the previous batch is consumed
        for (int x = tid; x < nb; x += 256) s_off[x] = (int64_t)q * L + d.pair_off[ct_pair[tb + x]];
        for (int x = tid; x < nb * KC; x += 256) {
          const int tt = x / KC, kk = x - tt * KC;
          const double *pt = ph + 2 * ((tb + tt) * n_k + k0 + kk);
          s_ph[tt][kk] = kk < nk ? dbl2{sign * pt[0], sign * pt[1]} : dbl2{0.0, 0.0};
        }
        __syncthreads();  // the batch is visible
        // BS_PF contributions at a time, the next ones' values loaded while
        // these are added (past the last one: it again, not added)
        double v[2][BS_PF][BS_EPT];
        auto load = [&](int tt, double (&w)[BS_PF][BS_EPT]) {
#pragma unroll
          for (int u = 0; u < BS_PF; ++u) {
            const double *b = store + s_off[min(tt + u, nb - 1)];
#pragma unroll
            for (int x = 0; x < BS_EPT; ++x) w[u][x] = b[at[x]];
          }
        };
        auto sum = [&](int tt, const double (&w)[BS_PF][BS_EPT]) {
#pragma unroll
          for (int u = 0; u < BS_PF; ++u)
            if (tt + u < nb) {  // workgroup-uniform
#pragma unroll
              for (int kk = 0; kk < KC; ++kk) {
                const dbl2 f = s_ph[tt + u][kk];
#pragma unroll
                for (int x = 0; x < BS_EPT; ++x) {
                  re[x][kk] = fma(f[0], w[u][x], re[x][kk]);
                  im[x][kk] = fma(f[1], w[u][x], im[x][kk]);
                }
              }
            }
        };
        load(0, v[0]);
        for (int tt = 0; tt < nb; tt += 2 * BS_PF) {
          load(tt + BS_PF, v[1]);
          __builtin_amdgcn_sched_barrier(0);
          sum(tt, v[0]);
          __builtin_amdgcn_sched_barrier(0);
          load(tt + 2 * BS_PF, v[0]);
          __builtin_amdgcn_sched_barrier(0);
          sum(tt + BS_PF, v[1]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    int64_t at[BS_EPT], turned[BS_EPT];
#pragma unroll
    for (int x = 0; x < BS_EPT; ++x) {
      const int64_t le = min<int64_t>(eb + tid + 256 * x, blk - 1);  // beyond the block: its last element, not written
      const int64_t i = le / ncol, j = le - i * ncol;
      at[x] = le;
      turned[x] = j * nrow + i;
    }
    if (t0 < tm && whole) {
      add(t0, tm, at, sq);
#pragma unroll
      for (int kk = 0; kk < KC; ++kk) {
        if (kk < nk) {      // workgroup-uniform
          __syncthreads();  // the previous k-point is read
#pragma unroll
          for (int x = 0; x < BS_EPT; ++x) s_turn[tid + 256 * x] = dbl2{re[x][kk], im[x][kk]};
          __syncthreads();
#pragma unroll
          for (int x = 0; x < BS_EPT; ++x) {
            re[x][kk] = s_turn[turned[x]][0];
            im[x][kk] = s_turn[turned[x]][1];
          }
        }
      }
    } else {
      add(t0, tm, turned, sq);
    }
    add(tm, t1, at, 1.0);
#pragma unroll
    for (int x = 0; x < BS_EPT; ++x) {
      const int64_t le = eb + tid + 256 * x;
      if (le < blk) {
#pragma unroll
        for (int kk = 0; kk < KC; ++kk)
          if (kk < nk)
            *reinterpret_cast<dbl2 *>(out + 2 * (((int64_t)(k0 + kk) * n_parts + q) * clen + e0 + le)) =
                dbl2{re[x][kk], im[x][kk]};
      }
    }
  }
}

// The reverse direction (the periodic density matrix of Sec. II C): a group
// of up to kBlochGroup stored image pairs p = (A', B') of one cell pair in one
// orientation, one thread per element (i, j):
//   coef = f Re sum_k w_k exp(i k.(T_B' - T_A')) rho_ab(k)[i][j],
// rho_ab(k)[i][j] = conj(rho_ba(k)[j][i]) when the cell atoms run a > b,
// f = 2 off the self pairs.  Each rho value read serves the whole group.
// Bound: L2 reads of rho, once per group (one pair per workgroup read it for
// every pair: 168 -> 50 us for 15k pairs and 18 k-points).  ph:
// [n_pairs][n_k] weighted phases of this chunk (uniform per workgroup); rho:
// this chunk's [n_k][n_parts][clen] complex; acc: add to coef.
__global__ __launch_bounds__(256) void k_bloch_density(DevPlan d, int n_parts, int64_t n_groups, int64_t ncp,
                                                       const int64_t *cp_off, const int32_t *pc_cp,
                                                       const int32_t *pc_flag, const int32_t *pc_order,
                                                       const int32_t *pc_group, int n_k,
                                                       const double *__restrict__ ph,
                                                       const double *__restrict__ rho, int acc,
                                                       double *__restrict__ coef) {
  constexpr int G = kBlochGroup;
  // the groups of one cell pair run one after another on one XCD
  const int64_t g = xcd_map(blockIdx.x, n_groups);
  const int first = pc_group[g], np = pc_group[g + 1] - first;
  const int64_t p0 = pc_order[first];
  const int64_t L = d.store_len, clen = cp_off[ncp];
  const int na = d.pair_na[p0], nb = d.pair_nb[p0];
  const int64_t blk = (int64_t)na * nb;
  const int64_t e = (int64_t)blockIdx.y * 256 + threadIdx.x;
  if (e >= blk) return;
  const bool tr = pc_flag[p0] != 0;
  const double sg = tr ? 1.0 : -1.0;  // Re(e^{i t} r) = c Re r - s Im r; conj(r): c Re r + s Im r
  // element of the cell-pair block: (i, j) of (a, b), or (j, i) of (b, a)
  const int i = (int)(e / nb), j = (int)(e - (int64_t)i * nb);
  const int64_t ce = cp_off[pc_cp[p0]] + (tr ? (int64_t)j * na + i : e);
  const double *pp[G];  // the pairs' phases (uniform)
#pragma unroll
  for (int x = 0; x < G; ++x) pp[x] = ph + 2 * (int64_t)pc_order[first + min(x, np - 1)] * n_k;
  for (int q = 0; q < n_parts; ++q) {
    double s[G];
#pragma unroll
    for (int x = 0; x < G; ++x) s[x] = 0.0;
#pragma unroll 2
    for (int k = 0; k < n_k; ++k) {
      const dbl2 r = *reinterpret_cast<const dbl2 *>(rho + 2 * (((int64_t)k * n_parts + q) * clen + ce));
      const double ri = sg * r[1];
#pragma unroll
      for (int x = 0; x < G; ++x) s[x] = fma(pp[x][2 * k + 1], ri, fma(pp[x][2 * k], r[0], s[x]));
    }
#pragma unroll
    for (int x = 0; x < G; ++x) {
      if (x < np) {  // workgroup-uniform
        const int64_t p = pc_order[first + x];
        const double f = d.pair_a[p] == d.pair_b[p] ? 1.0 : 2.0;
        double *o = coef + (int64_t)q * L + d.pair_off[p] + e;
        *o = acc ? *o + f * s[x] : f * s[x];
      }
    }
  }
}

}  // namespace

// Phase table, then the sums, for chunks of at most kchunk (<= KB) k-points;
// phase holds 2 kchunk n_contrib doubles.  timed: record the plan's profiling
// events (created on demand) when profiling is on.
static int launch_bloch_sum_chunks(const q4c_plan *p, int n_parts, const double *store, int n_k,
                                   const double *kpts_dev, double *phase, int kchunk, bool timed, double *out,
                                   hipStream_t s) {
  const int64_t ncp = (int64_t)p->cp_a.size();
  const int64_t clen = p->cp_off.back();
  const int64_t n_ct = p->n_contrib;
  if ((int64_t)n_k * n_parts * clen == 0) return Q4C_OK;
  for (int k0 = 0; k0 < n_k; k0 += kchunk) {
    const int nk = std::min(kchunk, n_k - k0);
    {
      std::optional<TimedLaunch> tl_;
      if (timed) tl_.emplace(p, Q4C_TIMER_OTHER, s);
      const int64_t tot = (int64_t)nk * n_ct;
      const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((tot + 255) / 256, 65536));
      hipLaunchKernelGGL(k_bloch_phase, dim3(grid), dim3(256), 0, s, nk, n_ct, kpts_dev + 3 * (int64_t)k0,
                         (const double *)nullptr, p->d_ct_T, phase);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_bloch_phase");
    {
      std::optional<TimedLaunch> tl_;
      if (timed) tl_.emplace(p, Q4C_TIMER_BLOCH, s);
      // k-points in equal groups of at most 9 (a thread's registers hold 3
      // elements x 9 complex sums)
      const int groups = (nk + 8) / 9, kper = (nk + groups - 1) / groups;
      auto launch = [&](auto kernel) {
        for_grids(ncp * n_parts * groups, [&](int64_t wg0, unsigned grid) {
          hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, s, p->dp, n_parts, ncp, p->d_cp_off, p->d_ct_off,
                             p->d_ct_pair, p->d_ct_flag, wg0, nk, groups, kper, (const double *)phase, store,
                             out + 2 * (int64_t)k0 * n_parts * clen);
        });
      };
      if (kper <= 2)
        launch(k_bloch_sum<2>);
      else if (kper <= 4)
        launch(k_bloch_sum<4>);
      else if (kper <= 6)
        launch(k_bloch_sum<6>);
      else
        launch(k_bloch_sum<9>);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_bloch_sum");
  }
  return Q4C_OK;
}

int launch_bloch_sum(const q4c_plan *p, int n_parts, const double *store, int n_k, const double *kpts_dev,
                     double *phase, double *out, hipStream_t s) {
  return launch_bloch_sum_chunks(p, n_parts, store, n_k, kpts_dev, phase, KB, true, out, s);
}

// Device address of `scratch` per device, looked up once per device (with
// that device current) on its first use.
static std::mutex g_scratch_mu;
static double *g_scratch_dev[kMaxDevices] = {};

int noalloc_scratch(int device, double **ptr) {
  if (device < 0 || device >= kMaxDevices) return fail_status(Q4C_EUNSUPPORTED, "device index beyond the scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[device]) {
    void *addr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    g_scratch_dev[device] = static_cast<double *>(addr);
  }
  *ptr = g_scratch_dev[device];
  return Q4C_OK;
}

int launch_bloch_sum_noalloc(const q4c_plan *p, int n_parts, const double *store, int n_k, const double *kpts_dev,
                             double *out, hipStream_t s) {
  double *phase = nullptr;
  int rc = noalloc_scratch(p->device, &phase);
  if (rc != Q4C_OK) return rc;
  // the phases of one k-point take 2 n_contrib doubles: as many k-points per
  // chunk as the scratch holds (at most KB)
  const int64_t per_k = 2 * std::max<int64_t>(p->n_contrib, 1);
  if (per_k > kNoAllocScratchDoubles)
    return fail_status(Q4C_ESIZE, "the phases of one k-point exceed the fixed scratch of q4c_bloch_sum_noalloc");
  const int kchunk = (int)std::min<int64_t>(KB, kNoAllocScratchDoubles / per_k);
  // no profiling events here: creating one may allocate
  return launch_bloch_sum_chunks(p, n_parts, store, n_k, kpts_dev, phase, kchunk, false, out, s);
}

int launch_bloch_density(const q4c_plan *p, int n_parts, const double *rho, int n_k, const double *kpts_dev,
                         const double *kw_dev, double *phase, double *coef, hipStream_t s) {
  const int64_t ncp = (int64_t)p->cp_a.size();
  const int64_t clen = p->cp_off.back();
  const int64_t L = p->store_len, np_ = p->n_pairs;
  if ((int64_t)n_parts * L == 0) return Q4C_OK;
  // no k-points: one pass with an empty sum writes zeros
  for (int k0 = 0; k0 < std::max(n_k, 1); k0 += KB) {
    const int nk = std::min(KB, n_k - k0);
    if (nk > 0) {
      TimedLaunch tl_(p, Q4C_TIMER_OTHER, s);
      const int64_t tot = (int64_t)nk * np_;
      const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((tot + 255) / 256, 65536));
      hipLaunchKernelGGL(k_bloch_phase, dim3(grid), dim3(256), 0, s, nk, np_, kpts_dev + 3 * (int64_t)k0,
                         kw_dev + k0, p->d_pc_T, phase);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_bloch_phase");
    {
      TimedLaunch tl_(p, Q4C_TIMER_BLOCH, s);
      const int64_t ng = p->n_bloch_groups;
      hipLaunchKernelGGL(k_bloch_density, dim3((unsigned)ng, (unsigned)((p->max_pair_block + 255) / 256)), dim3(256), 0,
                         s, p->dp, n_parts, ng, ncp, p->d_cp_off, p->d_pc_cp, p->d_pc_flag, p->d_pc_order,
                         p->d_pc_group, nk, (const double *)phase,
                         rho + 2 * (int64_t)k0 * n_parts * clen, k0 > 0 ? 1 : 0, coef);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_bloch_density");
  }
  return Q4C_OK;
}

}  // namespace q4c
