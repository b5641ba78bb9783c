// The kernels of density_on_grid: the transpose of the H integration
// (Eq. 39).  Per call the coefficients are folded once (k_coef_fold); then
// per pass every item of the batches' upper block triangles is contracted
// (k_density_items) and every point sums its partials in a fixed order
// (k_density_points).  The panel tabulation and the launches around these are
// in q4c_kernels.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "q4c_internal.h"
#include "q4c_device.h"

namespace q4c {
namespace {

// The adjoint's coefficients, folded once per call.  Eq. 39 sums every stored
// element ij of the selected terms; the items cover the upper 16 x 16 blocks
// of each batch, so in the diagonal block of one atom element (i, j), i < j,
// takes C_q(i, j) + s_q C_q(j, i) (s_q = +1 for V and Ws, -1 for the
// spin-orbit parts, whose terms change sign under i <-> j), (i, i) keeps
// C_q(i, i) and i > j is zero: every term is then carried once.  Blocks of two
// atoms are copied.  c' multiplies the W parts and unselected terms are zero.
// Each element holds kFold values: V, then for FP64 the coefficients of the
// six products D_m = a_m b_m, M_m (see k_density_items): with
// Wso_x = M_x - (D_y - D_z) and cyclic,
//   C^Dx = C^s + (C^y - C^z) and cyclic,  C^Mm = C^m;
// for the other forms C^s, C^x, C^y, C^z.  A zero element follows the last
// one (index store_len), for lanes without a stored element.  One workgroup
// per pair.
__global__ void k_coef_fold(DevPlan d, const double *coef, uint32_t terms, int six, double *cf) {
  const int64_t L = d.store_len;
  const int64_t q = blockIdx.x;
  const bool on[5] = {(terms & Q4C_TERM_LL) != 0, (terms & Q4C_TERM_SS) != 0, (terms & Q4C_TERM_SO) != 0,
                      (terms & Q4C_TERM_SO) != 0, (terms & Q4C_TERM_SO) != 0};
  if (q == 0 && threadIdx.x < kFold) cf[kFold * L + threadIdx.x] = 0.0;
  const int64_t po = d.pair_off[q];
  const int na = d.pair_na[q], nb = d.pair_nb[q];
  const bool diag = d.pair_a[q] == d.pair_b[q];
  for (int t = threadIdx.x; t < na * nb; t += blockDim.x) {
    const int i = t / nb, j = t - i * nb;
    double c[5];
#pragma unroll
    for (int p = 0; p < 5; ++p) {
      c[p] = coef[p * L + po + t];
      if (diag) {
        if (i < j)
          c[p] += mirror_sign(p) * coef[p * L + po + (int64_t)j * nb + i];
        else if (i > j)
          c[p] = 0.0;
      }
      c[p] = on[p] ? (p > 0 ? c[p] * d.cprime : c[p]) : 0.0;
    }
    dbl2 *o = reinterpret_cast<dbl2 *>(cf + kFold * (po + t));
    if (six) {
      o[0] = dbl2{c[0], c[1] + (c[3] - c[4])};
      o[1] = dbl2{c[1] + (c[4] - c[2]), c[1] + (c[2] - c[3])};
      o[2] = dbl2{c[2], c[3]};
      o[3] = dbl2{c[4], 0.0};
    } else {
      o[0] = dbl2{c[0], c[1]};
      o[1] = dbl2{c[2], c[3]};
      o[2] = dbl2{c[4], 0.0};
    }
  }
}

// Partials of one item: rows 16 rb .. (at most kDenRows blocks of 16, down to
// the diagonal), the 16 columns of block cb, all points of the batch:
//   partial[g] = sum over its stored elements ij of the selected terms
//     C^V phi_i phi_j + c' C^Ws a.b + c' sum_m C^m (a x b)_m,  a = grad phi_i, b = grad phi_j.
// The W terms come from six products of the row and column values,
//   C^Dm a_m b_m and C^Mx (a_y - a_z)(b_y + b_z) (and cyclic),
// as in the forward contraction: with V seven FP64 MFMAs per K step of 4 rows
// instead of ten.  The item's coefficients go into LDS once, shared by the four
// waves; each wave takes every fourth chunk of 16 points and runs through
// without barriers: per chunk seven accumulators (points x columns) over all
// rows of the item, then one sum over the columns.  Row values and column
// values come straight from the panel into registers, the next K pair's row
// values and coefficients (8 rows) while this one is multiplied.
//
// The MFMA takes the coefficients as its first operand, so that its result is
// columns x points: register r of lane (l16, lk) is a column at point l16, and
// the sum over the columns is a chain in the lane and two lane exchanges.
//
// Bound: FP64 matrix pipe, which an FP64 MFMA shares with every vector
// instruction of its SIMD (each costs about 5 cycles beside the MFMA's 64), so
// loads and LDS reads take no address arithmetic, the accumulators start from a
// zero operand and the drain is short.  Three workgroups of three row blocks
// (43 KB of LDS, at most 168 registers, hence the late loads of the column
// values) beat two of four (11.1 ms below) or four of two (10.8 ms); 8-byte
// loads whose neighbouring lanes read one point quad matter most (18.7 ms with
// points spread over the quads).  120-atom cluster 15.3 -> 9.6 ms, 17-atom
// molecule 0.52 -> 0.34 ms against ten products from LDS row images with a
// barrier every 16 points; FP32 W terms, 48 atoms, 2.84 -> 2.11 ms.  The
// seven MFMAs alone take 6.7 ms (cluster) at their peak rate, and the matrix pipe
// is busy for 72% of the active cycles.
//
// F32W (density_on_grid in FP32): the nine W products per K step run on FP32
// MFMA, coefficients and row values rounded to FP32; the FP32 sums over 32
// rows (at most 96 products per column and point) are drained into the FP64
// point sum, so the FP32 error of a point is at most gamma_98 (u = 2^-24)
// times the magnitudes of its W terms.  The V term stays FP64.
constexpr int NWD = 4, NTD = 64 * NWD;  // waves and threads of a workgroup

// The three kernels: FP64 with six products, FP32 W terms, and FP64 with nine
// products for calls with the spin-orbit terms but without V.  The six products
// round at the size of the D terms: beside V that does not show (RMS error of
// all terms 0.8-1.04 times that of nine products from 64-row tiles, 3 to 60
// atoms), in the spin-orbit terms alone it does (1.05-1.3; nine products here
// 0.91-1.05).
enum { DEN_F64 = 0, DEN_F32W = 1, DEN_SO = 2 };
__host__ __device__ constexpr int den_form(int precision, uint32_t terms) {
  return precision == Q4C_PREC_F32 ? DEN_F32W : (terms & Q4C_TERM_SO) && !(terms & Q4C_TERM_LL) ? DEN_SO : DEN_F64;
}

template <int FORM>
struct DenShared {
  static constexpr bool F32W = FORM == DEN_F32W;
  static constexpr int NC = FORM == DEN_F64 ? 7 : F32W ? 1 : 4;    // FP64 coefficients per element
  dbl2 c64[2 * kDenRows][NC][64];                                  // [K pair][part][lane], both K steps
  float c32[F32W ? 2 * kDenRows : 1][F32W ? 4 : 1][64][2];         // the FP32 W coefficients
};

// What an item's chunks need: the batch's panel, the item's partials, padded
// points and functions, points, first row and first column.
struct DenItem {
  const double *pb;
  int64_t plane;
  double *out;
  int Pp, np, P, i0, j0;
};

// The wave's chunks of an item of NB row blocks: chunks 16 wave + 16 NWD c.
// begin() issues the first loads (before the coefficients are in LDS), run()
// does the rest.
template <int FORM, int NB>
struct DenChunks {
  static constexpr bool F32W = FORM == DEN_F32W;
  static constexpr int NC = DenShared<FORM>::NC, Q0 = FORM == DEN_SO ? 1 : 0;  // Q0: the first panel component read
  const DenItem &x;
  const int lane, l16, lk;
  // lane offsets (bytes) in a chunk's four point quads: quad l16 / 4, the row
  // operand's function, point l16 % 4 (four neighbouring lanes read one quad);
  // and the column values, column lk + 4 r (FP64 MFMA) or 4 lk + r (FP32)
  const uint32_t vy, vz, vzw;
  // row values of a K pair (8 rows), the next pair's loaded while this one is
  // multiplied: two register sets
  double y[2][2][4];

  __device__ __forceinline__ DenChunks(const DenItem &x_, int lane_)
      : x(x_), lane(lane_), l16(lane_ & 15), lk(lane_ >> 4),
        vy(((uint32_t)(l16 >> 2) * x_.np + lk) * 32u + 8u * (l16 & 3)), vz(vy + (uint32_t)x_.j0 * 32u),
        vzw(vz + 96u * lk) {}

  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(int q, int k) const {
    return __builtin_amdgcn_make_buffer_rsrc((void *)(x.pb + (int64_t)q * x.plane + (int64_t)(k >> 2) * x.np * 4),
                                             (short)0, x.np * 128, 0x00020000);
  }
  template <int S>
  __device__ __forceinline__ void load_rows(int k, int kp) {
    const uint32_t so = (uint32_t)(x.i0 + 8 * kp) * 32u;
#pragma unroll
    for (int q = Q0; q < 4; ++q) {
      const __amdgpu_buffer_rsrc_t rs = rsrc(q, k);
#pragma unroll
      for (int h = 0; h < 2; ++h)
        y[S][h][q] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, vy + 128u * h, so, 0));
    }
  }
  __device__ __forceinline__ void begin(int wave) {
    if (16 * wave < x.Pp) load_rows<0>(16 * wave, 0);
  }
  // kp0: K pairs of the item before these rows
  __device__ __forceinline__ void chunk(int k, const DenShared<FORM> &sh, int kp0 = 0) {
    const int kn = k + 16 * NWD < x.Pp ? k + 16 * NWD : k;  // the wave's next chunk (the last: read again, unused)
    dbl4 u[NC];
    flt4 w[3];
    double z[4][4];
    double sum = 0.0, sumw = 0.0;  // V and W: one chain for both rounds W's six products at the size of V
    auto load_z = [&]() {
#pragma unroll
      for (int q = Q0; q < 4; ++q) {
        const __amdgpu_buffer_rsrc_t rs = rsrc(q, k);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          z[q][r] = __builtin_bit_cast(
              double, F32W && q ? __builtin_amdgcn_raw_buffer_load_b64(rs, vzw + 32u * r, 0, 0)
                                : __builtin_amdgcn_raw_buffer_load_b64(rs, vz + 128u * r, 0, 0));
      }
    };
    static_for<0, 2 * NB>([&](auto kc) {
      constexpr int KP = decltype(kc)::value, S = KP & 1;
      load_rows<S ^ 1>(KP + 1 < 2 * NB ? k : kn, KP + 1 < 2 * NB ? KP + 1 : 0);
      // the column values, for the drain: no earlier, so that three waves fit on a SIMD
      if constexpr (KP == (F32W && NB > 1 ? 3 : 2 * NB - 1)) load_z();
      __builtin_amdgcn_sched_barrier(0);
      dbl2 c[NC];
      float cw[F32W ? 4 : 1][2];
#pragma unroll
      for (int q = 0; q < NC; ++q) c[q] = sh.c64[kp0 + KP][q][lane];
      if constexpr (F32W) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          cw[q][0] = sh.c32[kp0 + KP][q][lane][0];
          cw[q][1] = sh.c32[kp0 + KP][q][lane][1];
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        // the sums start from zero (F32W: every 32 rows)
        const bool first = (F32W ? KP % 4 == 0 : KP == 0) && h == 0;
        const dbl4 z4 = dbl4{0.0, 0.0, 0.0, 0.0};
        const double y1 = y[S][h][1], y2 = y[S][h][2], y3 = y[S][h][3];
        if constexpr (FORM != DEN_SO) u[0] = mfma64(c[0][h], y[S][h][0], first ? z4 : u[0]);
        if constexpr (FORM == DEN_F64) {
          u[1] = mfma64(c[1][h], y1, first ? z4 : u[1]);
          u[2] = mfma64(c[2][h], y2, first ? z4 : u[2]);
          u[3] = mfma64(c[3][h], y3, first ? z4 : u[3]);
          u[4] = mfma64(c[4][h], y2 - y3, first ? z4 : u[4]);
          u[5] = mfma64(c[5][h], y3 - y1, first ? z4 : u[5]);
          u[6] = mfma64(c[6][h], y1 - y2, first ? z4 : u[6]);
        } else if constexpr (FORM == DEN_SO) {
          // grouped by the column component they meet: x: C^s dx - C^z dy + C^y dz, cyclic
          u[0] = mfma64(c[0][h], y1, first ? z4 : u[0]);
          u[1] = mfma64(c[3][h], y1, first ? z4 : u[1]);
          u[2] = mfma64(c[2][h], -y1, first ? z4 : u[2]);
          u[0] = mfma64(c[3][h], -y2, u[0]);
          u[1] = mfma64(c[0][h], y2, u[1]);
          u[2] = mfma64(c[1][h], y2, u[2]);
          u[0] = mfma64(c[2][h], y3, u[0]);
          u[1] = mfma64(c[1][h], -y3, u[1]);
          u[2] = mfma64(c[0][h], y3, u[2]);
        } else {  // the same in FP32
          const flt4 f4 = flt4{0.f, 0.f, 0.f, 0.f};
          const float f1 = (float)y1, f2 = (float)y2, f3 = (float)y3;
          w[0] = mfma32(cw[0][h], f1, first ? f4 : w[0]);
          w[1] = mfma32(cw[3][h], f1, first ? f4 : w[1]);
          w[2] = mfma32(cw[2][h], -f1, first ? f4 : w[2]);
          w[0] = mfma32(cw[3][h], -f2, w[0]);
          w[1] = mfma32(cw[0][h], f2, w[1]);
          w[2] = mfma32(cw[1][h], f2, w[2]);
          w[0] = mfma32(cw[2][h], f3, w[0]);
          w[1] = mfma32(cw[1][h], -f3, w[1]);
          w[2] = mfma32(cw[0][h], f3, w[2]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (KP + 1 == 2 * NB || (F32W && KP % 4 == 3)) {
        // drain: the lane's four columns
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (FORM != DEN_SO) sum = fma(u[0][r], z[0][r], sum);
          if constexpr (FORM == DEN_SO) {
            sumw = fma(u[0][r], z[1][r], sumw);
            sumw = fma(u[1][r], z[2][r], sumw);
            sumw = fma(u[2][r], z[3][r], sumw);
          } else if constexpr (F32W) {
            sumw = fma((double)w[0][r], z[1][r], sumw);
            sumw = fma((double)w[1][r], z[2][r], sumw);
            sumw = fma((double)w[2][r], z[3][r], sumw);
          } else {
            sumw = fma(u[1][r], z[1][r], sumw);
            sumw = fma(u[2][r], z[2][r], sumw);
            sumw = fma(u[3][r], z[3][r], sumw);
            sumw = fma(u[4][r], z[2][r] + z[3][r], sumw);
            sumw = fma(u[5][r], z[3][r] + z[1][r], sumw);
            sumw = fma(u[6][r], z[1][r] + z[2][r], sumw);
          }
        }
      }
    });
    sum += sumw;
    // the columns of the other lanes with this point
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    if (lk == 0 && k + l16 < x.P) x.out[k + l16] = sum;
  }
  __device__ __forceinline__ void run(int wave, const DenShared<FORM> &sh) {
    for (int k = 16 * wave; k < x.Pp; k += 16 * NWD) chunk(k, sh);
  }
};

template <int FORM, bool PERSIST>
__global__ __launch_bounds__(NTD, 3) void k_density_items(DevPlan d, const BlockItem *items, int64_t ni,
                                                          int global_queue, const double *cf, const double *panel,
                                                          double *partial, unsigned *tickets) {
  constexpr bool F32W = FORM == DEN_F32W;
  constexpr int NC = DenShared<FORM>::NC;
  __shared__ DenShared<FORM> sh;
  __shared__ int64_t s_pos;
  __shared__ double s_part[kDenRows][16];
  const bool gq = global_queue != 0;
  int64_t pos = PERSIST ? next_item(tickets, ni, gq, &s_pos) : (gq ? (int64_t)blockIdx.x : xcd_map_runs(blockIdx.x, ni, 128));
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  while (pos < ni) {  // workgroup-uniform
    const BlockItem it = items[pos];
    const int b = it.batch;
    const int g0 = d.batch_pt_off[b], P = d.batch_pt_off[b + 1] - g0;
    const int f0 = d.batch_fn_off[b], n = d.batch_fn_off[b + 1] - f0;
    const int Pp = (int)pad16(P), np = (int)pad16(n);
    const double *pb = panel + d.panel_off[b];
    const int64_t plane = (int64_t)Pp * np;
    const int i0 = 16 * it.rb, j0 = 16 * it.cb;
    const int nrb = min(kDenRows, it.cb + 1 - it.rb);  // row blocks
    double *out = partial + d.batch_part_off[b] + (int64_t)(den_items(it.cb) + it.rb / kDenRows) * P;
    const DenItem x{pb, plane, out, Pp, np, P, i0, j0};
    auto fill = [&]() {
      // coefficients: every thread one column, and rows i0 + e / 16 of the item
      constexpr int NE = (kDenRows * 256 + NTD - 1) / NTD;  // elements per thread
      const int ns = d.batch_slot_off[b + 1] - d.batch_slot_off[b];
      const int64_t spb = d.batch_sp_off[b];
      const int lj = j0 + (tid & 15);
      const SlotFn sj = lj < n ? slot_fn(d, f0, lj) : SlotFn{-1, 0, 0};
      int64_t ea[NE];
#pragma unroll
      for (int u = 0; u < NE; ++u) {
        const int il = (tid + u * NTD) >> 4, li = i0 + il;
        ea[u] = d.store_len;
        if (il < 16 * nrb && li < n && sj.slot >= 0) {
          const SlotFn si = slot_fn(d, f0, li);
          if (si.slot <= sj.slot) {
            const int64_t po = d.sp_poff[spb + (int64_t)si.slot * ns - (int64_t)si.slot * (si.slot - 1) / 2 +
                                         (sj.slot - si.slot)];
            if (po >= 0) ea[u] = po + (int64_t)(li - si.fnoff) * sj.nfn + (lj - sj.fnoff);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < NE; ++u) {
        const int il = (tid + u * NTD) >> 4;
        if (il >= 16 * nrb) break;
        const dbl2 *e = reinterpret_cast<const dbl2 *>(cf + kFold * ea[u]);
        double c[8];
#pragma unroll
        for (int k = 0; k < (FORM == DEN_F64 ? 4 : 3); ++k) {
          const dbl2 x = e[k];
          c[2 * k] = x[0];
          c[2 * k + 1] = x[1];
        }
        // row il is K index lk = il % 4 of K step il / 4
        const int kp = il >> 3, h = (il >> 2) & 1, cl = (tid & 15) + 16 * (il & 3);
#pragma unroll
        for (int q = 0; q < NC; ++q) reinterpret_cast<double *>(&sh.c64[kp][q][cl])[h] = c[FORM == DEN_SO ? 1 + q : q];
        if constexpr (F32W) {
#pragma unroll
          for (int q = 0; q < 4; ++q) sh.c32[kp][q][cl][h] = (float)c[1 + q];
        }
      }
    };
    auto run = [&](auto nb) {
      DenChunks<FORM, decltype(nb)::value> c(x, lane);
      c.begin(wave);
      fill();
      __syncthreads();  // the coefficients are visible
      c.run(wave, sh);
    };
    static_assert(kDenRows <= 3, "one branch per row block count");
    if (!F32W && Pp == 16) {
      // one chunk: the waves take the item's row blocks instead of its chunks,
      // and their sums are added in LDS (24 atoms, batches of 8 points: 1.62 -> 1.40
      // ms, of 16 0.87 -> 0.74)
      const DenItem xw{pb, plane, s_part[wave < kDenRows ? wave : 0], Pp, np, P, i0 + 16 * wave, j0};
      DenChunks<FORM, 1> c(xw, lane);
      const bool mine = wave < nrb;  // wave-uniform: the wave has a row block
      if (mine) c.begin(0);
      fill();
      __syncthreads();  // the coefficients are visible
      if (mine) c.chunk(0, sh, 2 * wave);
      __syncthreads();  // the waves' sums are visible
      if (tid < P) {
        double sum = s_part[0][tid];
        for (int r = 1; r < nrb; ++r) sum += s_part[r][tid];
        out[tid] = sum;
      }
    } else if (kDenRows > 2 && nrb == 3)
      run(std::integral_constant<int, 3>{});
    else if (nrb == 2)
      run(std::integral_constant<int, 2>{});
    else
      run(std::integral_constant<int, 1>{});
    if (!PERSIST) return;
    pos = next_item(tickets, ni, gq, &s_pos);  // its first barrier: the coefficients are consumed
  }
}

// Point sums: out[perm[g]] = (w_g if weighted) * sum over the batch's items, in
// eight chains of every eighth item (so their rounding stays small: RMS error of
// n 2.6e-17 -> 2.4e-17 of its terms on 60 atoms, and the loads are in flight together).
__global__ void k_density_points(DevPlan d, int64_t b0, const double *partial, int weight_mode, double *out) {
  const int64_t b = b0 + blockIdx.x;
  const int g0 = d.batch_pt_off[b], P = d.batch_pt_off[b + 1] - g0;
  const int m = (int)(pad16(d.batch_fn_off[b + 1] - d.batch_fn_off[b]) >> 4);
  const int ni = den_items(m);
  const double *pp = partial + d.batch_part_off[b];
  for (int g = threadIdx.x; g < P; g += blockDim.x) {
    double c[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int t = 0;
    for (; t + 8 <= ni; t += 8)
#pragma unroll
      for (int u = 0; u < 8; ++u) c[u] += pp[(int64_t)(t + u) * P + g];
#pragma unroll
    for (int u = 0; u < 7; ++u)
      if (t + u < ni) c[u] += pp[(int64_t)(t + u) * P + g];
    const double s = ((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]));
    out[d.perm[g0 + g]] = weight_mode ? d.pw[g0 + g] * s : s;
  }
}

}  // namespace

int launch_density_fold(const q4c_plan *p, const double *coef, uint32_t terms, int precision, hipStream_t s) {
  if (p->n_pairs <= 0) return Q4C_OK;
  TimedLaunch tl_(p, Q4C_TIMER_OTHER, s);
  hipLaunchKernelGGL(k_coef_fold, dim3((unsigned)p->n_pairs), dim3(256), 0, s, p->dp, coef, terms,
                     den_form(precision, terms) == DEN_F64, p->d_coef_fold);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? hip_fail(e, "k_coef_fold") : Q4C_OK;
}

int launch_density_pass(const q4c_plan *p, const Pass &ps, uint32_t terms, int precision, int weight_mode,
                        const double *panel, double *partial, unsigned *tickets, double *out, hipStream_t s) {
  const LaunchCfg cfg = p->cfg_density;
  const int64_t ni = ps.di1 - ps.di0, nb = ps.b1 - ps.b0;
  const BlockItem *items = (cfg.order ? p->d_den_cost : p->d_den) + ps.di0;
  const unsigned grid = (unsigned)(tickets ? std::min<int64_t>(cfg.persistent, ni) : ni);
  if (ni > 0) {
    {
      TimedLaunch tl_(p, Q4C_TIMER_DENSITY_TILES, s);
      auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(NTD), 0, s, p->dp, items, ni, (int)cfg.order,
                           (const double *)p->d_coef_fold, panel, partial, tickets);
      };
      switch (den_form(precision, terms)) {
        case DEN_F32W: tickets ? launch(k_density_items<DEN_F32W, true>) : launch(k_density_items<DEN_F32W, false>); break;
        case DEN_SO: tickets ? launch(k_density_items<DEN_SO, true>) : launch(k_density_items<DEN_SO, false>); break;
        default: tickets ? launch(k_density_items<DEN_F64, true>) : launch(k_density_items<DEN_F64, false>);
      }
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_density_items");
  }
  if (nb > 0) {
    {
      TimedLaunch tl_(p, Q4C_TIMER_DENSITY_POINTS, s);
      hipLaunchKernelGGL(k_density_points, dim3((unsigned)nb), dim3(256), 0, s, p->dp, ps.b0, (const double *)partial,
                         weight_mode, out);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "k_density_points");
  }
  return Q4C_OK;
}

}  // namespace q4c
