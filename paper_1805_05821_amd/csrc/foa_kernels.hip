// HIP kernels (gfx950) of one FOA push: one iteration of the snapshot loop of
// Algorithm 1 of Anantharamu & Mahesh, restructured as three fused row passes
// over the basis.
//
// The paper's literal schedule sweeps V five times per snapshot (forming w,
// the projection, the first orthogonalisation, the reprojection and the
// second orthogonalisation).  Each pair -- w and its projection, the first
// orthogonalisation and the reprojection, the second orthogonalisation and
// the norm -- is "apply a row-local update with coefficients known before the
// pass, then reduce over the rows", so one pass over V serves both halves;
// the two projections must finish globally before the next update, so three
// sweeps is the minimum for classical Gram-Schmidt with one
// reorthogonalisation.
//
//   pass A : w = (psi - V b) / beta_jj ; partial V^T w ; partial ||psi||^2
//   reduce : h = V^T w
//   pass B : w = w - V h ; partial V^T w
//   reduce : s = V^T w ; h = h + s
//   pass C : w = w - V s ; v_{j+1} <- w ; partial ||w||^2
//   finalize: h_{j+1,j} = ||w||, breakdown test, H_bar column, beta
//             completion, then the next push's partial beta column
//             (eq. betacolumnupdate) in a small multi-block kernel.
//
// The basis is stored unnormalised: column c holds fl(w_c) and
// v_c = sigma_c * column_c with sigma_c = 1 / h_{c,c-1} (sigma_1 = 1/beta_11).
// Every coefficient vector handed to a pass is pre-multiplied by sigma and every
// projection is post-multiplied by sigma, so the normalisation's division
// never needs its own sweep over n.  All dot products, norms and small-matrix arithmetic are FP64.
//
// Reductions are deterministic: every partial sum has a fixed association
// (per-lane register sums in panel order, butterfly within a wavefront, fixed
// per-block order); no floating-point atomics are used.

#include <type_traits>

#include "foa_device.h"


namespace foa {

template <typename TV, typename TX, int NW, int QW, int MODE, bool PREF, bool RED>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(pass_waves<TV, QW>()))) void k_pass(PassArgs a) {
  __shared__ double lds[pass_lds_doubles<TV, NW, QW, MODE>()];
  row_pass_body<TV, TX, NW, QW, MODE, PREF, false, RED, true>(a, blockIdx.x, a.P, gridDim.x, blockIdx.x, lds);
}

template <int MODE>
__global__ __launch_bounds__(256) void k_reduce(SmallArgs a) {
  reduce_body<MODE, false, true>(a, blockIdx.x * 4);
}

__global__ __launch_bounds__(256) void k_finalize(SmallArgs a) { finalize_body(a); }
__global__ __launch_bounds__(256) void k_finalize_init(SmallArgs a) { finalize_init_body(a); }
__global__ __launch_bounds__(1024) void k_finalize_next(SmallArgs a) {
  static_assert(kStreamSlots <= 4 * 256, "slots of a pass: one round of loads");
  finalize_next_body<kFinNextCols>(a);
}
__global__ __launch_bounds__(256) void k_nextb(SmallArgs a) { nextb_body(a, blockIdx.x); }

__global__ __launch_bounds__(256) void k_init_state(SmallArgs a, double tol) { init_state_body(a, tol); }

// Basis columns out of the panel layout: VEC consecutive rows of CU columns per
// thread, 256 VEC rows of a column per workgroup.  Where the caller's rows and
// columns are aligned to it, VEC is 16 bytes of the basis and a column at a time is
// enough; else a row at a time, four columns in flight.  Bound: HBM, half of it
// writes (a plain copy runs at 4.7 TB/s); those of an unaligned column end inside a
// line, so they go out in long pieces.  2^20 x 100, us, FP32 to FP32 / FP64 to FP64:
// aligned 158 / 311 (64 threads along the rows, four columns each, 163 / 339; an
// element per thread 259 / 334), 2^20 + 1 rows 185 / 337 (249 / 431; 270 / 347).
template <typename TV, typename TO, int VEC, int CU>
__global__ __launch_bounds__(256) void k_copy_basis(const TV *W, const double *sigma, int64_t r0, int64_t nrows,
                                                    int n_max, int ncols, TO *out, int64_t ld) {
  typedef TV tv __attribute__((ext_vector_type(VEC)));
  typedef TO to __attribute__((ext_vector_type(VEC)));
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * VEC;
  const int c0 = (int)blockIdx.y * CU;
  if (i >= nrows) return;
  const int64_t r = r0 + i;  // VEC rows from r lie in one panel
  const TV *src = W + (size_t)(r / PANEL) * n_max * PANEL + r % PANEL;
  tv v[CU];
#pragma unroll
  for (int u = 0; u < CU; ++u) v[u] = *reinterpret_cast<const tv *>(src + (size_t)min(c0 + u, ncols - 1) * PANEL);
#pragma unroll
  for (int u = 0; u < CU; ++u) {
    if (c0 + u >= ncols) break;
    const double sg = sigma[c0 + u];
    TO *o = out + (size_t)(c0 + u) * ld + i;
    if (i + VEC <= nrows) {
      to w;
#pragma unroll
      for (int e = 0; e < VEC; ++e) w[e] = (TO)(sg * (double)v[u][e]);
      *reinterpret_cast<to *>(o) = w;
    } else {
      for (int e = 0; i + e < nrows; ++e) o[e] = (TO)(sg * (double)v[u][e]);
    }
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Smallest QW in {1, 2, 4, 8, 16} whose instance covers j columns when one
// QW step spans cols_per_qw columns.
int pick_qw(int j, int cols_per_qw) {
  int qw = 1;
  while (qw < 16 && qw * cols_per_qw < j) qw *= 2;
  return qw;
}

int tile_slot(int qw) {
  switch (qw) {
    case 1: return 0;
    case 2: return 1;
    case 4: return 2;
    case 8: return 3;
    case 16: return 4;
    case 6: return 5;
    default: return 6;
  }
}

// The FP32 pass has 6- and 12-group tiles where the power-of-two tile would
// be a third to a half empty and the narrower one measured faster at
// n = 2^24: 8 x 6 for 129-192 columns (about 2%), 8 x 12 for 257-320 (about
// 2%) and 16 x 6 for 321-384 (about 5%; 16 x 6 for 257-320 was 6% slower
// than 8 x 16, and 8 x 12 for 321-384 no faster than 16 x 6).
int pass_qw(bool tv_f64, int nw, int j) {
  if (!tv_f64 && ((nw == 8 && j > 128 && j <= 192) || (nw == 16 && j > 320 && j <= 384))) return 6;
  if (!tv_f64 && nw == 8 && j > 256 && j <= 320) return 12;
  return pick_qw(j > 0 ? j : 1, nw * (tv_f64 ? 2 : 4));
}

// Tile widths QW that a workgroup of NW wavefronts is launched with: an FP64 basis
// takes each workgroup over its own range of basis sizes (pass_nw), an FP32 basis
// may be asked for any (option nw).
template <typename TV, int NW, int QW>
constexpr bool pass_shape() {
  if (sizeof(TV) == 8) return NW == 4 ? QW <= 8 && QW != 6 : (NW == 8 ? QW == 8 || QW == 16 : QW == 16);
  return QW == 6 ? NW >= 8 : (QW == 12 ? NW == 8 : NW * QW * 4 <= 512);
}

template <typename TV, typename TX, int NW, int QW, int MODE, bool PREF, bool RED>
static hipError_t launch_pass_s(int grid, const PassArgs &a, hipStream_t s) {
  if constexpr (MODE == PM_INIT || pass_shape<TV, NW, QW>()) {
    hipLaunchKernelGGL((k_pass<TV, TX, NW, QW, MODE, PREF, RED>), dim3(grid), dim3(NW * 64), 0, s, a);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <typename TV, typename TX, int NW, int MODE, bool PREF, bool RED>
static hipError_t launch_pass_q(int qw, int grid, const PassArgs &a, hipStream_t s) {
  switch (qw) {
    case 1: return launch_pass_s<TV, TX, NW, 1, MODE, PREF, RED>(grid, a, s);
    case 2: return launch_pass_s<TV, TX, NW, 2, MODE, PREF, RED>(grid, a, s);
    case 4: return launch_pass_s<TV, TX, NW, 4, MODE, PREF, RED>(grid, a, s);
    case 6: return launch_pass_s<TV, TX, NW, 6, MODE, PREF, RED>(grid, a, s);
    case 8: return launch_pass_s<TV, TX, NW, 8, MODE, PREF, RED>(grid, a, s);
    case 12: return launch_pass_s<TV, TX, NW, 12, MODE, PREF, RED>(grid, a, s);
    default: return launch_pass_s<TV, TX, NW, 16, MODE, PREF, RED>(grid, a, s);
  }
}

// Register budget: a 16-group FP64 tile (64 VGPRs) cannot be double buffered
// within the 128 VGPRs a 16-wavefront workgroup allows.
template <typename TV, int NW>
static bool prefetch_fits(int qw) {
  return !(sizeof(TV) == 8 && NW == 16 && qw >= 16);
}

template <typename TV, typename TX, int NW>
static hipError_t launch_pass_m(int mode, bool pref, int grid, const PassArgs &a, hipStream_t s) {
  const int qw = pass_qw(sizeof(TV) == 8, NW, a.j);
  if (qw * NW * Vec<TV>::EPL < a.j) return hipErrorInvalidValue;  // tile narrower than the basis
  pref = pref && prefetch_fits<TV, NW>(qw);
  auto go = [&](auto m) -> hipError_t {
    constexpr int M = decltype(m)::value;
    if (a.rstride)
      return pref ? launch_pass_q<TV, TX, NW, M, true, true>(qw, grid, a, s)
                  : launch_pass_q<TV, TX, NW, M, false, true>(qw, grid, a, s);
    return pref ? launch_pass_q<TV, TX, NW, M, true, false>(qw, grid, a, s)
                : launch_pass_q<TV, TX, NW, M, false, false>(qw, grid, a, s);
  };
  switch (mode) {
    case PM_INIT: return launch_pass_s<TV, TX, NW, 1, PM_INIT, false, false>(grid, a, s);
    case PM_A: return go(std::integral_constant<int, PM_A>{});
    case PM_B: return go(std::integral_constant<int, PM_B>{});
    default: return go(std::integral_constant<int, PM_C>{});
  }
}

// Wavefronts per row-pass workgroup: an FP64 basis 4 up to 64 columns, 8 up to 256
// and 16 beyond; an FP32 basis nw_opt (4, 8 or 16) if set, else 4 up to 128
// columns, 8 up to 320 and 16 beyond.  At small basis sizes a panel carries little
// data and the pass is bound by the per-panel barriers and LDS round trips, which
// smaller, independent workgroups overlap better.  FP64, us per push, 16
// wavefronts at every size / so: 2^20 x 32 163 / 98, 2^20 x 64 200 / 162, 2^18 x
// 64 62 / 50, 100037 x 200 66 / 60, 4096 x 64 20.5 / 18.9, 2^20 x 256 538 / 521
// (with 4 up to 128 columns 2^20 x 128 takes 293 instead of 288).  FP32 above 320
// columns: 16 wavefronts of 8 groups (128 VGPRs, 4 wavefronts per SIMD) beat 8 of
// 16 groups (one workgroup of 8 per CU).  Between 257 and 320 columns the
// 8-group tile is half empty and the n = 1e8 run was 2.5% slower with it.
int pass_nw(bool tv_f64, int nw_opt, int j) {
  if (tv_f64) return j <= 64 ? 4 : (j <= 256 ? 8 : 16);
  if (nw_opt == 4 && j > 256) return 8;  // 4 wavefronts cover at most 256 columns
  if (nw_opt > 0) return nw_opt;
  return j <= 128 ? 4 : (j <= 320 ? 8 : 16);
}

template <typename TV>
static hipError_t launch_pass_v(int mode, bool tx_f64, bool prefetch, int nw, int grid, const PassArgs &a,
                                hipStream_t s) {
  if (nw == 4)
    return tx_f64 ? launch_pass_m<TV, double, 4>(mode, prefetch, grid, a, s)
                  : launch_pass_m<TV, float, 4>(mode, prefetch, grid, a, s);
  if (nw == 8)
    return tx_f64 ? launch_pass_m<TV, double, 8>(mode, prefetch, grid, a, s)
                  : launch_pass_m<TV, float, 8>(mode, prefetch, grid, a, s);
  return tx_f64 ? launch_pass_m<TV, double, 16>(mode, prefetch, grid, a, s)
                : launch_pass_m<TV, float, 16>(mode, prefetch, grid, a, s);
}

hipError_t launch_pass(int mode, bool tv_f64, bool tx_f64, bool prefetch, int nw, int grid,
                       const PassArgs &a, hipStream_t s) {
  return tv_f64 ? launch_pass_v<double>(mode, tx_f64, prefetch, nw, grid, a, s)
                : launch_pass_v<float>(mode, tx_f64, prefetch, nw, grid, a, s);
}

// Resident workgroups per CU of the pass-A kernel for tile width qw (the
// widest register footprint of the three passes at that width).
template <typename TV, typename TX, int NW, int QW>
static int occ_q(bool pref) {
  int nb = 0;
  if constexpr (pass_shape<TV, NW, QW>()) {
    const void *f = pref ? reinterpret_cast<const void *>(&k_pass<TV, TX, NW, QW, PM_A, true, false>)
                         : reinterpret_cast<const void *>(&k_pass<TV, TX, NW, QW, PM_A, false, false>);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, NW * 64, 0) != hipSuccess) return 1;
  }
  return nb > 0 ? nb : 1;
}

template <typename TV, typename TX, int NW>
static int occ_m(int qw, bool pref) {
  pref = pref && prefetch_fits<TV, NW>(qw);
  switch (qw) {
    case 1: return occ_q<TV, TX, NW, 1>(pref);
    case 2: return occ_q<TV, TX, NW, 2>(pref);
    case 4: return occ_q<TV, TX, NW, 4>(pref);
    case 6: return occ_q<TV, TX, NW, 6>(pref);
    case 8: return occ_q<TV, TX, NW, 8>(pref);
    case 12: return occ_q<TV, TX, NW, 12>(pref);
    default: return occ_q<TV, TX, NW, 16>(pref);
  }
}

template <typename TV, typename TX>
static int occ_v(bool prefetch, int nw, int qw) {
  if (nw == 4) return occ_m<TV, TX, 4>(qw, prefetch);
  return nw == 8 ? occ_m<TV, TX, 8>(qw, prefetch) : occ_m<TV, TX, 16>(qw, prefetch);
}

int pass_occupancy(bool tv_f64, bool tx_f64, bool prefetch, int nw, int qw) {
  if (tv_f64) return tx_f64 ? occ_v<double, double>(prefetch, nw, qw) : occ_v<double, float>(prefetch, nw, qw);
  return tx_f64 ? occ_v<float, double>(prefetch, nw, qw) : occ_v<float, float>(prefetch, nw, qw);
}

hipError_t launch_reduce(int mode, const SmallArgs &a, hipStream_t s) {
  const int waves = a.j + (mode == 1 ? 1 : 0);
  const int blocks = (waves + 3) / 4;
  if (mode == 1)
    hipLaunchKernelGGL(k_reduce<1>, dim3(blocks), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(k_reduce<2>, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_finalize(const SmallArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_finalize_next(const SmallArgs &a, hipStream_t s) {
  if (a.j < 1 || a.j > kFinNextCols) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_finalize_next, dim3(1), dim3(1024), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_finalize_init(const SmallArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_finalize_init, dim3(1), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_nextb(const SmallArgs &a, hipStream_t s) {
  // J = q after the push is at most j + 1 (host expectation).
  const int J = a.j + 1;
  const int blocks = (J + 63) / 64;
  hipLaunchKernelGGL(k_nextb, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_init_state(const SmallArgs &a, double tol, hipStream_t s) {
  hipLaunchKernelGGL(k_init_state, dim3(64), dim3(256), 0, s, a, tol);
  return hipGetLastError();
}

template <typename TV, typename TO>
static hipError_t copy_basis_t(const void *W, const double *sigma, int64_t r0, int64_t nrows, int n_max, int ncols,
                               void *out, int64_t ld, hipStream_t s) {
  constexpr int VEC = Vec<TV>::EPL;
  const bool vec = r0 % VEC == 0 && ld % VEC == 0 && reinterpret_cast<uintptr_t>(out) % (VEC * sizeof(TO)) == 0;
  const int rows = 256 * (vec ? VEC : 1), cu = vec ? 1 : 4;
  const dim3 grid((unsigned)((nrows + rows - 1) / rows), (unsigned)((ncols + cu - 1) / cu));
  if (vec)
    hipLaunchKernelGGL((k_copy_basis<TV, TO, VEC, 1>), grid, dim3(256), 0, s, (const TV *)W, sigma, r0, nrows, n_max, ncols,
                       (TO *)out, ld);
  else
    hipLaunchKernelGGL((k_copy_basis<TV, TO, 1, 4>), grid, dim3(256), 0, s, (const TV *)W, sigma, r0, nrows, n_max, ncols,
                       (TO *)out, ld);
  return hipGetLastError();
}

hipError_t launch_copy_basis(bool tv_f64, const void *W, const double *sigma, int64_t r0, int64_t nrows,
                             int n_max, int ncols, void *out, int64_t ld, bool out_f64, hipStream_t s) {
  if (ncols <= 0 || nrows <= 0) return hipSuccess;
  if (tv_f64)
    return out_f64 ? copy_basis_t<double, double>(W, sigma, r0, nrows, n_max, ncols, out, ld, s)
                   : copy_basis_t<double, float>(W, sigma, r0, nrows, n_max, ncols, out, ld, s);
  return out_f64 ? copy_basis_t<float, double>(W, sigma, r0, nrows, n_max, ncols, out, ld, s)
                 : copy_basis_t<float, float>(W, sigma, r0, nrows, n_max, ncols, out, ld, s);
}

}  // namespace foa
