// Pushes of a small stream: one workgroup takes a run of snapshots through the
// whole push (passes A, B, C, the reductions, finalize and the next partial beta
// column, foa_device.h) in one launch, with the basis in its registers.
//
// Bound: latency.  Streams this small leave the chip idle whatever the split, and
// a push of four kernels (A, B, C, finalize) takes 17-19 us however few its rows:
// launches, and each kernel's first loads.  Here a push is a chain of five barriers
// on one CU with no memory between them but the snapshot and the new column.
//
// Tile: 16 wavefronts; wavefront w holds panels w, w + 16, .. (NP of them) of the
// basis, QB groups of 1 KiB each (16 bytes a lane, as in row_pass_body), so
// NP * QB = 16 groups are 64 of the 128 VGPRs a wavefront of such a workgroup
// has.  The rows' sums and w stay in the wavefront, one row of a panel per lane; a
// panel's column sums and norm go through LDS, where the small matrices of the run
// (H_bar, the coefficients) live as well, so nothing stored is read back.
//
// Every sum is formed in the order of the kernels this replaces (one workgroup per
// panel of 4 wavefronts there), so H_bar, beta and the basis are bitwise theirs.
#include "foa_device.h"

namespace foa {

// Sums of v[e], e < EPL, over the lanes that share rows (as xor_sum<16>, then
// xor_sum<32>), each lane keeping the one of row e = lane / (64 / EPL).
__device__ __forceinline__ double swap_add32(double a, double b) {
  const u32x2 x = __builtin_bit_cast(u32x2, a), y = __builtin_bit_cast(u32x2, b);
  const auto lo = __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false);
  return __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
}
__device__ __forceinline__ double swap_add16(double a, double b) {
  const u32x2 x = __builtin_bit_cast(u32x2, a), y = __builtin_bit_cast(u32x2, b);
  const auto lo = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
  return __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
}
__device__ __forceinline__ double row_scatter(const double (&v)[4]) {
  return swap_add32(swap_add16(v[0], v[1]), swap_add16(v[2], v[3]));
}
__device__ __forceinline__ double row_scatter(const double (&v)[2]) { return swap_add32(v[0], v[1]); }

// The inverse: every lane gets the values of the rows e < EPL.
__device__ __forceinline__ void row_gather(double v, double (&o)[2]) {
  const u32x2 x = __builtin_bit_cast(u32x2, v);
  const auto lo = __builtin_amdgcn_permlane32_swap(x.x, x.x, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(x.y, x.y, false, false);
  o[0] = __builtin_bit_cast(double, u32x2{lo[0], hi[0]});
  o[1] = __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
}
__device__ __forceinline__ void row_gather(double v, double (&o)[4]) {
  double h[2];
  row_gather(v, h);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const u32x2 x = __builtin_bit_cast(u32x2, h[k]);
    const auto lo = __builtin_amdgcn_permlane16_swap(x.x, x.x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(x.y, x.y, false, false);
    o[2 * k] = __builtin_bit_cast(double, u32x2{lo[0], hi[0]});
    o[2 * k + 1] = __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
  }
}

// Barrier of the workgroup for LDS contents only: stores to memory stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <typename TV, typename TX, int NP, int QB>
__global__ __launch_bounds__(1024) void k_push_small(PassArgs a, SmallArgs sa, int64_t ldx, int count) {
#pragma clang fp contract(off)  // as in row_pass_body
  constexpr int EPL = Vec<TV>::EPL, LPC = 64 / EPL, CPW = EPL, JC = QB * CPW;
  constexpr int NWO = 4;                         // wavefronts of a workgroup of k_pass at these sizes
  constexpr int LP = 16 * NP;                    // lanes of a column in the reductions
  static_assert(NP * QB <= 16 && 16 * (64 / LP) >= JC && JC <= 64, "register tile, one reduction step");
  __shared__ double s_coef[JC + 1], s_sig[JC + 1], s_bv[JC + 1], s_h[JC + 1], s_b[JC + 1];
  __shared__ double s_H[JC][JC + 1];  // [column][row]
  __shared__ double s_part[16 * NP][JC + 1];
  __shared__ double s_pn[2][16 * NP];
  __shared__ double s_p[8][64];
  __shared__ double s_xf, s_lim, s_xn, s_hn, s_bd, s_ihn, s_scale;
  __shared__ int s_bad, s_status;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cs = lane / LPC, rg = lane % LPC;
  const int row = rg * EPL + cs;  // this lane's row of a panel
  const int P = (int)a.P, j0 = a.j;
  const size_t pbytes = (size_t)a.n_max * PANEL * sizeof(TV);
  char *Wb = static_cast<char *>(const_cast<void *>(a.W));
  DevState *st = sa.st;

  auto load_x = [&](int k, int i) {
    const TX *x = static_cast<const TX *>(a.x) + (size_t)k * ldx;
    const int64_t r0 = (int64_t)(wave + 16 * i) * PANEL, rem = a.n - r0;
    const int rows = (int)(rem >= PANEL ? PANEL : (rem > 0 ? rem : 0));
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(x + (rows > 0 ? r0 : 0), (unsigned)(rows * sizeof(TX)));
    return buf_load_raw<TX>(rx, (unsigned)(row * sizeof(TX)));
  };

  const int status0 = uniform(st->status);
  if (status0 != ST_ACTIVE) {
    if (tid == 0) st->pushes += count;
    return;
  }
  TV t[NP][QB][EPL];
  TX xr[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int p = wave + 16 * i;
    const __amdgpu_buffer_rsrc_t r =
        make_rsrc(Wb + (size_t)(p < P ? p : 0) * pbytes, p < P ? (unsigned)(j0 * PANEL * sizeof(TV)) : 0u);
    xr[i] = load_x(0, i);
#pragma unroll
    for (int b = 0; b < QB; ++b)
      unpack16<TV>(__builtin_amdgcn_raw_buffer_load_b128(r, lane * 16 + b * 1024, 0, 0), t[i][b]);
  }
  // the state a push starts from; the scalars are the same in every thread
  double scale = uniform(st->scaleA), xfro2 = uniform(st->xfro2);
  double bjj = uniform(sa.beta[(size_t)(j0 - 1) * sa.ldB + (j0 - 1)]);
  const double tol = uniform(st->tol);
  for (int c = tid; c < JC + 1; c += 1024) {
    s_coef[c] = c < j0 ? sa.coefA[c] : 0.0;
    s_sig[c] = c < j0 ? sa.sigma[c] : 0.0;
    s_bv[c] = c < j0 ? sa.bvec[c] : 0.0;
  }
#pragma unroll
  for (int l0 = 0; l0 < JC; l0 += 16) {
    const int l = l0 + wave;
    if (l < j0 - 1 && lane < j0) s_H[l][lane] = sa.H[(size_t)l * sa.ldH + lane];
  }
  if (tid == 0) s_bad = 0;
  lds_barrier();

  int k = 0, status = ST_ACTIVE;
  double hlast = uniform(st->hlast);
  for (; k < count && status == ST_ACTIVE; ++k) {
    const int j = j0 + k;
    double w[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      w[i] = (double)xr[i];
      if (k + 1 < count) xr[i] = load_x(k + 1, i);
    }

    // the FP32 tile is converted anew by each use (FP64 copies would not fit)
    auto hold = [&](int i) {
#pragma unroll
      for (int b = 0; b < QB; ++b) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) asm volatile("" : "+v"(t[i][b][e]));
      }
    };
    // w - u with u_r = sum_c V_rc coef_c
    auto rows = [&](int i) {
      double us = 0.0;
      if constexpr (sizeof(TV) == 4) hold(i);
#pragma unroll
      for (int w2 = 0; w2 < (QB < NWO ? QB : NWO); ++w2) {
        double u[EPL];
#pragma unroll
        for (int e = 0; e < EPL; ++e) u[e] = 0.0;
#pragma unroll
        for (int b = w2; b < QB; b += NWO) {
          const double cf = s_coef[b * CPW + cs];
#pragma unroll
          for (int e = 0; e < EPL; ++e) u[e] = fma((double)t[i][b][e], cf, u[e]);
        }
        us += row_scatter(u);
        // a few at a time: interleaved, the chains and coefficients of all of them
        // outgrow the 128 VGPRs
        if (w2 % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
      return w[i] - us;
    };
    // V^T w over the panel, a row of s_part
    auto cols = [&](int i) {
      double wr[EPL];
      row_gather(w[i], wr);
      if constexpr (sizeof(TV) == 4) hold(i);
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        if (b % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        double acc = 0.0;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc = fma((double)t[i][b][e], wr[e], acc);
        acc = lanes_sum<LPC>(acc);
        if (rg == 0) s_part[wave + 16 * i][b * CPW + cs] = acc;
      }
    };
    // sum of squares of the panel's rows: butterflies of 64 / NWO rows, then
    // those sums in order
    auto norm2 = [&](double y) {
      double v = y * y;
      if constexpr (EPL == 4) v = xor_sum<16>(v);
      v = xor_sum<32>(v);
      v += dpp_mov<0xB1>(v);
      v += dpp_mov<0x4E>(v);
      if constexpr (EPL == 2) v += dpp_mov<0x141>(v);
      constexpr int LG = LPC / NWO;  // lanes of one such sum
      const u32x2 c = __builtin_bit_cast(u32x2, v);
      double s = 0.0;
#pragma unroll
      for (int g = 0; g < NWO; ++g)
        s += __builtin_bit_cast(double, u32x2{(unsigned)__builtin_amdgcn_readlane((int)c.x, g * LG),
                                              (unsigned)__builtin_amdgcn_readlane((int)c.y, g * LG)});
      return s;
    };
    // the panels' sums of column rc, in lane 0 of its LP lanes
    const int rc = wave * (64 / LP) + lane / LP, rp = lane % LP;
    auto reduce = [&]() { return lanes_sum<LP>(rc < JC && rp < P ? s_part[rp][rc < JC ? rc : 0] : 0.0); };

#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const double nx = norm2(w[i]);
      if (lane == 0) s_pn[0][wave + 16 * i] = nx;
      w[i] = rows(i) * scale;
      cols(i);
    }
    lds_barrier();
    {
      const double tc = reduce();
      if (rp == 0 && rc < j) {
        const double sg = s_sig[rc], v = sg * tc;
        s_h[rc] = v;
        s_coef[rc] = sg * v;
      }
      if (wave == 15) {  // ||psi||^2 and the breakdown limit
        const double xn = lanes_sum<64>(lane < P ? s_pn[0][lane < P ? lane : 0] : 0.0);
        if (lane == 0) {
          s_xn = xn;
          s_xf = xfro2 + xn;
          s_lim = tol * sqrt(xfro2 + xn);
        }
      }
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      w[i] = rows(i);
      cols(i);
    }
    lds_barrier();
    {
      const double tc = reduce();
      if (rp == 0 && rc < j) {
        const double sg = s_sig[rc], v = sg * tc, h = s_h[rc] + v;
        s_h[rc] = h;
        s_coef[rc] = sg * v;
        s_H[j - 1][rc] = h;
        s_b[rc] = fma(h, bjj, s_bv[rc]);  // beta completion
        if (!isfinite(h)) s_bad = 1;
      }
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int p = wave + 16 * i;
      w[i] = rows(i);
      const double wn = norm2(w[i]);
      if (lane == 0) s_pn[1][p] = wn;
      double wr[EPL];
      row_gather(w[i], wr);
      TV o[EPL];
#pragma unroll
      for (int e = 0; e < EPL; ++e) o[e] = (TV)wr[e];
      if (p < P && cs == 0) {
        TV *dst = reinterpret_cast<TV *>(Wb + (size_t)p * pbytes) + (size_t)j * PANEL + rg * EPL;
        *reinterpret_cast<u32x4 *>(dst) = __builtin_bit_cast(u32x4, o);
      }
      // the new column takes its place in the tile (dropped by a full one)
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        const bool in = b * CPW + cs == j;
#pragma unroll
        for (int e = 0; e < EPL; ++e) t[i][b][e] = in ? o[e] : t[i][b][e];
      }
    }
    lds_barrier();
    // finalize_next_body: wavefront 0 the scalars, wavefronts 4 .. 11 the sums of the
    // next partial beta column (64-row chunks x 4 l-slices, but row j)
    const int sl = wave & 3, i = ((wave >> 2) - 1) * 64 + lane;
    if (wave == 0) {
      double wn2 = lane < P ? s_pn[1][lane < P ? lane : 0] : 0.0;
      wn2 = xor_sum<16>(xor_sum<32>(wn2));
      wn2 += dpp_mov<0x128>(wn2);  // row_ror by 8, 4, 2, 1
      wn2 += dpp_mov<0x124>(wn2);
      wn2 += dpp_mov<0x122>(wn2);
      wn2 += dpp_mov<0x121>(wn2);
      const double hn = sqrt(wn2), bd = hn * bjj;
      const double ihn = 1.0 / hn, sc = 1.0 / bd;
      if (lane == 0) {
        s_hn = hn;
        s_bd = bd;
        s_ihn = ihn;
        s_scale = sc;
        s_status = s_bad || !isfinite(hn) || !isfinite(s_xn) ? ST_NONFINITE : (bd <= s_lim ? ST_INVARIANT : ST_ACTIVE);
      }
    } else if (wave >= 4 && wave < 12) {
      const int lo = i > 0 ? i - 1 : 0, len = i < j ? j - lo : 0;
      const int a0 = lo + (len * sl) / 4, a1 = lo + (len * (sl + 1)) / 4;
      double acc = 0.0;
      for (int l = a0; l < a1; ++l) acc = fma(s_H[l][i], s_b[l], acc);
      s_p[wave - 4][lane] = acc;
    }
    lds_barrier();
    status = uniform(s_status);
    if (status == ST_NONFINITE) continue;
    const double hn = s_hn;
    const bool inv = status == ST_INVARIANT;
    hlast = hn;
    xfro2 = s_xf;
    if (tid <= j) {
      sa.H[(size_t)(j - 1) * sa.ldH + tid] = tid < j ? s_h[tid] : (inv ? 0.0 : hn);
      sa.beta[(size_t)j * sa.ldB + tid] = tid < j ? s_b[tid] : (inv ? 0.0 : s_bd);
    }
    if (inv) continue;
    if (wave >= 4 && sl == 0 && i <= j) {
      const int g = wave - 4;
      // row j holds column j - 1 only
      const double b = i < j ? ((s_p[g][lane] + s_p[g + 1][lane]) + s_p[g + 2][lane]) + s_p[g + 3][lane]
                             : hn * s_b[j - 1];
      s_bv[i] = b;
      s_coef[i] = (i < j ? s_sig[i] : s_ihn) * b;
    }
    if (tid == 0) {
      s_sig[j] = s_ihn;
      if (j < JC) s_H[j - 1][j] = hn;
    }
    bjj = s_bd;
    scale = s_scale;
    lds_barrier();
  }

  // what the next launch starts from
  const int q = j0 + k - (status != ST_ACTIVE ? 1 : 0);  // columns committed
  for (int c = tid; c < q; c += 1024) {
    if (c >= j0) sa.sigma[c] = s_sig[c];
    if (status == ST_ACTIVE) {
      sa.bvec[c] = s_bv[c];
      sa.coefA[c] = s_coef[c];
    }
  }
  if (tid == 0) {
    st->q = q;
    st->status = status;
    st->pushes += count;  // those after a stop are offered and ignored
    st->xfro2 = xfro2;
    st->xn2 = s_xn;
    st->scaleA = scale;
    st->hlast = hlast;
  }
}

// Panels a wavefront holds, or 0 if the stream is too tall: with four panels a
// wavefront (4096 rows) the one CU is no faster than the kernels over 64 (FP32, 16
// columns: 19.4 / 17.5 us per push).
static int small_np(int64_t P) { return P <= 16 ? 1 : (P <= 32 ? 2 : 0); }

// A launch reads the tile and the small matrices once for its pushes.  With half
// the tile (8 groups a wavefront) that pays from one push on, with all of it from a
// run of kWideRun on.  us per push, this / the kernels: FP32, 1000 x 24, a run 7.2 /
// 17.6, one launch each 10.9 / 17.6; 1024 rows, 48..64 columns, a run 12.5 / 17.2,
// each 18.9 / 17.2; FP64, 1024 x 32, a run 7.9 / 18.3, each (kernels beyond 16
// columns) 12.9 / 18.5.
constexpr int kWideRun = 8;

int small_push_run(bool tv_f64, int64_t P, int j, int rem) {
  const int np = small_np(P), cpw = tv_f64 ? 2 : 4;
  if (np == 0 || j < 1) return 0;
  int qb = 4;
  while (np * qb <= 16 && qb * cpw < j) qb *= 2;
  if (np * qb > 16) return 0;
  const int room = qb * cpw - j + 1, run = rem < room ? rem : room;
  return np * qb == 16 && run < kWideRun ? 0 : run;
}

template <typename TV, typename TX>
static hipError_t push_small_t(const PassArgs &a, const SmallArgs &sa, int64_t ldx, int count, hipStream_t s) {
  const int np = small_np(a.P);
  int qb = 4;
  while (qb * Vec<TV>::EPL < a.j + count - 1) qb *= 2;
#define FOA_SMALL(NP, QB) \
  case NP * 100 + QB: hipLaunchKernelGGL((k_push_small<TV, TX, NP, QB>), dim3(1), dim3(1024), 0, s, a, sa, ldx, count); break;
  switch (np * 100 + qb) {
    FOA_SMALL(1, 4)
    FOA_SMALL(1, 8)
    FOA_SMALL(1, 16)
    FOA_SMALL(2, 4)
    FOA_SMALL(2, 8)
    default: return hipErrorInvalidValue;
  }
#undef FOA_SMALL
  return hipGetLastError();
}

hipError_t launch_push_small(bool tv_f64, bool tx_f64, const PassArgs &a, const SmallArgs &sa, int64_t ldx, int count,
                             hipStream_t s) {
  if (count < 1 || a.j < 1) return hipErrorInvalidValue;
  if (tv_f64)
    return tx_f64 ? push_small_t<double, double>(a, sa, ldx, count, s) : push_small_t<double, float>(a, sa, ldx, count, s);
  return tx_f64 ? push_small_t<float, double>(a, sa, ldx, count, s) : push_small_t<float, float>(a, sa, ldx, count, s);
}

}  // namespace foa
