// One-reduction form of the FOA step (gfx950).
//
// The modified FOA factorises the snapshots as X = V beta (the QR view of
// Section 3.1) with H_bar following from beta through eq. betacolumnupdate.
// Algorithm 1 orthogonalises with classical Gram-Schmidt applied twice, so a
// push needs three sweeps over the basis and three global reductions.  Here
// the snapshots themselves are orthogonalised and the two projections of
// consecutive snapshots share a sweep (delayed reorthogonalisation, Bielich et
// al., Parallel Computing 2022): the sweep of a push
//   * finishes the pending column: u - Q w, with w = Q^T u from the previous
//     reduction (the second projection);
//   * gives the pending snapshot copy its first projection: x - Q z - q_hat
//     R_tilde, with z = Q^T x and the coefficient on the column just finished,
//     R_tilde = (u^T x - w^T z) / rho_hat, from the previous reduction
//     (rho_hat = sqrt(||u||^2 - ||w||^2), the estimated norm);
//   * copies the new snapshot into the next basis column;
// and forms every column sum the next step needs in the same pass.  One
// fixed-order reduction then gives the exact norm of the finished column, w
// of the new pending column, and z of the new snapshot.  Per push: one sweep
// reading the final columns once, two pending columns read and written, the
// new snapshot read and stored -- about a third of the three-sweep form's
// traffic.  Columns become final two pushes after their snapshot; a flush
// (sweeps without a snapshot) finishes the pending ones.
//
// Storage: column c holds the unnormalised vector, v_c = sigma_c column_c
// with sigma_c = 1 / ||column_c|| (the exact norm of the stored values), as in
// the three-sweep form.  Every dot product, norm and small-matrix operation is
// FP64; stored columns are rounded to the basis precision, and every sum uses
// the rounded values the next sweep will read.
//
// Kernels (all on the context stream):
//   k_ls_pass     : the sweep (tile layout of the blocked passes; two coefficient
//                   vectors in phase 1, two or three right-hand sides in phase 2,
//                   six scalar sums); k_ls_rows: its row form, where that is the
//                   faster one for an FP64 basis;
//   k_ls_reduce   : fixed-order reduction of the workgroup partials;
//   k_ls_finalize : one workgroup: the finished column's norm, scale and
//                   breakdown test, H_bar's column from beta, beta's column of
//                   the new pending column, the next sweep's coefficients.
#include "foa_device.h"

namespace foa {

// ---------------------------------------------------------------------------
// Sweep body.  One workgroup walks units pstart, + pstep, ... < pend (in panels)
// of one stream and writes its partial sums to slot `slot`.  Called uniformly by
// the whole workgroup (it synchronises).
//
// Unit and tile are those of the blocked passes (foa_block.hip): BROWS rows of a
// panel (64 with an FP32 basis; 32 with an FP64 one, both halves up to 2 groups),
// lane l of a wavefront holding the 16-byte chunk l / 4 of column l % 4 of each of
// its QW groups of four of the q final columns.  Phase 1 sums the tile's rows against sigma o w and sigma o z
// (FMA per lane, DPP over the quad, LDS over the wavefronts); the update rows,
// contiguous per wavefront, read the pending column, the snapshot copy and the
// new snapshot; phase 2 forms the column sums on v_mfma_f64_4x4x4, whose four
// right-hand sides take the formed column, the snapshot and, with an FP32 basis,
// the rounding error of the finished column (the Gram correction of the second
// projection; an FP64 basis needs none).  That is one accumulator per group where
// vector FMAs took two FP64 and one FP32 and left the 16-group tile room to
// prefetch half; a tile's registers are refilled for the unit after next as
// phase 2 is done with them, the next unit's row inputs ahead of them.  The three
// columns go out 64 rows at a time.
// Bound: HBM, with three column writes per panel in the read stream.  FP32 basis,
// capacity 500, us per push at 2^21 / 2^22 rows: 225-256 columns 378 / 732, 449-480
// 664 / 1302 (with a 16-group tile 697 / 1357).
// ---------------------------------------------------------------------------
// 16-byte loads of a lane per column group and unit: two for the narrow tiles of an
// FP64 basis, whose units are then whole panels (fewer barriers per row, columns
// written 512 bytes at a time; 2^22 rows, 1-16 columns 175 -> 114 us per push, 17-32
// 219 -> 189; the 4-group tile has no registers for it).
template <typename TV, int NW, int QW>
constexpr int ls_loads() {
  return sizeof(TV) == 8 && QW <= 2 ? 2 : 1;
}
template <typename TV, int NW, int QW>
constexpr int ls_lds_doubles() {
  constexpr int BROWS = 16 * Vec<TV>::EPL * ls_loads<TV, NW, QW>();
  return 2 * QW * NW * 4 + 2 * NW * BROWS * 2 + BROWS * 4 + 3 * BROWS + NW * LS_NSC +
         (QW >= 16 ? LS_NSC * BROWS : 0);
}
template <typename TV, typename TX, int NW, int QW>
__device__ __forceinline__ void ls_pass_body(const LsArgs &a, int64_t pstart, int64_t pend_, int64_t pstep_,
                                             int slot, double *lds) {
#pragma clang fp contract(off)
  constexpr int LPL = Vec<TV>::EPL, EPL = LPL * ls_loads<TV, NW, QW>();  // elements of a load, of a lane
  constexpr int BROWS = 16 * EPL;
  constexpr int UPP = PANEL / BROWS;  // units per panel
  constexpr int JCAP = QW * NW * 4;
  constexpr int RPW = BROWS / NW;     // update rows of a wavefront
  constexpr int GSTRIDE = NW * 4;
  constexpr bool GRAM = sizeof(TV) == 4;

  double *s_coef = lds;                               // [column][w, z]
  double *s_red = s_coef + 2 * JCAP;                  // [parity][wavefront][row][w, z]
  double *s_w = s_red + 2 * NW * BROWS * 2;           // [row][right-hand side]
  TV *s_col = reinterpret_cast<TV *>(s_w + BROWS * 4);  // [finished, formed, copied][row of the unit]
  double (*s_sc)[LS_NSC] = reinterpret_cast<double (*)[LS_NSC]>(s_w + BROWS * 4 + 3 * BROWS);

  const DevState *st = a.st;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cl = lane & 3;

  // step state (uniform)
  const int q = uniform(st->q);
  const int hu = uniform(st->ls_u);
  const int hf = uniform(st->ls_x);
  const int hn = a.flush ? 0 : 1;
  const int cc = q;            // column under its second projection
  const int cf = q + hu;       // snapshot copy that gets its first projection
  const int cn = cf + hf;      // column the new snapshot is copied to
  const double cq = hu && hf ? uniform(st->ls_cq) : 0.0;

  __syncthreads();  // the previous call of this workgroup may still read LDS
  for (int c = tid; c < JCAP; c += NW * 64) {
    s_coef[2 * c] = c < q ? a.coefW[c] : 0.0;
    s_coef[2 * c + 1] = c < q ? a.coefZ[c] : 0.0;
  }
  __syncthreads();

  const int cbase = wave * 4 + cl;
  const unsigned goff0 = (unsigned)(cbase * PANEL * sizeof(TV)) + (unsigned)(lane >> 2) * 16u;
  constexpr unsigned GBYTES = (unsigned)(GSTRIDE * PANEL * sizeof(TV));  // group to group, in a scalar register
  const unsigned tile_bytes = (unsigned)(q * PANEL * sizeof(TV));
  const bool uact = lane < RPW;
  const int urow = wave * RPW + (lane & (RPW - 1));
  // its place in the tile's row order
  const int upos = (urow / (16 * LPL) * LPL + urow % LPL) * 16 + urow % (16 * LPL) / LPL;
  const unsigned pan_bytes = (unsigned)((size_t)a.n_max * PANEL * sizeof(TV));
  // byte offsets of the pending columns inside a panel (kOOR: absent)
  const unsigned ocu = hu ? (unsigned)(cc * PANEL * sizeof(TV)) : kOOR;
  const unsigned ocf = hf ? (unsigned)(cf * PANEL * sizeof(TV)) : kOOR;
  const unsigned ocn = hn ? (unsigned)(cn * PANEL * sizeof(TV)) : kOOR;
  const unsigned urb = (unsigned)(urow * sizeof(TV));

  double acc[QW];
#pragma unroll
  for (int g = 0; g < QW; ++g) acc[g] = 0.0;
  // the scalar sums of an update row; the widest tile leaves no registers for
  // them and keeps them in LDS (each read and written by its own lane only)
  constexpr bool SCL = QW >= 16;
  double *s_acc = s_w + BROWS * 4 + 3 * BROWS + NW * LS_NSC;
  double sc[LS_NSC];
#pragma unroll
  for (int k = 0; k < LS_NSC; ++k) sc[k] = 0.0;
  if (SCL && uact)
    for (int k = 0; k < LS_NSC; ++k) s_acc[k * BROWS + urow] = 0.0;

  char *Wb = static_cast<char *>(a.W);
  const size_t pbytes = (size_t)a.n_max * PANEL * sizeof(TV);
  TV ta[QW][EPL], tb[QW][EPL];

  // units (32-bit and scalar, see the blocked passes): u = unit * UPP + half
  const int pend = (int)pend_ * UPP, pstep = (int)pstep_;
  const int nfull = (int)(a.n / BROWS), nrem = (int)(a.n % BROWS);
  // walk of the workgroup: panels pstart, + pstep, ..., both halves of each
  auto unit_of = [&](int i) { return UPP == 1 ? (int)pstart + i * pstep : ((int)pstart + (i >> 1) * pstep) * 2 + (i & 1); };
  auto rsrc_of = [&](int u, unsigned bytes) {
    const int v = u < pend ? u : 0;
    const unsigned half = UPP > 1 ? (unsigned)(v % UPP) * (unsigned)(BROWS * sizeof(TV)) : 0u;
    return make_rsrc(Wb + (size_t)(v / UPP) * pbytes + half, u < pend && bytes > half ? bytes - half : 0u);
  };
  auto load_group = [&](const __amdgpu_buffer_rsrc_t &r, int g, TV (&dst)[EPL]) {
#pragma unroll
    for (int h = 0; h < EPL / LPL; ++h) {
      TV v[LPL];
      unpack16<TV>(__builtin_amdgcn_raw_buffer_load_b128(
                       r, (int)(goff0 + h * 16 * LPL * sizeof(TV)), (int)(g * GBYTES), kTileLoad), v);
#pragma unroll
      for (int e = 0; e < LPL; ++e) dst[h * LPL + e] = v[e];
    }
  };
  TV yu, yf;
  TX xr;
  auto load_rows = [&](int u) {
    const __amdgpu_buffer_rsrc_t rp = rsrc_of(u, pan_bytes);
    yu = buf_load_raw<TV>(rp, uact && hu ? ocu + urb : kOOR);
    yf = buf_load_raw<TV>(rp, uact && hf ? ocf + urb : kOOR);
    const int v = u < pend ? u : 0;
    const int valid = u >= pend || !hn ? 0 : (u < nfull ? BROWS : (u == nfull ? nrem : 0));
    xr = buf_load_raw<TX>(make_rsrc(static_cast<const TX *>(a.x) + (hn ? (size_t)v * BROWS : 0),
                                    (unsigned)(BROWS * sizeof(TX))),
                          uact && urow < valid ? (unsigned)(urow * sizeof(TX)) : kOOR);
  };

  int par = 0;
  auto step = [&](int u, int u1, int u2, TV (&t)[QW][EPL]) {
    const __amdgpu_buffer_rsrc_t rt = rsrc_of(u2, tile_bytes);
    // phase 1
    double s[2][EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) s[0][e] = s[1][e] = 0.0;
    // coefficients of group g + CD are read while group g's products run (read next
    // to their use, 385-416 columns of an FP32 basis took 2% longer)
    constexpr int CD = QW >= 8 ? 1 : 2;
    double cw[CD + 1][2];
    auto read_cf = [&](int g) {
#pragma unroll
      for (int k = 0; k < 2; ++k) cw[g % (CD + 1)][k] = s_coef[2 * (cbase + g * GSTRIDE) + k];
    };
#pragma unroll
    for (int g = 0; g < (CD < QW ? CD : QW); ++g) read_cf(g);
#pragma unroll
    for (int g = 0; g < QW; ++g) {
      if (g + CD < QW) read_cf(g + CD);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int e = 0; e < EPL; ++e) s[k][e] = fma((double)t[g][e], cw[g % (CD + 1)][k], s[k][e]);
      __builtin_amdgcn_sched_barrier(0);
    }
    double *red = s_red + par * NW * BROWS * 2;
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      const bool b0 = cl & 1;  // lanes 0, 2 of a quad end with the sum against w, 1, 3 against z
      double r = (b0 ? s[1][e] : s[0][e]) + dpp_mov<0xB1>(b0 ? s[0][e] : s[1][e]);
      r += dpp_mov<0x4E>(r);
      if (cl < 2) red[wave * BROWS * 2 + (e * 16 + (lane >> 2)) * 2 + cl] = r;
    }
    __syncthreads();
    double sw = 0.0, sz = 0.0;
#pragma unroll
    for (int w2 = 0; w2 < NW; ++w2) {
      sw += red[w2 * BROWS * 2 + upos * 2];
      sz += red[w2 * BROWS * 2 + upos * 2 + 1];
    }
    // row update: finished column, formed column, snapshot copy (each rounded
    // to the storage type; the sums below use the rounded values)
    const double yud = (double)yu, xv = (double)xr;
    const TV ut_s = (TV)(yud - sw);
    const double ut = (double)ut_s;
    const TV uf_s = (TV)(((double)yf - sz) - ut * cq);
    const double uf = (double)uf_s;
    const TV xs_s = (TV)xv;
    const double xs = (double)xs_s;
    if (uact) {
      auto add = [&](int k, double p, double q2) {
        if constexpr (SCL)
          s_acc[k * BROWS + urow] = fma(p, q2, s_acc[k * BROWS + urow]);
        else
          sc[k] = fma(p, q2, sc[k]);
      };
      add(LS_UU, ut, ut);
      add(LS_UF, ut, uf);
      add(LS_UX, ut, xs);
      add(LS_FF, uf, uf);
      add(LS_FX, uf, xs);
      add(LS_XX, xv, xv);
      s_w[upos * 4] = uf;
      s_w[upos * 4 + 1] = xs;
      s_w[upos * 4 + 2] = GRAM ? ut - (yud - sw) : 0.0;
      s_w[upos * 4 + 3] = 0.0;
      s_col[urow] = ut_s;
      s_col[BROWS + urow] = uf_s;
      s_col[2 * BROWS + urow] = xs_s;
    }
    __syncthreads();
    // a column per wavefront (or in turn), 64 or 32 rows to a store
    const __amdgpu_buffer_rsrc_t rp = rsrc_of(u, pan_bytes);
#pragma unroll
    for (int c = wave; c < 3; c += NW) {
      const unsigned off = c == 0 ? ocu : (c == 1 ? ocf : ocn);
      buf_store_scalar<TV>(s_col[c * BROWS + (lane & (BROWS - 1))], rp,
                           off != kOOR && lane < BROWS ? off + (unsigned)(lane * sizeof(TV)) : kOOR);
    }
    load_rows(u1);
    // phase 2
    if constexpr (sizeof(TV) == 4) {
#pragma unroll
      for (int g = 0; g < QW; ++g)
#pragma unroll
        for (int e = 0; e < EPL; ++e) asm volatile("" : "+v"(t[g][e]));
    }
    double we[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) we[e] = s_w[e * 64 + lane];
#pragma unroll
    for (int g4 = 0; g4 < QW; g4 += 4) {
#pragma unroll
      for (int e = 0; e < EPL; ++e)
#pragma unroll
        for (int g = g4; g < (g4 + 4 < QW ? g4 + 4 : QW); ++g)
          acc[g] = __builtin_amdgcn_mfma_f64_4x4x4f64((double)t[g][e], we[e], acc[g], 0, 0, 0);
#pragma unroll
      for (int g = g4; g < (g4 + 4 < QW ? g4 + 4 : QW); ++g) load_group(rt, g, t[g]);
      __builtin_amdgcn_sched_barrier(0);
    }
    par ^= 1;
  };

  // number of units of this workgroup's walk
  const int np = (int)((pend_ - pstart + pstep_ - 1) / pstep_);
  const int nu = pstart < pend_ ? np * UPP : 0;
  load_rows(unit_of(0));
  {
    const __amdgpu_buffer_rsrc_t r0 = rsrc_of(unit_of(0), tile_bytes), r1 = rsrc_of(unit_of(1), tile_bytes);
#pragma unroll
    for (int g = 0; g < QW; ++g) load_group(r0, g, ta[g]);
#pragma unroll
    for (int g = 0; g < QW; ++g) load_group(r1, g, tb[g]);
  }
  int i = 0;
  for (; i + 1 < nu; i += 2) {
    step(unit_of(i), unit_of(i + 1), unit_of(i + 2), ta);
    step(unit_of(i + 1), unit_of(i + 2), unit_of(i + 3), tb);
  }
  if (i < nu) step(unit_of(i), unit_of(i + 1), unit_of(i + 2), ta);

  // accumulators: lane = rhs + 4 * block + 16 * column
#pragma unroll
  for (int g = 0; g < QW; ++g) {
    const int c = wave * 4 + g * GSTRIDE + (lane >> 4);
    double v = acc[g] + dpp_mov<0x128>(acc[g]);
    v += dpp_mov<0x124>(v);
    if ((lane & 12) == 0 && c < q && cl < (GRAM ? 3 : 2))
      (cl == 0 ? a.part0 : (cl == 1 ? a.part1 : a.part2))[(size_t)c * a.ldg + slot] = v;
  }
#pragma unroll
  for (int k = 0; k < LS_NSC; ++k) {
    if (SCL && uact) sc[k] = s_acc[k * BROWS + urow];
    const double v = lanes_sum<64>(sc[k]);
    if (lane == 0) s_sc[wave][k] = v;
  }
  __syncthreads();
  if (tid < LS_NSC) {
    double v = 0.0;
    for (int w2 = 0; w2 < NW; ++w2) v += s_sc[w2][tid];
    a.part1[(size_t)(a.n_max + tid) * a.ldg + slot] = v;
  }
}

// ---------------------------------------------------------------------------
// Sweep of an FP64 basis for the sizes that ls_rows names (k_ls_rows) and in the
// batched form (panels pstart, + pstep, ... < pend as in ls_pass_body): the row
// passes' tile (8 wavefronts, a 16-byte load of 32 lanes covers a column's 64 rows,
// QW groups of two columns per wavefront), vector FMAs in both phases, the next
// panel's tile one panel ahead.  An FP64 basis has two right-hand sides in phase 2,
// for which the four of the matrix form bring nothing, and here a wavefront reads
// 1 KiB in one piece where the matrix tile takes 256 bytes of four columns.  Bound:
// HBM; 2^22 rows, capacity 250: 113-128 columns 702 us per push (matrix form 735),
// 225-249 1291 us (1386).
// ---------------------------------------------------------------------------
template <int QW>
constexpr int ls_rows_lds_doubles() {
  return 2 * QW * 16 + 4 * 8 * PANEL + 2 * PANEL + 8 * LS_NSC;
}

template <typename TX, int QW>
__device__ __forceinline__ void ls_rows_body(const LsArgs &a, int64_t pstart, int64_t pend, int64_t pstep, int slot,
                                             double *lds) {
#pragma clang fp contract(off)
  constexpr int NW = 8, EPL = 2, LPC = 32, CPW = 2;
  constexpr int JCAP = QW * NW * CPW;
  constexpr int RPW = PANEL / NW;
  constexpr int GSTRIDE = NW * CPW;
  double (*s_coef)[JCAP] = reinterpret_cast<double (*)[JCAP]>(lds);
  double (*s_red)[2][NW][PANEL] = reinterpret_cast<double (*)[2][NW][PANEL]>(lds + 2 * JCAP);
  double *s_u = lds + 2 * JCAP + 4 * NW * PANEL;
  double *s_x = s_u + PANEL;
  double (*s_sc)[LS_NSC] = reinterpret_cast<double (*)[LS_NSC]>(s_x + PANEL);

  const DevState *st = a.st;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cs = lane / LPC;
  const int rg = lane % LPC;

  // step state (uniform), as in ls_pass_body
  const int q = uniform(st->q);
  const int hu = uniform(st->ls_u);
  const int hf = uniform(st->ls_x);
  const int hn = a.flush ? 0 : 1;
  const int cc = q, cf = q + hu, cn = cf + hf;
  const double cq = hu && hf ? uniform(st->ls_cq) : 0.0;

  __syncthreads();  // the previous call of this workgroup may still read LDS
  for (int c = tid; c < JCAP; c += NW * 64) {
    s_coef[0][c] = c < q ? a.coefW[c] : 0.0;
    s_coef[1][c] = c < q ? a.coefZ[c] : 0.0;
  }
  __syncthreads();

  const int cbase = wave * CPW + cs;
  const unsigned goff0 = (unsigned)((wave * CPW * PANEL + lane * EPL) * 8);
  constexpr unsigned GBYTES = (unsigned)(GSTRIDE * PANEL * 8);
  const unsigned tile_bytes = (unsigned)(q * PANEL * 8);
  const bool uact = lane < RPW;
  const int urow = wave * RPW + (lane % RPW);
  const unsigned pan_bytes = (unsigned)((size_t)a.n_max * PANEL * 8);
  // per-row offsets of the pending columns inside a panel (kOOR: absent)
  const unsigned ocu = uact && hu ? (unsigned)((cc * PANEL + urow) * 8) : kOOR;
  const unsigned ocf = uact && hf ? (unsigned)((cf * PANEL + urow) * 8) : kOOR;
  const unsigned ocn = uact && hn ? (unsigned)((cn * PANEL + urow) * 8) : kOOR;

  double acc0[QW], acc1[QW], sc[LS_NSC];
#pragma unroll
  for (int g = 0; g < QW; ++g) acc0[g] = acc1[g] = 0.0;
#pragma unroll
  for (int k = 0; k < LS_NSC; ++k) sc[k] = 0.0;

  char *Wb = static_cast<char *>(a.W);
  const size_t pbytes = (size_t)a.n_max * PANEL * 8;
  double t[QW][EPL], tn[QW][EPL];
  auto load_tile = [&](int64_t p, double (&dst)[QW][EPL], unsigned bytes) {
    const __amdgpu_buffer_rsrc_t rt = make_rsrc(Wb + (size_t)p * pbytes, bytes);
#pragma unroll
    for (int g = 0; g < QW; ++g)
      unpack16<double>(__builtin_amdgcn_raw_buffer_load_b128(rt, (int)goff0, (int)(g * GBYTES), kTileLoad), dst[g]);
  };
  auto hold = [&](double (&v)[QW][EPL]) {
#pragma unroll
    for (int g = 0; g < QW; ++g)
#pragma unroll
      for (int e = 0; e < EPL; ++e) asm volatile("" : "+v"(v[g][e]));
  };

  int64_t p = pstart;
  if (p < pend) {
    load_tile(p, t, tile_bytes);
    hold(t);
  }
  int par = 0;
  for (; p < pend; p += pstep) {
    // per-row inputs, ahead of the next tile's loads
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(Wb + (size_t)p * pbytes, pan_bytes);
    const double yu = buf_load_scalar<double>(rp, ocu);
    const double yf = buf_load_scalar<double>(rp, ocf);
    const int64_t rem = a.n - p * PANEL;
    const unsigned xb = hn ? (unsigned)((rem >= PANEL ? PANEL : (rem > 0 ? rem : 0)) * sizeof(TX)) : 0u;
    const double xv =
        buf_load_scalar<TX>(make_rsrc(static_cast<const TX *>(a.x) + (hn ? p * PANEL : 0), xb),
                            uact ? (unsigned)(urow * sizeof(TX)) : kOOR);
    const bool more = p + pstep < pend;
    load_tile(more ? p + pstep : p, tn, more ? tile_bytes : 0u);

    // phase 1: row sums of the tile against sigma o w and sigma o z
    double u[2][EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) u[0][e] = u[1][e] = 0.0;
#pragma unroll
    for (int g = 0; g < QW; ++g)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const double cf_ = s_coef[k][cbase + g * GSTRIDE];
#pragma unroll
        for (int e = 0; e < EPL; ++e) u[k][e] = fma(t[g][e], cf_, u[k][e]);
      }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        u[k][e] = xor_sum<32>(u[k][e]);
      }
    // stores of their own: beside the sums they cost the 16-group tile 144 bytes of
    // scratch a lane
    if (cs == 0) {
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int e = 0; e < EPL; ++e) s_red[par][k][wave][rg * EPL + e] = u[k][e];
    }
    __syncthreads();
    double sw = 0.0, sz = 0.0;
#pragma unroll
    for (int w2 = 0; w2 < NW; ++w2) {
      sw += s_red[par][0][w2][urow];
      sz += s_red[par][1][w2][urow];
    }
    // row update: finished column, formed column, snapshot copy
    const double ut = yu - sw;
    const double uf = (yf - sz) - ut * cq;
    buf_store_scalar<double>(ut, rp, ocu);
    buf_store_scalar<double>(uf, rp, ocf);
    buf_store_scalar<double>(xv, rp, ocn);
    if (uact) {
      sc[LS_UU] = fma(ut, ut, sc[LS_UU]);
      sc[LS_UF] = fma(ut, uf, sc[LS_UF]);
      sc[LS_UX] = fma(ut, xv, sc[LS_UX]);
      sc[LS_FF] = fma(uf, uf, sc[LS_FF]);
      sc[LS_FX] = fma(uf, xv, sc[LS_FX]);
      sc[LS_XX] = fma(xv, xv, sc[LS_XX]);
      s_u[urow] = uf;
      s_x[urow] = xv;
    }
    __syncthreads();
    // phase 2: column sums of the tile against the formed column and the snapshot
    double wu[EPL], wx[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      wu[e] = s_u[rg * EPL + e];
      wx[e] = s_x[rg * EPL + e];
    }
#pragma unroll
    for (int g = 0; g < QW; ++g)
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        acc0[g] = fma(t[g][e], wu[e], acc0[g]);
        acc1[g] = fma(t[g][e], wx[e], acc1[g]);
      }
    hold(tn);
#pragma unroll
    for (int g = 0; g < QW; ++g)
#pragma unroll
      for (int e = 0; e < EPL; ++e) t[g][e] = tn[g][e];
    par ^= 1;
  }

#pragma unroll
  for (int g = 0; g < QW; ++g) {
    const double v0 = lanes_sum<LPC>(acc0[g]), v1 = lanes_sum<LPC>(acc1[g]);
    const int c = cbase + g * GSTRIDE;
    if (rg == 0 && c < q) {
      a.part0[(size_t)c * a.ldg + slot] = v0;
      a.part1[(size_t)c * a.ldg + slot] = v1;
    }
  }
#pragma unroll
  for (int k = 0; k < LS_NSC; ++k) {
    const double v = lanes_sum<64>(sc[k]);
    if (lane == 0) s_sc[wave][k] = v;
  }
  __syncthreads();
  if (tid < LS_NSC) {
    double v = 0.0;
    for (int w2 = 0; w2 < NW; ++w2) v += s_sc[w2][tid];
    a.part1[(size_t)(a.n_max + tid) * a.ldg + slot] = v;
  }
}

// Sweeps run while the stream is active; flush sweeps also after a
// non-finite snapshot stopped it (the snapshots before it are completed).
__device__ __forceinline__ bool ls_runs(const DevState *st, int flush) {
  const int s = st->status;
  return s == ST_ACTIVE || (flush && s == ST_NONFINITE);
}

// Register budget as waves per SIMD: two tiles and the accumulators, no spills
template <typename TV, int NW, int QW>
constexpr int ls_waves() {
  return NW == 16 || QW <= 4 ? 4 : (QW <= 8 ? 3 : 2);
}

template <typename TV, typename TX, int NW, int QW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(ls_waves<TV, NW, QW>()))) void k_ls_pass(
    LsArgs a) {
  if (!ls_runs(a.st, a.flush)) return;
  if (a.flush && !a.st->ls_u && !a.st->ls_x) return;
  __shared__ double lds[ls_lds_doubles<TV, NW, QW>()];
  ls_pass_body<TV, TX, NW, QW>(a, blockIdx.x, a.P, gridDim.x, blockIdx.x, lds);
}

template <typename TX, int QW>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(QW <= 4 ? 4 : 2))) void k_ls_rows(LsArgs a) {
  if (!ls_runs(a.st, a.flush)) return;
  if (a.flush && !a.st->ls_u && !a.st->ls_x) return;
  __shared__ double lds[ls_rows_lds_doubles<QW>()];
  ls_rows_body<TX, QW>(a, blockIdx.x, a.P, gridDim.x, blockIdx.x, lds);
}

// ---------------------------------------------------------------------------
// Reduction: one wavefront per value (part0 columns, part1 columns, scalars),
// lane-strided sums over the slots, then a butterfly: a fixed association.
// ---------------------------------------------------------------------------
// Where value v's partial sums lie (null: nothing to sum), and its place in red.
__device__ __forceinline__ const double *ls_reduce_src(const LsSmall &a, int v, int q, int *out) {
  if (v < a.nt) {
    *out = v;
    return v < q ? a.part0 + (size_t)v * a.ldg : nullptr;
  }
  if (v < 2 * a.nt) {
    *out = a.n_max + (v - a.nt);
    return v - a.nt < q ? a.part1 + (size_t)(v - a.nt) * a.ldg : nullptr;
  }
  const int sc = v - 2 * a.nt;
  *out = 2 * a.n_max + sc;
  if (sc < LS_NSC) return a.part1 + (size_t)(a.n_max + sc) * a.ldg;
  const int c = sc - LS_NSC;
  return a.gram && c < q && a.st->ls_u ? a.part2 + (size_t)c * a.ldg : nullptr;
}

// one wavefront per value; vblock selects four consecutive values
__device__ inline void ls_reduce_body(const LsSmall &a, int vblock) {
  const int lane = threadIdx.x & 63;
  int out;
  const double *src = ls_reduce_src(a, vblock * 4 + (threadIdx.x >> 6), a.st->q, &out);
  if (!src) return;
  const double t = strided_sum<false>(src, a.G, lane);
  if (lane == 0) a.red[out] = t;
}

__global__ __launch_bounds__(256) void k_ls_reduce(LsSmall a) {
  if (!ls_runs(a.st, a.flush)) return;
  if (a.flush && !a.st->ls_u && !a.st->ls_x) return;
  ls_reduce_body(a, blockIdx.x);
}

// ---------------------------------------------------------------------------
// Finalize (one workgroup of 512 threads, q <= 511 after the push).
// ---------------------------------------------------------------------------
// Sums of v[0 .. N) over the workgroup (wavefront sums, then over the wavefronts
// in order), in every thread; sh: N * NT / 64 doubles.
template <int NT, int N>
__device__ inline void ls_block_sums(double (&v)[N], double *sh) {
#pragma unroll
  for (int n = 0; n < N; ++n) {
    v[n] = lanes_sum<64>(v[n]);
    if ((threadIdx.x & 63) == 0) sh[n * (NT / 64) + (threadIdx.x >> 6)] = v[n];
  }
  __syncthreads();
#pragma unroll
  for (int n = 0; n < N; ++n) {
    v[n] = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) v[n] += sh[n * (NT / 64) + w];
  }
  __syncthreads();
}

// Two products for the coming finalize, both 64 rows x a contiguous l-slice per
// wavefront (NT / 64 of them) of slice `part` of `parts` of the l range, slices
// summed in order, one value per row to out[i] (i < c):
//  * KIND 0: the part of H_bar's column c-1 that the earlier columns give, for the
//    column c = q that the finalize finishes (eq. betacolumnupdate),
//    sum_{l = max(0, i-1)}^{c-2} H_bar[i, l] beta[l, c-1];
//  * KIND 1 (FP32 basis): E w over the earlier final columns for the column that
//    the finalize makes pending (w_l = sigma_l * its reduced sum l, l < q), E
//    symmetric with a zero diagonal; the terms of the column finished in the same
//    sweep are added by the finalize.
template <int KIND, int NT>
__device__ inline void ls_product_body(const LsSmall &a, int rblock, int part, int parts, double *out) {
  constexpr int NS = NT / 64;
  __shared__ double sh[NS][64];
  const int c = a.st->q;
  const int r = threadIdx.x & 63, sl = part * NS + (threadIdx.x >> 6), S = NS * parts;
  const int i = rblock * 64 + r;
  double t = 0.0;
  if (i < c) {
    const int lo = KIND == 0 && i > 0 ? i - 1 : 0, hi = KIND == 0 ? c - 1 : c, len = hi > lo ? hi - lo : 0;
    const int a0 = lo + (len * sl) / S, a1 = lo + (len * (sl + 1)) / S;
    const double *m = (KIND == 0 ? a.H : a.E) + i;
    const size_t ld = KIND == 0 ? (size_t)a.ldH : (size_t)a.n_max;
    const double *bprev = a.beta + (size_t)(c > 0 ? c - 1 : 0) * a.ldB;
    auto x = [&](int l) { return KIND == 0 ? bprev[l] : a.red[l] * a.sigma[l]; };
    // four independent chains, so the loads of several columns are in flight
    double t4[4] = {0.0, 0.0, 0.0, 0.0};
    int l = a0;
    for (; l + 4 <= a1; l += 4) {
#pragma unroll
      for (int k = 0; k < 4; ++k) t4[k] = fma(m[(size_t)(l + k) * ld], x(l + k), t4[k]);
    }
    for (; l < a1; ++l) t4[0] = fma(m[(size_t)l * ld], x(l), t4[0]);
    t = (t4[0] + t4[1]) + (t4[2] + t4[3]);
  }
  sh[threadIdx.x >> 6][r] = t;
  __syncthreads();
  if (threadIdx.x < 64 && i < c) {
    double o = sh[0][r];
#pragma unroll
    for (int k = 1; k < NS; ++k) o += sh[k][r];
    out[i] = o;
  }
}

// One stream: the l range of either product is cut into a.hs workgroups as well
// (grid: row chunks x slices x the two products) and the finalize adds the slices:
// a workgroup per 64 rows read H_bar and E through 8 CUs, 15.2 us at 250 columns.
__global__ __launch_bounds__(256) void k_ls_hprod(LsSmall a) {
  if (!ls_runs(a.st, a.flush)) return;
  double *out = a.hp + (size_t)(blockIdx.z * a.hs + blockIdx.y) * (a.n_max + 1);
  if (blockIdx.z == 0) {
    if (a.st->ls_u) ls_product_body<0, 256>(a, blockIdx.x, blockIdx.y, a.hs, out);
  } else if (a.st->ls_x) {
    ls_product_body<1, 256>(a, blockIdx.x, blockIdx.y, a.hs, out);
  }
}

// Row i of a product as the finalize reads it: the slices' sum, or (batched form)
// the whole product in p.
__device__ __forceinline__ double ls_product(const LsSmall &a, int kind, const double *p, int i) {
  if (!a.hp) return p[i];
  double v[8], t = 0.0;
#pragma unroll
  for (int s = 0; s < 8; ++s) v[s] = s < a.hs ? a.hp[(size_t)(kind * a.hs + s) * (a.n_max + 1) + i] : 0.0;
#pragma unroll
  for (int s = 0; s < 8; ++s) t += v[s];
  return t;
}

// H_bar's column c-1 once beta's column c is final: h = (beta_{0:c,c} -
// [b; 0]) / beta_{c-1,c-1} with b from k_ls_hprod.
template <int NT>
__device__ inline void ls_hbar_column(const LsSmall &a, int c) {
  const double *bcol = a.beta + (size_t)c * a.ldB;
  const double d = a.beta[(size_t)(c - 1) * a.ldB + (c - 1)];
  for (int i = threadIdx.x; i <= c; i += NT)
    a.H[(size_t)(c - 1) * a.ldH + i] = (bcol[i] - (i < c ? ls_product(a, 0, a.bvec, i) : 0.0)) / d;
}

template <int NT>
__device__ inline void ls_finalize_body(const LsSmall &a) {
  __shared__ double sh[2 * NT / 64];
  __shared__ int s_flag;
  DevState *st = a.st;
  const int tid = threadIdx.x;
  const bool push = !a.flush;
  if (!ls_runs(st, a.flush) || (a.flush && !st->ls_u && !st->ls_x)) {
    __syncthreads();
    if (tid == 0 && push) st->pushes += 1;
    return;
  }
  const int q0 = st->q;
  const int hu = st->ls_u, hf = st->ls_x;
  int hn = push ? 1 : 0;
  const double *red0 = a.red, *red1 = a.red + a.n_max, *sc = a.red + 2 * a.n_max;
  const double rhohat0 = st->ls_rhohat, rt0 = st->ls_rt;
  // the new snapshot: non-finite -> dropped, the stream stops; zero first -> q = 0
  if (hn) {
    const double xn2 = sc[LS_XX];
    if (!isfinite(xn2)) {
      hn = 0;
      __syncthreads();
      if (tid == 0) st->status = ST_NONFINITE;
    } else if (q0 == 0 && !hu && !hf && xn2 == 0.0) {
      __syncthreads();
      if (tid == 0) {
        st->status = ST_ZERO;
        st->pushes += 1;
      }
      return;
    }
  }
  // 1. the pending column is finished: exact norm, breakdown test, H_bar
  int q = q0;
  double rho = 0.0;
  if (hu) {
    rho = sqrt(sc[LS_UU]);
    const double xf = a.xpre[q0];
    if (tid == 0) s_flag = !(rho > st->tol * sqrt(xf)) ? (isfinite(rho) ? 1 : 2) : 0;
    __syncthreads();
    const int flag = s_flag;
    if (flag) {
      // dependent (or non-finite) column: the stream keeps the q0 columns before it
      if (flag == 1) {
        if (tid == 0) a.beta[(size_t)q0 * a.ldB + q0] = 0.0;
        __syncthreads();
        if (q0 > 0) ls_hbar_column<NT>(a, q0);
      }
      __syncthreads();
      if (tid == 0) {
        st->status = flag == 1 ? ST_INVARIANT : ST_NONFINITE;
        st->ls_u = 0;
        st->ls_x = 0;
        if (push) st->pushes += 1;
      }
      return;
    }
    if (tid == 0) {
      a.beta[(size_t)q0 * a.ldB + q0] = rho;
      a.sigma[q0] = 1.0 / rho;
    }
    if (a.gram) {
      // E's new column: q_i^T q_q0 = sigma_i (stored_i^T delta) / rho, delta the
      // rounding error of the stored column (the rest is O(||E||^2))
      const double *red2 = a.red + 2 * a.n_max + LS_NSC;
      for (int i = tid; i < q0; i += NT) {
        const double g = a.sigma[i] * red2[i] / rho;
        a.E[(size_t)q0 * a.n_max + i] = g;
        a.E[(size_t)i * a.n_max + q0] = g;
      }
      if (tid == 0) a.E[(size_t)q0 * a.n_max + q0] = 0.0;
    }
    __syncthreads();
    if (q0 > 0) ls_hbar_column<NT>(a, q0);
    q = q0 + 1;
  }
  __syncthreads();
  // 2. the snapshot copy became the pending column: its beta column is the
  // first projection plus the second (w), both on the final columns
  double alpha = 0.0, wn2 = 0.0;
  if (hf) {
    const int c = q;  // 0-based index of the new pending column
    const double sk = hu ? a.sigma[q0] : 0.0;
    // FP32 basis: E w.  The product over the earlier final columns is there; the
    // finished column q0 adds w_q0 E[i, q0] to rows i < q0 and the whole row q0,
    // sum_l E[q0, l] w_l.
    double eq0 = 0.0;
    if (a.gram && hu) {
      double t = 0.0;
      for (int l = tid; l < q0; l += NT) t = fma(a.E[(size_t)q0 * a.n_max + l], red0[l] * a.sigma[l], t);
      double v1[1] = {t};
      ls_block_sums<NT>(v1, sh);
      eq0 = v1[0];
    }
    for (int i = tid; i < c; i += NT) {
      double wi, pi, ewi = 0.0;
      if (i < q0) {
        wi = red0[i] * a.sigma[i];
        pi = a.z[i];
        if (a.gram) ewi = ls_product(a, 1, a.what, i) + (hu ? a.E[(size_t)q0 * a.n_max + i] * (sc[LS_UF] * sk) : 0.0);
      } else {  // i == q0: the column finished in this sweep
        wi = sc[LS_UF] * sk;
        pi = rhohat0 > 0.0 ? (rho / rhohat0) * rt0 : 0.0;
        ewi = eq0;
      }
      const double wh = wi - ewi;  // the second-projection coefficient used
      a.beta[(size_t)c * a.ldB + i] = pi + wh;
      a.w[i] = wi;
      a.what[i] = wh;
      a.coefW[i] = a.sigma[i] * wh;
    }
    alpha = sc[LS_FF];
  }
  __syncthreads();
  // 3. the new snapshot: first-projection coefficients on the final columns
  if (hn) {
    const double sk = hu ? a.sigma[q0] : 0.0;
    for (int i = tid; i < q; i += NT) {
      const double zi = i < q0 ? red1[i] * a.sigma[i] : sc[LS_UX] * sk;
      a.z[i] = zi;
      a.coefZ[i] = a.sigma[i] * zi;
    }
  }
  __syncthreads();
  // 4. scalars of the next sweep
  const int nu = hf ? 1 : 0;
  const int nx = hn ? 1 : 0;
  double wz = 0.0;
  if (nu) {
    // ||u - Q w_hat||^2 = ||u||^2 - w^T w_hat and the R_tilde identity with
    // w_hat (w_hat = w with an FP64 basis)
    double t = 0.0, t2 = 0.0;
    for (int i = tid; i < q; i += NT) {
      t = fma(a.w[i], a.what[i], t);
      if (nx) t2 = fma(a.what[i], a.z[i], t2);
    }
    double v2[2] = {t, t2};
    ls_block_sums<NT>(v2, sh);
    wn2 = v2[0];
    wz = v2[1];
  }
  if (tid == 0) {
    st->q = q;
    st->ls_u = nu;
    st->ls_x = nx;
    if (nu) st->ls_alpha = alpha;
    if (nx) {
      const double xn2 = sc[LS_XX];
      const int k = st->ls_nx;
      a.xpre[k] = (k > 0 ? a.xpre[k - 1] : 0.0) + xn2;
      st->ls_nx = k + 1;
      st->xfro2 += xn2;
      st->ls_gamma = nu ? sc[LS_FX] : 0.0;
    }
    double rh = 0.0, rt = 0.0, cq = 0.0;
    if (nu) {
      const double d = alpha - wn2;
      rh = d > 0.0 ? sqrt(d) : 0.0;
      if (nx && rh > 0.0) {
        rt = (st->ls_gamma - wz) / rh;
        cq = rt / rh;
      }
    }
    st->ls_rhohat = rh;
    st->ls_rt = rt;
    st->ls_cq = cq;
    if (push) st->pushes += 1;
  }
}

__global__ __launch_bounds__(512) void k_ls_finalize(LsSmall a) { ls_finalize_body<512>(a); }

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Tile shapes: the narrowest tile of 4 wavefronts that covers the final columns
// (up to 16 groups, 256 columns), 8 wavefronts beyond; option ls_nw = 16: sixteen
// for 129-256 columns of an FP32 basis.
//
// An FP64 basis takes k_ls_rows (8 wavefronts) where that is the faster one: at
// 33-64 columns, at 97-128 from 65536 rows on, and beyond 128 from 524288 rows on.
// Pushes of a stream, time of k_ls_pass over that of k_ls_rows: 33-64 columns 1.01
// - 1.16 at 3000 .. 2^22 rows; 65-96 0.91 - 1.02; 97-128 0.93 at 20000 rows, 0.99 at
// 50000, 1.02 at 100037, 1.08 at 2^21; 129-160 0.95 at 300007, 1.03 at 2^20;
// 225-256 0.98 at 100037, 1.09 at 300007, 1.12 at 2^21.
static bool ls_rows(bool tv_f64, int q, int64_t P) {
  return tv_f64 && (q > 128 ? P >= 8192 : (q > 96 ? P >= 1024 : q > 32 && q <= 64));
}

int ls_nw(bool tv_f64, int q, int nw_opt, int64_t P) {
  if (ls_rows(tv_f64, q, P)) return 8;
  if (!tv_f64 && nw_opt == 16 && q > 128 && q <= 256) return 16;
  return q <= 256 ? 4 : 8;
}

int ls_qw(bool tv_f64, int q, int nw_opt, int64_t P) {
  static const int qs[] = {1, 2, 4, 6, 8, 10, 12, 14, 15, 16};
  if (ls_rows(tv_f64, q, P)) return q <= 64 ? 4 : (q <= 128 ? 8 : 16);
  const int nw = ls_nw(tv_f64, q, nw_opt, P);
  if (nw == 16) return 4;
  for (int w : qs)
    if (nw * w * 4 >= q && (nw == 4 ? w != 15 : w >= 10)) return w;
  return 16;
}

bool ls_supported(bool tv_f64, int q) { return tv_f64 ? q <= 256 : q <= 512; }

template <typename TV, typename TX>
static const void *ls_fn(int nw, int qw) {
#define FOA_LS(NW, QW) \
  case NW * 100 + QW: return reinterpret_cast<const void *>(&k_ls_pass<TV, TX, NW, QW>);
  switch (nw * 100 + qw) {
    FOA_LS(4, 1)
    FOA_LS(4, 2)
    FOA_LS(4, 6)
    FOA_LS(4, 8)
    FOA_LS(4, 10)
    FOA_LS(4, 12)
    FOA_LS(4, 14)
    FOA_LS(4, 16)
    case 1604:
      if constexpr (sizeof(TV) == 4) return reinterpret_cast<const void *>(&k_ls_pass<TV, TX, 16, 4>);
      return nullptr;
  }
  if constexpr (sizeof(TV) == 4) {  // an FP64 basis holds at most 256 final columns (33-64: k_ls_rows)
    switch (nw * 100 + qw) {
      FOA_LS(4, 4)
      FOA_LS(8, 10)
      FOA_LS(8, 12)
      FOA_LS(8, 14)
      FOA_LS(8, 15)
      FOA_LS(8, 16)
    }
  }
#undef FOA_LS
  return nullptr;
}

template <typename TX>
static const void *ls_rows_fn(int qw) {  // covers 16 qw columns
  if (qw == 4) return reinterpret_cast<const void *>(&k_ls_rows<TX, 4>);
  return qw == 8 ? reinterpret_cast<const void *>(&k_ls_rows<TX, 8>) : reinterpret_cast<const void *>(&k_ls_rows<TX, 16>);
}

static const void *ls_kernel(bool tv_f64, bool tx_f64, int q, int nw_opt, int64_t P) {
  const int nw = ls_nw(tv_f64, q, nw_opt, P), qw = ls_qw(tv_f64, q, nw_opt, P);
  if (ls_rows(tv_f64, q, P)) return tx_f64 ? ls_rows_fn<double>(qw) : ls_rows_fn<float>(qw);
  if (qw * nw * 4 < q) return nullptr;  // tile narrower than the basis
  if (tv_f64) return tx_f64 ? ls_fn<double, double>(nw, qw) : ls_fn<double, float>(nw, qw);
  return tx_f64 ? ls_fn<float, double>(nw, qw) : ls_fn<float, float>(nw, qw);
}

hipError_t launch_ls_pass(bool tv_f64, bool tx_f64, int q, int nw_opt, int grid, const LsArgs &a, hipStream_t s) {
  if (!ls_supported(tv_f64, q)) return hipErrorInvalidValue;
  const void *f = ls_kernel(tv_f64, tx_f64, q, nw_opt, a.P);
  if (!f) return hipErrorInvalidValue;
  void *args[] = {const_cast<LsArgs *>(&a)};
  return hipLaunchKernel(f, dim3(grid), dim3(64 * ls_nw(tv_f64, q, nw_opt, a.P)), args, 0, s);
}

int ls_occupancy(bool tv_f64, bool tx_f64, int q, int nw_opt, int64_t P) {
  int nb = 0;
  const void *f = ls_kernel(tv_f64, tx_f64, q, nw_opt, P);
  if (!f || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, 64 * ls_nw(tv_f64, q, nw_opt, P), 0) != hipSuccess)
    return 1;
  return nb > 0 ? nb : 1;
}

hipError_t launch_ls_reduce(const LsSmall &a, hipStream_t s) {
  const int waves = (a.gram ? 3 : 2) * a.nt + LS_NSC;
  hipLaunchKernelGGL(k_ls_reduce, dim3((waves + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_ls_finalize(const LsSmall &a, hipStream_t s) {
  // the H_bar product for the column the finalize finishes (1 <= q <= nt;
  // for q = 1 it writes the empty product 0)
  if (a.nt >= 1) {
    hipLaunchKernelGGL(k_ls_hprod, dim3((a.nt + 63) / 64, a.hs, a.gram ? 2 : 1), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_ls_finalize, dim3(1), dim3(512), 0, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Batched one-reduction form.  The per-step plan of the three-sweep batched
// form (k_batch_plan with ls_mode) buckets the streams by final columns q
// and cuts each bucket's panels into workgroup ranges; here each bucket runs
// one sweep over its ranges, then every active stream its reduction, H_bar
// product and finalize.
// ---------------------------------------------------------------------------
__device__ __forceinline__ LsSmall ls_small_of(const BatchStream &d, int flush) {
  LsSmall a{};
  a.st = d.st;
  a.H = d.H;
  a.beta = d.beta;
  a.sigma = d.sigma;
  a.w = d.h;
  a.z = d.s;
  a.coefW = d.coefA;
  a.coefZ = d.coefB;
  a.red = d.red;
  a.bvec = d.bvec;
  a.xpre = d.xpre;
  a.part0 = d.part;
  a.part1 = d.part1;
  a.part2 = d.part2;
  a.E = d.E;
  a.what = d.what;
  a.gram = d.E != nullptr ? 1 : 0;
  a.ldH = d.ldH;
  a.ldB = d.ldB;
  a.n_max = d.n_max;
  a.ldg = d.ldg;
  a.G = d.st->nseg;
  a.nt = d.st->jstep;
  a.flush = flush;
  return a;
}

// ROWS: the sweep is ls_rows_body's (FP64 basis, NW = 8)
template <typename TV, typename TX, int NW, int QW, int BK, bool ROWS>
__global__ __launch_bounds__(NW * 64)
    __attribute__((amdgpu_waves_per_eu(ROWS ? (QW <= 4 ? 4 : 2) : ls_waves<TV, NW, QW>()))) void k_ls_pass_batch(BatchArgs b) {
  __shared__ double lds[ROWS ? ls_rows_lds_doubles<QW>() : ls_lds_doubles<TV, NW, QW>()];
  const int G = uniform(b.meta[2 * BK + 1]);
  if ((int)blockIdx.x >= G) return;
  const int cnt = uniform(b.meta[2 * BK]);
  const int64_t *pre = b.pre + (size_t)BK * (b.S + 1);
  const int *list = b.list + (size_t)BK * b.S;
  const int64_t T = pre[cnt];
  int64_t lo = uniform((int64_t)blockIdx.x * T / G);
  const int64_t hi = uniform((int64_t)(blockIdx.x + 1) * T / G);
  int i = uniform(b.first[BK * kMaxBatchGrid + blockIdx.x]);
  const int flush = b.ls_mode == 2 ? 1 : 0;
  while (lo < hi) {
    const int s = uniform(list[i]);
    const int64_t ps = uniform(pre[i]), pe = uniform(pre[i + 1]);
    const int64_t e = pe < hi ? pe : hi;
    const BatchStream &d = b.streams[s];
    const DevState *st = uniform(d.st);
    LsArgs a{};
    a.W = uniform(d.W);
    a.x = flush ? nullptr : uniform(b.xptrs[s]);
    a.coefW = uniform(d.coefA);
    a.coefZ = uniform(d.coefB);
    a.st = st;
    a.part0 = uniform(d.part);
    a.part1 = uniform(d.part1);
    a.part2 = uniform(d.part2);
    a.n = uniform(d.n);
    a.P = uniform(d.P);
    a.n_max = uniform(d.n_max);
    a.ldg = uniform(d.ldg);
    a.flush = flush;
    const int slot = (int)blockIdx.x - uniform(st->seg0);
    if constexpr (ROWS)
      ls_rows_body<TX, QW>(a, lo - ps, e - ps, 1, slot, lds);
    else
      ls_pass_body<TV, TX, NW, QW>(a, lo - ps, e - ps, 1, slot, lds);
    lo = e;
    ++i;
  }
}

// Four values a wavefront, their loads in flight together: a stream has few partial
// sums per value, and a value per wavefront made the launch 14 000 workgroups (64
// streams of 20..300 columns: 8.2 us, 5.5 us so).
__global__ __launch_bounds__(256) void k_ls_reduce_batch(BatchArgs b) {
  const BatchStream &d = b.streams[blockIdx.y];
  if (!d.st->act) return;
  const LsSmall a = ls_small_of(d, b.ls_mode == 2);
  const int v0 = blockIdx.x * 16 + 4 * __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (v0 >= (a.gram ? 3 : 2) * a.nt + LS_NSC) return;
  const int lane = threadIdx.x & 63, q = a.st->q;
  const double *p[4];
  int out[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) p[k] = ls_reduce_src(a, v0 + k, q, &out[k]);
  double t[4];
  strided_sum4(p, a.G, lane, t);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (lane == k && p[k]) a.red[out[k]] = t[k];
}

// A workgroup of 16 l-slices per 64 rows and product (64 streams of 20..300 columns:
// 4 slices and both products in a workgroup 12.5 us, 7.8 us so).
__global__ __launch_bounds__(1024) void k_ls_hprod_batch(BatchArgs b) {
  const BatchStream &d = b.streams[blockIdx.y];
  const LsSmall a = ls_small_of(d, b.ls_mode == 2);
  if (!d.st->act || ((int)blockIdx.x * 64 >= d.st->q && blockIdx.x > 0)) return;
  if (blockIdx.z == 0) {
    if (d.st->ls_u) ls_product_body<0, 1024>(a, blockIdx.x, 0, 1, a.bvec);
  } else if (a.gram && d.st->ls_x) {
    ls_product_body<1, 1024>(a, blockIdx.x, 0, 1, a.what);
  }
}

__global__ __launch_bounds__(512) void k_ls_finalize_batch(BatchArgs b) {
  const int s = blockIdx.x;
  const BatchStream &d = b.streams[s];
  DevState *st = d.st;
  const int flush = b.ls_mode == 2 ? 1 : 0;
  if (!flush) {
    if (b.xptrs[s] == nullptr) return;  // idle this step
    if (!st->act) {                     // offered to a stream that takes no snapshot
      if (threadIdx.x == 0) st->pushes += 1;
      return;
    }
  } else if (!st->act) {
    return;
  }
  ls_finalize_body<512>(ls_small_of(d, flush));
}

// Kernel shape of bucket k (basis sizes up to 32, 64, 128, 256, 512 final
// columns; an empty basis is in bucket 1): 1, 2, 4, 8, 8 wavefronts with 8, 8, 8, 8,
// 16 groups of four columns.  An FP64 basis (at most 256 columns) from 33 columns
// on takes the row form, 8 wavefronts with 4, 8, 16 groups of two: 64 streams of
// 2^12..2^18 rows and 20..250 columns 93.3 ms, from bucket 3 or 4 on 93.7 and 95.1,
// the matrix form throughout 102.1; 24 streams of 1000..20000 rows 13.8 ms (14.5).
bool ls_batch_supported(bool tv_f64, int k) { return k >= 1 && (!tv_f64 || k <= 4); }

template <typename TV, typename TX, int BK>
static const void *ls_batch_fn(int *nt) {
  constexpr bool ROWS = sizeof(TV) == 8 && BK >= 2;
  constexpr int NW = BK <= 1 ? 1 : (ROWS ? 8 : (BK == 2 ? 2 : (BK == 3 ? 4 : 8)));
  constexpr int QW = ROWS ? 2 << (BK - 1) : (BK == 5 ? 16 : 8);
  *nt = NW * 64;
  return reinterpret_cast<const void *>(&k_ls_pass_batch<TV, TX, NW, QW, BK, ROWS>);
}

template <typename TV, typename TX>
static const void *ls_batch_fn_k(int k, int *nt) {
  switch (k) {
    case 1: return ls_batch_fn<TV, TX, 1>(nt);
    case 2: return ls_batch_fn<TV, TX, 2>(nt);
    case 3: return ls_batch_fn<TV, TX, 3>(nt);
    case 4: return ls_batch_fn<TV, TX, 4>(nt);
    default:
      if constexpr (sizeof(TV) == 4) return ls_batch_fn<TV, TX, 5>(nt);
      return nullptr;
  }
}

static const void *ls_batch_kernel(bool tv_f64, bool tx_f64, int k, int *nt) {
  if (tv_f64) return tx_f64 ? ls_batch_fn_k<double, double>(k, nt) : ls_batch_fn_k<double, float>(k, nt);
  return tx_f64 ? ls_batch_fn_k<float, double>(k, nt) : ls_batch_fn_k<float, float>(k, nt);
}

int ls_batch_occupancy(bool tv_f64, int k) {
  int nt = 0, nb = 0;
  const void *f = ls_batch_kernel(tv_f64, false, k, &nt);
  if (!f || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, nt, 0) != hipSuccess) return 1;
  return nb > 0 ? nb : 1;
}

hipError_t launch_ls_batch_pass(bool tv_f64, bool tx_f64, int k, int grid, const BatchArgs &b, hipStream_t s) {
  int nt = 0;
  const void *f = ls_batch_kernel(tv_f64, tx_f64, k, &nt);
  if (!f) return hipErrorInvalidValue;
  void *args[] = {const_cast<BatchArgs *>(&b)};
  return hipLaunchKernel(f, dim3(grid), dim3(nt), args, 0, s);
}

hipError_t launch_ls_batch_small(const BatchArgs &b, int cols, hipStream_t s) {
  const int vblocks = (3 * cols + LS_NSC + 15) / 16;
  hipLaunchKernelGGL(k_ls_reduce_batch, dim3(vblocks, b.S), dim3(256), 0, s, b);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_ls_hprod_batch, dim3(std::max((cols + 63) / 64, 1), b.S, 2), dim3(1024), 0, s, b);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_ls_finalize_batch, dim3(b.S), dim3(512), 0, s, b);
  return hipGetLastError();
}

}  // namespace foa
