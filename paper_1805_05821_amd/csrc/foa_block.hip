// Blocked form of the FOA push: BPK snapshots per step.
//
// The modified FOA builds the thin QR factorisation X = V beta together with
// H_bar, where beta_{:,c+1} = H_bar_{:,1:c} beta_{1:c,c} (eq. betacolumnupdate;
// the QR view of Section 3.1).  The blocked form reaches the same factors in
// exact arithmetic with a block Y of snapshots at a time:
//   R1 = V^T Y;  Z = Y - V R1;  R2 = V^T Z;  Z = Z - V R2     (block CGS2)
//   [R3 = V^T Z;  Z = Z - V R3]    when two projections may not be enough
//   Z = Q S by shifted CholeskyQR3 (Fukaya et al., SIAM J. Sci. Comput. 2020)
//   beta's new columns [R1 + R2 (+ R3); S], V's new columns Q, and H_bar's new
//   columns from the recurrence above solved column by column.
// So the basis is swept three times per block (twice within a run, where a block's
// last sweep forms the next one's R1) instead of three times per snapshot.  The third projection: a stored FP32 basis is orthonormal only to
// E = V^T V - I, the part of Z left along V after two passes is about E R2,
// and where the block's new directions are as small as ||E|| ||Y|| (noise-
// floor snapshots at small n) that part is as large as Z itself.  The test
// estimates ||E|| by ||R2||_F / ||R1||_F and takes the third pass when
// ||E|| ||R2_k|| > u_V ||Z_k|| / 10 for some k (u_V the basis's unit
// roundoff); its kernels are always enqueued and return at once otherwise.  A block is committed only if its Cholesky steps succeed and every
// new diagonal entry of beta is above the breakdown threshold; otherwise the
// device state is left as it was and the host takes those snapshots one at a
// time (the sequential kernels then apply the paper's breakdown rule).
//
// Kernels (all on the context stream, all no-ops once the block is rejected):
//   k_bpass   : the block row passes over V (FP64 accumulation, BPK right-hand
//               sides, column sums on FP64 MFMA);
//   k_zgram   : passes over the n x BPK block (||y||^2, the Gram matrix of Z T,
//               the final Q written into V);
//   k_breduce : fixed-order reduction of the pass partials into R1 / R2 and
//               the next pass's coefficients;
//   k_bthird  : the test for the third projection (sets the gate of its
//               BP_D pass, reduction and BP_Z2 pass);
//   k_bchol   : Gram reduction, (shifted) Cholesky and triangular inverse;
//   k_bcommit, k_bcommit_h : breakdown test, beta, sigma and the scalar state; H_bar.
#include <mutex>
#include <type_traits>

#include "foa.h"
#include "foa_device.h"

// Block workspace of foa_push_blocked_static, for callers that cannot
// allocate device memory: one copy per device the library runs on, held
// until the process ends.  Host code never uses this name as an address:
// block_static_scratch() looks the device address up once per device and
// every launch takes that address.
static __device__ __align__(256) char scratch[FOA_BLOCK_STATIC_BYTES];

namespace foa {

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char *g_scratch_addr[kMaxDevices] = {};
hipError_t g_scratch_err[kMaxDevices] = {};
bool g_scratch_done[kMaxDevices] = {};
}  // namespace

hipError_t block_static_scratch(int device, char **ptr) {
  *ptr = nullptr;
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_done[device]) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e == hipSuccess && cur != device) e = hipSetDevice(device);
    void *addr = nullptr;
    if (e == hipSuccess) e = hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch));
    if (cur >= 0 && cur != device) {
      const hipError_t e2 = hipSetDevice(cur);
      if (e == hipSuccess) e = e2;
    }
    g_scratch_addr[device] = e == hipSuccess ? static_cast<char *>(addr) : nullptr;
    g_scratch_err[device] = e;
    g_scratch_done[device] = true;
  }
  *ptr = g_scratch_addr[device];
  return g_scratch_err[device];
}

enum { BP_R1 = 0, BP_Z1 = 1, BP_Z2 = 2, BP_D = 3, BP_ZR = 4 };
enum { ZG_YNORM = 0, ZG_GRAM = 1, ZG_WRITEV = 2, ZG_YNQ = 3 };

// ---------------------------------------------------------------------------
// Block row pass over the j basis columns.  MODE BP_R1: D = W^T Y (column sums
// only).  BP_Z1: Z = Y - W C, D = W^T Z.  BP_Z2: Z = Z - W C.  BP_D: D = W^T Z
// (the third projection).  BP_ZR: Z = Z - W C and D = W^T Y' for the next
// block's snapshots Y' (a.xn) in the same sweep (the next block's first
// projection over these columns; the two phases are independent, so Y' goes to
// LDS at phase 1's barrier).  BP_Z2 and BP_ZR also leave the partial Gram matrix
// of the Z they form in partg (a.G slots).  W is the stored basis (the sigma
// scaling of its columns is folded into C and into the reduction of D).
//
// Unit of work: BROWS rows of a panel, 16 chunks of one 16-byte load each (64
// rows with an FP32 basis, 32 with an FP64 one), walked by persistent
// workgroups.  Lane l of a wavefront holds chunk l / 4 of column l % 4 of each
// of its QW groups of four columns (wavefront w: groups w, w + NW, ...).
//   phase 1 (row sums against BPK coefficient vectors): FMA per lane over its
//     groups; then over the four lanes of a quad by DPP moves, each lane keeping
//     one right-hand side; then over the wavefronts through LDS;
//   update: (row, right-hand side) pairs, pos = e * 64 + chunk * 4 + k for row
//     chunk * EPL + e, spread over the wavefronts; Z is kept in that order;
//   phase 2 (column sums): the lanes hold a tile as the A operand of
//     v_mfma_f64_4x4x4 (four blocks: columns x rows), the pairs of row e as its
//     B operand, so a group's sums against the four right-hand sides take one
//     accumulator per lane.  The FP64 matrix and vector rates are the same here
//     (18.7 cycles per 256 FMAs, both on one pipe); what the matrix form buys is
//     registers: 4 x QW FP64 accumulators per lane became QW, so tiles of every
//     width are prefetched whole and an FP64 basis needs no column windows.
// Bound: HBM.  2^22 rows, FP32 basis of 449-496 columns: BP_Z1 1382 us and BP_ZR
// 1470 us (5.8 and 5.4 TB/s of basis reads beside the write stream of Z), 1925
// and 1980 us with vector FMAs for phase 2 and no room to prefetch; with the
// next tile loaded whole but one iteration ahead 1520 and 1680 us, and with each
// unit's y loaded at its own start (or through a divergent resource) 1540 us.
// FP64 basis, 300007 rows x 257-320 columns: 128 and 144 us, in two column
// windows 330 us.
// ---------------------------------------------------------------------------
template <typename TV, typename TX, int NW, int QW, int MODE>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(QW >= 10 ? 2 : 1))) void k_bpass(BlockArgs a) {
  constexpr int EPL = Vec<TV>::EPL;
  constexpr int BROWS = 16 * EPL;
  constexpr int UPP = PANEL / BROWS;    // units per panel
  constexpr int PAIRS = BROWS * BPK;
  constexpr int UL = PAIRS / NW;        // update lanes of a wavefront
  constexpr int JCAP = QW * NW * 4;
  constexpr int GSTRIDE = NW * 4;       // columns between a wavefront's groups
  constexpr bool NEXT_Y = MODE == BP_ZR;
  constexpr bool HAS_P1 = MODE == BP_Z1 || MODE == BP_Z2 || NEXT_Y;
  constexpr bool HAS_P2 = MODE == BP_R1 || MODE == BP_Z1 || MODE == BP_D || NEXT_Y;
  constexpr bool SRC_X = MODE == BP_R1 || MODE == BP_Z1;
  constexpr bool GRAM = MODE == BP_Z2 || NEXT_Y;
  static_assert(BPK == 4 && UL <= 64 && UL % 4 == 0, "update lanes");

  if (a.st->status != ST_ACTIVE || *a.flag || (a.gate && !*a.gate)) return;

  __shared__ double s_coef[HAS_P1 ? JCAP * BPK : 1];
  __shared__ double s_red[HAS_P1 ? 2 * NW * PAIRS : 1];
  __shared__ double s_w[2][PAIRS];
  __shared__ double s_g[GRAM ? NW * 12 : 1];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cl = lane & 3;
  const int j = a.j;
  const int slot = blockIdx.x;

  if (HAS_P1)
    for (int c = tid; c < JCAP * BPK; c += NW * 64) s_coef[c] = (c < j * BPK) ? a.coef[c] : 0.0;
  __syncthreads();

  const int cbase = wave * 4 + cl;
  const unsigned goff0 = (unsigned)(cbase * PANEL * sizeof(TV)) + (unsigned)(lane >> 2) * 16u;
  constexpr unsigned GBYTES = (unsigned)(GSTRIDE * PANEL * sizeof(TV));  // group to group, in a scalar register
  const unsigned tile_bytes = (unsigned)(j * PANEL * sizeof(TV));
  const bool uact = lane < UL;
  const int pos = wave * UL + (lane & (UL - 1));
  const int uk = pos & 3;
  const int urow = ((pos & 63) >> 2) * EPL + (pos >> 6);

  double acc[QW];
#pragma unroll
  for (int g = 0; g < QW; ++g) acc[g] = 0.0;
  double g0 = 0.0, g1 = 0.0, g2 = 0.0;

  const char *Wb = static_cast<const char *>(a.W);
  const size_t pbytes = (size_t)a.n_max * PANEL * sizeof(TV);
  TV ta[QW][EPL], tb[QW][EPL];

  // the unit's rows of column c start at c * PANEL + half * BROWS of its panel;
  // past the last unit every load is out of range and returns 0 without traffic
  // (unit numbers, below 2^31 for any basis that fits the card, and the choices
  // made from them are 32-bit and scalar: a resource that the compiler takes for
  // divergent costs a loop per load)
  const int pend = (int)a.P * UPP, pstep = (int)gridDim.x;
  auto tile_rsrc = [&](int u) {
    const int v = u < pend ? u : 0;
    const unsigned half = UPP > 1 ? (unsigned)(v % UPP) * (unsigned)(BROWS * sizeof(TV)) : 0u;
    return make_rsrc(Wb + (size_t)(v / UPP) * pbytes + half, u < pend ? tile_bytes - half : 0u);
  };
  auto load_group = [&](const __amdgpu_buffer_rsrc_t &r, int g, TV (&dst)[EPL]) {
    unpack16<TV>(__builtin_amdgcn_raw_buffer_load_b128(r, (int)goff0, (int)(g * GBYTES), kTileLoad), dst);
  };
  // snapshot rows of a unit: snapshot k's row r at byte (k * ldx + r) * sizeof(TX);
  // rows past the end are masked with the range itself, which may pass kOOR
  const unsigned xbytes = block_x_bytes(a.ldx, BROWS, sizeof(TX));
  const unsigned xoff0 = (unsigned)((uk * a.ldx + urow) * sizeof(TX));
  const int nfull = (int)(a.n / BROWS), nrem = (int)(a.n % BROWS);  // whole units, rows of the one after
  auto load_xs = [&](const void *x, int u) {
    const int v = u < pend ? u : 0;
    const int valid = u < nfull ? BROWS : (u == nfull ? nrem : 0);
    return buf_load_raw<TX>(make_rsrc(static_cast<const TX *>(x) + (size_t)v * BROWS, xbytes),
                            uact && urow < valid ? xoff0 : xbytes);
  };
  typedef typename std::conditional<SRC_X, TX, double>::type TY;
  auto load_y = [&](int u) -> TY {
    if constexpr (SRC_X) {
      return load_xs(a.x, u);
    } else {
      const int v = u < pend ? u : 0;
      return buf_load_raw<double>(make_rsrc(a.Z + (size_t)v * PAIRS, PAIRS * 8),
                                  uact && u < pend ? (unsigned)(pos * 8) : kOOR);
    }
  };

  TY y;
  TX yn = 0;
  int par = 0;
  // One unit, tile t; the tile of the unit after next is loaded into the same
  // registers group by group as the last phase is done with them, so between
  // one and two tiles per wavefront are always on their way.  The next unit's
  // y goes out before those loads: loads complete in order.
  auto step = [&](int p, TV (&t)[QW][EPL]) {
    const __amdgpu_buffer_rsrc_t rt = tile_rsrc(p + 2 * pstep);
    double wv = 0.0;
    if constexpr (!HAS_P1) wv = (double)y;
    if constexpr (HAS_P1) {
      double u[EPL][BPK];
#pragma unroll
      for (int e = 0; e < EPL; ++e)
#pragma unroll
        for (int k = 0; k < BPK; ++k) u[e][k] = 0.0;
      // the coefficients of group g + CD are read while group g's products run
      // (left to itself the compiler reads them next to their use)
      constexpr int CD = QW <= 12 ? 2 : 1;
      double cf[CD + 1][BPK];
      auto read_cf = [&](int g) {
#pragma unroll
        for (int k = 0; k < BPK; ++k) cf[g % (CD + 1)][k] = s_coef[(cbase + g * GSTRIDE) * BPK + k];
      };
#pragma unroll
      for (int g = 0; g < (CD < QW ? CD : QW); ++g) read_cf(g);
#pragma unroll
      for (int g = 0; g < QW; ++g) {
        if (g + CD < QW) read_cf(g + CD);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < BPK; ++k) {
#pragma unroll
          for (int e = 0; e < EPL; ++e) u[e][k] = fma((double)t[g][e], cf[g % (CD + 1)][k], u[e][k]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      // over the quad: lane cl ends with right-hand side cl of every row
      double *red = s_red + par * NW * PAIRS;
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const bool b0 = cl & 1, b1 = cl & 2;
        const double r01 = (b0 ? u[e][1] : u[e][0]) + dpp_mov<0xB1>(b0 ? u[e][0] : u[e][1]);
        const double r23 = (b0 ? u[e][3] : u[e][2]) + dpp_mov<0xB1>(b0 ? u[e][2] : u[e][3]);
        red[wave * PAIRS + e * 64 + lane] = (b1 ? r23 : r01) + dpp_mov<0x4E>(b1 ? r01 : r23);
      }
      if (NEXT_Y && uact) s_w[par][pos] = (double)yn;
      __syncthreads();
      double us = 0.0;
#pragma unroll
      for (int w2 = 0; w2 < NW; ++w2) us += red[w2 * PAIRS + pos];
      wv = (double)y - us;
      buf_store_scalar<double>(wv, make_rsrc(a.Z + (size_t)p * PAIRS, PAIRS * 8), uact ? (unsigned)(pos * 8) : kOOR);
    }
    if constexpr (GRAM) {
      // z_k z_k, z_k z_{k+1}, z_k z_{k+2} (k in the quad's lanes, mod 4)
      const double z = uact ? wv : 0.0;
      g0 = fma(z, z, g0);
      g1 = fma(z, dpp_mov<0x39>(z), g1);  // quad_perm 1,2,3,0
      g2 = fma(z, dpp_mov<0x4E>(z), g2);  // quad_perm 2,3,0,1
    }
    if (HAS_P2 && !NEXT_Y) {
      if (uact) s_w[par][pos] = wv;
      __syncthreads();
    }
    y = load_y(p + pstep);
    if constexpr (NEXT_Y) yn = load_xs(a.xn, p + pstep);
    if constexpr (HAS_P2) {
      if constexpr (sizeof(TV) == 4) {
        // keep only the FP32 tile live across the phases: convert again
#pragma unroll
        for (int g = 0; g < QW; ++g)
#pragma unroll
          for (int e = 0; e < EPL; ++e) asm volatile("" : "+v"(t[g][e]));
      }
      double we[EPL];
#pragma unroll
      for (int e = 0; e < EPL; ++e) we[e] = s_w[par][e * 64 + lane];
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
    } else {
#pragma unroll
      for (int g = 0; g < QW; ++g) load_group(rt, g, t[g]);
    }
    par ^= 1;
  };

  int p = blockIdx.x;
  y = load_y(p);
  if constexpr (NEXT_Y) yn = load_xs(a.xn, p);
  {
    const __amdgpu_buffer_rsrc_t r0 = tile_rsrc(p), r1 = tile_rsrc(p + pstep);
#pragma unroll
    for (int g = 0; g < QW; ++g) load_group(r0, g, ta[g]);
#pragma unroll
    for (int g = 0; g < QW; ++g) load_group(r1, g, tb[g]);
  }
  for (; p + pstep < pend; p += 2 * pstep) {
    step(p, ta);
    step(p + pstep, tb);
  }
  if (p < pend) step(p, ta);

  // accumulators: lane = rhs + 4 * block + 16 * column; the blocks (chunks mod
  // 4) are added by rotations within a row of 16 lanes
  if constexpr (HAS_P2) {
#pragma unroll
    for (int g = 0; g < QW; ++g) {
      const int c = wave * 4 + g * GSTRIDE + (lane >> 4);
      double v = acc[g] + dpp_mov<0x128>(acc[g]);
      v += dpp_mov<0x124>(v);
      if ((lane & 12) == 0 && c < j) a.partb[((size_t)c * BPK + cl) * a.ldg + slot] = v;
    }
  }
  if constexpr (GRAM) {
    double gv[3] = {g0, g1, g2};
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      double v = gv[m] + dpp_mov<0x128>(gv[m]);
      v += dpp_mov<0x124>(v);
      v = xor_sum<32>(xor_sum<16>(v));
      if (lane < 4) s_g[wave * 12 + m * 4 + lane] = v;
    }
    __syncthreads();
    if (tid < 12) {
      const int m = tid >> 2, k = tid & 3, l = (k + m) & 3;
      double v = 0.0;
      for (int w2 = 0; w2 < NW; ++w2) v += s_g[w2 * 12 + tid];
      if (m < 2 || k < 2) {
        a.partg[(size_t)slot * BPK * BPK + k * BPK + l] = v;
        a.partg[(size_t)slot * BPK * BPK + l * BPK + k] = v;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Passes over the n x BPK block, one thread per row (rows grid-strided).
// ZG_YNORM: partial ||y_k||^2 of the snapshots.  ZG_YNQ: the same and the
// partial products q_c^T y_k of the previous block's new columns with the
// snapshots (partq), when the sweep before formed V^T Y over the older
// columns (BP_ZR).  ZG_GRAM: the partial Gram
// matrix of Z T_0 .. T_{tlev-1} (T_t upper triangular, the inverses of the
// Cholesky steps so far), formed row by row from Z, which is never
// rewritten: the products are those a pass that stored Z T_0, then read it
// back for T_1, ... would form, in the same order, without the write streams.
// ZG_WRITEV: V's columns j .. j+BPK-1 <- Z T_0 T_1 T_2, rounded to the
// storage type.  Partials: partg[slot * GSLOT + (k * BPK + l)], slot =
// workgroup.
// ---------------------------------------------------------------------------
constexpr int GSLOT = BPK * BPK;
constexpr int GTRI = BPK * (BPK + 1) / 2;
constexpr int kBhRows = 576;  // rows of a column of H_bar products (j + BPK <= 512, in whole chunks)

// Sums of v[0 .. N) over a workgroup of 256 threads into sh[0 .. N) (wavefront
// sums, then over the wavefronts in order); sh: 5 N doubles.
template <int N>
__device__ __forceinline__ void wg_sums(const double (&v)[N], double *sh) {
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const double t = lanes_sum<64>(v[n]);
    if ((threadIdx.x & 63) == 0) sh[N + (threadIdx.x >> 6) * N + n] = t;
  }
  __syncthreads();
  if (threadIdx.x < N) {
    const double *w = sh + N + threadIdx.x;
    sh[threadIdx.x] = ((w[0] + w[N]) + w[2 * N]) + w[3 * N];
  }
  __syncthreads();
}

template <typename TV, typename TX, int MODE>
__global__ __launch_bounds__(256) void k_zgram(BlockArgs a) {
  __shared__ double sh[5 * (BPK + BPK * BPK)];
  __shared__ double sT[3 * BPK * BPK];
  const int tid = threadIdx.x;
  const int tlev = a.tlev;
  // Whether the block still runs is fetched with the rows and looked at before
  // anything is stored (the rows are there either way): a round trip of its own
  // costs each of these latency-bound passes most of a microsecond.
  const int status = a.st->status, rejected = *a.flag;
  // Z's order: units of BROWS rows (see k_bpass), row chunk * EPL + e of a
  // unit at e * 16 + chunk
  constexpr int EPL = Vec<TV>::EPL, BROWS = 16 * EPL;
  const int64_t npad = a.P * PANEL;
  const int64_t stride = (int64_t)gridDim.x * 256;
  if constexpr (MODE == ZG_YNORM || MODE == ZG_YNQ) {
    // ||y_k||^2 and (ZG_YNQ) h[c][k] = q_c^T y_k for the previous block's new
    // columns q_c = V(:, j - BPK + c), R rows in flight per thread (each sum takes
    // its rows in order)
    constexpr bool Q = MODE == ZG_YNQ;
    constexpr int R = Q ? 2 : 4;
    const TX *x = static_cast<const TX *>(a.x);
    const TV *W = static_cast<const TV *>(a.W);
    double s[Q ? BPK + BPK * BPK : BPK];
#pragma unroll
    for (int k = 0; k < (Q ? BPK + BPK * BPK : BPK); ++k) s[k] = 0.0;
    auto rows = [&](int64_t r, auto nr) {
      constexpr int N = decltype(nr)::value;
      double y[N][BPK], q[N][BPK];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const int64_t ru = r + u * stride;
#pragma unroll
        for (int k = 0; k < BPK; ++k) y[u][k] = (double)x[(int64_t)k * a.ldx + ru];
        if constexpr (Q) {
          const TV *qr = W + ((ru / PANEL) * a.n_max + (a.j - BPK)) * PANEL + ru % PANEL;
#pragma unroll
          for (int c = 0; c < BPK; ++c) q[u][c] = (double)qr[c * PANEL];
        }
      }
#pragma unroll
      for (int u = 0; u < N; ++u) {
#pragma unroll
        for (int k = 0; k < BPK; ++k) s[k] = fma(y[u][k], y[u][k], s[k]);
        if constexpr (Q) {
#pragma unroll
          for (int c = 0; c < BPK; ++c)
#pragma unroll
            for (int k = 0; k < BPK; ++k) s[BPK + c * BPK + k] = fma(q[u][c], y[u][k], s[BPK + c * BPK + k]);
        }
      }
    };
    int64_t r = (int64_t)blockIdx.x * 256 + tid;
    for (; r + (R - 1) * stride < a.n; r += R * stride) rows(r, std::integral_constant<int, R>{});
    for (; r < a.n; r += stride) rows(r, std::integral_constant<int, 1>{});
    wg_sums(s, sh);
    if (status != ST_ACTIVE || rejected) return;
    if (tid < BPK) a.partg[(size_t)blockIdx.x * GSLOT + tid * BPK + tid] = sh[tid];
    if (Q && tid < GSLOT) a.partq[(size_t)blockIdx.x * GSLOT + tid] = sh[BPK + tid];
    return;
  }
  double g[GTRI];  // upper triangle by rows
#pragma unroll
  for (int k = 0; k < GTRI; ++k) g[k] = 0.0;
  // z <- z T_0 .. T_{tlev-1}
  auto transform = [&](double (&z)[BPK]) {
    for (int t = 0; t < tlev; ++t) {
      const double *T = sT + t * BPK * BPK;
      double o[BPK];
#pragma unroll
      for (int l = 0; l < BPK; ++l) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k <= l; ++k) s = fma(z[k], T[k * BPK + l], s);  // T[k][l], k <= l
        o[l] = s;
      }
#pragma unroll
      for (int l = 0; l < BPK; ++l) z[l] = o[l];
    }
  };
  // two rows at a time, the next two in flight (a second past the end reads the
  // first again)
  double z[2][BPK];
  auto load = [&](int64_t r) {
    if (r >= npad) return;
    const int64_t r2 = r + stride < npad ? r + stride : r;
#pragma unroll
    for (int k = 0; k < BPK; ++k) {
      z[0][k] = a.Z[r * BPK + k];
      z[1][k] = a.Z[r2 * BPK + k];
    }
  };
  int64_t r = (int64_t)blockIdx.x * 256 + tid;
  const double tv = tid < tlev * BPK * BPK ? a.sm[SM_T + tid] : 0.0;
  load(r);
  if (tid < tlev * BPK * BPK) sT[tid] = tv;
  __syncthreads();
  if (MODE == ZG_WRITEV && (status != ST_ACTIVE || rejected)) return;
  for (; r < npad; r += 2 * stride) {
    double y[2][BPK];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int k = 0; k < BPK; ++k) y[u][k] = z[u][k];
    const bool two = r + stride < npad;
    load(r + 2 * stride);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      transform(y[u]);
      if (u && !two) break;
      if (MODE == ZG_WRITEV) {
        const int64_t ru = r + u * stride;
        const int rr = (int)(ru % PANEL), ri = rr % BROWS;
        TV *vc = static_cast<TV *>(a.W) + (size_t)(ru / PANEL) * a.n_max * PANEL + (size_t)a.j * PANEL + (rr - ri) +
                 (ri % 16) * EPL + ri / 16;
#pragma unroll
        for (int k = 0; k < BPK; ++k) vc[k * PANEL] = (TV)y[u][k];
        continue;
      }
      int m = 0;
#pragma unroll
      for (int k = 0; k < BPK; ++k)
#pragma unroll
        for (int l = k; l < BPK; ++l, ++m) g[m] = fma(y[u][k], y[u][l], g[m]);
    }
  }
  if (MODE == ZG_WRITEV) return;
  wg_sums(g, sh);
  if (status != ST_ACTIVE || rejected) return;
  if (tid < GSLOT) {
    const int k = min(tid / BPK, tid % BPK), l = max(tid / BPK, tid % BPK);
    a.partg[(size_t)blockIdx.x * GSLOT + tid] = sh[k * BPK - k * (k - 1) / 2 + l - k];
  }
}

// ---------------------------------------------------------------------------
// Reduction of the block-pass partials: one wavefront per (column, rhs) pair
// in a fixed order.  MODE 1 (after BP_R1): R = sigma o D, coef = sigma o R,
// and (extra wavefronts) ||y_k||^2 from the ZG_YNORM partials.  MODE 2 (after
// BP_Z1): R2 = sigma o D, R += R2, coef = sigma o R2.  MODE 3 (after BP_D):
// R += sigma o D, coef = sigma o (sigma o D).  MODE 1 with a.qy: D of the
// columns before the previous block's from dnext (summed by MODE 4 during
// that block), of the previous block's 4 from the ZG_YNQ partials.  MODE 4
// (after BP_ZR): the raw sums D into dnext, for the next block.
// ---------------------------------------------------------------------------
// sum of p[g * GSLOT], g < G, by one wavefront, eight loads in flight per lane
__device__ __forceinline__ double slot_sum(const double *p, int G, int lane) {
  double t = 0.0;
  for (int g = lane; g < G; g += 64 * 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = g + 64 * u < G ? p[(size_t)(g + 64 * u) * GSLOT] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) t += v[u];
  }
  return lanes_sum<64>(t);
}

template <int MODE>
__global__ __launch_bounds__(256) void k_breduce(BlockArgs a) {
  if (a.gate && !*a.gate) return;
  const bool run = a.st->status == ST_ACTIVE && !*a.flag;  // looked at before anything is stored
  const int lane = threadIdx.x & 63;
  const int wv = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int npairs = a.j * BPK;
  if (wv < npairs) {
    const int c = wv / BPK, k = wv % BPK;
    double t = 0.0;
    if (MODE == 1 && a.qy && c < a.j - BPK) {
      t = a.dnext[wv];
    } else if (MODE == 1 && a.qy) {
      const int e = (c - (a.j - BPK)) * BPK + k;
      t = slot_sum(a.partq + e, a.Gz, lane);
    } else {
      t = strided_sum<false>(a.partb + (size_t)wv * a.ldg, a.G, lane);
    }
    if (MODE == 4) {
      if (lane == 0 && run) a.dnext[wv] = t;
      return;
    }
    if (lane == 0 && run) {
      const double r = a.sigma[c] * t;
      const size_t idx = (size_t)c * BPK + k;
      if (MODE == 1) {
        a.sm[SM_R + idx] = r;
      } else {
        a.sm[SM_R + idx] += r;
      }
      if (MODE == 2) a.sm[SM_R2 + idx] = r;
      a.coef[idx] = a.sigma[c] * r;
    }
  } else if (MODE == 1 && wv < npairs + BPK) {
    const int k = wv - npairs;
    const double t = slot_sum(a.partg + k * BPK + k, a.Gz, lane);
    if (lane == 0 && run) a.sm[SM_YN2 + k] = t;
  }
}

// ---------------------------------------------------------------------------
// The Gram partials of the workgroups of a block pass, reduced in a fixed
// order into sG[0 .. GSLOT): thread t sums entry t % GSLOT over the slots
// t / GSLOT, + 64, ... (at most 1024 / 64 = 16, all in flight); the four
// slot lanes of a wavefront are then added by lane swaps, the wavefronts in
// order.  One workgroup of kGramThreads threads; sG is complete on return.
// (256 threads, eight loads at a time: 6 of k_bchol's 12 us.)
// ---------------------------------------------------------------------------
constexpr int kGramThreads = 1024;
static_assert(GSLOT == 16, "four slot lanes of 16 entries per wavefront");
__device__ inline void gram_reduce(const BlockArgs &a, int tid, double *sh, double *sG) {
  constexpr int SL = kGramThreads / GSLOT;  // slot lanes per entry
  const int e = tid % GSLOT, s0 = tid / GSLOT;
  double v[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) v[m] = s0 + m * SL < a.Gg ? a.partg[(size_t)(s0 + m * SL) * GSLOT + e] : 0.0;
  double t = 0.0;
#pragma unroll
  for (int m = 0; m < 16; ++m) t += v[m];
  t = xor_sum<32>(xor_sum<16>(t));
  if ((tid & 63) < GSLOT) sh[(tid >> 6) * GSLOT + e] = t;
  __syncthreads();
  if (tid < GSLOT) {
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < kGramThreads / 64; ++w) r += sh[w * GSLOT + tid];
    sG[tid] = r;
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Cholesky step ROUND (0: shifted; 0, 1, 2) of the block QR: reduce the Gram
// partials (fixed order), factor G (+ s I) = S^T S, store T_ROUND = S^{-1}
// and accumulate S_total = S S_total.  A non-finite Gram matrix or a non-positive pivot
// rejects the block.  One workgroup; the 4 x 4 algebra runs in thread 0.
// ---------------------------------------------------------------------------
template <int ROUND>
__global__ __launch_bounds__(kGramThreads) void k_bchol(BlockArgs a) {
  __shared__ double sh[256];
  __shared__ double sG[GSLOT];
  const int tid = threadIdx.x;
  // all of it is fetched at once; nothing is stored for a block that has stopped
  const int status = a.st->status, rejected = *a.flag;
  double Stot[BPK * BPK] = {};
  if (ROUND > 0 && tid == 0) {
#pragma unroll
    for (int k = 0; k < BPK * BPK; ++k) Stot[k] = a.sm[SM_S + k];
  }
  gram_reduce(a, tid, sh, sG);
  if (tid != 0 || status != ST_ACTIVE || rejected) return;
  // every loop unrolled, the matrices in registers (indexed at run time they lived
  // in scratch memory: 7.5 us a step, 4.9 us so)
  double G[BPK][BPK], S[BPK][BPK] = {}, T[BPK][BPK] = {};
  bool ok = true;
#pragma unroll
  for (int k = 0; k < BPK; ++k)
#pragma unroll
    for (int l = 0; l < BPK; ++l) {
      // symmetric part (the two triangles are sums of the same products)
      G[k][l] = 0.5 * (sG[k * BPK + l] + sG[l * BPK + k]);
      ok = ok && isfinite(G[k][l]);
    }
  if (ROUND == 0) {
    double tr = 0.0;
#pragma unroll
    for (int k = 0; k < BPK; ++k) tr += G[k][k];
    const double s = 11.0 * ((double)a.n * BPK + BPK * (BPK + 1)) * 0x1p-53 * tr;
#pragma unroll
    for (int k = 0; k < BPK; ++k) G[k][k] += s;
  }
  // G = S^T S, S upper triangular with a positive diagonal (a bad pivot goes on with
  // values that nothing stores)
#pragma unroll
  for (int k = 0; k < BPK; ++k) {
    double d = G[k][k];
#pragma unroll
    for (int i = 0; i < k; ++i) d -= S[i][k] * S[i][k];
    ok = ok && d > 0.0 && isfinite(d);
    S[k][k] = sqrt(d);
#pragma unroll
    for (int l = k + 1; l < BPK; ++l) {
      double v = G[k][l];
#pragma unroll
      for (int i = 0; i < k; ++i) v -= S[i][k] * S[i][l];
      S[k][l] = v / S[k][k];
    }
  }
  if (!ok) {
    *a.flag = 1;
    return;
  }
  // T = S^{-1} (upper triangular), column by column: S T_{:,l} = e_l
#pragma unroll
  for (int l = 0; l < BPK; ++l) {
#pragma unroll
    for (int k = BPK - 1; k >= 0; --k) {
      if (k > l) continue;
      double v = (k == l) ? 1.0 : 0.0;
#pragma unroll
      for (int i = k + 1; i <= l; ++i) v -= S[k][i] * T[i][l];
      T[k][l] = v / S[k][k];
    }
  }
#pragma unroll
  for (int k = 0; k < BPK; ++k)
#pragma unroll
    for (int l = 0; l < BPK; ++l) {
      double v = 0.0;
      if (ROUND == 0) {
        v = S[k][l];
      } else {
#pragma unroll
        for (int i = k; i <= l; ++i) v += S[k][i] * Stot[i * BPK + l];
      }
      a.sm[SM_S + k * BPK + l] = v;
      a.sm[SM_T + ROUND * GSLOT + k * BPK + l] = T[k][l];
    }
}

// ---------------------------------------------------------------------------
// Commit of an accepted block (one workgroup): breakdown test on the new
// diagonal of beta, then beta's columns j .. j+BPK-1, sigma and the scalar
// state.  On rejection nothing is written except the flag.  H_bar follows in
// k_bcommit_h; workgroups 1, 2, ... form the products it starts from (they need
// nothing of the commit).
// ---------------------------------------------------------------------------
// Sums over the old columns l < j-1 of H_bar[i, l] beta[l, j-1+k], k < BPK (beta's
// new columns from the small area): 64 rows x 4 slices of the l range of one of
// bh_slices(j) workgroups per row chunk, into partb[(slice * BPK + k) * kBhRows + i].
// One workgroup per row chunk read all of H_bar through 8 CUs: 32 us at 250
// columns.
__host__ __device__ constexpr int bh_slices(int j) { return j < 128 ? 1 : (j < 512 ? j / 64 : 8); }
__device__ inline void bcommit_products(const BlockArgs &a, int wg) {
  __shared__ double sh[4][64][BPK];
  const int j = a.j;
  const int S = bh_slices(j), chunk = wg / S, sl = (wg - chunk * S) * 4 + (threadIdx.x >> 6);
  const int r = threadIdx.x & 63, i = chunk * 64 + r;  // 0-based row, below j - 1 + BPK
  double t[BPK];
#pragma unroll
  for (int k = 0; k < BPK; ++k) t[k] = 0.0;
  const int lo = i > 0 ? i - 1 : 0, hi = j - 1, len = hi > lo ? hi - lo : 0;
  const int a0 = lo + (len * sl) / (4 * S), a1 = lo + (len * (sl + 1)) / (4 * S);
  const double *bj = a.beta + (size_t)(j - 1) * a.ldB;
  int l = a0;
  for (; l + 4 <= a1; l += 4) {
    double h[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) h[u] = a.H[(size_t)(l + u) * a.ldH + i];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      t[0] = fma(h[u], bj[l + u], t[0]);
#pragma unroll
      for (int k = 1; k < BPK; ++k) t[k] = fma(h[u], a.sm[SM_R + (l + u) * BPK + k - 1], t[k]);
    }
  }
  for (; l < a1; ++l) {
    const double h = a.H[(size_t)l * a.ldH + i];
    t[0] = fma(h, bj[l], t[0]);
#pragma unroll
    for (int k = 1; k < BPK; ++k) t[k] = fma(h, a.sm[SM_R + l * BPK + k - 1], t[k]);
  }
#pragma unroll
  for (int k = 0; k < BPK; ++k) sh[threadIdx.x >> 6][r][k] = t[k];
  __syncthreads();
  if (threadIdx.x < 64) {
#pragma unroll
    for (int k = 0; k < BPK; ++k)
      a.partb[(size_t)((wg - chunk * S) * BPK + k) * kBhRows + i] = ((sh[0][r][k] + sh[1][r][k]) + sh[2][r][k]) + sh[3][r][k];
  }
}

__global__ __launch_bounds__(256) void k_bcommit(BlockArgs a) {
  DevState *st = a.st;
  if (st->status != ST_ACTIVE) return;
  // without a look at the flag, which workgroup 0 may be setting: nothing reads the
  // products of a rejected block
  if (blockIdx.x > 0) {
    bcommit_products(a, (int)blockIdx.x - 1);
    return;
  }
  if (*a.flag) return;
  __shared__ int s_ok;
  const int tid = threadIdx.x;
  const int j = a.j;
  const double *Stot = a.sm + SM_S;
  int bad = 0;
  for (int e = tid; e < j * BPK; e += 256) bad |= !isfinite(a.sm[SM_R + e]);
  bad = __syncthreads_or(bad);
  if (tid == 0) {
    bool ok = !bad;
    double xf = st->xfro2;
    for (int k = 0; k < BPK; ++k) {
      const double yk = a.sm[SM_YN2 + k];
      ok = ok && isfinite(yk);
      xf += yk;
      const double skk = Stot[k * BPK + k];
      ok = ok && isfinite(skk) && skk > st->tol * sqrt(xf);
    }
    s_ok = ok ? 1 : 0;
    if (!ok) *a.flag = 1;
  }
  __syncthreads();
  if (!s_ok) return;
  // beta's new columns: rows 0..j-1 from R, rows j..j+BPK-1 from S
  for (int e = tid; e < j * BPK; e += 256) {
    const int c = e / BPK, k = e % BPK;
    a.beta[(size_t)(j + k) * a.ldB + c] = a.sm[SM_R + e];
  }
  if (tid < BPK * BPK) {
    const int k = tid / BPK, l = tid % BPK;
    if (k <= l) a.beta[(size_t)(j + l) * a.ldB + (j + k)] = Stot[k * BPK + l];
  }
  if (tid < BPK) a.sigma[j + tid] = 1.0;
  if (tid == 0) {
    double xf = st->xfro2;
    for (int k = 0; k < BPK; ++k) xf += a.sm[SM_YN2 + k];
    st->xfro2 = xf;
    st->q = j + BPK;
    st->pushes += BPK;
  }
}

// ---------------------------------------------------------------------------
// H_bar's new columns c = j-1 .. j+BPK-2 (0-based) of an accepted block, from
// H_bar_{:,c} beta_{c,c} = beta_{:,c+1} - H_bar_{:,0:c-1} beta_{0:c-1,c}.  The
// part of the sum over the old columns comes from k_bcommit's other workgroups
// (slices added in order); each row then runs the BPK-step recurrence over the
// new columns by itself.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_bcommit_h(BlockArgs a) {
  DevState *st = a.st;
  const int j = a.j;
  const int i = blockIdx.x * 64 + threadIdx.x;  // 0-based row
  const int rows = j + BPK;                     // rows 0 .. j+BPK-1 carry the new columns
  const int S = bh_slices(j);
  double t[BPK];
#pragma unroll
  for (int k = 0; k < BPK; ++k) {
    t[k] = 0.0;
    for (int q = 0; q < S; ++q) t[k] += a.partb[(size_t)(q * BPK + k) * kBhRows + i];
  }
  if (*a.flag || st->q != j + BPK || i >= rows) return;  // rejected, or nothing committed
  double hn[BPK];
#pragma unroll
  for (int k = 0; k < BPK; ++k) {
    const int c = j - 1 + k;
    double v = a.beta[(size_t)(c + 1) * a.ldB + i];
    v -= t[k];
    for (int kk = 0; kk < k; ++kk) v -= hn[kk] * a.beta[(size_t)c * a.ldB + (j - 1 + kk)];
    hn[k] = (i <= c + 1) ? v / a.beta[(size_t)c * a.ldB + c] : 0.0;
    a.H[(size_t)c * a.ldH + i] = hn[k];
  }
  if (i == rows - 1) st->hlast = hn[BPK - 1];
}

__global__ void k_bflag_clear(int *flag) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *flag = 0;
}

// ---------------------------------------------------------------------------
// Test for the third projection, after the Gram pass of Z = Y - V (R1 + R2):
// ||Z_k||^2 from the Gram partials (fixed order), ||R2||_F, ||R2_k|| and
// ||R1||_F = ||R - R2||_F from the small area.  *gate = 1 when
// (||R2||_F / ||R1||_F) ||R2_k|| > unit ||Z_k|| / 10 for some k, else 0
// (also for a rejected block).  One workgroup.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kGramThreads) void k_bthird(BlockArgs a, int *gate, double unit) {
  __shared__ double sh[kGramThreads / 64 * GSLOT];
  __shared__ double sG[GSLOT];
  __shared__ double s_w[kGramThreads / 64][BPK + 1];
  const int tid = threadIdx.x;
  if (a.st->status != ST_ACTIVE || *a.flag) {
    if (tid == 0) *gate = 0;
    return;
  }
  // thread t: right-hand side t % BPK of the columns t / BPK, + 256, ...
  const int npairs = a.j * BPK;
  double r1 = 0.0, r2 = 0.0;
  for (int e = tid; e < npairs; e += kGramThreads) {
    const double v2 = a.sm[SM_R2 + e];
    const double v1 = a.sm[SM_R + e] - v2;
    r1 = fma(v1, v1, r1);
    r2 = fma(v2, v2, r2);
  }
  r1 = lanes_sum<64>(r1);
  r2 = r2 + dpp_mov<0x128>(r2);  // over the lanes of equal t % BPK
  r2 = r2 + dpp_mov<0x124>(r2);
  r2 = xor_sum<32>(xor_sum<16>(r2));
  if ((tid & 63) < BPK) s_w[tid >> 6][tid & 63] = r2;
  if ((tid & 63) == BPK) s_w[tid >> 6][BPK] = r1;
  gram_reduce(a, tid, sh, sG);
  double s_r2[BPK], s_z2[BPK], r1s = 0.0;
#pragma unroll
  for (int k = 0; k < BPK; ++k) {
    s_r2[k] = 0.0;
    s_z2[k] = sG[k * BPK + k];
  }
  for (int w = 0; w < kGramThreads / 64; ++w) {
#pragma unroll
    for (int k = 0; k < BPK; ++k) s_r2[k] += s_w[w][k];
    r1s += s_w[w][BPK];
  }
  if (tid != 0) return;
  int third = 0;
  if (r1s > 0.0) {
    double r2f = 0.0;
    for (int k = 0; k < BPK; ++k) r2f += s_r2[k];
    const double e = sqrt(r2f) / sqrt(r1s);
    for (int k = 0; k < BPK; ++k) third |= e * sqrt(s_r2[k]) > 0.1 * unit * sqrt(s_z2[k]);
  }
  *gate = third;
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Workgroup shape of the block passes over j columns (tiles of QW groups of
// four columns on NW wavefronts): 4 wavefronts while their registers hold it
// (256 columns), 8 beyond, which fill a CU, and the narrowest tile that covers j,
// as the groups beyond it are arithmetic for nothing.  With widths of 1, 2, 4, 8
// and 16 groups alone: 2^22 x 500 FP32 230.7 ms (217.4 so), 2^22 x 256 67.8
// (65.6), 300007 x 320 FP64 19.5 (19.0), 100037 x 200 5.07 (4.98).
// Workgroups per CU: 4 up to 64 columns (2 take 12% longer, 1000003 x 30 FP64), 2 up
// to 256 (100037 x 200 FP32 4.74 ms, with the 3 that the registers hold 4.96, with
// 4 5.31; FP64 5.49, 5.72 and 5.98), 1 beyond (with 2, 30000 x 500 FP32 12.6 ms
// instead of 11.8).
BlockShape block_shape(int j) {
  static const int q4[] = {1, 2, 4, 6, 8, 10, 12, 14, 16}, q8[] = {10, 12, 14, 16};
  if (j <= 256) {
    for (int q : q4)
      if (16 * q >= j) return {4, q, q <= 4 ? 4 : 2};
  }
  for (int q : q8)
    if (32 * q >= j) return {8, q, 1};
  return {8, 16, 1};
}

template <typename TV, typename TX, int MODE>
static hipError_t launch_bpass_q(int nw, int qw, int grid, const BlockArgs &a, hipStream_t s) {
#define FOA_BPASS(NW, QW)                                                                              \
  case NW * 100 + QW:                                                                                  \
    hipLaunchKernelGGL((k_bpass<TV, TX, NW, QW, MODE>), dim3(grid), dim3(NW * 64), 0, s, a);           \
    break;
  switch (nw * 100 + qw) {
    FOA_BPASS(4, 1)
    FOA_BPASS(4, 2)
    FOA_BPASS(4, 4)
    FOA_BPASS(4, 6)
    FOA_BPASS(4, 8)
    FOA_BPASS(4, 10)
    FOA_BPASS(4, 12)
    FOA_BPASS(4, 14)
    FOA_BPASS(4, 16)
    FOA_BPASS(8, 10)
    FOA_BPASS(8, 12)
    FOA_BPASS(8, 14)
    FOA_BPASS(8, 16)
    default: return hipErrorInvalidValue;
  }
#undef FOA_BPASS
  return hipGetLastError();
}

template <typename TV, typename TX>
static hipError_t launch_bpass_m(int mode, const BlockShape &sh, int grid, const BlockArgs &a, hipStream_t s) {
  switch (mode) {
    case BP_R1: return launch_bpass_q<TV, TX, BP_R1>(sh.nw, sh.qw, grid, a, s);
    case BP_Z1: return launch_bpass_q<TV, TX, BP_Z1>(sh.nw, sh.qw, grid, a, s);
    case BP_D: return launch_bpass_q<TV, double, BP_D>(sh.nw, sh.qw, grid, a, s);
    case BP_ZR: return launch_bpass_q<TV, TX, BP_ZR>(sh.nw, sh.qw, grid, a, s);
    default: return launch_bpass_q<TV, double, BP_Z2>(sh.nw, sh.qw, grid, a, s);
  }
}

hipError_t launch_bpass(int mode, bool tv_f64, bool tx_f64, int grid, const BlockArgs &a, hipStream_t s) {
  const BlockShape sh = block_shape(a.j);
  if (sh.nw * sh.qw * 4 < a.j) return hipErrorInvalidValue;  // tile narrower than the basis
  if (tv_f64)
    return tx_f64 ? launch_bpass_m<double, double>(mode, sh, grid, a, s)
                  : launch_bpass_m<double, float>(mode, sh, grid, a, s);
  return tx_f64 ? launch_bpass_m<float, double>(mode, sh, grid, a, s)
                : launch_bpass_m<float, float>(mode, sh, grid, a, s);
}

template <typename TV, typename TX>
static hipError_t launch_zgram_t(int mode, int grid, const BlockArgs &a, hipStream_t s) {
  switch (mode) {
    case ZG_YNORM: hipLaunchKernelGGL((k_zgram<TV, TX, ZG_YNORM>), dim3(grid), dim3(256), 0, s, a); break;
    case ZG_GRAM: hipLaunchKernelGGL((k_zgram<TV, TX, ZG_GRAM>), dim3(grid), dim3(256), 0, s, a); break;
    case ZG_YNQ: hipLaunchKernelGGL((k_zgram<TV, TX, ZG_YNQ>), dim3(grid), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((k_zgram<TV, TX, ZG_WRITEV>), dim3(grid), dim3(256), 0, s, a); break;
  }
  return hipGetLastError();
}

hipError_t launch_zgram(int mode, bool tv_f64, bool tx_f64, int grid, const BlockArgs &a, hipStream_t s) {
  if (tv_f64)
    return tx_f64 ? launch_zgram_t<double, double>(mode, grid, a, s) : launch_zgram_t<double, float>(mode, grid, a, s);
  return tx_f64 ? launch_zgram_t<float, double>(mode, grid, a, s) : launch_zgram_t<float, float>(mode, grid, a, s);
}

hipError_t launch_breduce(int mode, const BlockArgs &a, hipStream_t s) {
  const int waves = a.j * BPK + (mode == 1 ? BPK : 0);
  const int blocks = (waves + 3) / 4;
  if (mode == 1)
    hipLaunchKernelGGL(k_breduce<1>, dim3(blocks), dim3(256), 0, s, a);
  else if (mode == 2)
    hipLaunchKernelGGL(k_breduce<2>, dim3(blocks), dim3(256), 0, s, a);
  else if (mode == 3)
    hipLaunchKernelGGL(k_breduce<3>, dim3(blocks), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(k_breduce<4>, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bchol(int round, const BlockArgs &a, hipStream_t s) {
  if (round == 0)
    hipLaunchKernelGGL(k_bchol<0>, dim3(1), dim3(kGramThreads), 0, s, a);
  else if (round == 1)
    hipLaunchKernelGGL(k_bchol<1>, dim3(1), dim3(kGramThreads), 0, s, a);
  else
    hipLaunchKernelGGL(k_bchol<2>, dim3(1), dim3(kGramThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bcommit(const BlockArgs &a, hipStream_t s) {
  const int chunks = (a.j + BPK + 63) / 64;
  if (chunks * 64 > kBhRows) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_bcommit, dim3(1 + chunks * bh_slices(a.j)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_bcommit_h, dim3(chunks), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_bflag_clear(int *flag, hipStream_t s) {
  hipLaunchKernelGGL(k_bflag_clear, dim3(1), dim3(64), 0, s, flag);
  return hipGetLastError();
}

hipError_t launch_bthird(const BlockArgs &a, int *gate, double unit, hipStream_t s) {
  hipLaunchKernelGGL(k_bthird, dim3(1), dim3(kGramThreads), 0, s, a, gate, unit);
  return hipGetLastError();
}

}  // namespace foa
