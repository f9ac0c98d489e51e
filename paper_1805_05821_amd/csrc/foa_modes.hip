// Mode reconstruction Phi = V B (the modes of Algorithm 1): the panel-layout
// basis W (n x k columns in use, FP32 or FP64) times the k x r coefficient
// matrix B (FP64, sigma folded in, packed real columns).  An FP32 basis with
// FP32 output runs on bf16 MFMA with every value split in three (FP32 MFMA for
// small products, few columns and coefficients outside the split's range), every
// other combination on FP64 MFMA.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "foa_buffer.h"
#include "foa_internal.h"

namespace foa {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// FP64-accumulating kernel (FP64 basis or FP64 output): Phi^T = B^T W^T on
// v_mfma_f64_16x16x4.  A wavefront owns 32 rows (two row tiles: the even and the
// odd rows, so a lane's load is two consecutive rows) x MB 16-mode blocks; four
// wavefronts share the coefficients, staged through LDS 16 basis columns at a
// time.  The basis goes straight from memory to the operand registers, the next
// stage's columns one stage ahead: each is used by its own wavefront alone.
// Coefficients are k-major without padding (a copy to the device beyond 16 KiB
// costs 4 us more), read as operand fragments: mode lane % 16, column lane / 16 (D:
// row = lane % 16, mode 4 t + lane / 16).
// Bound: the FP64 matrix rate (78.6 TFLOP/s); 2 n k r flops.  One thread per row
// with 16 modes' sums in registers (each reading the basis again, every product
// behind an LDS read) ran 2^18 x 149 x 60 in 438 us, 10.7 TFLOP/s.
constexpr int M64_K = 16, M64_MB = 8;

template <typename TV, typename TO, int MB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_modes_mfma64(
    const TV *W, int64_t n, int64_t P, int n_max, int kdim, const double *Bk, int r, TO *out, int64_t ld) {
  constexpr int KS = M64_K / 4;      // MFMA steps of a stage
  constexpr int FR = KS * MB;        // fragments of a stage (512 bytes each)
  constexpr int NL = (FR + 3) / 4;   // loads per wavefront
  __shared__ double sB[FR * 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m0 = (int64_t)blockIdx.x * 128 + wave * 32;
  const int64_t p = m0 / PANEL;
  const int mb0 = blockIdx.y * MB;
  // columns beyond kdim (and a panel beyond the last) read as 0
  const __amdgpu_buffer_rsrc_t rw =
      make_rsrc(W + (size_t)(p < P ? p : 0) * n_max * PANEL, p < P ? (unsigned)(kdim * PANEL * sizeof(TV)) : 0u);
  const unsigned woff = (unsigned)(((lane >> 4) * PANEL + (int)(m0 % PANEL) + 2 * (lane & 15)) * sizeof(TV));
  f64x4 acc[2][MB];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < MB; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  // coefficient rows beyond kdim and modes beyond r read as 0
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(Bk, (unsigned)(kdim * r * 8));
  TV w[KS][2];
  double bn[NL];
  auto load_w = [&](int k0) {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const unsigned off = woff + (unsigned)((k0 + 4 * s) * PANEL * sizeof(TV));
      if constexpr (sizeof(TV) == 8) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)off, 0, kTileLoad);
        w[s][0] = __builtin_bit_cast(double, u32x2{v.x, v.y});
        w[s][1] = __builtin_bit_cast(double, u32x2{v.z, v.w});
      } else {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rw, (int)off, 0, kTileLoad);
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        const f32x2 f = __builtin_bit_cast(f32x2, v);
        w[s][0] = f.x;
        w[s][1] = f.y;
      }
    }
  };
  auto load_b = [&](int k0) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int f = wave + 4 * i;  // fragment of the stage: step f / MB, mode block f % MB
      const int mode = (mb0 + f % MB) * 16 + (lane & 15), l = k0 + f / MB * 4 + (lane >> 4);
      if (f < FR)
        bn[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                               rb, mode < r ? (l * r + mode) * 8 : (int)kOOR, 0, 0));
    }
  };
  load_b(0);
  load_w(0);
  for (int k0 = 0; k0 < kdim; k0 += M64_K) {
    if (k0) __syncthreads();
#pragma unroll
    for (int i = 0; i < NL; ++i)
      if (wave + 4 * i < FR) sB[(wave + 4 * i) * 64 + lane] = bn[i];
    __syncthreads();
    TV wc[KS][2];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      wc[s][0] = w[s][0];
      wc[s][1] = w[s][1];
    }
    if (k0 + M64_K < kdim) {
      load_b(k0 + M64_K);
      load_w(k0 + M64_K);
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const double w0 = (double)wc[s][0], w1 = (double)wc[s][1];
#pragma unroll
      for (int b = 0; b < MB; ++b) {
        const double c = sB[(s * MB + b) * 64 + lane];
        acc[0][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(c, w0, acc[0][b], 0, 0, 0);
        acc[1][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(c, w1, acc[1][b], 0, 0, 0);
      }
    }
  }
  const int64_t row = m0 + 2 * (lane & 15);
  if (row >= n) return;
  const bool both = row + 1 < n;
#pragma unroll
  for (int b = 0; b < MB; ++b)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int mode = (mb0 + b) * 16 + 4 * t + (lane >> 4);
      if (mode < r) {
        TO *o = out + (size_t)mode * ld + row;
        o[0] = (TO)acc[0][b][t];
        if (both) o[1] = (TO)acc[1][b][t];
      }
    }
}

// FP32 basis and FP32 output on the bf16 matrix units: every FP32 value is the
// sum of three bf16 values exactly, w = w1 + w2 + w3 (each the rest rounded to
// nearest, so |w2| <= 2^-8 and |w3| <= 2^-17 for a significand in [1, 2)) and b
// likewise (by k_modes_split_coefs), and the six products
//   b1 w1 + (b1 w2 + b2 w1) + (b1 w3 + b2 w2 + b3 w1)
// are accumulated in FP32; what is left out, b2 w3 + b3 w2 + b3 w3, is below 2^-24
// |b w|.  A product accumulated into a sum costs a rounding of that sum's size,
// so b1 w1 alone enters the running sum, 16 columns at once, and the small five of
// 32 columns are added to it together: three roundings where FP32 products summed
// in turn take 32.  Measured against 64 bits, error of this kernel over that of
// k_modes_mfma (norm over all modes / of the worst mode): travelling oscillations
// of 34, 64 and 160 modes 0.49 / 0.48, 0.43 / 0.38 and 0.39 / 0.37; Gaussian streams
// of 33, 39, 48, 64 and 160 modes 1.05 / 0.88, 0.96 / 0.78, 0.87 / 0.69, 0.73 / 0.57
// and 0.49 / 0.38; modes that are one column of the basis 1.05 / 1.13, the sum of two
// far apart 1.28 / 1.39 (both below one FP32 rounding of the result).  All six into
// one sum: 0.79 / 0.80 for 160 travelling oscillations, 1.6 / 1.6 for single columns;
// b2 w3 and b3 w2 as well: 0.38 / 0.37 and 1.00 / 1.00, 2^22 x 160 modes 1.78 ms.
// Tile: 128 rows x 32 NB modes per workgroup, wavefront w its rows 32 w .. + 31.
// The basis goes from memory straight to registers (lane: row lane % 32, eight
// columns from 8 (lane / 32)) and is split there, one stage of 32 columns ahead;
// the coefficients are staged through LDS as operand fragments, [k / 16][mode /
// 32][piece][lane][8].
// Bound: HBM (n k + n r values of 4 bytes) up to about 200 modes per pass, the
// bf16 rate beyond.  2^22 x 160 modes 1.54 ms; on the FP32 matrix units
// (k_modes_mfma) 2.07 ms.
constexpr int MS_K = 32;

template <int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_modes_split(
    const float *W, int64_t n, int64_t P, int n_max, int kdim, const u32x4 *Bf, int rblocks, int r, float *out,
    int64_t ld) {
  constexpr int KS = MS_K / 16;
  constexpr int FR = KS * NB * 3;
  constexpr int NL = (FR + 3) / 4;
  __shared__ u32x4 sB[FR * 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m0 = (int64_t)blockIdx.x * 128 + wave * 32;
  const int64_t p = m0 / PANEL;
  const int rb0 = blockIdx.y * NB;
  const __amdgpu_buffer_rsrc_t rw =
      make_rsrc(W + (size_t)(p < P ? p : 0) * n_max * PANEL, p < P ? (unsigned)(kdim * PANEL * 4) : 0u);
  const unsigned woff = (unsigned)(((lane >> 5) * 8 * PANEL + (int)(m0 % PANEL) + (lane & 31)) * 4);
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(Bf, (unsigned)((kdim + MS_K - 1) / MS_K * KS * rblocks * 3 * 1024));
  f32x16 acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int t = 0; t < 16; ++t) acc[b][t] = 0.f;
  unsigned w[KS][8];
  u32x4 bn[NL];
  auto load_w = [&](int k0) {
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int m = 0; m < 8; ++m)
        w[s][m] = __builtin_amdgcn_raw_buffer_load_b32(rw, (int)woff, (k0 + 16 * s + m) * PANEL * 4, kTileLoad);
  };
  auto load_b = [&](int k0) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int f = wave + 4 * i;  // step f / (3 NB), block and piece f % (3 NB)
      if (f < FR)
        bn[i] = __builtin_amdgcn_raw_buffer_load_b128(
            rb, lane * 16, (((k0 / 16 + f / (3 * NB)) * rblocks + rb0) * 3 + f % (3 * NB)) * 1024, 0);
    }
  };
  load_b(0);
  load_w(0);
  for (int k0 = 0; k0 < kdim; k0 += MS_K) {
    if (k0) __syncthreads();
#pragma unroll
    for (int i = 0; i < NL; ++i)
      if (wave + 4 * i < FR) sB[(wave + 4 * i) * 64 + lane] = bn[i];
    // the three pieces of this stage's values, two columns to a register
    u32x4 w1[KS], w2[KS], w3[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const unsigned x0 = w[s][2 * q], x1 = w[s][2 * q + 1];
        const float f0 = __builtin_bit_cast(float, x0), f1 = __builtin_bit_cast(float, x1);
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const unsigned c1 = __builtin_bit_cast(unsigned, bf16x2{(__bf16)f0, (__bf16)f1});
        w1[s][q] = c1;
        const float r0 = f0 - __builtin_bit_cast(float, c1 << 16);
        const float r1 = f1 - __builtin_bit_cast(float, c1 & 0xffff0000u);
        const unsigned c2 = __builtin_bit_cast(unsigned, bf16x2{(__bf16)r0, (__bf16)r1});
        w2[s][q] = c2;
        const float t0 = r0 - __builtin_bit_cast(float, c2 << 16);
        const float t1 = r1 - __builtin_bit_cast(float, c2 & 0xffff0000u);
        w3[s][q] = __builtin_bit_cast(unsigned, bf16x2{(__bf16)t0, (__bf16)t1});
      }
    __syncthreads();
    if (k0 + MS_K < kdim) {
      load_b(k0 + MS_K);
      load_w(k0 + MS_K);
    }
    // a mode block at a time; the five small products of the stage are summed on
    // their own and added once
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      f32x16 small;
#pragma unroll
      for (int t = 0; t < 16; ++t) small[t] = 0.f;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const bf16x8 W1 = __builtin_bit_cast(bf16x8, w1[s]), W2 = __builtin_bit_cast(bf16x8, w2[s]),
                     W3 = __builtin_bit_cast(bf16x8, w3[s]);
        bf16x8 B;
        auto piece = [&](int c) { B = __builtin_bit_cast(bf16x8, sB[((s * NB + b) * 3 + c) * 64 + lane]); };
        auto term = [&](const bf16x8 &w) { small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(B, w, small, 0, 0, 0); };
        piece(2);
        term(W1);
        piece(1);
        term(W2);
        term(W1);
        piece(0);
        term(W3);
        term(W2);
        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(B, W1, acc[b], 0, 0, 0);
      }
#pragma unroll
      for (int t = 0; t < 16; ++t) acc[b][t] += small[t];
    }
  }
  // D[i][j]: j = lane % 32 (data row), i = 8 (t / 4) + 4 (lane / 32) + t % 4 (mode)
  const int64_t row = m0 + (lane & 31);
  if (row >= n) return;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const int mode = (rb0 + b) * 32 + 8 * (t >> 2) + 4 * (lane >> 5) + (t & 3);
      if (mode < r) out[(size_t)mode * ld + row] = acc[b][t];
    }
  }
}

// FP32-product kernel (FP32 basis, FP32 output, what modes_split_pays and
// modes_split_ok keep from k_modes_split): Phi^T = B^T W^T on 32x32x2 FP32 MFMA
// with FP32 accumulation.  Tile: 128 data rows (two panels) x 32*NB mode
// columns per workgroup; wavefront w owns data rows 32w..32w+31 and all NB
// 32-mode blocks, so for r <= 256 the basis is read exactly once.  k advances
// in chunks of 32 staged through LDS, the next chunk's global loads in flight
// in registers while the current one is multiplied: W as As[k][row] (rows
// contiguous, as in the panel layout), B as Bs[k][mode], both with row strides
// that put the two half-wavefronts of a fragment read 32 banks apart.  B
// arrives as FP32, k-major and zero-padded to whole chunks and mode blocks, so
// its loads need no masks.  Operands: A = B^T (lane l holds mode l%32,
// k-offset l/32), B = W^T (lane l holds data row l%32, k-offset l/32); the
// result D[i][j] has j = lane % 32, so each store instruction writes 32
// consecutive rows of one mode column.
constexpr int MT_ROWS = 128, MT_K = 32, MT_LDA = 160;

// 32-mode blocks per workgroup (at most 8): the blocks of r modes split evenly
// over the fewest workgroups
__host__ __device__ constexpr int mfma_nb(int r) {
  const int all = r <= 32 ? 1 : (r + 31) / 32, wgs = (all + 7) / 8;
  return (all + wgs - 1) / wgs;
}

int modes_kpad(int k) { return (k + MT_K - 1) / MT_K * MT_K; }
int modes_rpad(int r) {
  const int t = 32 * mfma_nb(r);
  return (r + t - 1) / t * t;
}

// mode blocks of 16 per workgroup of the FP64 kernel, and all of them (whole workgroups)
static int m64_mb(int r) {
  const int all = r <= 16 ? 1 : (r + 15) / 16, wgs = (all + M64_MB - 1) / M64_MB;
  return (all + wgs - 1) / wgs;
}
static int m64_blocks(int r) {
  const int mb = m64_mb(r), all = (r + 15) / 16;
  return (all + mb - 1) / mb * mb;
}

// Rule for the split products of an FP32 basis and output: from 2^31 multiply-adds
// on, the splitting launch (3 us) is less than they save (5e-15 s each against the
// FP32 units), and from kSplitCols basis columns on, where its error is no larger
// (k_modes_split; with up to 33 columns the FP32 products' may be smaller) and it
// is the faster one: 2^21 rows, us, split / FP32: 32 columns 132 / 125, 48 columns
// 204 / 254, 64 columns 259 / 310.
constexpr int kSplitCols = 48;
bool modes_split_pays(int64_t n, int k, int r) { return k >= kSplitCols && (double)n * k * r >= 0x1p31; }

// Where the FP32 coefficients lie that k_modes_split_coefs splits: behind the split
// ones.
size_t modes_split_bytes(int k, int r) { return (size_t)modes_kpad(k) * modes_rpad(r) * 6; }

// An upper bound of every path's packed size: splitting the blocks evenly over
// up to 2 (32-mode) or 4 (16-mode) workgroups adds at most 1 or 3 blocks.
size_t modes_coef_bytes(int n_max) {
  const size_t k = (size_t)modes_kpad(n_max);
  return std::max(k * ((n_max + 31) / 32 + 1) * 32 * (6 + 4), k * ((n_max + 15) / 16 + 3) * 16 * 8);
}

// The range in which three bf16 pieces carry an FP32 coefficient and the basis
// values beside it: a coefficient is a column's scale sigma (the stored column has
// norm 1 / sigma) times an entry of a unit vector, so a largest coefficient of at
// least 2^-60 keeps the values of its basis column below 2^60, far from where the
// rounding of w1 overflows; a column without a coefficient says nothing of its
// values.  Products outside go to the FP32 kernel.  (The last piece of a value
// below 2^-109 is under the smallest bf16: an error of 2^-134, in a column whose
// norm is at least 2^-60.)
bool modes_split_ok(const float *B, int k, int r, size_t ldp) {
  for (int l = 0; l < k; ++l) {
    float m = 0.f;
    for (int c = 0; c < r; ++c) {
      const float v = std::fabs(B[(size_t)l * ldp + c]);
      if (!(v <= 0x1p60f)) return false;  // also NaN
      m = std::max(m, v);
    }
    if (m < 0x1p-60f) return false;
  }
  return true;
}

int modes_path(bool tv_f64, bool out_f64) { return !tv_f64 && !out_f64 ? MODES_F32 : MODES_F64; }


void modes_pack(int path, const double *B, int k, int r, std::vector<char> &out) {
  if (path == MODES_F64) {
    out.resize((size_t)k * r * 8);
    double *o = reinterpret_cast<double *>(out.data());
    for (int c = 0; c < r; ++c)
      for (int l = 0; l < k; ++l) o[(size_t)l * r + c] = B[(size_t)c * k + l];
    return;
  }
  const int kp = modes_kpad(k), rp = modes_rpad(r);
  out.assign((size_t)kp * rp * 4, 0);
  float *o = reinterpret_cast<float *>(out.data());
  for (int c = 0; c < r; ++c)
    for (int l = 0; l < k; ++l) o[(size_t)l * rp + c] = (float)B[(size_t)c * k + l];
}

// The coefficients Bt (k-major, padded) as the operand fragments of k_modes_split:
// three bf16 pieces of each, to nearest even (finite, at most 2^60 in size).
__global__ __launch_bounds__(256) void k_modes_split_coefs(const float *Bt, int kp, int rp, uint16_t *o) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= kp * rp) return;
  const int l = e / rp, c = e - l * rp;
  float v = Bt[e];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    unsigned u = __builtin_bit_cast(unsigned, v);
    u = (u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u;
    o[((((size_t)(l / 16) * (rp / 32) + c / 32) * 3 + i) * 64 + (l % 16) / 8 * 32 + c % 32) * 8 + l % 8] =
        (uint16_t)(u >> 16);
    v -= __builtin_bit_cast(float, u);
  }
}

// Up to NB = 5 the registers fit three wavefronts per SIMD (three workgroups
// per CU), so one workgroup's staging and epilogue overlap the others' MFMA.
template <int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NB <= 5 ? 3 : 2))) void k_modes_mfma(const float *W, int64_t n, int64_t P, int n_max, int kdim,
                                                    const float *Bt, int rpad, int r, float *out, int64_t ld) {
  constexpr int LDB = 32 * NB + (NB % 2 == 0 ? 32 : 0);
  constexpr int GPR = 8 * NB;  // 16-byte groups per staged B row
  __shared__ float As[MT_K * MT_LDA];
  __shared__ float Bs[MT_K * LDB];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int64_t m0 = (int64_t)blockIdx.x * MT_ROWS;
  const int64_t p0 = m0 / PANEL;
  const int npan = (int)(P - p0 < 2 ? P - p0 : 2);
  const int n0 = blockIdx.y * 32 * NB;
  // This tile's (at most two) panels of W: rows of a missing second panel and
  // basis columns >= kdim read as 0.
  const unsigned pbytes = (unsigned)n_max * PANEL * 4;
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(W + (size_t)p0 * n_max * PANEL, npan * pbytes);
  f32x16 acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int t = 0; t < 16; ++t) acc[b][t] = 0.f;

  f32x4v ra[4], rb[NB];
  auto load_chunk = [&](int k0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = (tid + u * 256) * 4;  // first of 4 consecutive rows
      const int c = e / MT_ROWS, row = e % MT_ROWS;
      const unsigned off = k0 + c < kdim ? (row / PANEL) * pbytes + ((k0 + c) * PANEL + row % PANEL) * 4u : kOOR;
      ra[u] = __builtin_bit_cast(f32x4v, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)off, 0, kTileLoad));
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int e = tid + u * 256;
      rb[u] = *reinterpret_cast<const f32x4v *>(Bt + (size_t)(k0 + e / GPR) * rpad + n0 + (e % GPR) * 4);
    }
  };
  auto store_chunk = [&]() {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = (tid + u * 256) * 4;
      *reinterpret_cast<f32x4v *>(&As[(e / MT_ROWS) * MT_LDA + e % MT_ROWS]) = ra[u];
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int e = tid + u * 256;
      *reinterpret_cast<f32x4v *>(&Bs[(e / GPR) * LDB + (e % GPR) * 4]) = rb[u];
    }
  };
  // operand fragments of k-step kk
  float wf[2], bf[2][NB];
  auto read_frag = [&](int kk, float &w, float (&b)[NB]) {
    const int kr = kk + (lane >> 5);
    w = As[kr * MT_LDA + wave * 32 + (lane & 31)];
#pragma unroll
    for (int i = 0; i < NB; ++i) b[i] = Bs[kr * LDB + i * 32 + (lane & 31)];
  };

  load_chunk(0);
  for (int k0 = 0; k0 < kdim; k0 += MT_K) {
    store_chunk();
    __syncthreads();
    if (k0 + MT_K < kdim) load_chunk(k0 + MT_K);
    // the fragments of step kk + 2 are read while step kk's products run
    read_frag(0, wf[0], bf[0]);
#pragma unroll
    for (int kk = 0; kk < MT_K; kk += 2) {
      const int cur = (kk / 2) & 1;
      if (kk + 2 < MT_K) read_frag(kk + 2, wf[cur ^ 1], bf[cur ^ 1]);
      // keep the scheduler from sinking those reads next to their use
      __builtin_amdgcn_sched_barrier(0);
      if (k0 + kk < kdim) {  // ragged last chunk (uniform branch)
#pragma unroll
        for (int i = 0; i < NB; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(bf[cur][i], wf[cur], acc[i], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
  }
  // D[i][j]: j = lane % 32 (data row), i = 8 (t / 4) + 4 (lane / 32) + t % 4 (mode)
  const int64_t row = m0 + wave * 32 + (lane & 31);
  if (row >= n) return;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const int mode = n0 + b * 32 + 8 * (t >> 2) + 4 * (lane >> 5) + (t & 3);
      if (mode < r) out[(size_t)mode * ld + row] = acc[b][t];
    }
  }
}

template <int NB>
static void launch_mfma_nb(const float *W, int64_t n, int n_max, int k, const float *Bt, int r, float *out,
                           int64_t ld, hipStream_t s) {
  const int64_t P = (n + PANEL - 1) / PANEL;
  dim3 g((unsigned)((n + MT_ROWS - 1) / MT_ROWS), (unsigned)((r + 32 * NB - 1) / (32 * NB)));
  hipLaunchKernelGGL((k_modes_mfma<NB>), g, dim3(256), 0, s, W, n, P, n_max, k, Bt, modes_rpad(r), r, out, ld);
}

static void launch_mfma(const float *W, int64_t n, int n_max, int k, const float *Bt, int r, float *out,
                        int64_t ld, hipStream_t s) {
  switch (mfma_nb(r)) {
    case 1: launch_mfma_nb<1>(W, n, n_max, k, Bt, r, out, ld, s); break;
    case 2: launch_mfma_nb<2>(W, n, n_max, k, Bt, r, out, ld, s); break;
    case 3: launch_mfma_nb<3>(W, n, n_max, k, Bt, r, out, ld, s); break;
    case 4: launch_mfma_nb<4>(W, n, n_max, k, Bt, r, out, ld, s); break;
    case 5: launch_mfma_nb<5>(W, n, n_max, k, Bt, r, out, ld, s); break;
    case 6: launch_mfma_nb<6>(W, n, n_max, k, Bt, r, out, ld, s); break;
    case 7: launch_mfma_nb<7>(W, n, n_max, k, Bt, r, out, ld, s); break;
    default: launch_mfma_nb<8>(W, n, n_max, k, Bt, r, out, ld, s); break;
  }
}

template <int NB>
static void launch_split_nb(const float *W, int64_t n, int n_max, int k, const u32x4 *Bf, int r, float *out, int64_t ld,
                            hipStream_t s) {
  const int rb = modes_rpad(r) / 32;
  dim3 g((unsigned)((n + 127) / 128), (unsigned)(rb / NB));
  hipLaunchKernelGGL((k_modes_split<NB>), g, dim3(256), 0, s, W, n, (n + PANEL - 1) / PANEL, n_max, k, Bf, rb, r, out,
                     ld);
}

static void launch_split(const float *W, int64_t n, int n_max, int k, const u32x4 *Bf, int r, float *out, int64_t ld,
                         hipStream_t s) {
  switch (mfma_nb(r)) {
    case 1: launch_split_nb<1>(W, n, n_max, k, Bf, r, out, ld, s); break;
    case 2: launch_split_nb<2>(W, n, n_max, k, Bf, r, out, ld, s); break;
    case 3: launch_split_nb<3>(W, n, n_max, k, Bf, r, out, ld, s); break;
    case 4: launch_split_nb<4>(W, n, n_max, k, Bf, r, out, ld, s); break;
    case 5: launch_split_nb<5>(W, n, n_max, k, Bf, r, out, ld, s); break;
    case 6: launch_split_nb<6>(W, n, n_max, k, Bf, r, out, ld, s); break;
    case 7: launch_split_nb<7>(W, n, n_max, k, Bf, r, out, ld, s); break;
    default: launch_split_nb<8>(W, n, n_max, k, Bf, r, out, ld, s); break;
  }
}

template <typename TV, typename TO, int MB>
static void launch_m64_mb(const TV *W, int64_t n, int n_max, int k, const double *Bf, int r, TO *out, int64_t ld,
                          hipStream_t s) {
  const int rb = m64_blocks(r);
  dim3 g((unsigned)((n + 127) / 128), (unsigned)(rb / MB));
  hipLaunchKernelGGL((k_modes_mfma64<TV, TO, MB>), g, dim3(256), 0, s, W, n, (n + PANEL - 1) / PANEL, n_max, k, Bf, r, out,
                     ld);
}

template <typename TV, typename TO>
static void launch_m64(const void *W, int64_t n, int n_max, int k, const double *Bf, int r, void *out, int64_t ld,
                       hipStream_t s) {
  const TV *w = (const TV *)W;
  TO *o = (TO *)out;
  // few rows: fewer mode blocks a workgroup rather than idle CUs
  int mb = m64_mb(r);
  while (mb > 1 && (n + 127) / 128 * (m64_blocks(r) / mb) < 256) {
    int d = mb - 1;
    while (mb % d) --d;
    mb = d;
  }
  switch (mb) {
    case 1: launch_m64_mb<TV, TO, 1>(w, n, n_max, k, Bf, r, o, ld, s); break;
    case 2: launch_m64_mb<TV, TO, 2>(w, n, n_max, k, Bf, r, o, ld, s); break;
    case 3: launch_m64_mb<TV, TO, 3>(w, n, n_max, k, Bf, r, o, ld, s); break;
    case 4: launch_m64_mb<TV, TO, 4>(w, n, n_max, k, Bf, r, o, ld, s); break;
    case 5: launch_m64_mb<TV, TO, 5>(w, n, n_max, k, Bf, r, o, ld, s); break;
    case 6: launch_m64_mb<TV, TO, 6>(w, n, n_max, k, Bf, r, o, ld, s); break;
    case 7: launch_m64_mb<TV, TO, 7>(w, n, n_max, k, Bf, r, o, ld, s); break;
    default: launch_m64_mb<TV, TO, 8>(w, n, n_max, k, Bf, r, o, ld, s); break;
  }
}

hipError_t launch_modes_gemm(int path, bool tv_f64, const void *W, int64_t n, int n_max, int k, const void *Bv, int r,
                             void *out, int64_t ld, bool out_f64, hipStream_t s) {
  if (r <= 0 || k <= 0) return hipSuccess;
  if (k > 512 || k > n_max) return hipErrorInvalidValue;
  if (path == MODES_SPLIT && !tv_f64 && !out_f64) {
    const int kp = modes_kpad(k), rp = modes_rpad(r);
    char *b = static_cast<char *>(const_cast<void *>(Bv));
    hipLaunchKernelGGL(k_modes_split_coefs, dim3((kp * rp + 255) / 256), dim3(256), 0, s,
                       (const float *)(b + modes_split_bytes(k, r)), kp, rp, (uint16_t *)b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    launch_split((const float *)W, n, n_max, k, (const u32x4 *)Bv, r, (float *)out, ld, s);
  } else if (path == MODES_F32 && !tv_f64 && !out_f64)
    launch_mfma((const float *)W, n, n_max, k, (const float *)Bv, r, (float *)out, ld, s);
  else if (path != MODES_F64)
    return hipErrorInvalidValue;
  else if (tv_f64 && out_f64)
    launch_m64<double, double>(W, n, n_max, k, (const double *)Bv, r, out, ld, s);
  else if (tv_f64)
    launch_m64<double, float>(W, n, n_max, k, (const double *)Bv, r, out, ld, s);
  else if (out_f64)
    launch_m64<float, double>(W, n, n_max, k, (const double *)Bv, r, out, ld, s);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace foa
