// Matrices whose short side m' is at most NS_SMALL_MAX (32): Newton-Schulz in
// the Gram space, in float64.
//
// The bf16 matrix-core path would pad such a matrix to a whole tile, and with
// few singular values its rounding is not averaged away: the quintic is still
// far from converged on the small ones and magnifies the rounding of X there.
// Every B_k = a I + b A_k + c A_k^2 is a polynomial in A_0 = X_0 X_0^T, so
//     A_{k+1} = B_k A_k B_k,   O = (B_{s-1} ... B_0) X_0,
// and X is read twice, once for A_0 and once for the product with P = B_{s-1}
// ... B_0.  That holds for a bounded number of iterations only: rounding moves
// the eigenvalues of A_0 by about 1e-16 of the largest, either way, and the error
// grows by a^2 = 12 per iteration.  Where X has a zero singular value (a gradient
// of low rank) A's eigenvalue can come out negative, and then nothing bounds it:
// a + b x + c x^2 grows with |x| (16 x 1024 of rank 1: NaN at 20 iterations).  So
// after SmallArgs::span iterations (small_span: 8 with the default quintic, the
// error then 4e-8 at most) X becomes P X, in float32, A is formed from it anew,
// positive semidefinite by construction, and P starts over.  Up to span
// iterations, X is read twice.
// Products run on v_mfma_f64_16x16x4 (lane l holds A(l % 16, l / 16),
// B(l / 16, l % 16); result register r holds C(l / 16 + 4 r, l % 16)); only the
// final O is rounded to bf16.
//
// Two routes:
//   whole step   a matrix of at most TINY_ELEMS elements (of long ones only where
//                there are many, choose_whole_steps) takes its whole step
//                in one workgroup (tiny_step_kernel): one launch for all such
//                matrices of a plan, in place of 21.  What bounds it is the
//                chain of its phases, and for the larger ones what one CU can
//                read.
//   three launches   larger ones take the plan's elementwise passes, and here
//                a Gram over column chunks, one workgroup per matrix for the
//                iteration, and the product with P over column chunks.
// Measured (us per step): one 5 x 5 matrix 108 -> 16; 96 matrices of rank 16
// (16 x 1024, 1024 x 16, 3072 x 16) 580 -> 76, of which the GPU 65.
#include <type_traits>

#include "malt_internal.h"

namespace malt {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float sm_f32x4 __attribute__((ext_vector_type(4)));

constexpr int SM_M = NS_SMALL_MAX;          // 32
constexpr int SM_LD = SM_M + 1;             // row pitch of an m' x m' matrix in LDS (doubles)
constexpr int SM_PITCH = 64 + 1;            // row pitch of a wave's 64 staged columns (floats)
constexpr int SM_TALL = SM_M + 1;           // pitch of the same columns as rows of a tall W
constexpr int SM_WAVE = 64 * SM_TALL + 1;   // one wave's staging area (floats)
static_assert(SM_M * SM_PITCH <= SM_WAVE, "columns staged by row");

// Blocks of 16 rows, and of 16 x 16 upper blocks, of m' <= MC.
template <int MC>
struct SmDim {
  static constexpr int NB = MC > 16 ? 2 : 1;
  static constexpr int NBLK = NB * (NB + 1) / 2;
};

// The iteration's matrices (five of them), and what shares their memory.
struct SmCore {
  double A[SM_M * SM_LD], B[SM_M * SM_LD], T[SM_M * SM_LD], P[2][SM_M * SM_LD];
};

__device__ __forceinline__ f64x4 sm_zero() { return f64x4{0.0, 0.0, 0.0, 0.0}; }

// A wave's 64 columns (one per lane, rows >= MC absent) into its staging rows.
template <int MC>
__device__ __forceinline__ void sm_stage(float* buf, const float (&x)[MC], int lane) {
#pragma unroll
  for (int i = 0; i < MC; ++i) buf[i * SM_PITCH + lane] = x[i];
}

// Element (row, col) of the staged columns, 0 past MC rows.
template <int MC>
__device__ __forceinline__ double sm_at(const float* buf, int row, int col) {
  return MC >= 16 || row < MC ? (double)buf[row * SM_PITCH + col] : 0.0;
}

// acc += X X^T over the staged columns, upper 16 x 16 blocks (0,0), (0,1), (1,1).
template <int MC>
__device__ __forceinline__ void sm_gram(const float* buf, f64x4 (&acc)[SmDim<MC>::NBLK], int lane) {
#pragma unroll 4
  for (int k = 0; k < 16; ++k) {
    const int col = 4 * k + (lane >> 4);
    const double a0 = sm_at<MC>(buf, lane & 15, col);
    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, a0, acc[0], 0, 0, 0);
    if constexpr (SmDim<MC>::NB == 2) {
      const double a1 = sm_at<MC>(buf, 16 + (lane & 15), col);
      acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, a1, acc[1], 0, 0, 0);
      acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, a1, acc[2], 0, 0, 0);
    }
  }
}

// Block (bi, bj) of S1 S2, K = 16 NB.
__device__ __forceinline__ f64x4 sm_mul(const double* S1, const double* S2, int bi, int bj, int NB, int lane) {
  f64x4 c = sm_zero();
  for (int k = 0; k < 4 * NB; ++k) {
    const int kk = 4 * k + (lane >> 4);
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(S1[(16 * bi + (lane & 15)) * SM_LD + kk],
                                             S2[kk * SM_LD + 16 * bj + (lane & 15)], c, 0, 0, 0);
  }
  return c;
}

__device__ __forceinline__ void sm_put(double* D, const f64x4& c, int bi, int bj, int lane) {
#pragma unroll
  for (int r = 0; r < 4; ++r) D[(16 * bi + (lane >> 4) + 4 * r) * SM_LD + 16 * bj + (lane & 15)] = c[r];
}

// `steps` iterations on s.A (16 NB rows and columns); returns P.  Every thread
// of the workgroup of NWAVES waves calls it; it ends with a barrier.
template <int NWAVES>
__device__ __forceinline__ const double* sm_iterate(SmCore& s, int NB, const SmallArgs& ns, int steps) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nblk = NB * NB;
  int cur = 0;
  for (int it = 0; it < steps; ++it) {
    for (int w = wave; w < nblk; w += NWAVES) {   // B = a I + b A + c A A
      const int bi = w / NB, bj = w % NB;
      f64x4 v = sm_mul(s.A, s.A, bi, bj, NB, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * bi + (lane >> 4) + 4 * r, j = 16 * bj + (lane & 15);
        v[r] = ns.b * s.A[i * SM_LD + j] + ns.c * v[r] + (i == j ? ns.a : 0.0);
      }
      sm_put(s.B, v, bi, bj, lane);
      if (it == 0) sm_put(s.P[0], v, bi, bj, lane);
    }
    __syncthreads();
    if (it > 0) {   // P <- B P
      for (int w = wave; w < nblk; w += NWAVES)
        sm_put(s.P[cur ^ 1], sm_mul(s.B, s.P[cur], w / NB, w % NB, NB, lane), w / NB, w % NB, lane);
      cur ^= 1;
    }
    if (it + 1 < steps) {   // A <- B A B, on the waves the product above left free first
      for (int w = (wave + NWAVES - (it > 0 ? nblk % NWAVES : 0)) % NWAVES; w < nblk; w += NWAVES)
        sm_put(s.T, sm_mul(s.B, s.A, w / NB, w % NB, NB, lane), w / NB, w % NB, lane);
      __syncthreads();
      for (int w = wave; w < nblk; w += NWAVES)
        sm_put(s.A, sm_mul(s.T, s.B, w / NB, w % NB, NB, lane), w / NB, w % NB, lane);
    }
    __syncthreads();
  }
  return s.P[cur];
}

// The product with P for a wave's 64 columns: x becomes P x, staged in buf.
template <int MC>
__device__ __forceinline__ void sm_product(float* buf, const double (&pa)[SmDim<MC>::NB][MC > 16 ? 8 : 4], int lane,
                                           const float (&x)[MC]) {
  constexpr int NB = SmDim<MC>::NB, KS = MC > 16 ? 8 : 4;
  sm_stage<MC>(buf, x, lane);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int cl = 16 * g + (lane & 15);
    f64x4 y[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) y[b] = sm_zero();
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const double xb = sm_at<MC>(buf, 4 * k + (lane >> 4), cl);
#pragma unroll
      for (int b = 0; b < NB; ++b) y[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(pa[b][k], xb, y[b], 0, 0, 0);
    }
    // Back in place: this group's columns have been read.
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * b + (lane >> 4) + 4 * r;
        if (MC >= 16 || i < MC) buf[i * SM_PITCH + cl] = (float)y[b][r];
      }
  }
}

// x <- P x (0 past mc rows and past the matrix); in: this lane's column lies in
// the matrix.
template <int MC>
__device__ __forceinline__ void sm_advance(float* buf, const double (&pa)[SmDim<MC>::NB][MC > 16 ? 8 : 4], bool in,
                                           int mc, int lane, float (&x)[MC]) {
  sm_product<MC>(buf, pa, lane, x);
#pragma unroll
  for (int i = 0; i < MC; ++i) x[i] = in && i < mc ? buf[i * SM_PITCH + lane] : 0.f;
}

// The last product: x becomes O = P x rounded to bf16 (0 past mc rows and past
// the matrix), (o2, d2) gain its sums of o^2 and (Lm o Ln)^2.  rowf: canonical
// row factors (0 past mc); cf: this lane's column factor.
template <int MC>
__device__ __forceinline__ void sm_apply(float* buf, const double (&pa)[SmDim<MC>::NB][MC > 16 ? 8 : 4],
                                         const float* rowf, float cf, bool in, int mc, int lane, float (&x)[MC],
                                         double& o2, double& d2) {
  sm_product<MC>(buf, pa, lane, x);
  float so = 0.f, sd = 0.f;
#pragma unroll
  for (int i = 0; i < MC; ++i) {
    const float o = in && i < mc ? bf16_lo(pack_bf16x2(buf[i * SM_PITCH + lane], 0.f)) : 0.f;
    const float lm = rowf[i];
    x[i] = o;
    so += o * o;
    sd += lm * lm * (o * o);
  }
  o2 += (double)so;
  d2 += (double)(cf * cf * sd);
}

// The iterate between two Grams: canonical float32 rows < mc of pitch np, in the
// bf16 iterate buffer that the final O does not take (mc <= 32 rows of 4 bytes in
// NS_TILE of 2).
__device__ __forceinline__ MALT_GLOBAL float* sm_iterate_x(const MatDesc& d, int o_parity) {
  return reinterpret_cast<MALT_GLOBAL float*>(gptr(d.X[o_parity ^ 1]));
}
static_assert(SM_M * sizeof(float) <= NS_TILE * sizeof(bf16_t), "the float32 iterate fits a bf16 iterate buffer");

// Column c of the canonical O, already rounded (rows < mc).
template <int MC>
__device__ __forceinline__ void sm_store_o(MALT_GLOBAL bf16_t* O, int np, int mc, int c, bool in, const float (&x)[MC]) {
  if (!in) return;
#pragma unroll
  for (int i = 0; i < MC; ++i)
    if (i < mc) O[(size_t)i * np + c] = (bf16_t)(__float_as_uint(x[i]) >> 16);
}

// MFMA operand of P scaled by sigma: pa[b][k] = sigma P(16 b + l % 16, 4 k + l / 16).
template <int MC>
__device__ __forceinline__ void sm_operand(const double* P, double sigma, double (&pa)[SmDim<MC>::NB][MC > 16 ? 8 : 4],
                                           int lane) {
#pragma unroll
  for (int b = 0; b < SmDim<MC>::NB; ++b)
#pragma unroll
    for (int k = 0; k < (MC > 16 ? 8 : 4); ++k)
      pa[b][k] = sigma * P[(16 * b + (lane & 15)) * SM_LD + 4 * k + (lane >> 4)];
}

__device__ __forceinline__ double sm_wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Fixed-order sums of (v0, v1) over the workgroup, given to every thread.
template <int NWAVES>
__device__ __forceinline__ void sm_block_sum(double& v0, double& v1, double (*red)[2]) {
  v0 = sm_wave_sum(v0);
  v1 = sm_wave_sum(v1);
  __syncthreads();   // red is free
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6][0] = v0;
    red[threadIdx.x >> 6][1] = v1;
  }
  __syncthreads();
  v0 = v1 = 0.0;
#pragma unroll
  for (int w = 0; w < NWAVES; ++w) {
    v0 += red[w][0];
    v1 += red[w][1];
  }
}

// (v + eps)^(-1/8): three square roots and a quotient, each correctly rounded.
__device__ __forceinline__ float sm_inv_eighth(double v) { return (float)(1.0 / sqrt(sqrt(sqrt(v)))); }

// ---------------------------------------------------------------------------
// The whole step of one matrix.
// ---------------------------------------------------------------------------
constexpr int TY_NW = TINY_THREADS / 64;

struct TinyLds {
  union {
    float stage[TY_NW * SM_WAVE];
    struct {
      double red[TY_NW][3][64 * 4];   // Gram blocks of the waves
      SmCore core;
    };
  };
  float rowf[SM_M];
  double rows[TY_NW][SM_M];
  double red2[TY_NW][2];
};
static_assert(sizeof(TinyLds) <= 160 * 1024, "LDS of a whole-step workgroup");

// The columns of a wave in memory: canonical columns c0 .. c0 + 63 of a W-shaped
// array.  Of a wide matrix (canonical (i, c) = W(i, c)) lane l takes column c0 +
// l row by row.  Of a tall one (W(c, i), n = mc columns) the 64 columns are 64 n
// consecutive floats: they are read in that order, so that every access is
// whole cache lines, and change places through the wave's staging area.
struct TinyCols {
  bool tall;
  int n, mc, nc, c0, lane;
  uint32_t inv;   // floor(e / n) = (e * inv) >> 16 for e < 64 n <= 2048
};

// FULL: m' = MC rows and whole rounds of 64 columns, nothing to test.  Otherwise
// loads stay unconditional, at clamped positions (behind a bounds branch each,
// the compiler waits for one before it issues the next), and tiny_mask zeroes
// what lies past the matrix.
template <int MC, bool FULL>
__device__ __forceinline__ void tiny_load(const MALT_GLOBAL float* p, const TinyCols& t, float (&x)[MC]) {
  if constexpr (FULL) {
    if (!t.tall) {
#pragma unroll
      for (int i = 0; i < MC; ++i) x[i] = p[i * t.n + (t.c0 + t.lane)];
    } else {
#pragma unroll
      for (int i = 0; i < MC; ++i) x[i] = p[t.c0 * MC + t.lane + i * 64];
    }
  } else {
    const int c = t.c0 + t.lane, total = (t.nc - t.c0) * t.n;
    const int cc = min(c, t.nc - 1), base = t.c0 * t.n;
#pragma unroll
    for (int i = 0; i < MC; ++i)
      x[i] = p[t.tall ? base + min(i * 64 + t.lane, total - 1) : min(i, t.mc - 1) * t.n + cc];
  }
}

template <int MC, bool FULL>
__device__ __forceinline__ void tiny_mask(const TinyCols& t, float (&x)[MC]) {
  if constexpr (FULL) return;
  const int c = t.c0 + t.lane, total = (t.nc - t.c0) * t.n;
#pragma unroll
  for (int i = 0; i < MC; ++i) {
    const bool in = i < t.mc && (t.tall ? i * 64 + t.lane < total : c < t.nc);
    x[i] = in ? x[i] : 0.f;
  }
}

// Place in the staging area of the i-th value a lane reads of a tall matrix;
// the spare element past the columns where there is none.
template <int MC, bool FULL>
__device__ __forceinline__ int tiny_place(const TinyCols& t, int i) {
  const uint32_t e = i * 64 + t.lane;
  if constexpr (FULL) return (e / MC) * SM_TALL + e % MC;
  const uint32_t c = (e * t.inv) >> 16;
  return i < t.mc ? c * SM_TALL + (e - c * t.n) : 64 * SM_TALL;
}

// What tiny_load read, as this lane's column.
template <int MC, bool FULL>
__device__ __forceinline__ void tiny_own(float* buf, const TinyCols& t, float (&x)[MC]) {
  if (!t.tall) return;
#pragma unroll
  for (int i = 0; i < MC; ++i) buf[tiny_place<MC, FULL>(t, i)] = x[i];
#pragma unroll
  for (int i = 0; i < MC; ++i) x[i] = FULL || i < t.mc ? buf[t.lane * SM_TALL + i] : 0.f;
}

// The opposite: this lane's column, in the order of memory.
template <int MC, bool FULL>
__device__ __forceinline__ void tiny_give(float* buf, const TinyCols& t, float (&x)[MC]) {
  if (!t.tall) return;
#pragma unroll
  for (int i = 0; i < MC; ++i) buf[t.lane * SM_TALL + i] = x[i];
#pragma unroll
  for (int i = 0; i < MC; ++i) x[i] = buf[tiny_place<MC, FULL>(t, i)];
}

// Stores values in the order tiny_load reads them.
template <int MC, bool FULL>
__device__ __forceinline__ void tiny_put(MALT_GLOBAL float* p, const TinyCols& t, const float (&x)[MC]) {
  if constexpr (FULL) {
    if (!t.tall) {
#pragma unroll
      for (int i = 0; i < MC; ++i) p[i * t.n + (t.c0 + t.lane)] = x[i];
    } else {
#pragma unroll
      for (int i = 0; i < MC; ++i) p[t.c0 * MC + t.lane + i * 64] = x[i];
    }
  } else {
    const int c = t.c0 + t.lane, total = (t.nc - t.c0) * t.n;
#pragma unroll
    for (int i = 0; i < MC; ++i) {
      const bool in = i < t.mc && (t.tall ? i * 64 + t.lane < total : c < t.nc);
      if (in) p[t.tall ? t.c0 * t.n + i * 64 + t.lane : i * t.n + c] = x[i];
    }
  }
}

// Canonical bf16 column c of X0 or O.
template <int MC, bool FULL>
__device__ __forceinline__ void tiny_put16(MALT_GLOBAL bf16_t* p, const TinyCols& t, int np, const float (&x)[MC]) {
  const int c = t.c0 + t.lane;
#pragma unroll
  for (int i = 0; i < MC; ++i) {
    const bf16_t h = (bf16_t)(pack_bf16x2(x[i], 0.f) & 0xffffu);
    if (FULL || (i < t.mc && c < t.nc)) p[i * np + c] = h;
  }
}

// This lane's column of the float32 iterate.
template <int MC>
__device__ __forceinline__ void tiny_load_x(const MALT_GLOBAL float* X, const TinyCols& t, int np, float (&x)[MC]) {
  const int c = t.c0 + t.lane;
#pragma unroll
  for (int i = 0; i < MC; ++i) {
    const float y = X[(size_t)min(i, t.mc - 1) * np + min(c, t.nc - 1)];
    x[i] = i < t.mc && c < t.nc ? y : 0.f;
  }
}

// One exchange of halves: 2 N entries per lane in, the sums of N of them with the
// lane `off` away out (the upper half where lane & off).
template <int N, class F>
__device__ __forceinline__ void tiny_halve(F* v, int lane, int off) {
  const bool up = lane & off;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const F send = up ? v[k] : v[k + N], keep = up ? v[k + N] : v[k];
    v[k] = keep + __shfl_xor(send, off, 64);
  }
}

// Adds x over the wave's lanes; afterwards lane l holds the sum of entry
// l >> (6 - log2 N) (halves exchanged: N - 1 shuffles, not 6 N).  The first two
// exchanges in F, the others in float64.
template <int N, class F>
__device__ __forceinline__ double tiny_reduce(F (&x)[N], int lane) {
  tiny_halve<N / 2>(x, lane, 32);
  tiny_halve<N / 4>(x, lane, 16);
  double v[N / 4];
#pragma unroll
  for (int k = 0; k < N / 4; ++k) v[k] = (double)x[k];
  int off = 8;
  if constexpr (N >= 8) { tiny_halve<N / 8>(v, lane, off); off >>= 1; }
  if constexpr (N >= 16) { tiny_halve<N / 16>(v, lane, off); off >>= 1; }
  if constexpr (N >= 32) { tiny_halve<N / 32>(v, lane, off); off >>= 1; }
  double s = v[0];
  for (; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  return s;
}

// m' <= MC. Four passes over the matrix's columns, 64 per wave and round: the
// momentum and sums, L M R with its norms and Gram, the product with P, the
// update of W. The rounds are loops, not unrolled: with L M R in registers
// between the passes, every round unrolled, the code ran to hundreds of
// kilobytes executed once, and the step of a 3072 x 16 matrix took 98 us.  A
// round's loads are issued before the previous round is worked on, so that
// waiting for them does not wait for that round's stores.  us of a step: 16 x
// 1024 27 (55 with a bounds branch per row, 39 with clamped positions only),
// 3072 x 16 62, 32 x 1024 63, 8 x 4096 54.
// LONG: also more than ns.span iterations (see the top of this file), and steps
// that leave W to tiny_write_kernel.
template <bool MALTER, int MC, bool FULL, bool LONG>
__device__ __forceinline__ void tiny_step(const SmallArgs& ns, int mat, TinyLds& S) {
  constexpr int NB = SmDim<MC>::NB;
  constexpr int LOG = MC == 32 ? 5 : MC == 16 ? 4 : 3;
  const EwArgs& a = ns.e;
  const MatDesc& d = a.desc[mat];
  const EwView v = ew_view(a, mat);
  const int mc = d.mc, nc = d.nc, np = v.np;
  const bool tall = v.tall != 0;
  MALT_GLOBAL double* const scal = gptr(d.scal);
  MALT_GLOBAL float* const nu_p = gptr(d.nu);
  MALT_GLOBAL bf16_t* const O = gptr(d.X[a.o_parity]);
  // Column and row factors of the canonical orientation, and their EMAs.
  MALT_GLOBAL float* const cema = gptr(tall ? d.l : d.r);
  MALT_GLOBAL float* const cinv = gptr(tall ? d.Lv : d.Rv);
  MALT_GLOBAL float* const rema = gptr(tall ? d.r : d.l);
  MALT_GLOBAL float* const rinv = gptr(tall ? d.Rv : d.Lv);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float* const buf = S.stage + wave * SM_WAVE;
  TinyCols t{tall, v.n, mc, nc, 0, lane, 65536u / (uint32_t)v.n + 1u};

  auto next = [](TinyCols q) {
    q.c0 += TINY_THREADS;
    return q;
  };
  auto copy = [](float (&to)[MC], const float (&from)[MC]) {
#pragma unroll
    for (int i = 0; i < MC; ++i) to[i] = from[i];
  };

  // Momentum, and the row and column sums of G^2.  Those along the long side (up
  // to 65536 terms) are float64; past 16 rows, whose at most 3855 columns are
  // eight terms a lane, from float32 sums of four lanes (in float64 throughout the
  // 64 registers more cost 32 x 2048 100 -> 118 us).  Those over a column's rows
  // are float32.
  {
    typedef typename std::conditional<(MC > 16), float, double>::type sum_t;
    static_assert(TINY_ELEMS / 17 <= 8 * TINY_THREADS, "few float32 terms a lane");
    sum_t rs[MC];
#pragma unroll
    for (int i = 0; i < MC; ++i) rs[i] = 0;
    float gn[MC], mn[MC], en;
    auto fetch = [&](const TinyCols& t) {
      tiny_load<MC, FULL>(v.G, t, gn);
      tiny_load<MC, FULL>(v.M, t, mn);
      en = cema[min(t.c0 + lane, nc - 1)];
    };
    t.c0 = wave * 64;
    if (t.c0 < nc) fetch(t);
#pragma unroll 1
    for (; t.c0 < nc; t.c0 += TINY_THREADS) {
      const int c = t.c0 + lane;
      float g[MC], m[MC];
      copy(g, gn);
      copy(m, mn);
      const double old = (double)en;
      if (const TinyCols nx = next(t); nx.c0 < nc) fetch(nx);
      tiny_mask<MC, FULL>(t, g);
#pragma unroll
      for (int i = 0; i < MC; ++i) {
        m[i] = a.mu1 * m[i] + a.one_minus_mu1 * g[i];
        g[i] *= g[i];
      }
      tiny_put<MC, FULL>(v.M, t, m);
      tiny_own<MC, FULL>(buf, t, g);
      float cs = 0.f;
#pragma unroll
      for (int i = 0; i < MC; ++i) {
        cs += g[i];
        rs[i] += (sum_t)g[i];
      }
      if (FULL || c < nc) {
        const double e = a.mu2 * old + (1.0 - a.mu2) * (double)cs;
        cema[c] = (float)e;
        cinv[c] = a.identity ? 1.f : sm_inv_eighth(e + a.eps);
      }
    }
    const double s = tiny_reduce<MC>(rs, lane);
    if ((lane & ((64 >> LOG) - 1)) == 0) S.rows[wave][lane >> (6 - LOG)] = s;
  }
  __syncthreads();
  if (tid < SM_M) {
    float f = 0.f;
    if (tid < mc) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < TY_NW; ++w) s += S.rows[w][tid];
      const double e = a.mu2 * (double)rema[tid] + (1.0 - a.mu2) * s;
      rema[tid] = (float)e;
      f = a.identity ? 1.f : sm_inv_eighth(e + a.eps);
      rinv[tid] = f;
    }
    S.rowf[tid] = f;
  }
  __syncthreads();

  // Column c of L M R (or L G R) from M (G), in W's order of the two products.
  auto scale = [&](float (&x)[MC], float cf) {
#pragma unroll
    for (int i = 0; i < MC; ++i) x[i] = tall ? cf * x[i] * S.rowf[i] : S.rowf[i] * x[i] * cf;
  };

  // L M R (X0 before its normalisation), its Gram and norm, MALTER's ||L G R||.
  double s2 = 0.0, q2 = 0.0;
  f64x4 acc[SmDim<MC>::NBLK];
#pragma unroll
  for (int b = 0; b < SmDim<MC>::NBLK; ++b) acc[b] = sm_zero();
  float xn[MC], gn[MC], cn;
  auto fetch = [&](const MALT_GLOBAL float* p, const TinyCols& t) {
    tiny_load<MC, FULL>(p, t, xn);
    cn = cinv[min(t.c0 + lane, nc - 1)];
  };
  t.c0 = wave * 64;
  if (t.c0 < nc) {
    fetch(v.M, t);
    if constexpr (MALTER) tiny_load<MC, FULL>(v.G, t, gn);
  }
#pragma unroll 1
  for (; t.c0 < nc; t.c0 += TINY_THREADS) {
    const int c = t.c0 + lane;
    float x[MC], g[MC];
    copy(x, xn);
    if constexpr (MALTER) copy(g, gn);
    const float cf = FULL || c < nc ? cn : 0.f;
    if (const TinyCols nx = next(t); nx.c0 < nc) {
      fetch(v.M, nx);
      if constexpr (MALTER) tiny_load<MC, FULL>(v.G, nx, gn);
    }
    tiny_mask<MC, FULL>(t, x);
    tiny_own<MC, FULL>(buf, t, x);
    scale(x, cf);
    float sx = 0.f, sg = 0.f;
#pragma unroll
    for (int i = 0; i < MC; ++i) sx += x[i] * x[i];
    if constexpr (MALTER) {
      tiny_mask<MC, FULL>(t, g);
      tiny_own<MC, FULL>(buf, t, g);
      scale(g, cf);
#pragma unroll
      for (int i = 0; i < MC; ++i) sg += g[i] * g[i];
    }
    s2 += (double)sx;
    q2 += (double)sg;
    tiny_put16<MC, FULL>(v.X0, t, np, x);
    sm_stage<MC>(buf, x, lane);
    sm_gram<MC>(buf, acc, lane);
  }
  sm_block_sum<TY_NW>(s2, q2, S.red2);   // its barriers also free the staging rows for the blocks
  const double s = sqrt(s2), sigma = 1.0 / (s + a.ns_eps);
  double nu = 0.0, alpha = 1.0;
  if constexpr (MALTER) {
    nu = a.mu2 * (double)nu_p[0] + (1.0 - a.mu2) * q2;
    alpha = a.bc * s / (sqrt(nu) + a.eps);
  }
  // A = sg^2 times the Gram in acc, then `steps` iterations on it; pa = sg P.
  double pa[NB][MC > 16 ? 8 : 4];
  auto iterate = [&](double sg, int steps) {
#pragma unroll
    for (int b = 0; b < SmDim<MC>::NBLK; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) S.red[wave][b][lane * 4 + e] = acc[b][e];
    __syncthreads();
    for (int q = tid; q < SmDim<MC>::NBLK * 256; q += TINY_THREADS) {
      const int b = q >> 8, ln = (q & 255) >> 2, e = q & 3;
      double sum = 0.0;
#pragma unroll
      for (int w = 0; w < TY_NW; ++w) sum += S.red[w][b][q & 255];
      sum *= sg * sg;
      const int i = (b == 2 ? 16 : 0) + (ln >> 4) + 4 * e, j = (b > 0 ? 16 : 0) + (ln & 15);
      S.core.A[i * SM_LD + j] = sum;
      if (b == 1) S.core.A[j * SM_LD + i] = sum;
    }
    __syncthreads();
    sm_operand<MC>(sm_iterate<TY_NW>(S.core, NB, ns, steps), sg, pa, lane);
    __syncthreads();   // P is in registers; the staging rows are free again
  };
  iterate(sigma, LONG ? min(ns.steps, ns.span) : ns.steps);

  MALT_GLOBAL float* const X = sm_iterate_x(d, a.o_parity);
  // This lane's column of L M R, or of the float32 iterate; cf its column factor.
  auto long_column = [&](bool first, float cf, float (&x)[MC]) {
    if (first) {
      tiny_load<MC, FULL>(v.M, t, x);
      tiny_mask<MC, FULL>(t, x);
      tiny_own<MC, FULL>(buf, t, x);
      scale(x, cf);
    } else {
      tiny_load_x<MC>(X, t, np, x);
    }
  };
  if constexpr (LONG) {
    // X = P X (P L M R the first time, with sigma in P) and its Gram, until at
    // most span iterations are left.
    for (int left = ns.steps - ns.span; left > 0; left -= ns.span) {
#pragma unroll
      for (int b = 0; b < SmDim<MC>::NBLK; ++b) acc[b] = sm_zero();
#pragma unroll 1
      for (t.c0 = wave * 64; t.c0 < nc; t.c0 += TINY_THREADS) {
        const int c = t.c0 + lane;
        float x[MC];
        long_column(left == ns.steps - ns.span, c < nc ? cinv[c] : 0.f, x);
        sm_advance<MC>(buf, pa, c < nc, mc, lane, x);
#pragma unroll
        for (int i = 0; i < MC; ++i)
          if (i < mc && c < nc) X[(size_t)i * np + c] = x[i];
        sm_stage<MC>(buf, x, lane);
        sm_gram<MC>(buf, acc, lane);
      }
      __syncthreads();   // the staging rows are free for the blocks
      iterate(1.0, min(left, ns.span));
    }
  }

  // O = sigma P (L M R), or P X, its norm and ||L O R||.
  double o2 = 0.0, d2 = 0.0;
  t.c0 = wave * 64;
  if (!LONG && t.c0 < nc) fetch(v.M, t);
#pragma unroll 1
  for (; t.c0 < nc; t.c0 += TINY_THREADS) {
    const int c = t.c0 + lane;
    float x[MC], cf;
    if constexpr (LONG) {
      cf = c < nc ? cinv[c] : 0.f;
      long_column(ns.steps <= ns.span, cf, x);
    } else {
      copy(x, xn);
      cf = FULL || c < nc ? cn : 0.f;
      if (const TinyCols nx = next(t); nx.c0 < nc) fetch(v.M, nx);
      tiny_mask<MC, FULL>(t, x);
      tiny_own<MC, FULL>(buf, t, x);
      scale(x, cf);
    }
    sm_apply<MC>(buf, pa, S.rowf, cf, FULL || c < nc, FULL ? MC : mc, lane, x, o2, d2);
    tiny_put16<MC, FULL>(O, t, np, x);
  }
  sm_block_sum<TY_NW>(o2, d2, S.red2);
  const double graft = sqrt(o2) / (sqrt(d2) + a.eps), coef_d = a.lr * alpha * graft;
  if (tid == 0) {
    if constexpr (MALTER) nu_p[0] = (float)nu;
    scal[SC_S] = s;
    scal[SC_SIGMA] = sigma;
    scal[SC_NU] = nu;
    scal[SC_Q] = q2;
    scal[SC_ALPHA] = alpha;
    scal[SC_O2] = o2;
    scal[SC_D2] = d2;
    scal[SC_GRAFT] = graft;
    scal[SC_COEF] = coef_d;
  }

  if (LONG && ns.defer) return;

  // W <- decay W - coef L O R.
  const float coef = (float)coef_d;
  bf16_t on[MC];
  auto fetch_o = [&](const TinyCols& t) {
    const int c = FULL ? t.c0 + lane : min(t.c0 + lane, nc - 1);
#pragma unroll
    for (int i = 0; i < MC; ++i) on[i] = O[(FULL ? i : min(i, mc - 1)) * np + c];
  };
  t.c0 = wave * 64;
  if (t.c0 < nc) {
    fetch(v.W, t);
    fetch_o(t);
  }
#pragma unroll 1
  for (; t.c0 < nc; t.c0 += TINY_THREADS) {
    float w[MC], o[MC];
    copy(w, xn);
#pragma unroll
    for (int i = 0; i < MC; ++i) o[i] = bf16_lo(on[i]);
    const float cf = cn;
    if (const TinyCols nx = next(t); nx.c0 < nc) {
      fetch(v.W, nx);
      fetch_o(nx);
    }
    tiny_own<MC, FULL>(buf, t, w);
#pragma unroll
    for (int i = 0; i < MC; ++i) {
      const float f = S.rowf[i];
      w[i] = tall ? a.decay * w[i] - coef * cf * o[i] * f : a.decay * w[i] - coef * f * o[i] * cf;
    }
    tiny_give<MC, FULL>(buf, t, w);
    tiny_put<MC, FULL>(v.W, t, w);
  }
}

template <bool MALTER>
__global__ __launch_bounds__(TINY_THREADS) void tiny_step_kernel(SmallArgs ns) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  TinyLds& S = *reinterpret_cast<TinyLds*>(lds);
  const Tile t = ns.e.tiles[blockIdx.x];   // (mat, rows held per column, -, -)
  const MatDesc& d = ns.e.desc[t.mat];
  const bool full = d.mc == t.ti && d.nc % 64 == 0;
  if (t.ti == 8) {
    if (full) tiny_step<MALTER, 8, true, false>(ns, t.mat, S);
    else tiny_step<MALTER, 8, false, false>(ns, t.mat, S);
  } else if (t.ti == 16) {
    if (full) tiny_step<MALTER, 16, true, false>(ns, t.mat, S);
    else tiny_step<MALTER, 16, false, false>(ns, t.mat, S);
  } else {
    if (full) tiny_step<MALTER, 32, true, false>(ns, t.mat, S);
    else tiny_step<MALTER, 32, false, false>(ns, t.mat, S);
  }
}

// The LONG steps; one instance for every m'.
template <bool MALTER>
__global__ __launch_bounds__(TINY_THREADS) void tiny_long_step_kernel(SmallArgs ns) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  tiny_step<MALTER, SM_M, false, true>(ns, ns.e.tiles[blockIdx.x].mat, *reinterpret_cast<TinyLds*>(lds));
}

// The update of W by itself, after every gradient of the step has been read: for
// a set in which another matrix's gradient overlaps a W of this route.
__global__ __launch_bounds__(TINY_THREADS) void tiny_write_kernel(EwArgs a) {
  const Tile t = a.tiles[blockIdx.x];
  const EwView v = ew_view(a, t.mat);
  const float coef = (float)v.scal[SC_COEF];
  for (int e = threadIdx.x; e < v.m * v.n; e += TINY_THREADS) {
    const int i = e / v.n, j = e % v.n;
    const float o = bf16_lo(v.O[v.tall ? (size_t)j * v.np + i : (size_t)i * v.np + j]);
    v.W[e] = a.decay * v.W[e] - coef * v.Lv[i] * o * v.Rv[j];
  }
}

// ---------------------------------------------------------------------------
// The three launches of larger matrices, once per span iterations.
// ---------------------------------------------------------------------------
constexpr int SL_NW = NTHREADS / 64;
static_assert(SM_CH_U == NTHREADS, "one column per thread in the product");

// Column c, in the canonical orientation (rows < SM_M), of L M R (FIRST) or of
// the float32 iterate.  (Instances: chosen at run time, the product took 124
// registers in place of 72.)
template <bool FIRST>
__device__ __forceinline__ void sm_column(const MatDesc& d, const SmallArgs& ns, int c, float (&x)[SM_M]) {
  if constexpr (!FIRST) {
    const MALT_GLOBAL float* const X = sm_iterate_x(d, ns.e.o_parity);
#pragma unroll
    for (int i = 0; i < SM_M; ++i) x[i] = i < d.mc && c < d.nc ? X[(size_t)i * d.np + c] : 0.f;
    return;
  }
  const float cf = c < d.nc ? gptr(d.tall ? d.Lv : d.Rv)[c] : 0.f;
  const MALT_GLOBAL float* const rf = gptr(d.tall ? d.Rv : d.Lv);
  const MALT_GLOBAL float* const M = gptr(d.M);
#pragma unroll
  for (int i = 0; i < SM_M; ++i) {
    if (i >= d.mc || c >= d.nc) x[i] = 0.f;
    else if (!d.tall) x[i] = rf[i] * M[(size_t)i * d.n + c] * cf;
    else x[i] = cf * M[(size_t)c * d.n + i] * rf[i];
  }
}

template <bool FIRST>
__global__ __launch_bounds__(NTHREADS) void sm_gram_kernel(SmallArgs ns) {
  __shared__ union { float stage[SL_NW * SM_WAVE]; double red[SL_NW][3][64 * 4]; } S;
  const Tile t = ns.e.tiles[blockIdx.x];   // (mat, chunk, -, -)
  const MatDesc& d = ns.e.desc[t.mat];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* const buf = S.stage + wave * SM_WAVE;
  f64x4 acc[3] = {sm_zero(), sm_zero(), sm_zero()};
  const int c0 = t.ti * d.sm_chunk, c1 = min(c0 + d.sm_chunk, d.nc);
  for (int c = c0 + wave * 64; c < c1; c += NTHREADS) {
    float x[SM_M];
    sm_column<FIRST>(d, ns, c + lane < c1 ? c + lane : d.nc, x);
    sm_stage<SM_M>(buf, x, lane);
    sm_gram<SM_M>(buf, acc, lane);
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) S.red[wave][b][lane * 4 + e] = acc[b][e];
  __syncthreads();
  // Blocks as they lie in the accumulators; the iteration unpacks them.
  MALT_GLOBAL double* const out = gptr(d.Ap) + (size_t)t.ti * SM_PART;
  for (int q = threadIdx.x; q < SM_PART; q += NTHREADS)
    out[q] = (S.red[0][q >> 8][q & 255] + S.red[1][q >> 8][q & 255]) + (S.red[2][q >> 8][q & 255] + S.red[3][q >> 8][q & 255]);
}

__global__ __launch_bounds__(SM_PART) void sm_iterate_kernel(SmallArgs ns) {
  __shared__ SmCore s;
  const MatDesc& d = ns.e.desc[ns.e.tiles[blockIdx.x].mat];
  const int tid = threadIdx.x;
  double sg = 1.0;   // the iterate has been normalised
  if (ns.first && ns.norms) {   // the norm scalars are formed here
    __shared__ double sh[SM_PART / 64][2];
    double sums[2];
    block_sum_pairs<SM_PART>(d.k2part, d.k2_tiles, sh, sums);
    sg = 1.0 / (sqrt(sums[0]) + ns.e.ns_eps);
    if (tid == 0) norm_scalars(ns.e, d, sums);
  } else if (ns.first) {
    sg = gptr(d.scal)[SC_SIGMA];
  }
  {
    const MALT_GLOBAL double* const Ap = gptr(d.Ap);
    double sum = 0.0;
#pragma unroll 8
    for (int ch = 0; ch < d.sm_gchunks; ++ch) sum += Ap[(size_t)ch * SM_PART + tid];
    sum *= sg * sg;
    const int b = tid >> 8, ln = (tid & 255) >> 2, e = tid & 3;
    const int i = (b == 2 ? 16 : 0) + (ln >> 4) + 4 * e, j = (b > 0 ? 16 : 0) + (ln & 15);
    s.A[i * SM_LD + j] = sum;
    if (b == 1) s.A[j * SM_LD + i] = sum;
  }
  __syncthreads();
  const double* const P = sm_iterate<SM_PART / 64>(s, 2, ns, ns.steps);
  for (int q = tid; q < SM_M * SM_M; q += SM_PART) gptr(d.Bs)[q] = sg * P[(q / SM_M) * SM_LD + q % SM_M];
}

template <bool FIRST, bool LAST>
__global__ __launch_bounds__(NTHREADS) void sm_apply_kernel(SmallArgs ns) {
  __shared__ float stage[SL_NW * SM_WAVE];
  __shared__ double P[SM_M * SM_LD];
  __shared__ float rowf[SM_M];
  __shared__ double red[SL_NW][2];
  const Tile t = ns.e.tiles[blockIdx.x];   // (mat, chunk, -, partial slot)
  const MatDesc& d = ns.e.desc[t.mat];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int mc = d.mc, nc = d.nc, c = t.ti * SM_CH_U + tid;
  for (int q = tid; q < SM_M * SM_M; q += NTHREADS) P[(q / SM_M) * SM_LD + q % SM_M] = gptr(d.Bs)[q];
  if (tid < SM_M) rowf[tid] = tid < mc ? gptr(d.tall ? d.Rv : d.Lv)[tid] : 0.f;
  const float cf = c < nc ? gptr(d.tall ? d.Lv : d.Rv)[c] : 0.f;
  float x[SM_M];
  sm_column<FIRST>(d, ns, c, x);
  __syncthreads();
  double pa[2][8], o2 = 0.0, d2 = 0.0;
  sm_operand<SM_M>(P, 1.0, pa, lane);
  if constexpr (!LAST) {   // X = P X, in place where it came from X
    sm_advance<SM_M>(stage + wave * SM_WAVE, pa, c < nc, mc, lane, x);
    MALT_GLOBAL float* const X = sm_iterate_x(d, ns.e.o_parity);
#pragma unroll
    for (int i = 0; i < SM_M; ++i)
      if (i < mc && c < nc) X[(size_t)i * d.np + c] = x[i];
    return;
  }
  sm_apply<SM_M>(stage + wave * SM_WAVE, pa, rowf, cf, c < nc, mc, lane, x, o2, d2);
  sm_store_o<SM_M>(gptr(d.X[ns.e.o_parity]), d.np, mc, c, c < nc, x);
  sm_block_sum<SL_NW>(o2, d2, red);
  if (tid == 0) {
    gptr(d.gpart)[2 * (size_t)t.idx + 0] = (float)o2;
    gptr(d.gpart)[2 * (size_t)t.idx + 1] = (float)d2;
  }
}

}  // namespace

// Iterations in the Gram space before A is formed from X again: as many as keep
// 1e-16 a^(2 k) below 1e-7, at most 8 (8 with the default quintic, whose a is
// 3.4445).
int small_span(double a) {
  int k = 1;
  for (double g = a * a * a * a; k < 8 && g <= 1e9; g *= a * a) ++k;
  return k;
}

namespace {
const void* tiny_kernel(bool malter, bool lng) {
  if (lng)
    return malter ? reinterpret_cast<const void*>(&tiny_long_step_kernel<true>)
                  : reinterpret_cast<const void*>(&tiny_long_step_kernel<false>);
  return malter ? reinterpret_cast<const void*>(&tiny_step_kernel<true>)
                : reinterpret_cast<const void*>(&tiny_step_kernel<false>);
}
}  // namespace

// The whole-step kernels use more dynamic LDS than the default limit (see
// ns_sym_setup).
hipError_t tiny_step_setup(bool malter) {
  for (int lng = 0; lng < 2; ++lng) {
    const hipError_t e =
        hipFuncSetAttribute(tiny_kernel(malter, lng), hipFuncAttributeMaxDynamicSharedMemorySize, sizeof(TinyLds));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_tiny_step(const SmallArgs& a, hipStream_t s) {
  if (a.e.ntiles == 0) return hipSuccess;
  const dim3 grid(a.e.ntiles), block(TINY_THREADS);
  if (a.steps > a.span || a.defer) {
    if (a.e.malter) hipLaunchKernelGGL(tiny_long_step_kernel<true>, grid, block, sizeof(TinyLds), s, a);
    else hipLaunchKernelGGL(tiny_long_step_kernel<false>, grid, block, sizeof(TinyLds), s, a);
  } else {
    if (a.e.malter) hipLaunchKernelGGL(tiny_step_kernel<true>, grid, block, sizeof(TinyLds), s, a);
    else hipLaunchKernelGGL(tiny_step_kernel<false>, grid, block, sizeof(TinyLds), s, a);
  }
  return hipGetLastError();
}

hipError_t launch_tiny_write(const EwArgs& a, hipStream_t s) {
  if (a.ntiles == 0) return hipSuccess;
  hipLaunchKernelGGL(tiny_write_kernel, dim3(a.ntiles), dim3(TINY_THREADS), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_small_ns(const SmallArgs& a, int phase, hipStream_t s) {
  if (a.e.ntiles == 0) return hipSuccess;
  const dim3 grid(a.e.ntiles), block(NTHREADS);
  if (phase == PH_POLY) {
    hipLaunchKernelGGL(sm_iterate_kernel, grid, dim3(SM_PART), 0, s, a);
  } else if (phase == PH_GRAM) {
    if (a.first) hipLaunchKernelGGL((sm_gram_kernel<true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((sm_gram_kernel<false>), grid, block, 0, s, a);
  } else if (a.first) {
    if (a.last) hipLaunchKernelGGL((sm_apply_kernel<true, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((sm_apply_kernel<true, false>), grid, block, 0, s, a);
  } else {
    if (a.last) hipLaunchKernelGGL((sm_apply_kernel<false, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((sm_apply_kernel<false, false>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace malt
