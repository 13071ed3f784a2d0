// Internal device-side structures and kernel launchers of libmalt (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace malt {

// Elementwise tiles (momentum / back-map): EW_TR rows x EW_TC cols per
// EW_THREADS-thread workgroup; each lane owns 4 consecutive columns and each
// wave EW_TR / 16 = 2 rows, whose loads it issues before any arithmetic.
// (A streaming pass runs closest to HBM's rate with few loads in flight per
// wave and no loop per wave.)
constexpr int EW_TR = 32;
constexpr int EW_TC = 256;
constexpr int EW_THREADS = 1024;
// Scale+convert of wide matrices (canonical = W): K2W_R rows x EW_TC cols per
// K2W_THREADS-thread workgroup, one float4 per lane and row, four rows per
// wave (measured against 1-8 rows per wave and 256-1024 threads: within 2%,
// this the fastest).
constexpr int K2W_R = 64;
constexpr int K2W_THREADS = 1024;
// Scale+convert of tall matrices (canonical = W^T, through an LDS transpose):
// K2_T x K2_T tiles; a K2T_THREADS-thread workgroup takes K2_GROUP consecutive
// tiles of one row band (padded W dimensions are multiples of 256, so bands
// hold whole groups).
constexpr int K2_T = 64;
constexpr int K2_GROUP = 2;
constexpr int K2T_THREADS = 512;
// Newton-Schulz output tile and padding unit of the bf16 buffers.
constexpr int NS_TILE = 256;
constexpr int NS_BK = 64;
// Matrices whose short side is at most this carry B = b A + c A^2 as a bf16
// pair (hi, lo = bf16(B - hi)) into the update product: with few singular
// values the rounding of the small m' x m' polynomial is not averaged away.
constexpr int NS_SPLIT_MAX = 128;
// Threads of a workgroup of the finalise, scalar, zero-fill and condition-number
// kernels and of the short sides' Gram and product.
constexpr int NTHREADS = 256;
// Preconditioner finalise: rows or columns per workgroup, NTHREADS / FIN_W
// threads each; FIN_W_LONG of them where each has more than FIN_LONG partials.
constexpr int FIN_W = 64;
constexpr int FIN_W_LONG = 8;
constexpr int FIN_LONG = 512;
// Matrices whose short side is at most this run Newton-Schulz in the Gram space
// in float64 (small_ns.hip).  Those of at most TINY_ELEMS elements can take their
// whole step in one workgroup (choose_whole_steps); the others take a Gram over chunks of at least SM_CH_G
// columns, at most SM_CHUNKS of them, and the final product over SM_CH_U columns
// (one per thread).
constexpr int NS_SMALL_MAX = 32;
constexpr int TINY_THREADS = 512;
constexpr int TINY_ELEMS = 65536;
constexpr int SM_CH_G = 1024;
constexpr int SM_CHUNKS = 128;
constexpr int SM_CH_U = 256;
constexpr int SM_PART = 3 * 256;   // values of one chunk's Gram: three upper 16 x 16 blocks

typedef uint16_t bf16_t;   // bf16 storage

// Device pointers read from the descriptor tables are generic (flat) to the
// compiler, and flat memory instructions count against lgkmcnt as well as
// vmcnt: every later wait for an LDS read, a scalar load or a cross-lane
// shuffle would then also wait for them. Accesses through gptr() are global.
#define MALT_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ MALT_GLOBAL T* gptr(T* p) {
  return (MALT_GLOBAL T*)p;
}

typedef float malt_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 malt_bf16x2 __attribute__((ext_vector_type(2)));

// Two floats -> two bf16 (round to nearest even; one v_cvt_pk_bf16_f32),
// packed low | high << 16.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const malt_f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, malt_bf16x2));
}
__device__ __forceinline__ float bf16_lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }

// Per-matrix scalar slots (float64) in the workspace.
enum {
  SC_S = 0,       // ||L M R||_F
  SC_SIGMA = 1,   // 1 / (s + ns_eps)
  SC_NU = 2,      // nu_t (MALTER)
  SC_ALPHA = 3,   // alpha_t (1 for MALT)
  SC_O2 = 4,      // ||O||_F^2
  SC_D2 = 5,      // ||L O R||_F^2
  SC_GRAFT = 6,   // ||O|| / (||D|| + eps)
  SC_COEF = 7,    // lr * alpha * graft
  SC_Q = 8,       // ||L G R||_F^2 (MALTER)
  MAT_SCALARS = 16
};

struct MatDesc {
  int32_t m, n;        // W rows, cols
  int32_t mc, nc;      // canonical orientation: mc = min(m,n) rows, nc = max(m,n) cols
  int32_t mp, np;      // canonical dims padded to NS_TILE
  int32_t tall;        // 1 when m > n: canonical = W^T
  int32_t split;       // 1: B stored as [hi | lo] (row pitch 2*mp)
  int32_t k1_ct;       // column tiles of the momentum pass (row partial count)
  int32_t k1_rt;       // row tiles of the momentum pass (column partial count)
  int32_t k2_tiles;    // scale+convert tiles (norm partial count)
  int32_t upd_tiles;   // NS update tiles (graft partial count)
  float* M;
  float* l;
  float* r;
  float* nu;           // nullptr for MALT
  float* Lv;           // m
  float* Rv;           // n
  float* rowpart;      // [k1_ct][m]
  float* colpart;      // [k1_rt][n]
  float* k2part;       // [k2_tiles][2]: sum (LMR)^2, sum (LGR)^2
  float* gpart;        // [upd_tiles][2]: sum O^2, sum (LOR)^2
  bf16_t* X[2];        // canonical mp x np, row-major (double-buffered iterate)
  bf16_t* A;           // mp x mp  (Gram / A)
  bf16_t* B;           // mp x mp, or mp x 2mp [hi | lo] when split (b A + c A^2)
  double* scal;        // MAT_SCALARS
  // short side <= NS_SMALL_MAX; null otherwise
  int32_t small;       // 1: Newton-Schulz in the Gram space (small_ns.hip)
  int32_t tiny;        // 1: the whole step in one workgroup; the other passes skip this matrix
  int32_t sm_gchunks;  // Gram partial count
  int32_t sm_chunk;    // columns per Gram partial
  double* Ap;          // [sm_gchunks][SM_PART] Gram partials
  double* Bs;          // [32][32] P = B_{s-1} ... B_0 (times sigma the first time)
  // Newton-Schulz domain: canonical dims rounded up to the plan's largest
  // Newton-Schulz tile (<= mp, np); no Newton-Schulz kernel works past it
  int32_t dm, dn;
  int32_t gsplit;      // parts of the Gram's contraction (1: not cut)
};

// Per-step caller pointers; vec = 1 when W, G and M rows allow 16-byte access.
struct PtrPair {
  float* W;
  const float* G;
  int32_t vec;
  int32_t pad_;
};

// One unit of work of a grouped launch.
//   momentum/back-map: (mat, row tile, col tile, -)
//   preconditioner finalise: (mat, 0 = rows | 1 = cols, chunk, rows or columns per chunk)
//   scale+convert: (mat, row tile, col tile, partial slot)
//   NS: (mat, tile row, tile col, partial slot), stored in dispatch order:
//       entry b runs on XCD b % 8; mat = -1 pads the shorter XCD runs
//       On the smaller tiles a Gram's idx is its part of the contraction;
//       reduction of the parts: (mat, tile row, tile col, 16-row piece)
//   short sides: Gram (mat, chunk, -, -), iteration (mat, -, -, -), product
//            (mat, chunk, -, partial slot); whole step (mat, rows per column, -, -)
struct Tile {
  int32_t mat, ti, tj, idx;
};

enum { PH_GRAM = 0, PH_POLY = 1, PH_UPDATE = 2, PH_REDUCE = 3 };

struct EwArgs {
  const MatDesc* desc;
  const PtrPair* ptrs;
  const Tile* tiles;
  int32_t ntiles;
  float mu1, one_minus_mu1;
  double mu2, eps;
  double bc;             // sqrt(1 - mu2^t) / (1 - mu1^t + eps)
  double ns_eps;
  double lr;
  float decay;           // 1 - lr * weight_decay
  int32_t malter;
  int32_t identity;
  int32_t o_parity;      // which X buffer holds the final O
};

// Short sides: the step's arguments and the Newton-Schulz coefficients.
struct SmallArgs {
  EwArgs e;
  double a, b, c;
  int32_t steps;         // iterations: the step's, or those of these three launches
  int32_t span;          // iterations before A is formed from X again (small_span)
  int32_t norms;         // the first iteration kernel also forms the norm scalars
  int32_t first, last;   // three launches: X is L M R; O follows
  int32_t defer;         // whole step: all but W, which launch_tiny_write does
};

struct NsArgs {
  const MatDesc* desc;
  const Tile* tiles;
  int32_t ntiles;
  int32_t phase;
  int32_t first;         // iteration 0: apply sigma
  int32_t last;          // final iteration: write O and graft partials
  int32_t src;           // X[src] is the current iterate, X[src ^ 1] receives the next
  float a, b, c;
  int32_t norms;         // the first Gram also forms the norm scalars (of ew)
  EwArgs ew;
};

// Per-step pointer table written by a kernel whose arguments carry the
// pointers: the runtime copies kernel arguments at enqueue, so a step needs no
// host staging buffer and never waits for an earlier upload.
constexpr int PTR_CHUNK = 128;
struct PtrUploadArgs {
  PtrPair* dst;
  int32_t count;       // <= PTR_CHUNK
  PtrPair p[PTR_CHUNK];
};

// Launchers (stream-ordered, no synchronisation).
hipError_t launch_ptr_upload(const PtrUploadArgs& a, hipStream_t s);
hipError_t launch_zero_fill(void* dst, size_t bytes, hipStream_t s);   // dst 16-byte aligned
hipError_t launch_momentum_rowcol(const EwArgs& a, hipStream_t s);
hipError_t launch_precond_finalize(const EwArgs& a, hipStream_t s);
hipError_t launch_scale_convert(const EwArgs& a, bool tall, hipStream_t s);
hipError_t launch_norm_scalars(const EwArgs& a, int32_t nmat, hipStream_t s);
hipError_t launch_graft_scalars(const EwArgs& a, int32_t nmat, hipStream_t s);
hipError_t launch_backmap_write(const EwArgs& a, bool graft, hipStream_t s);   // graft: forms the graft scalars too
hipError_t launch_precond_cond(const MatDesc* desc, int32_t nmat, double* out, hipStream_t s);
hipError_t ns_sym_setup(int phase);      // LDS limits, once per plan that launches the kernel, on its device
hipError_t launch_ns_gemm(const NsArgs& a, hipStream_t s);
hipError_t ns_update_setup();
hipError_t launch_ns_update(const NsArgs& a, hipStream_t s);
hipError_t launch_ns_mid(const NsArgs& a, int tile, hipStream_t s);   // 64 or 128 tiles, all phases (ns_mid.hip)
int small_span(double a);
hipError_t tiny_step_setup(bool malter);
hipError_t launch_small_ns(const SmallArgs& a, int phase, hipStream_t s);
hipError_t launch_tiny_step(const SmallArgs& a, hipStream_t s);
hipError_t launch_tiny_write(const EwArgs& a, hipStream_t s);

// One matrix's descriptor fields and caller pointers, as the tile passes use
// them, read in one place before any branch: the compiler then issues them as
// one batch of scalar loads, not a chain of load-and-wait behind each test.
struct EwView {
  int m, n, np, tall;
  bool vec;
  MALT_GLOBAL float* W;
  const MALT_GLOBAL float* G;
  MALT_GLOBAL float* M;
  const MALT_GLOBAL float* Lv;
  const MALT_GLOBAL float* Rv;
  MALT_GLOBAL float* rowpart;
  MALT_GLOBAL float* colpart;
  MALT_GLOBAL float* k2part;
  MALT_GLOBAL bf16_t* X0;
  const MALT_GLOBAL bf16_t* O;   // back-map: the buffer holding the final iterate
  MALT_GLOBAL double* scal;
};

__device__ __forceinline__ EwView ew_view(const EwArgs& a, int mat) {
  const MatDesc& d = a.desc[mat];
  const PtrPair& p = a.ptrs[mat];
  EwView v;
  v.m = d.m;
  v.n = d.n;
  v.np = d.np;
  v.tall = d.tall;
  v.vec = p.vec != 0;
  v.W = gptr(p.W);
  v.G = gptr(p.G);
  v.M = gptr(d.M);
  v.Lv = gptr(d.Lv);
  v.Rv = gptr(d.Rv);
  v.rowpart = gptr(d.rowpart);
  v.colpart = gptr(d.colpart);
  v.k2part = gptr(d.k2part);
  v.X0 = gptr(d.X[0]);
  v.O = gptr(d.X[a.o_parity]);
  v.scal = gptr(d.scal);
  return v;
}

// Fixed-order sums in float64 of `count` float pairs (stride 2) over a
// workgroup of THREADS, given to every thread; sh is free again at the next
// barrier.  The two scalar kernels and the passes that take their place share
// it; a thread adds every THREADS-th pair, so the result depends on THREADS.
template <int THREADS>
__device__ __forceinline__ void block_sum_pairs(const float* __restrict__ p, int count, double (*sh)[2], double out[2]) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const MALT_GLOBAL f32x2* const q = reinterpret_cast<const MALT_GLOBAL f32x2*>(gptr(p));   // 256-byte aligned
  double s0 = 0.0, s1 = 0.0;
  int k = threadIdx.x;
  // Eight pairs in flight, added one by one (an embedding of 50257 x 768 has
  // 9456: 15 us with one in flight).
  for (; k + 7 * THREADS < count; k += 8 * THREADS) {
    f32x2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = q[k + u * THREADS];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      s0 += (double)v[u].x;
      s1 += (double)v[u].y;
    }
  }
  for (; k < count; k += THREADS) {
    s0 += (double)q[k].x;
    s1 += (double)q[k].y;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_xor(s0, off, 64);
    s1 += __shfl_xor(s1, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    sh[threadIdx.x >> 6][0] = s0;
    sh[threadIdx.x >> 6][1] = s1;
  }
  __syncthreads();
  out[0] = out[1] = 0.0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) {
    out[0] += sh[w][0];
    out[1] += sh[w][1];
  }
}

// ||Mt||_F, sigma = 1/(s+ns_eps), nu_t and alpha_t (Alg. 2; displayed alpha_t)
// from the sums of (LMR)^2 and (LGR)^2; one thread writes them.
__device__ __forceinline__ void norm_scalars(const EwArgs& a, const MatDesc& d, const double sums[2]) {
  const double s = sqrt(sums[0]);
  MALT_GLOBAL double* const sc = gptr(d.scal);
  double nu = 0.0, alpha = 1.0;
  if (a.malter) {
    nu = a.mu2 * (double)gptr(d.nu)[0] + (1.0 - a.mu2) * sums[1];
    gptr(d.nu)[0] = (float)nu;
    alpha = a.bc * s / (sqrt(nu) + a.eps);
  }
  sc[SC_S] = s;
  sc[SC_SIGMA] = 1.0 / (s + a.ns_eps);
  sc[SC_NU] = nu;
  sc[SC_Q] = a.malter ? sums[1] : 0.0;
  sc[SC_ALPHA] = alpha;
}

// ||O||^2, ||D||^2, graft and step coefficient from the sums of O^2 and
// (L O R)^2; returns the coefficient, `write` also stores them.
__device__ __forceinline__ double graft_scalars(const EwArgs& a, MALT_GLOBAL double* sc, const double sums[2], bool write) {
  const double g = sqrt(sums[0]) / (sqrt(sums[1]) + a.eps);
  const double coef = a.lr * sc[SC_ALPHA] * g;
  if (write) {
    sc[SC_O2] = sums[0];
    sc[SC_D2] = sums[1];
    sc[SC_GRAFT] = g;
    sc[SC_COEF] = coef;
  }
  return coef;
}

// XCDs of the chip; workgroups are dispatched to them round-robin.
constexpr int NXCD = 8;

// Map a workgroup id to a work index so that the workgroups that land on one
// XCD (dispatched round-robin over 8 XCDs) take a contiguous run of the work
// list; a bijection on [0, n).
__device__ __forceinline__ int xcd_remap(int b, int n) {
  const int q = n >> 3, r = n & 7;
  const int x = b & 7, k = b >> 3;
  return (x < r) ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

}  // namespace malt
