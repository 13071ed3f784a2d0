// Newton-Schulz phases on smaller tiles (T x T, T = 64 or 128), for sets whose
// 256 x 256 tiles (ns_sym.hip, ns_update.hip) would leave most of the chip
// idle, and the Gram of long matrices cut along k:
//   Gram        A  = s X X^T   (upper tiles, mirrored on write); cut along k,
//               the tiles leave fp32 partials and the reduction adds them in a
//               fixed order, rounds once and mirrors
//   Polynomial  B' = a I + b A + c A A^T   (upper tiles, mirrored)
//   Update      X' = s B' X, as C^T = X^T B'^T blocks
// Same operands, instruction (v_mfma_f32_16x16x32_bf16) and roundings to bf16 as
// the 256-tile kernels, and the same accumulation order in k except in the
// polynomial: b A is added in fp32 after the sum here, where the 256-tile kernel
// adds (b / c) A within it (c != 0).  One workgroup of 4 waves per tile,
// two or three workgroups per CU, so one tile's prologue and epilogue run
// beside another's main loop.
//
// What bounds them: a small set is bound by the length of its longest tile (a
// 64-tile with a CU to itself takes 0.22 us per 64-k stage and 3.5 us around
// them, against 1.3 and 6-11 for a 256-tile); with the chip full, by operand
// delivery: 64- and 128-tiles move 4 and 2 times a 256-tile's operand bytes per
// flop, and a CU takes about 28 and 20 B/clk of them (64-tile update of 96
// GPT-2 Medium matrices 1130 us, without its MFMAs 1270; without its loads
// 830).  Measured against the 256-tile kernels alone, us per step: one 256 x 512
// matrix 216 -> 83; one GPT-2 Small block (MALTER) 608 -> 302; eight ragged
// matrices 787 -> 243; GPT-2 Small with its embeddings, whose 50257 x 768 Gram
// was 6 tiles of 788 stages, 6375 -> 2720.
#include "ns_common.h"

namespace malt {

using namespace ns;

namespace {

constexpr int RED_THREADS = 256;

// Upper tiles of one symmetric product.
template <int T, int PHASE>
__global__ __launch_bounds__(MidGeom<T>::NT) __attribute__((amdgpu_waves_per_eu(MidGeom<T>::WPE, MidGeom<T>::WPE)))
void ns_mid_sym_kernel(NsArgs args) {
  using G = MidGeom<T>;
  using ML = MidLoads<T>;
  constexpr int WT = G::WT, I = WT / 16, NL = G::LOADS, H = G::H, RB = G::RB;
  // Epilogue: per-wave copies, transposed (padded by 16 bytes) and as is (8).
  constexpr int PITCH_T = WT * 2 + 16, PITCH_R = WT * 2 + 8;
  constexpr int WREG = WT * PITCH_T;
  static_assert(G::NW * WREG <= G::RING_BYTES, "epilogue copies fit the ring");
  __shared__ __attribute__((aligned(16))) char lds[G::RING_BYTES];

  const Tile t = args.tiles[blockIdx.x];
  if (t.mat < 0) return;
  const MatDesc* __restrict__ d = args.desc + t.mat;
  const int mp = d->mp, np = d->np, dm = d->dm, dn = d->dn;
  const bool split = d->split != 0;
  const int S = PHASE == PH_GRAM ? d->gsplit : 1;
  bf16_t* const Am = d->A;
  bf16_t* const Bm = d->B;
  const bf16_t* P = PHASE == PH_GRAM ? d->X[args.src] : Am;
  float* const part = reinterpret_cast<float*>(d->X[args.src ^ 1]);
  const bool norms = PHASE == PH_GRAM && args.first && args.norms;
  float sig = (args.first && PHASE == PH_GRAM && !norms) ? (float)d->scal[SC_SIGMA] : 1.f;
  const int ld = PHASE == PH_GRAM ? np : mp;
  const int row0 = t.ti * T, col0 = t.tj * T;
  const bool diag = t.ti == t.tj;
  const int KT = (PHASE == PH_GRAM ? dn : dm) / G::BK;
  const int k0 = mid_k0(t.idx, S, KT), nk = mid_k0(t.idx + 1, S, KT) - k0;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 1, wc = wave & 1;
  const int rl0 = wr * WT + 4 * (lane >> 4), cl0 = wc * WT + (lane & 15);   // tile row / column of i = j = e = 0

  // The b A term: A is symmetric, so the four rows of a lane's column are 8
  // contiguous bytes of A's row; in flight during the main loop.
  uint2 av[I][I];
  if constexpr (PHASE == PH_POLY) {
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
      for (int j = 0; j < I; ++j)
        av[i][j] = __builtin_bit_cast(
            uint2, *reinterpret_cast<const MALT_GLOBAL uint64_t*>(gptr(Am) + (size_t)(col0 + cl0 + j * 16) * mp + row0 +
                                                                  rl0 + i * 16));
  }

  f32x4 acc[I][I];
#pragma unroll
  for (int i = 0; i < I; ++i)
#pragma unroll
    for (int j = 0; j < I; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  const i32x4 rsP = buf_rsrc(P);
  // KIND 0: off-diagonal tile; 1: diagonal tile (one operand panel, both
  // operands read from it); 2: the wave of a diagonal tile whose sub-tile is
  // the mirror of another's, which only loads.
  auto main_loop = [&](auto kind_tag) {
    constexpr int KIND = decltype(kind_tag)::value;
    constexpr int NLD = KIND == 0 ? NL : NL / 2;
    uint32_t voff[NL];
    int dst_off[NL];
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int o = q / (NL / 2), g = wave + (q % (NL / 2)) * G::NW;
      voff[q] = (uint32_t)ML::voff_rk(g, lane, o ? col0 : row0, ld);
      dst_off[q] = o * G::OPER_BYTES + g * 1024;
    }
    int offa[H], offb[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int kc = 4 * h + (lane >> 4);
      offa[h] = G::swz_rk(wr * WT + (lane & 15), kc);
      offb[h] = (KIND ? 0 : G::OPER_BYTES) + G::swz_rk(wc * WT + (lane & 15), kc);
    }
    bf16x8 fa[2][I], fb[2][I];
    mid_pipeline<G, 1>(
        nk, NLD, lds,
        [&](int kt, char* st, int i) { dma16(rsP, voff[i], (uint32_t)ML::soff_rk(k0 + kt), lds_u32(st + dst_off[i])); },
        [&](int buf, const char* st, int h) {
          if constexpr (KIND != 2) {
#pragma unroll
            for (int i = 0; i < I; ++i) fa[buf][i] = *reinterpret_cast<const bf16x8*>(st + offa[h] + i * 16 * RB);
#pragma unroll
            for (int j = 0; j < I; ++j) fb[buf][j] = *reinterpret_cast<const bf16x8*>(st + offb[h] + j * 16 * RB);
          }
        },
        [&](int buf, auto&& after) {
#pragma unroll
          for (int i = 0; i < I; ++i)
#pragma unroll
            for (int j = 0; j < I; ++j) {
              if constexpr (KIND != 2)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[buf][i], fb[buf][j], acc[i][j], 0, 0, 0);
              after(i * I + j);
            }
        });
  };
  if (!diag) main_loop(std::integral_constant<int, 0>{});
  else if (wr <= wc) main_loop(std::integral_constant<int, 1>{});
  else main_loop(std::integral_constant<int, 2>{});

  // ---------------------------------------------------------------- epilogue
  // acc[i][j][e] = C(r, c), r = rl0 + 16 i + e, c = cl0 + 16 j.
  const bool idle = diag && wr > wc;
  if constexpr (PHASE == PH_GRAM) {
    // The norm scalars, by every workgroup for itself; the first tile's stores
    // them for the kernels after this one.
    if (norms) {
      double sums[2];
      __syncthreads();   // every wave is done reading the operand ring
      block_sum_pairs<G::NT>(d->k2part, d->k2_tiles, reinterpret_cast<double(*)[2]>(lds), sums);
      sig = (float)(1.0 / (sqrt(sums[0]) + args.ew.ns_eps));
      if (t.ti == 0 && t.tj == 0 && t.idx == 0 && tid == 0) norm_scalars(args.ew, *d, sums);
    }
  }
  if (PHASE == PH_GRAM && S > 1) {
    // Partial tile, stored transposed ([c][r]): four consecutive r per lane.
    if (idle) return;
    MALT_GLOBAL float* out = gptr(part) + mid_part(t.ti, t.tj, t.idx, dm / T, S, T);
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
      for (int j = 0; j < I; ++j)
        *reinterpret_cast<MALT_GLOBAL f32x4*>(out + (size_t)(cl0 + j * 16) * T + rl0 + i * 16) = acc[i][j];
    return;
  }
  const float sc = sig * sig;
  constexpr bool poly = PHASE == PH_POLY;
  const int lo_off = (poly && split) ? mp : 0;
  bf16_t* const out = poly ? Bm : Am;
  const int ldo = lo_off ? 2 * mp : mp;
  if (poly && diag && t.ti == dm / T - 1) {
    // B' = a I on the padding past the last tile, which no kernel reads: the
    // documented B' of malt_debug_layout, padded to whole 256-tiles.
    const uint32_t h = pack_bf16x2(args.a, 0.f);
    const uint32_t l = pack_bf16x2(args.a - bf16_lo(h), 0.f);
    for (int r = dm + tid; r < mp; r += G::NT) {
      gptr(out)[(size_t)r * ldo + r] = (bf16_t)(h & 0xffffu);
      if (lo_off) gptr(out)[(size_t)r * ldo + lo_off + r] = (bf16_t)(l & 0xffffu);
    }
  }
  __syncthreads();   // every wave is done reading the operand ring
  if (idle) return;
  uint2 hv[I][I];
#pragma unroll
  for (int i = 0; i < I; ++i)
#pragma unroll
    for (int j = 0; j < I; ++j) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = acc[i][j][e];
      if constexpr (poly) {
        const int R = row0 + rl0 + i * 16, C = col0 + cl0 + j * 16;
        const float a4[4] = {bf16_lo(av[i][j].x), bf16_hi(av[i][j].x), bf16_lo(av[i][j].y), bf16_hi(av[i][j].y)};
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = args.b * a4[e] + args.c * v[e] + (R + e == C ? args.a : 0.f);
      }
      hv[i][j].x = pack_bf16x2(sc * v[0], sc * v[1]);
      hv[i][j].y = pack_bf16x2(sc * v[2], sc * v[3]);
      if (lo_off) {
        acc[i][j][0] = v[0] - bf16_lo(hv[i][j].x);
        acc[i][j][1] = v[1] - bf16_hi(hv[i][j].x);
        acc[i][j][2] = v[2] - bf16_lo(hv[i][j].y);
        acc[i][j][3] = v[3] - bf16_hi(hv[i][j].y);
      }
    }
  const int p = lane & 3;
  char* const wreg = lds + wave * WREG;
  // Each wave moves its own sub-tile through a private region: transposed to
  // the mirror place, then as is.  A sub-tile on the block diagonal equals its
  // transpose and leaves once.
  auto emit = [&](int off) {
    constexpr int CH = WT * 2 / 16;   // 16-byte pieces per row
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
      for (int j = 0; j < I; ++j)
        *reinterpret_cast<uint2*>(wreg + ((lane & 15) + j * 16) * PITCH_T + (4 * (lane >> 4) + i * 16) * 2) = hv[i][j];
#pragma unroll
    for (int it = 0; it < WT * CH / 64; ++it) {
      const int q = lane + 64 * it, r = q / CH, ch = q % CH;
      const u32x4 v = *reinterpret_cast<const u32x4*>(wreg + r * PITCH_T + ch * 16);
      *reinterpret_cast<MALT_GLOBAL u32x4*>(gptr(out) + (size_t)(col0 + wc * WT + r) * ldo + off + row0 + wr * WT +
                                            ch * 8) = v;
    }
    if (diag && wr == wc) return;
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
      for (int j = 0; j < I; ++j)
        *reinterpret_cast<uint2*>(wreg + (4 * (lane >> 4) + i * 16 + p) * PITCH_R + (j * 16 + ((lane & 15) & ~3)) * 2) =
            quad_transpose(hv[i][j], p);
#pragma unroll
    for (int it = 0; it < WT * CH / 64; ++it) {
      const int q = lane + 64 * it, r = q / CH, ch = q % CH;
      const char* src = wreg + r * PITCH_R + ch * 16;
      const uint2 lo = *reinterpret_cast<const uint2*>(src);
      const uint2 hi = *reinterpret_cast<const uint2*>(src + 8);
      const u32x4 v = {lo.x, lo.y, hi.x, hi.y};
      *reinterpret_cast<MALT_GLOBAL u32x4*>(gptr(out) + (size_t)(row0 + wr * WT + r) * ldo + off + col0 + wc * WT +
                                            ch * 8) = v;
    }
  };
  emit(0);
  if (lo_off) {
#pragma unroll
    for (int i = 0; i < I; ++i)
#pragma unroll
      for (int j = 0; j < I; ++j) {
        hv[i][j].x = pack_bf16x2(acc[i][j][0], acc[i][j][1]);
        hv[i][j].y = pack_bf16x2(acc[i][j][2], acc[i][j][3]);
      }
    emit(lo_off);
  }
}

// Adds the partial tiles of a Gram cut along k, in split order, scales, rounds
// and writes the tile and its mirror.  Tile list (mat, ti, tj, 16-row piece of
// the transposed tile).
template <int T>
__global__ __launch_bounds__(RED_THREADS) void ns_mid_reduce_kernel(NsArgs args) {
  constexpr int V = 16 * T / (RED_THREADS * 4);   // float4 per thread
  constexpr int TPR = T / 4;                      // threads per row
  __shared__ bf16_t tr[T][16 + 4];
  const Tile t = args.tiles[blockIdx.x];
  const MatDesc* __restrict__ d = args.desc + t.mat;
  const int mp = d->mp, S = d->gsplit;
  const float sig = args.first ? (float)d->scal[SC_SIGMA] : 1.f;
  const float sc = sig * sig;
  MALT_GLOBAL bf16_t* const A = gptr(d->A);
  const MALT_GLOBAL float* src = gptr(reinterpret_cast<const float*>(d->X[args.src ^ 1])) +
                                 mid_part(t.ti, t.tj, 0, d->dm / T, S, T) + t.idx * 16 * T;
  const int row0 = t.ti * T, col0 = t.tj * T + t.idx * 16;
  const bool diag = t.ti == t.tj;
  f32x4 s[V];
#pragma unroll
  for (int v = 0; v < V; ++v) s[v] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int k = 0; k < S; ++k)
#pragma unroll
    for (int v = 0; v < V; ++v)
      s[v] += *reinterpret_cast<const MALT_GLOBAL f32x4*>(src + (size_t)k * T * T + (threadIdx.x + v * RED_THREADS) * 4);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int q = threadIdx.x + v * RED_THREADS, c = q / TPR, r = (q % TPR) * 4;
    const uint2 pk = make_uint2(pack_bf16x2(sc * s[v][0], sc * s[v][1]), pack_bf16x2(sc * s[v][2], sc * s[v][3]));
    // A diagonal tile holds its 16 x 16 blocks with row block <= column block.
    if (!diag || r / 16 <= t.idx)
      *reinterpret_cast<MALT_GLOBAL uint64_t*>(A + (size_t)(col0 + c) * mp + row0 + r) = __builtin_bit_cast(uint64_t, pk);
    tr[r][c] = (bf16_t)(pk.x & 0xffffu);
    tr[r + 1][c] = (bf16_t)(pk.x >> 16);
    tr[r + 2][c] = (bf16_t)(pk.y & 0xffffu);
    tr[r + 3][c] = (bf16_t)(pk.y >> 16);
  }
  __syncthreads();
  // Mirror: row row0 + r, columns col0 .. + 15 (two 16-byte pieces).
  for (int q = threadIdx.x; q < T * 2; q += RED_THREADS) {
    const int r = q >> 1, h = (q & 1) * 8;
    if (diag && r / 16 >= t.idx) continue;
    const uint2 lo = *reinterpret_cast<const uint2*>(&tr[r][h]);
    const uint2 hi = *reinterpret_cast<const uint2*>(&tr[r][h + 4]);
    const u32x4 v = {lo.x, lo.y, hi.x, hi.y};
    *reinterpret_cast<MALT_GLOBAL u32x4*>(A + (size_t)(row0 + r) * mp + col0 + h) = v;
  }
}

// Update tile (see ns_update.hip for the operand and output layouts).
template <int T>
__global__ __launch_bounds__(MidGeom<T>::NT) __attribute__((amdgpu_waves_per_eu(MidGeom<T>::WPE, MidGeom<T>::WPE)))
void ns_mid_update_kernel(NsArgs args) {
  using G = MidGeom<T>;
  using ML = MidLoads<T>;
  constexpr int WT = G::WT, N = WT / 16, NL = G::LOADS, H = G::H, RB = G::RB;
  constexpr int PITCH = WT * 2 + 8, WREG = WT * PITCH;
  static_assert(G::NW * WREG + 2 * G::NW * 4 <= G::RING_BYTES, "epilogue copies fit the ring");
  __shared__ __attribute__((aligned(16))) char lds[G::RING_BYTES];

  const Tile t = args.tiles[blockIdx.x];
  if (t.mat < 0) return;
  const MatDesc* __restrict__ d = args.desc + t.mat;
  const int mp = d->mp, np = d->np, dm = d->dm, mc = d->mc, nc = d->nc;
  const bool tall = d->tall != 0;
  const int ldb = d->split ? 2 * mp : mp;
  const int KH = dm / G::BK, KT = d->split ? 2 * KH : KH;
  bf16_t* const Xn = d->X[args.src ^ 1];
  const float* const Lm = tall ? d->Rv : d->Lv;   // factor indexed by the canonical row
  const float* const Ln = tall ? d->Lv : d->Rv;   // factor indexed by the canonical column
  float* const gpart = d->gpart;
  const float sc = args.first ? (float)d->scal[SC_SIGMA] : 1.f;
  const int row0 = t.ti * T, col0 = t.tj * T;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 1, wc = wave & 1;

  const i32x4 rsB = buf_rsrc(d->B);
  const i32x4 rsX = buf_rsrc(d->X[args.src]);
  uint32_t voff[NL];
  int dst_off[NL];
#pragma unroll
  for (int q = 0; q < NL; ++q) {
    const int o = q / (NL / 2), g = wave + (q % (NL / 2)) * G::NW;
    voff[q] = (uint32_t)(o ? ML::voff_kn(g, lane, col0, np) : ML::voff_rk(g, lane, row0, ldb));
    dst_off[q] = o * G::OPER_BYTES + g * 1024;
  }
  int offb[H], offx[N][2];
#pragma unroll
  for (int h = 0; h < H; ++h) offb[h] = G::swz_rk(wr * WT + (lane & 15), 4 * h + (lane >> 4));
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int r2 = 0; r2 < 2; ++r2)
      offx[a][r2] = G::OPER_BYTES +
                    G::swz_kn(8 * (lane >> 4) + 4 * r2 + ((lane & 15) >> 2), wc * WT + a * 16 + 4 * (lane & 3));

  f32x4 acc[N][N];
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[a][b][e] = 0.f;
  bf16x8 fx[2][N], fb[2][N];
  // Reads per sub-step: N of B' and 2 N transposed ones of X, against N * N MFMAs.
  constexpr int RPM = 3 * N > N * N ? 2 : 1;
  mid_pipeline<G, RPM>(
      KT, NL, lds,
      [&](int kt, char* st, int q) {
        const uint32_t la = lds_u32(st + dst_off[q]);
        if (q < NL / 2) dma16(rsB, voff[q], (uint32_t)ML::soff_b(kt, KH, mp), la);
        else dma16(rsX, voff[q], (uint32_t)ML::soff_x(kt, KH, np), la);
      },
      [&](int buf, const char* st, int h) {
#pragma unroll
        for (int b = 0; b < N; ++b) fb[buf][b] = *reinterpret_cast<const bf16x8*>(st + offb[h] + b * 16 * RB);
#pragma unroll
        for (int a = 0; a < N; ++a) {
          const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(st + offx[a][0] + h * 32 * T * 2));
          const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(st + offx[a][1] + h * 32 * T * 2));
          fx[buf][a] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
      },
      [&](int buf, auto&& after) {
#pragma unroll
        for (int a = 0; a < N; ++a)
#pragma unroll
          for (int b = 0; b < N; ++b) {
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx[buf][a], fb[buf][b], acc[a][b], 0, 0, 0);
            after(a * N + b);
          }
      });

  // ---------------------------------------------------------------- epilogue
  // acc[a][b][e] = C(m, n + e), m = wr*WT + 16 b + (lane & 15),
  // n = wc*WT + 16 a + 4 (lane >> 4).
  const int sr0 = lane & 15, sc0 = 4 * (lane >> 4);
  char* const sto = lds + wave * WREG;
  __syncthreads();   // every wave is done reading the operand ring
  float o2 = 0.f, d2 = 0.f;
#pragma unroll
  for (int a = 0; a < N; ++a) {
    const int n = col0 + wc * WT + sc0 + a * 16;
    float ln2[4];
    if (args.last) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float l = n + e < nc ? gptr(Ln)[n + e] : 0.f;
        ln2[e] = l * l;
      }
    }
#pragma unroll
    for (int b = 0; b < N; ++b) {
      uint2 pk;
      pk.x = pack_bf16x2(sc * acc[a][b][0], sc * acc[a][b][1]);
      pk.y = pack_bf16x2(sc * acc[a][b][2], sc * acc[a][b][3]);
      *reinterpret_cast<uint2*>(sto + (sr0 + b * 16) * PITCH + (sc0 + a * 16) * 2) = pk;
      if (args.last) {
        // Sums of O^2 and (L O R)^2 from the rounded O.
        const int m = row0 + wr * WT + sr0 + b * 16;
        const float ov[4] = {bf16_lo(pk.x), bf16_hi(pk.x), bf16_lo(pk.y), bf16_hi(pk.y)};
        float rowo = 0.f, rowd = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float q = (n + e < nc) ? ov[e] * ov[e] : 0.f;
          rowo += q;
          rowd += ln2[e] * q;
        }
        if (m < mc) {
          const float l = gptr(Lm)[m];
          o2 += rowo;
          d2 += l * l * rowd;
        }
      }
    }
  }
  constexpr int CH = WT * 2 / 16;
#pragma unroll
  for (int it = 0; it < WT * CH / 64; ++it) {
    const int q = lane + 64 * it, r = q / CH, ch = q % CH;
    const char* src = sto + r * PITCH + ch * 16;
    const uint2 lo = *reinterpret_cast<const uint2*>(src);
    const uint2 hi = *reinterpret_cast<const uint2*>(src + 8);
    const u32x4 v = {lo.x, lo.y, hi.x, hi.y};
    *reinterpret_cast<MALT_GLOBAL u32x4*>(gptr(Xn) + (size_t)(row0 + wr * WT + r) * np + col0 + wc * WT + ch * 8) = v;
  }
  if (!args.last) return;
  float* red = reinterpret_cast<float*>(lds + G::NW * WREG);
  o2 = wsum(o2);
  d2 = wsum(d2);
  if (lane == 0) {
    red[wave] = o2;
    red[G::NW + wave] = d2;
  }
  __syncthreads();
  if (tid == 0) {
    float so = 0.f, sd = 0.f;
#pragma unroll
    for (int w = 0; w < G::NW; ++w) {
      so += red[w];
      sd += red[G::NW + w];
    }
    gptr(gpart)[2 * (size_t)t.idx + 0] = so;
    gptr(gpart)[2 * (size_t)t.idx + 1] = sd;
  }
}

template <int T>
hipError_t launch_mid(const NsArgs& a, hipStream_t s) {
  using G = MidGeom<T>;
  const dim3 grid(a.ntiles);
  if (a.phase == PH_GRAM)
    hipLaunchKernelGGL((ns_mid_sym_kernel<T, PH_GRAM>), grid, dim3(G::NT), 0, s, a);
  else if (a.phase == PH_POLY)
    hipLaunchKernelGGL((ns_mid_sym_kernel<T, PH_POLY>), grid, dim3(G::NT), 0, s, a);
  else if (a.phase == PH_UPDATE)
    hipLaunchKernelGGL((ns_mid_update_kernel<T>), grid, dim3(G::NT), 0, s, a);
  else
    hipLaunchKernelGGL((ns_mid_reduce_kernel<T>), grid, dim3(RED_THREADS), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_ns_mid(const NsArgs& a, int tile, hipStream_t s) {
  if (a.ntiles == 0) return hipSuccess;
  if (tile == 64) return launch_mid<64>(a, s);
  if (tile == 128) return launch_mid<128>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace malt
