// Complex GEMMs on pre-split operands for the reduced-precision inner
// solves: split-BF16 (below) and FP32 Gauss planes (after it).
//
// Split-BF16.
// Every real component x of a complex128 operand is split into bf16 numbers,
// hi = bf16(x) and lo = bf16(x - hi), so x = hi + lo to about 2^-17
// relative.  A real product of two split operands is formed from three bf16
// MFMA products, hi*hi + hi*lo + lo*hi (the lo*lo term is below the split's
// own error; CCLR_BF16X3), or, with the second operand kept as hi only, from
// two, hi*hi + lo*hi (CCLR_BF16X2: the second operand then carries bf16
// rounding, about 2^-9 relative, which the FP64 refinement of the solver
// absorbs).  Products accumulate in FP32 on v_mfma_f32_16x16x32_bf16.
//
// A complex block takes three accumulators holding Ar Br, Ai Bi and
// Ar Bi + Ai Br, so Re = acc0 - acc1 and Im = acc2: twelve (X3) or eight (X2)
// bf16 MFMAs per complex block.  (Gauss's three-product form would save a
// quarter of the MFMAs but needs the (re + im) planes too, 1.5 times the
// operand traffic through LDS, which the kernel cannot afford: LDS reads and
// the direct loads already take about half of the MFMA time.)
//
// Operands are stored pre-split: a rows x K complex matrix becomes
// [K/32][rows_pad][4P] 16-byte chunks for P planes (re_hi, re_lo, im_hi,
// im_lo, or re_hi, im_hi).  Logical chunk c = 4p + g of row r holds the eight
// bf16 values k = 32 kc + 8 g ... + 7 of plane p and is stored at position
// c ^ sw(r) of the row, sw(r) = r mod 16 (P = 4) or (r / 2) mod 8 (P = 2):
// the MFMA operand reads (one chunk of 16 consecutive rows per 16 lanes) then
// fall in 16 different 16-byte bank groups.  Rows are padded to the 128-row
// tile and K to the MFMA's 32 with zeros.  One tile of one k step is
// contiguous and a multiple of 256 chunks, so it is copied into LDS by
// direct global-to-LDS loads, every lane active (no registers, no LDS store
// instructions, no branches in the loop).  The Jacobian's ladder and ring
// operators are split once per set of amplitudes and kept; the trial vectors
// are split per product.
#include <algorithm>

#include "internal.h"

namespace {
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned u4v __attribute__((ext_vector_type(4)));

constexpr int TN = 128;  // tile columns, and row padding of the B side

// plane codes of a split operand
enum { P_RH = 0, P_RL, P_IH, P_IL };

// The two kernel forms: planes of the A and B operands and the MFMA list
// (A plane, B plane, accumulator), small terms first, ordered so that
// consecutive MFMAs go to different accumulators.
struct FormDesc {
  int pa, pb;  // planes per operand
  int planes_a[4], planes_b[4];
  int nprod;
  int prod[12][3];
};
constexpr FormDesc kForms[2] = {
    // X3: both operands split, 12 MFMAs per complex block
    {4, 4, {P_RH, P_RL, P_IH, P_IL}, {P_RH, P_RL, P_IH, P_IL}, 12,
     {{1, 0, 0}, {3, 2, 1}, {1, 2, 2}, {0, 1, 0}, {2, 3, 1}, {3, 0, 2},
      {0, 0, 0}, {2, 2, 1}, {0, 3, 2}, {0, 2, 2}, {2, 1, 2}, {2, 0, 2}}},
    // X2: B planes re_hi, im_hi; 8 MFMAs per complex block
    {4, 2, {P_RH, P_RL, P_IH, P_IL}, {P_RH, P_IH}, 8,
     {{1, 0, 0}, {3, 1, 1}, {1, 1, 2}, {0, 0, 0}, {2, 1, 1}, {3, 0, 2}, {0, 1, 2}, {2, 0, 2}}},
};

// position of logical chunk c in row r of a split operand with P planes
__host__ __device__ constexpr int swz(int P, int r, int c) { return c ^ (P == 4 ? (r & 15) : ((r >> 1) & 7)); }

// round-to-nearest-even bf16 bits of a finite float
__device__ __forceinline__ unsigned bf16_bits(float x) {
  const unsigned u = __float_as_uint(x);
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// bits of plane `code` of the complex value (re, im)
__device__ __forceinline__ unsigned plane_bits(int code, double re, double im) {
  const double x = code < P_IH ? re : im;
  const unsigned hi = bf16_bits((float)x);
  if (!(code & 1)) return hi;
  return bf16_bits((float)(x - (double)__uint_as_float(hi << 16)));
}

// One thread reads eight k values of one row and writes their chunk in every
// plane.  Threads run along k when the source's unit stride is k, along rows
// otherwise, so the reads coalesce.
template <int P>
__global__ __launch_bounds__(256) void k_split(int rows, int K, const cplx* __restrict__ src, i64 sR, i64 sK,
                                               int conj, u4v* __restrict__ dst, int rows_pad, int nkc, int p0, int p1,
                                               int p2, int p3, int rows_fast) {
  const int code[4] = {p0, p1, p2, p3};
  const i64 units = (i64)rows_pad * nkc * 4;
  const double si = conj ? -1.0 : 1.0;
  for (i64 u = blockIdx.x * (i64)blockDim.x + threadIdx.x; u < units; u += (i64)gridDim.x * blockDim.x) {
    i64 r, kc;
    int g;
    if (rows_fast) {
      r = u % rows_pad;
      const i64 q = u / rows_pad;
      g = (int)(q & 3);
      kc = q >> 2;
    } else {
      g = (int)(u & 3);
      const i64 q = u >> 2;
      r = q % rows_pad;
      kc = q / rows_pad;
    }
    cplx x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const i64 k = kc * 32 + g * 8 + e;
      x[e] = (r < rows && k < K) ? src[r * sR + k * sK] : make_double2(0.0, 0.0);
      x[e].y *= si;
    }
    u4v* o = dst + (kc * rows_pad + r) * (4 * P);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      u4v w;
#pragma unroll
      for (int e = 0; e < 8; e += 2)
        w[e >> 1] = plane_bits(code[p], x[e].x, x[e].y) | (plane_bits(code[p], x[e + 1].x, x[e + 1].y) << 16);
      o[swz(P, (int)r, 4 * p + g)] = w;
    }
  }
}

__device__ __forceinline__ bf8 as_bf8(u4v x) { return __builtin_bit_cast(bf8, x); }

#define MF(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0)

// Copy CH contiguous 16-byte chunks (a multiple of 64) from global memory
// into LDS with direct loads; each wave instruction moves 64 consecutive chunks.
template <int NT, int CH>
__device__ __forceinline__ void dma_tile(const u4v* __restrict__ g, u4v* lds, int tid) {
  static_assert(CH % 64 == 0, "tile must be a whole number of wave loads");
#pragma unroll
  for (int e0 = 0; e0 < CH; e0 += NT) {
    if (e0 + NT > CH && e0 + (tid & ~63) >= CH) break;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(g + e0 + tid),
                                     (__attribute__((address_space(3))) void*)(lds + e0 + (tid & ~63)), 16, 0, 0);
  }
}

// The workgroups of one XCD (hardware index modulo 8) take consecutive
// positions of the work order.
__device__ __forceinline__ int xcd_position(int w, int n) {
  const int x = w & 7, l = w >> 3, per = n >> 3, rem = n & 7;
  return (x < rem ? x * (per + 1) : rem * (per + 1) + (x - rem) * per) + l;
}

// Deals a product to this workgroup: its whole tiles first, then its run over
// the k steps of the cut ones (at most nk steps, so at most two tiles).
// seg(tile, first step, end, slot): slot < 0 a whole tile, else partial sums
// to that slot of the workspace.
template <class Seg>
__device__ __forceinline__ void deal(const SplitPlan& p, const Seg& seg) {
  const int pos = xcd_position((int)blockIdx.x, (int)gridDim.x);
  const i64 total = (p.tiles - p.whole) * p.nk;
  i64 t = pos, it = 0, end = 0;
  if (pos < p.cutters) {
    it = (i64)pos * total / p.cutters;
    end = (i64)(pos + 1) * total / p.cutters;
  }
  i64 slot = 2 * (i64)pos;
  while (t < p.whole || it < end) {
    i64 tile = t, to = -1;
    int k0 = 0, k1 = p.nk;
    if (t < p.whole) {
      t += gridDim.x;
    } else {
      const i64 c = it / p.nk;
      tile = p.whole + c;
      k0 = (int)(it - c * p.nk);
      k1 = (int)min((i64)p.nk, k0 + (end - it));
      if (k0 > 0 || k1 < p.nk) to = slot;
      ++slot;
      it += k1 - k0;
    }
    seg(tile, k0, k1, to);
  }
}

__device__ __forceinline__ void put(cplx* dst, double xr, double xi, double ar, double ai, int beta) {
  cplx y = make_double2(ar * xr - ai * xi, ar * xi + ai * xr);
  if (beta) {
    const cplx o = *dst;
    y.x += o.x;
    y.y += o.y;
  }
  *dst = y;
}

// the accumulators of a cut tile's run, as they are: 16 bytes a lane, fragment
// after fragment ([accumulator][i][j][thread of 512][row of 4]), so that the
// stores of a wave and the loads of k_split_join are whole lines (4-byte
// stores into rows: 4 to 13 us more, 264x4005x4005 in X3 103 us against 95)
template <int FM, int FN>
__device__ __forceinline__ void keep(float* __restrict__ W, i64 slot, const f4 (&acc)[3][FM][FN]) {
  f4* w = (f4*)W + slot * (3 * FM * FN * 512) + threadIdx.x;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) w[((a * FM + i) * FN + j) * 512] = acc[a][i][j];
}

// C[m][n] (+)= alpha * sum_k A[m][k] B[n][k] on split operands.  BM x 128
// tile per workgroup of eight waves (2 x 4, each BM/2 x 32 in 16x16 MFMA
// blocks; two waves per SIMD, which hide each other's LDS and barrier
// waits: about 1.2 times faster than four waves of 64 x 64 with one wave per
// SIMD), double-buffered LDS filled by direct loads one k step ahead: each
// step requests the next step's tiles into the other stage, then reads its
// operand fragments and runs its MFMAs while the loads are in flight; the
// wait for the loads and the barrier come before the MFMAs of its last row
// block, whose time covers the reads of the next step's first fragments
// (3-5% faster than a barrier after the last MFMA).  The
// stages are separate LDS arrays, so the compiler does not make the reads of
// one wait for the direct loads into the other.
//
// The LDS holds one workgroup per compute unit.  A solve's transforms have
// few tiles (a ladder of four vectors at o = 12, v = 90 is 264 x 4005: 96 of
// 128 x 128, padded by 45%): then 256 workgroups take whole tiles while those
// fill all of them and equal runs of the k steps of the others (deal), and
// k_split_join adds the partial sums.  Products that gain nothing from that
// run one workgroup per tile, the XCDs on contiguous ranges of tiles, m
// fastest, so that the B tile of a step is shared in an XCD's L2: a ring of 12
// vectors, 48000x4000x4000, 13.1 ms in X3 and 9.7 in X2 (14.3 and 11.5 on 256
// workgroups in rounds).  BM is 64, 96 or 128, by estimated time (split_plan).
// Bound by the bf16 MFMAs (1.28 us of a
// 128-row k step; 1.5 to 2.0 measured, by how many compute units compete for
// the operands).  Against whole 128 x 128 tiles, X3, us: 264x4005x4005 103 / 218,
// 66x4005x4005 50 / 205, 1080x1080x1080 42 / 62, 4320x1080x1080 110 / 138,
// 570x19900x19900 3920 / 4900.
template <int F, int BM>
__global__ __launch_bounds__(512) void k_cgemm_bf16s(const u4v* __restrict__ As, const u4v* __restrict__ Bs,
                                                     int Mpad, int Npad, int M, int N, cplx* __restrict__ C, i64 sCm,
                                                     i64 sCn, double ar, double ai, int beta, SplitPlan p,
                                                     float* __restrict__ W) {
  constexpr FormDesc D = kForms[F];
  constexpr int PA = D.pa, PB = D.pb;
  constexpr int RSA = 4 * PA, RSB = 4 * PB;  // chunks per row
  constexpr int NT = 512;  // eight waves: two along m, four along n
  constexpr int WM = BM / 2, WN = TN / 4;
  constexpr int FM = WM / 16, FN = WN / 16;
  constexpr int CA = BM * RSA, CB = TN * RSB;  // chunks per tile and k step
  // the two stages in separate arrays, so the compiler can tell a read of
  // one stage from the direct loads into the other and does not make the
  // reads wait for the loads
  __shared__ u4v sA0[CA], sA1[CA];
  __shared__ u4v sB0[CB], sB1[CB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave & 1) * WM, wn = (wave >> 1) * WN;
  const int rr = lane & 15, g = lane >> 4;
  // LDS offsets of this lane's fragments (rows wm + 16 i + rr, wn + 16 j + rr;
  // the swizzle depends on the row only through rr)
  int offa[PA], offb[PB];
#pragma unroll
  for (int p = 0; p < PA; ++p) offa[p] = (wm + rr) * RSA + swz(PA, rr, 4 * p + g);
#pragma unroll
  for (int p = 0; p < PB; ++p) offb[p] = (wn + rr) * RSB + swz(PB, rr, 4 * p + g);
  auto segment = [&](i64 t, int k0, int k1, i64 slot) {
    const int m0 = (int)(t % p.tm) * BM, n0 = (int)(t / p.tm) * TN;
    auto fetch = [&](int kc, u4v* la, u4v* lb) {
      dma_tile<NT, CA>(As + ((i64)kc * Mpad + m0) * RSA, la, tid);
      dma_tile<NT, CB>(Bs + ((i64)kc * Npad + n0) * RSB, lb, tid);
    };
    f4 acc[3][FM][FN];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[a][i][j] = f4{0.f, 0.f, 0.f, 0.f};
    auto mfma_i = [&](int i, const bf8 (&a)[PA], const bf8 (&b)[FN][PB]) {
#pragma unroll
      for (int q = 0; q < D.nprod; ++q)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[D.prod[q][2]][i][j] = MF(a[D.prod[q][0]], b[j][D.prod[q][1]], acc[D.prod[q][2]][i][j]);
    };
    auto read_b = [&](const u4v* cb, bf8 (&b)[FN][PB]) {
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int p = 0; p < PB; ++p) b[j][p] = as_bf8(cb[offb[p] + 16 * j * RSB]);
    };
    auto read_a = [&](const u4v* ca, int i, bf8 (&a)[PA]) {
#pragma unroll
      for (int p = 0; p < PA; ++p) a[p] = as_bf8(ca[offa[p] + 16 * i * RSA]);
    };
    bf8 bq[FN][PB], aq[PA];  // the first fragments of the next step, read ahead
    // one k step on the stage (ca, cb) while the next step's tiles load into (na, nb)
    auto step = [&](int kc, const u4v* ca, const u4v* cb, u4v* na, u4v* nb) {
      // the last step reloads its own tiles into the idle stage (no branch)
      fetch(kc + 1 < k1 ? kc + 1 : kc, na, nb);
      __builtin_amdgcn_sched_barrier(0);  // the loads are requested first, not scheduled between the MFMAs
      // the wait and the barrier come once the last fragments of this stage
      // are read; the next stage's first fragments are read while the MFMAs
      // of the last row block run
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        bf8 a[PA];
        if (i == 0) {
#pragma unroll
          for (int p = 0; p < PA; ++p) a[p] = aq[p];
        } else {
          read_a(ca, i, a);
        }
        if (i + 1 < FM) {
          mfma_i(i, a, bq);
        } else {
          bf8 bn[FN][PB], an[PA];
          __builtin_amdgcn_sched_barrier(0);
          __builtin_amdgcn_s_waitcnt(0);
          __syncthreads();
          read_b(nb, bn);
          read_a(na, 0, an);
          mfma_i(i, a, bq);
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int p = 0; p < PB; ++p) bq[j][p] = bn[j][p];
#pragma unroll
          for (int p = 0; p < PA; ++p) aq[p] = an[p];
        }
      }
    };
    __syncthreads();  // every wave is done with the stages of the previous segment
    fetch(k0, sA0, sB0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    read_b(sB0, bq);
    read_a(sA0, 0, aq);
    for (int kc = k0; kc < k1; kc += 2) {
      step(kc, sA0, sB0, sA1, sB1);
      if (kc + 1 < k1) step(kc + 1, sA1, sB1, sA0, sB0);
    }
    if (slot >= 0) {
      keep(W, slot, acc);
      return;
    }
    // output block (i, j): row 16i + 4*(lane/16) + r, column 16j + lane%16
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + wm + 16 * i + 4 * g + r, n = n0 + wn + 16 * j + rr;
          const double xr = (double)acc[0][i][j][r] - (double)acc[1][i][j][r], xi = (double)acc[2][i][j][r];
          if (m < M && n < N) put(C + (i64)m * sCm + (i64)n * sCn, xr, xi, ar, ai, beta);
        }
  };
  deal(p, segment);
}
#undef MF

// ---------------------------------------------------------------- FP32 form
// Three real products per complex block (Gauss): k1 = (Ar + Ai) Br,
// k2 = Ar (Bi - Br), k3 = Ai (Br + Bi), Re = k1 - k3, Im = k1 + k2, on
// v_mfma_f32_16x16x4f32 with FP32 accumulation.  Split layout: [K/16][rows_pad]
// [12] 16-byte chunks; logical chunk c = 4p + g of a row holds the four FP32
// values k = 16 kb + 4g ... + 3 of plane p (A: Ar + Ai, Ar, Ai; B: Br,
// Bi - Br, Br + Bi), stored at position (c + (r / 4) mod 4) mod 12, which
// puts one chunk of 16 consecutive rows in 16 different bank groups.  A lane
// reads its four k values with one 16-byte read and feeds them to the four
// MFMAs of the k-step (lane group g takes k = 4g + s in MFMA s: the k order
// within the step is the same on both operands, so the sum is unchanged).
__host__ __device__ constexpr int f32pos(int r, int c) { return (c + ((r >> 2) & 3)) % 12; }

__global__ __launch_bounds__(256) void k_split_f32(int rows, int K, const cplx* __restrict__ src, i64 sR, i64 sK,
                                                   int conj, int side, u4v* __restrict__ dst, int rows_pad, int nkb,
                                                   int rows_fast) {
  const i64 units = (i64)rows_pad * nkb * 4;
  const double si = conj ? -1.0 : 1.0;
  for (i64 u = blockIdx.x * (i64)blockDim.x + threadIdx.x; u < units; u += (i64)gridDim.x * blockDim.x) {
    i64 r, kb;
    int g;
    if (rows_fast) {
      r = u % rows_pad;
      const i64 q = u / rows_pad;
      g = (int)(q & 3);
      kb = q >> 2;
    } else {
      g = (int)(u & 3);
      const i64 q = u >> 2;
      r = q % rows_pad;
      kb = q / rows_pad;
    }
    float pl[3][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const i64 k = kb * 16 + g * 4 + e;
      cplx x = (r < rows && k < K) ? src[r * sR + k * sK] : make_double2(0.0, 0.0);
      const double re = x.x, im = si * x.y;
      if (side == 0) {
        pl[0][e] = (float)(re + im);
        pl[1][e] = (float)re;
        pl[2][e] = (float)im;
      } else {
        pl[0][e] = (float)re;
        pl[1][e] = (float)(im - re);
        pl[2][e] = (float)(re + im);
      }
    }
    u4v* o = dst + (kb * rows_pad + r) * 12;
#pragma unroll
    for (int p = 0; p < 3; ++p)
      o[f32pos((int)r, 4 * p + g)] =
          u4v{__float_as_uint(pl[p][0]), __float_as_uint(pl[p][1]), __float_as_uint(pl[p][2]), __float_as_uint(pl[p][3])};
  }
}

// C[m][n] (+)= alpha * sum_k A[m][k] B[n][k] on FP32 split operands: the
// pipeline and the even split of k_cgemm_bf16s (BM x 128 tiles of eight
// BM/2 x 32 waves, direct loads one 16-deep k step ahead into the other of
// two LDS stages).  Without cut tiles the 128-row kernel takes one tile and no
// loop over tiles (CUT = false), which spares it registers: 2280x19900x19900
// 39.5 ms, 41.5 with the loop (the bf16 forms are the same with and without).
// One workgroup per compute unit by the attribute: with 64 rows the registers
// would do for two, which is slower (3240x1080x1080 250 us, 216).
// Against whole 128 x 128 tiles, us: 264x4005x4005 289 / 740, 4320x1080x1080
// 300 / 411, 570x19900x19900 11630 / 14700.
template <int BM, bool CUT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_cgemm_f32s(
    const u4v* __restrict__ As, const u4v* __restrict__ Bs, int Mpad, int Npad, int M, int N,
    cplx* __restrict__ C, i64 sCm, i64 sCn, double ar, double ai, int beta, SplitPlan p, float* __restrict__ W) {
  constexpr int RS = 12, NT = 512, WM = BM / 2, WN = TN / 4, FM = WM / 16, FN = WN / 16;
  constexpr int CA = BM * RS, CB = TN * RS;  // chunks per tile and k step
  __shared__ u4v sA0[CA], sA1[CA];
  __shared__ u4v sB0[CB], sB1[CB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave & 1) * WM, wn = (wave >> 1) * WN;
  const int rr = lane & 15, g = lane >> 4;
  // the rotation depends on the row only through rr (wm, wn and 16 i are multiples of 16)
  int off[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) off[p] = rr * RS + f32pos(rr, 4 * p + g);
  auto segment = [&](i64 t, int k0, int k1, i64 slot) {
    const int m0 = (int)(t % p.tm) * BM, n0 = (int)(t / p.tm) * TN;
    auto fetch = [&](int kb, u4v* la, u4v* lb) {
      dma_tile<NT, CA>(As + ((i64)kb * Mpad + m0) * RS, la, tid);
      dma_tile<NT, CB>(Bs + ((i64)kb * Npad + n0) * RS, lb, tid);
    };
    f4 acc[3][FM][FN];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[a][i][j] = f4{0.f, 0.f, 0.f, 0.f};
    auto mfma_i = [&](int i, const f4 (&a)[3], const f4 (&b)[FN][3]) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[p][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[p][s], b[j][p][s], acc[p][i][j], 0, 0, 0);
    };
    auto read_b = [&](const u4v* cb, f4 (&b)[FN][3]) {
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int p = 0; p < 3; ++p) b[j][p] = __builtin_bit_cast(f4, cb[(wn + 16 * j) * RS + off[p]]);
    };
    auto read_a = [&](const u4v* ca, int i, f4 (&a)[3]) {
#pragma unroll
      for (int p = 0; p < 3; ++p) a[p] = __builtin_bit_cast(f4, ca[(wm + 16 * i) * RS + off[p]]);
    };
    f4 bq[FN][3], aq[3];  // the first fragments of the next step, read ahead
    auto step = [&](int kb, const u4v* ca, const u4v* cb, u4v* na, u4v* nb) {
      fetch(kb + 1 < k1 ? kb + 1 : kb, na, nb);
      __builtin_amdgcn_sched_barrier(0);  // the loads are requested first, not scheduled between the MFMAs
      // as in the split-BF16 kernel: wait and barrier before the last row block's MFMAs
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        f4 a[3];
        if (i == 0) {
#pragma unroll
          for (int p = 0; p < 3; ++p) a[p] = aq[p];
        } else {
          read_a(ca, i, a);
        }
        if (i + 1 < FM) {
          mfma_i(i, a, bq);
        } else {
          f4 bn[FN][3], an[3];
          __builtin_amdgcn_sched_barrier(0);
          __builtin_amdgcn_s_waitcnt(0);
          __syncthreads();
          read_b(nb, bn);
          read_a(na, 0, an);
          mfma_i(i, a, bq);
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int p = 0; p < 3; ++p) bq[j][p] = bn[j][p];
#pragma unroll
          for (int p = 0; p < 3; ++p) aq[p] = an[p];
        }
      }
    };
    if (CUT) __syncthreads();  // every wave is done with the stages of the previous segment
    fetch(k0, sA0, sB0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    read_b(sB0, bq);
    read_a(sA0, 0, aq);
    for (int kb = k0; kb < k1; kb += 2) {
      step(kb, sA0, sB0, sA1, sB1);
      if (kb + 1 < k1) step(kb + 1, sA1, sB1, sA0, sB0);
    }
    if (!CUT || slot < 0) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int m = wm + 16 * i + 4 * g + r, n = wn + 16 * j + rr;
            const double g1 = acc[0][i][j][r], g2 = acc[1][i][j][r], g3 = acc[2][i][j][r];
            if (m0 + m < M && n0 + n < N)
              put(C + (i64)(m0 + m) * sCm + (i64)(n0 + n) * sCn, g1 - g3, g1 + g2, ar, ai, beta);
          }
    } else {
      keep(W, slot, acc);
    }
  };
  if (CUT) deal(p, segment);
  else segment(xcd_position((int)blockIdx.x, (int)gridDim.x), 0, p.nk, -1);
}

// Adds the accumulators of the runs of cut tile whole + blockIdx.x in the order
// of k, in FP64, forms the result of them and stores it: four rows of one
// 16 x 16 block a thread, as the product's waves hold them, blockIdx.y which of
// a wave's blocks.
__global__ __launch_bounds__(512) void k_split_join(int M, int N, cplx* __restrict__ C, i64 sCm, i64 sCn, double ar,
                                                    double ai, int beta, SplitPlan p, int gauss,
                                                    const f4* __restrict__ W) {
  const i64 total = (p.tiles - p.whole) * p.nk, t = blockIdx.x;
  const i64 lo = t * p.nk, hi = lo + p.nk;
  // run c covers the k steps [c total / cutters, (c + 1) total / cutters): the runs with a part of [lo, hi)
  i64 c0 = lo * p.cutters / total;
  while ((c0 + 1) * total / p.cutters <= lo) ++c0;
  const i64 b0 = c0 * total / p.cutters;
  if (b0 <= lo && (c0 + 1) * total / p.cutters >= hi) return;  // in one run: stored whole
  i64 c1 = c0 + 1;
  while (c1 < p.cutters && c1 * total / p.cutters < hi) ++c1;
  const i64 tile = p.whole + t;
  constexpr int FN = TN / 4 / 16;
  const int blocks = p.bm / 32 * FN, size = blocks * 512;  // 16-byte entries of one accumulator
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = blockIdx.y / FN, j = blockIdx.y % FN;
  const int m0 = (int)(tile % p.tm) * p.bm + (wave & 1) * (p.bm / 2) + 16 * i + 4 * (lane >> 4);
  const int n = (int)(tile / p.tm) * TN + (wave >> 1) * (TN / 4) + 16 * j + (lane & 15);
  if (m0 >= M || n >= N) return;
  const int e = blockIdx.y * 512 + threadIdx.x;
  double x[3][4];
  {
    // the first run may have begun in the tile before: then this is its second piece
    const f4* w = W + 3 * (2 * c0 + (b0 < lo ? 1 : 0)) * size + e;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const f4 v = w[q * size];
#pragma unroll
      for (int r = 0; r < 4; ++r) x[q][r] = v[r];
    }
  }
  constexpr int U = 4;
  for (i64 c = c0 + 1; c < c1; c += U) {
    f4 w[U][3];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < 3; ++q) w[u][q] = c + u < c1 ? W[(6 * (c + u) + q) * size + e] : f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) x[q][r] += (double)w[u][q][r];
  }
  // split-BF16: Ar Br, Ai Bi, Ar Bi + Ai Br; FP32: k1, k2, k3 of Gauss's form
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (m0 + r >= M) break;
    const double xr = x[0][r] - (gauss ? x[2][r] : x[1][r]), xi = gauss ? x[0][r] + x[1][r] : x[2][r];
    put(C + (i64)(m0 + r) * sCm + (i64)n * sCn, xr, xi, ar, ai, beta);
  }
}

template <int P>
void launch_split_p(const SplitMat& s, const cplx* src, i64 sR, i64 sK, int conj, hipStream_t st) {
  const i64 units = (i64)s.rows_pad * s.nkc * 4;
  i64 grid = (units + 255) / 256;
  if (grid > 65536) grid = 65536;
  const int* c = s.planes;
  hipLaunchKernelGGL(k_split<P>, dim3((unsigned)grid), dim3(256), 0, st, s.rows, s.K, src, sR, sK, conj,
                     (u4v*)s.p, s.rows_pad, s.nkc, c[0], c[1], c[2], c[3], sR == 1 ? 1 : 0);
}
}  // namespace

bool split_form_valid(int form) { return form == BF16_X3 || form == BF16_X2 || form == F32_G3; }

int split_form_of(int prec) { return prec == CCLR_FP32 ? F32_G3 : prec == CCLR_BF16X2 ? BF16_X2 : BF16_X3; }

SplitMat split_shape(int rows, int K, int form, int side, int tile) {
  REQUIRE(split_form_valid(form), CCLR_EINVAL, "split: unknown form");
  SplitMat s;
  s.rows = rows;
  s.K = K;
  s.rows_pad = (rows + tile - 1) / tile * tile;
  s.form = form;
  s.side = side;
  if (form == F32_G3) {
    s.nkc = (K + 15) / 16;
    s.nplanes = 3;
    s.chunks = 12;
    return s;
  }
  const FormDesc& d = kForms[form];
  s.nkc = (K + 31) / 32;
  s.nplanes = side == 0 ? d.pa : d.pb;
  s.chunks = 4 * s.nplanes;
  for (int p = 0; p < 4; ++p) s.planes[p] = p < s.nplanes ? (side == 0 ? d.planes_a[p] : d.planes_b[p]) : 0;
  return s;
}

size_t split_bytes(int rows, int K, int form, int side, int tile) {
  const SplitMat s = split_shape(rows, K, form, side, tile);
  return (size_t)s.rows_pad * (size_t)s.nkc * (size_t)s.chunks * 16;
}

SplitMat launch_split(int rows, int K, const cplx* src, i64 sR, i64 sK, int conj, void* dst, int form, int side,
                      hipStream_t st, int tile) {
  REQUIRE(rows > 0 && K > 0, CCLR_EINVAL, "split: empty operand");
  SplitMat s = split_shape(rows, K, form, side, tile);
  s.p = dst;
  if (form == F32_G3) {
    const i64 units = (i64)s.rows_pad * s.nkc * 4;
    i64 grid = (units + 255) / 256;
    if (grid > 65536) grid = 65536;
    hipLaunchKernelGGL(k_split_f32, dim3((unsigned)grid), dim3(256), 0, st, rows, K, src, sR, sK, conj, side,
                       (u4v*)dst, s.rows_pad, s.nkc, sR == 1 ? 1 : 0);
  } else if (s.nplanes == 4) {
    launch_split_p<4>(s, src, sR, sK, conj, st);
  } else {
    launch_split_p<2>(s, src, sR, sK, conj, st);
  }
  HIPCHK(hipGetLastError());
  return s;
}

SplitPlan split_plan_for(int M, int N, int K, int form, int bm, int cutters) {
  SplitPlan p;
  p.bm = bm;
  p.tm = (M + bm - 1) / bm;
  p.nk = split_shape(1, K, form, 0).nkc;
  p.tiles = (i64)p.tm * ((N + TN - 1) / TN);
  constexpr int G = 256;
  const i64 rounds = p.tiles / G, rest = p.tiles % G;
  p.whole = p.tiles;
  p.grid = (int)p.tiles;
  const i64 c = std::min<i64>(cutters, rest * p.nk / 4);  // runs of at least four steps
  if (c > rest) {
    p.whole = rounds * G;
    p.cutters = (int)c;
    p.grid = rounds ? G : (int)c;
  }
  return p;
}

// Estimated time in us of a plan: the k steps of the busiest workgroup (low:
// few compute units at work, full: all of them and their traffic), each whole
// tile's stores, and for cut tiles the partial sums, written and read at
// 4 TB/s, the second launch, and a tenth on their steps, since each workgroup
// starts at another k and neighbours no longer share operand panels.
static double split_cost(const SplitPlan& p, int form) {
  // us per k step with 128, 96 and 64 rows
  static const double low[3][3] = {{1.5, 1.15, 0.9}, {1.05, 0.84, 0.74}, {3.2, 2.55, 1.68}};
  static const double full[3][3] = {{2.0, 1.6, 1.37}, {1.4, 1.18, 1.0}, {3.2, 2.55, 1.68}};
  const int r = p.bm == 128 ? 0 : p.bm == 96 ? 1 : 2;
  const double lo = low[form][r], hi = full[form][r], tile = p.bm * TN / 4e6;  // us of one byte per element
  auto step = [&](i64 busy) { return lo + (hi - lo) * (double)busy / 256; };
  const i64 rounds = p.whole / 256, last = p.whole % 256;
  if (p.cutters == 0 && form == F32_G3 && r == 0) return (p.nk * 3.05 + 2.0 + 256 * 16 * tile) * (rounds + (last > 0));
  double t = (double)rounds * (p.nk * hi + 2.0 + 256 * 16 * tile);
  if (last) t += p.nk * step(last) + 2.0 + (double)last * 16 * tile;
  if (p.cutters) {
    const double rest = (double)(p.tiles - p.whole);
    t += 1.1 * rest * p.nk / p.cutters * step(p.cutters) + 8.0 + p.cutters * (6.0 / 256 + 24 * tile) + rest * 16 * tile;
  }
  return t;
}

// The tile height and the number of runs of least estimated time; cut tiles
// where they are estimated 2% faster than that without.  Over 65 products (10
// to 48000 rows, K 144 to 19900) in the three forms that is 2% off the fastest
// plan measured in the mean, 17% at most, and never behind whole 128 x 128
// tiles.  Cut on any gain in the estimate, and always into 256 runs, it was up
// to 29% behind those: 540x3160x3160 in X2 113 us cut, 85 whole;
// 55x2016x2016 in X2 29 us on 252 runs, 22 on 64 to 128.
SplitPlan split_plan(int M, int N, int K, int form, bool room) {
  REQUIRE(split_form_valid(form), CCLR_EINVAL, "split: unknown form");
  SplitPlan best;
  double t = 1e300;
  auto offer = [&](int cutters, double margin) {
    for (int bm : {128, 96, 64}) {
      const SplitPlan p = split_plan_for(M, N, K, form, bm, cutters);
      const double tp = split_cost(p, form) * margin;
      if (tp < t) best = p, t = tp;
    }
  };
  offer(0, 0.98);
  for (int cutters = 64; room && cutters <= 256; cutters += 32) offer(cutters, 1.0);
  return best;
}

size_t split_workspace(const SplitPlan& p) { return sizeof(float) * 6 * (size_t)p.cutters * p.bm * TN; }

namespace {
template <int BM>
void launch_bm(const SplitMat& A, const SplitMat& B, cplx* C, i64 sCm, i64 sCn, double ar, double ai, int beta,
               const SplitPlan& p, float* W, hipStream_t st) {
  const dim3 grid((unsigned)p.grid), block(512);
  const u4v *a = (const u4v*)A.p, *b = (const u4v*)B.p;
  if (A.form == F32_G3 && BM == 128 && p.cutters == 0)
    hipLaunchKernelGGL((k_cgemm_f32s<128, false>), grid, block, 0, st, a, b, A.rows_pad, B.rows_pad, A.rows, B.rows, C,
                       sCm, sCn, ar, ai, beta, p, W);
  else if (A.form == F32_G3)
    hipLaunchKernelGGL((k_cgemm_f32s<BM, true>), grid, block, 0, st, a, b, A.rows_pad, B.rows_pad, A.rows, B.rows, C,
                       sCm, sCn, ar, ai, beta, p, W);
  else if (A.form == BF16_X2)
    hipLaunchKernelGGL((k_cgemm_bf16s<BF16_X2, BM>), grid, block, 0, st, a, b, A.rows_pad, B.rows_pad, A.rows,
                       B.rows, C, sCm, sCn, ar, ai, beta, p, W);
  else
    hipLaunchKernelGGL((k_cgemm_bf16s<BF16_X3, BM>), grid, block, 0, st, a, b, A.rows_pad, B.rows_pad, A.rows,
                       B.rows, C, sCm, sCn, ar, ai, beta, p, W);
}
}  // namespace

void launch_split_gemm(const SplitMat& A, const SplitMat& B, cplx* C, i64 sCm, i64 sCn, double ar, double ai,
                       int beta, const SplitPlan& p, void* W, hipStream_t st) {
  REQUIRE(A.p && B.p, CCLR_EINVAL, "split GEMM: operand not split");
  REQUIRE(A.form == B.form && A.side == 0 && B.side == 1, CCLR_EINVAL, "split GEMM: operands of different forms");
  REQUIRE(A.K == B.K && A.nkc == B.nkc && A.nkc > 0, CCLR_EINVAL, "split GEMM: operands differ in K");
  REQUIRE(A.rows_pad == p.tm * p.bm && p.tiles == (i64)p.tm * (B.rows_pad / TN) && B.rows_pad % TN == 0 &&
              p.nk == A.nkc && (p.cutters == 0 || W),
          CCLR_EINVAL, "split GEMM: operands and plan differ");
  // uncut, a workgroup of 512 threads for each tile
  REQUIRE(p.tiles < (i64)1 << 23 && (p.cutters > 0 || p.grid == p.tiles), CCLR_EINVAL, "split GEMM: too many tiles");
  switch (p.bm) {
    case 64: launch_bm<64>(A, B, C, sCm, sCn, ar, ai, beta, p, (float*)W, st); break;
    case 96: launch_bm<96>(A, B, C, sCm, sCn, ar, ai, beta, p, (float*)W, st); break;
    case 128: launch_bm<128>(A, B, C, sCm, sCn, ar, ai, beta, p, (float*)W, st); break;
    default: throw CclrError(CCLR_EINVAL, "split GEMM: no such tile");
  }
  HIPCHK(hipGetLastError());
  if (p.cutters > 0) {
    hipLaunchKernelGGL(k_split_join, dim3((unsigned)(p.tiles - p.whole), p.bm * TN / 2048), dim3(512), 0, st, A.rows,
                       B.rows, C, sCm, sCn, ar, ai, beta, p, A.form == F32_G3 ? 1 : 0, (const f4*)W);
    HIPCHK(hipGetLastError());
  }
}
