// FP64 complex GEMM with an even split of the work over the compute units.
//
// The transforms' ladders and rings at o <= 20 have between a few dozen and
// a few hundred output tiles: whole tiles dealt to 256 compute units leave a
// last round that is partly empty, and a ladder of one vector (o(o-1)/2 = 45
// rows at o = 10) occupies half of them.  Here a persistent grid deals whole
// tiles first, while they fill every workgroup, and cuts the K loops of the
// remaining tiles into equal runs, one per workgroup; a second kernel adds a
// cut tile's partial sums in the order of k.  No workgroup waits for another.
//
// Bound by FP64 MFMA issue; what is left to 75 TFLOP/s is padding to 16 rows,
// the first loads of each run and the partial sums.  Against the fastest of
// the other tiles (us): 45x8385x8385 429 / 1223, 180x3160x3160 251 / 461,
// 240x7140x7140 1439 / 1833, 1300x1300x1300 299 / 343, 3840x1920x1920 1640 /
// 1765, 570x19900x19900 25980 / 27330, 144x144x10000 54 / 90 (split along K
// on 64x64 tiles), 100x144x10000 in a batch of 12 297 / 890.
#include <algorithm>

#include "gemm_dma.h"

namespace {
constexpr int SK_BN = 64, SK_BK = 16, SK_NT = 256;

// Tile t of the launch, M fastest within groups of gm row tiles that sweep
// the column tiles, the batch index slowest.
__device__ __forceinline__ void sk_tile(i64 t, const SkPlan& p, int& mi, int& ni, int& bz) {
  const int per_b = p.tm * p.tn;
  bz = (int)(t / per_b);
  const int r = (int)(t - (i64)bz * per_b);
  const int grp = r / (p.gm * p.tn), within = r - grp * p.gm * p.tn;
  const int gme = min(p.gm, p.tm - grp * p.gm);
  mi = grp * p.gm + within % gme;
  ni = within / gme;
}

// The workgroups of one XCD (hardware index modulo 8) take consecutive
// positions of the work order, so that they share operand panels in their L2.
__device__ __forceinline__ int sk_position(int w, int n) {
  const int x = w & 7, l = w >> 3, per = n >> 3, rem = n & 7;
  return (x < rem ? x * (per + 1) : rem * (per + 1) + (x - rem) * per) + l;
}

// Four waves side by side, each FM x 1 blocks of 16 x 16: tiles of 16 FM rows
// and 64 columns, so a product with 45 or 90 rows pads to 48 or 96 and not
// to 64 or 128.  Operand tiles go from memory to LDS by direct loads, two
// stages (at most 80 KiB, so two workgroups share a compute unit and one runs
// MFMAs while the other waits at its barrier); layouts as in k_zgemm_dma:
// an operand with unit-stride k as [row][16 slots], k in slot k ^ (row mod
// 16), one with unit-stride rows as [k][rows].
template <int FM, bool AK, bool BNF>
__global__ __launch_bounds__(SK_NT, 2) void k_zgemm_sk(GemmArgs g, SkPlan p, cplx* __restrict__ W) {
  constexpr int BM = 16 * FM, BN = SK_BN, BK = SK_BK;
  constexpr int JA = FM, JB = 4;  // 1 KiB chunks of a stage per wave (of BM / 4 and BN / 4)
  constexpr bool KCA = AK, KCB = !BNF;
  __shared__ cplx sA0[BM * BK], sA1[BM * BK], sB0[BN * BK], sB1[BN * BK];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rr = lane & 15, gq = lane >> 4, wn = wave * 16;
  const unsigned sgnA = g.conjA ? 0x80000000u : 0u, sgnB = g.conjB ? 0x80000000u : 0u;
  const i64 dA = (i64)BK * g.sAk, dB = (i64)BK * g.sBk;
  const int pos = sk_position((int)blockIdx.x, (int)gridDim.x);
  auto offa = [&](int q, int i) {
    return KCA ? (16 * i + rr) * BK + ((4 * q + gq) ^ rr) : (4 * q + gq) * BM + 16 * i + rr;
  };
  auto offb = [&](int q) { return KCB ? (wn + rr) * BK + ((4 * q + gq) ^ rr) : (4 * q + gq) * BN + wn + rr; };

  // K tiles [kt0, kt1) of output tile t; slot < 0: the whole tile, else its partial sums to W[slot]
  auto segment = [&](i64 t, int kt0, int kt1, i64 slot) {
    int mi, ni, bz;
    sk_tile(t, p, mi, ni, bz);
    const int m0 = mi * BM, n0 = ni * BN, kbeg = kt0 * BK, kend = min(g.K, kt1 * BK);
    const int nfull = (kend - kbeg) / BK, tail = kend - kbeg - nfull * BK;
    const cplx* __restrict__ A = g.A + boff(g, bz, g.sAb, g.sAb2);
    const cplx* __restrict__ B = g.B + boff(g, bz, g.sBb, g.sBb2);
    // this lane's element of each of its chunks of a K tile (rows past the
    // operand read its last row; their outputs are not stored)
    const cplx *pa[JA], *pb[JB];
    int ka[JA], kb[JB];
#pragma unroll
    for (int j = 0; j < JA; ++j) {
      const int c = 4 * j + wave, e = 64 * c + lane;
      const int row = KCA ? 4 * c + gq : e % BM;
      ka[j] = KCA ? rr ^ (row & 15) : e / BM;
      pa[j] = A + (i64)min(m0 + row, g.M - 1) * g.sAm + (i64)(kbeg + ka[j]) * g.sAk;
    }
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const int c = 4 * j + wave, e = 64 * c + lane;
      const int row = KCB ? 4 * c + gq : e % BN;
      kb[j] = KCB ? rr ^ (row & 15) : e / BN;
      pb[j] = B + (i64)min(n0 + row, g.N - 1) * g.sBn + (i64)(kbeg + kb[j]) * g.sBk;
    }
    auto fetch = [&](int t, cplx* la, cplx* lb) {
#pragma unroll
      for (int j = 0; j < JA; ++j) dma16(pa[j] + t * dA, la + 64 * (4 * j + wave));
#pragma unroll
      for (int j = 0; j < JB; ++j) dma16(pb[j] + t * dB, lb + 64 * (4 * j + wave));
    };
    d4 cr[FM], ci[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i) cr[i] = ci[i] = d4{0, 0, 0, 0};
    double2 fa[2][FM], fb[2];
    auto fread = [&](const cplx* la, const cplx* lb, int q, int s) {
#pragma unroll
      for (int i = 0; i < FM; ++i) fa[s][i] = flip_im(la[offa(q, i)], sgnA);
      fb[s] = flip_im(lb[offb(q)], sgnB);
    };
    auto mfma_q = [&](int s) {
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        cr[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s][i].x, fb[s].x, cr[i], 0, 0, 0);
        ci[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s][i].x, fb[s].y, ci[i], 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        cr[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s][i].y, fb[s].y, cr[i], 0, 0, kNegA);
        ci[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s][i].y, fb[s].x, ci[i], 0, 0, 0);
      }
    };
    // one K tile on stage (ca, cb) while the next one loads into (na, nb); the
    // wait and the barrier come once the last K step's fragments are in
    // registers, the next tile's first fragments are read behind them
    auto step = [&](int t, const cplx* ca, const cplx* cb, cplx* na, cplx* nb) {
      fetch(t + 1 < nfull ? t + 1 : t, na, nb);
      __builtin_amdgcn_sched_barrier(0);
      fread(ca, cb, 1, 1);
      mfma_q(0);
      fread(ca, cb, 2, 0);
      mfma_q(1);
      fread(ca, cb, 3, 1);
      mfma_q(0);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      fread(na, nb, 0, 0);
      mfma_q(1);
    };
    __syncthreads();  // every wave is done with the stages of the previous segment
    if (nfull > 0) {
      fetch(0, sA0, sB0);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      fread(sA0, sB0, 0, 0);
      for (int t = 0; t < nfull; t += 2) {
        step(t, sA0, sB0, sA1, sB1);
        if (t + 1 < nfull) step(t + 1, sA1, sB1, sA0, sB0);
      }
      __syncthreads();
    }
    if (tail > 0) {  // K remainder: through registers, zero beyond kend (both stages are idle here)
      const cplx z = make_double2(0.0, 0.0);
#pragma unroll
      for (int j = 0; j < JA; ++j) sA0[64 * (4 * j + wave) + lane] = ka[j] < tail ? pa[j][nfull * dA] : z;
#pragma unroll
      for (int j = 0; j < JB; ++j) sB0[64 * (4 * j + wave) + lane] = kb[j] < tail ? pb[j][nfull * dB] : z;
      __syncthreads();
      fread(sA0, sB0, 0, 0);
#pragma unroll
      for (int q = 0; q < BK / 4; ++q) {
        if (q + 1 < BK / 4) fread(sA0, sB0, q + 1, (q & 1) ^ 1);
        mfma_q(q & 1);
      }
    }
    if (slot >= 0) {
      cplx* __restrict__ w = W + slot * (BM * BN);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          w[(16 * i + 4 * r + gq) * BN + wn + rr] = make_double2(cr[i][r], ci[i][r]);
      return;
    }
    cplx* __restrict__ C = g.C + boff(g, bz, g.sCb, g.sCb2);
    const int n = n0 + wn + rr;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + 16 * i + 4 * r + gq;
        if (m < g.M && n < g.N) {
          const double xr = cr[i][r], xi = ci[i][r];
          cplx y = make_double2(g.ar * xr - g.ai * xi, g.ar * xi + g.ai * xr);
          cplx* dst = C + (i64)m * g.sCm + (i64)n * g.sCn;
          if (g.beta) {
            const cplx o = *dst;
            y.x += o.x;
            y.y += o.y;
          }
          *dst = y;
        }
      }
  };

  // the whole tiles of this workgroup, then its run over the cut ones (a run of
  // at most nk K tiles touches at most two output tiles)
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
    segment(tile, k0, k1, to);
  }
}

// Adds the partial sums of cut tile whole + blockIdx.x in the order of k and
// stores the result, one element per thread (blockIdx.y: which 256 of the
// tile); eight partial sums are loaded before they are added.
__global__ __launch_bounds__(256) void k_zgemm_sk_join(GemmArgs g, SkPlan p, int bm, const cplx* __restrict__ W) {
  const i64 total = (p.tiles - p.whole) * p.nk, t = blockIdx.x;
  const i64 lo = t * p.nk, hi = lo + p.nk;
  // run c covers the K tiles [c total / cutters, (c + 1) total / cutters): the runs with a part of [lo, hi)
  i64 c0 = lo * p.cutters / total;
  while ((c0 + 1) * total / p.cutters <= lo) ++c0;
  const i64 b0 = c0 * total / p.cutters;
  if (b0 <= lo && (c0 + 1) * total / p.cutters >= hi) return;  // in one run: stored whole
  i64 c1 = c0 + 1;
  while (c1 < p.cutters && c1 * total / p.cutters < hi) ++c1;
  int mi, ni, bz;
  sk_tile(p.whole + t, p, mi, ni, bz);
  const int size = bm * SK_BN, e = blockIdx.y * 256 + threadIdx.x;
  const int m = mi * bm + e / SK_BN, n = ni * SK_BN + e % SK_BN;
  if (e >= size || m >= g.M || n >= g.N) return;
  // the first run may have begun in the tile before: then this is its second piece
  const cplx first = W[(2 * c0 + (b0 < lo ? 1 : 0)) * size + e];
  double xr = first.x, xi = first.y;
  constexpr int U = 8;
  for (i64 c = c0 + 1; c < c1; c += U) {
    cplx w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) w[u] = c + u < c1 ? W[2 * (c + u) * size + e] : make_double2(0.0, 0.0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      xr += w[u].x;
      xi += w[u].y;
    }
  }
  cplx y = make_double2(g.ar * xr - g.ai * xi, g.ar * xi + g.ai * xr);
  cplx* dst = g.C + boff(g, bz, g.sCb, g.sCb2) + (i64)m * g.sCm + (i64)n * g.sCn;
  if (g.beta) {
    const cplx o = *dst;
    y.x += o.x;
    y.y += o.y;
  }
  *dst = y;
}

template <int FM>
void launch_fm(const GemmArgs& g, const SkPlan& p, cplx* W, hipStream_t s) {
  const bool ak = g.sAk == 1, bn = g.sBn == 1;
  const dim3 grid((unsigned)p.grid), block(SK_NT);
  if (ak && bn) hipLaunchKernelGGL((k_zgemm_sk<FM, true, true>), grid, block, 0, s, g, p, W);
  else if (ak) hipLaunchKernelGGL((k_zgemm_sk<FM, true, false>), grid, block, 0, s, g, p, W);
  else if (bn) hipLaunchKernelGGL((k_zgemm_sk<FM, false, true>), grid, block, 0, s, g, p, W);
  else hipLaunchKernelGGL((k_zgemm_sk<FM, false, false>), grid, block, 0, s, g, p, W);
}
}  // namespace

size_t sk_workspace(const SkPlan& p) {
  return p.cutters > 0 ? sizeof(cplx) * 2 * (size_t)p.cutters * (16 * p.fm) * SK_BN : 0;
}

SkPlan sk_plan_for(const GemmArgs& g, int fm, int max_cutters) {
  SkPlan p{};
  p.fm = fm;
  p.tm = (g.M + 16 * fm - 1) / (16 * fm);
  p.tn = (g.N + SK_BN - 1) / SK_BN;
  p.gm = std::min(p.tm, 8);
  p.nk = (g.K + SK_BK - 1) / SK_BK;
  p.tiles = (i64)p.tm * p.tn * g.batch;
  constexpr int G = 512, kMinRun = 8;
  const i64 rounds = p.tiles / G, rest = p.tiles % G;
  p.whole = p.tiles;
  p.cutters = 0;
  p.grid = (int)std::min<i64>(p.tiles, G);
  if (rest && max_cutters > 0) {
    const i64 c = std::min<i64>(std::min<i64>(G, max_cutters), rest * p.nk / kMinRun);
    if (c > rest) {
      p.whole = rounds * G;
      p.cutters = (int)c;
      p.grid = rounds ? G : (int)c;
    }
  }
  return p;
}

void launch_zgemm_sk(const GemmArgs& g, const SkPlan& p, cplx* W, hipStream_t s) {
  REQUIRE(g.M >= 1 && g.N >= 1 && g.K >= 1 && g.batch >= 1 && g.kchunk == 0 && (p.cutters == 0 || W) &&
              p.tiles == (i64)p.tm * p.tn * g.batch && (i64)p.tm * p.tn < (1ll << 31),
          CCLR_EINVAL, "evenly split product: arguments outside the kernel's contract");
  switch (p.fm) {
    case 2: launch_fm<2>(g, p, W, s); break;
    case 3: launch_fm<3>(g, p, W, s); break;
    case 4: launch_fm<4>(g, p, W, s); break;
    case 5: launch_fm<5>(g, p, W, s); break;
    case 6: launch_fm<6>(g, p, W, s); break;
    default: throw CclrError(CCLR_EINVAL, "evenly split product: no such tile");
  }
  HIPCHK(hipGetLastError());
  if (p.cutters > 0) {
    hipLaunchKernelGGL(k_zgemm_sk_join, dim3((unsigned)(p.tiles - p.whole), 4 * p.fm), dim3(256), 0, s, g,
                       p, 16 * p.fm, W);
    HIPCHK(hipGetLastError());
  }
}
