// Small FP64 complex products: outputs of at most a few hundred 16 x 16 blocks.
//
// The MFMA tiles of the other kernels stage operands through LDS behind a
// barrier per 16 values of k, in one workgroup per output tile; a product such
// as 16 x 4 x 480 then is one workgroup that waits for memory 30 times in a
// row.  Here the waves of a workgroup share one tile of 16 FM x 16 FN and
// split its K loop: each loads its operand fragments straight into the
// registers of v_mfma_f64_16x16x4_f64 (a load takes 16 rows and four
// consecutive k, 64 contiguous bytes of each row where k has unit stride), the
// next tile's loads in flight while the MFMAs of the current one run, and the
// waves' sums are added in LDS at the end.  A long reduction is cut over
// workgroups as well; the partial sums go to a workspace that
// launch_chunk_reduce adds in a fixed order.
//
// Bound by the latency of a few loads per wave (3-4 us a launch up to K = 96,
// 8 us at 16x4x480; 44 us on a 64x32 tile) and, for long reductions, by the
// operands' bytes, which the tiles of a chunk read through one XCD's L2:
// 12x100x120000 43 us = 5.4 TB/s (585 us on the vector kernel with its serial
// chunk sums), 90x48x48060 43, 80x30x31600 26, 130x10x83850 42, 20x200x38000 in
// a batch of 3 126 (83, 36, 58 and 188 with chunks over all XCDs, 516 to 525
// workgroups for 512 places, and loads of 16 bytes out of 64 per row).
#include <algorithm>

#include "gemm_dma.h"

namespace {
template <int FM, int FN, int NW>
__global__ __launch_bounds__(64 * NW, (FM * FN == 4 ? 2 : 4)) void k_zgemm_frag(GemmArgs g, int tm, int nt, int kc, int S,
                                                          int xcd, cplx* __restrict__ W) {
  constexpr int BM = 16 * FM, BN = 16 * FN;
  constexpr int U = FM * FN >= 2 ? 2 : 4, KT = 4 * U;  // MFMA steps and depth of a K tile
  __shared__ cplx red[NW > 1 ? NW : 1][NW > 1 ? BM * BN : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, rr = lane & 15, gq = lane >> 4;
  // xcd: all tiles of a chunk run on one XCD (workgroups are dealt to the 8
  // XCDs round-robin), which then reads the chunk's operands into its L2 once
  int t = blockIdx.x, q = 0;
  if (xcd) {
    const int l = t >> 3, c = l / nt;
    q = 8 * c + (t & 7);
    t = l - c * nt;
    if (q >= S) return;
  } else if (S > 1) {
    q = t / nt;
    t -= q * nt;
  }
  const int m0 = (t % tm) * BM, n0 = (t / tm) * BN;
  const i64 bz = blockIdx.y;
  const int k0 = q * kc, k1 = min(g.K, k0 + kc);
  const unsigned sgnA = g.conjA ? 0x80000000u : 0u, sgnB = g.conjB ? 0x80000000u : 0u;
  // rows past the operand read its last row; their outputs are not stored
  const cplx *pa[FM], *pb[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
    pa[i] = g.A + boff(g, bz, g.sAb, g.sAb2) + (i64)min(m0 + 16 * i + rr, g.M - 1) * g.sAm + gq * g.sAk;
#pragma unroll
  for (int j = 0; j < FN; ++j)
    pb[j] = g.B + boff(g, bz, g.sBb, g.sBb2) + (i64)min(n0 + 16 * j + rr, g.N - 1) * g.sBn + gq * g.sBk;
  d4 cr[FM][FN], ci[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) cr[i][j] = ci[i][j] = d4{0, 0, 0, 0};
  cplx fa[2][U][FM], fb[2][U][FN];
  // this lane's elements of the K tile at kb; zero beyond the chunk, in both operands
  auto load = [&](int kb, int s) {
    if (kb + KT <= k1) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const i64 oa = (i64)(kb + 4 * u) * g.sAk, ob = (i64)(kb + 4 * u) * g.sBk;
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[s][u][i] = pa[i][oa];
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[s][u][j] = pb[j][ob];
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = kb + 4 * u + gq;
        const bool in = k < k1;
        const i64 kk = (in ? k : k1 - 1) - gq;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const cplx x = pa[i][kk * g.sAk];
          fa[s][u][i] = in ? x : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const cplx x = pb[j][kk * g.sBk];
          fb[s][u][j] = in ? x : make_double2(0.0, 0.0);
        }
      }
    }
  };
  auto mfma = [&](int s) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      cplx a[FM], b[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) a[i] = flip_im(fa[s][u][i], sgnA);
#pragma unroll
      for (int j = 0; j < FN; ++j) b[j] = flip_im(fb[s][u][j], sgnB);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          cr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].x, cr[i][j], 0, 0, 0);
          ci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].x, b[j].y, ci[i][j], 0, 0, 0);
        }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          cr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].y, b[j].y, cr[i][j], 0, 0, kNegA);
          ci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i].y, b[j].x, ci[i][j], 0, 0, 0);
        }
    }
  };
  int kb = k0 + KT * wave;
  if (kb < k1) {
    load(kb, 0);
    for (;;) {
      if (kb + KT * NW < k1) load(kb + KT * NW, 1);
      mfma(0);
      kb += KT * NW;
      if (kb >= k1) break;
      if (kb + KT * NW < k1) load(kb + KT * NW, 0);
      mfma(1);
      kb += KT * NW;
      if (kb >= k1) break;
    }
  }
  auto store = [&](int m, int n, double xr, double xi) {
    if (m >= g.M || n >= g.N) return;
    if (S > 1) {
      W[((bz * S + q) * (i64)g.M + m) * g.N + n] = make_double2(xr, xi);
      return;
    }
    cplx y = make_double2(g.ar * xr - g.ai * xi, g.ar * xi + g.ai * xr);
    cplx* dst = g.C + boff(g, bz, g.sCb, g.sCb2) + (i64)m * g.sCm + (i64)n * g.sCn;
    if (g.beta) {
      const cplx o = *dst;
      y.x += o.x;
      y.y += o.y;
    }
    *dst = y;
  };
  if (NW == 1) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          store(m0 + 16 * i + 4 * r + gq, n0 + 16 * j + rr, cr[i][j][r], ci[i][j][r]);
    return;
  }
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        red[wave][(16 * i + 4 * r + gq) * BN + 16 * j + rr] = make_double2(cr[i][j][r], ci[i][j][r]);
  __syncthreads();
  for (int e = threadIdx.x; e < BM * BN; e += 64 * NW) {
    double xr = 0.0, xi = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      xr += red[w][e].x;
      xi += red[w][e].y;
    }
    store(m0 + e / BN, n0 + e % BN, xr, xi);
  }
}

// C[b][m][n] = (beta ? C : 0) + alpha * sum_s W[b][s][m][n].  P threads share
// an output element: thread p adds the chunks p, p + P, ..., four loads in
// flight, and the P sums are added in order.  One thread per output, adding
// 60 to 1900 chunks one after another, took 20-60 us for outputs of a thousand
// entries (500 us for 1875 chunks); this takes 4-8.
template <int P>
__global__ __launch_bounds__(256) void k_chunk_reduce(GemmArgs g, int S, const cplx* __restrict__ W) {
  constexpr int E = 256 / P;
  __shared__ cplx part[P][E + 1];
  const i64 mn = (i64)g.M * g.N, total = mn * g.batch;
  const int o = threadIdx.x % E, p = threadIdx.x / E;
  const i64 e = (i64)blockIdx.x * E + o;
  double xr = 0.0, xi = 0.0;
  i64 b = 0, r = 0;
  if (e < total) {
    b = e / mn;
    r = e - b * mn;
    const cplx* __restrict__ w = W + b * S * mn + r;
    int s = p;
    for (; s + 3 * P < S; s += 4 * P) {
      const cplx w0 = w[s * mn], w1 = w[(s + P) * mn], w2 = w[(s + 2 * P) * mn], w3 = w[(s + 3 * P) * mn];
      xr += (w0.x + w1.x) + (w2.x + w3.x);
      xi += (w0.y + w1.y) + (w2.y + w3.y);
    }
    for (; s < S; s += P) {
      const cplx x = w[s * mn];
      xr += x.x;
      xi += x.y;
    }
  }
  if (P > 1) {
    part[p][o] = make_double2(xr, xi);
    __syncthreads();
    if (p > 0) return;
    xr = xi = 0.0;
#pragma unroll
    for (int t = 0; t < P; ++t) {
      xr += part[t][o].x;
      xi += part[t][o].y;
    }
  }
  if (e >= total) return;
  cplx y = make_double2(g.ar * xr - g.ai * xi, g.ar * xi + g.ai * xr);
  cplx* dst = g.C + boff(g, b, g.sCb, g.sCb2) + r / g.N * g.sCm + r % g.N * g.sCn;
  if (g.beta) {
    const cplx x = *dst;
    y.x += x.x;
    y.y += x.y;
  }
  *dst = y;
}
}  // namespace

void launch_chunk_reduce(const GemmArgs& g, int S, const cplx* W, hipStream_t s) {
  const i64 total = (i64)g.M * g.N * g.batch;
  if (total <= 0) return;
  REQUIRE(total < (1ll << 31) * 16, CCLR_EINVAL, "chunk sums: output too large");
  // enough threads per output for about a thousand workgroups, at most one for every four chunks
  auto grid = [&](int P) { return dim3((unsigned)((total * P + 255) / 256)); };
  const i64 want = (1024 * 256 + total - 1) / total, most = std::max(1, S / 4);
  const i64 P = std::min(want, most);
  if (P >= 32) hipLaunchKernelGGL(k_chunk_reduce<32>, grid(32), dim3(256), 0, s, g, S, W);
  else if (P >= 16) hipLaunchKernelGGL(k_chunk_reduce<16>, grid(16), dim3(256), 0, s, g, S, W);
  else if (P >= 8) hipLaunchKernelGGL(k_chunk_reduce<8>, grid(8), dim3(256), 0, s, g, S, W);
  else if (P >= 4) hipLaunchKernelGGL(k_chunk_reduce<4>, grid(4), dim3(256), 0, s, g, S, W);
  else hipLaunchKernelGGL(k_chunk_reduce<1>, grid(1), dim3(256), 0, s, g, S, W);
  HIPCHK(hipGetLastError());
}

FragPlan frag_plan(const GemmArgs& g) {
  FragPlan p{};
  const auto blocks = [&](int fm, int fn) {
    return (i64)((g.M + 16 * fm - 1) / (16 * fm)) * ((g.N + 16 * fn - 1) / (16 * fn)) * g.batch;
  };
  const int kt = (g.K + 15) / 16;
  // Long reductions are cut into chunks that fill each XCD once: 128 workgroups
  // of four waves on each, 64 with 32 x 32 tiles (registers).  Ten more of 1000
  // took a second round: 20x200x38000, batch 3 121 us with 24 chunks, 173 with
  // 25.  Tile height and width by the rate their operand reads, out of L2, were
  // measured at (16-row panels over 9, 7.5 and 6.5 TB/s): 90x48x48060 43 us on
  // 32 x 16, 53 on 32 x 32; 32x120x114240 93 and 84.
  if (kt >= 32 && blocks(1, 1) <= 512) {
    static const struct { int fm, fn, slots; double cost; } shapes[] = {
        {1, 1, 1024, 0.222}, {2, 1, 1024, 0.4}, {1, 2, 1024, 0.4}, {2, 2, 512, 0.61}};
    double best = 1e300;
    for (const auto& x : shapes) {
      const i64 nb = blocks(x.fm, x.fn), per = x.slots / 8 / nb;
      const i64 S = std::min<i64>(per ? 8 * per : x.slots / nb, kt / 8);
      if (S < 2 || (double)nb * x.cost >= best) continue;
      best = (double)nb * x.cost;
      p.fm = x.fm, p.fn = x.fn, p.nw = 4;
      p.xcd = S >= 8 && (S % 8 == 0 || S >= 64);
      p.kc = (int)(((g.K + S - 1) / S + 15) / 16 * 16);
    }
    if (p.kc > 0) {
      p.S = (g.K + p.kc - 1) / p.kc;
      return p;
    }
  }
  // larger tiles read each operand fewer times, once they alone keep the compute units busy
  const i64 work = blocks(1, 1) * ((g.K + 255) / 256);
  p.fm = p.fn = 1;
  if (g.M > 16 && work >= 1024) p.fm = 2;
  if (g.N > 16 && work >= 2048) p.fn = 2;
  const i64 nb = blocks(p.fm, p.fn);
  // one wave a tile where the tiles alone are two a SIMD (97200x12x90 32 us, 36 with four)
  p.nw = kt <= 1 || (nb >= 2048 && kt <= 8) ? 1 : (p.fm * p.fn == 1 && kt > 4 ? 8 : 4);
  // cut the reduction until there are about 512 workgroups, each wave with at least 4 K tiles
  i64 S = std::min<i64>((512 + nb - 1) / nb, kt / (4 * p.nw));
  S = std::max<i64>(1, std::min<i64>(S, 4096));
  i64 kc = ((g.K + S - 1) / S + 15) / 16 * 16;
  p.S = (int)((g.K + kc - 1) / kc);
  p.kc = (int)kc;
  return p;
}

void launch_zgemm_frag(const GemmArgs& g, const FragPlan& p, cplx* W, hipStream_t s) {
  const int tm = (g.M + 16 * p.fm - 1) / (16 * p.fm), tn = (g.N + 16 * p.fn - 1) / (16 * p.fn);
  REQUIRE(g.M >= 1 && g.N >= 1 && g.K >= 1 && g.batch >= 1 && g.batch < 65536 && g.kchunk == 0 && p.S >= 1 &&
              p.S < 65536 && (p.S == 1 || W) && (i64)p.kc * p.S >= g.K && (i64)tm * tn < (1ll << 31),
          CCLR_EINVAL, "small product: arguments outside the kernel's contract");
  const i64 wgs = (i64)tm * tn * (p.xcd ? (p.S + 7) / 8 * 8 : p.S);
  REQUIRE(wgs < (1ll << 31), CCLR_EINVAL, "small product: too many workgroups");
  const dim3 grid((unsigned)wgs, (unsigned)g.batch);
#define FRAG(FM, FN, NW) hipLaunchKernelGGL((k_zgemm_frag<FM, FN, NW>), grid, dim3(64 * NW), 0, s, g, tm, tm * tn, p.kc, p.S, p.xcd, W)
  if (p.fm == 1 && p.fn == 1) {
    if (p.nw == 1) FRAG(1, 1, 1);
    else if (p.nw == 4) FRAG(1, 1, 4);
    else FRAG(1, 1, 8);
  } else if (p.fm == 2 && p.fn == 1) {
    if (p.nw == 1) FRAG(2, 1, 1);
    else FRAG(2, 1, 4);
  } else if (p.fm == 1) {
    if (p.nw == 1) FRAG(1, 2, 1);
    else FRAG(1, 2, 4);
  } else {
    if (p.nw == 1) FRAG(2, 2, 1);
    else FRAG(2, 2, 4);
  }
#undef FRAG
  HIPCHK(hipGetLastError());
  if (p.S > 1) launch_chunk_reduce(g, p.S, W, s);
}
