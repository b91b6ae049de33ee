// Small complex GEMM straight from the operands' own layouts.
//
// A vertex with a short k (a few bits) or few entries spends its time not on
// products but on launches: two permutations of some microseconds and a GEMM
// kernel that fills a 128 x 128 tile for them.  Here one launch reads both
// operands through offset tables (entry (m, k) of A sits at row[m] + ka[k], entry
// (k, n) of B at col[n] + kb[k]: an operand's offset is linear in its legs),
// so neither is permuted, and multiplies on the vector units.
//
// Bound: the result's bytes for short k, else launch latency: operands of at
// most a few hundred KB come from the L2.  Tile T x T (64, or 32 when there
// are few tiles), 256 threads of (T / 16)^2 results, 16 k a round through LDS; the next
// round's entries are fetched while this one is multiplied.  One launch of
// 4-7 us in place of 20-30 us (permutations 3.5 us each, GEMM 8-17 us).
//
// MODE 0 multiplies in FP32 (four real products).  A BF16x3 plan keeps its
// products: MODE 1 (4M) splits each value into two bfloat16 terms and adds
// ha hb + ha lb + la hb, MODE 2 (3M) the same of re, im and their sum; a
// product of two bfloat16 is exact in FP32, so only the order of the
// additions differs from the matrix cores'.
#include "tn_device.h"

namespace tn {

template <int MODE>
__device__ __forceinline__ void small_split(float2 v, float (&h)[3], float (&l)[3]) {
  const float x[3] = {v.x, v.y, v.x + v.y};
#pragma unroll
  for (int c = 0; c < (MODE == 2 ? 3 : 2); ++c) {
    const float t = (float)(__bf16)x[c];
    h[c] = t;
    l[c] = (float)(__bf16)(x[c] - t);
  }
}

template <int MODE, int T>
__global__ __launch_bounds__(256) void k_cgemm_small(SmallGemm g) {
  constexpr int R = T / 16;           // results per thread along each side
  constexpr int KS = 16;              // k per round
  constexpr int LD = T * KS / 256;    // entries per thread, operand and round
  __shared__ __align__(16) float2 As[KS][T], Bs[KS][T + 2];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int q = blockIdx.z;
  const int m0 = blockIdx.y * T, n0 = blockIdx.x * T;
  const float2 *A = g.A + q * g.abs, *B = g.B + q * g.bbs;
  const Slot *sa = g.sa + q * g.sabs, *sb = g.sb + q * g.sbbs;
  Slot *sc = g.sc + q * g.scbs;
  const int ea = tn_scale_exp(sa->maxbits), eb = tn_scale_exp(sb->maxbits);
  const float fa = ldexpf(1.0f, -ea), fb = ldexpf(1.0f, -eb);
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) sc->log2s = sa->log2s + sb->log2s + (double)(ea + eb);
  const int32_t *row = g.tab, *col = row + g.M, *ka = col + g.N, *kb = ka + g.K;
  // this thread's rows, columns and k of a round: 16 consecutive threads take
  // 16 rows of one k
  int ro[LD], co[LD], kk[LD], mm[LD];
#pragma unroll
  for (int i = 0; i < LD; ++i) {
    const int e = tid + 256 * i;
    mm[i] = e % T;
    kk[i] = e / T;
    ro[i] = m0 + mm[i] < g.M ? row[m0 + mm[i]] : -1;
    co[i] = n0 + mm[i] < g.N ? col[n0 + mm[i]] : -1;
  }
  float2 av[LD], bv[LD];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      const int k = k0 + kk[i];
      av[i] = bv[i] = make_float2(0.f, 0.f);
      if (k < g.K) {
        if (ro[i] >= 0) av[i] = A[ro[i] + ka[k]];
        if (co[i] >= 0) bv[i] = B[co[i] + kb[k]];
      }
    }
  };
  float acc[R][R][MODE == 2 ? 3 : 2];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
      for (int c = 0; c < (MODE == 2 ? 3 : 2); ++c) acc[i][j][c] = 0.f;
  fetch(0);
  for (int k0 = 0; k0 < g.K; k0 += KS) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      As[kk[i]][mm[i]] = make_float2(av[i].x * fa, av[i].y * fa);
      Bs[kk[i]][mm[i]] = make_float2(bv[i].x * fb, bv[i].y * fb);
    }
    __syncthreads();
    if (k0 + KS < g.K) fetch(k0 + KS);
    const int kn = g.K - k0 < KS ? g.K - k0 : KS;
    for (int k = 0; k < kn; ++k) {
      float2 a[R], b[R];
#pragma unroll
      for (int i = 0; i < R; ++i) {
        a[i] = As[k][ty + 16 * i];
        b[i] = Bs[k][tx + 16 * i];
      }
      if (MODE == 0) {
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
          for (int j = 0; j < R; ++j) {
            acc[i][j][0] = fmaf(a[i].x, b[j].x, acc[i][j][0]);
            acc[i][j][0] = fmaf(-a[i].y, b[j].y, acc[i][j][0]);
            acc[i][j][1] = fmaf(a[i].x, b[j].y, acc[i][j][1]);
            acc[i][j][1] = fmaf(a[i].y, b[j].x, acc[i][j][1]);
          }
      } else {
        float ah[R][3], al[R][3], bh[R][3], bl[R][3];
#pragma unroll
        for (int i = 0; i < R; ++i) {
          small_split<MODE>(a[i], ah[i], al[i]);
          small_split<MODE>(b[i], bh[i], bl[i]);
        }
        // one real product of the split values
        auto prod = [](float xh, float xl, float yh, float yl, float c) {
          return fmaf(xh, yh, fmaf(xh, yl, fmaf(xl, yh, c)));
        };
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
          for (int j = 0; j < R; ++j) {
            if (MODE == 1) {
              acc[i][j][0] = prod(ah[i][0], al[i][0], bh[j][0], bl[j][0], acc[i][j][0]);
              acc[i][j][0] = prod(-ah[i][1], -al[i][1], bh[j][1], bl[j][1], acc[i][j][0]);
              acc[i][j][1] = prod(ah[i][0], al[i][0], bh[j][1], bl[j][1], acc[i][j][1]);
              acc[i][j][1] = prod(ah[i][1], al[i][1], bh[j][0], bl[j][0], acc[i][j][1]);
            } else {
#pragma unroll
              for (int c = 0; c < 3; ++c)
                acc[i][j][c % (MODE == 2 ? 3 : 2)] =
                    prod(ah[i][c], al[i][c], bh[j][c], bl[j][c], acc[i][j][c % (MODE == 2 ? 3 : 2)]);
            }
          }
      }
    }
  }
  float2 *C = g.C + q * g.cbs;
  float mx = 0.f;
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int m = m0 + ty + 16 * i, n = n0 + tx + 16 * j;
      float re = acc[i][j][0], im = acc[i][j][1];
      if (MODE == 2) {
        im = acc[i][j][MODE == 2 ? 2 : 0] - re - im;
        re = re - acc[i][j][1];
      }
      if (m < g.M && n < g.N) {
        C[(int64_t)m * g.N + n] = make_float2(re, im);
        mx = fmaxf(mx, fmaxf(fabsf(re), fabsf(im)));
      }
    }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  // one record update per block
  __syncthreads();
  float *red = (float *)&As[0][0];
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
  if (tid == 0) slot_max(&sc->maxbits, fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])));
}

hipError_t launch_gemm_small(hipStream_t st, const SmallGemm &g, int prec, int form, int nbatch) {
  if (g.M < 1 || g.N < 1 || g.K < 1 || nbatch < 1 || nbatch > 65535) return hipErrorInvalidValue;
  const int mode = prec == kPrecFP32 ? 0 : form == kForm4M ? 1 : 2;
  // 64 x 64 tiles when they alone give every CU a block, 32 x 32 otherwise
  const int64_t big = (int64_t)((g.M + 63) / 64) * ((g.N + 63) / 64) * nbatch;
  const int t = big >= 256 ? 64 : 32;
  const dim3 grid((g.N + t - 1) / t, (g.M + t - 1) / t, nbatch);
  if (grid.y > 65535) return hipErrorInvalidValue;
#define TN_SMALL(MODE)                                                                         \
  if (t == 64) hipLaunchKernelGGL((k_cgemm_small<MODE, 64>), grid, dim3(256), 0, st, g);       \
  else hipLaunchKernelGGL((k_cgemm_small<MODE, 32>), grid, dim3(256), 0, st, g)
  if (mode == 0) {
    TN_SMALL(0);
  } else if (mode == 1) {
    TN_SMALL(1);
  } else {
    TN_SMALL(2);
  }
#undef TN_SMALL
  return hipGetLastError();
}

}  // namespace tn
