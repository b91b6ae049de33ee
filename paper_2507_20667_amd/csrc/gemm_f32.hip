// FP32 complex GEMM from k-tiled float planes, on the bfloat16 matrix cores.
//
// The permutation that puts a vertex's operands in GEMM order writes them as
// two float planes (re, im), divided by 2^e of the operand's scale record and
// k-tiled: row r, k sits at ((k / 16) * rows + r) * 16 + k % 16, so that one
// 16-deep stage of a 128-row tile is a contiguous 8 KB block of each plane.
// Stages stream straight from global memory into two LDS slots
// (global_load_lds_dwordx4, no staging registers), one stage ahead (the 32-wide
// wave tiles: four slots, three stages ahead).  The wait
// for a stage is a vmcnt on the wave's own loads followed by a barrier.  Past
// the last stage the request repeats the last stage into the free slot, so
// the number of loads in flight never changes.  The slots are distinct arrays
// named statically (the loop is unrolled by their number), which lets the compiler see
// that a read of one slot does not wait on loads into the other.
//
// Products.  A value is the sum of three bfloat16 terms, x = h + m + l with
// h = bf16(x), m = bf16(x - h), l = x - h - m, exactly (24 significant bits
// are 3 times 8), for |x| from 2^-110 (SplitRange), and a product is ha hb +
// ha mb + ma hb + ma mb + ha lb + la hb: the dropped terms are at most 2^-24
// of it (the rounding of one FP32 addition; 2^-27.5 in the mean square of
// pairs in [1, 2), 2^-26.5 with both mantissas below 1 + 2^-8, of which 2.8 %
// pass 2^-25).  An operand with an entry outside that range, as its record's
// mark says, is multiplied on the FP32 matrix cores.
// Six v_mfma_f32_32x32x16_bf16 do 16 k in 192 cycles where eight
// v_mfma_f32_32x32x2_f32 took 512, and an accumulator is added to 12 times per
// 16 k (two real products) instead of 32, the small terms of both products
// first, so that only the last two additions round in the last bits of a short
// sum (product by product, 0.6 % faster, the first and last columns were 0.69e-7 at
// K = 16 and 0.52e-7).  Error against 64 bits of 1024 x 1152 outputs (2-norm),
// here and on the FP32 matrix cores:
//              normal          positive      modulus 1     one entry a row
//     K = 16   0.38e-7 1.03e-7 0.38e-7 0.85e-7 0.36e-7 1.03e-7 0.35e-7 0.31e-7
//     K = 64   1.52e-7 2.03e-7 1.17e-7 1.59e-7 1.50e-7 2.03e-7 0.35e-7 0.31e-7
//     K = 256  3.36e-7 4.06e-7 2.35e-7 3.06e-7 3.29e-7 4.05e-7 0.35e-7 0.31e-7
// (one complex64 multiplication: 0.38e-7).  The two products of order three as
// well change these numbers in the third digit, at 1.19 times the time.
// The terms are formed in registers from the float fragments (seven
// instructions for two values, 32 rows x 16 k of each operand half per wave
// and stage), so the planes, the permutations and the fused epilogues stay FP32
// and no operand takes more memory.
// The complex product takes four real ones whatever the form flag says
// (Gauss's three would need a third accumulator set: one block per CU).
//
// Bound: the matrix cores, at the clock their power allows.  The five GEMMs of
// eight 30-qubit amplitudes: 43.3 ms, against 66.5 on the FP32 matrix cores in
// their 3M form; 1636 TFLOP/s of bf16 products, 0.91 of the 1800 that the matrix
// cores sustain with no memory traffic on operands that change; matrix cores
// busy 0.66-0.68.
//
// Block = 4 waves in a 2 x 2 grid over a 128 x 128 output tile, two blocks per
// CU (64 KB of LDS, 248 registers): one block's splits, fragment reads and
// barrier overlap the other's products.  Each wave has 64 x 64 outputs as 2 x 2
// MFMA tiles: lane l supplies A[l%32][8(l/32) .. + 7] and the same k of column
// l%32 of B, and holds C[8(v/4) + 4(l/32) + v%4][l%32] in accumulator v.  Rows
// are 64 bytes; row r's chunk c sits at position c ^ swz(r), so the rows one
// LDS access touches fall on distinct banks.  A stage is 96 MFMAs per wave.
#include <type_traits>

#include "tn_device.h"

namespace tn {

typedef float v16f_c __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int v4u_f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf_f __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void lds_void_f;

constexpr int FBK = 16;               // k per stage

// s_waitcnt immediate: vmcnt(v) expcnt(7) lgkmcnt(0)
__host__ __device__ constexpr int f_wait_imm(int v) { return (v & 15) | ((v >> 4) << 14) | (7 << 4); }

// (b3 ^ b1, b2) of the row index: rows r..r+15 cover every (r % 4, chunk)
// pair and rows r..r+7 every (r % 2, chunk) pair once
__device__ __forceinline__ int fswz(int r) {
  return ((((r >> 3) ^ (r >> 1)) & 1) << 1) | ((r >> 2) & 1);
}

__device__ __forceinline__ v16f_c mfma_bf(v4u_f a, v4u_f b, v16f_c c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf_f, a), __builtin_bit_cast(v8bf_f, b), c, 0, 0, 0);
}

// term indices (0 = h, 1 = m, 2 = l) of the six products
__device__ constexpr int kSplitA[6] = {1, 0, 2, 0, 1, 0};
__device__ constexpr int kSplitB[6] = {1, 2, 0, 1, 0, 0};

// WMW = waves along M (the four waves form a WMW x 4/WMW grid, WT x WT
// outputs each).  WT = 64: 2 gives a 128 x 128 tile, 1 a 64 x 256 tile (for
// M <= 64), 4 a 256 x 64 tile (for N <= 64).  WT = 32: 64 x 64, 32 x 128 and 128 x
// 32, for launches of few blocks and for skinny results (24 MFMAs a stage and
// wave).  Those wait on the stages' way from memory rather than on the matrix
// cores, so four slots keep three stages in flight (64 or 80 KB, two blocks
// per CU).  M 128 x N 512 x K 256, 3 queries: 46 -> 21 us against the 128 x 128
// tile; 16 queries of 16 x 128 x 8192 85 -> 33 us, 4.1 TB/s.

// Two values split at once: v = h + m + l, each term the bfloat16 nearest to
// what the terms before it leave (bits 0-15 of h, m, l: a's terms, bits 16-31:
// b's).  a - h is one dot product of the pair h with (-1, 0), b - h with
// (0, -1): exact, and an instruction less per value than widening h first.
__device__ __forceinline__ void split3(float a, float b, uint32_t lo1, uint32_t hi1, uint32_t &h, uint32_t &m,
                                       uint32_t &l) {
  const tn_bf16x2 e0 = __builtin_bit_cast(tn_bf16x2, lo1), e1 = __builtin_bit_cast(tn_bf16x2, hi1);
  const tn_bf16x2 hv = __builtin_convertvector((tn_f32x2{a, b}), tn_bf16x2);
  const float ra = __builtin_amdgcn_fdot2_f32_bf16(hv, e0, a, false);
  const float rb = __builtin_amdgcn_fdot2_f32_bf16(hv, e1, b, false);
  const tn_bf16x2 mv = __builtin_convertvector((tn_f32x2{ra, rb}), tn_bf16x2);
  const float sa = __builtin_amdgcn_fdot2_f32_bf16(mv, e0, ra, false);
  const float sb = __builtin_amdgcn_fdot2_f32_bf16(mv, e1, rb, false);
  h = __builtin_bit_cast(uint32_t, hv);
  m = __builtin_bit_cast(uint32_t, mv);
  l = __builtin_bit_cast(uint32_t, __builtin_convertvector((tn_f32x2{sa, sb}), tn_bf16x2));
}

template <int WMW, int WT>
__global__ __launch_bounds__(256, 2) void k_cgemm_f32_planes(GemmArgs g) {
  constexpr int WNW = 4 / WMW;
  constexpr int MB = WT / 32;                          // MFMA tiles a wave has each way
  constexpr int BM = WT * WMW, BN = WT * WNW;          // tile rows of A and of B
  constexpr int APL = BM * FBK, BPL = BN * FBK;        // floats per plane tile
  constexpr int FSTAGE = 2 * (APL + BPL);              // A re, A im, B re, B im
  // load instructions per wave and plane (a 32-row plane takes two waves; the
  // other two load the other plane)
  constexpr int JA = BM > 32 ? BM / 64 : 1, JB = BN > 32 ? BN / 64 : 1;
  constexpr int PA = BM > 32 ? 2 : 1, PB = BN > 32 ? 2 : 1;
  constexpr int NSLOT = WT == 64 ? 2 : 4;
  constexpr int NLOAD = PA * JA + PB * JB;             // a wave's loads of a stage
  __shared__ __align__(16) float ring0[FSTAGE], ring1[FSTAGE];
  __shared__ __align__(16) float ring2[NSLOT == 4 ? FSTAGE : 4], ring3[NSLOT == 4 ? FSTAGE : 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WNW, wn = wave % WNW;
  const int q = blockIdx.y;
  const float *A = (const float *)g.A + q * g.abs;
  const float *B = (const float *)g.B + q * g.bbs;
  const Slot *sa = g.sa + q * g.sabs;
  const Slot *sb = g.sb + q * g.sbbs;
  Slot *sc = g.sc + q * g.scbs;
  int ks;
  int64_t t;
  gemm_block_tile(g, ks, t);  // XCD-aware block -> (k chunk, tile)
  const int64_t m0 = (t % g.tiles_m) * BM, n0 = (t / g.tiles_m) * BN;
  const int64_t kbeg = (int64_t)ks * g.kchunk;
  const int64_t kend = g.K < kbeg + g.kchunk ? g.K : kbeg + g.kchunk;
  const int ea = tn_scale_exp(sa->maxbits), eb = tn_scale_exp(sb->maxbits);
  if (blockIdx.x == 0 && tid == 0) sc->log2s = sa->log2s + sb->log2s + (double)(ea + eb);

  v16f_c acc[MB][MB][2];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][c][v] = 0.0f;

  // this lane's loads: instruction j covers rows (R / 4) * wave + 16 * j +
  // lane / 4 of an R-row plane tile (R = 32: 16 * (wave % 2) + lane / 4 of
  // plane wave / 2); position lane % 4 of the row holds
  // logical chunk (lane % 4) ^ fswz(row) (rows past M or N clamped to the
  // last one)
  const uint8_t *abase = (const uint8_t *)(A + m0 * FBK);
  const uint8_t *bbase = (const uint8_t *)(B + n0 * FBK);
  uint32_t aoff[JA], boff[JB];
  constexpr int WA = BM > 32 ? BM / 4 : 16, WB = BN > 32 ? BN / 4 : 16;
  const int wa = BM > 32 ? wave : wave & 1, wb = BN > 32 ? wave : wave & 1;
  // the plane this wave loads where it loads one
  const int apl = BM > 32 ? 0 : wave >> 1, bpl = BN > 32 ? 0 : wave >> 1;
#pragma unroll
  for (int j = 0; j < JA; ++j) {
    const int r = WA * wa + 16 * j + (lane >> 2);
    const int c = (lane & 3) ^ fswz(r);
    const int64_t ra_ = m0 + r < g.M ? r : g.M - 1 - m0;
    aoff[j] = (uint32_t)((ra_ * FBK + c * 4) * 4);
  }
#pragma unroll
  for (int j = 0; j < JB; ++j) {
    const int r = WB * wb + 16 * j + (lane >> 2);
    const int c = (lane & 3) ^ fswz(r);
    const int64_t rb_ = n0 + r < g.N ? r : g.N - 1 - n0;
    boff[j] = (uint32_t)((rb_ * FBK + c * 4) * 4);
  }
  const int64_t nk = (kend - kbeg) / FBK;
#define TN_FRING(S) ((S) == 0 ? ring0 : (S) == 1 ? ring1 : (S) == 2 ? ring2 : ring3)
  auto issue = [&](auto slot, int64_t stg) {
    constexpr int S = decltype(slot)::value;
    float *rb = TN_FRING(S);
    const int64_t kb = kbeg / FBK + (stg < nk ? stg : nk - 1);
    const uint8_t *ak = abase + kb * g.M * FBK * 4, *bk = bbase + kb * g.N * FBK * 4;
#pragma unroll
    for (int pl = 0; pl < 2; ++pl) {
      if (pl < PA) {
        const int p = pl + apl;
#pragma unroll
        for (int j = 0; j < JA; ++j)
          __builtin_amdgcn_global_load_lds((const void *)(ak + p * g.pa * 4 + aoff[j]),
                                           (lds_void_f *)(rb + p * APL + (WA * wa + 16 * j) * FBK), 16, 0, 0);
      }
      if (pl < PB) {
        const int p = pl + bpl;
#pragma unroll
        for (int j = 0; j < JB; ++j)
          __builtin_amdgcn_global_load_lds((const void *)(bk + p * g.pb * 4 + boff[j]),
                                           (lds_void_f *)(rb + 2 * APL + p * BPL + (WB * wb + 16 * j) * FBK),
                                           16, 0, 0);
      }
    }
  };
  // a lane's eight k (8h .. 8h + 7 of lane half h) of row `row` of a plane
  // tile: logical chunks 2h and 2h + 1
  const int fr = lane & 31, fh = lane >> 5;
  const int fp0 = ((2 * fh) ^ fswz(fr)) * 4, fp1 = ((2 * fh + 1) ^ fswz(fr)) * 4;
  // the constant pairs of split3, kept in scalar registers (opaque, so that
  // they are not folded into packed inline constants)
  uint32_t lo1 = 0x0000bf80u, hi1 = 0xbf800000u;
  asm volatile("" : "+s"(lo1), "+s"(hi1));
  auto split = [&](const float *row, v4u_f (&t3)[3]) {
    const v4f x = *(const v4f *)(row + fp0), y = *(const v4f *)(row + fp1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t h, m, l;
      split3(i < 2 ? x[2 * i] : y[2 * i - 4], i < 2 ? x[2 * i + 1] : y[2 * i - 3], lo1, hi1, h, m, l);
      t3[0][i] = h;
      t3[1][i] = m;
      t3[2][i] = l;
    }
  };
  auto stage = [&](auto slot, int64_t kt) {
    constexpr int S = decltype(slot)::value;
    const float *rb = TN_FRING(S);
    __builtin_amdgcn_s_waitcnt(f_wait_imm((NSLOT - 2) * NLOAD));
    __builtin_amdgcn_s_barrier();
    issue(std::integral_constant<int, (S + NSLOT - 1) % NSLOT>(), kt + NSLOT - 1);
    v4u_f a[MB][2][3];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int pl = 0; pl < 2; ++pl) split(rb + pl * APL + (wm * WT + mb * 32 + fr) * FBK, a[mb][pl]);
#pragma unroll
    for (int nb = 0; nb < MB; ++nb) {
      v4u_f b[2][3];
#pragma unroll
      for (int pl = 0; pl < 2; ++pl) split(rb + 2 * APL + pl * BPL + (wn * WT + nb * 32 + fr) * FBK, b[pl]);
      // the six products of total order at most two, smallest first, and of
      // both of a part's real products before the next larger
#pragma unroll
      for (int pi = 0; pi < 6; ++pi) {
        const int x = kSplitA[pi], y = kSplitB[pi];
        const v4u_f bn = b[1][y] ^ 0x80008000u;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          acc[mb][nb][0] = mfma_bf(a[mb][0][x], b[0][y], acc[mb][nb][0]);
          acc[mb][nb][1] = mfma_bf(a[mb][1][x], b[0][y], acc[mb][nb][1]);
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          acc[mb][nb][0] = mfma_bf(a[mb][1][x], bn, acc[mb][nb][0]);
          acc[mb][nb][1] = mfma_bf(a[mb][0][x], b[1][y], acc[mb][nb][1]);
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // the same stage on the FP32 matrix cores (four real products per complex
  // one), for an operand with entries that three terms do not hold
  auto stage32 = [&](auto slot, int64_t kt) {
    constexpr int S = decltype(slot)::value;
    const float *rb = TN_FRING(S);
    __builtin_amdgcn_s_waitcnt(f_wait_imm((NSLOT - 2) * NLOAD));
    __builtin_amdgcn_s_barrier();
    issue(std::integral_constant<int, (S + NSLOT - 1) % NSLOT>(), kt + NSLOT - 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int fp = h ? fp1 : fp0;
      v4f a[MB][2], b[MB][2];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int pl = 0; pl < 2; ++pl) {
          a[mb][pl] = *(const v4f *)(rb + pl * APL + (wm * WT + mb * 32 + fr) * FBK + fp);
          b[mb][pl] = *(const v4f *)(rb + 2 * APL + pl * BPL + (wn * WT + mb * 32 + fr) * FBK + fp);
        }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int nb = 0; nb < MB; ++nb) {
            const float ar = a[mb][0][s], ai = a[mb][1][s], br = b[nb][0][s], bi = b[nb][1][s];
            acc[mb][nb][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar, br, acc[mb][nb][0], 0, 0, 0);
            acc[mb][nb][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar, bi, acc[mb][nb][1], 0, 0, 0);
            acc[mb][nb][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(-ai, bi, acc[mb][nb][0], 0, 0, 0);
            acc[mb][nb][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(ai, br, acc[mb][nb][1], 0, 0, 0);
          }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
#undef TN_FRING
  const std::integral_constant<int, 0> s0;
  const std::integral_constant<int, 1> s1;
  const std::integral_constant<int, NSLOT == 4 ? 2 : 0> s2;
  const std::integral_constant<int, NSLOT == 4 ? 3 : 1> s3;
  __builtin_amdgcn_s_waitcnt(0);  // nothing else in flight when the ring starts
  issue(s0, 0);
  if (NSLOT == 4) {
    issue(s1, 1);
    issue(s2, 2);
  }
  auto run = [&](auto one) {
    int64_t kt = 0;
    if (NSLOT == 4) {
      for (; kt + 4 <= nk; kt += 4) {
        one(s0, kt);
        one(s1, kt + 1);
        one(s2, kt + 2);
        one(s3, kt + 3);
      }
      if (kt < nk) one(s0, kt);
      if (kt + 1 < nk) one(s1, kt + 1);
      if (kt + 2 < nk) one(s2, kt + 2);
    } else {
      for (; kt + 2 <= nk; kt += 2) {
        one(s0, kt);
        one(s1, kt + 1);
      }
      if (kt < nk) one(s0, kt);
    }
  };
  if ((sa->mark | sb->mark) == 0u)
    run(stage);
  else
    run(stage32);
  __builtin_amdgcn_s_waitcnt(0);  // no load may still write LDS when the block ends

  const bool partial = g.ksplit > 1;
  float2 *C = partial ? g.part + q * g.partbs + (int64_t)ks * g.M * g.N : g.C + q * g.cbs;
  const int64_t ldc = partial ? g.N : g.ldc;
  // an operand read as it is (raw) scales the result instead: exact
  const float post = (g.raw_a | g.raw_b) ? ldexpf(1.0f, -(g.raw_a ? ea : 0) - (g.raw_b ? eb : 0)) : 1.0f;
  // or the result as its parent's operand planes
  const bool fo = g.fo_on != 0;
  uint8_t *P = (uint8_t *)(g.C + q * g.cbs), *P1 = P + g.fo_plane * 4;
  PlaneOut<4> po;
  if (fo) po.init(g, m0 + wm * WT + (lane >> 5) * 4, n0 + wn * WT + (lane & 31));
  float mx = 0.0f;
  SplitRange range;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < MB; ++nb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = wm * WT + mb * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
        const int col = wn * WT + nb * 32 + (lane & 31);
        const int64_t cm = m0 + row, cn = n0 + col;
        const float re = acc[mb][nb][0][v] * post, im = acc[mb][nb][1][v] * post;
        if (cm < g.M && cn < g.N) {
          if (fo) {
            const uint32_t d = po.at(mb, nb, v);
            *(float *)(P + d) = re;
            *(float *)(P1 + d) = im;
            range.add(re);
            range.add(im);
          } else {
            C[cm * ldc + cn] = make_float2(re, im);
          }
          mx = fmaxf(mx, fmaxf(fabsf(re), fabsf(im)));
        }
      }
  if (!partial) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    if (lane == 0) slot_max(&sc->maxbits, mx);
    if (fo) range.mark(sc);
  }
}

// Tile shape of variant v: 0 = 128 x 128, 1 = 64 x 256, 2 = 256 x 64, 3 = 64 x
// 64, 4 = 32 x 128, 5 = 128 x 32.
int gemm_planes_tile_m(int v) { return v == 1 || v == 3 ? 64 : v == 2 ? 256 : v == 4 ? 32 : 128; }
int gemm_planes_tile_n(int v) { return v == 1 ? 256 : v == 2 || v == 3 ? 64 : v == 5 ? 32 : 128; }

hipError_t launch_gemm_f32_planes(hipStream_t st, const GemmArgs &g0, int form, int nbatch) {
  GemmArgs g = g0;
  if (g.opA != 0 || g.opB != 1 || g.planes != 2 || !g.ktile || g.K % FBK != 0 ||
      (form != kForm4M && form != kForm3M) || g.tile < 0 || g.tile > 5 || (g.fo_on && g.ksplit > 1))
    return hipErrorInvalidValue;
  const int tm = gemm_planes_tile_m(g.tile), tn = gemm_planes_tile_n(g.tile);
  g.tiles_m = (int)((g.M + tm - 1) / tm);
  g.tiles_n = (int)((g.N + tn - 1) / tn);
  if (g.ksplit < 1) g.ksplit = 1;
  if (g.ksplit == 1) g.kchunk = g.K;
  if (g.kchunk < 1 || g.kchunk % FBK != 0 || (int64_t)g.ksplit * g.kchunk < g.K ||
      (g.ksplit > 1 && !g.part))
    return hipErrorInvalidValue;
  const int64_t blocks = (int64_t)g.tiles_m * g.tiles_n * g.ksplit;
  if (blocks <= 0 || blocks > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks, nbatch);
#define TN_F32P(W, T) hipLaunchKernelGGL((k_cgemm_f32_planes<W, T>), grid, dim3(256), 0, st, g)
  if (g.tile == 0) TN_F32P(2, 64);
  else if (g.tile == 1) TN_F32P(1, 64);
  else if (g.tile == 2) TN_F32P(4, 64);
  else if (g.tile == 3) TN_F32P(2, 32);
  else if (g.tile == 4) TN_F32P(1, 32);
  else TN_F32P(4, 32);
#undef TN_F32P
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || g.ksplit == 1) return e;
  return launch_splitk_reduce(st, g, nbatch);
}

}  // namespace tn
