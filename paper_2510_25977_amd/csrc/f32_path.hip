// fp32 debug path: fp32 storage and arithmetic everywhere (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 fused
// multiply-adds), every intermediate in fp32.  It exists to validate the boundary, the input generators and the oracle
// plumbing independently of the bf16 kernels, takes any extents, reads the factors as the caller stores them, and serves
// the single factored linear layer O = (X U) V (paper Sec. 4.2.1).
#include "common.h"
#include "row4.h"

namespace svdmlp {

// C[M,N] = A[M,K] B[K,N]           (GATED == false; blockIdx.z = 1: B2 in place of B, C one strip further)
// C[M,N] = SiLU(A B) .* (A2 B2)    (GATED == true; epilogue of paper Alg. 3)
// Row-major with leading dimensions lda / ldb / ldc.
//
// What bounds it: the fp32 matrix rate (256 FLOP per clock and CU, a quarter of an 8 KiB operand panel per 64 clocks)
// while there are enough tiles, memory round trips otherwise.  A workgroup of eight waves owns BM x 64 outputs
// (BM = 64, or 32 for up to 32 rows) and takes 64 of the contraction per step; a wave owns 32 x 32 of them and
// 64 / WK of each step, so that small tiles still keep two waves per SIMD busy and a step's loads (all issued before
// the previous step's arithmetic) are wide: 16 bytes per lane, four rows of 256 bytes per wave.  Short outputs with a
// long contraction are cut into ranges over K on top (blockIdx.y, f32_ranges), whose partial tiles k_f32_reduce adds.
// Measured at M = 512, d = 2048, ffn = 8192, r = r_down = 256: 2559 us per forward with 64 x 64 x 16 tiles of scalar
// FMAs and scalar loads, no ranges; 102 us with this kernel, 79 TFLOP/s.  Traced one by one the launches take 15.6 + 4.8,
// 54.0, 28.0 + 4.7 and 9.2 us, 116 in all: in a stream each starts while the one before it ends.  Rows that do not start at
// 16 bytes are read 16 bytes at a time all the same (load4); with four loads of a float each, factored layers and blocks of
// odd extents took a quarter longer: M = 20, d = 1999, ffn = 6001, r = 333 53.6 -> 41.4 us; M = 250, 1001, 2503, 203
// 59.3 -> 48.1; O = (X U) V of 512 rows, 777, 3333, r = 99 28.8 -> 21.8; aligned extents level.  The matrix cores are
// busy half of the second product's time and a third of the others', without LDS bank conflicts.
//
// Rounding: every 16 contraction indices are summed from zero in one accumulator tile and then added to the running
// total, which keeps the fp32 rounding error of long contractions (K = ffn) well below 1e-6 relative.
struct F32Args {
  const float *A, *A2, *B, *B2;
  float* C;
  float* part;              // ranges > 1: [range][z][tile][BM][64]
  int lda, ldb, ldc;
  int M, N, K;
  int strip;                // distance of the second product's columns in C (z = 1)
  int nt;                   // 64-column tiles
  int ranges, klen;         // ranges over K and their length (a multiple of 64)
  int tiles, nz;            // ranges > 1: output tiles of one product, products in the launch
};

typedef f32x4 __attribute__((aligned(4))) f32x4u;   // at any float

constexpr int BN = 64;
constexpr int SB = BN + 8;  // row length of the B panel in LDS: rows 4 apart (the two halves of a wave) shift by 32 banks

template <int BM, bool GATED, bool VEC_A, bool VEC_B>
__global__ __launch_bounds__(512) void k_f32_mm(F32Args a) {
  constexpr int WM = BM / 32, WN = BN / 32, WK = 8 / (WM * WN);
  constexpr int NG = GATED ? 2 : 1;
  // contraction per step: a gated product of 64 rows takes half as much, or its operands and partial sums would take 195
  // registers a lane, which is one workgroup on the CU; with 127 it is two (the forward of the sizes above 111.2 us with
  // steps of 64, 102.1 with steps of 32)
  constexpr int BK = GATED && BM == 64 ? 32 : 64;
  constexpr int SA = BK + 4;                // row length of the A panel: 16 rows fall into different banks (16-byte reads)
  constexpr int CH = BK / WK / 16;          // 16-wide pieces of a step per wave
  constexpr int GP = 4 / WK;                // groups of four accumulator registers a wave finishes
  constexpr int PANEL = BM * SA + BK * SB;
  constexpr int RED = 8 * (4 - GP) * 256;   // floats the waves hand each other at the end
  __shared__ __attribute__((aligned(16))) float lds[NG * (PANEL > RED ? PANEL : RED)];
  const int t = threadIdx.x, lane = t % 64, w = __builtin_amdgcn_readfirstlane(t / 64);
  const int wk = w / (WM * WN), wm = (w / WN) % WM, wn = w % WN;
  const int il = lane % 32, h = lane / 32;
  // rows and columns in grid dimensions of their own: their product may pass what one dimension takes
  const int z = (int)blockIdx.z >= a.ranges, range = blockIdx.z - z * a.ranges;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int kbeg = range * a.klen, kend = kbeg + a.klen < a.K ? kbeg + a.klen : a.K;

  const float* Ap[NG] = {};
  const float* Bp[NG] = {};
  Ap[0] = a.A;
  Bp[0] = z ? a.B2 : a.B;
  if (GATED) { Ap[NG - 1] = a.A2; Bp[NG - 1] = a.B2; }
  // panel loads, four floats per thread and pass
  constexpr int TA = BK / 4, RA = 512 / TA < BM ? 512 / TA : BM, PA = BM / RA;   // threads per row of A, rows and number of passes
  constexpr int PB = BK / 32;
  const int arow = t / TA, acol = 4 * (t % TA), brow = t / 16, bcol = 4 * (t % 16);
  f32x4 ra[NG][PA], rb[NG][PB];
  // Four floats of a row.  Nothing looks at the values here, so that the loads stay in flight over the arithmetic of
  // the step before.  Wide loads take any row that has four floats, aligned to 16 bytes or not: four that would pass the end of
  // the row (lim) are its last four and are shifted into place on the way to LDS, in the steps and tiles that have such
  // columns at all.  What lies beyond the contraction is zeroed there.
  auto load4 = [&](const float* row, int c, int lim, bool wide) __attribute__((always_inline)) {
    f32x4 v;
    if (wide) {
      v = *reinterpret_cast<const f32x4u*>(row + row4_start(c, lim));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = row[c + e < lim ? c + e : 0];
    }
    return v;
  };
  auto load = [&](int k) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < NG; ++n) {
#pragma unroll
      for (int p = 0; p < PA; ++p) {
        const int m = m0 + RA * p + arow;   // rows beyond M only feed outputs that are not stored
        ra[n][p] = load4(Ap[n] + (size_t)(m < a.M ? m : a.M - 1) * a.lda, k + acol, a.K, VEC_A);
      }
#pragma unroll
      for (int p = 0; p < PB; ++p) {        // ... and so do columns beyond N
        const int kk = k + 32 * p + brow;
        rb[n][p] = load4(Bp[n] + (size_t)(kk < kend ? kk : kbeg) * a.ldb, n0 + bcol, a.N, VEC_B);
      }
    }
  };
  auto zero_tail = [&](int k) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < NG; ++n) {
#pragma unroll
      for (int p = 0; p < PA; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) ra[n][p][e] = k + acol + e < kend ? ra[n][p][e] : 0.f;
#pragma unroll
      for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) rb[n][p][e] = k + 32 * p + brow < kend ? rb[n][p][e] : 0.f;
    }
  };

  f32x16 acc[NG];
#pragma unroll
  for (int n = 0; n < NG; ++n)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[n][e] = 0.f;
  load(kbeg);
  for (int k = kbeg; k < kend; k += BK) {
    if (VEC_B && n0 + BN > a.N && a.N % 4) {
#pragma unroll
      for (int n = 0; n < NG; ++n)
#pragma unroll
        for (int p = 0; p < PB; ++p) row4_place(rb[n][p], n0 + bcol, a.N);
    }
    if (k + BK > kend) {
      if (VEC_A && k + BK > a.K && a.K % 4) {
#pragma unroll
        for (int n = 0; n < NG; ++n)
#pragma unroll
          for (int p = 0; p < PA; ++p) row4_place(ra[n][p], k + acol, a.K);
      }
      zero_tail(k);
    }
#pragma unroll
    for (int n = 0; n < NG; ++n) {
      float* sA = lds + n * PANEL;
      float* sB = sA + BM * SA;
#pragma unroll
      for (int p = 0; p < PA; ++p) *reinterpret_cast<f32x4*>(sA + (RA * p + arow) * SA + acol) = ra[n][p];
#pragma unroll
      for (int p = 0; p < PB; ++p) *reinterpret_cast<f32x4*>(sB + (32 * p + brow) * SB + bcol) = rb[n][p];
    }
    __syncthreads();
    if (k + BK < kend) load(k + BK);
    // the order of a contraction is free: lane half h takes indices 4 h .. 4 h + 3 of every eight.  All operands of the
    // step are read first and the independent sums of its pieces take turns, so that neither an LDS round trip nor the
    // latency of a dependent MFMA stands between two of them.
    f32x4 av[NG][CH][2], bv[NG][CH][2];
#pragma unroll
    for (int n = 0; n < NG; ++n)
#pragma unroll
      for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const float* sA = lds + n * PANEL;
          const float* sB = sA + BM * SA;
          const int kk = (wk * CH + c) * 16 + 8 * g + 4 * h;
          av[n][c][g] = *reinterpret_cast<const f32x4*>(sA + (32 * wm + il) * SA + kk);
#pragma unroll
          for (int e = 0; e < 4; ++e) bv[n][c][g][e] = sB[(kk + e) * SB + 32 * wn + il];
        }
    __builtin_amdgcn_sched_barrier(0);
    f32x16 part[NG][CH];
#pragma unroll
    for (int n = 0; n < NG; ++n)
#pragma unroll
      for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) part[n][c][e] = 0.f;
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < NG; ++n)
#pragma unroll
          for (int c = 0; c < CH; ++c)
            part[n][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[n][c][g][e], bv[n][c][g][e], part[n][c], 0, 0, 0);
#pragma unroll
    for (int n = 0; n < NG; ++n)
#pragma unroll
      for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[n][e] += part[n][c][e];
    __syncthreads();
  }

  // Sum the WK waves that share outputs, in order: wave wk finishes register groups GP wk .. of the 32 x 32 tile and
  // leaves the others for its partners.
  auto slot = [&](int n, int wave, int k, int g) __attribute__((always_inline)) {   // k: the wave's share of the step
    return lds + n * RED + (wave * (4 - GP) + (g < k * GP ? g : g - GP)) * 256 + lane * 4;
  };
#pragma unroll
  for (int n = 0; n < NG; ++n)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if (g / GP != wk)
        *reinterpret_cast<f32x4*>(slot(n, w, wk, g)) = f32x4{acc[n][4 * g], acc[n][4 * g + 1], acc[n][4 * g + 2], acc[n][4 * g + 3]};
  __syncthreads();
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    if (g / GP != wk) continue;
    f32x4 v[NG];
#pragma unroll
    for (int n = 0; n < NG; ++n) {
      v[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < WK; ++q) {
        if (q == wk) v[n] += f32x4{acc[n][4 * g], acc[n][4 * g + 1], acc[n][4 * g + 2], acc[n][4 * g + 3]};
        else v[n] += *reinterpret_cast<const f32x4*>(slot(n, q * WM * WN + wm * WN + wn, q, g));
      }
    }
    if (GATED)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[0][e] = v[0][e] / (1.0f + expf(-v[0][e])) * v[NG - 1][e];
    // registers 4 g .. 4 g + 3 of a lane: rows 8 g + 4 h + e of column il
    const int rl = 32 * wm + 8 * g + 4 * h, cl = 32 * wn + il;
    if (a.ranges > 1) {
      float* dst = a.part + ((size_t)(range * a.nz + z) * a.tiles + blockIdx.y * a.nt + blockIdx.x) * (BM * BN) + cl;
#pragma unroll
      for (int e = 0; e < 4; ++e) dst[(rl + e) * BN] = v[0][e];
    } else if (n0 + cl < a.N) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (m0 + rl + e < a.M) a.C[(size_t)(m0 + rl + e) * a.ldc + z * a.strip + n0 + cl] = v[0][e];
    }
  }
}

// C = sum of the ranges' partial tiles, in order; one thread per four columns of a row of a tile
__global__ __launch_bounds__(256) void k_f32_reduce(F32Args a, int BM) {
  const int q = blockIdx.x * 256 + threadIdx.x;
  const int per = BM * BN / 4, zt = q / per, o = q % per;
  if (zt >= a.nz * a.tiles) return;
  const float* src = a.part + (size_t)zt * (BM * BN) + 4 * o;
  const size_t stride = (size_t)a.nz * a.tiles * (BM * BN);
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < a.ranges; s0 += 4) {   // four loads in flight, additions in order
    f32x4 x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = *reinterpret_cast<const f32x4*>(src + (s0 + j < a.ranges ? s0 + j : a.ranges - 1) * stride);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (s0 + j < a.ranges) v += x[j];
  }
  const int z = zt / a.tiles, tile = zt % a.tiles;
  const int m = tile / a.nt * BM + o / (BN / 4), n = tile % a.nt * BN + 4 * (o % (BN / 4));
  if (m >= a.M) return;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (n + e < a.N) a.C[(size_t)m * a.ldc + z * a.strip + n + e] = v[e];
}

int f32_rows(int64_t M) { return M <= 32 ? 32 : 64; }

// Ranges over K: two workgroups per CU if the contraction has that many pieces of 256 (four steps: fewer and a range
// is all latency), at most sixteen; none where the tiles fill the chip by themselves.
int f32_ranges(int64_t tiles, int64_t K) {
  if (tiles > 256) return 1;
  int64_t s = (512 + tiles - 1) / tiles;
  if (s > K / 256) s = K / 256;
  if (s > 16) s = 16;
  return s < 1 ? 1 : (int)s;
}

// floats of partial tiles a product of M rows takes (nz products of N columns at once)
size_t f32_part_floats(int64_t M, int64_t N, int64_t K, int nz) {
  const int64_t bm = f32_rows(M), tiles = (M + bm - 1) / bm * ((N + BN - 1) / BN) * nz;
  const int s = f32_ranges(tiles, K);
  return s > 1 ? (size_t)s * tiles * bm * BN : 0;
}

F32Cut f32_cut(int64_t M, int64_t N, int64_t K, int nz, bool gated) {
  F32Cut c;
  c.rows = f32_rows(M);
  c.mt = (int)((M + c.rows - 1) / c.rows);
  c.nt = (int)((N + BN - 1) / BN);
  const int want = gated ? 1 : f32_ranges((int64_t)c.mt * c.nt * nz, K);
  c.klen = (int)((K + (int64_t)want * 64 - 1) / ((int64_t)want * 64)) * 64;
  c.ranges = (int)((K + c.klen - 1) / c.klen);
  return c;
}

template <bool GATED, bool VEC_A, bool VEC_B>
static void launch(int BM, dim3 grid, const F32Args& a, hipStream_t st) {
  if (BM == 32) hipLaunchKernelGGL((k_f32_mm<32, GATED, VEC_A, VEC_B>), grid, dim3(512), 0, st, a);
  else hipLaunchKernelGGL((k_f32_mm<64, GATED, VEC_A, VEC_B>), grid, dim3(512), 0, st, a);
}

static int mm(const Ctx* c, const float* A, const float* A2, int64_t lda, const float* B, const float* B2, int64_t N, bool gated,
              float* C, int64_t ldc, int64_t strip, int64_t M, int64_t K, hipStream_t st) {
  const int nz = strip ? 2 : 1;
  const F32Cut cut = f32_cut(M, N, K, nz, gated);
  const int BM = cut.rows;
  const int64_t tiles = (int64_t)cut.mt * cut.nt;
  F32Args a;
  a.A = A; a.A2 = A2; a.B = B; a.B2 = B2; a.C = C;
  a.part = reinterpret_cast<float*>(c->ws) + c->plan.f32_part;
  a.lda = (int)lda; a.ldb = (int)N; a.ldc = (int)ldc;
  a.M = (int)M; a.N = (int)N; a.K = (int)K;
  a.strip = (int)strip;
  a.nt = cut.nt;
  a.klen = cut.klen;
  a.ranges = cut.ranges;
  a.tiles = a.ranges > 1 ? (int)tiles : 0;
  a.nz = nz;
  const dim3 grid(cut.nt, cut.mt, a.ranges * nz);
  // rows of A / B have four floats or not (the gated product's A is an intermediate, whose rows always do)
  const bool va = lda >= 4, vb = N >= 4;
  if (gated) {
    if (vb) launch<true, true, true>(BM, grid, a, st);
    else launch<true, true, false>(BM, grid, a, st);
  } else if (va) {
    if (vb) launch<false, true, true>(BM, grid, a, st);
    else launch<false, true, false>(BM, grid, a, st);
  } else {
    if (vb) launch<false, false, true>(BM, grid, a, st);
    else launch<false, false, false>(BM, grid, a, st);
  }
  const int e = (int)hipGetLastError();
  if (e || a.ranges == 1) return e;
  const int64_t threads = nz * tiles * BM * BN / 4;
  hipLaunchKernelGGL(k_f32_reduce, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, a, BM);
  return (int)hipGetLastError();
}

int f32_forward(const Ctx* c, const void* Xv, int64_t M, void* Yv, hipStream_t st) {
  const Plan& p = c->plan;
  const svdmlp_desc& de = c->desc;
  const float* X = static_cast<const float*>(Xv);
  float* Y = static_cast<float*>(Yv);
  float* ws = reinterpret_cast<float*>(c->ws);
  const int64_t d = p.d, ffn = p.ffn, r = p.r, rd = p.rd;
  const int64_t rs = f32_stride(r), hs = f32_stride(ffn), ds = f32_stride(rd);
  const float *Ug = (const float*)de.Ug, *Vg = (const float*)de.Vg, *Uu = (const float*)de.Uu, *Vu = (const float*)de.Vu;
  int e;
  float* T = ws + p.f32_T;    // [M, rs], gated: [M, 2 rs] with the gate strip in columns [0, r), the up strip from rs on
  if (p.kind == SVDMLP_LINEAR) {
    if ((e = mm(c, X, nullptr, d, Ug, nullptr, r, false, T, rs, 0, M, d, st))) return e;
    return mm(c, T, nullptr, rs, Vg, nullptr, ffn, false, Y, ffn, 0, M, r, st);
  }
  float* H = ws + p.f32_H;    // [M, hs]
  float* Td = ws + p.f32_Td;  // [M, ds]
  if ((e = mm(c, X, nullptr, d, Ug, Uu, r, false, T, 2 * rs, rs, M, d, st))) return e;
  if ((e = mm(c, T, T + rs, 2 * rs, Vg, Vu, ffn, true, H, hs, 0, M, r, st))) return e;
  if ((e = mm(c, H, nullptr, hs, (const float*)de.Ud, nullptr, rd, false, Td, ds, 0, M, ffn, st))) return e;
  return mm(c, Td, nullptr, ds, (const float*)de.Vd, nullptr, d, false, Y, d, 0, M, rd, st);
}

}  // namespace svdmlp
