// bf16 weight-streaming (decode) path: M <= 128 rows, weight-bandwidth bound.
//
// Each of the four products of the factored MLP (paper Alg. 2) is one launch: up to 32 rows D2 of k_stream_gu16 and the
// others of k_stream16 (16-row activation operands), from 33 rows on D2 of k_stream_gu and the others of k_stream, where
// the row tiles of D1, D4 and D5 may get workgroups of their own:
//   D1  T^T  = [Ug|Uu]^T X^T          split-K over d
//   D2  H^T  = SiLU(Vg^T Tg^T) .* (Vu^T Tu^T)
//   D4  Td^T = Ud^T H^T               split-K over ffn
//   D5  Y^T  = Vd^T Td^T
// Every weight frag (common.h) is read exactly once, straight from HBM into registers with one
// coalesced 16-byte-per-lane load, and multiplied on the matrix cores against the (tiny, L2-resident)
// activation: up to 32 rows one or two operands of the rows that exist, beyond that the frags of the RT = 2 or 4 tiles of
// 32 rows that the batch is padded to.  The contraction range
// of a workgroup is split over its 8 waves; their partial tiles are summed through LDS, and, when the
// contraction is also split over workgroups, through a partial buffer in which the last workgroup to
// arrive (an atomic ticket, no spinning) adds the partials in a fixed order, so results are
// bit-reproducible.  Products are computed transposed (lane = activation row), so each output tile is
// already the chain-order frag the next product consumes.
#include "common.h"
#include <mutex>
#include <type_traits>

namespace svdmlp {

enum { PH_D1 = 0, PH_D2 = 1, PH_D4 = 2, PH_D5 = 3 };
constexpr int SW = 8;  // waves per workgroup

struct StreamArgs {
  const char* W0;       // weight frags (D2: gate)
  const char* W1;       // D2: up frags
  const void* act;      // D1: X row-major bf16; otherwise activation frags [row tile][kb] (D2: Tg at 0, Tu at KB frags),
                        // of k_stream16 and k_stream_gu16 the layout given there
  void* out;            // D1: T frags; D2: H frags; D4: Td frags; D5: Y row-major
  float* part;          // split-K partial tiles [tile][split][accumulator][row tile][16][64]
  int* cnt;             // arrival counters [tile], TICKET_STRIDE ints apart
  int M, KB, tiles, S;  // contraction blocks, output tiles, workgroup-level splits
  int ldx;              // D1: row length of X (= d); D5: row length of Y (= d)
  int r;                // D1: rank (separates gate tiles from up tiles)
  int kb_major;         // weight frag order (1 for Ud)
  int act_rt, out_rt;   // frags between consecutive 32-row tiles of the activation / of the output
  int rtw;              // k_stream: groups of RT row tiles, each group with workgroups of its own (the batch has rtw RT row tiles)
  int* clear;           // D2, D5 of a forward on the static array: ticket lines to set to zero (D2: D4's, D5: D1's); or null
};

constexpr int TICKET_LINES = 2048;   // of each split phase

// A launch has at least a.tiles workgroups.  (gridDim would do, but a kernel that reads it takes 256 bytes of hidden
// arguments more, which the host fills on every launch, whether or not there is anything to clear: 0.6 us of it, eight
// factored layers of 2 .. 22 rows called from Python 96.9 -> 92.4 us.)
__device__ __forceinline__ void clear_tickets(const StreamArgs& a) {
  if (!a.clear) return;
  for (int i = blockIdx.x * SW * 64 + threadIdx.x; i < TICKET_LINES * SW; i += a.tiles * SW * 64)
    a.clear[i / SW * TICKET_STRIDE + i % SW] = 0;
}

// The contraction loop of a wave: blocks k0 .. k1 - 1, U at a time.
// NB = 2: two register buffers.  The loads of a group are issued before the matrix instructions of the group before it,
// so 1 to 2 U weight frags per wave are in flight all the way; one buffer, refilled only once used up, leaves a memory
// round trip open between groups.  The gain of this loop and of k_stream_gu together is given there.  Blocks of the last
// group that lie beyond k1 are loaded from block k1 - 1 again and not multiplied, so U should divide the range well
// (stream_unroll).
// NB = 1: one buffer, for launches of many workgroups, whose waves cover each other's round trips: half the registers
// are worth more there (launch_stream_rt).
// load(buffer, u, kb) and mma(buffer, u) are the caller's.
template <int U, int NB, class Load, class Mma>
__device__ __forceinline__ void stream_loop(int k0, int k1, Load&& load, Mma&& mma) {
  if (k0 >= k1) return;
  constexpr std::integral_constant<int, 0> B0{};
  if constexpr (NB == 1) {
    auto group = [&](auto n, int kb) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < n; ++u) load(B0, u, kb + u);
#pragma unroll
      for (int u = 0; u < n; ++u) mma(B0, u);
    };
    static_assert(U == 4 || U == 2, "groups of four, two, one");
    int kb = k0;
    for (; kb + U <= k1; kb += U) group(std::integral_constant<int, U>{}, kb);
    if (U == 4 && kb + 2 <= k1) {
      group(std::integral_constant<int, 2>{}, kb);
      kb += 2;
    }
    if (kb < k1) group(std::integral_constant<int, 1>{}, kb);
  } else {
    constexpr std::integral_constant<int, 1> B1{};
    auto fill = [&](auto buf, int kb) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < U; ++u) load(buf, u, kb + u < k1 ? kb + u : k1 - 1);
    };
    auto use = [&](auto buf, int kb) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (kb + u < k1) mma(buf, u);
    };
    fill(B0, k0);
    for (int kb = k0; kb < k1; kb += 2 * U) {
      if (kb + U < k1) fill(B1, kb + U);
      use(B0, kb);
      if (kb + U >= k1) break;
      if (kb + 2 * U < k1) fill(B0, kb + 2 * U);
      use(B1, kb + U);
    }
  }
}

// After a wave's write-through stores of its partial tile: takes a ticket once they are acknowledged and returns whether
// it was the last of S; the last one leaves the ticket at zero for the next forward.
__device__ __forceinline__ bool last_to_arrive(int* ticket, int S, int lane) {
  asm volatile("" ::: "memory");
  wait_vmcnt<0>();
  int n = 0;
  if (lane == 0) n = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const bool last = __builtin_amdgcn_readfirstlane(n) == S - 1;
  asm volatile("" ::: "memory");
  if (last && lane == 0) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return last;
}

template <int PH, int RT, int U, int NB>
__global__ __launch_bounds__(SW * 64) void k_stream(StreamArgs a) {
  static_assert(PH == PH_D1 || PH == PH_D4 || PH == PH_D5, "D2 is k_stream_gu");
  // staging of accumulator tiles: [row tile][wave][registers 4 p .. 4 p + 3][lane], 16 bytes per lane
  __shared__ f32x4 red[RT][SW][4][64];
  // the wave index as a scalar: the contraction loop below then has wave-uniform bounds
  const int lane = threadIdx.x % 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  if (PH == PH_D5) clear_tickets(a);
  // Workgroups b, b + 8, .. b + 8 (rtw - 1) run on the same XCD and take the rtw row-tile groups of one (tile, range):
  // the first of them brings the weight frags into that XCD's L2, the others find them there.
  const int idx = (blockIdx.x / (8 * a.rtw)) * 8 + blockIdx.x % 8;
  if (idx >= a.tiles * a.S) return;
  const int rt0 = (blockIdx.x / 8) % a.rtw * RT;          // first row tile of this workgroup
  const int tile = idx / a.S, sp = idx % a.S;
  const int unit = tile * a.rtw + rt0 / RT;               // output tile x row-tile group: owner of partials and ticket
  const int kbs = (a.KB + a.S - 1) / a.S;                 // contraction blocks of this workgroup
  const int kw = (kbs + SW - 1) / SW;                     // ... of each wave
  int k0 = sp * kbs + w * kw;
  int k1 = k0 + kw;
  const int kend = (sp + 1) * kbs < a.KB ? (sp + 1) * kbs : a.KB;
  if (k1 > kend) k1 = kend;

  const int il = lane % 32, h = lane / 32;
  const size_t wstride = a.kb_major ? (size_t)a.tiles * FRAG_BYTES : (size_t)FRAG_BYTES;
  const char* wp = a.W0 + (a.kb_major ? (size_t)tile : (size_t)tile * a.KB) * FRAG_BYTES + lane * 16;
  const uint16_t* xrow[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int row = 32 * (rt0 + rt) + il;
    xrow[rt] = (PH == PH_D1) ? static_cast<const uint16_t*>(a.act) + (size_t)(row < a.M ? row : a.M - 1) * a.ldx + 8 * h : nullptr;
  }
  const char* af = static_cast<const char*>(a.act) + lane * 16;
  // wave t < 2 RT finishes registers 8 (t % 2) .. + 7 (= one chain-order frag) of row tile t / 2
  const int t = w;
  const int rtf = t / 2, hf = t % 2;

  f32x16 acc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[rt][e] = 0.f;
  bf16x8 wv[NB][U], av[NB][U][RT];
  stream_loop<U, NB>(k0, k1,
      [&](auto b, int u, int kb) __attribute__((always_inline)) {
        wv[b][u] = *reinterpret_cast<const bf16x8*>(wp + (size_t)kb * wstride);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          av[b][u][rt] = PH == PH_D1 ? *reinterpret_cast<const bf16x8*>(xrow[rt] + 16 * kb)
                                     : *reinterpret_cast<const bf16x8*>(af + ((size_t)(rt0 + rt) * a.act_rt + kb) * FRAG_BYTES);
      },
      [&](auto b, int u) __attribute__((always_inline)) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt] = mfma32(wv[b][u], av[b][u][rt], acc[rt]);
      });

  // ---- sum the 8 waves' partial tiles through LDS (fixed order) ----
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int pl = 0; pl < 4; ++pl)
      red[rt][w][pl][lane] = f32x4{acc[rt][4 * pl], acc[rt][4 * pl + 1], acc[rt][4 * pl + 2], acc[rt][4 * pl + 3]};
  __syncthreads();
  if (t >= 2 * RT) return;
  float v[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) v[s] = 0.f;
#pragma unroll
  for (int ww = 0; ww < SW; ++ww) {
    const f32x4 x0 = red[rtf][ww][2 * hf][lane], x1 = red[rtf][ww][2 * hf + 1][lane];
#pragma unroll
    for (int s = 0; s < 4; ++s) { v[s] += x0[s]; v[4 + s] += x1[s]; }
  }
  if (a.S > 1) {
    // Partials cross workgroups (possibly on different XCDs, whose L2s are not coherent with each other) as
    // device-scope relaxed atomics: such stores write through to memory and such loads bypass the local L2,
    // so no cache write-back / invalidate (which a device-scope fence would cost every workgroup) is needed.
    // Ordering: a wave waits for its own stores to be acknowledged, then takes a ticket.  Every finishing wave has a
    // ticket of its own (t-th word of the unit's line): no workgroup barrier in the hand-over.
    const int eo = rtf * 1024 + (8 * hf) * 64 + lane;
    float* mine = a.part + ((size_t)unit * a.S + sp) * RT * 1024 + eo;
#pragma unroll
    for (int s = 0; s < 8; ++s) __hip_atomic_store(mine + s * 64, v[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!last_to_arrive(a.cnt + unit * TICKET_STRIDE + t, a.S, lane)) return;
#pragma unroll
    for (int s = 0; s < 8; ++s) v[s] = 0.f;
    // four partial tiles' worth of loads in flight at a time; the additions stay in split order
    for (int q0 = 0; q0 < a.S; q0 += 4) {
      float tmp[4][8];
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {
        const int q = q0 + qq < a.S ? q0 + qq : a.S - 1;
        const float* src = a.part + ((size_t)unit * a.S + q) * RT * 1024 + eo;
#pragma unroll
        for (int s = 0; s < 8; ++s) tmp[qq][s] = __hip_atomic_load(src + s * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
      for (int qq = 0; qq < 4; ++qq)
        if (q0 + qq < a.S) {
#pragma unroll
          for (int s = 0; s < 8; ++s) v[s] += tmp[qq][s];
        }
    }
  }

  // ---- epilogue ----
  if (PH == PH_D5) {
    // lane = row m; slots s <-> columns 32 tile + 16 hf + 8 (s / 4) + 4 h + s % 4
    const int row = 32 * (rt0 + rtf) + il;
    if (row < a.M) {
      uint16_t* y = static_cast<uint16_t*>(a.out) + (size_t)row * a.ldx + 32 * tile + 16 * hf + 4 * h;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        bf16x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = (__bf16)v[4 * g + i];
        *reinterpret_cast<bf16x4*>(y + 8 * g) = o;
      }
    }
    return;
  }
  bf16x8 o;
#pragma unroll
  for (int s = 0; s < 8; ++s) o[s] = (__bf16)v[s];
  size_t frag = (size_t)(rt0 + rtf) * a.out_rt;
  if (PH == PH_D1) {
    const int p0 = 32 * tile;
    const int which = p0 >= a.r ? 1 : 0;
    frag += (size_t)which * (a.r / 16) + (p0 - which * a.r) / 16 + hf;
  } else {
    frag += (size_t)2 * tile + hf;
  }
  *reinterpret_cast<bf16x8*>(static_cast<char*>(a.out) + (frag * 64 + lane) * 16) = o;
}

// ------------------------------------------------------------------------------------------------
// D2: H^T = SiLU(Vg^T Tg^T) .* (Vu^T Tu^T), one tile of 32 ffn columns per workgroup.  A wave takes one of the two
// products and one of KS = 4 ranges of the contraction: every weight frag is loaded by one wave of the chip, straight
// from HBM, a wave holds one accumulator tile per row tile, and eight tiles per row tile meet in LDS, behind one barrier.
// (Both products in every wave and eight ranges, as before, put twice the tiles through LDS in two to four rounds and
// left registers for half the loads.)  Bound by the weights from HBM up to 32 rows, beyond that also by the activation
// frags, which every workgroup reads from L2.  Two column tiles per workgroup halve those reads but fill the chip
// worse: 2 % faster at 64 rows and r = 1024, 1 to 9 % slower everywhere else.
// Forwards before and after this kernel, the two-buffer loop and the hand-over without barriers: d = 4096, ffn = 14336,
// r = 512, 1 / 16 rows 25.3 -> 23.5 / 25.8 -> 24.0 us; r = 1024, 64 rows 49.3 -> 45.3 us; d = 2048, ffn = 8192,
// r = 256, 128 rows 22.9 -> 19.4 us; d = 8192, ffn = 28672, r = 1536, 8 rows 89.7 -> 85.3 us.
// ------------------------------------------------------------------------------------------------
template <int RT, int U>
__global__ __launch_bounds__(SW * 64) void k_stream_gu(StreamArgs a) {
  constexpr int KS = SW / 2;             // contraction ranges
  __shared__ f32x4 red[SW][RT][4][64];    // [product, range][row tile][registers 4 p .. 4 p + 3][lane]
  const int lane = threadIdx.x % 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int up = w / KS, ks = w % KS;
  clear_tickets(a);
  const int tile = blockIdx.x;
  const int kw = (a.KB + KS - 1) / KS;
  const int k0 = ks * kw, k1 = k0 + kw < a.KB ? k0 + kw : a.KB;
  const char* wp = (up ? a.W1 : a.W0) + (size_t)tile * a.KB * FRAG_BYTES + lane * 16;
  const char* af = static_cast<const char*>(a.act) + (size_t)(up * a.KB) * FRAG_BYTES + lane * 16;
  f32x16 acc[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[rt][e] = 0.f;
  bf16x8 wv[2][U], av[2][U][RT];
  stream_loop<U, 2>(k0, k1,
      [&](auto b, int u, int kb) __attribute__((always_inline)) {
        wv[b][u] = *reinterpret_cast<const bf16x8*>(wp + (size_t)kb * FRAG_BYTES);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          av[b][u][rt] = *reinterpret_cast<const bf16x8*>(af + ((size_t)rt * a.act_rt + kb) * FRAG_BYTES);
      },
      [&](auto b, int u) __attribute__((always_inline)) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt] = mfma32(wv[b][u], av[b][u][rt], acc[rt]);
      });
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int pl = 0; pl < 4; ++pl)
      red[w][rt][pl][lane] = f32x4{acc[rt][4 * pl], acc[rt][4 * pl + 1], acc[rt][4 * pl + 2], acc[rt][4 * pl + 3]};
  __syncthreads();
  // wave w < 2 RT finishes one of the tile's 2 RT frags: registers 8 hf .. + 7 of row tile rt
  static_assert(2 * RT <= SW, "a wave for each of them");
  if (w >= 2 * RT) return;
  const int rt = w / 2, hf = w % 2;
  float v[2][8];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
#pragma unroll
    for (int s = 0; s < 8; ++s) v[n][s] = 0.f;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const f32x4 x0 = red[n * KS + k][rt][2 * hf][lane], x1 = red[n * KS + k][rt][2 * hf + 1][lane];
#pragma unroll
      for (int s = 0; s < 4; ++s) { v[n][s] += x0[s]; v[n][4 + s] += x1[s]; }
    }
  }
  bf16x8 o;
#pragma unroll
  for (int s = 0; s < 8; ++s) o[s] = (__bf16)(v[0][s] * __builtin_amdgcn_rcpf(1.0f + __expf(-v[0][s])) * v[1][s]);
  *reinterpret_cast<bf16x8*>(static_cast<char*>(a.out) + (((size_t)rt * a.out_rt + 2 * tile + hf) * 64 + lane) * 16) = o;
}

// ------------------------------------------------------------------------------------------------
// Up to 32 rows: the same products on 16 x 16 x 32 MFMAs.
// Bound by waiting for memory (requests times their latency, over the launch: 30 lines of 128 bytes open per CU on average in
// D1 and D5, 55 in D4, 85 in D2 at 16 rows).  In the 32-row frags that these phases used to hand over, an activation took as
// many requests as the weights it met, whatever the number of rows.  With operands of 16 rows that hold nothing but the rows
// of the batch it takes half as many at 16 rows and one in sixteen at one row.  d = 4096, ffn = 14336, r = 512 (weights from
// HBM), 1 / 16 rows 23.6 -> 21.6 / 24.0 -> 22.8 us; d = 5120, ffn = 13824, r = 640, 2 rows 30.7 -> 26.7; d = 8192,
// ffn = 28672, r = 1024, 4 rows 53.3 -> 48.8; d = 3072, ffn = 9216, r = 1500, 30 rows 37.0 -> 36.9.
// Contractions are cut over the waves in blocks of 32, those of the 32-row kernels in blocks of 16.  So the order of a sum
// differs from theirs in D2 where r is an odd multiple of 64 (r = 192: ranges of 64, 64, 64, 0 instead of 48, four times) and
// in a last product on 32-column tiles whose rank is an odd multiple of 128; elsewhere the ranges are the same.
// D1 and D4 take one 16-column output tile per workgroup.  They split their contraction over workgroups, and what the split
// costs (the partial tile written through, and above all the read-back of all S partial tiles by one workgroup, past its L2
// and through one CU's bounded fetch rate) goes with the tile size: a 16 x 16 fp32 tile is 1 KiB instead of 4 KiB, and twice
// as many tiles need half as many ranges.  The weight frags are the same ones (32 rows x 16 k, lane-major): a 16-row
// operand of contraction block pair (2 kb2, 2 kb2 + 1) is lanes 16 hn .. + 15 and 32 + 16 hn .. + 15 of those two
// frags, i.e. four 256-byte runs per load; every cache line of a frag is still read by exactly one workgroup.
// Lane l of a wave: row / column i = l % 16, contraction group g = l / 16 (k = 32 kb2 + 8 g .. + 7).
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Activations of these kernels (T, H, Td): [32 contraction indices][g][row < M][8 values], the operand of one MFMA with
// the rows that exist and no others.
template <int MT>
__device__ __forceinline__ void act16_offsets(unsigned (&off)[MT], int M, int i, int g) {
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int row = 16 * mt + i;
    off[mt] = (unsigned)(g * M + (row < M ? row : M - 1)) * 16u;
  }
}
// Columns 16 ct + 4 gp .. + 3 of row m: chain order puts them into half gp / 2 of group 2 (ct % 2) + gp % 2.
__device__ __forceinline__ char* act16_slot(char* act, int M, int ct, int gp, int m) {
  return act + ((size_t)(ct / 2) * 4 + 2 * (ct % 2) + gp % 2) * M * 16 + m * 16 + gp / 2 * 8;
}

// MT = 16-row tiles of the batch (M <= 16 MT <= 32); NH = 16-column tiles per workgroup
template <int PH, int MT, int NH, int U, int NB>
__global__ __launch_bounds__(SW * 64) void k_stream16(StreamArgs a) {
  static_assert(PH == PH_D1 || PH == PH_D4 || PH == PH_D5, "D2 is k_stream_gu16");
  static_assert(MT == 1 || MT == 2, "one 32-row activation tile");
  static_assert(NH == 1 || (NH == 2 && PH == PH_D5), "the cut phases run on 16-column tiles");
  __shared__ f32x4 red[SW][NH * MT][64];
  const int lane = threadIdx.x % 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  if (PH == PH_D5) clear_tickets(a);
  const int tile = blockIdx.x / a.S, sp = blockIdx.x % a.S;   // tile of 16 NH columns, contraction range
  const int KB2 = a.KB / 2;                                // contraction blocks of 32
  const int kbs = (KB2 + a.S - 1) / a.S;
  const int kw = (kbs + SW - 1) / SW;
  int k0 = sp * kbs + w * kw;
  int k1 = k0 + kw;
  const int kend = (sp + 1) * kbs < KB2 ? (sp + 1) * kbs : KB2;
  if (k1 > kend) k1 = kend;

  const int i = lane % 16, g = lane / 16;
  const int tile32 = NH == 2 ? tile : tile / 2, hn0 = NH == 2 ? 0 : tile % 2, tiles32 = NH == 2 ? a.tiles : a.tiles / 2;
  // this lane's 16 bytes within a weight frag, and which frag of the pair
  const size_t wstride = a.kb_major ? (size_t)tiles32 * FRAG_BYTES : (size_t)FRAG_BYTES;   // per 16-k frag
  const char* wbase = a.W0 + (a.kb_major ? (size_t)tile32 : (size_t)tile32 * a.KB) * FRAG_BYTES + (g / 2) * wstride +
                      (16 * hn0 + i + 32 * (g % 2)) * 16;
  unsigned ao[MT];
  if (PH == PH_D1) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int row = 16 * mt + i;
      ao[mt] = (unsigned)(row < a.M ? row : a.M - 1) * (unsigned)a.ldx * 2u + 16 * g;
    }
  } else {
    act16_offsets<MT>(ao, a.M, i, g);
  }
  const size_t astride = PH == PH_D1 ? 64 : (size_t)a.M * 64;

  f32x4 acc[NH][MT];
#pragma unroll
  for (int n = 0; n < NH; ++n)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[n][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 wv[NB][U][NH], av[NB][U][MT];
  stream_loop<U, NB>(k0, k1,
      [&](auto b, int u, int kb) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NH; ++n) wv[b][u][n] = *reinterpret_cast<const bf16x8*>(wbase + (size_t)(2 * kb) * wstride + n * 256);
        const char* ap = static_cast<const char*>(a.act) + kb * astride;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) av[b][u][mt] = *reinterpret_cast<const bf16x8*>(ap + ao[mt]);
      },
      [&](auto b, int u) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NH; ++n)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[n][mt] = mfma16(wv[b][u][n], av[b][u][mt], acc[n][mt]);
      });
  // lane (m = l % 16, g): acc[n][mt][e] = element (output column 4 g + e of tile n, row 16 mt + m)
#pragma unroll
  for (int n = 0; n < NH; ++n)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) red[w][n * MT + mt][lane] = acc[n][mt];
  __syncthreads();
  if (w >= NH * MT) return;   // wave n MT + mt finishes that tile
  const int hn = w / MT, row = 16 * (w % MT) + i;
  f32x4 v = red[0][w][lane];
#pragma unroll
  for (int ww = 1; ww < SW; ++ww) v += red[ww][w][lane];
  if (PH != PH_D5 && a.S > 1) {
    // same exchange as in k_stream: write-through partial, ticket (a word for each of the MT finishing waves), the last
    // one adds in range order
    float* mine = a.part + (((size_t)tile * a.S + sp) * MT + w) * 256;
#pragma unroll
    for (int e = 0; e < 4; ++e) __hip_atomic_store(&mine[e * 64 + lane], v[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!last_to_arrive(a.cnt + tile * TICKET_STRIDE + w, a.S, lane)) return;
    v = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int QB = 8;   // partial tiles in flight (8 KiB); additions in range order
    for (int q0 = 0; q0 < a.S; q0 += QB) {
      f32x4 tmp[QB];
#pragma unroll
      for (int qq = 0; qq < QB; ++qq) {
        const int q = q0 + qq < a.S ? q0 + qq : a.S - 1;
        const float* src = a.part + (((size_t)tile * a.S + q) * MT + w) * 256 + lane;
#pragma unroll
        for (int e = 0; e < 4; ++e) tmp[qq][e] = __hip_atomic_load(src + e * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
      for (int qq = 0; qq < QB; ++qq)
        if (q0 + qq < a.S) v += tmp[qq];
    }
  }
  if (row >= a.M) return;
  bf16x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (__bf16)v[e];
  if (PH == PH_D5)
    *reinterpret_cast<bf16x4*>(static_cast<uint16_t*>(a.out) + (size_t)row * a.ldx + 16 * (NH * tile + hn) + 4 * g) = o;
  else *reinterpret_cast<bf16x4*>(act16_slot(static_cast<char*>(a.out), a.M, tile, g, row)) = o;
}

// D2 for the same batches: 32 ffn columns per workgroup, waves as in k_stream_gu.  Groups of up to four pairs of frags with
// one 16-row tile, of two with two (two with one tile: 2 % slower at d = 4096, r = 512; four with two: 1 % slower at 24 rows).
template <int MT, int U>
__global__ __launch_bounds__(SW * 64) void k_stream_gu16(StreamArgs a) {
  constexpr int KS = SW / 2;             // contraction ranges
  __shared__ f32x4 red[SW][2 * MT][64];   // [product, range][16-column tile, 16-row tile][lane]
  const int lane = threadIdx.x % 64, w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int up = w / KS, ks = w % KS, i = lane % 16, g = lane / 16;
  clear_tickets(a);
  const int tile = blockIdx.x, KB2 = a.KB / 2;
  const int kw = (KB2 + KS - 1) / KS;
  const int k0 = ks * kw, k1 = k0 + kw < KB2 ? k0 + kw : KB2;
  const char* wbase = (up ? a.W1 : a.W0) + ((size_t)tile * a.KB + g / 2) * FRAG_BYTES + (i + 32 * (g % 2)) * 16;
  const char* abase = static_cast<const char*>(a.act) + (size_t)(up * KB2) * a.M * 64;
  unsigned ao[MT];
  act16_offsets<MT>(ao, a.M, i, g);
  f32x4 acc[2][MT];
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[n][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 wv[2][U][2], av[2][U][MT];
  stream_loop<U, 2>(k0, k1,
      [&](auto b, int u, int kb) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < 2; ++n) wv[b][u][n] = *reinterpret_cast<const bf16x8*>(wbase + (size_t)(2 * kb) * FRAG_BYTES + n * 256);
        const char* ap = abase + (size_t)kb * a.M * 64;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) av[b][u][mt] = *reinterpret_cast<const bf16x8*>(ap + ao[mt]);
      },
      [&](auto b, int u) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[n][mt] = mfma16(wv[b][u][n], av[b][u][mt], acc[n][mt]);
      });
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) red[w][n * MT + mt][lane] = acc[n][mt];
  __syncthreads();
  if (w >= 2 * MT) return;
  const int hn = w / MT, row = 16 * (w % MT) + i;
  f32x4 v[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    v[n] = red[n * KS][w][lane];
#pragma unroll
    for (int k = 1; k < KS; ++k) v[n] += red[n * KS + k][w][lane];
  }
  if (row >= a.M) return;
  bf16x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (__bf16)(v[0][e] * __builtin_amdgcn_rcpf(1.0f + __expf(-v[0][e])) * v[1][e]);
  *reinterpret_cast<bf16x4*>(act16_slot(static_cast<char*>(a.out), a.M, 2 * tile + hn, g, row)) = o;
}

// ranges for k_stream16: `tiles` 16-column tiles, KB2 contraction blocks of 32, mt 16-row tiles
int stream_splits16(int tiles, int KB2, int mt) {
  int s = (256 + tiles - 1) / tiles;
  int smax = KB2 / SW;
  if (s > smax) s = smax;
  if (s > 64) s = 64;
  if (s < 1) s = 1;
  const size_t part_floats = ((size_t)8 << 20) / 4;   // the partial-tile buffer of the workspace
  while (s > 1 && (size_t)tiles * s * mt * 256 > part_floats) --s;
  return s;
}
// 16-row tiles k_stream16 pads a batch to
int stream_tiles16(int64_t M) { return M <= 16 ? 1 : 2; }
// whether the two split phases of a forward of M rows run on 16-column tiles
bool stream_uses_tile16(int64_t M, int64_t d, int64_t ffn, int64_t r, int64_t rd) {
  // beyond 32 rows the activation frags, re-read for every 16-column weight tile, cost more than the smaller partials
  // save (the 32-column tiles with row-tile groups of their own measure faster there)
  return M <= 32 && d % 32 == 0 && ffn % 32 == 0 && 2 * r / 16 <= 2048 && rd / 16 <= 2048;
}

// The last product on 16-column tiles too: while the 32-column tiles would leave CUs without a workgroup (a phase
// streams its weights at the chip's rate only if every CU pulls: 128 of 256 CUs reach 3.6 of 7.1 TB/s).  Measured at
// the decode shape (128 -> 256 workgroups for 4 MB of Vd): the forward 0.9 us shorter at 1..16 rows, 0.55 us at 32.
bool stream_last_uses_tile16(bool tile16, int tiles32) { return tile16 && tiles32 < 256; }

// Row-tile groups of the two split phases (k_stream; `rt` row tiles in the batch, `tiles` 32-column tiles, KB
// contraction blocks).  With all row tiles in one workgroup the weights are fetched once, but the workgroup that adds
// the partial tiles reads ranges x rt of them through one CU's bounded fetch rate (mlp_small, 128 rows: 512 KiB
// in the down projection).  Groups with workgroups of their own need fewer ranges to fill the chip and spread that
// read-back; in exchange rtw workgroups (of one XCD) fetch the same weight frags, which occupies rtw times the
// requests in flight chip-wide while they stream from HBM.  Measured: at 128 rows phases with 2 and 4 MB of weights
// take 35-40 % less time with four groups, 8 MB 25 % less with four groups, 15 MB 10 % less with two (and no less with
// four when the weights come from HBM); at 64 rows two groups on these 32-column tiles beat the 16-column tiles of
// k_stream16 (whose workgroups re-read twice the activation bytes) by 2.3 us (D1, 8 MB) and 2.5 us (D4, 15 MB).
int stream_row_groups(int rt, int tiles, int KB, bool first) {
  const double weight_mb = (double)tiles * KB * FRAG_BYTES / 1.0e6;
  int rtw = rt;
  // the first phase (activation = the rows of X) takes more copies of a fetch than the down projection, whose
  // workgroups also stream the ffn-wide activation: cold, every row tile on its own still pays with 17 MB of [Ug|Uu]
  // (r = 1024, 128 rows: the forward 67.8 -> 65.4 us), two groups lose a little with 34 MB (r = 2048), and the down
  // projection loses with four groups at 15 MB and 29 MB
  const double lim = first && weight_mb <= 20.0 ? 1.0e9 : 30.0;
  while (rtw > 1 && (weight_mb * (rtw - 1) > lim || tiles * rtw > 2048)) rtw /= 2;
  return rtw;
}

// ... of the last product, whose contraction is not split: groups only while there are fewer workgroups than CUs
int stream_row_groups_whole(int rt, int tiles) {
  int rtw = 1;
  while (2 * rtw <= rt && 2 * rtw * tiles <= 256) rtw *= 2;
  return rtw;
}

int stream_splits(int tiles, int KB, int rt) {
  int s = (256 + tiles - 1) / tiles;      // aim at one workgroup per CU
  int smax = KB / SW;                     // at least one contraction block per wave
  if (s > smax) s = smax;
  if (s > 64) s = 64;
  if (s < 1) s = 1;
  const size_t part_floats = ((size_t)8 << 20) / 4;   // the partial-tile buffer of the workspace
  while (s > 1 && (size_t)tiles * s * rt * 1024 > part_floats) --s;
  return s;
}

// Contraction blocks per register buffer of stream_loop, for waves of kw blocks: as few groups of up to `most` as the
// range needs, all of about the same length, so that little is loaded for nothing.  Four at a time whatever the range
// made small layers slower than the single buffer before had been; factored layers replayed from a graph, single buffer
// / always four / this rule: 22 rows, d = 1536, r = 256, n = 4736 (8 layers) 65.8 / 76.2 / 64.9 us; 18 rows, d = 4224,
// r = 384, n = 14592 (8) 86.7 / 91.0 / 83.6 us; 30 rows, d = 4096, r = 1536, n = 24576 (2) 49.2 / 52.2 / 49.0 us.  (Skipping
// the loads beyond the range instead, by branches in the loop: 2 to 4 % slower at 64 rows and at d = 5120.)
// `most`: 8 costs the 16-row kernels 3 to 15 %.  k_stream of several row tiles: 2 (4 takes the registers: gated blocks
// of 65 .. 128 rows up to 1.6 % slower, single layers 1 to 2 % faster).  k_stream_gu: 4, with two row tiles 2 (4 there: 0 to
// 2 % slower at 33 .. 64 rows; 2 with four row tiles, where one workgroup fills the CU's LDS whatever its registers:
// 2 % slower at d = 2048, r = 256, 0.5 % at d = 4096).
static int stream_unroll(int kw, int most) {
  if (kw <= 1) return 1;
  const int groups = (kw + most - 1) / most;
  return (kw + groups - 1) / groups;
}

// Three workgroups share a CU if a wave takes at most 80 registers, four at 64: two buffers of two blocks, or one of
// four.  With the 96 of two buffers of four (two workgroups on a CU) the last product of 768 tiles
// ran in two rounds: 7 layers of 8 rows, d = 6784, r = 1024, n = 24576 141.9 us; one buffer of four 130.7, two of two 134.3
// (before the two-buffer loop 134.2); 12 rows, d = 5120, r = 640, n = 17920 (4 layers) 58.0 / 51.4 us with / without.  For a cut
// phase two buffers of two are better: 128 rows of a gated block, d = 2176, r = 2176 (544 workgroups in D1, 4 layers) 265.6
// against 273.0 us with one buffer, 268.4 with two of four.
// Those figures are from when up to 32 rows ran here too.  Now one row tile means one of several groups, at most 256
// workgroups, or up to 32 rows with r > 16384 or r_down > 32768, where one buffer is left.  Where two buffers load two blocks
// for nothing they are the better choice all the same: layers of d = 4096, n = 2048, one buffer / two, r = 1280 40 rows
// 15.0 / 14.8 us, r = 1792 40 / 128 rows 18.7 / 18.3, 22.4 / 22.0; n = 4096 level to 1 % (before, such ranges took one).
template <int PH, int RT>
static void launch_stream_rt(const StreamArgs& a, hipStream_t st) {
  const dim3 grid((a.tiles * a.S + 7) / 8 * 8 * a.rtw), block(SW * 64);
  const int kw = ((a.KB + a.S - 1) / a.S + SW - 1) / SW;
  if constexpr (RT == 1) {
    const bool many = grid.x > 512;
    const int u = stream_unroll(kw, PH != PH_D5 && many ? 2 : 4);
    if (u == 1) hipLaunchKernelGGL((k_stream<PH, 1, 1, 2>), grid, block, 0, st, a);
    else if (u == 2) hipLaunchKernelGGL((k_stream<PH, 1, 2, 2>), grid, block, 0, st, a);
    else if (PH == PH_D5 && many) hipLaunchKernelGGL((k_stream<PH, 1, 4, PH == PH_D5 ? 1 : 2>), grid, block, 0, st, a);
    else if (u == 3) hipLaunchKernelGGL((k_stream<PH, 1, 3, 2>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((k_stream<PH, 1, 4, 2>), grid, block, 0, st, a);
  } else {
    if (stream_unroll(kw, 2) == 1) hipLaunchKernelGGL((k_stream<PH, RT, 1, 2>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((k_stream<PH, RT, 2, 2>), grid, block, 0, st, a);
  }
}
template <int PH>
static void launch_stream(int rt, const StreamArgs& a, hipStream_t st) {   // rt: row tiles per workgroup
  if (rt == 1) launch_stream_rt<PH, 1>(a, st);
  else if (rt == 2) launch_stream_rt<PH, 2>(a, st);
  else launch_stream_rt<PH, 4>(a, st);
}

template <int RT>
static void launch_gu_rt(const StreamArgs& a, hipStream_t st) {
  const dim3 grid(a.tiles), block(SW * 64);
  const int u = stream_unroll((a.KB + SW / 2 - 1) / (SW / 2), 4);
  if (RT == 2 || u <= 2) hipLaunchKernelGGL((k_stream_gu<RT, 2>), grid, block, 0, st, a);
  else if (u == 3) hipLaunchKernelGGL((k_stream_gu<RT, RT == 2 ? 2 : 3>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((k_stream_gu<RT, RT == 2 ? 2 : 4>), grid, block, 0, st, a);
}
static void launch_gu(int rt, const StreamArgs& a, hipStream_t st) {
  if (rt == 1) launch_gu_rt<1>(a, st);
  else if (rt == 2) launch_gu_rt<2>(a, st);
  else launch_gu_rt<4>(a, st);
}

template <int PH, int MT>
static void launch_stream16_mt(const StreamArgs& a, hipStream_t st) {
  const dim3 grid(a.tiles * a.S), block(SW * 64);
  const int u = stream_unroll(((a.KB / 2 + a.S - 1) / a.S + SW - 1) / SW, 4);
  if (u == 1) hipLaunchKernelGGL((k_stream16<PH, MT, 1, 1, 2>), grid, block, 0, st, a);
  else if (u == 2) hipLaunchKernelGGL((k_stream16<PH, MT, 1, 2, 2>), grid, block, 0, st, a);
  else if (u == 3) hipLaunchKernelGGL((k_stream16<PH, MT, 1, 3, 2>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((k_stream16<PH, MT, 1, 4, 2>), grid, block, 0, st, a);
}
template <int PH>
static void launch_stream16(int mt, const StreamArgs& a, hipStream_t st) {
  if (mt == 1) launch_stream16_mt<PH, 1>(a, st);
  else launch_stream16_mt<PH, 2>(a, st);
}
// The last product on tiles of 32 columns: from 256 of them on, where all CUs have one and the wider tile halves the
// requests for the activation.
// Register buffers of two pairs of frags (four: 28 rows, r = 1024, n = 24576 (3 layers, d = 6784) 53.8 against 51.5 us).
// Layers of d = 4096, two buffers / one.  Two row tiles, beyond 512 tiles (two workgroups per CU): one (28 rows, n = 24576,
// r = 384 .. 1280 1.5 to 7 % faster, other n and r from 5 % faster to 1.7 % slower).  One row tile: two up to 768 tiles (2 rows,
// n = 24576, r = 1024 15.2 / 16.9 us, r = 1280 18.0 / 18.6, r = 384 10.1 / 10.3), one beyond, where a fourth workgroup shares a
// CU (n = 28672, -9 to 3 %).  Up to 512 tiles one for waves of an odd number kw of blocks, where two load a block for nothing, if
// some CU has two workgroups to cover each other's round trips; 2 rows: n = 9216, r = 640 (kw = 3) 10.1 / 9.6 us, r = 1152 (5)
// 13.0 / 12.2, r = 1664 (7) 16.1 / 14.8; n = 16384 level to 2 % faster with one; 28 rows 1 to 4 %.  With a workgroup per CU
// (n = 8192) one buffer is level to 5 % slower, and where kw is even (r = 1024, 1536, 2048; n = 12288 .. 16384, up to 16 rows)
// -3 to 5 %.
int stream_last_buffers(int tiles32, int KB2, int mt) {
  const int kw = (KB2 + SW - 1) / SW;
  if (kw <= 1 || tiles32 <= 256) return 2;
  return (tiles32 > 512 ? mt == 2 || tiles32 > 768 : kw % 2 == 1) ? 1 : 2;
}
template <int MT>
static void launch_last32_mt(const StreamArgs& a, hipStream_t st) {
  const dim3 grid(a.tiles), block(SW * 64);
  if (a.KB / 2 <= SW) hipLaunchKernelGGL((k_stream16<PH_D5, MT, 2, 1, 2>), grid, block, 0, st, a);   // a block per wave
  else if (stream_last_buffers(a.tiles, a.KB / 2, MT) == 1)
    hipLaunchKernelGGL((k_stream16<PH_D5, MT, 2, 2, 1>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((k_stream16<PH_D5, MT, 2, 2, 2>), grid, block, 0, st, a);
}
static void launch_last32(int mt, const StreamArgs& a, hipStream_t st) {
  if (mt == 1) launch_last32_mt<1>(a, st);
  else launch_last32_mt<2>(a, st);
}
template <int MT>
static void launch_gu16_mt(const StreamArgs& a, hipStream_t st) {
  const dim3 grid(a.tiles), block(SW * 64);
  constexpr int most = MT == 1 ? 4 : 2;
  const int u = stream_unroll((a.KB / 2 + SW / 2 - 1) / (SW / 2), most);
  if (u == 1) hipLaunchKernelGGL((k_stream_gu16<MT, 1>), grid, block, 0, st, a);
  else if (u == 2) hipLaunchKernelGGL((k_stream_gu16<MT, 2>), grid, block, 0, st, a);
  else if (u == 3) hipLaunchKernelGGL((k_stream_gu16<MT, most == 4 ? 3 : 2>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((k_stream_gu16<MT, most == 4 ? 4 : 2>), grid, block, 0, st, a);
}
static void launch_gu16(int mt, const StreamArgs& a, hipStream_t st) {
  if (mt == 1) launch_gu16_mt<1>(a, st);
  else launch_gu16_mt<2>(a, st);
}

// The per-forward buffers of the path: the rank-r strips T, the ffn-wide activation H of its (at most 128) rows, the
// down strip Td, the partial tiles of the two phases that split their contraction over workgroups, and their tickets.
struct StreamBufs {
  char* T;
  char* H;
  char* Td;
  float* part;
  int* cnt;
  bool clear;   // of tickets that an earlier caller may have left behind
};

static int stream_forward_on(const Ctx* c, const StreamBufs& b, const void* X, int64_t M, void* Y, hipStream_t st);

int bf16_stream_forward(const Ctx* c, const void* X, int64_t M, void* Y, hipStream_t st) {
  const Plan& p = c->plan;
  char* ws = c->ws;
  const StreamBufs b = {ws + p.off_T, ws + p.off_H, ws + p.off_Td, reinterpret_cast<float*>(ws + p.off_part),
                        reinterpret_cast<int*>(ws + p.off_cnt + CNT_ONE_KERNEL_BYTES), false};
  return stream_forward_on(c, b, X, M, Y, st);
}

// Whether the weight-streaming path takes a forward of M rows of this plan: up to 128 rows, and no more units (output
// tile x row-tile group) in either split phase than there are ticket lines (2048 per phase: ranks beyond 32768).
bool stream_supported(const Plan& p, int64_t M) {
  if (M < 1 || M > STREAM_MAX_M) return false;
  const int rt = M <= 32 ? 1 : M <= 64 ? 2 : 4;
  if (p.kind == SVDMLP_LINEAR) {
    if (M <= 32 && p.d % 32 == 0 && p.r / 16 <= 2048) return true;   // 16-column tiles
    const int t1 = (int)(p.r / 32);
    return t1 * stream_row_groups(rt, t1, (int)(p.d / 16), true) <= 2048;
  }
  if (stream_uses_tile16(M, p.d, p.ffn, p.r, p.rd)) return true;     // its own limits are part of that predicate
  const int t1 = (int)(2 * p.r / 32), t4 = (int)(p.rd / 32);
  return t1 * stream_row_groups(rt, t1, (int)(p.d / 16), true) <= 2048 &&
         t4 * stream_row_groups(rt, t4, (int)(p.ffn / 16), false) <= 2048;
}

static int stream_forward_on(const Ctx* c, const StreamBufs& b, const void* X, int64_t M, void* Y, hipStream_t st) {
  const Plan& p = c->plan;
  char* ws = c->ws;
  int* cnt = b.cnt;
  float* part = b.part;
  if (M > STREAM_MAX_M) return (int)hipErrorInvalidValue;
  const int rt = M <= 32 ? 1 : M <= 64 ? 2 : 4;   // 32-row tiles the batch is padded to
  const bool t16 = stream_uses_tile16(M, p.d, p.ffn, p.r, p.rd);
  const int mt16 = stream_tiles16(M);
  int e;
  static const char* const names[4] = {"k_stream_d1", "k_stream_d2", "k_stream_d4", "k_stream_d5"};
  const int ps = prof_open_forward(c, 4, names);
  const int fT = (int)(2 * p.r / 16), fH = (int)(p.ffn / 16), fTd = (int)(p.rd / 16);   // frags per 32-row tile

  StreamArgs a;
  // D1
  a = StreamArgs{ws + p.off_wU, nullptr, X, b.T, part, cnt, (int)M, (int)(p.d / 16), (int)(2 * p.r / 32), 1,
                 (int)p.d, (int)p.r, 0, 0, fT, 1};
  a.rtw = stream_row_groups(rt, a.tiles, a.KB, true);
  a.S = stream_splits(a.tiles * a.rtw, a.KB, rt / a.rtw);
  if (a.tiles * a.rtw > 2048) return (int)hipErrorInvalidValue;
  prof_mark(c, ps, 0, 0, st);
  if (t16) {
    a.tiles *= 2;
    a.S = stream_splits16(a.tiles, a.KB / 2, mt16);
    launch_stream16<PH_D1>(mt16, a, st);
  } else {
    launch_stream<PH_D1>(rt / a.rtw, a, st);
  }
  prof_mark(c, ps, 0, 1, st);
  if ((e = (int)hipGetLastError())) return e;
  // D2 (never split over workgroups: its contraction is only r long)
  a = StreamArgs{ws + p.off_wVg, ws + p.off_wVu, b.T, b.H, part, cnt, (int)M, (int)(p.r / 16),
                 (int)(p.ffn / 32), 1, 0, (int)p.r, 0, fT, fH, 1, b.clear ? cnt + TICKET_LINES * TICKET_STRIDE : nullptr};
  prof_mark(c, ps, 1, 0, st);
  if (t16) launch_gu16(mt16, a, st);
  else launch_gu(rt, a, st);
  prof_mark(c, ps, 1, 1, st);
  if ((e = (int)hipGetLastError())) return e;
  // D4
  a = StreamArgs{ws + p.off_wUd, nullptr, b.H, b.Td, part, cnt + TICKET_LINES * TICKET_STRIDE, (int)M, (int)(p.ffn / 16),
                 (int)(p.rd / 32), 1, 0, (int)p.r, 1, fH, fTd, 1};
  a.rtw = stream_row_groups(rt, a.tiles, a.KB, false);
  a.S = stream_splits(a.tiles * a.rtw, a.KB, rt / a.rtw);
  if (a.tiles * a.rtw > 2048) return (int)hipErrorInvalidValue;
  prof_mark(c, ps, 2, 0, st);
  if (t16) {
    a.tiles *= 2;
    a.S = stream_splits16(a.tiles, a.KB / 2, mt16);
    launch_stream16<PH_D4>(mt16, a, st);
  } else {
    launch_stream<PH_D4>(rt / a.rtw, a, st);
  }
  prof_mark(c, ps, 2, 1, st);
  if ((e = (int)hipGetLastError())) return e;
  // D5
  a = StreamArgs{ws + p.off_wVd, nullptr, b.Td, Y, part, cnt, (int)M, (int)(p.rd / 16), (int)(p.d / 32), 1,
                 (int)p.d, (int)p.r, 0, fTd, 0, 1, b.clear ? cnt : nullptr};
  a.rtw = stream_row_groups_whole(rt, a.tiles);
  prof_mark(c, ps, 3, 0, st);
  if (stream_last_uses_tile16(t16, a.tiles)) {
    a.tiles *= 2;
    launch_stream16<PH_D5>(mt16, a, st);
  } else if (t16) {
    launch_last32(mt16, a, st);
  } else {
    launch_stream<PH_D5>(rt / a.rtw, a, st);
  }
  prof_mark(c, ps, 3, 1, st);
  return (int)hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// The same forward with its per-forward buffers in a static device array instead of the caller's workspace, for
// callers that may not allocate device memory and hold no workspace of their own for intermediates (code under graph
// capture, tight serving loops).  Layout of the array: partial tiles (8 MiB, the capacity stream_splits assumes), the
// ticket lines of D1 and D4, then T, H and Td of the call, each 256-byte aligned.  Every GPU the library's code is
// loaded on holds its own copy of the array until the process ends; all calls on one GPU share it, so calls that
// overlap on one GPU race (as forwards on one context do).
// ------------------------------------------------------------------------------------------------
constexpr size_t SCRATCH_PART_BYTES = (size_t)8 << 20;
constexpr size_t SCRATCH_TICKET_BYTES = (size_t)2 * TICKET_LINES * TICKET_STRIDE * 4;
constexpr size_t SCRATCH_ACT_OFF = SCRATCH_PART_BYTES + SCRATCH_TICKET_BYTES;
static_assert(STATIC_SCRATCH_BYTES > SCRATCH_ACT_OFF, "room for the activations");
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

// Device address of this GPU's copy of the array.  The array's name is only a host-side handle; the address comes
// from the runtime, once per device, with that device current (svdmlp_create calls this, so the lookup, which may load
// the code object, never happens inside a forward).
constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mutex;
static char* g_scratch_ptr[MAX_DEVICES] = {};

int static_scratch_resolve(int device, char** out) {
  if (device < 0 || device >= MAX_DEVICES) return (int)hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[device]) {
    char* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    if (!ptr) return (int)hipErrorInvalidSymbol;
    g_scratch_ptr[device] = ptr;
  }
  *out = g_scratch_ptr[device];
  return 0;
}

size_t stream_static_scratch_need(const Plan& p, int64_t M) {
  const size_t rows = M <= 32 ? 32 : M <= 64 ? 64 : 128;
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  return SCRATCH_ACT_OFF + up(rows * 2 * p.r * 2) + up(rows * p.ffn * 2) + up(rows * p.rd * 2);
}

int bf16_stream_forward_static(const Ctx* c, const void* X, int64_t M, void* Y, hipStream_t st) {
  const Plan& p = c->plan;
  char* base = c->static_scratch;   // resolved at create for this context's device
  if (!base || stream_static_scratch_need(p, M) > STATIC_SCRATCH_BYTES) return (int)hipErrorInvalidValue;
  const size_t rows = M <= 32 ? 32 : M <= 64 ? 64 : 128;
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  StreamBufs b;
  b.part = reinterpret_cast<float*>(base);
  b.cnt = reinterpret_cast<int*>(base + SCRATCH_PART_BYTES);
  b.T = base + SCRATCH_ACT_OFF;
  b.H = b.T + up(rows * 2 * p.r * 2);
  b.Td = b.H + up(rows * p.ffn * 2);
  // The tickets are zero when the library is loaded and a forward leaves them at zero.  But the array is shared by every
  // caller on this GPU and outlives them, and forwards that overlapped (which they may not) can leave any count on a
  // ticket while they run.  A forward that is ordered after all of them finds D1's tickets at zero all the same: D5 of
  // every forward clears them after all arrivals of its own D1, so the last of those clears comes after all arrivals
  // of all of them.  D4's tickets are cleared by D2 of the forward that is about to use them.  Both clear in their own
  // launches (a launch for it cost 1 us of a 23 us forward; tickets that count from an epoch, which need no clearing,
  // 0.4 us of 20).  The other buffers are written before they are read.
  b.clear = true;
  return stream_forward_on(c, b, X, M, Y, st);
}

// Testing aid: `arrivals` on every ticket of one split phase (0: D1, 1: D4).
__global__ __launch_bounds__(256) void k_preset_tickets(int* cnt, int arrivals) {
  const int i = blockIdx.x * 256 + threadIdx.x;   // the launch has TICKET_LINES SW threads
  cnt[i / SW * TICKET_STRIDE + i % SW] = arrivals;
}

int static_scratch_preset_tickets(const Ctx* c, int phase, int arrivals, hipStream_t st) {
  if (!c->static_scratch) return (int)hipErrorInvalidValue;
  int* cnt = reinterpret_cast<int*>(c->static_scratch + SCRATCH_PART_BYTES) + phase * TICKET_LINES * TICKET_STRIDE;
  static_assert(TICKET_LINES * SW % 256 == 0, "whole workgroups");
  hipLaunchKernelGGL(k_preset_tickets, dim3(TICKET_LINES * SW / 256), dim3(256), 0, st, cnt, arrivals);
  return (int)hipGetLastError();
}

// Whether the single factored layer of M <= 128 rows streams: every workgroup of a phase re-reads the activation of
// its rows from L2, (r / 32) d + (n / 32) r elements per row over the two phases; beyond about 0.5 GB of that the
// MFMA-tiled kernels are faster (measured: d = 8192, r = 4096, n = 16384 at 96 / 128 rows 85 / 91 us against 79 us
// tiled, at 64 rows 57 against 78 us; every smaller layer tried streams 1.3 - 3x faster up to 128 rows).
bool linear_stream_pays(int64_t M, int64_t d, int64_t r, int64_t n) {
  const int64_t rows = M <= 32 ? 32 : M <= 64 ? 64 : 128;
  return M <= STREAM_MAX_M && (double)((r / 32) * d + (n / 32) * r) * (double)rows * 2.0 <= 512.0e6;
}

// Single factored layer O = (X U) V for up to 128 rows (paper Sec. 4.2.1 at decode sizes): the first and the last
// phase of the path above back to back.  T = X U is phase D1 with one strip of r columns, O = T V is phase D5 with
// the row length of O; U and V frags are the ones the tiled kernels of this kind read.
int bf16_linear_stream_forward(const Ctx* c, const void* X, int64_t M, void* Y, hipStream_t st) {
  const Plan& p = c->plan;
  char* ws = c->ws;
  int* cnt = reinterpret_cast<int*>(ws + p.off_cnt + CNT_ONE_KERNEL_BYTES);
  float* part = reinterpret_cast<float*>(ws + p.off_part);
  if (M > STREAM_MAX_M) return (int)hipErrorInvalidValue;
  const int rt = M <= 32 ? 1 : M <= 64 ? 2 : 4;
  const bool t16 = M <= 32 && p.d % 32 == 0 && p.r / 16 <= 2048;
  const int mt16 = stream_tiles16(M);
  static const char* const names[2] = {"k_stream_d1", "k_stream_d5"};
  const int ps = prof_open_forward(c, 2, names);
  const int fT = (int)(p.r / 16);   // frags of T per 32-row tile
  int e;
  StreamArgs a;
  a = StreamArgs{ws + p.off_wU, nullptr, X, ws + p.off_T, part, cnt, (int)M, (int)(p.d / 16), (int)(p.r / 32), 1,
                 (int)p.d, (int)p.r, 0, 0, fT, 1};
  a.rtw = stream_row_groups(rt, a.tiles, a.KB, true);
  a.S = stream_splits(a.tiles * a.rtw, a.KB, rt / a.rtw);
  if (a.tiles * a.rtw > 2048) return (int)hipErrorInvalidValue;
  prof_mark(c, ps, 0, 0, st);
  if (t16) {
    a.tiles *= 2;
    a.S = stream_splits16(a.tiles, a.KB / 2, mt16);
    launch_stream16<PH_D1>(mt16, a, st);
  } else {
    launch_stream<PH_D1>(rt / a.rtw, a, st);
  }
  prof_mark(c, ps, 0, 1, st);
  if ((e = (int)hipGetLastError())) return e;
  a = StreamArgs{ws + p.off_wVd, nullptr, ws + p.off_T, Y, part, cnt, (int)M, (int)(p.r / 16), (int)(p.ffn / 32), 1,
                 (int)p.ffn, (int)p.r, 0, fT, 0, 1};
  a.rtw = stream_row_groups_whole(rt, a.tiles);
  prof_mark(c, ps, 1, 0, st);
  if (stream_last_uses_tile16(t16, a.tiles)) {
    a.tiles *= 2;
    launch_stream16<PH_D5>(mt16, a, st);
  } else if (t16) {
    launch_last32(mt16, a, st);
  } else {
    launch_stream<PH_D5>(rt / a.rtw, a, st);
  }
  prof_mark(c, ps, 1, 1, st);
  return (int)hipGetLastError();
}

}  // namespace svdmlp
