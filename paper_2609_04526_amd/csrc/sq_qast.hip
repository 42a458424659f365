// One QAST low-rank scale step on gfx950 (paper Section 3, "Scale-QLoRA
// forward" and "QAST makes merge exact by construction"; stability recipe
// items (ii)-(iii)).
//
//   Delta_S = (alpha/r) B A            B bf16 [O, r], A bf16 [r, G]
//   eff'    = eff + Delta_S            rounded onto the grid by grid_update,
//                                      the same function the merge uses
//   dB = (alpha/r) (dS * m) A^T        m = 0 where the NVFP4 ceiling clamp bound
//   dA = (alpha/r) B^T (dS * m)
//
// The MoE path stacks E experts (rows e*O .. e*O + O - 1 of every [rows, G]
// or [rows, r] plane; A as [E, r, G]) and runs every expert's step in the
// same launches.
//
// All three contractions run on the fp32 matrix cores, which do twice the
// fused multiply-adds per cycle of the vector units and take their operands
// from one register per lane instead of LDS reads per term.  Their terms are
// added in increasing k, each with one rounding, so Delta_S equals a chain of
// r fused multiply-adds (each product of two bf16 values is exact in fp32) and
// the scale bytes are fixed bit for bit.  The factor gradients are summed in a
// fixed order that depends on the shape alone: deterministic, and the same
// for an expert alone and in a batch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sq_device.h"
#include "sq_grid.h"
#include "sq_launch.h"

namespace sq {

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------------ scales
// Loads below are issued without a branch, from an address moved inside the
// plane where there is nothing to load, and their values dropped afterwards
// (a branch per load made each wait for the one before).  blockIdx.y is the
// expert: rows e O .. e O + O - 1 of base, B, out and mask belong to it, its A
// is A + e r G and its ws2 ws2.v[e].  With vec (G % 4 == 0 and 4-byte aligned
// byte planes) the MFMA's rows are scale blocks g and its columns output rows o,
// so that a lane ends with four consecutive bytes of one row, one word each
// way.  Else its operands change places: a lane ends with one byte of each of
// four rows, and 16 lanes with 16 consecutive bytes of a row (14336 x 129 at
// rank 58, NVFP4: 27.0 -> 18.0 us, 128 experts of 1536 x 65 at rank 2 54.2 -> 36.2,
// against vector multiply-adds fed from LDS).

// The sums s[0..3] of a lane to scales: blocks g .. g + 3 of row o (vec), or
// block g of rows o .. o + 3.  The base bytes come from base4 of the same place.
template <int FMT>
__device__ __forceinline__ void scale4(const float (&s)[4], const uint32_t (&in)[4], float c, const Ws2Div& wd,
                                       uint8_t* out, uint8_t* mask, size_t rows0, int o, int g, int O, int G,
                                       int vec) {
  uint32_t n[4], m[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    bool clamped;
    n[j] = grid_update<FMT>(in[j], __fmul_rn(s[j], c), wd, clamped);
    m[j] = clamped ? 0u : 1u;
  }
  if (o >= O || g >= G) return;
  const size_t at = (rows0 + o) * G + g;
  if (vec) {
    *reinterpret_cast<uint32_t*>(out + at) = n[0] | (n[1] << 8) | (n[2] << 16) | (n[3] << 24);
    if (mask) *reinterpret_cast<uint32_t*>(mask + at) = m[0] | (m[1] << 8) | (m[2] << 16) | (m[3] << 24);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (o + j >= O) break;
      out[at + (size_t)j * G] = (uint8_t)n[j];
      if (mask) mask[at + (size_t)j * G] = (uint8_t)m[j];
    }
  }
}
__device__ __forceinline__ void base4(uint32_t (&in)[4], const uint8_t* base, size_t rows0, int o, int g, int O, int G,
                                      int vec) {
  const size_t inside = rows0 * G, at = (rows0 + o) * G + g;
  const bool ok = o < O && g < G;
  if (vec) {
    const uint32_t w = *reinterpret_cast<const uint32_t*>(base + (ok ? at : inside));
#pragma unroll
    for (int j = 0; j < 4; ++j) in[j] = (w >> (8 * j)) & 0xFFu;
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) in[j] = base[ok && o + j < O ? at + (size_t)j * G : inside];
  }
}

// n consecutive bf16 values (a workgroup's rows of a factor are one run of
// memory) to LDS, w of them per load (w = 8 or 2: their place and n allow it),
// and the RMAX x COLS tile of A at block g0 (zeros past r and G).
__device__ __forceinline__ void stage_run(uint16_t* dst, const uint16_t* __restrict__ src, int n, int w) {
  auto copy = [&](auto Z) {
    typedef decltype(Z) V;
    const V* s = reinterpret_cast<const V*>(src);
    const int m = n / (int)(sizeof(V) / 2);
    for (int i = threadIdx.x; i < m; i += 1024) {
      V v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = s[i + 256 * u < m ? i + 256 * u : 0];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i + 256 * u < m) reinterpret_cast<V*>(dst)[i + 256 * u] = v[u];
    }
  };
  if (w == 8) copy(uint4{});
  else if (w == 2) copy(uint32_t{});
  else copy(uint16_t{});
}
template <int RMAX, int COLS>
struct ATile {
  static constexpr int kPer = (RMAX * COLS + 255) / 256;
  uint16_t v[kPer];
  __device__ __forceinline__ void load(const uint16_t* __restrict__ ap, int g0, int G, int r) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = threadIdx.x + 256 * u, k = i / COLS, g = g0 + i % COLS;
      v[u] = ap[k < r && g < G ? (size_t)k * G + g : 0];
    }
  }
  __device__ __forceinline__ void store(uint16_t (*lds)[COLS], int g0, int G, int r) const {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int i = threadIdx.x + 256 * u, k = i / COLS, g = g0 + i % COLS;
      if (RMAX * COLS < 256 && k >= RMAX) break;
      lds[k][i % COLS] = k < r && g < G ? v[u] : (uint16_t)0;
    }
  }
};

// One linear: latency is what bounds it, so a wave takes a single 16 x 16
// block and four ranks per MFMA (v_mfma_f32_16x16x4 adds its four terms in
// increasing k, each with its own rounding: every byte the tests compare
// depends on it).  GB of a workgroup's four waves lie along g, the rest along
// o.  STAGED: a workgroup's rows of B and columns of A come through LDS in wide
// loads, since at high ranks a load per rank and lane costs more than the
// products (4096 x 256 at rank 64 11.5 us so, 8.8 through LDS; scales_staged has
// the line).  4096 x 256 scales at rank 58, NVFP4: 10.1 us on vector multiply-adds
// fed from LDS, 7.3 here; 7384 x 77 5.7 -> 4.9 at rank 11.
template <int FMT, int RMAX, int GB, bool STAGED>
__global__ __launch_bounds__(256, 4) void qast_scales_kernel(const uint8_t* __restrict__ base,
                                                          const uint16_t* __restrict__ B,
                                                          const uint16_t* __restrict__ A, int O, int G, int r,
                                                          float c, Ws2Table ws2, uint8_t* out, uint8_t* mask,
                                                          int vec, int w) {
  constexpr int COLS = 16 * GB, ROWS = 64 / GB, N = RMAX / 4;
  __shared__ uint16_t at_lds[STAGED ? RMAX : 1][COLS];
  __shared__ __attribute__((aligned(16))) uint16_t b_lds[STAGED ? ROWS * RMAX : 8];
  const int e = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
  const int gtiles = (G + COLS - 1) / COLS;
  const int gw = (int)blockIdx.x % gtiles * COLS, ow = (int)blockIdx.x / gtiles * ROWS;   // of the workgroup
  const int g0 = gw + wave % GB * 16, ro = wave / GB * 16, o0 = ow + ro;
  const size_t rows0 = (size_t)e * O;
  const bool g_ok = g0 + n < G, o_ok = o0 + n < O;
  const int g = vec ? g0 + 4 * q : g0 + n, o = vec ? o0 + n : o0 + 4 * q;
  uint32_t in[4];
  uint16_t ar[N], br[N];
  ATile<RMAX, COLS> at;
  if constexpr (STAGED) {
    at.load(A + (size_t)e * r * G, gw, G, r);
    base4(in, base, rows0, o, g, O, G, vec);            // before the wait for B, whose loads go straight on to LDS
    stage_run(b_lds, B + (rows0 + ow) * r, min(ROWS, O - ow) * r, w);
  } else {
    const uint16_t* ap = A + (size_t)e * r * G + (g_ok ? g0 + n : 0);
    const uint16_t* bp = B + (rows0 + (o_ok ? o0 + n : 0)) * r;
#pragma unroll
    for (int st = 0; st < N; ++st) {
      const int k = 4 * st + q, kc = k < r ? k : 0;
      ar[st] = ap[(size_t)kc * G];
      br[st] = bp[kc];
    }
  }
  if constexpr (!STAGED) base4(in, base, rows0, o, g, O, G, vec);
  if constexpr (STAGED) at.store(at_lds, gw, G, r);
  const Ws2Div wd = make_ws2_div(ws2.v[e]);
  if constexpr (STAGED) {
    __syncthreads();
    const uint16_t* bl = b_lds + (o_ok ? (ro + n) * r : 0);
#pragma unroll
    for (int st = 0; st < N; ++st) {
      const int k = 4 * st + q;
      ar[st] = at_lds[k][wave % GB * 16 + n];
      br[st] = bl[k < r ? k : 0];
    }
  }
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int st = 0; st < N; ++st) {
    const bool in_r = 4 * st + q < r;                    // ranks past r add exact zeros
    const float av = g_ok && in_r ? bf16_bits_to_f32(ar[st]) : 0.0f;
    const float bv = o_ok && in_r ? bf16_bits_to_f32(br[st]) : 0.0f;
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(vec ? av : bv, vec ? bv : av, acc, 0, 0, 0);
  }
  const float sum[4] = {acc[0], acc[1], acc[2], acc[3]};
  scale4<FMT>(sum, in, c, wd, out, mask, rows0, o, g, O, G, vec);
}

// Many scales (stacked experts, the widest linears): the address unit bounds
// it, so a wave takes four 16 x 16 blocks with one-deep MFMAs
// (v_mfma_f32_16x16x1: a register of A and one of B per rank serve all four),
// GB of them along g; the workgroup's waves lie below one another and share
// the A columns, of which each loads a quarter of the ranks into LDS; a row
// of B comes W ranks per load or, at odd ranks, through LDS, since the rows of a
// workgroup are one run of memory (128 experts of 768 x 128 at rank 47 76 us a rank
// per load, 41 so).  128 experts of 768 x 128 scales at rank 58 (NVFP4): 85 us on
// vector multiply-adds fed from LDS, 44 here, at rank 64 86 -> 35; at rank 5, where
// the bytes bound it, 21.8 -> 22.1.  VEC is a parameter: with both orders of the
// operands in one kernel the compiler spilled (128 experts of 2048 x 24 at rank 58
// 77 us instead of 29).
template <int FMT, int RMAX, int GB, int W, bool VEC>
__global__ __launch_bounds__(256, 4) void qast_scales_wide_kernel(const uint8_t* __restrict__ base,
                                                               const uint16_t* __restrict__ B,
                                                               const uint16_t* __restrict__ A, int O, int G, int r,
                                                               float c, Ws2Table ws2, uint8_t* out, uint8_t* mask,
                                                               int w) {
  constexpr int OB = 4 / GB, COLS = 16 * GB, ROWS = 64 * OB;
  __shared__ uint16_t at_lds[RMAX][COLS];
  __shared__ __attribute__((aligned(16))) uint16_t b_lds[W == 1 ? ROWS * RMAX : 8];
  const int e = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
  const int gtiles = (G + COLS - 1) / COLS;
  const int g0 = ((int)blockIdx.x % gtiles) * COLS;
  const int ow = ((int)blockIdx.x / gtiles) * ROWS, ro = wave * 16 * OB, o0 = ow + ro;
  const size_t rows0 = (size_t)e * O;
  ATile<RMAX, COLS> at;
  at.load(A + (size_t)e * r * G, g0, G, r);
  const int rl = 16 * (q / GB) + n;                     // this lane's operand row
  const bool o_ok = o0 + rl < O;
  uint32_t br[W > 1 ? RMAX / 2 : 1];                    // pairs of ranks
  if constexpr (W > 1) {
    const uint16_t* bp = B + (rows0 + (o_ok ? o0 + rl : 0)) * r;
#pragma unroll
    for (int k = 0; k < RMAX; k += W) {
      const int kc = k < r ? k : 0;                     // r is a multiple of W
      if constexpr (W == 8) {
        const uint4 v = *reinterpret_cast<const uint4*>(bp + kc);
        br[k / 2] = v.x; br[k / 2 + 1] = v.y; br[k / 2 + 2] = v.z; br[k / 2 + 3] = v.w;
      } else {
        br[k / 2] = *reinterpret_cast<const uint32_t*>(bp + kc);
      }
    }
  }
  // the result: block b, register 4 b + j is MFMA row 4 q + j, column n.  With VEC
  // the MFMA's row 4 q + j of block b is scale block g0 + 4 GB q + 4 (b % GB) + j, so
  // that a lane's GB words of a row lie side by side; else rows and columns are
  // output rows and scale blocks in their order.
  auto row = [&](int b) { return o0 + 16 * (b / GB) + (VEC ? n : 4 * q); };
  auto blk = [&](int b) { return g0 + (VEC ? 4 * GB * q + 4 * (b % GB) : 16 * (b % GB) + n); };
  const int acol = VEC ? 4 * GB * (n >> 2) + 4 * (q % GB) + (n & 3) : 16 * (q % GB) + n;
  uint32_t in[4][4];
#pragma unroll
  for (int b = 0; b < 4; ++b) base4(in[b], base, rows0, row(b), blk(b), O, G, VEC);
  if constexpr (W == 1) stage_run(b_lds, B + (rows0 + ow) * r, min(ROWS, O - ow) * r, w);
  at.store(at_lds, g0, G, r);
  __syncthreads();
  const uint16_t* bl = b_lds + (W == 1 && o_ok ? (ro + rl) * r : 0);
  f32x16 acc;
#pragma unroll
  for (int j = 0; j < 16; ++j) acc[j] = 0.0f;
#pragma unroll
  for (int k = 0; k < RMAX; ++k) {
    uint32_t bw;
    if constexpr (W == 1) bw = (uint32_t)bl[k < r ? k : 0] << 16;
    else bw = k & 1 ? br[k / 2] & 0xFFFF0000u : br[k / 2] << 16;
    const float av = bf16_bits_to_f32(at_lds[k][acol]);
    const float bv = o_ok && k < r ? __uint_as_float(bw) : 0.0f;
    acc = __builtin_amdgcn_mfma_f32_16x16x1f32(VEC ? av : bv, VEC ? bv : av, acc, 0, 0, 0);
  }
  const Ws2Div wd = make_ws2_div(ws2.v[e]);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const float sum[4] = {acc[4 * b], acc[4 * b + 1], acc[4 * b + 2], acc[4 * b + 3]};
    scale4<FMT>(sum, in[b], c, wd, out, mask, rows0, row(b), blk(b), O, G, VEC);
  }
}

// ------------------------------------------------------------------ dB, dA
// v = dS * m.  Both products run in one launch (workgroups below ndb take dB
// rows, the rest dA chunks; they are independent and short), every operand
// loaded straight into MFMA registers: lane (n, q) of v_mfma_f32_16x16x4
// holds row n of A, column n of B and the term q of the four.
//
// dB[o, k] = c sum_g v[o, g] A[k, g]: a workgroup takes 16 rows and all RT * 16
// ranks; wave w takes the 16-block steps w, w + 4, ... of g, in which MFMA j
// adds the terms g = 4 q + j (a lane's four consecutive blocks: one 16-byte
// load of dS, one word of the mask, 8 bytes of A where vec).  The waves'
// sums meet in LDS in wave order.
//
// part[chunk][k][g] = sum over a chunk of 64 rows of B[o, k] v[o, g]: a
// workgroup takes 16 U blocks and all ranks, its waves 16 rows each, four per
// MFMA in increasing order; the waves' sums again meet in LDS in a fixed
// order.  Column n of tile u is block U n + u, so that a lane's blocks are one
// load of dS (RUNS: block 16 u + n, see kDaRunsGrid), and row n of tile t is rank
// RT n + t.  U = 4, but 2 for ranks over
// 32: with 16 accumulator tiles a wave, too few waves fit a SIMD (128 experts
// of 768 x 128 at rank 54: 113 us, 69 with 8).  Chunks are added in order by
// qast_da_reduce_kernel.
// 4096 x 256 scales at rank 58: vector multiply-adds fed from LDS tiles took
// 30.0 us, this 11.2; the reduction of 128 partial planes of 32 rows (a wave
// per output, lanes striding over the planes) 12.3, of 64 in rows 3.9.
// The launch bounds of the MFMA kernels here ask for four waves per SIMD: left
// free, the compiler kept the accumulators in accumulation registers and
// moved every operand through them (128 experts of 2048 x 24 at rank 32: the
// gradients 45 -> 36 us).
constexpr int kDaRows = 64;         // rows per dA chunk
// Workgroups from which on dA of narrow dS rows (no vec) takes columns 16 u + n of
// the block tile instead of U n + u, one run of dS per load (128 experts of 1536 x
// 65 at rank 5 79 -> 67 us, 16 of 7384 x 77 52 -> 47; below, a lane's own
// neighbours serve better: 1536 x 65 8.1 against 9.1, 16 experts of 2048 x 130 at
// rank 32 37 against 40).
constexpr int64_t kDaRunsGrid = 4096;
template <int RT>
__host__ __device__ constexpr int da_u() { return RT == 4 ? 2 : 4; }

// v at blocks g .. g + U - 1 of row o; zeros outside the plane (loaded from
// inside it without a branch, then dropped).  vec: whole words (G % 4 == 0, dS
// 16-byte and the mask 4-byte aligned).
template <int U>
__device__ __forceinline__ void load_v(float (&v)[U], const float* __restrict__ dS, const uint8_t* __restrict__ mask,
                                       int O, int G, int o, int g, int vec) {
  const size_t row = o < O ? (size_t)o * G : 0;
  if (U > 1 && vec) {
    const size_t at_ = row + (g < G ? g : 0);
    if constexpr (U == 4) {
      const f32x4 w = *reinterpret_cast<const f32x4*>(dS + at_);
#pragma unroll
      for (int j = 0; j < U; ++j) v[j] = w[j];
    } else if constexpr (U == 2) {
      const f32x2 w = *reinterpret_cast<const f32x2*>(dS + at_);
      v[0] = w[0];
      v[1] = w[1];
    }
    if (mask) {
      const uint32_t m = U == 4 ? *reinterpret_cast<const uint32_t*>(mask + at_)
                                : (uint32_t)*reinterpret_cast<const uint16_t*>(mask + at_);
#pragma unroll
      for (int j = 0; j < U; ++j) v[j] *= (float)((m >> (8 * j)) & 0xFFu);
    }
  } else {
#pragma unroll
    for (int j = 0; j < U; ++j) v[j] = dS[row + (g + j < G ? g + j : 0)];
    if (mask) {
#pragma unroll
      for (int j = 0; j < U; ++j) v[j] *= (float)mask[row + (g + j < G ? g + j : 0)];
    }
  }
#pragma unroll
  for (int j = 0; j < U; ++j) v[j] = o < O && g + j < G ? v[j] : 0.0f;
}

template <int RT>
__device__ __forceinline__ void db_tile(int bx, int e, float* lds, const float* __restrict__ dS,
                                        const uint8_t* __restrict__ mask, const uint16_t* __restrict__ A, int O,
                                        int G, int r, float c, float* __restrict__ dB, int vec) {
  constexpr int S = 16 * RT + 1;                        // LDS row of one output row's ranks
  dS += (size_t)e * O * G;
  if (mask) mask += (size_t)e * O * G;
  A += (size_t)e * r * G;
  dB += (size_t)e * O * r;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
  // few steps (G <= 64): every wave its own 16 rows and all steps
  const bool split = G > 64;
  const int o0 = split ? bx * 16 : bx * 64 + 16 * wave, o = o0 + n;
  f32x4 acc[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int steps = (G + 15) / 16;
#pragma unroll 2
  for (int st = split ? wave : 0; st < steps; st += split ? 4 : 1) {
    const int g = 16 * st + 4 * q;
    float v[4];
    load_v<4>(v, dS, mask, O, G, o, g, vec);
    float a[RT][4];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int k = 16 * t + n;
      const uint16_t* ap = A + (size_t)(k < r ? k : 0) * G;
      if (vec) {
        const u32x2 w = *reinterpret_cast<const u32x2*>(ap + (g < G ? g : 0));
        a[t][0] = __uint_as_float(w[0] << 16);
        a[t][1] = __uint_as_float(w[0] & 0xFFFF0000u);
        a[t][2] = __uint_as_float(w[1] << 16);
        a[t][3] = __uint_as_float(w[1] & 0xFFFF0000u);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) a[t][j] = bf16_bits_to_f32(ap[g + j < G ? g + j : 0]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) a[t][j] = k < r && g + j < G ? a[t][j] : 0.0f;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int t = 0; t < RT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][j], v[j], acc[t], 0, 0, 0);
  }
  // register e of tile t: rank 16 t + 4 q + e of row n
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int x = 0; x < 4; ++x) lds[(wave * 16 + n) * S + 16 * t + 4 * q + x] = acc[t][x];
  __syncthreads();
  const int first = split ? bx * 16 : bx * 64, rows = min(split ? 16 : 64, O - first);
  for (int i = threadIdx.x; i < rows * r; i += 256) {
    const int ro = i / r, k = i - ro * r;
    float s = lds[ro * S + k];
    if (split) {
#pragma unroll
      for (int w = 1; w < 4; ++w) s += lds[(w * 16 + ro) * S + k];
    }
    dB[(size_t)first * r + i] = __fmul_rn(s, c);
  }
}

template <int RT, bool RUNS>
__device__ __forceinline__ void da_tile(int bx, int e, float* lds, const float* __restrict__ dS,
                                        const uint8_t* __restrict__ mask, const uint16_t* __restrict__ B, int O,
                                        int G, int r, float* __restrict__ part, int vec, int bvec) {
  constexpr int U = da_u<RT>(), COLS = 16 * U, S = COLS + 4;      // S: LDS row of one rank's blocks
  const int chunks = (O + kDaRows - 1) / kDaRows;
  dS += (size_t)e * O * G;
  if (mask) mask += (size_t)e * O * G;
  B += (size_t)e * O * r;
  part += (size_t)e * chunks * r * G;
  const int gtiles = (G + COLS - 1) / COLS;
  const int chunk = bx / gtiles, g0 = (bx % gtiles) * COLS;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, q = lane >> 4;
  const int o0 = chunk * kDaRows + 16 * wave;
  f32x4 acc[RT][U];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int u = 0; u < U; ++u) acc[t][u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  float v[4][U], b[4][RT];
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    const int o = o0 + 4 * st + q, k0 = RT * n;
    if constexpr (!RUNS) {
      load_v<U>(v[st], dS, mask, O, G, o, g0 + U * n, vec);
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) load_v<1>(*reinterpret_cast<float (*)[1]>(&v[st][u]), dS, mask, O, G, o, g0 + 16 * u + n, 0);
    }
    const uint16_t* bp = B + (o < O ? (size_t)o * r : 0);
    if (RT > 1 && bvec) {                               // r even, B 4-byte aligned: pairs of ranks
#pragma unroll
      for (int t = 0; t + 1 < RT; t += 2) {
        const uint32_t w = *reinterpret_cast<const uint32_t*>(bp + (k0 + t < r ? k0 + t : 0));
        b[st][t] = __uint_as_float(w << 16);
        b[st][t + 1] = __uint_as_float(w & 0xFFFF0000u);
      }
    } else {
#pragma unroll
      for (int t = 0; t < RT; ++t) b[st][t] = bf16_bits_to_f32(bp[k0 + t < r ? k0 + t : 0]);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) b[st][t] = o < O && k0 + t < r ? b[st][t] : 0.0f;
  }
#pragma unroll
  for (int st = 0; st < 4; ++st)
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int u = 0; u < U; ++u)
        acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[st][t], v[st][u], acc[t][u], 0, 0, 0);
  // register x of tile (t, u): rank RT (4 q + x) + t, column U n + u of LDS.  Waves 2
  // and 3 park their sums, waves 0 and 1 add theirs (half the LDS of four
  // planes, so twice the workgroups per CU), then the two planes are added.
  auto at = [&](int w, int t, int x, int u) -> float& {
    return lds[(w * 16 * RT + RT * (4 * q + x) + t) * S + U * n + u];
  };
  if (wave >= 2) {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int u = 0; u < U; ++u) at(wave - 2, t, x, u) = acc[t][u][x];
  }
  __syncthreads();
  if (wave < 2) {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int u = 0; u < U; ++u) at(wave, t, x, u) = acc[t][u][x] + at(wave, t, x, u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < r * COLS; i += 256) {
    const int k = i / COLS, gi = i % COLS;
    const int at_ = k * S + (RUNS ? U * (gi % 16) + gi / 16 : gi);
    if (g0 + gi < G) part[((size_t)chunk * r + k) * G + g0 + gi] = lds[at_] + lds[16 * RT * S + at_];
  }
}

template <int RT, bool RUNS>
__global__ __launch_bounds__(256, 4) void qast_grads_kernel(const float* __restrict__ dS,
                                                         const uint8_t* __restrict__ mask,
                                                         const uint16_t* __restrict__ A,
                                                         const uint16_t* __restrict__ B, int O, int G, int r,
                                                         float c, float* __restrict__ dB, float* __restrict__ part,
                                                         int ndb, int vec, int bvec) {
  constexpr int kDb = 4 * 16 * (16 * RT + 1), kDa = 2 * 16 * RT * (16 * da_u<RT>() + 4);
  __shared__ __attribute__((aligned(16))) float lds[kDb > kDa ? kDb : kDa];
  const int bx = (int)blockIdx.x, e = (int)blockIdx.y;
  if (bx < ndb)
    db_tile<RT>(bx, e, lds, dS, mask, A, O, G, r, c, dB, vec);
  else
    da_tile<RT, RUNS>(bx - ndb, e, lds, dS, mask, B, O, G, r, part, vec, bvec);
}

// dA[i] = c sum over the chunk partials in order.  64 consecutive outputs per
// workgroup; its four waves take every fourth group of 8 chunks (eight loads in
// flight each), and their sums are added in wave order.
__global__ __launch_bounds__(256) void qast_da_reduce_kernel(const float* __restrict__ part, int chunks, int r,
                                                             int G, int E, float c, float* __restrict__ dA) {
  __shared__ float sum[4][64];
  const int64_t n = (int64_t)r * G;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  float s = 0.0f;
  if (i < (int64_t)E * n) {
    const int64_t e = i / n, ie = i - e * n;
    const float* pe = part + (size_t)e * chunks * n + ie;
    for (int c0 = 8 * wave; c0 < chunks; c0 += 32) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = c0 + u < chunks ? pe[(size_t)(c0 + u) * n] : 0.0f;
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
  }
  sum[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && i < (int64_t)E * n)
    dA[i] = __fmul_rn(((sum[0][lane] + sum[1][lane]) + sum[2][lane]) + sum[3][lane], c);
}

// ------------------------------------------------------------------ launch
// Whether a launch of so many 16 x 16 blocks takes the wide kernel, by the width of
// the loads of B's rows.  Eight ranks: 4096 blocks (4096 x 256, rank 32) 6.0 us
// either way, 6144 (16 experts of 1536 x 64, rank 32) 7.2 there and 7.5 on the
// narrow kernel, 7168 7.2 and 7.8.  Two: 9216 (48 experts of 768 x 64, rank 58)
// 15.0 and 13.2, 12,288 (64 experts) 15.3 and 16.3.  One: 12,288 at rank 31 10.8 and
// 13.4, but at rank 5 8.4 and 7.3 (24,576 13.0 and 12.7, at 128 experts of 768 x 128
// 22.1 and 23.0); without words of bytes never (128 experts of 1536 x 65 at rank
// 31 61.5 and 47.5).
static bool scales_wide(int64_t blocks, int r, int w, int vec) {
  if (w == 8) return blocks >= 6144;
  if (w == 2) return blocks >= 12288;
  return vec && blocks >= (r > 8 ? 12288 : 24576);
}

// Whether the narrow kernel's factors come through LDS: in 16-byte loads from rank
// 32 on (4096 x 64 at rank 48 5.2 us a rank per load, 4.9 so, at rank 24 3.8 and
// 4.0), and where workgroups share the CUs from rank 16 on (4096 x 256 at rank 16
// 5.7 and 5.2, at rank 8 4.2 and 4.8) or, at odd ranks, in the 64-rank kernel
// (rank 63 8.5 and 7.6, rank 31 6.3 and 6.2, rank 11 4.6 and 5.2).
static bool scales_staged(int r, int w, int64_t grid) {
  if (grid <= 512) return w == 8 && r >= 32;
  return w > 1 ? r >= 16 : r > 32;
}

template <int F, int R, int GB>
static void scales_go(bool wide, int w, int64_t gtiles, int m, hipStream_t s, const uint8_t* bp, const uint16_t* Bp,
                      const uint16_t* Ap, int O, int G, int r, float c, const Ws2Table& t, uint8_t* op, uint8_t* mp,
                      int vec) {
  const int rows = (wide ? 4 : 1) * 16 * (4 / GB);                   // of a workgroup
  const dim3 grid((unsigned)(((O + rows - 1) / rows) * gtiles), (unsigned)m);
  const auto go = [&](auto k, auto... last) {
    hipLaunchKernelGGL(k, grid, dim3(256), 0, s, bp, Bp, Ap, O, G, r, c, t, op, mp, last...);
  };
  if (wide && vec) {
    if (w == 8) go(qast_scales_wide_kernel<F, R, GB, 8, true>, w);
    else if (w == 2) go(qast_scales_wide_kernel<F, R, GB, 2, true>, w);
    else go(qast_scales_wide_kernel<F, R, GB, 1, true>, w);
  } else if (wide) {
    if (w == 8) go(qast_scales_wide_kernel<F, R, GB, 8, false>, w);
    else go(qast_scales_wide_kernel<F, R, GB, 2, false>, w);
  } else if (R > 8 && scales_staged(r, w, (int64_t)grid.x * m)) {
    go(qast_scales_kernel<F, R, GB, (R > 8)>, vec, w);
  } else {
    go(qast_scales_kernel<F, R, GB, false>, vec, w);
  }
}
template <int F, int R>
static void scales_gb(bool wide, int gb, int w, int m, hipStream_t s, const uint8_t* bp, const uint16_t* Bp,
                      const uint16_t* Ap, int O, int G, int r, float c, const Ws2Table& t, uint8_t* op, uint8_t* mp,
                      int vec) {
  const int64_t gtiles = (G + 16 * gb - 1) / (16 * gb);
  if (gb == 4) scales_go<F, R, 4>(wide, w, gtiles, m, s, bp, Bp, Ap, O, G, r, c, t, op, mp, vec);
  else if (gb == 2) scales_go<F, R, 2>(wide, w, gtiles, m, s, bp, Bp, Ap, O, G, r, c, t, op, mp, vec);
  else scales_go<F, R, 1>(wide, w, gtiles, m, s, bp, Bp, Ap, O, G, r, c, t, op, mp, vec);
}
int qast_scales_launch(int fmt, int E, int O, int G, int r, const uint8_t* base, const void* B, const void* A,
                       float c, const float* ws2, uint8_t* out, uint8_t* mask, hipStream_t s) {
  const uint16_t* b = static_cast<const uint16_t*>(B);
  const uint16_t* a = static_cast<const uint16_t*>(A);
  // the widest wave tile along g that pads no more 16-block columns than a narrower one
  const int cols = (G + 15) / 16;
  const auto padded = [cols](int b) { return (cols + b - 1) / b * b; };
  const int gb = padded(4) == cols || padded(4) == padded(2) ? 4 : padded(2) == cols || padded(2) == padded(1) ? 2 : 1;
  const auto al = [](const void* q, uintptr_t n) { return (reinterpret_cast<uintptr_t>(q) & (n - 1)) == 0; };
  const int w = r % 8 == 0 && al(b, 16) ? 8 : r % 2 == 0 && al(b, 4) ? 2 : 1;
  for (int e0 = 0; e0 < E; e0 += kWs2TableMax) {          // per-expert ws2 travels by value
    const int m = E - e0 < kWs2TableMax ? E - e0 : kWs2TableMax;
    Ws2Table t;
    for (int e = 0; e < m; ++e) t.v[e] = fmt == kNV ? ws2[e0 + e] : 1.0f;
    const size_t rows0 = (size_t)e0 * O;
    const uint8_t* bp = base + rows0 * G;
    const uint16_t* Bp = b + rows0 * r;
    const uint16_t* Ap = a + (size_t)e0 * r * G;
    uint8_t* op = out + rows0 * G;
    uint8_t* mp = mask ? mask + rows0 * G : nullptr;
    const int vec = G % 4 == 0 && al(bp, 4) && al(op, 4) && (mp == nullptr || al(mp, 4)) ? 1 : 0;
    const bool wide = scales_wide((int64_t)cols * ((O + 15) / 16) * m, r, w, vec);
#define SQ_QAST_SCALES(F, R) scales_gb<F, R>(wide, gb, w, m, s, bp, Bp, Ap, O, G, r, c, t, op, mp, vec)
    if (fmt == kMX) {
      if (r <= 8) SQ_QAST_SCALES(kMX, 8);
      else if (r <= 16) SQ_QAST_SCALES(kMX, 16);
      else if (r <= 32) SQ_QAST_SCALES(kMX, 32);
      else SQ_QAST_SCALES(kMX, 64);
    } else {
      if (r <= 8) SQ_QAST_SCALES(kNV, 8);
      else if (r <= 16) SQ_QAST_SCALES(kNV, 16);
      else if (r <= 32) SQ_QAST_SCALES(kNV, 32);
      else SQ_QAST_SCALES(kNV, 64);
    }
#undef SQ_QAST_SCALES
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// (callers were given room for partials of 32-row chunks, and still are)
size_t qast_grads_workspace(int E, int O, int G, int r) {
  return (size_t)E * ((O + 31) / 32) * r * G * sizeof(float);
}

template <int RT>
static void qast_grads_r(int E, int O, int G, int r, const float* dS, const uint8_t* mask, const uint16_t* B,
                         const uint16_t* A, float c, float* dB, float* dA, float* part, hipStream_t s) {
  const int chunks = (O + kDaRows - 1) / kDaRows;
  const auto al = [](const void* q, uintptr_t n) { return (reinterpret_cast<uintptr_t>(q) & (n - 1)) == 0; };
  const int vec = G % 4 == 0 && al(dS, 16) && al(A, 8) && (mask == nullptr || al(mask, 4)) ? 1 : 0;
  const int ndb = G > 64 ? (O + 15) / 16 : (O + 63) / 64, nda = ((G + 16 * da_u<RT>() - 1) / (16 * da_u<RT>())) * chunks;
  const int bvec = r % 2 == 0 && al(B, 4) ? 1 : 0;
  const bool runs = !vec && (int64_t)(ndb + nda) * E >= kDaRunsGrid;
  hipLaunchKernelGGL((runs ? qast_grads_kernel<RT, true> : qast_grads_kernel<RT, false>),
                     dim3((unsigned)(ndb + nda), (unsigned)E), dim3(256), 0, s, dS, mask, A, B, O, G, r, c, dB, part,
                     ndb, vec, bvec);
  const int64_t n = (int64_t)E * r * G;
  hipLaunchKernelGGL(qast_da_reduce_kernel, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, s, part, chunks, r, G, E, c,
                     dA);
}

int qast_grads_launch(int E, int O, int G, int r, const float* dS, const uint8_t* mask, const void* B, const void* A,
                      float c, float* dB, float* dA, void* workspace, hipStream_t s) {
  const uint16_t* b = static_cast<const uint16_t*>(B);
  const uint16_t* a = static_cast<const uint16_t*>(A);
  float* part = static_cast<float*>(workspace);
  if (r <= 16) qast_grads_r<1>(E, O, G, r, dS, mask, b, a, c, dB, dA, part, s);
  else if (r <= 32) qast_grads_r<2>(E, O, G, r, dS, mask, b, a, c, dB, dA, part, s);
  else qast_grads_r<4>(E, O, G, r, dS, mask, b, a, c, dB, dA, part, s);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace sq
