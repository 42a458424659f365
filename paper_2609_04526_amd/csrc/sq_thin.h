// Forward and dX for few tokens (decode, a serving batch, experts with a
// handful of routed rows) on gfx950.
//
// With few tokens the weight plane is the largest operand, a 128 x 128 tile
// is mostly padding and a grid of O / 128 workgroups leaves most CUs idle,
// each of them walking the whole contraction alone.  Here a workgroup owns a
// narrow strip of the output (16 MT tokens x 16 NT outputs of the forward, x
// 32 input features of dX) and its 8 waves split the contraction: wave w
// takes the K steps w, w + 8, ..., D of them in flight, through LDS buffers of
// its own (no barrier in the loop), and the 8 partial sums are added through
// LDS in wave order.  Every weight is read and dequantised once per 16 MT
// tokens.  The summation order of an output element depends on the
// contraction length alone (not on MT, NT, D or the launch), so an expert of a
// grouped call equals its single call bit for bit.
//
// MFMA operands of v_mfma_f32_16x16x32_bf16: lane l = (n, q) = (l % 16, l /
// 16) holds row (A) or column (B) n and the 8 consecutive k from 8 q;
// register r of the result holds row 4 q + r, column n.  Loading the token
// rows straight into that layout puts four rows under every four consecutive
// lanes, which the address unit serves at a third of the rate of whole
// 64-byte runs (the 4096 x 4096 forward at 64 tokens 18 us), so they are
// copied to LDS in whole rows instead.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sq_device.h"
#include "sq_gemm_args.h"

namespace sq {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Which calls (and experts) take these kernels: T tokens over a contraction of
// length K (I in the forward, O in dX).  Single products are faster here up to
// 64 tokens at every size tried (see thin_fwd_pick).  But a strip is a third
// as efficient as a tile once experts fill the chip, and an expert has to
// take the path its single call takes.  So contractions as short as the
// 30B-A3B MoE's (768 and 2048) stay on tiles: with 64 tokens for every K its
// layer at 4096 tokens (a tenth of the experts under 65 rows) went from 512 to
// 528 us with the small experts in a launch of their own and to 561 with them
// among the tiles, and with 16 tokens its layer at 326 tokens from 154 to 185
// (single products of that length are near the launch's own time either way).
__host__ __device__ inline bool thin_takes(int T, int K) { return K > 2048 && T <= 64; }

constexpr int kThinKWaves = 8;             // waves that split the contraction
constexpr int kThinThreads = 64 * kThinKWaves;

// Every wave has an LDS region of its own (region(w)), which first holds its
// operand buffers and in the end its partial sums: a [16][cols + 4] fp32 plane
// per token tile (the pad spreads the four rows a lane group stores over all
// banks).
constexpr int thin_red_bytes(int mt, int cols) { return mt * 16 * (cols + 4) * 4; }

// Adds the waves' partial planes in wave order and stores the strip: rows
// t0 .. t0 + 16 MT - 1, columns c0 .. c0 + COLS - 1 of the [T, N] output.
template <int FMT, int MT, int COLS, typename Region>
__device__ __forceinline__ void thin_store(const GemmArgs& g, Region region, int t0, int c0, int T, int N) {
  constexpr int S = COLS + 4;
#pragma unroll
  for (int u = 0; u < (MT * 16 * COLS + kThinThreads - 1) / kThinThreads; ++u) {
    const int e = (int)threadIdx.x + kThinThreads * u;
    if (MT * 16 * COLS % kThinThreads != 0 && e >= MT * 16 * COLS) break;
    const int m = e / (16 * COLS), r = e / COLS % 16, c = e % COLS;
    const int at_ = (m * 16 + r) * S + c;
    float v = ((const SQ_LDS float*)region(0))[at_];
#pragma unroll
    for (int w = 1; w < kThinKWaves; ++w) v += ((const SQ_LDS float*)region(w))[at_];
    if constexpr (FMT == kNV) v *= g.ws2;
    const int t = t0 + 16 * m + r, n = c0 + c;
    if (t >= T || n >= N) continue;
    const uint32_t at = (uint32_t)t * (uint32_t)N + (uint32_t)n;
    if (g.out_bf16)
      reinterpret_cast<uint16_t*>(g.out)[at] = (uint16_t)f32_to_bf16_rne(v);
    else
      reinterpret_cast<float*>(g.out)[at] = v;
  }
}

// The wave's accumulators into its partial planes.
template <int MT, int NT>
__device__ __forceinline__ void thin_park(const f32x4 (&acc)[MT][NT], SQ_LDS float* red, int n, int q) {
  constexpr int S = 16 * NT + 4;
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        red[(m * 16 + 4 * q + e) * S + 16 * j + n] = acc[m][j][e];
}

// ------------------------------------------------------------------ forward
// A step is 128 deep.  LDS of a wave, per step in flight: the token rows
// [16 MT][256 bytes], 16-byte chunk c of row r at chunk c ^ (r % 16), copied
// four whole 256-byte runs per instruction; and the packed codes [16 NT][64
// bytes], chunk c of row r at c ^ (r / 4 % 4).  MFMA kk takes k = 32 kk + 8 q:
// the token chunk 4 kk + q and the code word q of chunk kk, both free of bank
// conflicts (16 rows at one chunk; 16 rows x 4 words).  The scale bytes stay
// in registers: block kk (MXFP4) or 2 kk + q / 2 (NVFP4) of the step.  Reads
// past an operand's row or end give zeros (their offset is moved past the
// buffer), so ragged sizes take no branch.
template <int MT, int NT, int D>
constexpr int thin_fwd_wave_bytes() { return D * (MT * 4096 + NT * 1024); }

template <int FMT, int MT, int NT, int D, typename Region>
__device__ __forceinline__ void thin_fwd_tile(const GemmArgs& g, int tm, int tn, Region region) {
  static_assert(thin_red_bytes(MT, 16 * NT) <= thin_fwd_wave_bytes<MT, NT, D>(), "the partial sums fit the region");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int n = lane & 15, q = lane >> 4;
  const int T = g.T, O = g.O, I = g.I, G = g.G;
  const int t0 = tm * 16 * MT, o0 = tn * 16 * NT;
  const DmaRsrc rx = make_dma_rsrc(g.a, (uint32_t)((size_t)T * I * 2));
  const DmaRsrc rc = make_dma_rsrc(g.codes, (uint32_t)((size_t)O * (I >> 1)));
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(g.scales, (uint32_t)((size_t)O * G));
  SQ_LDS uint8_t* mine = region(wave);

  // copies: lane l moves stored chunk l % 16 of token row 4 i + l / 16, and
  // stored chunk l % 4 of code row l / 4.  A row outside the operand starts
  // past the buffer and stays there (offsets below 2^31 are added to 2^31).
  uint32_t xo[MT][4], co[NT], so[NT];
  int xk[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 4 * i + q, c = n ^ r;
    xk[i] = 8 * c;                                        // first k of the chunk within the step
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int t = t0 + 16 * m + r;
      xo[m][i] = t < T ? (uint32_t)t * (uint32_t)I * 2u + 16u * (uint32_t)c : kOOB;
    }
  }
  const int cr = lane >> 2, cc = (lane & 3) ^ ((cr >> 2) & 3);
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int oc = o0 + 16 * j + cr, on = o0 + 16 * j + n;
    co[j] = oc < O ? (uint32_t)oc * (uint32_t)(I >> 1) + 16u * (uint32_t)cc : kOOB;
    so[j] = on < O ? (uint32_t)on * (uint32_t)G : kOOB;
  }
  // whole scale words per row and step: one load instead of four bytes
  const bool words = G % 4 == 0 && (reinterpret_cast<uintptr_t>(g.scales) & 3) == 0;

  f32x4 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[m][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  const int steps = (I + 127) / 128;
  for (int sb = wave; sb < steps; sb += kThinKWaves * D) {
    uint32_t sw[D][NT];                                   // the lane's four scale bytes of the step
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int k0 = 128 * (sb + kThinKWaves * d);
      SQ_LDS uint8_t* xs = mine + d * (MT * 4096 + NT * 1024);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          dma16(rx, xs + m * 4096 + i * 1024, k0 + xk[i] < I ? xo[m][i] + (uint32_t)k0 * 2u : kOOB);
#pragma unroll
      for (int j = 0; j < NT; ++j)
        dma16(rc, xs + MT * 4096 + j * 1024, k0 + 32 * cc < I ? co[j] + (uint32_t)(k0 >> 1) : kOOB);
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        if (words) {
          if constexpr (FMT == kMX) {
            sw[d][j] = __builtin_amdgcn_raw_buffer_load_b32(
                rs, (int)(k0 < I ? so[j] + (uint32_t)(k0 >> 5) : kOOB), 0, 0);
          } else {
            const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b32(
                rs, (int)(k0 < I ? so[j] + (uint32_t)(k0 >> 4) : kOOB), 0, 0);
            const uint32_t hi = __builtin_amdgcn_raw_buffer_load_b32(
                rs, (int)(k0 + 64 < I ? so[j] + (uint32_t)(k0 >> 4) + 4u : kOOB), 0, 0);
            // bytes h, 2 + h of each word, h = q / 2
            sw[d][j] = __builtin_amdgcn_perm(hi, lo, q & 2 ? 0x07050301u : 0x06040200u);
          }
        } else {
          uint32_t b[4];
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) {
            const int k = k0 + 32 * kk + (FMT == kNV ? 16 * (q >> 1) : 0);
            b[kk] = __builtin_amdgcn_raw_buffer_load_b8(
                rs, (int)(k < I ? so[j] + (uint32_t)(k >> (FMT == kNV ? 4 : 5)) : kOOB), 0, 0);
          }
          sw[d][j] = b[0] | (b[1] << 8) | (b[2] << 16) | (b[3] << 24);
        }
      }
    }
    wait_vm_lgkm0<0>();                                   // the copies have landed (and only this wave reads them)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const SQ_LDS uint8_t* xs = mine + d * (MT * 4096 + NT * 1024);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        bf16x8 a[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m)
          a[m] = *(const SQ_LDS bf16x8*)(xs + m * 4096 + n * 256 + 16 * ((4 * kk + q) ^ n));
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const uint32_t w = *(const SQ_LDS uint32_t*)(xs + MT * 4096 + j * 1024 + n * 64 +
                                                       16 * (kk ^ ((n >> 2) & 3)) + 4 * q);
          const uint4 v = ScaleOperand<FMT>::dequant8(w, ScaleOperand<FMT>::of((sw[d][j] >> (8 * kk)) & 0xFFu));
          bf16x8 b;
          __builtin_memcpy(&b, &v, 16);
          // an 8-code word past the row's end (NVFP4 rows may end inside a
          // chunk) belongs to the next row: its tokens read zeros, and so must it
          if (FMT == kNV && 128 * (sb + kThinKWaves * d) + 32 * kk + 8 * q >= I) b = bf16x8{};
#pragma unroll
          for (int m = 0; m < MT; ++m)
            acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b, acc[m][j], 0, 0, 0);
        }
      }
    }
    wait_vm_lgkm0<0>();                                   // every read is done before the buffers are refilled
    __builtin_amdgcn_sched_barrier(0);
  }
  thin_park<MT, NT>(acc, (SQ_LDS float*)mine, n, q);
  __syncthreads();
  thin_store<FMT, MT, 16 * NT>(g, region, t0, o0, T, O);
}

// ------------------------------------------------------------------ dX
// A step is 64 rows of W (64 k) x 32 input features: lane l loads the 16
// bytes of row l (one MXFP4 block, two NVFP4 blocks), dequantises them and
// writes them to the wave's own [64][32] bf16 tile, from which the transposing
// read gives each lane 8 consecutive k of its column (16-byte chunk c of tile
// row k at chunk c ^ (k / 4 % 4)).  The token rows of dY are copied to LDS as
// [16 MT][128 bytes] per step, chunk c of row r at c ^ ((r ^ r / 8) % 8).
// Neighbouring strips read the same 128-byte lines of W and are dealt to one
// XCD, whose L2 fetches them once.
constexpr int kThinDxCols = 32;
constexpr int kThinDxTileBytes = 64 * kThinDxCols * 2;

__device__ __forceinline__ int thin_dx_off(int k, int col) {
  return k * kThinDxCols + ((((col >> 3) ^ (k >> 2)) & 3) << 3) + (col & 7);
}

template <int MT, int D>
constexpr int thin_dx_wave_bytes() { return kThinDxTileBytes + D * MT * 2048; }

template <int FMT, int MT, int D, typename Region>
__device__ __forceinline__ void thin_dx_tile(const GemmArgs& g, int tm, int tn, Region region) {
  static_assert(thin_red_bytes(MT, kThinDxCols) <= thin_dx_wave_bytes<MT, D>(), "the partial sums fit the region");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int n = lane & 15, q = lane >> 4;
  const int T = g.T, O = g.O, I = g.I, G = g.G;
  const int t0 = tm * 16 * MT, i0 = tn * kThinDxCols;
  const DmaRsrc ry = make_dma_rsrc(g.a, (uint32_t)((size_t)T * O * 2));
  const __amdgpu_buffer_rsrc_t rc = make_rsrc(g.codes, (uint32_t)((size_t)O * (I >> 1)));
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(g.scales, (uint32_t)((size_t)O * G));
  SQ_LDS uint8_t* mine = region(wave);
  SQ_LDS uint16_t* tile = (SQ_LDS uint16_t*)mine;
  SQ_LDS uint8_t* ys = mine + kThinDxTileBytes;

  // copies of dY: lane l moves stored chunk l % 8 of row 8 i + l / 8
  uint32_t yo[MT][2];
  int yk[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = 8 * i + (lane >> 3), c = (lane & 7) ^ ((r ^ (r >> 3)) & 7);
    yk[i] = 8 * c;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int t = t0 + 16 * m + r;
      yo[m][i] = t < T ? (uint32_t)t * (uint32_t)O * 2u + 16u * (uint32_t)c : kOOB;
    }
  }
  f32x4 acc[MT][2];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[m][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  const int steps = (O + 63) / 64;
  for (int sb = wave; sb < steps; sb += kThinKWaves * D) {
    u32x4 cw[D];
    uint32_t sc[D][FMT == kNV ? 2 : 1];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int k0 = 64 * (sb + kThinKWaves * d);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 2; ++i)                       // O is a multiple of 8
          dma16(ry, ys + (d * MT + m) * 2048 + i * 1024, k0 + yk[i] < O ? yo[m][i] + (uint32_t)k0 * 2u : kOOB);
      const int o = k0 + lane;
      const uint32_t co = (uint32_t)o * (uint32_t)(I >> 1) + (uint32_t)(i0 >> 1);
      if constexpr (FMT == kMX) {
        const bool in = o < O;                            // i0 < I, and I is a multiple of 32
        cw[d] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rc, (int)(in ? co : kOOB), 0, 0));
        sc[d][0] = __builtin_amdgcn_raw_buffer_load_b8(
            rs, (int)(in ? (uint32_t)o * (uint32_t)G + (uint32_t)(i0 >> 5) : kOOB), 0, 0);
      } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {                     // the row may end between the two blocks
          const bool in = o < O && i0 + 16 * h < I;
          const u32x2 v = __builtin_bit_cast(
              u32x2, __builtin_amdgcn_raw_buffer_load_b64(rc, (int)(in ? co + 8u * h : kOOB), 0, 0));
          cw[d][2 * h] = v[0];
          cw[d][2 * h + 1] = v[1];
          sc[d][h] = __builtin_amdgcn_raw_buffer_load_b8(
              rs, (int)(in ? (uint32_t)o * (uint32_t)G + (uint32_t)(i0 >> 4) + h : kOOB), 0, 0);
        }
      }
    }
    wait_vm_lgkm0<0>();                                   // the copies have landed (and only this wave reads them)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint4 v = ScaleOperand<FMT>::dequant8(cw[d][c], ScaleOperand<FMT>::of(sc[d][FMT == kNV ? c >> 1 : 0]));
        u32x4 w;
        __builtin_memcpy(&w, &v, 16);
        *(SQ_LDS u32x4*)(tile + thin_dx_off(lane, 8 * c)) = w;
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        bf16x8 a[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m)
          a[m] = *(const SQ_LDS bf16x8*)(ys + (d * MT + m) * 2048 + n * 128 +
                                         16 * ((4 * kk + q) ^ ((n ^ (n >> 3)) & 7)));
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          // the 16-lane group of k = 32 kk + 8 q .. + 7: lane n addresses row
          // n / 4 of a 4 x 16 block and receives its column n
          const int k = 32 * kk + 8 * q + (n >> 2), col = 16 * j + 4 * (n & 3);
          const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SQ_LDS v4i16*)(tile + thin_dx_off(k, col)));
          const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SQ_LDS v4i16*)(tile + thin_dx_off(k + 4, col)));
          bf16x8 b;
          __builtin_memcpy(&b, &lo, 8);
          __builtin_memcpy(reinterpret_cast<char*>(&b) + 8, &hi, 8);
#pragma unroll
          for (int m = 0; m < MT; ++m)
            acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b, acc[m][j], 0, 0, 0);
        }
      }
    }
    wait_vm_lgkm0<0>();                                   // every read is done before the buffers are refilled
    __builtin_amdgcn_sched_barrier(0);
  }
  thin_park<MT, 2>(acc, (SQ_LDS float*)mine, n, q);
  __syncthreads();
  thin_store<FMT, MT, kThinDxCols>(g, region, t0, i0, T, I);
}

template <int FMT, int MT, int NT, int D>
__global__ __launch_bounds__(kThinThreads) void thin_fwd_kernel(GemmArgs g, int tiles_m) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kThinKWaves * thin_fwd_wave_bytes<MT, NT, D>()];
  static_assert(sizeof(lds) <= 160 * 1024, "LDS budget");
  const int b = xcd_stretch((int)blockIdx.x, (int)gridDim.x);
  thin_fwd_tile<FMT, MT, NT, D>(g, b % tiles_m, b / tiles_m,
                                 [&](int w) { return (SQ_LDS uint8_t*)lds + w * thin_fwd_wave_bytes<MT, NT, D>(); });
}

template <int FMT, int MT, int D>
__global__ __launch_bounds__(kThinThreads) void thin_dx_kernel(GemmArgs g, int tiles_m) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kThinKWaves * thin_dx_wave_bytes<MT, D>()];
  static_assert(sizeof(lds) <= 160 * 1024, "LDS budget");
  const int b = xcd_stretch((int)blockIdx.x, (int)gridDim.x);
  thin_dx_tile<FMT, MT, D>(g, b % tiles_m, b / tiles_m,
                           [&](int w) { return (SQ_LDS uint8_t*)lds + w * thin_dx_wave_bytes<MT, D>(); });
}

// Experts of a grouped call (or the one product of a single call's group):
// positions [tile_begin[e], tile_begin[e + 1]) are expert e's strips, its token
// tiles next to each other so that one XCD reads a strip's weights once.
template <int ROWS>
__device__ __forceinline__ bool thin_expert(const GemmGroup& gg, GemmArgs& g, int strips, int& tm, int& tn) {
  const int b = xcd_stretch((int)blockIdx.x, (int)gridDim.x);
  int lo = 0, hi = gg.count - 1;                 // last e with tile_begin[e] <= b
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (gg.tile_begin[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  g = gg.base;
  g.a = gg.act(lo);
  g.codes = gg.code_plane(lo);
  g.scales = gg.second(lo);
  g.out = gg.output(lo);
  g.T = gg.T[lo];
  g.ws2 = gg.ws2[lo];
  const int local = b - gg.tile_begin[lo], tiles_m = (g.T + ROWS - 1) / ROWS;
  tm = local % tiles_m;
  tn = local / tiles_m;
  return tn < strips;
}

template <int FMT, int MT, int NT, int D>
__global__ __launch_bounds__(kThinThreads) void thin_fwd_grouped_kernel(GemmGroup gg) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kThinKWaves * thin_fwd_wave_bytes<MT, NT, D>()];
  GemmArgs g;
  int tm, tn;
  if (!thin_expert<16 * MT>(gg, g, (gg.base.O + 16 * NT - 1) / (16 * NT), tm, tn)) return;
  thin_fwd_tile<FMT, MT, NT, D>(g, tm, tn,
                                [&](int w) { return (SQ_LDS uint8_t*)lds + w * thin_fwd_wave_bytes<MT, NT, D>(); });
}

template <int FMT, int MT, int D>
__global__ __launch_bounds__(kThinThreads) void thin_dx_grouped_kernel(GemmGroup gg) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[kThinKWaves * thin_dx_wave_bytes<MT, D>()];
  GemmArgs g;
  int tm, tn;
  if (!thin_expert<16 * MT>(gg, g, (gg.base.I + kThinDxCols - 1) / kThinDxCols, tm, tn)) return;
  thin_dx_tile<FMT, MT, D>(g, tm, tn,
                           [&](int w) { return (SQ_LDS uint8_t*)lds + w * thin_dx_wave_bytes<MT, D>(); });
}

// ------------------------------------------------------------------ launch
// Strip of the forward for experts of T[0 .. n-1] tokens: the (MT, NT) of the
// least time by a model of one workgroup, a token copies (MT), b dequantises
// (NT) and c multiplies (MT NT) per step, times the rounds its grid takes (160
// KB of LDS: one workgroup per CU from MT = 4 or 2 x 4 on).  Fitted to
// sweeps at 4096 x 4096, 14336 x 4096 and 4096 x 14336 (microseconds over the
// launch at I = 4096): MXFP4 a = 1.2, b = 0.5, c = 0.35; NVFP4, whose codes
// take four times the instructions, b = 2.  T = 64: 4096 x 4096 39.7 -> 7.9
// us with 2 x 2 tiles (4 x 4: 15.0), 14336 x 4096 39.9 -> 16.3 with 4 x 4 (2
// x 2: 22.6).
struct ThinPick {
  int mt, nt;
};
inline ThinPick thin_fwd_pick(int fmt, const int* T, int n, int O) {
  static constexpr ThinPick kPicks[] = {{1, 1}, {1, 2}, {1, 4}, {2, 1}, {2, 2}, {2, 4}, {4, 1}, {4, 2}, {4, 4}};
  int most = 0;
  for (int e = 0; e < n; ++e) most = T[e] > most ? T[e] : most;
  ThinPick best = kPicks[0];
  double best_t = 1e30;
  for (const ThinPick& p : kPicks) {
    if (p.mt > 1 && most <= 8 * p.mt) continue;           // half the tile's rows or more would be padding
    int64_t wgs = 0;
    for (int e = 0; e < n; ++e) wgs += (T[e] + 16 * p.mt - 1) / (16 * p.mt);
    wgs *= (O + 16 * p.nt - 1) / (16 * p.nt);
    const bool one_per_cu = p.mt * 4 + p.nt > 10;         // more than 80 KB of LDS
    double rounds = (double)wgs / kCUs;
    if (one_per_cu) rounds = (double)((wgs + kCUs - 1) / kCUs);
    if (rounds < 1.0) rounds = 1.0;
    const double t = rounds * (1.2 * p.mt + (fmt == kNV ? 2.0 : 0.5) * p.nt + 0.35 * p.mt * p.nt);
    if (t < best_t) {
      best_t = t;
      best = p;
    }
  }
  return best;
}

}  // namespace sq
