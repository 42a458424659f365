// Forward and dX for few tokens (decode, a serving batch, experts with a
// handful of routed rows) on gfx950.
//
// With few tokens the weight plane is the largest operand, a 128 x 128 tile
// is mostly padding and a grid of a layer's tiles leaves most CUs idle.  Here a
// workgroup owns a narrow strip of the output and walks the whole contraction
// in steps, its waves each with a job of their own and many steps of loads in
// flight.
//
// Every output element is one chain of matrix instructions in the order of the
// tiles (sq_gemm.hip): v_mfma_f32_16x16x32_bf16 gives, bit for bit, what the
// tiles' v_mfma_f32_32x32x16_bf16 gives in two, the first 16 terms in its lane
// groups 0 and 1 and the second 16 in groups 2 and 3 (compared over normal,
// widely spread and subnormal products).  So a row's result does not depend on
// how many rows come with it, an expert of a grouped call equals its single
// call on either path, and a launch takes whichever is the faster.
//
// MFMA operands of v_mfma_f32_16x16x32_bf16: lane l = (n, q) = (l % 16, l /
// 16) holds row (A) or column (B) n and 8 consecutive k; register r of the
// result holds row 4 q + r, column n.  Loading the token rows straight into
// that layout puts four rows under every four consecutive lanes, which the
// address unit serves at a third of the rate of whole 64-byte runs, so they are
// copied to LDS in whole rows instead.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sq_device.h"
#include "sq_gemm_args.h"

namespace sq {

typedef float f32x4 __attribute__((ext_vector_type(4)));

enum ThinMode { kThinFwd = 0, kThinDx = 1 };

// Waits until at most n copies of this wave are in flight and its LDS operations
// are done, then (BARRIER) for the other waves.  The copies are inline assembly
// and the waits builtins that name no memory: the empty statements keep the
// compiler from moving an LDS access, which another lane may depend on, across
// them.
template <int n, bool BARRIER>
__device__ __forceinline__ void thin_wait() {
  asm volatile("" ::: "memory");
  wait_vm_lgkm0<n>();
  if (BARRIER) __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
constexpr int kThinAnyLoads = 63;          // a wait that leaves register loads in flight

// f(0), .., f(N - 1) with the index as a constant.
template <int N, int I = 0, typename F>
__device__ __forceinline__ void thin_each(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    thin_each<N, I + 1>(f);
  }
}

// A workgroup takes 16 MT tokens x 16 NT columns of the output (outputs of the
// forward, input features of dX), in steps of 32 KF k (input features of the
// forward, rows of W of dX), with one barrier a step:
//   NT chain waves: the MFMA chains of one 16-column tile, MT of them.  In step
//     s they read the operands of s from LDS while they multiply what they read
//     before.
//   one loader wave: copies the token rows [16 MT][64 KF bytes] of step s + D - 1
//     into the ring slot of step s - 1, 16-byte chunk c of row r at c ^ (r % 16),
//     one KiB per copy; D - 2 steps stay in flight at the wait.
//   NT KF / 2 dequantising waves: 16 codes (one scale, whole within their row) a
//     lane, loaded P steps ahead into registers and written as the operands of
//     step s + 1 into the other of two buffers.  Forward: a wave takes 64 k of
//     the 16 rows of a tile; an operand is [4 lane groups][16][16 bytes], padded
//     so that the four parts of a row a store spans fall in different banks.
//     dX: a wave takes 32 rows of W; the operands are a [32 KF][32] bf16 tile,
//     chunk c of row k at c ^ (k / 4 % 4), from which the transposing read gives
//     each lane 8 consecutive k of its column.
// The chains are serial and the dequantising is not: this way both run at once,
// neither waits for its loads, and the waits of one kind do not hold up the
// other's (the copies are counted by hand, the register loads by the compiler).
// MFMA i of a step takes, in lane group q, the 8 k of chunk 4 i + q; in the
// order of the register forward (g.reg_order: it adds k = 8 j .. and 32 + 8 j ..
// of a 64-deep stage together) chunk 8 (i / 2) + 2 (i % 2) + q / 2 + 4 (q % 2).
// Reads past an operand's row or end give zeros (their offset is moved past
// the buffer), so ragged sizes take no branch.
constexpr int kThinLq = 256 + 64, kThinOp = 4 * kThinLq + 64;   // LDS bytes of a lane group, of an operand
constexpr int kThinDxCols = 32;

// Bytes of one operand buffer; MFMAs a chain wave reads ahead (its register sets
// hold MT + 1 operands for each).
template <int MODE, int NT, int KF>
constexpr int thin_ops() { return MODE == kThinFwd ? NT * KF * kThinOp : 32 * KF * kThinDxCols * 2; }
template <int MODE, int MT, int NT, int KF, int D>
constexpr int thin_lds() { return D * MT * KF * 1024 + 2 * thin_ops<MODE, NT, KF>(); }
template <int NT, int KF>
constexpr int thin_threads() { return 64 * (NT + 1 + NT * KF / 2); }
template <int MT>
constexpr int thin_part() { return MT == 1 ? 8 : MT == 2 ? 4 : 2; }

__device__ __forceinline__ int thin_dx_off(int k, int col) {
  return 2 * (k * kThinDxCols + ((((col >> 3) ^ (k >> 2)) & 3) << 3) + (col & 7));
}

template <int MODE, int FMT, int MT, int NT, int KF, int D, int P>
__device__ __forceinline__ void thin_tile(const GemmArgs& g, int tm, int tn, SQ_LDS uint8_t* lds) {
  constexpr int KS = 32 * KF, PX = MT * KF;               // k per step, copies per step
  constexpr int BLK = ScaleOperand<FMT>::kBlock;
  constexpr int kSlot = MT * KF * 1024, kOps = thin_ops<MODE, NT, KF>();
  static_assert(KF % 4 == 0 && KF <= 16, "a token row of 16 chunks or more, 64 at most");
  static_assert(MODE == kThinFwd || 16 * NT == kThinDxCols, "dX tiles are 32 columns wide");
  static_assert(D >= 3 && (D - 1) * PX <= 63, "the wait counts every copy in flight");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int T = g.T, O = g.O, I = g.I, G = g.G;
  const int K = MODE == kThinFwd ? I : O, N = MODE == kThinFwd ? O : I;
  const int t0 = tm * 16 * MT, n0 = tn * 16 * NT;
  const int steps = (K + KS - 1) / KS;
  SQ_LDS uint8_t* ops = lds + D * kSlot;

  if (wave < NT) {                                        // ---- chains of columns n0 + 16 wave ..
    const int n = lane & 15, q = lane >> 4;
    const bool regs = MODE == kThinFwd && g.reg_order;
    int xat[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int ch = regs ? 8 * (i >> 1) + 2 * (i & 1) + (q >> 1) + 4 * (q & 1) : 4 * i + q;
      xat[i] = n * (64 * KF) + 16 * (ch ^ n);             // 16 chunks on: 256 bytes on
    }
    // dX: the 16-lane group of k = 32 i + 8 q .. + 7 reads two 4 x 16 blocks; lane
    // n addresses row n / 4 of a block and receives its column n.  32 rows on, the
    // same place 64 x 32 bytes on.
    const int lo_at = thin_dx_off(8 * q + (n >> 2), 16 * wave + 4 * (n & 3));
    const int hi_at = thin_dx_off(8 * q + (n >> 2) + 4, 16 * wave + 4 * (n & 3));
    f32x4 acc[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int HF = thin_part<MT>() < KF ? thin_part<MT>() : KF, H = KF / HF;   // MFMAs of a part, parts of a step
    static_assert(H <= 2, "one or two parts");
    bf16x8 a[2][HF][MT], b[2][HF];
    int slot = 0;
    // part h of step s into register set u; the set before it is multiplied
    // while those reads are under way
    auto read = [&](int s, auto PART, auto SET) {
      constexpr int h = decltype(PART)::value, u = decltype(SET)::value & 1;
      const SQ_LDS uint8_t* x = lds + slot;
      const SQ_LDS uint8_t* w = ops + (s & 1) * kOps;
#pragma unroll
      for (int f = 0; f < HF; ++f) {
        const int i = h * HF + f;
        if constexpr (MODE == kThinFwd) {
          b[u][f] = *(const SQ_LDS bf16x8*)(w + (wave * KF + i) * kThinOp + q * kThinLq + n * 16);
        } else {
          const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SQ_LDS v4i16*)(w + lo_at + i * 64 * kThinDxCols));
          const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SQ_LDS v4i16*)(w + hi_at + i * 64 * kThinDxCols));
          __builtin_memcpy(&b[u][f], &lo, 8);
          __builtin_memcpy(reinterpret_cast<char*>(&b[u][f]) + 8, &hi, 8);
        }
#pragma unroll
        for (int m = 0; m < MT; ++m)
          a[u][f][m] = *(const SQ_LDS bf16x8*)(x + m * KF * 1024 + xat[i & 3] + 256 * (i >> 2));
      }
    };
    auto multiply = [&](auto SET) {
      constexpr int u = decltype(SET)::value & 1;
#pragma unroll
      for (int f = 0; f < HF; ++f)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][f][m], b[u][f], acc[m], 0, 0, 0);
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    // a step whose first part goes to set SET
    auto step = [&](int s, auto SET) {
      constexpr int u = decltype(SET)::value;
      thin_wait<kThinAnyLoads, true>();
      read(s, S0{}, std::integral_constant<int, u>{});
      if (s > 0) multiply(std::integral_constant<int, u + 1>{});
      if constexpr (H > 1) {
        read(s, S1{}, std::integral_constant<int, u + 1>{});
        multiply(std::integral_constant<int, u>{});
      }
      slot = slot + kSlot == D * kSlot ? 0 : slot + kSlot;
    };
    if constexpr (H == 2) {
      for (int s = 0; s < steps; ++s) step(s, S0{});
      multiply(S1{});
    } else {
      for (int s = 0; s < steps; s += 2) {
        step(s, S0{});
        if (s + 1 < steps) step(s + 1, S1{});
      }
      if (steps & 1) multiply(S0{});
      else multiply(S1{});
    }
    const int c = n0 + 16 * wave + n;
    if (c >= N) return;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int t = t0 + 16 * m + 4 * q + e;
        if (t >= T) break;
        const float v = FMT == kNV ? acc[m][e] * g.ws2 : acc[m][e];
        const uint32_t at = (uint32_t)t * (uint32_t)N + (uint32_t)c;
        if (g.out_bf16)
          reinterpret_cast<uint16_t*>(g.out)[at] = (uint16_t)f32_to_bf16_rne(v);
        else
          reinterpret_cast<float*>(g.out)[at] = v;
      }
  } else if (wave == NT) {                                // ---- token rows
    const DmaRsrc rx = make_dma_rsrc(g.a, (uint32_t)((size_t)T * K * 2));
    constexpr int kRows = 16 / KF, kCh = 4 * KF;          // rows of one copy, chunks of a row
    uint32_t xo[PX];
    int xk[PX];
#pragma unroll
    for (int u = 0; u < PX; ++u) {
      const int r = kRows * u + lane / kCh, c = (lane % kCh) ^ (r & 15), t = t0 + r;
      xk[u] = K - 8 * c;                                  // the chunk is inside while k0 < xk (K is a multiple of 8)
      xo[u] = t < T ? (uint32_t)t * (uint32_t)K * 2u + 16u * (uint32_t)c : kOOB;
    }
    auto issue = [&](int s, int slot) {
      const int k0 = KS * s;
#pragma unroll
      for (int u = 0; u < PX; ++u)
        dma16(rx, lds + slot + u * 1024, k0 < xk[u] ? xo[u] + (uint32_t)k0 * 2u : kOOB);
    };
#pragma unroll
    for (int d = 0; d < D - 1; ++d) issue(d, d * kSlot);
    int wr = (D - 1) * kSlot;
    for (int s = 0; s < steps; ++s) {
      thin_wait<(D - 2) * PX, true>();
      issue(s + D - 1, wr);
      wr = wr + kSlot == D * kSlot ? 0 : wr + kSlot;
    }
    thin_wait<0, false>();                                // the copies past the last step have landed
  } else {                                                // ---- weights
    const int d = wave - NT - 1;
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(g.codes, (uint32_t)((size_t)O * (I >> 1)));
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(g.scales, (uint32_t)((size_t)O * G));
    // the lane's 16 codes at step 0, inside while k0 < lim, and how far a step
    // moves them; where their two 8-code operand parts go
    uint32_t co, so, cstep, sstep;
    int lim, wat[2];
    if constexpr (MODE == kThinFwd) {
      const int j = d % NT, n = lane >> 2, c0 = 8 * (d / NT) + 2 * (lane & 3);    // tile, row, chunk within the step
      const int o = n0 + 16 * j + n;
      lim = o < O ? I - 8 * c0 : 0;
      co = (uint32_t)o * (uint32_t)(I >> 1) + 4u * (uint32_t)c0;
      so = (uint32_t)o * (uint32_t)G + (uint32_t)(8 * c0 / BLK);
      cstep = KS / 2;
      sstep = KS / BLK;
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const int c = c0 + w;
        const int i = g.reg_order ? 2 * (c >> 3) + ((c >> 1) & 1) : c >> 2;
        const int lq = g.reg_order ? 2 * (c & 1) + ((c >> 2) & 1) : c & 3;
        wat[w] = (j * KF + i) * kThinOp + lq * kThinLq + n * 16;
      }
    } else {
      const int k = 32 * d + (lane >> 1), i = n0 + 16 * (lane & 1);
      lim = i < I ? O - k : 0;
      co = (uint32_t)k * (uint32_t)(I >> 1) + (uint32_t)(i >> 1);
      so = (uint32_t)k * (uint32_t)G + (uint32_t)(i / BLK);
      cstep = (uint32_t)KS * (uint32_t)(I >> 1);
      sstep = (uint32_t)KS * (uint32_t)G;
#pragma unroll
      for (int w = 0; w < 2; ++w) wat[w] = thin_dx_off(k, 16 * (lane & 1) + 8 * w);
    }
    u32x2 cw[P];
    uint32_t sb[P];
    auto load = [&](int s, auto SET) {
      constexpr int u = decltype(SET)::value;
      const bool in = KS * s < lim;
      cw[u] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rc, (int)(in ? co + (uint32_t)s * cstep : kOOB), 0, 0));
      sb[u] = __builtin_amdgcn_raw_buffer_load_b8(rs, (int)(in ? so + (uint32_t)s * sstep : kOOB), 0, 0);
    };
    auto fill = [&](int s, auto SET) {
      constexpr int u = decltype(SET)::value;
      SQ_LDS uint8_t* p = ops + (s & 1) * kOps;
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const uint4 v = ScaleOperand<FMT>::dequant8(cw[u][w], ScaleOperand<FMT>::of(sb[u]));
        u32x4 x;
        __builtin_memcpy(&x, &v, 16);
        *(SQ_LDS u32x4*)(p + wat[w]) = x;
      }
    };
    // the buffer of step s was last read in step s - 2, before the barrier of s - 1
    thin_each<P>([&](auto SET) { load(decltype(SET)::value, SET); });
    for (int s0 = 0; s0 < steps; s0 += P)
      thin_each<P>([&](auto SET) {
        const int s = s0 + decltype(SET)::value;
        if (s >= steps) return;
        fill(s, SET);
        load(s + P, SET);
        thin_wait<kThinAnyLoads, true>();
      });
  }
}

template <int MODE, int FMT, int MT, int NT, int KF, int D, int P>
__global__ __launch_bounds__((thin_threads<NT, KF>())) void thin_kernel(GemmArgs g, int tiles_m) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[thin_lds<MODE, MT, NT, KF, D>()];
  static_assert(sizeof(lds) <= 160 * 1024, "LDS budget");
  const int b = xcd_stretch((int)blockIdx.x, (int)gridDim.x);
  thin_tile<MODE, FMT, MT, NT, KF, D, P>(g, b % tiles_m, b / tiles_m, (SQ_LDS uint8_t*)lds);
}

// Experts of a grouped call: positions [tile_begin[e], tile_begin[e + 1]) are
// expert e's strips, its token tiles next to each other so that one XCD reads
// a strip's weights once.
template <int MODE, int FMT, int MT, int NT, int KF, int D, int P>
__global__ __launch_bounds__((thin_threads<NT, KF>())) void thin_grouped_kernel(GemmGroup gg) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[thin_lds<MODE, MT, NT, KF, D>()];
  const int b = xcd_stretch((int)blockIdx.x, (int)gridDim.x);
  int lo = 0, hi = gg.count - 1;                          // last e with tile_begin[e] <= b
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (gg.tile_begin[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  GemmArgs g = gg.base;
  g.a = gg.act(lo);
  g.codes = gg.code_plane(lo);
  g.scales = gg.second(lo);
  g.out = gg.output(lo);
  g.T = gg.T[lo];
  g.ws2 = gg.ws2[lo];
  const int local = b - gg.tile_begin[lo], tiles_m = (g.T + 16 * MT - 1) / (16 * MT);
  thin_tile<MODE, FMT, MT, NT, KF, D, P>(g, local % tiles_m, local / tiles_m, (SQ_LDS uint8_t*)lds);
}

}  // namespace sq
