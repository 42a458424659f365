// Kernel arguments and small device helpers shared by the GEMM kernels
// (sq_gemm.hip) and the few-token kernels (sq_thin.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sq_device.h"
#include "sq_launch.h"

namespace sq {

constexpr int kXcds = 8;                // MI355X: workgroups are dealt round-robin to 8 XCDs
constexpr uint32_t kOOB = 0x80000000u;  // a buffer offset past every operand: reads zero
constexpr int kCUs = 256;               // MI355X compute units

#define SQ_LDS __attribute__((address_space(3)))
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct GemmArgs {
  const uint16_t* a;      // FWD: X [T,I]   DX: dY [T,O]   DS: X [T,I]
  const uint16_t* b;      // DS: dY [T,O]
  const uint8_t* codes;   // [O, I/2]
  const uint8_t* scales;  // [O, G]  (FWD, DX)
  void* out;              // FWD: Y [T,O]  DX: dX [T,I]  DS: dS [O,G] fp32
  int M, N, K;
  int T, O, I, G;
  float ws2;              // NV epilogue factor (1 for MX)
  int out_bf16;
  int reg_order;          // few-token forward: sum in the order of the register path (kFwdC)
  int ksplit;             // DS: K (token) ranges per tile; >1 writes partial planes to `out`
  int ksteps_per;         // DS: K stages per range
  // the launch covers output rows [m_off, m_off + m_cnt) and columns
  // [n_off, n_off + n_cnt) (a count of 0: up to M or N)
  int m_off, m_cnt, n_off, n_cnt;
};

// Up to kGroupMax experts per grouped launch, passed by value (kernel
// arguments stay under 4 KiB): each kind of pointer is a base and a 32-bit
// byte offset per expert, so the run of experts a launch takes is cut short
// where the pointers of one kind would span 4 GiB or more.  The second
// operand is dS's dY, or the forward's and dX's scale plane.  An operand an
// expert does not have (null, read with a size of zero) gets offset 0.
struct GemmGroup {
  GemmArgs base;                  // shared: O, I, G, N (fwd/dx) or M, N (ds), out_bf16
  const uint8_t* a0;
  const uint8_t* p0;
  const uint8_t* codes0;
  uint8_t* out0;
  uint32_t a[kGroupMax];
  uint32_t p[kGroupMax];
  uint32_t codes[kGroupMax];
  uint32_t out[kGroupMax];
  int T[kGroupMax];
  float ws2[kGroupMax];
  int tile_begin[kGroupMax];
  int count;
  __device__ const uint16_t* act(int e) const { return reinterpret_cast<const uint16_t*>(a0 + a[e]); }
  __device__ const uint8_t* second(int e) const { return p0 + p[e]; }
  __device__ const uint8_t* code_plane(int e) const { return codes0 + codes[e]; }
  __device__ void* output(int e) const { return out0 + out[e]; }
};
static_assert(sizeof(GemmGroup) <= 4096, "kernel argument budget");

// Bases and offsets of experts p[0, n) (dS: the second operand is b, else
// the scale plane); false when one kind's pointers span 4 GiB or more.
inline bool set_experts(GemmGroup& gg, const ExpertProblem* p, int n, bool ds) {
  auto pack = [&](auto get, const uint8_t*& base, uint32_t* off) {
    uintptr_t lo = UINTPTR_MAX, hi = 0;
    for (int e = 0; e < n; ++e) {
      const uintptr_t v = reinterpret_cast<uintptr_t>(get(p[e]));
      if (v == 0) continue;
      lo = v < lo ? v : lo;
      hi = v > hi ? v : hi;
    }
    if (lo == UINTPTR_MAX) lo = hi = 0;
    if (hi - lo > 0xFFFFFFFFu) return false;
    base = reinterpret_cast<const uint8_t*>(lo);
    for (int e = 0; e < n; ++e) {
      const uintptr_t v = reinterpret_cast<uintptr_t>(get(p[e]));
      off[e] = v == 0 ? 0u : (uint32_t)(v - lo);
    }
    return true;
  };
  const uint8_t* out0 = nullptr;
  const bool ok = pack([](const ExpertProblem& x) { return x.a; }, gg.a0, gg.a) &&
                  pack([ds](const ExpertProblem& x) { return ds ? x.b : static_cast<const void*>(x.scales); },
                       gg.p0, gg.p) &&
                  pack([](const ExpertProblem& x) { return x.codes; }, gg.codes0, gg.codes) &&
                  pack([](const ExpertProblem& x) { return x.out; }, out0, gg.out);
  gg.out0 = const_cast<uint8_t*>(out0);
  return ok;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// Buffer descriptor of the global -> LDS copies: base, num_records = bytes
// (offsets at or past it read zeros), raw buffer flags.
typedef int i32x4 __attribute__((ext_vector_type(4)));
struct DmaRsrc {
  i32x4 v;
};
__device__ __forceinline__ DmaRsrc make_dma_rsrc(const void* p, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  DmaRsrc r;
  r.v = i32x4{__builtin_amdgcn_readfirstlane((int)(uint32_t)a), __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32) & 0xFFFF),
              __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
  return r;
}

// 16 bytes per lane, global -> LDS; lane l writes dst + 16 l.  Written as
// the instruction itself: the compiler's wait insertion cannot tell the LDS
// tile a copy fills from the tile being read, and would otherwise stall
// every later LDS read until the copy lands.  The loop waits for the copies
// explicitly (vmcnt) before the barrier that publishes a stage.  The s_nop is
// the wait state that gfx9 needs between a write of M0 and a load to LDS; the
// compiler does not look for hazards inside the block.
__device__ __forceinline__ void dma16(DmaRsrc r, SQ_LDS void* dst, uint32_t voff) {
  const int lds = __builtin_amdgcn_readfirstlane((int)(uint32_t)reinterpret_cast<uintptr_t>(dst));
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(r.v)
               : "memory", "m0");
}

// Wait until at most n vector-memory loads of this wave are outstanding and
// all of its LDS operations are done (raw s_barrier has no memory semantics).
template <int n>
__device__ __forceinline__ void wait_vm_lgkm0() {
  static_assert(n >= 0 && n < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt(0x0070 | (n & 15) | ((n >> 4) << 14));
}

// Position in the tile order of workgroup bid of nb: XCD x = bid % 8 takes
// the x-th contiguous stretch of the order (stretches differ by at most one).
__device__ __forceinline__ int xcd_stretch(int bid, int nb) {
  const int x = bid % kXcds, q = nb / kXcds, r = nb % kXcds;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + bid / kXcds;
}

}  // namespace sq
