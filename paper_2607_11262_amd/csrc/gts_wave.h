// gts_wave.h — wave-level helpers shared by the simulation kernels: cross-lane
// sums, minima and max-plus scans by DPP, global-memory pointer types, and
// the node record held in registers.
#pragma once
#include <hip/hip_runtime.h>

#include "../../include/gts.h"
#include "gts_common.h"
#include "gts_dev.h"

namespace gts {

namespace {

// Node state: latest release cycle (low word) | released in-edges (high word).
__device__ __forceinline__ uint32_t* st_acc(uint64_t* st) { return reinterpret_cast<uint32_t*>(st); }
__device__ __forceinline__ uint32_t* st_cnt(uint64_t* st) { return reinterpret_cast<uint32_t*>(st) + 1; }

// A pointer into global memory (address space 1).
template <typename T>
using gmem = __attribute__((address_space(1))) T;

// Four consecutive words of global memory (one 16-B load).
__device__ __forceinline__ uint4 ld4(const gmem<const uint32_t>* p) { return make_uint4(p[0], p[1], p[2], p[3]); }

// Loads of words that global atomics may change bypass the L1.
template <typename T>
__device__ __forceinline__ T gld(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void mem_wait() { __builtin_amdgcn_s_waitcnt(0); }
__device__ __forceinline__ void wsync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Cross-lane steps by DPP (VALU lane shifts inside rows of 16 and row
// broadcasts) rather than LDS-crossbar shuffles: row_shr:n gives lane l the
// value of lane l - n of its row (lanes without one keep `old`); row_bcast:15
// / :31 give rows 1, 3 / rows 2, 3 lane 15 / lane 31 (other rows keep `old`).
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143;
template <int ctrl, int row_mask = 0xF>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, ctrl, row_mask, 0xF, false);
}
__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int l) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}

__device__ __forceinline__ uint32_t wave_incl_sum_u32(uint32_t x) {
  x += dpp<kRowShr1>(0u, x);
  x += dpp<kRowShr2>(0u, x);
  x += dpp<kRowShr4>(0u, x);
  x += dpp<kRowShr8>(0u, x);
  x += dpp<kRowBcast15, 0xA>(0u, x);
  x += dpp<kRowBcast31, 0xC>(0u, x);
  return x;
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) { return lane_u32(wave_incl_sum_u32(x), 63); }
__device__ __forceinline__ uint32_t wave_excl_scan_u32(uint32_t x) { return wave_incl_sum_u32(x) - x; }

// Wave-wide min / max of a u64 (uniform result): row reductions by DPP, then
// the four row results.
template <bool kMax>
__device__ __forceinline__ uint64_t wave_ext_u64(uint64_t x) {
  uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
  const uint32_t id = kMax ? 0u : ~0u;
#define GTS_EXT_STEP(C)                                              \
  {                                                                  \
    const uint32_t plo = dpp<C>(id, lo), phi = dpp<C>(id, hi);       \
    const bool less = phi < hi || (phi == hi && plo < lo);           \
    if (kMax ? (!less && (phi != hi || plo != lo)) : less) {         \
      lo = plo;                                                      \
      hi = phi;                                                      \
    }                                                                \
  }
  GTS_EXT_STEP(kRowShr1)
  GTS_EXT_STEP(kRowShr2)
  GTS_EXT_STEP(kRowShr4)
  GTS_EXT_STEP(kRowShr8)
#undef GTS_EXT_STEP
  uint64_t r = kMax ? 0ull : ~0ull;
#pragma unroll
  for (int l = 15; l < 64; l += 16) {
    const uint64_t v = ((uint64_t)lane_u32(hi, l) << 32) | lane_u32(lo, l);
    r = kMax ? (v > r ? v : r) : (v < r ? v : r);
  }
  return r;
}
// Wave-wide max of a u32 (uniform result).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  auto mx = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
  x = mx(x, dpp<kRowShr1>(0u, x));
  x = mx(x, dpp<kRowShr2>(0u, x));
  x = mx(x, dpp<kRowShr4>(0u, x));
  x = mx(x, dpp<kRowShr8>(0u, x));
  x = mx(x, dpp<kRowBcast15, 0xA>(0u, x));
  x = mx(x, dpp<kRowBcast31, 0xC>(0u, x));
  return lane_u32(x, 63);
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) { return ~wave_max_u32(~x); }

__device__ __forceinline__ uint64_t wmin64(uint64_t x) { return wave_ext_u64<false>(x); }
__device__ __forceinline__ uint64_t wmax64(uint64_t x) { return wave_ext_u64<true>(x); }

struct Compose {  // f(x) = max(x, a) + o on int64
  int64_t a, o;
};
constexpr int64_t kNegCycle = -(int64_t(1) << 62);  // below every cycle: max(x, kNegCycle) = x
// The DPP moves of dpp_c stay moves of their own in front of this subtraction:
// in 64 bits it is a pair with a carry, which the compiler gives no DPP
// operand (in 32 bits it does, wrongly for lanes without a source: the team
// kernel's MaxPlus32 keeps them apart).
__device__ __forceinline__ Compose compose(Compose f, Compose g) {  // g after f
  const int64_t ga = g.a - f.o;
  return Compose{f.a > ga ? f.a : ga, f.o + g.o};
}
template <int ctrl, int row_mask = 0xF>
__device__ __forceinline__ Compose dpp_c(Compose c) {  // lanes without a source get the identity
  const uint64_t a = (uint64_t)c.a, o = (uint64_t)c.o, na = (uint64_t)kNegCycle;
  const uint32_t alo = dpp<ctrl, row_mask>((uint32_t)na, (uint32_t)a);
  const uint32_t ahi = dpp<ctrl, row_mask>((uint32_t)(na >> 32), (uint32_t)(a >> 32));
  const uint32_t olo = dpp<ctrl, row_mask>(0u, (uint32_t)o);
  const uint32_t ohi = dpp<ctrl, row_mask>(0u, (uint32_t)(o >> 32));
  return Compose{(int64_t)(((uint64_t)ahi << 32) | alo), (int64_t)(((uint64_t)ohi << 32) | olo)};
}
// Inclusive scan of compositions across the wave (lane 0 first).
__device__ __forceinline__ Compose wave_incl_compose(Compose c) {
  c = compose(dpp_c<kRowShr1>(c), c);
  c = compose(dpp_c<kRowShr2>(c), c);
  c = compose(dpp_c<kRowShr4>(c), c);
  c = compose(dpp_c<kRowShr8>(c), c);
  c = compose(dpp_c<kRowBcast15, 0xA>(c), c);
  c = compose(dpp_c<kRowBcast31, 0xC>(c), c);
  return c;
}
__device__ __forceinline__ Compose lane_c(Compose c, int l) {
  const uint64_t a = (uint64_t)c.a, o = (uint64_t)c.o;
  return Compose{(int64_t)(((uint64_t)lane_u32((uint32_t)(a >> 32), l) << 32) | lane_u32((uint32_t)a, l)),
                 (int64_t)(((uint64_t)lane_u32((uint32_t)(o >> 32), l) << 32) | lane_u32((uint32_t)o, l))};
}

// A node record held in registers: a = {op | out-degree << 16, cta,
// succ_begin, succ0}, b = {succ1, succ2, indeg0 | indeg1 << 16, indeg2}.
struct Rec {
  uint4 a, b;
  __device__ __forceinline__ uint32_t op() const { return a.x & 0xFFFFu; }
  __device__ __forceinline__ uint32_t nsucc() const { return a.x >> 16; }
  __device__ __forceinline__ uint32_t cta() const { return a.y; }
  __device__ __forceinline__ uint32_t sb() const { return a.z; }
  __device__ __forceinline__ uint32_t succ(uint32_t k) const { return k == 0 ? a.w : k == 1 ? b.x : b.y; }
  __device__ __forceinline__ uint32_t sindeg(uint32_t k) const {
    return k == 0 ? (b.z & 0xFFFFu) : k == 1 ? (b.z >> 16) : (b.w & 0xFFFFu);
  }
};
__device__ __forceinline__ Rec load_rec(const NodeDev* nodes, uint32_t v) {
  const uint4* p = reinterpret_cast<const uint4*>(nodes + v);
  return Rec{p[0], p[1]};
}

// Does a node need the one-edge-at-a-time path (more than three successors,
// or an inline successor that is a shared node)?
__device__ __forceinline__ bool needs_slow(const Rec r) {
  const uint32_t n = r.nsucc();
  if (n > kInlineSucc) return true;
  bool sh = false;
#pragma unroll
  for (uint32_t k = 0; k < kInlineSucc; ++k) sh |= k < n && ((r.succ(k) >> GTS_EDGE_KIND_SHIFT) & kDevShared);
  return sh;
}

}  // namespace

}  // namespace gts
