// Wave-level pieces of the packet traversals: wave-uniform values and lane
// access, the segment-box test, and the traversal stack in VGPR lanes.
#pragma once
#pragma clang fp contract(off)

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pr {
namespace {  // each translation unit keeps its own copy

__device__ __forceinline__ uint64_t ballot(bool b) { return __ballot(b); }

__device__ __forceinline__ int lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ int32_t uni(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint64_t uni64(uint64_t v) {
  uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// v_writelane_b32: `old` with lane `lane` replaced by the uniform value v
// (the LLVM intrinsic; this clang has no builtin spelling for it).
__device__ int32_t lane_write(int32_t v, int32_t lane, int32_t old) __asm("llvm.amdgcn.writelane.i32");

__device__ __forceinline__ bool meet6(const float* g, float lx, float ly, float lz, float hx, float hy, float hz) {
  return (g[0] <= hx) & (lx <= g[3]) & (g[1] <= hy) & (ly <= g[4]) & (g[2] <= hz) & (lz <= g[5]);
}

__device__ __forceinline__ float lane_f(float v, int j) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), j));
}

__device__ __forceinline__ uint64_t lane_u64(uint64_t v, int j) {
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, j);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), j);
  return ((uint64_t)hi << 32) | lo;
}

// Segment-box test (conservative): slab test on t in [0, 1] for the segment
// p + t (q - p), with t computed as (plane - p) * fl(1 / fl(q - p)); every t
// carries a relative error of at most gamma_4 = 4 eps / (1 - 4 eps), so
// accepting when t_min <= t_max (1 + 2^-19) + 2^-120 never rejects a box the
// exact segment touches (closed boxes).  A zero direction component uses a
// large finite reciprocal (2^100) and a bias of 2^16 that turns the slab into
// "no constraint" or "empty" exactly.  Valid for FP32-safe coordinates; for
// other meshes every box is accepted and every leaf test is deferred.
constexpr float kSlabK = 1.0f + 0x1p-19f;
constexpr float kSlabS = 0x1p-120f;
constexpr float kZeroInv = 0x1p100f;
constexpr float kZeroBias = 0x1p16f;

struct Ray {
  float px, py, pz, ix, iy, iz, bx, by, bz;
};

__device__ __forceinline__ void axis_setup(float d, bool safe, float& inv, float& bias) {
  if (!safe) { inv = 0.f; bias = INFINITY; return; }
  if (d != 0.f) { inv = 1.0f / d; bias = 0.f; }
  else { inv = kZeroInv; bias = kZeroBias; }
}

// t = (plane - p) * inv -+ bias as one fused multiply-add: with bias 0 (a
// non-zero direction component) the value is the rounded product, as two
// separate operations would give; with a zero component the sign of
// (plane - p) is kept exactly and the bias opens the slab to all t, or
// pushes it away from [0, 1].
__device__ __forceinline__ bool slab(const Ray& r, float lx, float ly, float lz, float hx, float hy, float hz) {
  float t0x = fmaf(lx - r.px, r.ix, -r.bx), t1x = fmaf(hx - r.px, r.ix, r.bx);
  float t0y = fmaf(ly - r.py, r.iy, -r.by), t1y = fmaf(hy - r.py, r.iy, r.by);
  float t0z = fmaf(lz - r.pz, r.iz, -r.bz), t1z = fmaf(hz - r.pz, r.iz, r.bz);
  float tn = fmaxf(fmaxf(fminf(t0x, t1x), fminf(t0y, t1y)), fmaxf(fminf(t0z, t1z), 0.f));
  float tf = fminf(fminf(fmaxf(t0x, t1x), fmaxf(t0y, t1y)), fminf(fmaxf(t0z, t1z), 1.f));
  return tn <= fmaf(tf, kSlabK, kSlabS);
}

// The same values in fewer instructions: the hardware reciprocal (1 ulp) and one
// Newton step are the correctly rounded quotient 1 / d for every d of magnitude
// 2^-64 ... 2^43 (compared for all of them on gfx950); FP32-safe coordinates
// differ by 0 or by 2^-63 ... 2^41.
__device__ __forceinline__ void axis_rcp(float d, bool safe, float& inv, float& bias) {
  const bool zero = d == 0.f;
  const float r = __builtin_amdgcn_rcpf(d);
  inv = zero ? kZeroInv : fmaf(fmaf(-d, r, 1.0f), r, r);
  bias = zero ? kZeroBias : 0.f;
  if (!safe) { inv = 0.f; bias = INFINITY; }
}

// Stack entries kept in VGPR lanes.
constexpr int kRegStack = 64;


struct WaveStack {
  int32_t ref;
  int32_t mlo, mhi;
  int32_t* lref;
  uint64_t* lmask;
  int32_t top;
  // entries reg_lo .. reg_lo + kRegStack - 1 live in VGPR lanes 0 .. 63, the
  // others at LDS index i - lds_lo (plain integers, so that the placement
  // of an entry is decided by scalar instructions)
  int32_t reg_lo;
  int32_t lds_lo;
};

// Pushes onto a stack whose first kRegStack entries live in VGPR lanes and the
// others in LDS.
__device__ __forceinline__ void push_node(WaveStack& s, int32_t ref, uint64_t m) {
  if (s.top < kRegStack) {
    s.ref = lane_write(ref, s.top, s.ref);
    s.mlo = lane_write((int32_t)(uint32_t)m, s.top, s.mlo);
    s.mhi = lane_write((int32_t)(uint32_t)(m >> 32), s.top, s.mhi);
  } else if ((threadIdx.x & 63) == 0) {
    s.lref[s.top - kRegStack] = ref;
    s.lmask[s.top - kRegStack] = m;
  }
  ++s.top;
}

}  // namespace
}  // namespace pr
