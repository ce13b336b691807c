// Device helpers shared by the libsx kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sx {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// bfloat16 stored as the upper half of a float32: widening is exact.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Two float32 -> packed bfloat16, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  bf16x2_t v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// Value of v in lane src of the wave (src taken mod 64).
__device__ __forceinline__ int lane_value(int v, int src) { return __builtin_amdgcn_ds_bpermute(src << 2, v); }

// Request-major position of a workgroup: position idx of the concatenation of every request's
// items (cnt(r) items of request r, requests in order) -> request *r and item *q inside it; *r = -1
// past the last item.  Every wave computes the same answer (no LDS, no barrier); cnt is called for
// requests in runs of 64, one per lane.  lane: the caller's lane index (threadIdx.x & 63; a kernel
// that loops over items passes a copy the compiler cannot hoist, so the shuffle indices built from
// it are not kept live across the loop).
template <typename CountF>
__device__ __forceinline__ void locate_request(int idx, int n_req, CountF cnt, int* r, int* q, int lane) {
  int base = 0;
  for (int c0 = 0; c0 < n_req; c0 += 64) {
    const int rr = c0 + lane;
    const int c = rr < n_req ? cnt(rr) : 0;
    int x = c;   // inclusive prefix over the lanes
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = lane_value(x, lane - o);
      if (lane >= o) x += y;
    }
    const int tot = __builtin_amdgcn_readlane(x, 63);
    if (idx < base + tot) {
      const uint64_t m = __ballot(base + x > idx);
      const int l = __ffsll((unsigned long long)m) - 1;
      *r = c0 + l;
      *q = idx - (base + __builtin_amdgcn_readlane(x, l) - __builtin_amdgcn_readlane(c, l));
      return;
    }
    base += tot;
  }
  *r = -1;
  *q = 0;
}

// Largest and smallest v over the wave (lane as for locate_request).
__device__ __forceinline__ int wave_max_i(int v, int lane) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = max(v, lane_value(v, lane ^ o));
  return v;
}

__device__ __forceinline__ int wave_min_i(int v, int lane) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = min(v, lane_value(v, lane ^ o));
  return v;
}

// Number of values of the ascending list x[0, n) below v, by the whole wave: 64 probes of the list per
// round (two dependent loads for up to 4096 values, three for 262144; a binary search takes 12 and 18).
__device__ __forceinline__ int lower_bound_wave(const int32_t* x, int n, int v, int lane) {
  int lo = 0;   // x[lo - 1] < v <= x[lo + n]
  while (n > 0) {
    const int step = (n + 63) >> 6;
    const int i = (lane + 1) * step - 1;   // last of this lane's values
    const int below = __popcll(__ballot(i < n && x[lo + i] < v));
    lo += below * step;
    n = min(n - below * step, step - 1);
  }
  return lo;
}

typedef short shortx4_t __attribute__((ext_vector_type(4)));

// XOR applied to the 16-byte chunk index of row r of a V tile.  Each transposed read touches 4
// consecutive rows; this spreads their 32-byte (per 16 lanes) and 64-byte (per 32 lanes) pieces over
// distinct banks for both 128- and 256-byte-per-clock LDS service.  D = 64 rows have 8 chunks.
template <int NCH>
__device__ __forceinline__ int v_swz(int r) {
  return NCH >= 16 ? ((0xCA60 >> ((r & 3) * 4)) & 15) : ((0x4260 >> ((r & 3) * 4)) & 7);
}
typedef __attribute__((address_space(3))) shortx4_t lds_shortx4_t;

// Scheduling groups (instruction classes of the sched_group_barrier builtin): the next `n`
// instructions of class `mask` are placed here, in program order of the groups.
#define SX_SG(mask, n) __builtin_amdgcn_sched_group_barrier(mask, n, 0)
constexpr int kSgMfma = 0x8, kSgDsRead = 0x100;
// Order of a matrix phase of NM MFMAs whose operands come from NR LDS reads each: the reads of
// the first PRE MFMAs go first, then every MFMA is followed by the reads of the MFMA PRE places
// later, so each read has PRE MFMAs (32 cycles each) to complete.
template <int NM, int NR, int PRE>
__device__ __forceinline__ void sched_pipelined() {
  SX_SG(kSgDsRead, NR * PRE);
#pragma unroll
  for (int i = 0; i < NM - PRE; ++i) {
    SX_SG(kSgMfma, 1);
    SX_SG(kSgDsRead, NR);
  }
  SX_SG(kSgMfma, PRE);
}

// Grid of the kernels that tile one request's columns: x = KV head fastest, then kTilesX tiles; y = further
// tiles; z = request.  With the KV head fastest the round-robin dispatch over the 8 XCDs keeps a head's
// K and V in one L2 (8 heads) or a few.
constexpr int kTilesX = 64;

// Pool offset (elements) of (slot, head) in a [blocks][Hkv][16][D] pool.
__device__ __forceinline__ int64_t pool_off(int32_t slot, int head, int Hkv, int D) {
  return ((((int64_t)(slot >> 4)) * Hkv + head) * 16 + (slot & 15)) * (int64_t)D;
}

}  // namespace sx
