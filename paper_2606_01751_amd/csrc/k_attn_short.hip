// bfloat16 attention for launches with few query rows (short requests, small batches, the Sparse-Q rows of
// a short selecting layer), where the 256-column workgroups of k_attn.hip leave most of the chip idle and
// a workgroup walks all keys by itself.
//
// A workgroup of 4 waves takes 32 columns of one KV head (a column is a (row, query head) pair, row
// major, so any group size fills the tile) and splits the keys: pieces of 32 keys go to the waves in
// turn, each wave keeps its own online softmax, and the waves are merged through LDS in wave order.  The
// waves share nothing but the query columns, so the loop has no barrier: K and V pieces go to the wave's
// own LDS buffers (global -> LDS, whole rows; K read straight into operand registers, 32 bytes of each of
// 32 rows per instruction, cost the address unit three times as long), each refilled as soon as it is
// read, so a piece has half an iteration of this wave and all of the SIMD's other one to land.
#include <algorithm>

#include "sx_device.h"
#include "sx_internal.h"

namespace sx {
namespace {

constexpr int SW = 4;   // waves per workgroup
// Grid: x = KV head fastest, then kTilesX tiles; y = further tiles; z = request.  With the KV head
// fastest the round-robin dispatch over the 8 XCDs keeps a head's K and V in one L2 (8 heads) or a few.
constexpr int kTilesX = 64;

struct AttnS {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  uint16_t* out;
  float* lse;
  const ReqDev* reqs;
  const int32_t* bt;
  const int32_t* rows;
  const int32_t* n_rows;
  const int32_t* cu;
  int Hq, Hkv, G;
  uint32_t g_inv;  // ceil(2^32 / G): n / G = (n g_inv) >> 32 for the column counts that fit
  int grid_rows;   // paged: rows of a request beyond this bound are not processed
  float scale_log2;
  int lse_base2;
};

typedef short shortx4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4_t lds_shortx4_t;

// XOR of the 16-byte chunk index of row r of a V piece: spreads the 4 rows of a transposed read over
// distinct banks.
template <int NCH>
__device__ __forceinline__ int v_swz(int r) {
  return NCH >= 16 ? ((0xCA60 >> ((r & 3) * 4)) & 15) : ((0x4260 >> ((r & 3) * 4)) & 7);
}

// Order of NM MFMAs whose operands come from NR LDS reads each: the reads of the first PRE MFMAs go
// first, then every MFMA is followed by the reads of the MFMA PRE places later.
template <int NM, int NR, int PRE>
__device__ __forceinline__ void sched_pipelined() {
  constexpr int kMfma = 0x8, kDsRead = 0x100;   // sched_group_barrier instruction classes
  __builtin_amdgcn_sched_group_barrier(kDsRead, NR * PRE, 0);
#pragma unroll
  for (int i = 0; i < NM - PRE; ++i) {
    __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
    __builtin_amdgcn_sched_group_barrier(kDsRead, NR, 0);
  }
  __builtin_amdgcn_sched_group_barrier(kMfma, PRE, 0);
}

template <int D, bool PAGED, bool PV>
__global__ __launch_bounds__(SW * 64, 2) void attn_short_kernel(AttnS a) {
  constexpr int CT = 32;                    // columns
  constexpr int ROWB = D * 2;               // bytes of one key row
  constexpr int NCH = ROWB / 16;            // 16-byte chunks per row
  constexpr int NK = D / 16;                // K pieces (and MFMAs) per key tile
  constexpr int RPK = 1024 / ROWB;          // rows per 1 KB transfer
  constexpr int NT = 32 / RPK;              // transfers of a K or V piece
  constexpr int PB = 32 * ROWB;             // bytes of one
  constexpr int WB = (PV ? 2 : 1) * PB;     // a wave's pieces
  constexpr int NU = D / 8;                 // 4-value groups of a lane's O^T
  static_assert(!PV || WB == NU * 1024, "a wave's pieces are as large as its O^T in the merge");
  // [wave][K | V], rows row-major, 16-byte chunk c of row n at c ^ (n mod NCH) (K) or c ^ v_swz(n) (V)
  __shared__ __attribute__((aligned(1024))) char smem[SW * WB];
  __shared__ float ms[SW][CT], ls[SW][CT];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hg = lane >> 5;
  const int kvh = blockIdx.x % a.Hkv;
  const int tile = (int)(blockIdx.y * kTilesX + blockIdx.x / a.Hkv);
  const int r = blockIdx.z;
  int tok_off, bt_off = 0, nrows;
  if constexpr (PAGED) {
    const ReqDev rq = a.reqs[r];
    tok_off = rq.tok_off;
    bt_off = rq.bt_off;
    nrows = min(a.n_rows[r], a.grid_rows);
  } else {
    tok_off = a.cu[r];
    nrows = a.cu[r + 1] - tok_off;
  }
  const int ncols = nrows * a.G;
  const int ntiles = (ncols + CT - 1) / CT;
  if (tile >= ntiles) return;
  const int c0 = (ntiles - 1 - tile) * CT;   // the tiles with the most keys first
  // this lane's column (past the end: the last row's first head)
  const int c = c0 + l32;
  const bool valid = c < ncols;
  const int my_row = a.G == 1 ? min(c, ncols - 1) : (int)__umulhi((uint32_t)min(c, ncols - 1), a.g_inv);
  const int h = kvh * a.G + (valid ? c - my_row * a.G : 0);
  const int pos = PAGED ? a.rows[tok_off + my_row] : my_row;
  // Q^T as the B operand: lane owns column l32, d 16 s + 8 hg .. + 7
  bf16x8_t qb[NK];
  const uint16_t* qp = a.q + ((int64_t)(tok_off + pos) * a.Hq + h) * D + hg * 8;
#pragma unroll
  for (int s = 0; s < NK; ++s) qb[s] = *(const bf16x8_t*)(qp + 16 * s);
  // rows ascend: the last key that any column sees, and the last that every column sees
  const int cmax = __builtin_amdgcn_readlane(pos, 31), cmin = __builtin_amdgcn_readfirstlane(pos);
  const int np = cmax / 32 + 1;
  // 16-key block b of the request: element offset of its first row (uniform; the block id by a scalar
  // load).  Keys past the last visible one read that one's row (they are masked).
  const int bmax = cmax >> 4;
  auto blk_off = [&](int b) -> int64_t {
    b = min(b, bmax);
    if constexpr (PAGED) {
      const __attribute__((address_space(4))) int32_t* btc = (const __attribute__((address_space(4))) int32_t*)a.bt;
      return ((int64_t)btc[__builtin_amdgcn_readfirstlane(bt_off + b)] * a.Hkv + kvh) * 16 * D;
    } else {
      return ((int64_t)(tok_off + 16 * b) * a.Hkv + kvh) * D;
    }
  };
  const int rstep = PAGED ? D : a.Hkv * D;   // elements between the rows of a block
  auto row_off = [&](int b, int i) { return (min(16 * b + i, cmax) - 16 * min(b, bmax)) * rstep; };
  // transfers of the K or V piece t into this wave's buffer: 1 KB is RPK whole rows
  const uint32_t kb = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + (uint32_t)(w * WB);
  const uint32_t vb = kb + (uint32_t)PB;
  const int trow = lane / NCH, tch = lane % NCH;
  auto issue = [&](const uint16_t* base, int t, const int64_t (&bo)[2], uint32_t dst, bool is_v) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int row = RPK * i + trow;
      const int ch = tch ^ (is_v ? v_swz<NCH>(row) : (row & (NCH - 1)));
      const uint16_t* p = base + bo[RPK * i / 16] + row_off(2 * t + RPK * i / 16, row & 15) + ch * 8;
      const uint32_t m0 = __builtin_amdgcn_readfirstlane(dst + (uint32_t)(i * 1024));
      asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p), "s"(m0) : "m0", "memory");
    }
  };
  uint32_t ko[NK];   // K operand: lane reads row l32, chunk 2 s + hg
#pragma unroll
  for (int s = 0; s < NK; ++s) ko[s] = kb + (uint32_t)(l32 * ROWB + (((2 * s + hg) ^ (l32 & (NCH - 1))) << 4));
  // V^T operand: lane 4 tk + tc of each 16-lane group points at row tk, dims 4 tc .. + 3 of its slice
  const int tg = lane >> 4, tk = (lane & 15) >> 2, tc = lane & 3;
  uint32_t vtr[PV ? D / 32 : 1];
#pragma unroll
  for (int dt = 0; dt < (PV ? D / 32 : 1); ++dt) {
    const int dchunk = 4 * dt + 2 * (tg & 1) + (tc >> 1);
    vtr[dt] = vb + (uint32_t)((4 * (tg >> 1) + tk) * ROWB + ((dchunk ^ v_swz<NCH>(tk)) << 4) + (tc & 1) * 8);
  }
  float m = -INFINITY, l = 0.f;
  f32x16_t o[PV ? D / 32 : 1];
#pragma unroll
  for (int dt = 0; dt < (PV ? D / 32 : 1); ++dt) o[dt] = f32x16_t{};
  // Q has landed before the first transfer, whose waits count transfers only
#pragma unroll
  for (int s = 0; s < NK; ++s) asm volatile("" : "+v"(qb[s]));
  int64_t bo[2] = {blk_off(2 * w), blk_off(2 * w + 1)};   // blocks of the wave's piece
  if (w < np) {
    issue(a.k, w, bo, kb, false);
    if constexpr (PV) issue(a.v, w, bo, vb, true);
  }
  for (int t = w; t < np; t += SW) {
    const int kbase = t * 32;
    const bool more = t + SW < np;
    const int64_t bn[2] = {blk_off(2 * (t + SW)), blk_off(2 * (t + SW) + 1)};   // of its next one
    // K has landed (this piece's V is younger)
    if constexpr (PV) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NT) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    f32x16_t sacc = f32x16_t{};
#pragma unroll
    for (int s = 0; s < NK; ++s) {
      const bf16x8_t ka = *(const __attribute__((address_space(3))) bf16x8_t*)(uintptr_t)ko[s];
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb[s], sacc, 0, 0, 0);
    }
    sched_pipelined<NK, 1, 4>();
    // its buffer takes the next piece's K
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (more) issue(a.k, t + SW, bn, kb, false);
    // online softmax in the log2 domain: lane value e is key kbase + 8 (e / 4) + 4 hg + e % 4
    bf16x8_t pb[2];
    if (kbase + 31 > cmin) {
      const int lim = pos - kbase - hg * 4;
#pragma unroll
      for (int e = 0; e < 16; ++e) sacc[e] = (e >> 2) * 8 + (e & 3) > lim ? -INFINITY : sacc[e];
    }
    float mx = sacc[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sacc[e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * a.scale_log2;   // (the scale is positive)
    const float mn = fmaxf(m, mx);
    if (__ballot(mn > m)) {
      const float f = mn == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - mn);
      l *= f;
      if constexpr (PV) {
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
          for (int e = 0; e < 16; ++e) o[dt][e] *= f;
      }
      m = mn;
    }
    const float mneg = m == -INFINITY ? 0.f : -m;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      float p[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[8 * kk + e], a.scale_log2, mneg));
        l += p[e];
      }
      if constexpr (PV)
        pb[kk] = __builtin_bit_cast(bf16x8_t, make_uint4(pack_bf16x2(p[0], p[1]), pack_bf16x2(p[2], p[3]),
                                                         pack_bf16x2(p[4], p[5]), pack_bf16x2(p[6], p[7])));
    }
    if constexpr (PV) {
      // V has landed (the next K is younger)
      if (more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NT) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) {
          uint2 h2[2];
#pragma unroll
          for (int i = 0; i < 2; ++i)   // slots 8 hg + 4 i + x <-> key 16 kk + 8 i + 4 hg + x
            h2[i] = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_t*)(uintptr_t)(
                                                  vtr[dt] + (uint32_t)((16 * kk + 8 * i) * ROWB))));
          const bf16x8_t va = __builtin_bit_cast(bf16x8_t, make_uint4(h2[0].x, h2[0].y, h2[1].x, h2[1].y));
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[kk], o[dt], 0, 0, 0);
        }
      sched_pipelined<D / 16, 2, 4>();
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (more) issue(a.v, t + SW, bn, vb, true);
    }
    bo[0] = bn[0];
    bo[1] = bn[1];
  }
  // ---- merge: every wave leaves its O^T (in place of its pieces), maximum and sum in LDS and adds up
  // its share of the O^T of the waves that had a piece, in wave order ----
  const int na = min(np, SW);
  l += __shfl_xor(l, 32, 64);
  if (hg == 0) {
    ms[w][l32] = m;
    ls[w][l32] = l;
  }
  f32x4_t* const red = (f32x4_t*)smem;
  if constexpr (PV) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const f32x16_t& x = o[u / 4];
      red[(w * NU + u) * 64 + lane] = f32x4_t{x[4 * (u % 4)], x[4 * (u % 4) + 1], x[4 * (u % 4) + 2], x[4 * (u % 4) + 3]};
    }
  }
  __syncthreads();
  float M = -INFINITY, L = 0.f, f[SW];
#pragma unroll
  for (int i = 0; i < SW; ++i) M = fmaxf(M, ms[i][l32]);
#pragma unroll
  for (int i = 0; i < SW; ++i) {
    const float mi = ms[i][l32];
    f[i] = mi == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(mi - M);
    L += ls[i][l32] * f[i];
  }
  if constexpr (PV) {
    if (valid) {
      const float inv = 1.f / L;
      uint16_t* op = a.out + ((int64_t)(tok_off + my_row) * a.Hq + h) * D;
#pragma unroll
      for (int x = 0; x < NU / SW; ++x) {
        const int u = w * (NU / SW) + x;
        f32x4_t y = red[u * 64 + lane] * f[0];
#pragma unroll
        for (int i = 1; i < SW; ++i)
          if (i < na) y += red[(i * NU + u) * 64 + lane] * f[i];
        uint2 t;
        t.x = pack_bf16x2(y[0] * inv, y[1] * inv);
        t.y = pack_bf16x2(y[2] * inv, y[3] * inv);
        *(uint2*)(op + (u / 4) * 32 + (u % 4) * 8 + hg * 4) = t;
      }
    }
  }
  if (a.lse && w == 0 && hg == 0 && valid) {
    const float lse2 = M + __log2f(L);
    a.lse[(int64_t)(tok_off + my_row) * a.Hq + h] = a.lse_base2 ? lse2 : lse2 * 0.69314718055994531f;
  }
}

template <int D>
hipError_t launch_d(const AttnLaunch& L, bool paged, hipStream_t s) {
  AttnS a{};
  a.q = (const uint16_t*)L.q;
  a.k = (const uint16_t*)L.k;
  a.v = (const uint16_t*)L.v;
  a.out = (uint16_t*)L.out;
  a.lse = L.lse;
  a.reqs = L.reqs;
  a.bt = L.bt;
  a.rows = L.rows;
  a.n_rows = L.n_rows;
  a.cu = L.cu;
  a.Hq = L.Hq;
  a.Hkv = L.Hkv;
  a.G = L.Hq / L.Hkv;
  a.grid_rows = L.grid_rows;
  a.scale_log2 = L.scale * 1.4426950408889634f;
  a.lse_base2 = L.lse_base2;
  a.g_inv = (uint32_t)((((uint64_t)1 << 32) + a.G - 1) / a.G);
  const int64_t tiles = ((int64_t)L.grid_rows * a.G + 31) / 32;
  const dim3 grid((unsigned)(L.Hkv * std::min<int64_t>(tiles, kTilesX)), (unsigned)((tiles + kTilesX - 1) / kTilesX),
                  (unsigned)L.n_req);
  if (!paged) hipLaunchKernelGGL((attn_short_kernel<D, false, true>), grid, dim3(SW * 64), 0, s, a);
  else if (L.out) hipLaunchKernelGGL((attn_short_kernel<D, true, true>), grid, dim3(SW * 64), 0, s, a);
  else hipLaunchKernelGGL((attn_short_kernel<D, true, false>), grid, dim3(SW * 64), 0, s, a);
  return hipGetLastError();
}

}  // namespace

// Whether the launch goes here.  The 256-column grid runs at most one workgroup per compute unit up to
// 256 items (row tile x KV head x request), so it takes as long as its longest item, 9 us and 26 ns per
// key; this kernel's time is the K / V bytes that its tiles read, about 0.14 ns per item and key (d = 128)
// for a causal request, half at d = 64.  They meet at about 140 items, more where the 9 us weigh in.
// Measured (whole layer calls, 256-column / this): 56 items of 777 keys 35 / 20 us, 104 of 800 31 / 23.6,
// 126 of 4000 91 / 75, 150 of 3000 80 / 76; 200 of 1600 49 / 55, 240 of 5000 120 / 155 us.  The
// log-sum-exp pass of the 256-column kernel splits the keys too and reads K only, so it is left earlier:
// 32 items of 1000 keys 67 / 52, 96 of 3000 112 / 113, 256 of 8192 279 / 318 us.
bool attn_short_fits(const AttnLaunch& L) {
  const int rpw = 256 / (L.Hq / L.Hkv);
  const int64_t items = (int64_t)(L.grid_rows + rpw - 1) / rpw * L.Hkv * L.n_req * L.D / 128;
  return items <= (L.out ? 140 : 20) + 80000 / std::max(1, L.max_keys);
}

hipError_t launch_attn_short(const AttnLaunch& L, bool paged, hipStream_t s) {
  return L.D == 128 ? launch_d<128>(L, paged, s) : launch_d<64>(L, paged, s);
}

}  // namespace sx
