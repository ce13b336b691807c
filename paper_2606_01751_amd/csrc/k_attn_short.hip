// bfloat16 attention for launches with few query rows (short requests, small batches, the Sparse-Q rows of
// a short selecting layer), where the 256-column workgroups of k_attn.hip leave most of the chip idle and
// a workgroup walks all keys by itself.
//
//   attn_short_kernel  attention with output, the same arithmetic as k_attn.hip's, column by column: which of
//                      the two runs is chosen by the size of the whole launch, and must not show in a result
//   lse_short_kernel   the log-sum-exp pass of the probe rows (no output to keep alike: that pass splits
//                      its keys by the size of the launch in k_attn.hip too)
//
// Both take 32 columns of one KV head per workgroup (a column is a (row, query head) pair, row major) and
// move K and V through LDS (global -> LDS, whole rows; K read straight into operand registers, 32 bytes of
// each of 32 rows per instruction, cost the address unit three times as long).
#include <algorithm>
#include <type_traits>

#include "sx_device.h"
#include "sx_internal.h"

namespace sx {
namespace {

constexpr int COLS = 256;   // columns of a row tile of k_attn.hip
constexpr int SW = 4;       // waves per workgroup of the log-sum-exp pass

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
  int grid_rows;   // paged: rows of a request beyond this bound are not processed
  float scale_log2;
  int lse_base2;
};

// Attention of 32 columns, formed as a wave of attn_mfma_kernel forms them (the same 32 columns of a row tile of
// 256 / G rows, 64-key tiles in order, the running maximum raised for the whole wave when a probability would
// reach 2^64, the same sums in the same order), with the work of NW / 2 key tiles at a time spread over NW
// waves: wave w forms S and the probabilities of 32 of the round's 32 NW keys, passes P^T on through LDS, and
// adds P.V of the whole round to 32 dims of O^T (waves past D / 32 rest then).  Only the sum of a tile's
// probabilities is serial: its second half goes on from the first half's.
// Bound by a column's chain of rounds while few workgroups run (1.5 us per 128 keys with 4 waves: S 0.2,
// transfers into LDS 0.2 and 0.25 (22 cycles per 1 KB and compute unit), probabilities 0.35, P.V 0.25, the rest
// barriers and the LDS trips behind them), by those transfers, K and V whole for every 32 columns, once the
// chip is full: hence three widths (see the dispatch).  Two buffers for K and V and transfers placed between
// the MFMAs and exponentials were no faster.  Measured (whole calls, this / the 256-column grid / four waves that
// split the keys and merge, whose sums were others): 777 tokens, 388 rows of 32/8/128 15.9 / 28.3 / 14.8 us,
// 777 rows 19.5 / 29.6 / 21.2, 1200 rows of 6000 tokens of 8/2/128 57 / 124 / 62, six requests of 250 tokens
// 21 / 29 / 22.
template <int D, bool PAGED, int NW>
__global__ __launch_bounds__(NW * 64, 2) void attn_short_kernel(AttnS a) {
  constexpr int KR = 32 * NW;               // keys per round
  constexpr int TR = KR / 64;               // key tiles per round
  constexpr int ROWB = D * 2;               // bytes of one key row
  constexpr int NCH = ROWB / 16;            // 16-byte chunks per row
  constexpr int NK = D / 16;                // k-slices (and MFMAs) of S
  constexpr int RPK = 1024 / ROWB;          // rows per 1 KB transfer
  constexpr int NT = 32 / RPK;              // transfers of a wave's 32 rows of K or V
  constexpr int PB = 32 * ROWB;             // bytes of them
  constexpr int BB = NW * PB;               // bytes of a round's K or V
  // K [wave][32 rows], V [KR rows] (16-byte chunk c of row n at c ^ (n mod NCH) (K) or
  // c ^ v_swz(n) (V)), P^T operands [tile][kk][lane]
  __shared__ __attribute__((aligned(1024))) char smem[2 * BB + TR * 4096];
  __shared__ float s_half[TR][64];          // sum of the first 32 keys of a tile
  __shared__ float s_sum[TR][64];           // sum of a tile
  __shared__ float s_max[NW][32];
  __shared__ int s_flag[NW];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hg = lane >> 5;
  const int kvh = blockIdx.x % a.Hkv;
  const int idx = (int)(blockIdx.y * kTilesX + blockIdx.x / a.Hkv);
  const int r = blockIdx.z;
  int T, tok_off, bt_off = 0, nrows;
  if constexpr (PAGED) {
    const ReqDev rq = a.reqs[r];
    T = rq.T;
    tok_off = rq.tok_off;
    bt_off = rq.bt_off;
    nrows = min(a.n_rows[r], a.grid_rows);
  } else {
    tok_off = a.cu[r];
    T = nrows = a.cu[r + 1] - tok_off;
  }
  if (nrows <= 0) return;
  // groups of 32 columns, those of the last row tile only as far as it has rows; most keys first
  const int rpw = COLS / a.G, gpt = (rpw * a.G + 31) / 32;
  const int full = (nrows - 1) / rpw;
  const int groups = full * gpt + ((nrows - full * rpw) * a.G + 31) / 32;
  if (idx >= groups) return;
  const int grp = groups - 1 - idx, row_tile = grp / gpt;
  const int col = (grp - row_tile * gpt) * 32 + l32;
  const int lrow = col / a.G;
  const int ridx = row_tile * rpw + lrow;
  const bool valid = lrow < rpw && ridx < nrows;
  const int h = kvh * a.G + col - lrow * a.G;
  int pos = -1;
  if (valid) pos = PAGED ? a.rows[tok_off + ridx] : ridx;
  // Q^T as the B operand: lane owns column l32, d 16 s + 8 hg .. + 7
  bf16x8_t qb[NK];
  const uint16_t* qp = a.q + ((int64_t)(tok_off + max(pos, 0)) * a.Hq + (valid ? h : 0)) * D + hg * 8;
#pragma unroll
  for (int s = 0; s < NK; ++s)
    qb[s] = __builtin_bit_cast(bf16x8_t, valid ? *(const uint4*)(qp + 16 * s) : make_uint4(0, 0, 0, 0));
  const int wave_max = __builtin_amdgcn_readfirstlane(wave_max_i(pos, lane));
  const int wave_min = __builtin_amdgcn_readfirstlane(wave_min_i(valid ? pos : 0x7fffffff, lane));
  const int nkt = wave_max / 64 + 1;   // key tiles
  const float c2 = a.scale_log2;

  // ---- transfers: 1 KB is RPK whole rows; keys past the request's end read row T - 1 (they are masked) ----
  const int last_key = T - 1, bmax = last_key >> 4;
  const int64_t rstride = PAGED ? D : (int64_t)a.Hkv * D;   // elements between the rows of a block
  // element offset of the first row of block b of the request (uniform; the block id by a scalar load)
  auto blk_off = [&](int b) -> int64_t {
    b = min(b, bmax);
    if constexpr (PAGED) {
      const __attribute__((address_space(4))) int32_t* btc = (const __attribute__((address_space(4))) int32_t*)a.bt;
      return ((int64_t)btc[__builtin_amdgcn_readfirstlane(bt_off + b)] * a.Hkv + kvh) * 16 * D;
    } else {
      return ((int64_t)(tok_off + 16 * b) * a.Hkv + kvh) * D;
    }
  };
  const int trow = lane / NCH, tch = lane % NCH;
  // byte offsets of the transfers of a 16-key block (those of its two blocks are alike)
  uint32_t off_k[NT / 2], off_v[NT / 2];
#pragma unroll
  for (int i = 0; i < NT / 2; ++i) {
    const int row = RPK * i + trow;
    off_k[i] = (uint32_t)((row * rstride + (tch ^ (row & (NCH - 1))) * 8) * 2);
    off_v[i] = (uint32_t)((row * rstride + (tch ^ v_swz<NCH>(row)) * 8) * 2);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const uint32_t kb = lds0 + (uint32_t)(w * PB), vb0 = lds0 + (uint32_t)(BB);
  const uint32_t vb = vb0 + (uint32_t)(w * PB);
  // this wave's 32 rows of K or V from `key` on; bo: blk_off of their two blocks
  auto issue = [&](const uint16_t* base, int key, const int64_t (&bo)[2], uint32_t dst, bool is_v) {
    if (key + 31 <= last_key) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const uint64_t sb = (uint64_t)(uintptr_t)(base + bo[b]);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)sb);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(sb >> 32));
        const uint64_t sbu = ((uint64_t)hi << 32) | (uint64_t)lo;
#pragma unroll
        for (int i = 0; i < NT / 2; ++i) {
          const uint32_t m0 = __builtin_amdgcn_readfirstlane(dst + (uint32_t)((b * NT / 2 + i) * 1024));
          asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(is_v ? off_v[i] : off_k[i]), "s"(sbu),
                       "s"(m0)
                       : "m0", "memory");
        }
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int row = RPK * i + trow;
      const int b = min((key >> 4) + RPK * i / 16, bmax);
      const int ch = tch ^ (is_v ? v_swz<NCH>(row) : (row & (NCH - 1)));
      const uint16_t* p = base + bo[RPK * i / 16] + (min(key + row, last_key) - 16 * b) * rstride + ch * 8;
      const uint32_t m0 = __builtin_amdgcn_readfirstlane(dst + (uint32_t)(i * 1024));
      asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p), "s"(m0) : "m0", "memory");
    }
  };

  uint32_t ko[NK];   // K operand: lane reads row l32, chunk 2 s + hg
#pragma unroll
  for (int s = 0; s < NK; ++s) ko[s] = kb + (uint32_t)(l32 * ROWB + (((2 * s + hg) ^ (l32 & (NCH - 1))) << 4));
  // V^T operand of this wave's 32 dims: lane 4 tk + tc of each 16-lane group points at row tk, dims 4 tc .. + 3
  // of its slice
  const int tg = lane >> 4, tk = (lane & 15) >> 2, tc = lane & 3;
  const int dt = w % (D / 32);
  const int dchunk = 4 * dt + 2 * (tg & 1) + (tc >> 1);
  const uint32_t vtr = vb0 + (uint32_t)((4 * (tg >> 1) + tk) * ROWB + ((dchunk ^ v_swz<NCH>(tk)) << 4) + (tc & 1) * 8);
  const uint32_t pt = vb0 + (uint32_t)(BB + lane * 16);   // P^T operands of this lane
  const int ti = w >> 1, mt = w & 1;                           // this wave's key tile of the round, and half of it

  float m = valid ? -INFINITY : 0.f, l = 0.f;
  f32x16_t o = f32x16_t{}, sacc;
  float x[16], ps;
  // probabilities 2^(c2 s + mneg) of this wave's keys (lane value e is key 8 (e / 4) + 4 hg + e % 4) and their sum
  auto expo = [&](float mneg) {
    ps = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      x[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[e], c2, mneg));
      ps += x[e];
    }
    if (mt == 0) s_half[ti][lane] = ps;
  };
  auto put_p = [&]() {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const float* y = x + 8 * kk;
      *(__attribute__((address_space(3))) bf16x8_t*)(uintptr_t)(pt + (uint32_t)(ti * 4096 + (2 * mt + kk) * 1024)) =
          __builtin_bit_cast(bf16x8_t, make_uint4(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]),
                                                  pack_bf16x2(y[6], y[7])));
    }
  };
  auto put_max = [&]() {
    float mx = sacc[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sacc[e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (hg == 0) s_max[w][l32] = mx;
  };
  // the running maximum raised to that of tile t of the round; returns the factor of what is summed so far
  auto raise = [&](int t) -> float {
    const float mn = fmaxf(m, fmaxf(s_max[2 * t][l32], s_max[2 * t + 1][l32]) * c2);
    const float f = mn == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - mn);
    m = mn;
    return f;
  };

  // Q has landed before the first transfer, whose waits count transfers only
#pragma unroll
  for (int s = 0; s < NK; ++s) asm volatile("" : "+v"(qb[s]));
  if (ti < nkt) {
    const int64_t bo[2] = {blk_off(2 * w), blk_off(2 * w + 1)};
    issue(a.k, 32 * w, bo, kb, false);
    issue(a.v, 32 * w, bo, vb, true);
  }
  for (int t0 = 0; t0 < nkt; t0 += TR) {   // round of tiles t0 .. t0 + TR - 1
    const int key = 64 * t0 + 32 * w;      // this wave's first
    const bool live = t0 + ti < nkt, more = t0 + TR + ti < nkt;   // whether it has any, in this round and the next
    // blocks of its next keys, whose ids are on their way while this round is computed
    const int64_t bo[2] = {blk_off((key + KR) >> 4), blk_off(((key + KR) >> 4) + 1)};
    if (live) {
      // K has landed (this round's V is younger)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NT) : "memory");
      sacc = f32x16_t{};
#pragma unroll
      for (int s = 0; s < NK; ++s) {
        const bf16x8_t ka = *(const __attribute__((address_space(3))) bf16x8_t*)(uintptr_t)ko[s];
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb[s], sacc, 0, 0, 0);
      }
      sched_pipelined<NK, 1, 4>();
      // its buffer takes the next round's K
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (more) issue(a.k, key + KR, bo, kb, false);
      if (key + 31 > wave_min) {
        const int lim = pos - key - hg * 4;
#pragma unroll
        for (int e = 0; e < 16; ++e) sacc[e] = (e >> 2) * 8 + (e & 3) > lim ? -INFINITY : sacc[e];
      }
    }
    // the first tile always raises the maximum (from -inf: nothing is summed yet)
    if (t0 == 0) {
      if (ti == 0) put_max();
      __syncthreads();
      (void)raise(0);
    }
    int flag = 0;
    if (live) {
      const bool first = t0 + ti == 0;
      expo(first && m == -INFINITY ? 0.f : -m);
      put_p();
      // a tile whose halves both stay below 2^62 stays below 2^64
      flag = !first && __ballot(!(ps < 0x1p62f)) != 0;
      // V has landed (the next K is younger)
      if (more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NT) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    if (lane == 0) s_flag[w] = flag;
    __syncthreads();
    bool grow = false;
#pragma unroll
    for (int i = 0; i < NW; ++i) grow |= s_flag[i] != 0;
    float f[TR];
#pragma unroll
    for (int t = 0; t < TR; ++t) f[t] = 1.f;
    if (grow) {   // (rare, and the same in every wave: tile by tile, as one wave would)
#pragma unroll
      for (int t = 0; t < TR; ++t) {
        if (t0 + t == 0 || t0 + t >= nkt) continue;
        __syncthreads();
        if (ti == t) {
          expo(-m);
          put_max();
        }
        __syncthreads();
        if (ti == t && mt == 1) {
          float sum = s_half[t][lane];
#pragma unroll
          for (int e = 0; e < 16; ++e) sum += x[e];
          const int over = __ballot(!(sum < 0x1p64f)) != 0;
          if (lane == 0) s_flag[w] = over;
        }
        __syncthreads();
        if (s_flag[2 * t + 1]) {
          f[t] = raise(t);
          if (ti == t) expo(m == -INFINITY ? 0.f : -m);
        }
      }
      if (live) put_p();
      __syncthreads();
    }
    if (live && mt == 1) {
      float sum = s_half[ti][lane];
#pragma unroll
      for (int e = 0; e < 16; ++e) sum += x[e];
      s_sum[ti][lane] = sum;
    }
    // O^T += V^T P^T of the round's tiles
#pragma unroll
    for (int t = 0; t < TR; ++t) {
      if (t0 + t >= nkt || w >= D / 32) break;
      if (grow) {
#pragma unroll
        for (int e = 0; e < 16; ++e) o[e] *= f[t];
      }
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const bf16x8_t pb = *(const __attribute__((address_space(3))) bf16x8_t*)(uintptr_t)(pt + (uint32_t)(t * 4096 + kk * 1024));
        uint2 h2[2];
#pragma unroll
        for (int i = 0; i < 2; ++i)   // slots 8 hg + 4 i + x <-> key 16 kk + 8 i + 4 hg + x
          h2[i] = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_t*)(uintptr_t)(
                                                vtr + (uint32_t)((64 * t + 16 * kk + 8 * i) * ROWB))));
        const bf16x8_t va = __builtin_bit_cast(bf16x8_t, make_uint4(h2[0].x, h2[0].y, h2[1].x, h2[1].y));
        o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb, o, 0, 0, 0);
      }
    }
    // V and P^T are read: their buffers take the next round's
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (more) issue(a.v, key + KR, bo, vb, true);
#pragma unroll
    for (int t = 0; t < TR; ++t) {
      if (t0 + t >= nkt) break;
      if (grow) {
        l *= f[t];
        asm volatile("" : "+v"(l));   // (the product is rounded before the sum)
      }
      l += s_sum[t][lane];
    }
  }

  l += __shfl_xor(l, 32, 64);
  if (!valid || w >= D / 32) return;
  const float inv = 1.f / l;
  uint16_t* op = a.out + ((int64_t)(tok_off + ridx) * a.Hq + h) * D + 32 * w + hg * 4;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint2 t;
    t.x = pack_bf16x2(o[4 * j] * inv, o[4 * j + 1] * inv);
    t.y = pack_bf16x2(o[4 * j + 2] * inv, o[4 * j + 3] * inv);
    *(uint2*)(op + 8 * j) = t;
  }
  if (a.lse && w == 0 && hg == 0) {
    const float lse2 = m + __log2f(l);
    a.lse[(int64_t)(tok_off + ridx) * a.Hq + h] = a.lse_base2 ? lse2 : lse2 * 0.69314718055994531f;
  }
}

// Log-sum-exp of 32 columns (paged): 4 waves take the keys in pieces of 32 in turn, each with its own online
// sum, merged through LDS in wave order.  The waves share nothing but the columns, so the loop has no barrier: K
// pieces go to the wave's own LDS buffer, refilled as soon as it is read.
template <int D>
__global__ __launch_bounds__(SW * 64, 2) void lse_short_kernel(AttnS a) {
  constexpr int CT = 32;                    // columns
  constexpr int ROWB = D * 2;               // bytes of one key row
  constexpr int NCH = ROWB / 16;            // 16-byte chunks per row
  constexpr int NK = D / 16;                // k-slices (and MFMAs) of S
  constexpr int RPK = 1024 / ROWB;          // rows per 1 KB transfer
  constexpr int NT = 32 / RPK;              // transfers of a piece
  constexpr int PB = 32 * ROWB;             // bytes of one
  __shared__ __attribute__((aligned(1024))) char smem[SW * PB];   // chunk c of row n at c ^ (n mod NCH)
  __shared__ float ms[SW][CT], ls[SW][CT];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hg = lane >> 5;
  const int kvh = blockIdx.x % a.Hkv;
  const int tile = (int)(blockIdx.y * kTilesX + blockIdx.x / a.Hkv);
  const ReqDev rq = a.reqs[blockIdx.z];
  const int tok_off = rq.tok_off, bt_off = rq.bt_off;
  const int ncols = min(a.n_rows[blockIdx.z], a.grid_rows) * a.G;
  const int ntiles = (ncols + CT - 1) / CT;
  if (tile >= ntiles) return;
  const int c0 = (ntiles - 1 - tile) * CT;   // the tiles with the most keys first
  // this lane's column (past the end: the last row's first head)
  const int c = c0 + l32;
  const bool valid = c < ncols;
  const int my_row = min(c, ncols - 1) / a.G;
  const int h = kvh * a.G + (valid ? c - my_row * a.G : 0);
  const int pos = a.rows[tok_off + my_row];
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
    const __attribute__((address_space(4))) int32_t* btc = (const __attribute__((address_space(4))) int32_t*)a.bt;
    return ((int64_t)btc[__builtin_amdgcn_readfirstlane(bt_off + min(b, bmax))] * a.Hkv + kvh) * 16 * D;
  };
  auto row_off = [&](int b, int i) { return (min(16 * b + i, cmax) - 16 * min(b, bmax)) * D; };
  // transfers of the K piece t into this wave's buffer: 1 KB is RPK whole rows
  const uint32_t kb = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + (uint32_t)(w * PB);
  const int trow = lane / NCH, tch = lane % NCH;
  auto issue = [&](int t, const int64_t (&bo)[2]) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int row = RPK * i + trow;
      const uint16_t* p = a.k + bo[RPK * i / 16] + row_off(2 * t + RPK * i / 16, row & 15) + (tch ^ (row & (NCH - 1))) * 8;
      const uint32_t m0 = __builtin_amdgcn_readfirstlane(kb + (uint32_t)(i * 1024));
      asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(p), "s"(m0) : "m0", "memory");
    }
  };
  uint32_t ko[NK];   // K operand: lane reads row l32, chunk 2 s + hg
#pragma unroll
  for (int s = 0; s < NK; ++s) ko[s] = kb + (uint32_t)(l32 * ROWB + (((2 * s + hg) ^ (l32 & (NCH - 1))) << 4));
  float m = -INFINITY, l = 0.f;
  // Q has landed before the first transfer, whose waits count transfers only
#pragma unroll
  for (int s = 0; s < NK; ++s) asm volatile("" : "+v"(qb[s]));
  int64_t bo[2] = {blk_off(2 * w), blk_off(2 * w + 1)};   // blocks of the wave's piece
  if (w < np) issue(w, bo);
  for (int t = w; t < np; t += SW) {
    const int kbase = t * 32;
    const int64_t bn[2] = {blk_off(2 * (t + SW)), blk_off(2 * (t + SW) + 1)};   // of its next one
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    f32x16_t sacc = f32x16_t{};
#pragma unroll
    for (int s = 0; s < NK; ++s) {
      const bf16x8_t ka = *(const __attribute__((address_space(3))) bf16x8_t*)(uintptr_t)ko[s];
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qb[s], sacc, 0, 0, 0);
    }
    sched_pipelined<NK, 1, 4>();
    // its buffer takes the next piece's K
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (t + SW < np) issue(t + SW, bn);
    // online softmax in the log2 domain: lane value e is key kbase + 8 (e / 4) + 4 hg + e % 4
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
      l *= mn == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - mn);
      m = mn;
    }
    const float mneg = m == -INFINITY ? 0.f : -m;
#pragma unroll
    for (int e = 0; e < 16; ++e) l += __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[e], a.scale_log2, mneg));
    bo[0] = bn[0];
    bo[1] = bn[1];
  }
  l += __shfl_xor(l, 32, 64);
  if (hg == 0) {
    ms[w][l32] = m;
    ls[w][l32] = l;
  }
  __syncthreads();
  float M = -INFINITY, L = 0.f;
#pragma unroll
  for (int i = 0; i < SW; ++i) M = fmaxf(M, ms[i][l32]);
#pragma unroll
  for (int i = 0; i < SW; ++i) L += ms[i][l32] == -INFINITY ? ls[i][l32] : ls[i][l32] * __builtin_amdgcn_exp2f(ms[i][l32] - M);
  if (w == 0 && hg == 0 && valid) {
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
  // groups of 32 columns of one request and KV head
  const int rpw = COLS / a.G, gpt = (rpw * a.G + 31) / 32;
  const int64_t tiles = L.out ? (int64_t)(L.grid_rows / rpw) * gpt + ((int64_t)(L.grid_rows % rpw) * a.G + 31) / 32
                              : ((int64_t)L.grid_rows * a.G + 31) / 32;
  const dim3 grid((unsigned)(L.Hkv * std::min<int64_t>(tiles, kTilesX)), (unsigned)((tiles + kTilesX - 1) / kTilesX),
                  (unsigned)L.n_req);
  if (!L.out) {
    hipLaunchKernelGGL(lse_short_kernel<D>, grid, dim3(SW * 64), 0, s, a);
    return hipGetLastError();
  }
  // Waves: the more, the fewer rounds a column takes, and the fewer columns a compute unit carries (LDS: one
  // workgroup of 8, two of 4 at d = 128 and three at 64, seven of 2), so 8 up to 1.5 groups per compute unit and
  // 4 beyond; d = 64, where only 2 waves have P.V, 2 from four groups per compute unit.  Measured, 8 / 4 waves:
  // 8/2/128, 300 groups of 6000 tokens 57 / 73 us, 376 of 1500 19.4 / 23.8, 392 of 777 16.4 / 17.7; 480 of 800
  // 21.8 / 16.5, 600 of 3000 (32/8) 47.5 / 43.0; 8/8/64, 384 of 3000 25.4 / 32.8, 600 (16/4) 38 / 34; 16/4/64, 4 / 2
  // waves: 684 of 1500 24.0 / 27.9, 784 of 777 14.8 / 17.2, 960 of 800 18.4 / 17.9, 1216 of 300 15.7 / 11.9.
  const int64_t groups = tiles * L.Hkv * L.n_req, n_cu = std::max(1, L.n_cu);
  const int nw = 2 * groups <= 3 * n_cu ? 8 : D == 64 && groups > 4 * n_cu ? 2 : 4;
  auto go = [&](auto waves) {
    constexpr int NW = decltype(waves)::value;
    if (paged) hipLaunchKernelGGL((attn_short_kernel<D, true, NW>), grid, dim3(NW * 64), 0, s, a);
    else hipLaunchKernelGGL((attn_short_kernel<D, false, NW>), grid, dim3(NW * 64), 0, s, a);
  };
  if (nw == 8) go(std::integral_constant<int, 8>{});
  else if (nw == 4) go(std::integral_constant<int, 4>{});
  else if constexpr (D == 64) go(std::integral_constant<int, 2>{});
  return hipGetLastError();
}

}  // namespace

// Whether the launch goes here.  The 256-column grid runs at most one workgroup per compute unit up to
// 256 items (row tile x KV head x request), so it takes as long as its longest item, 9 us and 26 ns per
// key (d = 64: 7 and 17); attn_short_kernel's time is the K / V bytes that its tiles read, about 0.14 ns per
// item and key (d = 128) for a causal request.  They meet at about 140 items, more where the 9 us weigh in
// and where the requests are of unequal lengths (the bound counts every one as the longest); at d = 64 at about
// 180.  Measured (calls, 256-column / this): 56 items of 777 keys 28.3 / 15.9 us, 104 of 777 29.6 / 19.5, 152 of
// 3000 70 / 64, 152 of 6000 125 / 114; 192 of 1500 43 / 46, 240 of 800 35 / 43; d = 64: 192 of 3000 63 / 61, 152 of
// 6000 110 / 92, 304 of 6000 114 / 135.  The log-sum-exp pass of the 256-column kernel splits the keys too
// and reads K only, so it is left earlier: 32 items of 1000 keys 67 / 52, 96 of 3000 112 / 113, 256 of 8192
// 279 / 318 us.
// (The request is a grid dimension here, of at most 65535; the 256-column grid has no such bound.)
bool attn_short_fits(const AttnLaunch& L) {
  if (L.n_req > 65535) return false;
  const int rpw = 256 / (L.Hq / L.Hkv);
  const int64_t items = (int64_t)(L.grid_rows + rpw - 1) / rpw * L.Hkv * L.n_req * L.D / 128;
  return items <= (!L.out ? 20 : L.D == 128 ? 140 : 90) + 80000 / std::max(1, L.max_keys);
}

hipError_t launch_attn_short(const AttnLaunch& L, bool paged, hipStream_t s) {
  return L.D == 128 ? launch_d<128>(L, paged, s) : launch_d<64>(L, paged, s);
}

}  // namespace sx
