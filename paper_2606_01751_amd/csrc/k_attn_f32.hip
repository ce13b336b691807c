// float32 attention and Sparse-Q column sums on v_mfma_f32_32x32x2_f32 / _16x16x4_f32: float32 operands
// and accumulators throughout.  Used when the layer stores float32 (small, accuracy-first
// configurations, 64 to a few thousand tokens); the bfloat16 path runs on the bf16 matrix cores.
//
// Both kernels give one tile of 16 or 32 columns (or keys) to a workgroup of 8 waves and split the
// other dimension over the waves, so that a short request still fills the chip; the waves' results are
// merged through LDS in wave order.  Operands come straight from global memory (L2) into registers: the
// float32 MFMAs are slow enough (64 FLOP per cycle and SIMD) to hide the loads, and the waves of a
// workgroup share nothing but the stationary tile.
//
// Operand order: an MFMA multiplies one value of d per lane group, and the order in which the d
// products are summed is free as long as both operands use it.  Group g of NG takes d = 4 NG j + 4 g + i
// at step (j, i), so every operand row is read in 16-byte pieces.
//
// The tile width is chosen by the size of the launch, so it must not show in a result: a request gives the
// same bits in any batch.  An MFMA adds its products to the accumulator one after the other in group order, so
// two of a 32-wide tile (two products each) taken in the order of one of a 16-wide tile (four) form the same
// sum; what a lane of a 32-wide tile sums on the vector ALU it keeps in two parts, those of the two lanes that
// share the work on a 16-wide tile (Tile::PH), added in the 16-wide tile's order.
#include <algorithm>

#include "sx_device.h"
#include "sx_internal.h"

namespace sx {
namespace {

constexpr int FW = 8;     // waves per workgroup
constexpr int kWideTiles = 256;   // 32-column tiles from which the attention uses them (one per compute unit)

struct AttnF {
  const float* q;
  const float* k;
  const float* v;
  float* out;
  float* lse;
  const ReqDev* reqs;
  const int32_t* bt;
  const int32_t* rows;
  const int32_t* n_rows;
  const int32_t* cu;
  int Hq, Hkv, G;
  int grid_rows;   // paged: rows of a request beyond this bound are not processed
  float scale;
};

// LDS written by other lanes of the wave before it is read by this one after it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ f32x4_t ld4(const float* p) { return *(const f32x4_t*)p; }

// CT x CT tiles of v_mfma_f32: NG lane groups hold one value of the contraction each, a lane owns
// column lc and rows row_in(e) of the result.
template <int CT>
struct Tile {
  static constexpr int NG = 64 / CT, AE = CT * CT / 64;
  static constexpr int PH = 4 / NG;   // parts (MFMAs) of a lane for one 16-wide tile's lane group (MFMA)
  typedef float acc_t __attribute__((ext_vector_type(AE)));
  static __device__ __forceinline__ acc_t mfma(float x, float y, acc_t c) {
    if constexpr (CT == 32) return __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row_in(int e, int g) { return 8 * (e >> 2) + 4 * g + (e & 3); }   // (CT = 16: e < 4)
};

// Attention of CT query columns of one KV head (a column is a (listed row, query head) pair, row
// major, so any group size fills the tile).  Pieces of 32 keys go to the waves in turn.
// S^T = K Q^T on CT x CT tiles: a lane owns one column (lc) and KPP keys of the piece, so the softmax
// stays in the NG lanes of a column; O^T += V^T P^T takes one of those keys per lane group and MFMA, so
// P^T is the lane's own registers and a V row is read whole, VW consecutive values per lane
// (d = VW lc + j).
// Matrix-core bound (64 FLOP per cycle and SIMD at either CT), with the loads and the softmax of the
// other wave of the SIMD beside the MFMAs.  The column tile is the least work a compute unit can get:
// 32 columns of 1500 keys at D = 64 take it 20 us, so launches of few tiles use 16 columns, which
// doubles the K/V reads per column (see the dispatch).
// Measured: 1500 tokens, 576 rows, 8/2/64 27 us (237 with one wave per row and head on the vector
// ALU), the 192 probe rows of a 512-token layer 8.6 us (20), 4096 rows of 32/8/128 1.45 ms or
// 95 TFLOP/s (29 ms).  expf takes 6 % of that over v_exp_f32 of x log2 e with the product's rounding made up
// for, which is as exact for probabilities near 1 but drops those below 2^-126.
template <int D, int CT, bool PAGED, bool PV>
__global__ __launch_bounds__(FW * 64, 1) void attn_f32_kernel(AttnF a) {
  constexpr int NG = Tile<CT>::NG, AE = Tile<CT>::AE, PH = Tile<CT>::PH;
  constexpr int KT = 32 / CT;               // key tiles per piece
  constexpr int KPP = KT * AE;              // keys per lane and piece
  constexpr int QS = D + 4;                 // floats per Q row in LDS
  constexpr int VW = D / CT;                // V values per lane and key
  constexpr int RS = D * CT;                // floats of one wave's O^T in the merge buffer
  constexpr int NJ = D / (4 * NG);          // 16-byte operand pieces per lane and row
  typedef typename Tile<CT>::acc_t acc_t;
  __shared__ __attribute__((aligned(16))) float qs[CT * QS];
  __shared__ __attribute__((aligned(16))) float red[PV ? FW / 2 * RS : 4];
  __shared__ float ms[FW][CT], ls[FW][CT];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lc = lane % CT, g = lane / CT;
  // key of the piece that a lane's value x is
  auto key_in = [&](int x) { return (CT == 32 ? 8 : 16) * (x >> 2) + 4 * g + (x & 3); };
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
  auto row_of = [&](int c) { return min(c, ncols - 1) / a.G; };
  auto pos_of = [&](int n) -> int { return PAGED ? a.rows[tok_off + n] : n; };
  const int my_row = row_of(c0 + lc);
  const bool valid = c0 + lc < ncols;
  const int pos = pos_of(my_row);
  // Q tile into LDS, 16 bytes per thread and step
  for (int x = tid; x < CT * (D / 4); x += FW * 64) {
    const int c = x / (D / 4), d4 = x % (D / 4);
    const int n = row_of(c0 + c), h = min(c0 + c, ncols - 1) - n * a.G;
    *(f32x4_t*)(qs + c * QS + 4 * d4) = ld4(a.q + ((int64_t)(tok_off + pos_of(n)) * a.Hq + kvh * a.G + h) * D + 4 * d4);
  }
  const int cmax = wave_max_i(pos, lane), cmin = wave_min_i(pos, lane);   // last visible key of any / every column
  const int np = cmax / 32 + 1;
  // 16-key block b of the request: element offset of its first row (uniform; the block id by a scalar
  // load).  Keys past the tile's last visible one read that one's row (they are masked).
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
  f32x4_t kr[KT][NJ];
  auto load_k = [&](int t, const int64_t (&bo)[2]) {
#pragma unroll
    for (int b = 0; b < KT; ++b) {
      const int i = CT * b + lc, bb = i >> 4;
      const float* p = a.k + (bb ? bo[1] : bo[0]) + row_off(2 * t + bb, i & 15) + 4 * g;
#pragma unroll
      for (int j = 0; j < NJ; ++j) kr[b][j] = ld4(p + 4 * NG * j);
    }
  };
  float m = -INFINITY, l[PH];
#pragma unroll
  for (int h = 0; h < PH; ++h) l[h] = 0.f;
  acc_t o[PV ? VW : 1];
#pragma unroll
  for (int j = 0; j < (PV ? VW : 1); ++j) o[j] = acc_t{};
  // the next piece's K is read ahead where the registers allow it
  constexpr bool PRE = !(PV && D == 128 && CT == 32);
  int64_t bo[2] = {blk_off(2 * w), blk_off(2 * w + 1)};   // blocks of the wave's piece
  if (PRE && w < np) load_k(w, bo);
  __syncthreads();
  for (int t = w; t < np; t += FW) {
    const int kbase = t * 32;
    const int64_t bn[2] = {blk_off(2 * (t + FW)), blk_off(2 * (t + FW) + 1)};   // of its next one
    if constexpr (!PRE) load_k(t, bo);
    float vr[PV ? KPP : 1][VW];
    if constexpr (PV) {
      // (keys 0-15 and 16-31 of the piece are one block each)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int x = b * KPP / 2; x < (b + 1) * KPP / 2; ++x) {
          const float* p = a.v + bo[b] + row_off(2 * t + b, key_in(x) & 15) + VW * lc;
#pragma unroll
          for (int j = 0; j < VW; j += VW == 2 ? 2 : 4) {
            if constexpr (VW == 2) {
              const float2 y = *(const float2*)p;
              vr[x][0] = y.x;
              vr[x][1] = y.y;
            } else {
              const f32x4_t y = ld4(p + j);
#pragma unroll
              for (int i = 0; i < 4; ++i) vr[x][j + i] = y[i];
            }
          }
        }
      }
    }
    acc_t s[KT];
#pragma unroll
    for (int b = 0; b < KT; ++b) s[b] = acc_t{};
#pragma unroll
    for (int j = 0; j < NJ; j += PH) {
      f32x4_t qj[PH];
#pragma unroll
      for (int h = 0; h < PH; ++h) qj[h] = ld4(qs + lc * QS + 4 * NG * (j + h) + 4 * g);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < PH; ++h)
#pragma unroll
          for (int b = 0; b < KT; ++b) s[b] = Tile<CT>::mfma(kr[b][j + h][i], qj[h][i], s[b]);
    }
    if (PRE && t + FW < np) load_k(t + FW, bn);
    float p[KPP];
    float mx = -INFINITY;
#pragma unroll
    for (int x = 0; x < KPP; ++x) {
      p[x] = kbase + key_in(x) > pos ? -INFINITY : s[x / AE][x % AE] * a.scale;
      mx = fmaxf(mx, p[x]);
    }
#pragma unroll
    for (int i = CT; i < 64; i <<= 1) mx = fmaxf(mx, __shfl_xor(mx, i, 64));
    const float mn = fmaxf(m, mx);
    if (__ballot(mn > m)) {
      const float f = mn == -INFINITY ? 1.f : expf(m - mn);
#pragma unroll
      for (int h = 0; h < PH; ++h) l[h] *= f;
      if constexpr (PV) {
#pragma unroll
        for (int j = 0; j < VW; ++j)
#pragma unroll
          for (int e = 0; e < AE; ++e) o[j][e] *= f;
      }
      m = mn;
    }
    const float msub = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int x = 0; x < KPP; ++x) {
      p[x] = expf(p[x] - msub);
      l[(x >> 2) % PH] += p[x];   // (keys 16 b + 8 h + 4 g ..: part h)
    }
    if constexpr (PV) {
      // A masked key must not reach a column even when its V is infinite or NaN (0 x inf): on pieces
      // with masked keys such values are left out of the product and added to the columns that see them
      bool odd = false;
      if (kbase + 31 > cmin) {
#pragma unroll
        for (int x = 0; x < KPP; ++x)
#pragma unroll
          for (int j = 0; j < VW; ++j) {
            const bool fin = fabsf(vr[x][j]) < INFINITY;
            odd |= !fin;
            vr[x][j] = fin ? vr[x][j] : 0.f;
          }
      }
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int h = 0; h < PH; ++h) {
            const int x = (b * PH + h) * 4 + i;
#pragma unroll
            for (int j = 0; j < VW; ++j) o[j] = Tile<CT>::mfma(vr[x][j], p[x], o[j]);
          }
      if (__ballot(odd)) {
        // rare: key by key, the probabilities through this wave's part of the merge buffer
        static_assert(FW / 2 * RS / FW >= 32 * CT, "a wave's part of the merge buffer holds a piece");
        float* pw = red + w * (FW / 2 * RS / FW);
        wave_sync();
#pragma unroll
        for (int x = 0; x < KPP; ++x) pw[key_in(x) * CT + lc] = p[x];
        wave_sync();
        for (int kk = 0; kk < 32; ++kk) {
          const int key = kbase + kk;
          const float pk = pw[kk * CT + lc];
          const float* vp = a.v + (kk < 16 ? bo[0] : bo[1]) + row_off(key >> 4, kk & 15);
#pragma unroll
          for (int e = 0; e < AE; ++e)
#pragma unroll
            for (int j = 0; j < VW; ++j) {
              const float y = vp[VW * Tile<CT>::row_in(e, g) + j];
              if (key <= pos && !(fabsf(y) < INFINITY)) o[j][e] += pk * y;
            }
        }
        wave_sync();
      }
    }
    bo[0] = bn[0];
    bo[1] = bn[1];
  }
#pragma unroll
  for (int h = 0; h < PH; ++h)
#pragma unroll
    for (int i = CT; i < 64; i <<= 1) l[h] += __shfl_xor(l[h], i, 64);
  if (g == 0) {
    ms[w][lc] = m;
    ls[w][lc] = PH == 1 ? l[0] : l[0] + l[PH - 1];
  }
  __syncthreads();
  float M = -INFINITY, L = 0.f;
#pragma unroll
  for (int i = 0; i < FW; ++i) M = fmaxf(M, ms[i][lc]);
#pragma unroll
  for (int i = 0; i < FW; ++i) L += ms[i][lc] == -INFINITY ? ls[i][lc] : ls[i][lc] * expf(ms[i][lc] - M);
  const int h = c0 + lc - my_row * a.G;
  if constexpr (PV) {
    const float f = m == -INFINITY ? 1.f : expf(m - M);   // (no key seen: O is 0, or NaN as L then is)
#pragma unroll
    for (int j = 0; j < VW; ++j)
#pragma unroll
      for (int e = 0; e < AE; ++e) o[j][e] *= f;
    // O^T of the upper half of the waves onto the lower half's, until wave 0 holds the sum
#pragma unroll
    for (int n = FW / 2; n >= 1; n >>= 1) {
      if (w >= n && w < 2 * n) {
#pragma unroll
        for (int j = 0; j < VW; ++j)
#pragma unroll
          for (int e = 0; e < AE; ++e) red[(w - n) * RS + (j * AE + e) * 64 + lane] = o[j][e];
      }
      __syncthreads();
      if (w < n) {
#pragma unroll
        for (int j = 0; j < VW; ++j)
#pragma unroll
          for (int e = 0; e < AE; ++e) o[j][e] += red[w * RS + (j * AE + e) * 64 + lane];
      }
      __syncthreads();
    }
    if (w == 0 && valid) {
      float* op = a.out + ((int64_t)(tok_off + my_row) * a.Hq + kvh * a.G + h) * D;
#pragma unroll
      for (int e = 0; e < AE; ++e) {
        const int d0 = VW * Tile<CT>::row_in(e, g);
        if constexpr (VW == 2) {
          *(float2*)(op + d0) = make_float2(o[0][e] / L, o[1][e] / L);
        } else {
#pragma unroll
          for (int j = 0; j < VW; j += 4) {
            f32x4_t y;
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = o[j + i][e] / L;
            *(f32x4_t*)(op + d0 + j) = y;
          }
        }
      }
    }
  }
  if (a.lse && w == 0 && g == 0 && valid)
    a.lse[(int64_t)(tok_off + my_row) * a.Hq + kvh * a.G + h] = M + logf(L);   // natural log of sum exp(scale q.k)
}

// Column sums of the Sparse-Q probabilities of CT keys of one KV head: S = Q K^T with the keys
// stationary in registers as the B operand (a lane owns one key), the probe columns (probe row x head
// of the group, row major) streamed as the A operand in pieces of 32 that go to the waves in turn:
// sum over the columns i >= j of exp(scale q.k - lse), each probability added in float64, then the lane
// groups, then the waves in order.
// Measured (512 tokens, 192 probe rows, 8/2/64): 12.2 us; with one key per thread walking all
// columns, in 4 workgroups, 1351 us.
struct ColsumF {
  const float* q;
  const float* k;
  const float* lse;
  const ReqDev* reqs;
  const int32_t* bt;
  const int32_t* probe;
  double* colsum;
  int64_t total;
  int Hq, Hkv, G;
  float scale;
  int lse_tok;   // 0: lse indexed by probe; 1: indexed by token position
};

template <int D, int CT>
__global__ __launch_bounds__(FW * 64, 1) void colsum_f32_kernel(ColsumF a) {
  constexpr int NG = Tile<CT>::NG, AE = Tile<CT>::AE, PH = Tile<CT>::PH;
  constexpr int KT = 32 / CT;               // column tiles per piece
  constexpr int NJ = D / (4 * NG);          // 16-byte operand pieces per lane and row
  typedef typename Tile<CT>::acc_t acc_t;
  __shared__ __attribute__((aligned(16))) float s_lse[FW][32];
  __shared__ __attribute__((aligned(16))) int s_pos[FW][32];
  __shared__ double s_sum[FW][CT];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lc = lane % CT, g = lane / CT;
  const int kvh = blockIdx.x % a.Hkv;
  const int tile = (int)(blockIdx.y * kTilesX + blockIdx.x / a.Hkv);
  const ReqDev rq = a.reqs[blockIdx.z];
  const int j0 = tile * CT;   // first keys first: the most probe rows see them
  if (j0 >= rq.T) return;
  const int key = j0 + lc;
  f32x4_t kb[NJ];
  {
    const int jj = min(key, rq.T - 1);
    const int32_t blk = a.bt[rq.bt_off + (jj >> 4)];
    const float* kp = a.k + (((int64_t)blk * a.Hkv + kvh) * 16 + (jj & 15)) * D + 4 * g;
#pragma unroll
    for (int j = 0; j < NJ; ++j) kb[j] = ld4(kp + 4 * NG * j);
  }
  const int32_t* probe = a.probe + rq.tok_off;
  // first probe row that sees a key of the 32 (the pieces start there at either tile width)
  const int lo = lower_bound_wave(probe, rq.n_probe, j0 & ~31, lane);
  const int ncols = (rq.n_probe - lo) * a.G;
  // piece t: the query rows of this lane's columns, and the log-sum-exp and position of column lane % 32
  // (position -1 past the end)
  f32x4_t qr[KT][NJ];
  float ql = 0.f;
  int qp = -1;
  auto load = [&](int t) {
    int pos[KT];
#pragma unroll
    for (int b = 0; b < KT; ++b) {
      const int c = min(t * 32 + CT * b + lc, ncols - 1);
      const int n = c / a.G;
      pos[b] = probe[lo + n];
      const float* p = a.q + ((int64_t)(rq.tok_off + pos[b]) * a.Hq + kvh * a.G + c - n * a.G) * D + 4 * g;
#pragma unroll
      for (int j = 0; j < NJ; ++j) qr[b][j] = ld4(p + 4 * NG * j);
    }
    const int c = t * 32 + (lane & 31), cc = min(c, ncols - 1);
    const int n = cc / a.G;
    const int cp = KT == 1 ? pos[0] : (g & 1) ? pos[KT - 1] : pos[0];
    ql = a.lse[(int64_t)(rq.tok_off + (a.lse_tok ? cp : lo + n)) * a.Hq + kvh * a.G + cc - n * a.G];
    qp = c < ncols ? cp : -1;
  };
  double acc[PH];
#pragma unroll
  for (int h = 0; h < PH; ++h) acc[h] = 0.0;
  const int np = (ncols + 31) / 32;
  if (w < np) load(w);
  for (int t = w; t < np; t += FW) {
    wave_sync();
    if (lane < 32) {
      s_lse[w][lane] = ql;
      s_pos[w][lane] = qp;
    }
    wave_sync();
    acc_t s[KT];
#pragma unroll
    for (int b = 0; b < KT; ++b) s[b] = acc_t{};
#pragma unroll
    for (int j = 0; j < NJ; j += PH)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < PH; ++h)
#pragma unroll
          for (int b = 0; b < KT; ++b) s[b] = Tile<CT>::mfma(qr[b][j + h][i], kb[j + h][i], s[b]);
    if (t + FW < np) load(t + FW);
#pragma unroll
    for (int b = 0; b < KT; ++b)
#pragma unroll
      for (int e = 0; e < AE; e += 4) {
        const int c = CT * b + Tile<CT>::row_in(e, g);
        const f32x4_t l4 = *(const f32x4_t*)&s_lse[w][c];
        const int4 p4 = *(const int4*)&s_pos[w][c];
        const int ps[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float pr = expf(s[b][e + i] * a.scale - l4[i]);
          acc[(e >> 2) % PH] += (double)(key <= ps[i] ? pr : 0.f);
        }
      }
  }
#pragma unroll
  for (int h = 0; h < PH; ++h)
#pragma unroll
    for (int i = CT; i < 64; i <<= 1) acc[h] += __shfl_xor(acc[h], i, 64);
  if (g == 0) s_sum[w][lc] = PH == 1 ? acc[0] : acc[0] + acc[PH - 1];
  __syncthreads();
  if (tid < CT && key < rq.T) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < FW; ++i) t += s_sum[i][tid];
    a.colsum[(int64_t)kvh * a.total + rq.tok_off + key] = t;
  }
}

dim3 grid_of(int64_t tiles, int Hkv, int n_req) {
  return dim3((unsigned)(Hkv * std::min<int64_t>(tiles, kTilesX)), (unsigned)((tiles + kTilesX - 1) / kTilesX), (unsigned)n_req);
}

}  // namespace

hipError_t launch_attn_f32(const AttnLaunch& L, bool paged, hipStream_t s) {
  AttnF a{};
  a.q = (const float*)L.q;
  a.k = (const float*)L.k;
  a.v = (const float*)L.v;
  a.out = (float*)L.out;
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
  a.scale = L.scale;
  // 32 columns per workgroup read each K/V row half as often; 16 columns give twice the workgroups and
  // halve the longest one, which is what bounds a launch with fewer tiles than compute units.  Measured
  // (calls, 16 / 32 columns): 144 tiles 27 / 41 us, 250 38 / 52; 304 41 / 34, 400 80 / 74, 600 121 / 109, 4096
  // 1627 / 1455 us
  const bool wide = ((int64_t)L.grid_rows * a.G + 31) / 32 * L.Hkv * L.n_req >= kWideTiles;
  const int ct = wide ? 32 : 16;
  const dim3 grid = grid_of(((int64_t)L.grid_rows * a.G + ct - 1) / ct, L.Hkv, L.n_req);
  const bool pv = L.out != nullptr;
#define SX_F32_LAUNCH(D_, P_, V_)                                                                           \
  do {                                                                                                      \
    if (wide) hipLaunchKernelGGL((attn_f32_kernel<D_, 32, P_, V_>), grid, dim3(FW * 64), 0, s, a);         \
    else hipLaunchKernelGGL((attn_f32_kernel<D_, 16, P_, V_>), grid, dim3(FW * 64), 0, s, a);              \
  } while (0)
  if (L.D == 128) {
    if (paged) { if (pv) SX_F32_LAUNCH(128, true, true); else SX_F32_LAUNCH(128, true, false); }
    else SX_F32_LAUNCH(128, false, true);
  } else {
    if (paged) { if (pv) SX_F32_LAUNCH(64, true, true); else SX_F32_LAUNCH(64, true, false); }
    else SX_F32_LAUNCH(64, false, true);
  }
#undef SX_F32_LAUNCH
  return hipGetLastError();
}

hipError_t launch_colsum_f32(const sx_plan* p, double* colsum, const void* q, const void* kc, const float* lse,
                             int lse_tok, hipStream_t s) {
  ColsumF a{};
  a.q = (const float*)q;
  a.k = (const float*)kc;
  a.lse = lse;
  a.lse_tok = lse_tok;
  a.reqs = p->d_req;
  a.bt = p->d_bt;
  a.probe = p->d_probe;
  a.colsum = colsum;
  a.total = p->total;
  a.Hq = p->desc.n_q_heads;
  a.Hkv = p->desc.n_kv_heads;
  a.G = a.Hq / a.Hkv;
  a.scale = p->scale;
  // the tile width as for the attention above (512 tokens, 8/2/64: 16 / 32 keys 11.3 / 14.1 us)
  const bool wide = ((int64_t)p->max_T + 31) / 32 * a.Hkv * p->n_req >= kWideTiles;
  const int ct = wide ? 32 : 16;
  const dim3 grid = grid_of((p->max_T + ct - 1) / ct, a.Hkv, p->n_req);
#define SX_F32_COLSUM(D_)                                                                                \
  do {                                                                                                   \
    if (wide) hipLaunchKernelGGL((colsum_f32_kernel<D_, 32>), grid, dim3(FW * 64), 0, s, a);            \
    else hipLaunchKernelGGL((colsum_f32_kernel<D_, 16>), grid, dim3(FW * 64), 0, s, a);                 \
  } while (0)
  if (p->desc.head_dim == 128) SX_F32_COLSUM(128);
  else SX_F32_COLSUM(64);
#undef SX_F32_COLSUM
  return hipGetLastError();
}

}  // namespace sx
