// Row-sparse layer body (Algorithm 1 steps 19 and 22): the projections, normalisations and the
// feed-forward module evaluated on the rows of the recompute set R only.
//
//   gemm_rows_kernel     Y[row] = X[row] W^T (+ residual[row]): bfloat16 operands, float32
//                        accumulation on v_mfma_f32_16x16x32_bf16, W stored [n][k] (k contiguous,
//                        the layout of a linear layer's weight)
//   rmsnorm_rows_kernel  Y[row] = X[row] / sqrt(mean(X[row]^2) + eps) * gamma
//   rope_rows_kernel     RoPE of fresh query / key rows at their positions in the new sequence
//   silu_mul_rows_kernel Y[row] = silu(G[row]) * U[row] for a gate|up product [row][2f]
//
// Rows: for request r, the listed rows n < n_rows[r] of the row-list layout.  An operand row is
// addressed by slot (off_r + n: compact per request, like the sparse attention output) or by
// token (off_r + rows[off_r + n]: the request's token rows, like fresh Q/K/V and hidden states).
#include <type_traits>

#include "sx_device.h"
#include "sx_internal.h"

namespace sx {
namespace {

typedef float f32x2_t __attribute__((ext_vector_type(2)));

// s_waitcnt with vmcnt <= n (n < 16), expcnt and lgkmcnt left unconstrained (gfx9 encoding).
#define SX_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (0x7 << 4) | (0xF << 8))
// the same for n < 64 (the counter's two high bits sit at 15:14)
#define SX_WAIT_VMCNT6(n) \
  __builtin_amdgcn_s_waitcnt(((n) & 0xF) | ((((n) >> 4) & 3) << 14) | (0x7 << 4) | (0xF << 8))

__device__ __forceinline__ int64_t row_index(const ReqDev& rq, const int32_t* rows, int n, bool by_token) {
  return by_token ? (int64_t)rq.tok_off + rows[rq.tok_off + n] : (int64_t)rq.tok_off + n;
}

// ---------------------------------------------------------------------------------------------
// GEMM on listed rows.  Computed transposed, Y^T = W X^T: the MFMA A operand is a slice of W (16
// output features), the B operand a slice of X^T (16 rows), so each lane owns one row of the
// result and writes 4 consecutive features per store.
// Workgroup tile: BN features x BM rows; WN x WM waves, a wave owns BN / WN features x BM / WM rows.  The
// MFMA is v_mfma_f32_16x16x32_bf16: measured 1-12 % faster than v_mfma_f32_32x32x16_bf16 on the same
// tiles, most on the narrow products.  The k dimension moves in stages of 64 through NST LDS buffers:
// both operand tiles go global -> LDS directly (16 bytes per lane); stage t + NST is issued once its
// readers have read stage t, so a stage has about NST - 1 stages of compute to land.  A tile row (64 bf16)
// holds 8 chunks of 16 bytes, XOR-swizzled per row (chunk_swz) so that the rows a read instruction touches
// at one logical chunk hit distinct banks.
// Every tile sums an element over k in one order, MFMA after MFMA, so a row's result does not depend on
// the tile that the launch's size chose.  Two or four wave groups that share k on the small tiles, their
// sums added at the end, were no faster (394 rows, 4096 -> 4096 features: 26.3 / 27.2 us in two groups;
// 200 rows 20.2 / 20.7 in four).
// Matrix-core bound on 256 x 256 tiles with many rows (gate_up of 6712 rows, 4096 -> 28672: 1252 us,
// 1.26 PFLOP/s, 1370 with a stage's transfers issued together); with few rows a tile per compute unit
// bounds it (see the dispatch).
// ---------------------------------------------------------------------------------------------
constexpr int kGemmMaxParts = 4;
constexpr int kGemmGM = 8;          // row tiles per group of the tile order
constexpr int kGemmPart = 256;      // widths are multiples of this (a tile lies in one output part)
constexpr unsigned kGemmXcds = 8;   // XCDs of the chip, which deals workgroups round-robin

struct GemmRowsK {
  const ReqDev* reqs;
  const int32_t* rows;
  const int32_t* n_rows;
  const uint16_t* x;
  const uint16_t* w;
  const uint16_t* res;
  uint16_t* y[kGemmMaxParts];   // output part p: columns pn[p] .. pn[p + 1] - 1, row stride pn[p + 1] - pn[p]
  int pn[kGemmMaxParts + 1];
  int n_parts, K, N, n_req, m_tiles, max_rows, x_tok, y_tok;
};

// physical chunk of logical chunk c in tile row `row` (8 chunks per row): 16 consecutive rows
// read at one logical chunk cover the 16 four-bank groups of a 256-byte LDS line
__device__ __forceinline__ int chunk_swz(int c, int row) { return c ^ ((row >> 1) & 7); }   // (two rows per line)

template <int BN, int BM, int WN, int WM, int NST>
__global__ __launch_bounds__(WN * WM * 64, 1) void gemm_rows_kernel(GemmRowsK a) {
  constexpr int NW = WN * WM;
  constexpr int FI = BN / WN / 16;             // 16-feature fragments per wave
  constexpr int RJ = BM / WM / 16;             // 16-row fragments per wave
  constexpr int ROWB = 128;                    // bytes of one tile row (64 bf16)
  constexpr int CH = ROWB / 16;                // 16-byte chunks per row
  constexpr int RPT = 1024 / ROWB;             // rows per 1 KB transfer
  constexpr int STAGE = (BN + BM) * ROWB;
  constexpr int PW = BN / RPT / NW, PX = BM / RPT / NW;   // transfers per wave and operand
  static_assert(PW * NW * RPT == BN && PX * NW * RPT == BM, "transfers spread evenly over the waves");
  static_assert(kGemmPart % BN == 0, "a tile lies in one output part");
  __shared__ __attribute__((aligned(1024))) char smem[NST * STAGE];   // [stage][W | X]
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wu = __builtin_amdgcn_readfirstlane(tid >> 6);
  // tile order: groups of kGemmGM row tiles, the feature tile slowest within a group, so that a run of
  // consecutive tile indices covers a few feature tiles x all row tiles of the group.  The hardware
  // deals block b to XCD b mod 8; each XCD takes a contiguous run of tile indices, so the workgroups
  // running together on one XCD read the same W and X k-slices through that XCD's L2.
  const int n_mt = a.n_req * a.m_tiles;
  const int n_nt = a.N / BN;
  const unsigned per_xcd = gridDim.x / kGemmXcds;   // the grid is a multiple of kGemmXcds
  const int L = (int)((blockIdx.x % kGemmXcds) * per_xcd + blockIdx.x / kGemmXcds);
  if (L >= n_mt * n_nt) return;
  const int grp = L / (kGemmGM * n_nt);
  const int in_g = L - grp * kGemmGM * n_nt;
  const int gm = min(kGemmGM, n_mt - grp * kGemmGM);
  const int mt_all = grp * kGemmGM + in_g % gm;
  const int nt = in_g / gm;
  const int r = mt_all / a.m_tiles;
  const int m0 = (mt_all - r * a.m_tiles) * BM;
  const ReqDev rq = a.reqs[r];
  const int nr = min(a.n_rows[r], a.max_rows);
  if (m0 >= nr) return;
  const int n0 = nt * BN;
  const int K = a.K;

  // ---- transfers: 1 KB holds rows RPT q .. RPT q + RPT - 1 of a tile; lane l fills row RPT q + l / CH,
  // physical chunk l % CH with the logical chunk that chunk_swz maps there.  A wave moves transfers
  // wu + NW i of both tiles. ----
  const uint16_t* src[PW + PX];
#pragma unroll
  for (int i = 0; i < PW; ++i) {
    const int row = RPT * (wu + NW * i) + lane / CH;
    src[i] = a.w + (int64_t)(n0 + row) * K + chunk_swz(lane % CH, row) * 8;   // (an involution)
  }
#pragma unroll
  for (int i = 0; i < PX; ++i) {
    const int row = RPT * (wu + NW * i) + lane / CH;
    const int m = min(m0 + row, nr - 1);   // rows past the request's last read a valid row
    src[PW + i] = a.x + row_index(rq, a.rows, m, a.x_tok) * K + chunk_swz(lane % CH, row) * 8;
  }
  const uint32_t smem_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const int nk = K / 64;
  // transfer d of this wave for stage t, into buffer t mod NST
  auto dma = [&](int t, int d) {
    const uint32_t m0r = __builtin_amdgcn_readfirstlane(smem_lds + (uint32_t)((t % NST) * STAGE) +
                                                        (uint32_t)(d < PW ? (wu + NW * d) * 1024 : BN * ROWB + (wu + NW * (d - PW)) * 1024));
    asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src[d] + t * 64), "s"(m0r) : "m0", "memory");
  };
  // wait until this wave's transfers of every stage before the n youngest have landed
  auto wait_stages = [&](int n) {
    constexpr int P = PW + PX;
    static_assert((NST - 1) * P < 64 && NST <= 4, "wait table");
    switch (n) {
      case 1: SX_WAIT_VMCNT6(P); break;
      case 2: SX_WAIT_VMCNT6(2 * P & 63); break;
      case 3: SX_WAIT_VMCNT6(3 * P & 63); break;
      default: SX_WAIT_VMCNT6(0); break;
    }
  };
  // Before stage t is read: this wave's transfers of it have landed (the younger ones may be in flight),
  // its reads of the stages before are done (the barrier alone does not wait for them), and so are the
  // other waves'; past it the buffer of stage t - 1 is free.
  auto enter_stage = [&](int t) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wait_stages(min(NST - 2, nk - 1 - t));
    __syncthreads();
  };

  // ---- operand reads: a lane reads row lr of each 16-row fragment, 16 bytes of k starting at chunk
  // 4 s + cg: the lane part depends on s only, the fragment adds a constant (an immediate offset) ----
  const int wn = wu % WN, wm = wu / WN;
  const int lr = lane % 16, cg = lane / 16;
  uint32_t lane_off[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) lane_off[s] = (uint32_t)(lr * ROWB + (chunk_swz(4 * s + cg, lr) << 4));
  f32x4_t acc[FI][RJ];
#pragma unroll
  for (int i = 0; i < FI; ++i)
#pragma unroll
    for (int j = 0; j < RJ; ++j) acc[i][j] = f32x4_t{};

  // Software pipeline over slices: while the MFMAs of a slice run, the fragments of the next one are
  // read (the row fragments into the registers that the MFMAs have just read for the last time, the
  // feature fragments into a second set) and, once a stage's buffer is free, the transfers that refill
  // it are issued one by one between the MFMAs (issued together they hold every wave for as long as half
  // the stage's MFMAs take: the address unit takes about 22 cycles per transfer and compute unit).  A
  // stage is entered after the first MFMAs of the slice before it, so that they cover the last reads of
  // the stage that it ends.  The order is pinned: MFMA m, then the reads and transfers due.
  bf16x8_t fw[2][FI], fx[RJ];
  constexpr int NM = FI * RJ, ND = PW + PX;
  auto lds16 = [](uint32_t addr) { return *(const __attribute__((address_space(3))) bf16x8_t*)(uintptr_t)addr; };
  // MFMAs of a slice on feature set C; RD: read slice RS of stage rst beside them, EN: entering it
  // first; DM: refill with stage dst
  auto phase = [&](auto set, auto rd, auto en, int rst, auto rs, auto dm, int dst) {
    constexpr int C = decltype(set)::value, RS = decltype(rs)::value;
    constexpr bool RD = decltype(rd)::value, EN = decltype(en)::value, DM = decltype(dm)::value;
    constexpr int P0 = EN ? (RJ >= 4 ? 2 : 1) * FI : 0;   // MFMAs before the stage is entered
    uint32_t wb = 0, xb = 0;
    if constexpr (RD) {
      // one base register per matrix (the empty asm keeps the sums from being re-associated into one
      // register per read), the row blocks as immediate offsets
      const uint32_t sb = smem_lds + (uint32_t)((rst % NST) * STAGE);
      wb = sb + lane_off[RS] + (uint32_t)(wn * FI * 16 * ROWB);
      xb = sb + (uint32_t)(BN * ROWB) + lane_off[RS] + (uint32_t)(wm * RJ * 16 * ROWB);
      asm volatile("" : "+v"(wb), "+v"(xb));
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int i = m % FI, j = m / FI;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[C][i], fx[j], acc[i][j], 0, 0, 0);
      if (EN && m == P0 - 1) {
        __builtin_amdgcn_sched_barrier(0);
        enter_stage(rst);
      }
      if constexpr (RD) {
#pragma unroll
        for (int f = 0; f < FI; ++f)
          if (m == (P0 + f < NM ? P0 + f : NM - 1)) fw[1 - C][f] = lds16(wb + (uint32_t)(f * 16 * ROWB));
#pragma unroll
        for (int f = 0; f < RJ; ++f) {
          const int at = (f + 1) * FI - 1 > P0 + FI + f ? (f + 1) * FI - 1 : P0 + FI + f;
          if (m == (at < NM ? at : NM - 1)) fx[f] = lds16(xb + (uint32_t)(f * 16 * ROWB));
        }
      }
      if constexpr (DM) {
#pragma unroll
        for (int d = 0; d < ND; ++d)
          if (m == P0 + (2 * d + 1) * (NM - P0) / (2 * ND) ) dma(dst, d);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  // the row indices above are compiler-visible loads: complete before the first transfer wait
  SX_WAIT_VMCNT(0);
#pragma unroll
  for (int t = 0; t < NST; ++t)
    if (t < nk)
#pragma unroll
      for (int d = 0; d < ND; ++d) dma(t, d);
  wait_stages(min(NST - 1, nk - 1));   // stage 0 has landed
  __syncthreads();
  {
    const uint32_t wb = smem_lds + lane_off[0] + (uint32_t)(wn * FI * 16 * ROWB);
    const uint32_t xb = smem_lds + (uint32_t)(BN * ROWB) + lane_off[0] + (uint32_t)(wm * RJ * 16 * ROWB);
#pragma unroll
    for (int j = 0; j < RJ; ++j) fx[j] = lds16(xb + (uint32_t)(j * 16 * ROWB));
#pragma unroll
    for (int i = 0; i < FI; ++i) fw[0][i] = lds16(wb + (uint32_t)(i * 16 * ROWB));
    // stages that refill their buffer, stages that do not, the last one
    int t = 0;
    for (; t + NST < nk; ++t) {
      phase(c0, yes, no, t, c1, no, 0);
      phase(c1, yes, yes, t + 1, c0, yes, t + NST);
    }
    for (; t + 1 < nk; ++t) {
      phase(c0, yes, no, t, c1, no, 0);
      phase(c1, yes, yes, t + 1, c0, no, 0);
    }
    phase(c0, yes, no, t, c1, no, 0);
    phase(c1, no, no, 0, c0, no, 0);
  }

  // ---- epilogue: lane owns row 16 j + lr of the wave's rows; value e of accumulator (i, j) is feature
  // 16 i + 4 cg + e of the wave's features.  Part boundaries are multiples of the tile width, so the
  // output part is the tile's. ----
  int op = 0;
  while (op + 1 < a.n_parts && n0 >= a.pn[op + 1]) ++op;
  uint16_t* const yp = a.y[op];
  const int ld = a.pn[op + 1] - a.pn[op];
  const int col0 = n0 - a.pn[op] + wn * FI * 16 + 4 * cg;
#pragma unroll
  for (int f = 0; f < FI * RJ; ++f) {
    const int i = f % FI, j = f / FI;
    const int m = m0 + wm * RJ * 16 + 16 * j + lr;
    if (m >= nr) continue;
    const int64_t yr = row_index(rq, a.rows, m, a.y_tok) * ld + col0 + 16 * i;
    f32x4_t v = acc[i][j];
    if (a.res) {
      const uint2 rv = *(const uint2*)(a.res + yr);
      v[0] += bf16_lo(rv.x);
      v[1] += bf16_hi(rv.x);
      v[2] += bf16_lo(rv.y);
      v[3] += bf16_hi(rv.y);
    }
    uint2 o;
    o.x = pack_bf16x2(v[0], v[1]);
    o.y = pack_bf16x2(v[2], v[3]);
    *(uint2*)(yp + yr) = o;
  }
}

// ---------------------------------------------------------------------------------------------
// RMSNorm of listed rows: one workgroup per row, the row read once into registers (NC 16-byte pieces
// per thread; longer rows read their further pieces again), sum of squares in a fixed order (thread,
// wave, waves in order).  Sum and products in float64, which hides under the row's transfers and leaves
// the rounding to float32 and from there to bf16: a float32 product near a rounding boundary of bf16 is off by
// a whole unit for every later reader of the row.  Bound by HBM, for few rows by the latency of one read: 394 rows of
// 4096 5.3 us, 6750 rows 23 us; one wave per row reading it twice took 9.2 and 28.5.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rmsnorm_rows_kernel(const ReqDev* __restrict__ reqs, const int32_t* __restrict__ rows,
                                                           const int32_t* __restrict__ n_rows, int max_rows,
                                                           const uint16_t* __restrict__ x, int x_tok,
                                                           const uint16_t* __restrict__ gamma, float eps, int H,
                                                           uint16_t* __restrict__ y, int y_tok) {
  constexpr int NC = 2, STEP = 256 * 8;
  __shared__ double part[4];
  const ReqDev rq = reqs[blockIdx.y];
  const int n = blockIdx.x;
  if (n >= n_rows[blockIdx.y] || n >= max_rows) return;
  const uint16_t* xr = x + row_index(rq, rows, n, x_tok) * H;
  uint16_t* yr = y + row_index(rq, rows, n, y_tok) * H;
  const int c0 = threadIdx.x * 8;
  uint4 xv[NC], gv[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = c0 + i * STEP;
    xv[i] = c < H ? *(const uint4*)(xr + c) : make_uint4(0, 0, 0, 0);
    gv[i] = c < H ? *(const uint4*)(gamma + c) : make_uint4(0, 0, 0, 0);
  }
  double ss = 0.0;
  auto add = [&](const uint4& v) {
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double lo = bf16_lo(u[i]), hi = bf16_hi(u[i]);
      ss = __builtin_fma(lo, lo, ss);
      ss = __builtin_fma(hi, hi, ss);
    }
  };
#pragma unroll
  for (int i = 0; i < NC; ++i) add(xv[i]);
  for (int c = c0 + NC * STEP; c < H; c += STEP) add(*(const uint4*)(xr + c));
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = part[0] + part[1] + part[2] + part[3];
  const double inv = 1.0 / sqrt(ss / (double)H + (double)eps);
  auto put = [&](int c, const uint4& v, const uint4& g) {
    const uint32_t u[4] = {v.x, v.y, v.z, v.w}, gw[4] = {g.x, g.y, g.z, g.w};
    uint32_t o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      o[i] = pack_bf16x2((float)((double)bf16_lo(u[i]) * inv * (double)bf16_lo(gw[i])),
                         (float)((double)bf16_hi(u[i]) * inv * (double)bf16_hi(gw[i])));
    *(uint4*)(yr + c) = make_uint4(o[0], o[1], o[2], o[3]);
  };
#pragma unroll
  for (int i = 0; i < NC; ++i)
    if (c0 + i * STEP < H) put(c0 + i * STEP, xv[i], gv[i]);
  for (int c = c0 + NC * STEP; c < H; c += STEP) put(c, *(const uint4*)(xr + c), *(const uint4*)(gamma + c));
}

// ---------------------------------------------------------------------------------------------
// RoPE of the fresh query and key rows of listed tokens, in place.  A workgroup takes 256 / (D / 2)
// listed tokens: each thread forms the cos / sin of one (token, pair) (angle and cos / sin in float64,
// rounded to float32) into LDS, then the threads share the tokens' query and key heads in units of 8
// pairs (float32, no contraction, bf16 store with round to nearest even), consecutive threads on
// consecutive bytes.  Bound by the float64 cos / sin latency for few rows, by HBM for many: 394 rows of
// 32/8/128 7.7 us, 6750 rows 25 us; one thread per (token, 8 pairs) walking all heads took 27 and 42
// (13 workgroups at 394 rows, each thread's 16 float64 cos / sin one after the other).
// ---------------------------------------------------------------------------------------------
template <int D, bool NEOX>
__global__ __launch_bounds__(256) void rope_rows_kernel(const ReqDev* __restrict__ reqs, const int32_t* __restrict__ rows,
                                                        const int32_t* __restrict__ n_rows, int max_rows,
                                                        const int32_t* __restrict__ tok_pos,
                                                        const double* __restrict__ theta, uint16_t* __restrict__ q,
                                                        uint16_t* __restrict__ k, int Hq, int Hkv) {
  constexpr int TB = 256 / (D / 2);   // tokens per workgroup
  constexpr int UPH = D / 16;         // units of 8 pairs per head
  __shared__ __attribute__((aligned(16))) float cs[TB][D / 2], sn[TB][D / 2];
  const ReqDev rq = reqs[blockIdx.y];
  const int n0 = blockIdx.x * TB;
  const int nt = min(TB, min(n_rows[blockIdx.y], max_rows) - n0);   // tokens of this workgroup
  if (nt <= 0) return;
  {
    const int tb = threadIdx.x / (D / 2), p = threadIdx.x % (D / 2);
    const double phi = (double)tok_pos[row_index(rq, rows, n0 + min(tb, nt - 1), true)] * theta[p];
    cs[tb][p] = (float)cos(phi);
    sn[tb][p] = (float)sin(phi);
  }
  __syncthreads();
  const int per_tok = (Hq + Hkv) * UPH;
  for (int x = threadIdx.x; x < nt * per_tok; x += 256) {
#pragma clang fp contract(off)
    const int tb = x / per_tok;
    const int hu = x - tb * per_tok;
    const int h = hu / UPH, u = hu % UPH;
    const int64_t t = row_index(rq, rows, n0 + tb, true);
    uint16_t* row = h < Hq ? q + (t * Hq + h) * D : k + (t * Hkv + h - Hq) * D;
    float c[8], s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      c[e] = cs[tb][u * 8 + e];
      s[e] = sn[tb][u * 8 + e];
    }
    // pair p = 8u + e: NEOX (p, p + D/2); GPT-J (2p, 2p + 1)
    if constexpr (NEOX) {
      uint4* pa = (uint4*)(row + u * 8);
      uint4* pb = (uint4*)(row + D / 2 + u * 8);
      const uint4 va = *pa, vb = *pb;
      const uint32_t wa[4] = {va.x, va.y, va.z, va.w}, wb[4] = {vb.x, vb.y, vb.z, vb.w};
      uint32_t oa[4], ob[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float a0 = bf16_lo(wa[i]), a1 = bf16_hi(wa[i]), b0 = bf16_lo(wb[i]), b1 = bf16_hi(wb[i]);
        const int e0 = 2 * i, e1 = 2 * i + 1;
        oa[i] = pack_bf16x2(a0 * c[e0] - b0 * s[e0], a1 * c[e1] - b1 * s[e1]);
        ob[i] = pack_bf16x2(b0 * c[e0] + a0 * s[e0], b1 * c[e1] + a1 * s[e1]);
      }
      *pa = make_uint4(oa[0], oa[1], oa[2], oa[3]);
      *pb = make_uint4(ob[0], ob[1], ob[2], ob[3]);
    } else {
      uint4* pp = (uint4*)(row + u * 16);
      const uint4 v0 = pp[0], v1 = pp[1];
      const uint32_t w[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
      uint32_t o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x1 = bf16_lo(w[e]), x2 = bf16_hi(w[e]);
        o[e] = pack_bf16x2(x1 * c[e] - x2 * s[e], x2 * c[e] + x1 * s[e]);
      }
      pp[0] = make_uint4(o[0], o[1], o[2], o[3]);
      pp[1] = make_uint4(o[4], o[5], o[6], o[7]);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// SwiGLU activation of listed rows (slot-indexed): gu row = [gate (f) | up (f)] -> y row (f).
// silu(g) = g / (1 + e^-g) in float32.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void silu_mul_rows_kernel(const ReqDev* __restrict__ reqs,
                                                            const int32_t* __restrict__ n_rows, int max_rows,
                                                            const uint16_t* __restrict__ gu, int f,
                                                            uint16_t* __restrict__ y) {
  const ReqDev rq = reqs[blockIdx.y];
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int upr = f / 8;
  const int64_t n = g / upr;
  const int c = (int)(g - n * upr) * 8;
  if (n >= n_rows[blockIdx.y] || n >= max_rows) return;
  const int64_t row = (int64_t)rq.tok_off + n;
  const uint4 gv = *(const uint4*)(gu + row * 2 * f + c);
  const uint4 uv = *(const uint4*)(gu + row * 2 * f + f + c);
  const uint32_t gw[4] = {gv.x, gv.y, gv.z, gv.w}, uw[4] = {uv.x, uv.y, uv.z, uv.w};
  uint32_t o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float g0 = bf16_lo(gw[i]), g1 = bf16_hi(gw[i]);
    const float s0 = g0 / (1.0f + expf(-g0)), s1 = g1 / (1.0f + expf(-g1));
    o[i] = pack_bf16x2(s0 * bf16_lo(uw[i]), s1 * bf16_hi(uw[i]));
  }
  *(uint4*)(y + row * f + c) = make_uint4(o[0], o[1], o[2], o[3]);
}

}  // namespace

template <int BN, int BM, int WN, int WM, int NST>
static hipError_t launch_gemm_tiles(GemmRowsK& a, hipStream_t s) {
  a.m_tiles = (a.max_rows + BM - 1) / BM;
  const int64_t tiles = (int64_t)a.m_tiles * a.n_req * (a.N / BN);
  const int64_t blocks = (tiles + kGemmXcds - 1) / kGemmXcds * kGemmXcds;
  hipLaunchKernelGGL((gemm_rows_kernel<BN, BM, WN, WM, NST>), dim3((unsigned)blocks), dim3(WN * WM * 64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_gemm_rows(const sx_plan* p, const RowsArg& r, const void* x, int x_tok, const void* w, int k,
                            int n_parts, const int* part_n, void* const* ys, const void* res, int y_tok, hipStream_t s) {
  if (n_parts < 1 || n_parts > kGemmMaxParts) return hipErrorInvalidValue;
  GemmRowsK a{};
  a.reqs = p->d_req;
  a.rows = r.rows;
  a.n_rows = r.n_rows;
  a.x = (const uint16_t*)x;
  a.w = (const uint16_t*)w;
  a.res = (const uint16_t*)res;
  a.n_parts = n_parts;
  int n = 0;
  for (int i = 0; i < n_parts; ++i) {
    a.y[i] = (uint16_t*)ys[i];
    a.pn[i] = n;
    n += part_n[i];
  }
  a.pn[n_parts] = n;
  a.K = k;
  a.N = n;
  a.n_req = p->n_req;
  a.max_rows = r.max_rows;
  a.x_tok = x_tok;
  a.y_tok = y_tok;
  // The tile whose rounds over the compute units take least: a workgroup per compute unit, and one
  // 64-wide piece of k costs a round about 1.5 us on 256 x 256 tiles, 0.95 on 256 x 128, 0.60 on
  // 128 x 128, 0.46 on 128 x 64 and 0.35 on 64 x 64 (measured, K = 4096, weights from HBM; bound by the
  // LDS reads and transfers between barriers on all but the largest).  So wide products keep the large
  // tile and few rows take the one that gives every compute unit a tile: the rows' count at which two
  // neighbours cross depends on the width.  Measured for 384 rows (start: 256 x 256 always), K = 4096:
  // N = 6144 39 us (101), 4096 30 us (110); K = 14336: N = 4096 95 us (340).
  struct Shape {
    int bn, bm;
    double cost;
  };
  static const Shape shapes[] = {{256, 256, 1.5}, {256, 128, 0.95}, {128, 128, 0.60}, {128, 64, 0.46}, {64, 64, 0.35}};
  int best = 0;
  double best_cost = 0;
  for (int i = 0; i < 5; ++i) {
    const int64_t tiles = (int64_t)((r.max_rows + shapes[i].bm - 1) / shapes[i].bm) * p->n_req * (n / shapes[i].bn);
    const double cost = (double)((tiles + p->n_cu - 1) / p->n_cu) * shapes[i].cost;
    if (i == 0 || cost < 0.98 * best_cost) {
      best = i;
      best_cost = cost;
    }
  }
  switch (best) {
    case 0: return launch_gemm_tiles<256, 256, 4, 2, 2>(a, s);
    case 1: return launch_gemm_tiles<256, 128, 4, 2, 3>(a, s);
    case 2: return launch_gemm_tiles<128, 128, 4, 2, 4>(a, s);
    case 3: return launch_gemm_tiles<128, 64, 4, 2, 4>(a, s);
    default: return launch_gemm_tiles<64, 64, 2, 2, 4>(a, s);
  }
}

hipError_t launch_rmsnorm_rows(const sx_plan* p, const RowsArg& r, const void* x, int x_tok, const void* gamma,
                               float eps, int h, void* y, int y_tok, hipStream_t s) {
  const dim3 grid((unsigned)r.max_rows, (unsigned)p->n_req);
  hipLaunchKernelGGL(rmsnorm_rows_kernel, grid, dim3(256), 0, s, p->d_req, r.rows, r.n_rows, r.max_rows, (const uint16_t*)x, x_tok,
                     (const uint16_t*)gamma, eps, h, (uint16_t*)y, y_tok);
  return hipGetLastError();
}

hipError_t launch_rope_rows(const sx_plan* p, const RowsArg& r, void* q, void* k, hipStream_t s) {
  const int D = p->desc.head_dim;
  const int tb = 256 / (D / 2);   // tokens per workgroup
  const dim3 grid((unsigned)((r.max_rows + tb - 1) / tb), (unsigned)p->n_req);
  const bool neox = p->desc.rope_style == SX_ROPE_NEOX;
  const int Hq = p->desc.n_q_heads, Hkv = p->desc.n_kv_heads;
#define SX_ROPE(D_, N_)                                                                                               \
  hipLaunchKernelGGL((rope_rows_kernel<D_, N_>), grid, dim3(256), 0, s, p->d_req, r.rows, r.n_rows, r.max_rows, p->d_tok_pos,   \
                     p->d_theta, (uint16_t*)q, (uint16_t*)k, Hq, Hkv)
  if (D == 128) {
    if (neox) SX_ROPE(128, true); else SX_ROPE(128, false);
  } else {
    if (neox) SX_ROPE(64, true); else SX_ROPE(64, false);
  }
#undef SX_ROPE
  return hipGetLastError();
}

hipError_t launch_silu_mul_rows(const sx_plan* p, const RowsArg& r, const void* gu, int f, void* y, hipStream_t s) {
  const int64_t threads = (int64_t)r.max_rows * (f / 8);
  const dim3 grid((unsigned)((threads + 255) / 256), (unsigned)p->n_req);
  hipLaunchKernelGGL(silu_mul_rows_kernel, grid, dim3(256), 0, s, p->d_req, r.n_rows, r.max_rows, (const uint16_t*)gu, f,
                     (uint16_t*)y);
  return hipGetLastError();
}

}  // namespace sx
