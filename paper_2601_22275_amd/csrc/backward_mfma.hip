// bf16 MFMA kernels for the backward of one blocked-softmax pass with entropy (App. "Backward
// pass of Flash-Entropy-Attention", Alg. 2) on gfx950, d = 64 or 128.
//
// Alg. 2 adds into dQ in HBM from every key block.  Here the three results are produced by
// two passes that accumulate nothing across workgroups (bit-reproducible):
//   dQ pass:     a workgroup owns query rows and streams the frame's K and V tiles;
//   dK, dV pass: a workgroup owns key rows and streams the frame's Q and dO tiles; P and dS of a
//                tile pair are formed once and feed both products.
// Both are one kernel template.  The "owner" rows (32 per wave) stay in registers as B
// operands for the whole loop; the "stream" rows pass through LDS in 64-row tiles exactly as
// in the forward kernel (same direct global -> LDS loads, same swizzle, same transpose reads):
//   G^T  = X1 R1^T         rows = stream rows, columns = owner rows; lane owns one owner row
//   dP^T = X2 R2^T
//   E    = elementwise     P = exp(S - L), dS = P (dP - D) - dH P (S - L + H)   (Alg. 2)
//   acc^T += Xa^T E        B = E converted to bf16 in place, A = Xa^T by LDS transpose reads
// Per query row the elementwise step needs sc (logit scale), L, D, dH, H, reduced to four
// floats per row, {sc2, l2, a, b} with t = S_raw sc2 - l2 (log2 units), P = 2^t and
// dS = P (dP - a - b t):  a = D + dH H,  b = dH ln 2.  The dQ pass, which runs first, forms them
// (D from the dO rows it holds anyway) as per-lane scalars and stores them for the other.  In the dK, dV
// pass the stream rows are queries, and a lane needs the values of 16 of them per 32-row sub-tile: they
// travel with the Q tile as one LDS array per statistic, read four rows at a time.  Such a read costs as
// much LDS time as the operand of an MFMA, and LDS is the narrowest path here (an MFMA's worth of operand
// per MFMA already).  Without dH and c_R (row scale the same for all rows) sc2 and b are constants, two of
// the four arrays and a third of the vector arithmetic drop out: that is the PLAIN form.
// Measured inside back-to-back calls, three passes and a statistics kernel -> two passes: 12 x 21 frames of 1560, d =
// 128, plain form: dQ 506 -> 462 us (1019 TFLOP/s issued), dV + dK 381 + 608 -> 603 us (1042 TFLOP/s), statistics 36 us
// -> inside dQ; 10 x 9 frames of 943, d = 64, general form: 57 + 53 + 67 + 7 -> 42 + 60 us (739, 684 TFLOP/s).  At d =
// 128 the matrix pipes are busy for 0.54 of the cycles and two waves per SIMD (all that the registers allow) do not
// fill the rest; a large library product reaches 1150 TFLOP/s.  At d = 64 vector work per score weighs twice as much.
#include <type_traits>

#include "common.h"
#include "flash_select.h"

namespace vm {

namespace {

// Workgroups are NW waves of 32 owner rows: 4 at d = 64, two or three of them on a compute unit, 4 or 8 at d = 128.  Smaller blocks leave less of the
// last block and the last round idle and hide each other's start and end (all gradients, d = 64, eight -> four waves: 90 frames
// of 943 131 -> 114 us, 252 of 1560 722 -> 667, 128 of 512 level).  At d = 128 two workgroups leave LDS for tiles of 32 stream rows, a
// barrier for every 32 rows: which launch takes which: flash_select.h.
template <int D, int NW>
constexpr int tile_rows() {  // stream rows per LDS tile
  return D == 128 && NW == 4 ? 32 : 64;
}
constexpr int NSLOT = 3;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

enum { MODE_DQ = 0, MODE_DKV = 1, MODE_DKV_PLAIN = 2 };

struct BwdParams {
  const bf16_t* q;
  const bf16_t* k;
  const bf16_t* v;
  const bf16_t* dO;
  const bf16_t* o;       // the forward result, and per query row:
  const float* cR;       // may be null (= 1)
  const float* lse;
  const float* H;
  const float* dH;       // may be null (= 0)
  float4* stats;         // {sc2, l2, a, b}: written by the dQ pass, read by the dK, dV pass
  bf16_t* out;           // dq or dk
  bf16_t* out_v;         // dv
  int n;                 // rows per problem (b): owner rows and stream rows alike
  int nob;               // owner blocks per problem
  int total_blocks;
  int blocks_per_xcd;
  float row_scale;
  float cr_min;
};

__device__ __forceinline__ bf16x8 lds_read_b128(const char* p) { return *reinterpret_cast<const bf16x8*>(p); }
__device__ __forceinline__ bf16x4 lds_read_tr(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
      (bf16x4 __attribute__((address_space(3)))*)(reinterpret_cast<const bf16x4*>(p)));
}
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
  bf16x2 r;
  r[0] = (__bf16)a;
  r[1] = (__bf16)b;
  uint32_t u;
  __builtin_memcpy(&u, &r, 4);
  return u;
}

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

template <int D, int MODE, int NW>
constexpr int own_in_lds() {
  return D != 128 || MODE == MODE_DQ ? 0 : MODE == MODE_DKV ? 2 : NW == 4 ? 4 : 0;
}

template <int D, int MODE, int NW>
__global__ void __launch_bounds__(64 * NW, 2) bwd_kernel(BwdParams P) {
  using G = RowGeo<D>;
  constexpr int BK = tile_rows<D, NW>();
  constexpr int SR = 64;                              // floats of a tile's array of statistics (a wave's load fills 64)
  constexpr int BO = 32 * NW;
  constexpr int ROW_BYTES = G::ROW_BYTES;
  constexpr int TILE_BYTES = BK * ROW_BYTES;
  constexpr int SLOT_BYTES = 2 * TILE_BYTES;         // X1 tile, then X2 tile
  constexpr int KS = G::KS;
  constexpr int CT = G::CT;
  constexpr int CH = G::CH;
  constexpr int RPI = G::RPI;
  constexpr bool DKV = MODE != MODE_DQ;               // stream rows are queries
  constexpr bool PLAIN = MODE == MODE_DKV_PLAIN;
  constexpr int NST = !DKV ? 0 : PLAIN ? 2 : 4;      // arrays of stream statistics: l2, a (, sc2, b)
  constexpr int STATS_OFF = NSLOT * SLOT_BYTES;      // [NSLOT][NST][SR] floats
  constexpr int STATS_SLOT = NST * SR * 4;
  constexpr int NACC = DKV ? 2 : 1;                   // accumulator sets: [dQ or dK][dV]
  constexpr bool TIGHT = DKV && D == 128;             // the registers are just enough
  constexpr int NG = 2 * KS;                          // MFMAs of G^T and dP^T
  // The dK, dV pass at d = 128 just fills a wave's 256 registers (64 of owner rows, 128 of accumulators, 32 of logits); with
  // the general statistics in flight, or tiles of 32 rows, it is a few short, and the last NL k-steps of the second owner
  // tensor wait in LDS, private to the wave.  (One spilled operand instead waits, in order, behind the tile just requested:
  // 252 frames of 1536 1035 us instead of 1011.)
  constexpr int NL = own_in_lds<D, MODE, NW>();
  constexpr int OWN_OFF = STATS_OFF + NSLOT * STATS_SLOT;  // [NW][NL][64 lanes] 16 bytes
  auto swz = [](int row) { return G::swz(row); };
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int bid = blockIdx.x;
  const int wid = (bid & 7) * P.blocks_per_xcd + (bid >> 3);  // XCD-aware, as in the forward kernel
  if (wid >= P.total_blocks) return;
  const int prob = wid / P.nob;
  const int ob = wid - prob * P.nob;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int ql = lane & 31;
  const int g = lane >> 5;
  const int n = P.n;
  const int ntiles = (n + BK - 1) / BK;
  const long long row0 = (long long)prob * n;  // first row of the problem in every tensor

  // owner / stream tensors of this pass
  const bf16_t* r1 = (DKV ? P.k : P.q) + row0 * D;   // B of G^T
  const bf16_t* r2 = (DKV ? P.v : P.dO) + row0 * D;  // B of dP^T
  const bf16_t* x1 = (DKV ? P.q : P.k) + row0 * D;   // A of G^T; A^T of dQ (dK)
  const bf16_t* x2 = (DKV ? P.dO : P.v) + row0 * D;  // A of dP^T; A^T of dV
  const float4* stats = P.stats + row0;

  // ---- stream tiles: global -> LDS, as in the forward kernel --------------------------------
  static_assert(BK % (RPI * NW) == 0, "every wave issues the same number of loads per tile");
  // A tile's address is a wave-uniform base, a lane's place in it a 32-bit offset.
  const unsigned lds_base = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)smem;
  auto issue_tile = [&](int t) __attribute__((always_inline)) {
    const unsigned kb = lds_base + (t % NSLOT) * SLOT_BYTES;
    const bf16_t* s1 = x1 + (long long)t * BK * D;
    const bf16_t* s2 = x2 + (long long)t * BK * D;
    // the lane's place, derived anew for every tile where registers are short (opaque copy)
    int tid_i = tid;
    if (TIGHT) asm volatile("" : "+v"(tid_i));
    const int lane_i = tid_i & 63;
    const int st_row = RPI * wave + lane_i / CH;  // + RPI NW r
    const int st_lc = (lane_i % CH) ^ swz(st_row);
    const int last = n - 1 - t * BK;  // rows past the end: copies of the last one, weight zero below
#pragma unroll
    for (int r = 0; r < BK / (RPI * NW); ++r) {
      const unsigned off = (unsigned)(min(RPI * NW * r + st_row, last) * ROW_BYTES + st_lc * 16);
      const unsigned dst = __builtin_amdgcn_readfirstlane(kb + (RPI * NW * r + RPI * wave) * ROW_BYTES);
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(s1), "s"(dst) : "memory", "m0");
      const unsigned dst2 = dst + TILE_BYTES;
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(s2), "s"(dst2) : "memory", "m0");
    }
    if (DKV && wave < NST) {
      // wave w fetches statistic w of the tile's 64 query rows, one float per lane
      const float* s3 = reinterpret_cast<const float*>(stats + (long long)t * BK) + (wave == 0 ? 1 : wave == 1 ? 2 : wave == 2 ? 0 : 3);
      const unsigned off = (unsigned)(min(lane_i, last) * 16);
      const unsigned dst3 = __builtin_amdgcn_readfirstlane(lds_base + STATS_OFF + (t % NSLOT) * STATS_SLOT + wave * (SR * 4));
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" : : "v"(off), "s"(s3), "s"(dst3) : "memory", "m0");
    }
  };
  issue_tile(0);
  if (ntiles > 1) issue_tile(1);

  // ---- owner rows: B operands in registers -----------------------------------------------
  const int orow_raw = ob * BO + wave * 32 + ql;
  const bool ovalid = orow_raw < n;
  const int orow = ovalid ? orow_raw : n - 1;
  typedef __attribute__((address_space(3))) const bf16x8* lds_b128_ptr;
  typedef __attribute__((address_space(3))) bf16x8* lds_b128_wptr;
  bf16x8 reg1[KS], reg2[KS - NL];
  const unsigned own_base = lds_base + OWN_OFF + (wave * NL * 64 + lane) * 16;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    reg1[ks] = *reinterpret_cast<const bf16x8*>(r1 + (long long)orow * D + 8 * g + 16 * ks);
    const bf16x8 x = *reinterpret_cast<const bf16x8*>(r2 + (long long)orow * D + 8 * g + 16 * ks);
    if (ks < KS - NL) reg2[ks] = x;
    else *(lds_b128_wptr)(unsigned long long)(own_base + (ks - (KS - NL)) * 1024) = x;
  }
  float4 ost = {0.f, 0.f, 0.f, 0.f};        // dQ pass: the owner row is a query
  if (!DKV) {
    // D = dO . O (Alg. 2, before the loops) on the way: dO is here already, each half of the wave holds half of a row
    const bf16_t* op = P.o + (row0 + orow) * D + 8 * g;
    float dot = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 x = *reinterpret_cast<const bf16x8*>(op + 16 * ks);
#pragma unroll
      for (int i = 0; i < 8; ++i) dot = __builtin_fmaf((float)x[i], (float)reg2[DKV ? 0 : ks][i], dot);
    }
    dot += __shfl_xor(dot, 32);
    const float c = fmaxf(P.cR ? P.cR[row0 + orow] : 1.f, P.cr_min);
    const float gh = P.dH ? P.dH[row0 + orow] : 0.f;
    ost.x = P.row_scale / c * LOG2E;
    ost.y = P.lse[row0 + orow] * LOG2E;
    ost.z = dot + gh * P.H[row0 + orow];
    ost.w = gh * LN2;
    if (ovalid && g == 0) P.stats[row0 + orow] = ost;
  }
  if (PLAIN) ost = stats[0];                // .x is the same for every row, .w is zero

  // LDS byte addresses of a sub-tile's operands, relative to its first row in the X1 tile.  Row reads (A of G^T, dP^T):
  // row ql, logical chunk 2 ks + g; transpose reads: rows 8 hh + 4 g + rp / 4, logical chunk 4 ct + ...  The chunk
  // index only ever enters through XOR, so one base serves all ks (ct): base ^ (ks << 5), base ^ (ct << 6).
  const unsigned a_base = lds_base + ql * ROW_BYTES + ((g ^ swz(ql)) << 4);
  unsigned t_base[2];
  {
    const int rp = lane & 15;
    const int chh = (lane >> 4) & 1;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int row = 8 * hh + 4 * g + (rp >> 2);
      const int lc = 2 * chh + ((rp >> 1) & 1);
      t_base[hh] = lds_base + row * ROW_BYTES + ((lc ^ swz(row)) << 4) + ((rp & 1) << 3);
    }
  }
  typedef __attribute__((address_space(3))) bf16x4* lds_b64_ptr;
  typedef __attribute__((address_space(3))) const f32x4* lds_f32x4_ptr;
  auto rd_row = [&](unsigned addr) __attribute__((always_inline)) -> bf16x8 { return *(lds_b128_ptr)(unsigned long long)addr; };
  auto rd_tr = [&](unsigned lo, unsigned hi) __attribute__((always_inline)) -> bf16x8 {
    const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b64_ptr)(unsigned long long)lo);
    const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b64_ptr)(unsigned long long)hi);
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  auto rd_stat = [&](unsigned addr) __attribute__((always_inline)) -> f32x4 { return *(lds_f32x4_ptr)(unsigned long long)addr; };

  f32x16 acc[NACC][CT];
#pragma unroll
  for (int x = 0; x < NACC; ++x)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][ct][r] = 0.f;
  constexpr int NOP = NG + 2 * CT * NACC;  // MFMAs (and A operands) of a sub-tile: G, dP, then the products
  constexpr int PF = TIGHT ? 2 : 3;
  const bool active = ob * BO + wave * 32 < n;  // a wave whose owner rows are all padding only loads tiles

  // ---- one 32-row sub-tile of the stream ---------------------------------------------------
  // slot: byte offset of the tile's slot; sslot: of its statistics, from lds_base, the lane's first row included
  auto step = [&](unsigned slot, unsigned sslot, auto st_c, int rows_left) __attribute__((always_inline)) {
    constexpr int ST = decltype(st_c)::value;
    constexpr int SUB = ST * 32 * ROW_BYTES;
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = 0.f; }
    // The operands pass through a ring of four, requested PF ahead of their MFMA and no earlier (the fences): left to
    // itself the compiler requests a whole product's operands at once, which at d = 128 (64 registers of owner rows and
    // 128 of accumulators out of 256 in the dK, dV pass) spills the owner rows into the loop.
    // (opaque copies where registers are short: address terms are not kept across sub-tiles)
    unsigned ab = a_base + slot, tb0 = t_base[0] + slot, tb1 = t_base[1] + slot;
    if (TIGHT) asm volatile("" : "+v"(ab), "+v"(tb0), "+v"(tb1));
    bf16x8 ring[4], own[NL > 0 ? NL : 1];
    auto request = [&](auto ic) __attribute__((always_inline)) {
      constexpr int I = decltype(ic)::value;
      if constexpr (I < KS) {
        ring[I & 3] = rd_row((ab ^ (I << 5)) + SUB);
      } else if constexpr (I < NG) {
        ring[I & 3] = rd_row((ab ^ ((I - KS) << 5)) + SUB + TILE_BYTES);
        if constexpr (I >= NG - NL) own[I - (NG - NL)] = rd_row(own_base + (I - (NG - NL)) * 1024);
      } else if constexpr (I < NOP) {
        constexpr int c = (I - NG) / (CT * NACC), ct = (I - NG) / NACC % CT, x = (NACC - 1) - (I - NG) % NACC;  // dV first: P is there before dS
        constexpr int off = SUB + c * 16 * ROW_BYTES + (x == 1 ? TILE_BYTES : 0);
        ring[I & 3] = rd_tr((tb0 ^ (ct << 6)) + off, (tb1 ^ (ct << 6)) + off);
      }
    };
    static_for<0, PF>(request);
    static_for<0, NG>([&](auto ic) __attribute__((always_inline)) {
      constexpr int I = decltype(ic)::value;
      request(std::integral_constant<int, I + PF>{});
      if constexpr (I < KS) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[I & 3], reg1[I], s, 0, 0, 0);
      else if constexpr (I >= NG - NL) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[I & 3], own[I - (NG - NL)], dp, 0, 0, 0);
      else dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[I & 3], reg2[I - KS], dp, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    });
    // elementwise: register r is stream row 8 (r / 4) + 4 g + (r % 4) of the sub-tile
    bf16x8 pb[2], eb[2];  // P, dS
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      f32x4 l2 = {ost.y, ost.y, ost.y, ost.y}, av = {ost.z, ost.z, ost.z, ost.z};
      f32x4 sc2 = {ost.x, ost.x, ost.x, ost.x}, bv = {ost.w, ost.w, ost.w, ost.w};
      if (DKV) {
        const unsigned sa = sslot + (32 * ST + 8 * r4) * 4;
        l2 = rd_stat(sa);
        av = rd_stat(sa + SR * 4);
        if (!PLAIN) {
          sc2 = rd_stat(sa + 2 * SR * 4);
          bv = rd_stat(sa + 3 * SR * 4);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 4 * r4 + i;
        const float t = __builtin_fmaf(s[r], sc2[i], -l2[i]);
        const float p = __builtin_amdgcn_exp2f(t);
        if (DKV) pb[r >> 3][r & 7] = (__bf16)p;
        float ds = PLAIN ? p * (dp[r] - av[i]) : p * (dp[r] - av[i] - bv[i] * t);
        if (DKV && !PLAIN) ds *= sc2[i] * (1.0f / LOG2E);  // dK carries the query's logit scale
        eb[r >> 3][r & 7] = (__bf16)ds;
      }
      if (TIGHT || NST == 4 && (r4 & 1)) __builtin_amdgcn_sched_barrier(0);  // no more than half of the statistics in flight
    }
    if (rows_left < 32) {
      // ragged end of the stream: rows rows_left .. 31 are copies of the last row and get weight zero
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + 4 * g + (r & 3) >= rows_left) {
          if (DKV) pb[r >> 3][r & 7] = (__bf16)0.0f;
          eb[r >> 3][r & 7] = (__bf16)0.0f;
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    static_for<NG, NOP>([&](auto ic) __attribute__((always_inline)) {
      constexpr int I = decltype(ic)::value;
      constexpr int c = (I - NG) / (CT * NACC), ct = (I - NG) / NACC % CT, x = (NACC - 1) - (I - NG) % NACC;  // dV first: P is there before dS
      request(std::integral_constant<int, I + PF>{});
      if constexpr (x == 1) acc[x][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[I & 3], pb[c], acc[x][ct], 0, 0, 0);
      else acc[x][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[I & 3], eb[c], acc[0][ct], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // Tile t sits in slot t mod 3 and is requested two iterations ahead; the barrier at the top
  // of iteration t publishes it (every wave has waited for its own part) and retires tile t-1, whose slot
  // tile t+2 takes.
  for (int t = 0; t < ntiles; ++t) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t + 2 < ntiles) issue_tile(t + 2);
    if (active) {
      const unsigned slot = (t % NSLOT) * SLOT_BYTES;
      const unsigned sslot = lds_base + STATS_OFF + (t % NSLOT) * STATS_SLOT + 16 * g;
      const int left = n - t * BK;
      step(slot, sslot, std::integral_constant<int, 0>{}, left);
      if constexpr (BK == 64) step(slot, sslot, std::integral_constant<int, 1>{}, left - 32);
    }
  }

  // ---- epilogue: rows staged in LDS, written as whole lines ---------------------------------
  __syncthreads();
  // lane-dependent values derived again behind an opaque copy, so that none of them stays live across the loop
  int tid_e = threadIdx.x;
  asm volatile("" : "+v"(tid_e));
  const int lane_e = tid_e & 63;
  const int ql_e = lane_e & 31;
  const int g_e = lane_e >> 5;
  const float oscale = DKV && !PLAIN ? 1.0f : ost.x * (1.0f / LOG2E);  // dq (and dk in the plain form) carry the logit scale
  const int row_first = ob * BO + wave * 32;
  char* stage = smem + wave * (32 * ROW_BYTES);
  static_assert(NW * 32 * ROW_BYTES <= NSLOT * SLOT_BYTES, "staged rows fit the tile slots");
#pragma unroll
  for (int x = 0; x < NACC; ++x) {
    const float f = x == 1 ? 1.0f : oscale;
    bf16_t* dst = x == 1 ? P.out_v : P.out;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        uint2 w;
        w.x = pack_bf16(acc[x][ct][4 * c + 0] * f, acc[x][ct][4 * c + 1] * f);
        w.y = pack_bf16(acc[x][ct][4 * c + 2] * f, acc[x][ct][4 * c + 3] * f);
        *reinterpret_cast<uint2*>(stage + ql_e * ROW_BYTES + (((4 * ct + c) ^ swz(ql_e)) << 4) + 8 * g_e) = w;
      }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the staged rows are private to the wave
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int ps = 0; ps < 32 / RPI; ++ps) {
      const int lr = ps * RPI + lane_e / CH;
      const int pc = lane_e % CH;
      const int lc = pc ^ swz(lr);
      const uint4 w = *reinterpret_cast<const uint4*>(stage + lr * ROW_BYTES + pc * 16);
      if (row_first + lr < n) *reinterpret_cast<uint4*>(dst + (row0 + row_first + lr) * D + lc * 8) = w;
    }
    __builtin_amdgcn_wave_barrier();  // the next set is staged over these rows
  }
}

template <int D, int MODE, int NW>
hipError_t launch_bwd(BwdParams P, long long problems, hipStream_t st) {
  constexpr int LDS_BYTES = 2 * NSLOT * tile_rows<D, NW>() * D * 2 + NSLOT * 64 * 16 + NW * own_in_lds<D, MODE, NW>() * 1024;
  P.nob = (P.n + 32 * NW - 1) / (32 * NW);
  const long long total = problems * P.nob;
  if (total > 0x3fffffffLL) return hipErrorInvalidValue;
  P.total_blocks = (int)total;
  P.blocks_per_xcd = (P.total_blocks + 7) / 8;
  auto kern = bwd_kernel<D, MODE, NW>;
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
    if (e != hipSuccess) return e;
    configured = true;
  }
  hipLaunchKernelGGL(kern, dim3(P.blocks_per_xcd * 8), dim3(64 * NW), LDS_BYTES, st, P);
  return hipGetLastError();
}

}  // namespace

bool entropy_bwd_mfma_supported(const Dims& dm) { return dm.d == 128 || dm.d == 64; }
size_t entropy_bwd_mfma_scratch_bytes(const Dims& dm) { return (size_t)dm.BH * dm.N * sizeof(float4); }

hipError_t launch_entropy_bwd_mfma(const bf16_t* q, const float* cR, const bf16_t* k, const bf16_t* v,
                                   const bf16_t* o, const bf16_t* dO, const float* lse, const float* H,
                                   const float* dH, bf16_t* dq, bf16_t* dk, bf16_t* dv, void* scratch, const Dims& dm,
                                   float row_scale, float cr_min, hipStream_t st) {
  const long long rows = (long long)dm.BH * dm.N;
  if (rows > 0x7fffffffLL) return hipErrorInvalidValue;
  BwdParams P = {};
  P.q = q; P.k = k; P.v = v; P.dO = dO;
  P.o = o; P.cR = cR; P.lse = lse; P.H = H; P.dH = dH; P.stats = (float4*)scratch;
  P.row_scale = row_scale; P.cr_min = cr_min;
  P.n = dm.b;
  const long long problems = (long long)dm.BH * dm.T;
  const bool plain = cR == nullptr && dH == nullptr;
  auto run = [&](auto dc, auto wc) -> hipError_t {
    constexpr int D = decltype(dc)::value, NW = decltype(wc)::value;
    P.out = dq;
    hipError_t e2 = launch_bwd<D, MODE_DQ, NW>(P, problems, st);
    if (e2 != hipSuccess) return e2;
    P.out = dk;
    P.out_v = dv;
    return plain ? launch_bwd<D, MODE_DKV_PLAIN, NW>(P, problems, st) : launch_bwd<D, MODE_DKV, NW>(P, problems, st);
  };
  using four = std::integral_constant<int, 4>;
  if (dm.d == 64) return run(std::integral_constant<int, 64>{}, four{});
  if (backward_short_blocks(problems, dm.b, compute_units())) return run(std::integral_constant<int, 128>{}, four{});
  return run(std::integral_constant<int, 128>{}, std::integral_constant<int, 8>{});
}

}  // namespace vm
