// float32 kernels for spatio-temporal Monarch attention on the matrix cores of gfx950, d = 32, 64 or 128: every
// blocked-softmax pass (R-update with its statistics, exact attention of chosen rows, sink averaging) and the temporal
// factor for up to 32 frames.  v_mfma_f32_32x32x2_f32 multiplies and accumulates in fp32 (one rounding per product and
// sum, like an FMA), so results carry no less precision than the plain-ALU kernels' (generic.hip), whose exp and log
// functions are used here too.
//
// Bound by the fp32 matrix rate (256 FLOP per clock and CU: 64 cycles per 32x32x2 MFMA); the softmax of a 32x32 tile is
// 16 exponentials per lane against 4096 .. 12288 cycles of MFMA, so nothing is pipelined by hand.
//   S^T[key, q] = K Q^T      lane (q = lane & 31, g = lane >> 5) ends with the logits of query q for keys
//                            8 (r >> 2) + 4 g + (r & 3): max, sum and entropy are per-lane sums plus one exchange with
//                            lane ^ 32
//   O^T[ch, q] += X^T P^T    register r of P^T is the B operand as it stands: the two k-slots of the MFMA (g = 0, 1) then
//                            mean keys 8 (r >> 2) + (r & 3) and 4 more, and the A operand is one float per lane of just
//                            these two rows of X
// A contraction may visit its index in any order, which is what makes both operand layouts free of shuffles; the rows
// of a 32-key tile sit in LDS with 16 bytes of padding, so row reads (16 bytes per lane) and channel reads (4 bytes per
// lane) spread over all banks.
//
// 4 heads x 8 frames of 15 x 26, d = 64 (two sweeps and the first frame): 2.07 ms on the plain-ALU kernels, 0.106 ms here.
// Calls with very few keys stay on those (f32_select.h).
#include <type_traits>

#include "common.h"
#include "f32_select.h"

namespace vm {

namespace {

constexpr int BT = kF32Tile;            // query rows of a tile, key rows of a tile, frames of a position
constexpr int WAVES = kF32Waves;        // waves per workgroup of the blocked-softmax kernel
constexpr float F32_LOWEST = -3.0e38f;  // reference of a row that has seen no key yet

struct F32Params {
  const float* q;
  const float* cR;       // per query row, null: 1
  const float* k;
  const float* v;
  float* outk;           // softmax(z) K
  float* outv;           // softmax(z) V
  float* cl;             // sum p log p
  float* lse;            // null: not wanted
  float* part_o;         // key ranges: [range][problem][nq][D] sums relative to the range's reference
  float2* part_ms;       // ... and its {reference, sum of weights}
  const int* q_index;    // null, or the row numbers of the query rows; entries outside [0, q_limit) are skipped
  long long q_rows_per_problem, k_rows_per_problem, q_limit;
  int nq, nk;
  int nqt;               // query tiles per problem
  int nsplit;            // key ranges per query tile
  int tiles_per_split;
  int nproblems;
  int total;             // nproblems * nqt * nsplit items
  int groups_per_xcd;    // workgroups per XCD
  float row_scale, cr_min;
  int blend;             // outv <- (outv + result) / 2
};

__device__ __forceinline__ f32x16 mfma(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// LDS traffic between the lanes of one wave: DS operations of a wave complete in order, the compiler must not reorder them
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// KW waves share a query tile and take every KW-th key tile each (their sums meet in the epilogue); a workgroup holds
// WAVES / KW query tiles.
template <int D, bool OUT_K, bool OUT_V, int KW>
__global__ void __launch_bounds__(64 * WAVES) f32_attend_kernel(F32Params P) {
  constexpr int RS = D + 4;                // floats per LDS row
  constexpr int AREA = BT * RS;            // one tile of one tensor
  constexpr int NX = (OUT_K ? 1 : 0) + (OUT_V ? 1 : 0);
  constexpr int WAVE_FLOATS = (OUT_V ? 2 : 1) * AREA;  // K tile, V tile
  constexpr int NL = D / 8;                // 16-byte loads per lane and tile
  constexpr int RPL = 64 / (D / 4);        // rows per load instruction (8, 4, 2)
  constexpr int CT = D / 32;
  constexpr int XV = OUT_K ? 1 : 0;
  extern __shared__ __attribute__((aligned(16))) float sm[];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int ql = lane & 31;
  const int g = lane >> 5;
  const int kw = wave % KW;
  float* Ks = sm + wave * WAVE_FLOATS;
  float* Vs = Ks + (OUT_V ? AREA : 0);
  float* stat = sm + WAVES * WAVE_FLOATS;  // [WAVES][3][32]: reference, sum, entropy sum

  // XCD-aware: each XCD gets one contiguous range of items, whose query tiles share K and V in its L2
  const int grp = (blockIdx.x & 7) * P.groups_per_xcd + (blockIdx.x >> 3);
  const int item = grp * (WAVES / KW) + wave / KW;
  const bool active = item < P.total;
  const int it = active ? item : 0;
  const int prob = it / (P.nqt * P.nsplit);
  const int rem = it - prob * (P.nqt * P.nsplit);
  const int split = rem / P.nqt;
  const int qt = rem - split * P.nqt;
  const int all_tiles = (P.nk + BT - 1) / BT;
  const int t_end = active ? min(all_tiles, (split + 1) * P.tiles_per_split) : 0;
  int t = split * P.tiles_per_split + kw;

  const float* kb = P.k + (long long)prob * P.k_rows_per_problem * D;
  const float* vb = OUT_V ? P.v + (long long)prob * P.k_rows_per_problem * D : nullptr;
  f32x4 rk[NL], rv[OUT_V ? NL : 1];  // (HIP's float4 in these arrays would live in scratch memory)
  const int ld_row = lane / (D / 4);
  const int ld_col = (lane % (D / 4)) * 4;
  auto load = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const long long row = min(tile * BT + i * RPL + ld_row, P.nk - 1);  // rows past the end: copies, weight zero below
      rk[i] = *reinterpret_cast<const f32x4*>(kb + row * D + ld_col);
      if (OUT_V) rv[i] = *reinterpret_cast<const f32x4*>(vb + row * D + ld_col);
    }
    if (OUT_V && tile * BT + BT > P.nk) {
      // ... whose values are zeros: an infinite value of the last row times weight zero would be NaN
#pragma unroll
      for (int i = 0; i < NL; ++i)
        if (tile * BT + i * RPL + ld_row >= P.nk) rv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  auto to_lds = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      *reinterpret_cast<f32x4*>(Ks + (i * RPL + ld_row) * RS + ld_col) = rk[i];
      if (OUT_V) *reinterpret_cast<f32x4*>(Vs + (i * RPL + ld_row) * RS + ld_col) = rv[i];
    }
  };
  if (t < t_end) load(t);

  // query rows: B operand of S^T, channels 8 j + 4 g + c
  const int qr = qt * BT + ql;
  long long qrow = min(qr, P.nq - 1);
  bool qvalid = active && qr < P.nq;
  if (P.q_index != nullptr) {
    const long long x = P.q_index[qrow];
    qvalid = qvalid && x >= 0 && x < P.q_limit;
    qrow = x >= 0 && x < P.q_limit ? x : 0;
  }
  qrow += (long long)prob * P.q_rows_per_problem;
  f32x4 qreg[D / 8];
#pragma unroll
  for (int j = 0; j < D / 8; ++j) qreg[j] = *reinterpret_cast<const f32x4*>(P.q + qrow * D + 8 * j + 4 * g);
  const float sc = P.row_scale / fmaxf(P.cR ? P.cR[qrow] : 1.f, P.cr_min);

  f32x16 acc[NX][CT];
#pragma unroll
  for (int x = 0; x < NX; ++x)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][ct][r] = 0.f;
  float m = F32_LOWEST, S = 0.f, H = 0.f;  // App. B: reference, sum of p, sum of p t (this lane's keys only)

  while (t < t_end) {
    to_lds();
    wave_lds_fence();
    const int nt = t + KW;
    if (nt < t_end) load(nt);
    __builtin_amdgcn_sched_barrier(0);  // the next tile's loads stay in front of this tile's arithmetic
    f32x16 s, s2;  // two chains of half the channels: a shorter chain of roundings
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[r] = 0.f; s2[r] = 0.f; }
    f32x4 a[2];  // key rows, read one group of four MFMAs ahead
    a[0] = *reinterpret_cast<const f32x4*>(Ks + ql * RS + 4 * g);
#pragma unroll
    for (int j = 0; j < D / 8; ++j) {
      if (j + 1 < D / 8) a[(j + 1) & 1] = *reinterpret_cast<const f32x4*>(Ks + ql * RS + 8 * (j + 1) + 4 * g);
      __builtin_amdgcn_sched_barrier(0);
      s = mfma(a[j & 1][0], qreg[j][0], s);
      s2 = mfma(a[j & 1][1], qreg[j][1], s2);
      s = mfma(a[j & 1][2], qreg[j][2], s);
      s2 = mfma(a[j & 1][3], qreg[j][3], s2);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] += s2[r];
    const int left = P.nk - t * BT;  // keys of this tile that exist (copies past them cannot raise a maximum)
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32)) * sc;
    const float mn = fmaxf(m, mx);
    if (__any(mn > m)) {
      const float dl = m - mn;
      const float al = expf(dl);
      // App. B's rule; a row without keys so far has S = H = 0 and no finite shift
      H = S > 0.f ? H * al + S * al * dl : 0.f;
      S *= al;
      m = mn;
#pragma unroll
      for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[x][ct][r] *= al;
    }
    // step r: the probability of register r + 1 is formed while the products of register r run, the channel values of
    // step r + 1 are read
    auto prob = [&](int r) __attribute__((always_inline)) {
      float z = __builtin_fmaf(s[r], sc, -m);
      if (8 * (r >> 2) + 4 * g + (r & 3) >= left) z = -1.0e9f;
      const float p = expf(z);
      S += p;
      if (OUT_K) H = __builtin_fmaf(p, z, H);
      s[r] = p;
    };
    float xv[2][NX][CT];
    auto read_x = [&](int r) __attribute__((always_inline)) {
      const int row = (8 * (r >> 2) + 4 * g + (r & 3)) * RS + ql;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        if (OUT_K) xv[r & 1][0][ct] = Ks[row + 32 * ct];
        if (OUT_V) xv[r & 1][XV][ct] = Vs[row + 32 * ct];
      }
    };
    read_x(0);
    prob(0);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (r + 1 < 16) read_x(r + 1);
      __builtin_amdgcn_sched_barrier(0);
      if (r + 1 < 16) prob(r + 1);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int x = 0; x < NX; ++x) acc[x][ct] = mfma(xv[r & 1][x][ct], s[r], acc[x][ct]);
    }
    wave_lds_fence();
    t = nt;
  }

  // ---- epilogue: the KW waves of a query tile agree on a reference, stage their sums in LDS and add them up ----------
  S += __shfl_xor(S, 32);
  H += __shfl_xor(H, 32);
  if (g == 0) {
    stat[wave * 96 + ql] = m;
    stat[wave * 96 + 32 + ql] = S;
    stat[wave * 96 + 64 + ql] = H;
  }
  __syncthreads();
  const int w0 = wave - kw;
  float M = stat[w0 * 96 + ql];
#pragma unroll
  for (int w = 1; w < KW; ++w) M = fmaxf(M, stat[(w0 + w) * 96 + ql]);
  float St = 0.f, Ht = 0.f;
#pragma unroll
  for (int w = 0; w < KW; ++w) {
    const float sw = stat[(w0 + w) * 96 + 32 + ql];
    const float dl = stat[(w0 + w) * 96 + ql] - M;
    const float e = KW == 1 ? 1.f : expf(dl);
    St += sw * e;
    // no keys: nothing; NaN goes through
    if (!(sw == 0.f)) Ht += KW == 1 ? stat[(w0 + w) * 96 + 64 + ql] : (stat[(w0 + w) * 96 + 64 + ql] + sw * dl) * e;
  }
  const float inv = P.part_o != nullptr ? 1.f : 1.f / St;
  const float mine = (KW == 1 ? 1.f : expf(m - M)) * inv;
#pragma unroll
  for (int x = 0; x < NX; ++x) {
    float* dst = (x == XV && OUT_V) ? Vs : Ks;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float4 w = {acc[x][ct][4 * c] * mine, acc[x][ct][4 * c + 1] * mine, acc[x][ct][4 * c + 2] * mine,
                          acc[x][ct][4 * c + 3] * mine};
        *reinterpret_cast<float4*>(dst + ql * RS + 32 * ct + 8 * c + 4 * g) = w;
      }
  }
  if (kw == 0 && g == 0 && qvalid) {
    if (P.part_o != nullptr) {
      P.part_ms[((long long)split * P.nproblems + prob) * P.nq + qr] = make_float2(M, St);
    } else {
      if (OUT_K) P.cl[qrow] = -(logf(St) - Ht / St);  // c_L = -H
      if (P.lse != nullptr) P.lse[qrow] = M + logf(St);
    }
  }
  __syncthreads();
  const float* base = sm + w0 * WAVE_FLOATS;
#pragma unroll
  for (int u = 0; u < BT * D / 4 / (64 * KW); ++u) {
    const int e = u * 64 * KW + kw * 64 + lane;
    const int row = e / (D / 4);
    const int col = (e % (D / 4)) * 4;
    const int r = qt * BT + row;
    if (!active || r >= P.nq) continue;
    long long orow = r;
    if (P.q_index != nullptr && P.part_o == nullptr) {
      orow = P.q_index[r];
      if (orow < 0 || orow >= P.q_limit) continue;
    }
#pragma unroll
    for (int x = 0; x < NX; ++x) {
      const bool is_v = x == XV && OUT_V;
      const float* a = base + (is_v ? AREA : 0) + row * RS + col;
      float4 o = *reinterpret_cast<const float4*>(a);
#pragma unroll
      for (int w = 1; w < KW; ++w) {
        const float4 b = *reinterpret_cast<const float4*>(a + w * WAVE_FLOATS);
        o.x += b.x; o.y += b.y; o.z += b.z; o.w += b.w;
      }
      float* d = P.part_o != nullptr ? P.part_o + (((long long)split * P.nproblems + prob) * P.nq + orow) * D + col
                                     : (is_v ? P.outv : P.outk) + ((long long)prob * P.q_rows_per_problem + orow) * D + col;
      if (is_v && P.blend) {
        const float4 b = *reinterpret_cast<const float4*>(d);
        o.x = 0.5f * (o.x + b.x); o.y = 0.5f * (o.y + b.y); o.z = 0.5f * (o.z + b.z); o.w = 0.5f * (o.w + b.w);
      }
      *reinterpret_cast<float4*>(d) = o;
    }
  }
}

// Sums of the key ranges of one query row, 64 threads: out = sum_s o_s e^(m_s - M) / sum_s S_s e^(m_s - M).
__global__ void __launch_bounds__(64) f32_merge_kernel(const float* __restrict__ part_o, const float2* __restrict__ part_ms,
                                                       float* __restrict__ out, int nsplit, int nq, int nproblems,
                                                       long long rows_per_problem, int d) {
  const int r = blockIdx.x, prob = blockIdx.y;
  const long long step = (long long)nproblems * nq;
  const long long row = (long long)prob * nq + r;
  float M = F32_LOWEST;
  for (int s = 0; s < nsplit; ++s) M = fmaxf(M, part_ms[s * step + row].x);
  float S = 0.f;
  for (int s = 0; s < nsplit; ++s) S += part_ms[s * step + row].y * expf(part_ms[s * step + row].x - M);
  for (int c = threadIdx.x; c < d; c += 64) {
    float o = 0.f;
    for (int s = 0; s < nsplit; ++s) o += part_o[(s * step + row) * d + c] * expf(part_ms[s * step + row].x - M);
    out[((long long)prob * rows_per_problem + r) * d + c] = o / S;
  }
}

template <int D, bool OUT_K, bool OUT_V, int KW>
hipError_t launch_kw(F32Params& P, hipStream_t st) {
  constexpr int LDS = (WAVES * (OUT_V ? 2 : 1) * BT * (D + 4) + WAVES * 96) * 4;  // at most 134 KB (d = 128 with values)
  auto kern = f32_attend_kernel<D, OUT_K, OUT_V, KW>;
  if (LDS > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (e != hipSuccess) return e;
  }
  const int groups = (P.total + WAVES / KW - 1) / (WAVES / KW);
  P.groups_per_xcd = (groups + 7) / 8;
  hipLaunchKernelGGL(kern, dim3(P.groups_per_xcd * 8), dim3(64 * WAVES), LDS, st, P);
  return hipGetLastError();
}

// Waves per query tile: one each when the tiles alone give every SIMD (1024 of them) two waves, or when there is nothing
// to share; four otherwise, so that few query tiles still occupy the chip.
template <int D, bool OUT_K, bool OUT_V>
hipError_t launch_attend(F32Params& P, hipStream_t st) {
  const int tiles = P.tiles_per_split;
  if (P.total >= 2048 || tiles < 2) return launch_kw<D, OUT_K, OUT_V, 1>(P, st);
  if (tiles == 2) return launch_kw<D, OUT_K, OUT_V, 2>(P, st);
  return launch_kw<D, OUT_K, OUT_V, 4>(P, st);
}

template <bool OUT_K, bool OUT_V>
hipError_t launch_attend_d(F32Params& P, int d, hipStream_t st) {
  const long long total = (long long)P.nproblems * P.nqt * P.nsplit;
  if (!f32_attend_fits((long long)P.nproblems * P.nsplit, P.nq)) return hipErrorInvalidValue;
  P.total = (int)total;
  if (d == 128) return launch_attend<128, OUT_K, OUT_V>(P, st);
  if (d == 64) return launch_attend<64, OUT_K, OUT_V>(P, st);
  return launch_attend<32, OUT_K, OUT_V>(P, st);
}

// ---- temporal factor (Eq. L with Eq. alpha_R / c_R; the apply-to-V of App. A), T <= 32 ----------------------------------
// One wave per (position, head): the T rows of q, alpha_L (and y) in LDS, U^T = alpha_L Q^T as above (lane = query frame
// j), softmax over key frames in the lane.  Last sweep: O^T = y^T L^T straight from the registers.  Fitting sweep: the
// contraction runs over j, so L passes through LDS once to become lane = key frame.  Bound by memory: each row read and
// written once.
template <int D, bool FINAL>
__global__ void __launch_bounds__(64) f32_temporal_kernel(const float* __restrict__ q, const float* __restrict__ aL,
                                                          const float* __restrict__ cL, const float* __restrict__ y,
                                                          float* __restrict__ aR, float* __restrict__ cR,
                                                          float* __restrict__ out, int T, int b, float q_scale) {
  constexpr int RS = D + 4;
  constexpr int CT = D / 32;
  constexpr int LS = BT + 1;               // row stride of L in LDS
  constexpr int RPL = 64 / (D / 4);
  extern __shared__ __attribute__((aligned(16))) float sm[];
  float* Qs = sm;                          // [T][RS]
  float* As = Qs + T * RS;                 // [T][RS]
  float* Xs = As + T * RS;                 // last sweep: y [T][RS]; fitting sweep: L [32][LS]
  const int i = blockIdx.x;
  const long long row0 = (long long)blockIdx.y * T * b + i;  // row of frame 0
  const int lane = threadIdx.x;
  const int ql = lane & 31;
  const int g = lane >> 5;
  const int lr = lane / (D / 4);
  const int lc = (lane % (D / 4)) * 4;
  for (int r = lr; r < T; r += RPL) {
    const long long e = (row0 + (long long)r * b) * D + lc;
    *reinterpret_cast<float4*>(Qs + r * RS + lc) = *reinterpret_cast<const float4*>(q + e);
    *reinterpret_cast<float4*>(As + r * RS + lc) = *reinterpret_cast<const float4*>(aL + e);
    if (FINAL) *reinterpret_cast<float4*>(Xs + r * RS + lc) = *reinterpret_cast<const float4*>(y + e);
  }
  const float bias = cL[row0 + (long long)min(ql, T - 1) * b];  // of key frame ql
  wave_lds_fence();
  const int rl = min(ql, T - 1);           // frames past T: copies, weight zero below
  f32x16 u;
#pragma unroll
  for (int r = 0; r < 16; ++r) u[r] = 0.f;
#pragma unroll
  for (int j = 0; j < D / 8; ++j) {
    const float4 a = *reinterpret_cast<const float4*>(As + rl * RS + 8 * j + 4 * g);
    const float4 x = *reinterpret_cast<const float4*>(Qs + rl * RS + 8 * j + 4 * g);
    u = mfma(a.x, x.x, u);
    u = mfma(a.y, x.y, u);
    u = mfma(a.z, x.z, u);
    u = mfma(a.w, x.w, u);
  }
  float mx = F32_LOWEST;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int kf = 8 * (r >> 2) + 4 * g + (r & 3);
    u[r] = kf < T ? u[r] * q_scale - __shfl(bias, kf) : -INFINITY;
    mx = fmaxf(mx, u[r]);
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  float s = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    u[r] = expf(u[r] - mx);
    s += u[r];
  }
  s += __shfl_xor(s, 32);
  const float inv = ql < T ? 1.f / s : 0.f;  // query frames past T weigh nothing
#pragma unroll
  for (int r = 0; r < 16; ++r) u[r] *= inv;
  f32x16 acc[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[ct][r] = 0.f;
  if (!FINAL) {
#pragma unroll
    for (int r = 0; r < 16; ++r) Xs[ql * LS + 8 * (r >> 2) + 4 * g + (r & 3)] = ql < T ? u[r] : 0.f;
    wave_lds_fence();
    float c = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {  // now lane = key frame, register r = query frame
      u[r] = Xs[(8 * (r >> 2) + 4 * g + (r & 3)) * LS + ql];
      c += u[r];
    }
    c += __shfl_xor(c, 32);
    if (g == 0 && ql < T) cR[row0 + (long long)ql * b] = c;
  }
  const float* src = FINAL ? Xs : Qs;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (8 * (r >> 2) + (r & 3) >= T) continue;  // neither of the two frames of this step exists
    const int f = 8 * (r >> 2) + 4 * g + (r & 3);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const float x = src[min(f, T - 1) * RS + 32 * ct + ql];
      acc[ct] = mfma(f < T ? x : 0.f, u[r], acc[ct]);  // (not a copy: infinite values times weight zero)
    }
  }
  // staged over alpha_L (read for the last time above) and written as whole rows
  wave_lds_fence();
  if (ql < T) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        *reinterpret_cast<float4*>(As + ql * RS + 32 * ct + 8 * c + 4 * g) =
            make_float4(acc[ct][4 * c], acc[ct][4 * c + 1], acc[ct][4 * c + 2], acc[ct][4 * c + 3]);
  }
  wave_lds_fence();
  float* dst = FINAL ? out : aR;
  for (int r = lr; r < T; r += RPL)
    *reinterpret_cast<float4*>(dst + (row0 + (long long)r * b) * D + lc) = *reinterpret_cast<const float4*>(As + r * RS + lc);
}

template <int D, bool FINAL>
hipError_t launch_temporal(const float* q, const float* aL, const float* cL, const float* y, float* aR, float* cR, float* out,
                           const Dims& dm, float q_scale, hipStream_t st) {
  const int lds = (2 * dm.T * (D + 4) + (FINAL ? dm.T * (D + 4) : BT * (BT + 1))) * 4;  // at most 50 KB
  auto kern = f32_temporal_kernel<D, FINAL>;
  if (lds > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(dm.b, dm.BH), dim3(64), lds, st, q, aL, cL, y, aR, cR, out, dm.T, dm.b, q_scale);
  return hipGetLastError();
}

bool aligned16(std::initializer_list<const void*> ptrs) {
  for (const void* p : ptrs)
    if (((uintptr_t)p & 15) != 0) return false;
  return true;
}

bool head_dim_ok(const Dims& dm) { return dm.d == 32 || dm.d == 64 || dm.d == 128; }

}  // namespace

// The calls the blocked-softmax kernel takes, `problems` of nq query rows and nk keys: the head dimensions above, tensors on
// 16-byte boundaries (rows then are too), query tiles that one launch holds (a frame of one token is a tile too), and keys
// enough that it is the faster one.
bool f32_attend_supported(const Dims& dm, bool with_v, long long problems, long long nq, long long nk,
                          std::initializer_list<const void*> tensors) {
  return head_dim_ok(dm) && aligned16(tensors) && f32_attend_fits(problems, nq) &&
         !f32_few_keys(dm.d, with_v, problems, nq, nk);
}

hipError_t launch_r_update_f32(const float* aR, const float* cR, const float* k, const float* v, float* aL, float* cL,
                               float* y, float* lse, const Dims& dm, float row_scale, float cr_min, hipStream_t st) {
  F32Params P = {};
  P.q = aR; P.cR = cR; P.k = k; P.v = v; P.outk = aL; P.outv = y; P.cl = cL; P.lse = lse;
  P.q_rows_per_problem = dm.b; P.k_rows_per_problem = dm.b;
  P.nq = dm.b; P.nk = dm.b;
  P.nqt = (dm.b + BT - 1) / BT;
  P.nsplit = 1;
  P.tiles_per_split = P.nqt;
  P.nproblems = dm.BH * dm.T;
  P.row_scale = row_scale; P.cr_min = cr_min;
  return v != nullptr ? launch_attend_d<true, true>(P, dm.d, st) : launch_attend_d<true, false>(P, dm.d, st);
}

// scratch: room for the partial sums of several key ranges per row, used as far as it goes (none: one range).  Only the first
// frame inside vmonarch_attention_f32 brings any; the other calls take one range, which is still the faster way (one row of 4
// heads over 3120 / 32,760 keys, d = 128: 139 / 1343 us, plain-ALU kernel 963 / 19,900).
hipError_t launch_attend_rows_f32(const float* q, const float* k, const float* v, float* out, float* lse, const Dims& dm,
                                  int nrows, const int* rows, void* scratch, size_t scratch_bytes, hipStream_t st) {
  F32Params P = {};
  P.q = q; P.k = k; P.v = v; P.outv = out; P.lse = lse;
  P.q_index = rows; P.q_limit = dm.N;
  P.q_rows_per_problem = dm.N; P.k_rows_per_problem = dm.N;
  if (dm.N > 0x7fffffffLL - 2 * BT) return hipErrorInvalidValue;
  P.nq = nrows; P.nk = (int)dm.N;
  P.nqt = (nrows + BT - 1) / BT;
  P.nproblems = dm.BH;
  P.row_scale = 1.0f / sqrtf((float)dm.d);
  P.cr_min = 0.f;
  // Key ranges: as many four-wave items as 256 CUs hold at once (two workgroups' LDS fits one, d = 128: one) without
  // starting a second round, each of at least eight tiles (two per wave), within the scratch.
  const long long tiles = (dm.N + BT - 1) / BT;
  const long long items = (long long)dm.BH * P.nqt;
  long long ns = 1;
  if (rows == nullptr && lse == nullptr && scratch != nullptr) {
    ns = (dm.d == 128 ? 256 : 512) / items;
    ns = ns < tiles / 8 ? ns : tiles / 8;
    const long long per_range = (long long)dm.BH * nrows * (dm.d * (long long)sizeof(float) + (long long)sizeof(float2));
    const long long fit = (long long)(scratch_bytes / (size_t)per_range);
    ns = ns < fit ? ns : fit;
    if (ns < 1) ns = 1;
  }
  P.tiles_per_split = (int)((tiles + ns - 1) / ns);
  ns = (tiles + P.tiles_per_split - 1) / P.tiles_per_split;  // no empty range
  P.nsplit = (int)ns;
  if (ns > 1) {
    P.part_o = (float*)scratch;
    P.part_ms = (float2*)((char*)scratch + (size_t)ns * dm.BH * nrows * dm.d * sizeof(float));
  }
  hipError_t e = launch_attend_d<false, true>(P, dm.d, st);
  if (e != hipSuccess || ns == 1) return e;
  hipLaunchKernelGGL(f32_merge_kernel, dim3(nrows, dm.BH), dim3(64), 0, st, P.part_o, P.part_ms, out, P.nsplit, nrows, dm.BH,
                     dm.N, dm.d);
  return hipGetLastError();
}

hipError_t launch_sink_average_f32(const float* q, const float* k, const float* v, float* out, const Dims& dm, hipStream_t st) {
  F32Params P = {};
  P.q = q; P.k = k; P.v = v; P.outv = out;
  P.q_rows_per_problem = dm.N; P.k_rows_per_problem = dm.N;
  if (dm.N > 0x7fffffffLL - 2 * BT) return hipErrorInvalidValue;
  P.nq = (int)dm.N; P.nk = dm.b;
  P.nqt = (int)((dm.N + BT - 1) / BT);
  P.nsplit = 1;
  P.tiles_per_split = (dm.b + BT - 1) / BT;
  P.nproblems = dm.BH;
  P.row_scale = 1.0f / sqrtf((float)dm.d);
  P.cr_min = 0.f;
  P.blend = 1;
  return launch_attend_d<false, true>(P, dm.d, st);
}

bool l_update_f32_supported(const Dims& dm, std::initializer_list<const void*> tensors) {
  return dm.T <= BT && head_dim_ok(dm) && aligned16(tensors) && grid_fits(dm.b, 64);
}

hipError_t launch_l_update_f32(const float* q, const float* aL, const float* cL, const float* y, float* aR, float* cR,
                               float* out, const Dims& dm, float q_scale, hipStream_t st) {
  auto run = [&](auto dc) -> hipError_t {
    constexpr int D = decltype(dc)::value;
    return y != nullptr ? launch_temporal<D, true>(q, aL, cL, y, aR, cR, out, dm, q_scale, st)
                        : launch_temporal<D, false>(q, aL, cL, y, aR, cR, out, dm, q_scale, st);
  };
  if (dm.d == 128) return run(std::integral_constant<int, 128>{});
  if (dm.d == 64) return run(std::integral_constant<int, 64>{});
  return run(std::integral_constant<int, 32>{});
}

}  // namespace vm
