// bf16 MFMA kernel for the R-update (Eq. R with Eq. alpha_L/c_L; App. A R_update and y = R V) of short frames on
// gfx950: b <= 32 KT tokens, KT = 1 .. 8, d = 64 or 128.
//
// A short frame has no key loop to pipeline: its keys are one or a few 32-row tiles, the whole softmax of a query sits
// in one lane's registers and every tensor is read and written once, so the bounds are memory and the length of one
// block's dependent chain.  One workgroup therefore takes one frame with exactly KT waves, 32 queries each: no wave
// idles on padding (the streaming kernels' blocks of 256 or 128 query rows are padding for the most part here), a block
// needs 4 KT .. 16 KT KB of LDS, so that many frames are in flight on a compute unit, and all of a frame's loads are
// issued before the first is waited for.  Fitting / last update in us, streaming kernels -> this one, 12 heads, d = 64: 32 frames
// of 32 tokens (one block's chain) 7.9 / 10.4 -> 4.0 / 5.0; 512 frames of 64 70 / 100 -> 25 / 40 (6.0 / 6.3 TB/s of
// the tensors, which fit the last-level cache there: more than the 5.2 TB/s of a copy through HBM).
// Contractions and register layouts are the streaming kernels' (flash2.hip):
//
//   S^T = K Q^T     A = K rows from LDS, B = Q^T in registers; lane (q, g) holds query q's logits for half of the keys
//   X^T P^T         A = X^T (X = K, then V) by LDS transpose reads, B = P^T from the softmax registers
//
// The exact row maximum is the reference; c_L and the log-sum-exp come from fp32 sums (subtile_probs), the rows are divided
// by the sum of the bf16-rounded weights.
#include "common.h"
#include "flash_device.h"

namespace vm {

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

struct FrameParams {
  const bf16_t* q;
  const float* cR;  // may be null (= 1)
  const bf16_t* k;
  const bf16_t* v;
  bf16_t* aL;
  float* cL;
  bf16_t* y;
  float* lse;  // may be null
  int b;
  float row_scale;
  float cr_min;
};

// Row `row` from its reference m and the sums l of p = 2^t and h of p t (log2 units): c_L = -H, App. B's H = log S - L / S
__device__ __forceinline__ void store_statistics(const FrameParams& P, long long row, float m, float l, float h) {
  const float log_l = __log2f(l);
  P.cL[row] = LN2 * (h / l - log_l);
  if (P.lse != nullptr) P.lse[row] = LN2 * (m + log_l);
}

template <int D, int KT, bool WITH_V>
__global__ void __launch_bounds__(64 * KT) frame_kernel(FrameParams P) {
  using G = RowGeo<D>;
  constexpr int ROW_BYTES = G::ROW_BYTES;
  constexpr int KS = G::KS;
  constexpr int CT = G::CT;
  constexpr int CH = G::CH;
  constexpr int RPI = G::RPI;
  constexpr int NPS = 32 / RPI;                // 16-byte loads per lane that fetch a wave's 32 rows
  constexpr int V_OFF = 32 * KT * ROW_BYTES;
  auto swz = [](int row) { return G::swz(row); };
  extern __shared__ __attribute__((aligned(16))) char smem[];  // [K|V][32 KT rows][2 D bytes]

  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const int lane = tid & 63;
  const int ql = lane & 31;
  const int g = lane >> 5;
  const int b = P.b;
  const long long row0 = (long long)blockIdx.x * b;

  // ---- every load of the frame: wave w fetches key (and value) rows 32 w .. + 31 and its query rows.  Rows past the
  // end are copies of the last one (finite data; masked as keys, not stored as queries).
  const int st_row = lane / CH;  // + RPI ps
  const int pc = lane % CH;
  u32x4 rk[NPS], rv[NPS];
#pragma unroll
  for (int ps = 0; ps < NPS; ++ps) {
    const int r = 32 * wave + ps * RPI + st_row;
    const long long e = (row0 + min(r, b - 1)) * D + (pc ^ swz(r)) * 8;
    rk[ps] = *reinterpret_cast<const u32x4*>(P.k + e);
  }
  const int qrow = 32 * wave + ql;
  const bool qvalid = qrow < b;
  const long long qr = row0 + (qvalid ? qrow : b - 1);
  bf16x8 qreg[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(P.q + qr * D + 16 * ks + 8 * g);
  const float c = fmaxf(P.cR ? P.cR[qr] : 1.0f, P.cr_min);
  if (WITH_V) {
#pragma unroll
    for (int ps = 0; ps < NPS; ++ps) {
      const int r = 32 * wave + ps * RPI + st_row;
      const long long e = (row0 + min(r, b - 1)) * D + (pc ^ swz(r)) * 8;
      rv[ps] = *reinterpret_cast<const u32x4*>(P.v + e);
    }
  }
  const int st_off = (32 * wave + st_row) * ROW_BYTES + pc * 16;
#pragma unroll
  for (int ps = 0; ps < NPS; ++ps) *reinterpret_cast<u32x4*>(smem + st_off + ps * 1024) = rk[ps];
  // The values wait in registers until the softmax is done, or, where its logits need those (five tiles and more at
  // d = 128), go to LDS now.  Later is better where it fits: 64 against 78 us, 2432 frames of 160 at d = 64.
  constexpr bool EARLY_V = D == 128 && KT > 4;
  auto values_to_lds = [&]() __attribute__((always_inline)) {
    if (!WITH_V) return;
#pragma unroll
    for (int ps = 0; ps < NPS; ++ps) *reinterpret_cast<u32x4*>(smem + V_OFF + st_off + ps * 1024) = rv[ps];
  };
  if (EARLY_V) values_to_lds();
  __syncthreads();

  // ---- logits and softmax over the frame's keys ----------------------------------------------------------------
  f32x16 s[KT];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[kt][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 a = lds_read_b128(smem + (32 * kt + ql) * ROW_BYTES + (((2 * ks + g) ^ swz(ql)) << 4));
      s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[ks], s[kt], 0, 0, 0);
    }
  }
  const float sc = P.row_scale * LOG2E / c;
  auto past_end = [&](int kt, int r) {  // only the last 32 keys can lie past the end
    return kt == KT - 1 && 32 * kt + 8 * (r >> 2) + 4 * g + (r & 3) >= b;
  };
  float m = -3.0e38f;
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
#pragma unroll
    for (int r = 0; r < 16; ++r) m = fmaxf(m, past_end(kt, r) ? -3.0e38f : s[kt][r] * sc);
  m = fmaxf(m, __shfl_xor(m, 32));
  bf16x8 pb[KT][2];
  float lt = 0.f, l = 0.f, h = 0.f;
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[kt][r] = past_end(kt, r) ? -3.0e38f : __builtin_fmaf(s[kt][r], sc, -m);
    subtile_probs<true>(s[kt], 1.0f, 0.0f, lt, l, h, pb[kt]);
  }
  lt += __shfl_xor(lt, 32);
  l += __shfl_xor(l, 32);
  h += __shfl_xor(h, 32);
  const float inv = lt > 0.f ? 1.0f / lt : 0.f;  // no key with a finite logit: zeros, as in the streaming kernels
  if (qvalid && g == 0) store_statistics(P, qr, m, l, h);

  // ---- X^T P^T ---------------------------------------------------------------------------------------------------
  const int rp = lane & 15;
  const int chh = (lane >> 4) & 1;
  auto product = [&](int off, f32x16 (&acc)[CT]) __attribute__((always_inline)) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ct][r] = 0.f;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int cc = 0; cc < 2; ++cc)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          bf16x4 part[2];
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const int key = 8 * hh + 4 * g + (rp >> 2);
            const int lc = 4 * ct + 2 * chh + ((rp >> 1) & 1);
            part[hh] = lds_read_tr(smem + off + (32 * kt + 16 * cc + key) * ROW_BYTES + ((lc ^ swz(key)) << 4) + ((rp & 1) << 3));
          }
          const bf16x8 a = __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
          acc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[kt][cc], acc[ct], 0, 0, 0);
        }
  };
  // the wave's 32 result rows, over its own rows of the tensor that was just multiplied, and out as whole rows
  auto store_rows = [&](int off, const f32x16 (&acc)[CT], bf16_t* dst) __attribute__((always_inline)) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) {
        uint2 w;
        w.x = pack_bf16(acc[ct][4 * cc + 0] * inv, acc[ct][4 * cc + 1] * inv);
        w.y = pack_bf16(acc[ct][4 * cc + 2] * inv, acc[ct][4 * cc + 3] * inv);
        *reinterpret_cast<uint2*>(smem + off + qrow * ROW_BYTES + (((4 * ct + cc) ^ swz(ql)) << 4) + 8 * g) = w;
      }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the staged rows are private to the wave
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int ps = 0; ps < NPS; ++ps) {
      const int r = 32 * wave + ps * RPI + st_row;
      if (r < b) {
        const uint4 w = *reinterpret_cast<const uint4*>(smem + off + r * ROW_BYTES + pc * 16);
        *reinterpret_cast<uint4*>(dst + (row0 + r) * D + (pc ^ swz(r)) * 8) = w;
      }
    }
  };
  if (!EARLY_V) values_to_lds();
  f32x16 acc[CT];
  product(0, acc);
  __syncthreads();  // every wave is done with K; V is in place
  store_rows(0, acc, P.aL);
  if (WITH_V) {
    product(V_OFF, acc);
    __syncthreads();  // every wave is done with V
    store_rows(V_OFF, acc, P.y);
  }
}

template <int D, int KT, bool WITH_V>
hipError_t launch_kt(const FrameParams& P, unsigned frames, hipStream_t st) {
  constexpr int LDS_BYTES = (WITH_V ? 2 : 1) * 32 * KT * D * 2;
  auto kern = frame_kernel<D, KT, WITH_V>;
  if (LDS_BYTES > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(frames), dim3(64 * KT), LDS_BYTES, st, P);
  return hipGetLastError();
}

template <int D, bool WITH_V>
hipError_t launch_frames(const FrameParams& P, unsigned frames, hipStream_t st) {
  switch ((P.b + 31) / 32) {
    case 1: return launch_kt<D, 1, WITH_V>(P, frames, st);
    case 2: return launch_kt<D, 2, WITH_V>(P, frames, st);
    case 3: return launch_kt<D, 3, WITH_V>(P, frames, st);
    case 4: return launch_kt<D, 4, WITH_V>(P, frames, st);
    case 5: return launch_kt<D, 5, WITH_V>(P, frames, st);
    case 6: return launch_kt<D, 6, WITH_V>(P, frames, st);
    default: break;
  }
  if constexpr (D == 64 || !WITH_V)
    if (P.b <= 224) return launch_kt<D, 7, WITH_V>(P, frames, st);
  if constexpr (D == 64 && WITH_V) return launch_kt<D, 8, WITH_V>(P, frames, st);
  return hipErrorInvalidValue;
}

// Frames of 257 .. 384 tokens, d = 64 (b <= 32 KT, KT = 10, 12): a workgroup takes 128 query rows (four waves) of one frame.
// The streaming kernel's query blocks hold 256 rows, so a third to a half of them is padding here, and its last update has
// one workgroup on a compute unit: 130 frames are two rounds.  Blocks of 128 rows, two on a unit, waste less of both.
// All keys are requested at once (32 KT rows of LDS, which the values take over when the R K products are done), the logits
// are formed twice, first for the exact row maxima, then for the weights, which wait in registers (8 a tile) for both
// products.  Last update, before -> now: 768 frames of 257 89 -> 57 us, 1216 of 323 161 -> 107, 1024 of 384 130 -> 95.
template <int D, int KT, bool WITH_V>
__global__ void __launch_bounds__(256, 2) frame_rows_kernel(FrameParams P) {
  using G = RowGeo<D>;
  constexpr int ROW_BYTES = G::ROW_BYTES;
  constexpr int KS = G::KS;
  constexpr int CT = G::CT;
  constexpr int CH = G::CH;
  constexpr int RPI = G::RPI;
  constexpr int STAGE_OFF = 32 * KT * ROW_BYTES;
  auto swz = [](int row) { return G::swz(row); };
  extern __shared__ __attribute__((aligned(16))) char smem[];  // [32 KT key (value) rows][4 waves x 32 result rows]

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int ql = lane & 31;
  const int g = lane >> 5;
  const int b = P.b;
  const int nqb = (b + 127) / 128;
  const int frame = blockIdx.x / nqb;
  const int qb = blockIdx.x - frame * nqb;
  const long long row0 = (long long)frame * b;

  const unsigned lds_base = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)smem;
  auto issue_rows = [&](const bf16_t* x) __attribute__((always_inline)) {
    const bf16_t* base = x + row0 * D;
    constexpr int NR = 32 * KT / (4 * RPI);
    static_assert(32 * KT % (4 * RPI) == 0 && (4 * RPI) % 16 == 0, "whole instructions; the rows of one lane share a swizzle");
    const int r0 = RPI * wave + lane / CH;
    const int lc = (lane % CH) ^ swz(r0);
#pragma unroll
    for (int r = 0; r < NR; ++r) {  // rows past the end: copies of the last one, masked below
      const unsigned off = (unsigned)(min(4 * RPI * r + r0, b - 1) * ROW_BYTES + lc * 16);
      const unsigned dst = __builtin_amdgcn_readfirstlane(lds_base + (4 * RPI * r + RPI * wave) * ROW_BYTES);
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(dst) : "memory", "m0");
    }
  };
  issue_rows(P.k);
  const int row_first = qb * 128 + wave * 32;
  const bool active = row_first < b;  // a wave without rows only helps to load
  const int qrow = row_first + ql;
  const bool qvalid = qrow < b;
  const long long qr = row0 + (qvalid ? qrow : b - 1);
  bf16x8 qreg[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(P.q + qr * D + 16 * ks + 8 * g);
  const float sc = P.row_scale * LOG2E / fmaxf(P.cR ? P.cR[qr] : 1.0f, P.cr_min);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  f32x16 acc[CT];
  bf16x8 pb[KT][2];
  float m = -3.0e38f, lt = 0.f, l = 0.f, h = 0.f;
  auto logits = [&](int kt) __attribute__((always_inline)) -> f32x16 {
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 a = lds_read_b128(smem + (32 * kt + ql) * ROW_BYTES + (((2 * ks + g) ^ swz(ql)) << 4));
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[ks], s, 0, 0, 0);
    }
    return s;
  };
  const int rp = lane & 15;
  const int chh = (lane >> 4) & 1;
  auto product = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ct][r] = 0.f;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
      for (int cc = 0; cc < 2; ++cc)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          bf16x4 part[2];
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const int key = 8 * hh + 4 * g + (rp >> 2);
            const int lc = 4 * ct + 2 * chh + ((rp >> 1) & 1);
            part[hh] = lds_read_tr(smem + (32 * kt + 16 * cc + key) * ROW_BYTES + ((lc ^ swz(key)) << 4) + ((rp & 1) << 3));
          }
          const bf16x8 a = __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7);
          acc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[kt][cc], acc[ct], 0, 0, 0);
        }
      if (kt & 1) __builtin_amdgcn_sched_barrier(0);
    }
  };
  float inv = 0.f;
  auto store_rows = [&](bf16_t* dst) __attribute__((always_inline)) {
    char* stage = smem + STAGE_OFF + wave * 32 * ROW_BYTES;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) {
        uint2 w;
        w.x = pack_bf16(acc[ct][4 * cc + 0] * inv, acc[ct][4 * cc + 1] * inv);
        w.y = pack_bf16(acc[ct][4 * cc + 2] * inv, acc[ct][4 * cc + 3] * inv);
        *reinterpret_cast<uint2*>(stage + ql * ROW_BYTES + (((4 * ct + cc) ^ swz(ql)) << 4) + 8 * g) = w;
      }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the staged rows are private to the wave
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int ps = 0; ps < 32 / RPI; ++ps) {
      const int r = ps * RPI + lane / CH;
      const int pc = lane % CH;
      const uint4 w = *reinterpret_cast<const uint4*>(stage + r * ROW_BYTES + pc * 16);
      if (row_first + r < b) *reinterpret_cast<uint4*>(dst + (row0 + row_first + r) * D + (pc ^ swz(r)) * 8) = w;
    }
    __builtin_amdgcn_wave_barrier();  // the next result is staged over these rows
  };
  if (active) {
    // b > 32 (KT - 2): only the last two tiles can reach past the end
    auto past_end = [&](int kt, int r) { return kt >= KT - 2 && 32 * kt + 8 * (r >> 2) + 4 * g + (r & 3) >= b; };
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      const f32x16 s = logits(kt);
#pragma unroll
      for (int r = 0; r < 16; ++r) m = fmaxf(m, past_end(kt, r) ? -3.0e38f : s[r] * sc);
      if (kt & 1) __builtin_amdgcn_sched_barrier(0);  // operands of two tiles in flight, not of all
    }
    m = fmaxf(m, __shfl_xor(m, 32));
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      f32x16 s = logits(kt);
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = past_end(kt, r) ? -3.0e38f : __builtin_fmaf(s[r], sc, -m);
      subtile_probs<true>(s, 1.0f, 0.0f, lt, l, h, pb[kt]);
      if (kt & 1) __builtin_amdgcn_sched_barrier(0);
    }
    lt += __shfl_xor(lt, 32);
    l += __shfl_xor(l, 32);
    h += __shfl_xor(h, 32);
    inv = lt > 0.f ? 1.0f / lt : 0.f;
    if (qvalid && g == 0) store_statistics(P, qr, m, l, h);
    product();
  }
  if (WITH_V) {
    __syncthreads();  // every wave is done with the keys
    issue_rows(P.v);
  }
  if (active) store_rows(P.aL);
  if (WITH_V) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (active) {
      product();
      store_rows(P.y);
    }
  }
}

template <int D, int KT, bool WITH_V>
hipError_t launch_rows(const FrameParams& P, unsigned frames, hipStream_t st) {
  constexpr int LDS_BYTES = 32 * (KT + 4) * D * 2;
  auto kern = frame_rows_kernel<D, KT, WITH_V>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(frames * ((P.b + 127) / 128)), dim3(256), LDS_BYTES, st, P);
  return hipGetLastError();
}

}  // namespace

// Where the whole-frame kernel is the faster one, by sweeps of b = 1 .. 256 with 2 .. 3000 frames.  Without values up
// to 224 tokens: many frames 29 against 53 us at 128 tokens (d = 64), level from 161 on (50 / 49 us at 192), few frames
// 13 / 15 us there; at d = 128 59 / 97 us at 128 tokens, 101 / 112 at 224.  With values up to 256 tokens at d = 64 (66
// / 89 us there) and 192 at d = 128 (142 / 174 us): with a seventh tile of logits that one spills and is level.
bool frame_supported(const Dims& dm, bool with_v) {
  if (dm.d != 64 && dm.d != 128) return false;
  return dm.b <= (!with_v ? 224 : dm.d == 64 ? 256 : 192) && (long long)dm.BH * dm.T <= 0x7fffff;
}

// Where the 128-row blocks are taken (sweeps of 193 .. 512 tokens, 128 .. 2000 frames): d = 64, up to 384 tokens with
// values (see the kernel), 352 without (1216 frames of 323 87 -> 81 us; level at 384).  From 448 tokens on they lose
// (448, d = 64, without values: 71 -> 88 us).  Up to 128 frames the streaming kernel's two blocks a frame are one round
// of the 256 compute units; the two kernels are then within 4 % with values (19 / 20 us) and the blocks 4 .. 8 % ahead
// without (257 tokens 13.2 / 12.2 us): one line for both.  At d = 128 the keys leave room for one block on a unit: from
// 257 tokens on they lose nearly everywhere (257, 128 frames: 15.7 / 22.9 us, with values 25.9 / 32.0); at 193 and 256
// tokens they win while the blocks are one round (128 frames, with values: 22.0 / 16.6 and 23.3 / 18.4 us) and lose
// beyond (256 frames: 26.6 / 32.4 and 28.9 / 33.9), which is left alone.
bool frame_rows_supported(const Dims& dm, bool with_v) {
  const long long frames = (long long)dm.BH * dm.T;
  return dm.d == 64 && dm.b > 256 && dm.b <= (with_v ? 384 : 352) && frames > 128 && frames <= 0x7fffff;
}

hipError_t launch_r_update_frame(const bf16_t* aR, const float* cR, const bf16_t* k, const bf16_t* v, bf16_t* aL, float* cL,
                                 bf16_t* y, float* lse, const Dims& dm, float row_scale, float cr_min, hipStream_t st) {
  const bool with_v = v != nullptr, whole = frame_supported(dm, with_v);
  if (!(whole || frame_rows_supported(dm, with_v)) || with_v != (y != nullptr)) return hipErrorInvalidValue;
  FrameParams P = {aR, cR, k, v, aL, cL, y, lse, dm.b, row_scale, cr_min};
  const unsigned frames = (unsigned)((long long)dm.BH * dm.T);
  if (!whole) {
    if (dm.b <= 320) return with_v ? launch_rows<64, 10, true>(P, frames, st) : launch_rows<64, 10, false>(P, frames, st);
    return with_v ? launch_rows<64, 12, true>(P, frames, st) : launch_rows<64, 12, false>(P, frames, st);
  }
  if (dm.d == 128) return with_v ? launch_frames<128, true>(P, frames, st) : launch_frames<128, false>(P, frames, st);
  return with_v ? launch_frames<64, true>(P, frames, st) : launch_frames<64, false>(P, frames, st);
}

}  // namespace vm
