// bf16 MFMA kernel for the R-update (Eq. R with Eq. alpha_L/c_L; App. A R_update and y = R V) of short frames on
// gfx950: b <= 32 KT tokens, KT = 1 .. 7, d = 64 or 128.
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
#include "flash_select.h"

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
    default: break;
  }
  if constexpr (WITH_V) {
    if (P.b <= 192) return launch_kt<D, 6, true>(P, frames, st);
    if constexpr (D == 64) return launch_kt<D, 7, true>(P, frames, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace

bool frame_supported(const Dims& dm, bool with_v) {
  if (dm.d != 64 && dm.d != 128) return false;
  const long long frames = (long long)dm.BH * dm.T;
  return dm.b <= whole_frame_tokens(dm.d, with_v, frames, compute_units()) && frames <= 0x7fffff;
}

hipError_t launch_r_update_frame(const bf16_t* aR, const float* cR, const bf16_t* k, const bf16_t* v, bf16_t* aL, float* cL,
                                 bf16_t* y, float* lse, const Dims& dm, float row_scale, float cr_min, hipStream_t st) {
  const bool with_v = v != nullptr;
  if (!frame_supported(dm, with_v) || with_v != (y != nullptr)) return hipErrorInvalidValue;
  FrameParams P = {aR, cR, k, v, aL, cL, y, lse, dm.b, row_scale, cr_min};
  const unsigned frames = (unsigned)((long long)dm.BH * dm.T);
  if (dm.d == 128) return with_v ? launch_frames<128, true>(P, frames, st) : launch_frames<128, false>(P, frames, st);
  return with_v ? launch_frames<64, true>(P, frames, st) : launch_frames<64, false>(P, frames, st);
}

}  // namespace vm
