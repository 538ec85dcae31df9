// bf16 MFMA kernel for every blocked-softmax pass of spatio-temporal Monarch attention on gfx950,
// with one or two 32-query tiles per wave: the R-update of a fitting sweep
// (Eq. R + Eq. alpha_L/c_L: logits, alpha_L = R K and c_L), the R-update of the last sweep (the
// same plus y = R V of App. A, from ONE evaluation of the logits and of the softmax) and the
// first-frame recomputation (Sec. 3.3).  All three are Alg. 1 with the running max / sum /
// entropy of App. B.
//
// One workgroup = 4 waves.  With two tiles a wave owns 64 query rows for the whole key loop and, at d = 128 with values, the
// full register file of its SIMD (512 registers), which is what lets one wave hold both accumulator sets (R K and R V:
// 2 x 2 x 4 tiles of 16 registers) beside its queries and logits.  With one tile (32 rows, 128 in a workgroup) two or three
// workgroups share a compute unit; which launch takes which: flash_select.h.  Keys (and values) stream through LDS in tiles of 64 rows (32 where two
// workgroups would not fit a unit otherwise: tile_rows), four slots per tensor, loaded two tiles ahead.  Both contractions use v_mfma_f32_32x32x16_bf16:
//
//   S^T = K Q^T     A = K rows read from LDS (ds_read_b128), B = Q^T held in registers.  One A
//                   operand serves all query tiles of the wave: with two, half the
//                   LDS bytes per MFMA.  In the result lane (q, g) holds the logits of query q for
//                   16 of the 32 keys, so the sums are per-lane scalars.
//   O^T += X^T P^T  A = X^T (X = K for alpha_L, X = V for y) fetched from the same row-major
//                   LDS tile with the LDS transpose read (ds_read_b64_tr_b16), again shared by
//                   the query tiles; B = P^T, the S^T accumulator converted to bf16 in place.
//
// The 16-byte chunk c of key row r is stored at chunk c ^ swz(r) (RowGeo in common.h) so that
// both the row-wise b128 reads and the transpose reads spread over all banks.
#include "../../include/vmonarch.h"
#include <type_traits>

#include "common.h"
#include "flash_device.h"
#include "flash_select.h"

namespace vm {

namespace {

constexpr int W2 = 4;             // waves per workgroup
// No running row maximum is kept.  A row's reference comes from the maximum of its first 32 logits, and any reference gives the
// same outputs: the sums and the accumulators carry the common factor 2^-reference, the weights are formed in fp32 and rounded
// to bf16, which has fp32's exponent range, so a stale reference costs the outputs no precision until 2^t nears overflow.  What
// would overflow shows in the sums: a sub-tile whose weights add up to more than this in any lane is formed again, before its
// products, against references from its own row maxima (`redo`).  The maxima and their bookkeeping were 18 % of the vector
// instructions, which bound the loop (busy 0.85 of the cycles at d = 64 without values).  Measured, R-update without / with
// values: 12 x 32 frames of 2048, d = 64: 472 -> 441 / 713 -> 654 us (934, 945 TFLOP/s); 12 x 21 of 1536, d = 128: 317 -> 298 /
// 453 -> 431 us (1021, 1060).
// c_L needs two precautions.  The sum h of p t and the sum l of p must weigh every key alike, or their mismatch (about 1e-3
// relative when l holds the bf16-rounded p and h the unrounded ones) is multiplied by the mean of t, which a stale reference
// lets grow; both carry the UNROUNDED p here, beside the rounded sum that the outputs are divided by.  And c_L = h / l - log2 l is a
// difference of two numbers of the size of t at the keys that matter, so the reference belongs at the row's maximum: see
// HEADROOM2.
constexpr float STEP_MAX2 = 18446744073709551616.0f;  // 2^64
// Weights that large leave the accumulators 2^47 of room at 2^17 keys.  Sums above this one are rare (a row has grown by 2^32 and more since
// its reference was set); they send a wave to look whether the sub-tile multiplies elements of 2^40 or more, and then its references move too.
// (A limit of 2^64 alone overflows where values of 1e24 meet sharp rows; the look costs 252 frames of 1560 of deviation 20 / 30 1 / 5 %.)
constexpr float STEP_LARGE2 = 4294967296.0f;  // 2^32
// A reference is put at the row's maximum.  Only where attention is sharp it is put above it, by up to this much (log2 units), because
// moving one passes the accumulators through ordinary registers and forms a sub-tile twice, and the maxima of such rows jump from
// tile to tile (c_R raises logits up to tenfold): with first references and moves at the maximum itself 252 frames of 1560, d = 128, logits of
// deviation 20 / 30 in natural units, take 394 / 513 us without values, with this headroom 351 / 369 (ordinary logits 340).  Sharp are rows whose first 32 logits
// span more than 40 log2 units, and rows that have to move; the fp32 rounding of logits of that size costs c_L as much as the headroom does.
// Every row 2^64 above its maximum instead cost c_L a digit: largest error for deviations 1 / 3 / 20, 2 x 1560 rows, d = 128: 1.9e-5 /
// 3.5e-5 / 2.1e-5, now 1.3e-6 / 4.5e-6 / 8.4e-6; d = 64 2.0e-5 / 2.4e-5 / 1.9e-5, now 1.2e-6 / 4.9e-6 / 8.4e-6 (flash_kernel, at most 2^8
// below the maximum: 2.7e-6 / 8.5e-6 / 4.4e-6).  It also drove products with values below 2^-62 under the smallest normal number.
// STEP_MAX2 * 2^HEADROOM2 must stay below 2^102: the factor that a move rescales by is then normal wherever old sums still count.
constexpr float HEADROOM2 = 32.0f;
// A row that a wave's move finds this far above its reference (log2 units) is taken for sharp and moves along.
constexpr float MOVE_ALONG2 = 8.0f;

// The headroom of a row's first reference from its first 32 logits, which span `top` downwards.
__device__ __forceinline__ float first_headroom(const f32x16& s, float sc, float top) {
  f32x16 neg;
#pragma unroll
  for (int r = 0; r < 16; ++r) neg[r] = -s[r];
  const float bottom = fmaxf(-subtile_max(neg) * sc, NEG_BIG);
  return fminf(fmaxf(0.8f * (top - bottom) - 32.0f, 0.f), HEADROOM2);
}

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Nothing moves across this line in the instruction schedule.
#define F2_FENCE() __builtin_amdgcn_sched_barrier(0)
// The hardware does not interlock an MFMA's result against plain vector instructions: passes + 3 = 11 issue
// slots must lie between the issue of this 8-pass MFMA and the first instruction that reads (or
// overwrites) what it writes.  The MFMAs of this kernel are inline assembly, which the compiler's hazard
// handling cannot see, so wherever vector code follows an MFMA closely this wait is written out.
#define F2_MFMA_RESULT_WAIT() asm volatile("s_nop 7\n\ts_nop 3" ::: "memory")

// Key rows per LDS tile: 64, or 32 where two workgroups are to share a compute unit and the tiles of keys and values would leave LDS
// for one.
template <int D, bool OUT_V, int Q2, int BIAS, bool PAIRED = false>
constexpr int tile_rows() {
  return (D == 128 || BIAS != 0 || PAIRED) && OUT_V && Q2 == 1 ? 32 : 64;
}

// ENT: c_L not wanted (0), online (1) or in the identity form (2)
// Q2: 32-query tiles per wave; W2 Q2 of them are the workgroup's query block
// BIAS: the temporal factor's passes (launch_l_update_flash2): the logit of (query r, key l) is sc (q . k) + kb_scale kbias[key row l]
// (kbias indexed like the key rows), and rows of a problem need not be adjacent.  1: with OUT_K only the rows' log-sum-exp is
// wanted and no product formed, with OUT_V the products with the values.  2: the reference of query r is given, qb_scale qbias[query row r],
// the sums stay unnormalised and the sum of the weights goes to `cl`.
// PAIRED: one of two kinds of blocks in a launch (flash2_pair_kernel).
template <int D, bool OUT_K, bool OUT_V, int ENT, bool SPLIT, int Q2, int BIAS, bool PAIRED = false>
__device__ __forceinline__ void flash2_block(const FlashParams& P, const int bid) {
  using G = RowGeo<D>;
  constexpr int ROW_BYTES = G::ROW_BYTES;
  constexpr int BT = tile_rows<D, OUT_V, Q2, BIAS, PAIRED>();
  constexpr int TILE_BYTES = BT * ROW_BYTES;
  constexpr int KS = G::KS;                   // k-steps of S^T = K Q^T
  constexpr int CT = G::CT;                   // 32-channel tiles of an output row
  constexpr int CH = G::CH;                   // 16-byte chunks per row
  constexpr int RPI = G::RPI;                 // rows filled by one 64-lane global -> LDS load
  constexpr int V_OFF = NSLOT * TILE_BYTES;   // the V slots follow the K slots
  constexpr bool LSE_ONLY = BIAS == 1 && OUT_K;
  constexpr int NX = LSE_ONLY ? 0 : (OUT_K ? 1 : 0) + (OUT_V ? 1 : 0);  // accumulator sets: [R K][R V]
  constexpr int XV = OUT_K ? 1 : 0;                       // index of the R V set
  static_assert(OUT_K || OUT_V, "at least one product");
  static_assert(BIAS == 0 || (!SPLIT && ENT == 0 && OUT_K != OUT_V), "the biased modes are whole-range passes without entropy");
  constexpr bool TIGHT = D == 128 && NX == 2 && Q2 == 1;  // two workgroups on a unit: 128 + 128 registers are just enough
  constexpr int BQ2 = 32 * Q2 * W2;  // query rows per workgroup
  auto swz = [](int row) { return G::swz(row); };
  extern __shared__ __attribute__((aligned(16))) char smem[];  // [K|V][NSLOT][64 rows][2 D bytes]

  // XCD-aware placement: hardware deals workgroups to the 8 XCDs round-robin, so give each
  // XCD one contiguous range of work items; the query blocks of one (head, frame) then share
  // that XCD's L2 copy of the frame's K and V.
  const int wid = (bid & 7) * P.blocks_per_xcd + (bid >> 3);
  if (wid >= P.total_blocks) return;
  const int per_problem = P.nqb * P.nsplit;
  const int prob = wid / per_problem;
  const int rem = wid - prob * per_problem;
  // the query blocks of one key range are neighbours: they stream the same K and V tiles at
  // the same time and share them through the XCD's L2
  const int split = rem / P.nqb;
  const int qb = rem - split * P.nqb;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int ql = lane & 31;
  const int g = lane >> 5;

  const int kbeg = split * P.keys_per_split;
  const int kend = min(P.nk, kbeg + P.keys_per_split);
  const int nkeys = kend - kbeg;
  const int ntiles = (nkeys + BT - 1) / BT;
  const int last_left = nkeys - (ntiles - 1) * BT;  // 1 .. BT keys in the last tile
  const long long rs = BIAS != 0 ? P.row_stride : 1;  // distance between consecutive rows of a problem
  const int p_out = BIAS != 0 ? prob / P.inner : prob, p_in = BIAS != 0 ? prob - p_out * P.inner : 0;
  const long long qrow0 = (long long)p_out * P.q_rows_per_problem + p_in;
  const long long krow0 = (long long)p_out * P.k_rows_per_problem + p_in + kbeg * rs;
  const char* kbase = reinterpret_cast<const char*>(P.k + krow0 * D);
  const char* vbase = OUT_V ? reinterpret_cast<const char*>(P.v + krow0 * D) : nullptr;

  // ---- global -> LDS staging (global_load_lds_dwordx4) --------------------------------------
  // One wave instruction fills 64 consecutive 16-byte slots (RPI key rows); slot = key * CH +
  // physical chunk.  Wave w issues the instructions for key rows RPI (W2 r + w) .. + RPI - 1
  // (r = 0 .. NR - 1); each lane fetches the logical chunk that belongs in its slot: its byte offset
  // inside a tile is a per-lane constant (goff[r]), the tile's address a wave-uniform base.
  // Rows past the end of the key range are clamped to the last valid row: finite data whose
  // logits are pushed far down again before they are exponentiated (and which cannot change a row
  // maximum, being copies).
  // The loads are inline assembly on purpose: issued through the builtin, the compiler treats
  // them as LDS writes that any later LDS read may alias and waits for them (vmcnt(0)) in front of
  // the next LDS read, a few instructions after they were issued.  The loop below waits for them
  // itself, before the barrier that publishes a tile.  Loads the compiler does not know about
  // only make its own vmcnt waits longer, never shorter: the counter retires in order.
  constexpr int NR = BT / (RPI * W2);
  static_assert(BT % (RPI * W2) == 0, "every wave issues the same number of loads per tile");
  static_assert((RPI * W2) % 16 == 0, "the rows of one lane share a swizzle");
  const int st_key = RPI * wave + lane / CH;  // + RPI W2 r
  const int st_lc = (lane % CH) ^ swz(st_key);
  unsigned goff[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) goff[r] = (unsigned)((RPI * W2 * r + st_key) * ROW_BYTES + st_lc * 16);
  // Biased modes, whose rows lie far apart: the same in 64 bits.  Formed anew for every tile, the products with the row distance were 93
  // instructions of the one wave on a SIMD, 12 of them at a quarter of the rate.
  long long far[NR];
  if (BIAS != 0) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      far[r] = (RPI * W2 * r + st_key) * rs * ROW_BYTES + st_lc * 16;
      asm volatile("" : "+v"(far[r]));
    }
  }
  const unsigned lds_base = (unsigned)(unsigned long long)(__attribute__((address_space(3))) char*)smem;
  auto issue_tile = [&](int t) __attribute__((always_inline)) {  // into slot t & 3
    const unsigned kb = lds_base + (t & (NSLOT - 1)) * TILE_BYTES;
    const char* ksrc = kbase + t * rs * TILE_BYTES;
    const char* vsrc = OUT_V ? vbase + t * rs * TILE_BYTES : nullptr;
    const bool ragged = t == ntiles - 1 && last_left < BT;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      unsigned off = goff[r];
      if (ragged) off = (unsigned)(min(RPI * W2 * r + st_key, last_left - 1) * ROW_BYTES + st_lc * 16);
      // wave-uniform LDS byte address in M0; lane lands at + 16 * lane
      const unsigned dst = __builtin_amdgcn_readfirstlane(kb + (RPI * W2 * r + RPI * wave) * ROW_BYTES);
      if (BIAS != 0) {
        long long at = far[r];
        if (ragged) at = min(RPI * W2 * r + st_key, last_left - 1) * rs * ROW_BYTES + st_lc * 16;
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(ksrc + at), "s"(dst) : "memory", "m0");
        if (OUT_V) {
          const unsigned vdst = dst + V_OFF;
          asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(vsrc + at), "s"(vdst) : "memory", "m0");
        }
        continue;
      }
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(ksrc), "s"(dst) : "memory", "m0");
      if (OUT_V) {
        const unsigned vdst = dst + V_OFF;
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(vsrc), "s"(vdst) : "memory", "m0");
      }
    }
  };
  // the first two tiles go out before anything else so that they travel while Q is fetched
  if (ntiles > 0) issue_tile(0);
  if (ntiles > 1) issue_tile(1);
  // Step 0 has no predecessor and multiplies P^T = 0 with slot 3 of K (and of V): clear those
  // slots, LDS may hold NaN patterns from whoever used it last (0 * NaN would poison the
  // accumulators).
  {
    const uint4 z = {0u, 0u, 0u, 0u};
    static_assert(TILE_BYTES % (16 * 64 * W2) == 0, "the clear covers the slot exactly");
#pragma unroll
    for (int r = 0; r < TILE_BYTES / (16 * 64 * W2); ++r) {
      if (OUT_K) *reinterpret_cast<uint4*>(smem + 3 * TILE_BYTES + (r * 64 * W2 + tid) * 16) = z;
      if (OUT_V) *reinterpret_cast<uint4*>(smem + V_OFF + 3 * TILE_BYTES + (r * 64 * W2 + tid) * 16) = z;
    }
  }

  // Biased modes: the keys' terms behind the tile slots, in units of the raw product (divided by the scale of a logit), so that they can be
  // the value a logit's accumulation starts from.  One sub-tile past the end is read (and its logits dropped).
  constexpr int KB_OFF = (OUT_V ? 2 : 1) * NSLOT * TILE_BYTES;
  if (BIAS != 0) {
    float* kb_lds = reinterpret_cast<float*>(smem + KB_OFF);
    const float f = P.kb_scale / (P.row_scale * LOG2E);
    for (int l = tid; l < ntiles * BT + 32; l += 64 * W2) kb_lds[l] = l < nkeys ? f * P.kbias[krow0 + l * rs] : 0.f;
  }

  // The row of the problem that query row r stands for: the same, or (exact rows) what a list says; -1 if there is none.
  auto row_of = [&](int r) __attribute__((always_inline)) -> int {
    if (r >= P.nq) return -1;
    if (OUT_K || P.q_index == nullptr) return r;
    const int i = P.q_index[r];
    return i >= 0 && i < P.q_index_limit ? i : -1;
  };
  // Query row r as the B operand of S^T = K Q^T; returns its logit scale (log2 units).
  auto load_query = [&](int r, bf16x8 (&x)[KS]) __attribute__((always_inline)) -> float {
    const int row = max(row_of(min(r, P.nq - 1)), 0);
    const bf16_t* qp = P.q + (qrow0 + row * rs) * D + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) x[ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks);
    const float c = BIAS == 0 && P.cR ? P.cR[qrow0 + row] : 1.0f;
    if (BIAS != 0) return P.row_scale * LOG2E;
    return P.row_scale * LOG2E / fmaxf(c, P.cr_min);
  };

  // LDS read addresses, one register each, everything else of an address is an instruction immediate.
  // Row reads (A of S^T): key row = 32 st + ql, logical chunk 2 ks + g.
  unsigned a_off[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) a_off[ks] = lds_base + ql * ROW_BYTES + (((2 * ks + g) ^ swz(ql)) << 4);
  // Transpose reads (A of O^T += X^T P^T): 16-lane group u = lane / 16 -> g = u / 2, channel
  // half u & 1; lane r' of the group supplies key (r' / 4) and channels 4 (r' & 3) .. + 3.  The V slots
  // lie beyond the reach of the 16-bit offset field, hence a second set of registers for them.
  constexpr int NTO = NX == 2 && 2 * NSLOT * TILE_BYTES > 65536 ? 2 : 1;  // the 16-bit offset field reaches 64 KB
  constexpr int V_IMM = NX == 2 && NTO == 1 ? V_OFF : 0;
  unsigned t_off[NTO][CT][2];
  {
    const int rp = lane & 15;
    const int chh = (lane >> 4) & 1;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        const int key = 8 * hh + 4 * g + (rp >> 2);  // + 32 st + 16 c added as an immediate
        const int lc = 4 * ct + 2 * chh + ((rp >> 1) & 1);
        const unsigned o = lds_base + key * ROW_BYTES + ((lc ^ swz(key)) << 4) + ((rp & 1) << 3);
        if (OUT_K) t_off[0][ct][hh] = o;
        if (OUT_V && (!OUT_K || NTO == 2)) t_off[NTO - 1][ct][hh] = o + V_OFF;
      }
  }
  // keep the compiler from re-deriving these from one another inside the loop
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(a_off[ks]));
#pragma unroll
  for (int x = 0; x < NTO; ++x)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) asm volatile("" : "+v"(t_off[x][ct][0]), "+v"(t_off[x][ct][1]));
  typedef __attribute__((address_space(3))) const bf16x8* lds_b128_ptr;
  typedef __attribute__((address_space(3))) bf16x4* lds_b64_ptr;
  auto rd_row = [&](auto kc, int off) __attribute__((always_inline)) -> bf16x8 {  // A of k-step kc, keys at byte offset off
    return *(lds_b128_ptr)(unsigned long long)(a_off[decltype(kc)::value] + off);
  };
  auto rd_tr = [&](unsigned addr) __attribute__((always_inline)) -> bf16x4 {
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_b64_ptr)(unsigned long long)addr);
  };

  // ---- the MFMAs, as inline assembly ---------------------------------------------------------
  // With more than 256 registers per wave the compiler gives every MFMA it selects itself an
  // accumulation-register result, which plain vector instructions cannot read; here the logits must land in
  // ordinary registers (the softmax consumes them element by element) and the products in accumulation
  // registers.  Consecutive MFMAs that accumulate into exactly the registers the previous one wrote need
  // no wait; a vector instruction that reads a result does (F2_MFMA_RESULT_WAIT, or enough MFMAs issued in
  // between: each one waits for the pipe, 8 passes).
  auto mfma_first = [&](f32x16& acc, const bf16x8& a, const bf16x8& b) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
  };
  // acc = c + a b into registers of its own: a starting value put into acc itself could get there by plain moves right before the
  // MFMA, which it would not wait for
  auto mfma_from = [&](f32x16& acc, const bf16x8& a, const bf16x8& b, const f32x16& c) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(acc) : "v"(a), "v"(b), "v"(c));
  };
  auto mfma_v = [&](f32x16& acc, const bf16x8& a, const bf16x8& b) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
  };
  auto mfma_a = [&](f32x16& acc, const bf16x8& a, const bf16x8& b) __attribute__((always_inline)) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
  };

  // ---- queries: B operand of S^T = K Q^T, kept in registers -------------------------------
  bf16x8 qreg[Q2][KS];
  float sc[Q2];
#pragma unroll
  for (int qt = 0; qt < Q2; ++qt) sc[qt] = load_query(qb * BQ2 + wave * (32 * Q2) + qt * 32 + ql, qreg[qt]);

  // ---- accumulators and statistics ---------------------------------------------------------
  // The products accumulate in accumulation registers (constraint "a" below): with the two query tiles,
  // the logits and the queries in the 256 ordinary registers, 2 x 2 x CT tiles of 16 live there.
  f32x16 oacc[NX > 0 ? NX : 1][Q2][CT];
#pragma unroll
  for (int x = 0; x < NX; ++x)
#pragma unroll
    for (int qt = 0; qt < Q2; ++qt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[x][qt][ct][r] = 0.f;
  float msc[Q2], ltil[Q2], lsum[Q2], hsum[Q2];
#pragma unroll
  for (int qt = 0; qt < Q2; ++qt) {
    msc[qt] = NEG_BIG;
    ltil[qt] = 0.f;
    lsum[qt] = 0.f;
    hsum[qt] = 0.f;
    if (BIAS == 2) msc[qt] = P.qb_scale * P.qbias[qrow0 + min(qb * BQ2 + wave * (32 * Q2) + qt * 32 + ql, P.nq - 1) * rs];
  }

  // ---- one step = one 32-key sub-tile, as a fixed sequence of groups ------------------------
  // Software pipeline over sub-tiles n = 0, 1, ...  Step n carries, in the one wave,
  //   matrix:  S^T of sub-tile n+1 (all query tiles), then O^T += X^T P^T of sub-tile n-1;
  //   vector:  p = 2^t, sums and bf16 P^T of sub-tile n, whose sums then say whether its references held.
  // A group is the MFMAs (one per query tile) that share one A operand from LDS: KS groups of
  // logits, then 2 CT NX groups of products in the order (16-key half c, channel tile ct, product x).  The
  // operand of group i + PF is requested while group i runs (a ring of operand registers whose length divides NG, so that
  // ring positions repeat from step to step and, with two sub-tiles per tile, the requests run on across steps, tiles and barriers).  The vector work is cut into pieces that are dealt to the MFMA slots so that no
  // slot carries more than an MFMA's worth of it when there is enough matrix work to hide it.
  constexpr int NPV = 2 * CT * NX;
  constexpr int NG = KS + NPV;
  constexpr int NSL = Q2 * NG;  // MFMA slots per step
  constexpr int PF = TIGHT ? 1 : 2;  // groups between an operand's request and its use
  constexpr int RING = TIGHT ? 2 : 4;
  static_assert(NG % RING == 0 && RING > PF, "ring positions repeat from step to step");
  bf16x8 ring[RING];
  // request the A operand of group `gi` of a step whose logits come from byte offset s_off (slot and
  // sub-tile of the K tile) and whose products read byte offset pv_off (slot and sub-tile, K and V alike)
  auto request = [&](auto gc, int s_off, int pv_off) __attribute__((always_inline)) {
    constexpr int GI = decltype(gc)::value;
    if constexpr (GI < KS) {
      ring[GI % RING] = rd_row(gc, s_off);
    } else if constexpr (NX > 0) {
      constexpr int h = GI - KS;
      constexpr int c = h / (CT * NX);
      constexpr int ct = (h % (CT * NX)) / NX;
      constexpr int x = h % NX;
      const bf16x4 lo = rd_tr(t_off[NTO == 2 ? x : 0][ct][0] + pv_off + (c * 16 * ROW_BYTES + (x == 1 ? V_IMM : 0)));
      const bf16x4 hi = rd_tr(t_off[NTO == 2 ? x : 0][ct][1] + pv_off + (c * 16 * ROW_BYTES + (x == 1 ? V_IMM : 0)));
      ring[GI % RING] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  };
  // Biased modes: the terms of the keys of sub-tile `sub` (32 sub .. 32 sub + 31), which their logits start from
  const unsigned kb_base = lds_base + KB_OFF + 16 * g;
  typedef __attribute__((address_space(3))) const f32x4* lds_f32x4_ptr;
  f32x16 kterm;
  auto load_kterm = [&](int sub) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const f32x4 kb = *(lds_f32x4_ptr)(unsigned long long)(kb_base + 128 * sub + 32 * c);
#pragma unroll
      for (int e = 0; e < 4; ++e) kterm[4 * c + e] = kb[e];
    }
  };

  auto issue = [&](auto gc, auto qc, f32x16 (&snext)[Q2], bf16x8 (&pbprev)[Q2][2]) __attribute__((always_inline)) {
    constexpr int GI = decltype(gc)::value;
    constexpr int qt = decltype(qc)::value;
    if constexpr (GI == 0 && BIAS != 0) {
      mfma_from(snext[qt], ring[GI % RING], qreg[qt][GI], kterm);
    } else if constexpr (GI == 0) {
      mfma_first(snext[qt], ring[GI % RING], qreg[qt][GI]);
    } else if constexpr (GI < KS) {
      mfma_v(snext[qt], ring[GI % RING], qreg[qt][GI]);
    } else if constexpr (NX > 0) {
      constexpr int h = GI - KS;
      constexpr int c = h / (CT * NX);
      constexpr int ct = (h % (CT * NX)) / NX;
      constexpr int x = h % NX;
      mfma_a(oacc[x][qt][ct], ring[GI % RING], pbprev[qt][c]);
    }
  };

  // vector pieces
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
  bf16x2 ones2;
  ones2[0] = (__bf16)1.0f;
  ones2[1] = (__bf16)1.0f;
  // Two scores of one query tile: t = s sc - m, p = 2^t, bf16 pair, sums of the rounded p, of p and of p t.  The three
  // stages of a pair (scale, exponent, the rest) are dependent instructions; each stage goes to an MFMA slot of its
  // own (the stages that share a slot then belong to different pairs and issue back to back), so that a single
  // wave does not sit out the latency of its own chain.
  float tq[2][2], pq[2][2];  // in flight between the stages, by parity of the pair
  float ltstep[Q2], lstep[Q2], hstep[Q2];  // this step's part of the sums
  auto score_scale = [&](auto kc, f32x16 (&scur)[Q2]) __attribute__((always_inline)) {
    constexpr int K = decltype(kc)::value;  // 0 .. 8 Q2 - 1
    constexpr int qt = K % Q2;
    constexpr int j = K / Q2;
    tq[K & 1][0] = __builtin_fmaf(scur[qt][2 * j], sc[qt], -msc[qt]);
    tq[K & 1][1] = __builtin_fmaf(scur[qt][2 * j + 1], sc[qt], -msc[qt]);
  };
  auto score_exp = [&](auto kc) __attribute__((always_inline)) {
    constexpr int K = decltype(kc)::value;
    pq[K & 1][0] = __builtin_amdgcn_exp2f(tq[K & 1][0]);
    pq[K & 1][1] = __builtin_amdgcn_exp2f(tq[K & 1][1]);
  };
  auto score_sums = [&](auto kc, bf16x8 (&pbcur)[Q2][2]) __attribute__((always_inline)) {
    constexpr int K = decltype(kc)::value;
    constexpr int qt = K % Q2;
    constexpr int j = K / Q2;
    if (LSE_ONLY) {  // no weights: the sum of the unrounded ones
      ltstep[qt] = (j == 0 ? pq[K & 1][0] : ltstep[qt] + pq[K & 1][0]) + pq[K & 1][1];
      asm volatile("" : "+v"(ltstep[qt]));
      return;
    }
    bf16x2 pr;
    pr[0] = (__bf16)pq[K & 1][0];  // round to nearest even; the pair is one v_cvt_pk_bf16_f32
    pr[1] = (__bf16)pq[K & 1][1];
    if (ENT == 1) {
      lstep[qt] = j == 0 ? pq[K & 1][0] : lstep[qt] + pq[K & 1][0];
      hstep[qt] = j == 0 ? pq[K & 1][0] * tq[K & 1][0] : __builtin_fmaf(pq[K & 1][0], tq[K & 1][0], hstep[qt]);
      lstep[qt] += pq[K & 1][1];
      hstep[qt] = __builtin_fmaf(pq[K & 1][1], tq[K & 1][1], hstep[qt]);
    }
    // last, so that it does not wait for the conversion (12 x 32 frames of 2048, d = 64, last update: 753 -> 734 us)
    ltstep[qt] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones2, j == 0 ? 0.f : ltstep[qt], false);
    pbcur[qt][j >> 2][2 * (j & 3)] = pr[0];
    pbcur[qt][j >> 2][2 * (j & 3) + 1] = pr[1];
    asm volatile("" : "+v"(ltstep[qt]));
    if (ENT == 1) asm volatile("" : "+v"(lstep[qt]), "+v"(hstep[qt]));
  };
  // rows keys_left .. 31 of the last sub-tile are copies of the last valid row: push their logits far down so that they get
  // probability zero
  auto mask_tail = [&](f32x16 (&s)[Q2], int keys_left) __attribute__((always_inline)) {
    // register r is key 8 (r / 4) + 4 g + r % 4; compared as below the lane keeps one limit, not sixteen key numbers across the loop
    int limit = keys_left - 4 * g;
    asm volatile("" : "+v"(limit));
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float off = 8 * (r >> 2) + (r & 3) >= limit ? -1.0e9f : 0.f;
#pragma unroll
      for (int qt = 0; qt < Q2; ++qt) s[qt][r] += off;
    }
  };
  // logits of the 32 keys at byte offset `off` (slot and sub-tile), plain form, ready to be read
  auto plain_logits = [&](int off, f32x16 (&s)[Q2], int sub) __attribute__((always_inline)) {
    if (BIAS != 0) load_kterm(sub);
    static_for<0, KS>([&](auto kc) {
      constexpr int ks = decltype(kc)::value;
      const bf16x8 a = rd_row(kc, off);
      if constexpr (ks == 0) {
#pragma unroll
        for (int qt = 0; qt < Q2; ++qt) {
          if constexpr (BIAS != 0) mfma_from(s[qt], a, qreg[qt][ks], kterm);
          else mfma_first(s[qt], a, qreg[qt][ks]);
        }
      } else {
#pragma unroll
        for (int qt = 0; qt < Q2; ++qt) mfma_v(s[qt], a, qreg[qt][ks]);
      }
    });
    F2_MFMA_RESULT_WAIT();
    F2_FENCE();
  };
  // Rows of query tile qt that have outgrown their reference take one of HEADROOM2 above `cand`; everything so far is rescaled
  // (App. B: h <- a h + a log(a) l).
  auto move_reference = [&](int qt, float cand) __attribute__((always_inline)) {
    const float m = cand > msc[qt] + MOVE_ALONG2 ? cand + HEADROOM2 : msc[qt];
    const float dl = msc[qt] - m;  // log2 of the rescale factor, <= 0
    const float alpha = __builtin_amdgcn_exp2f(dl);
    if (ENT == 1) {
      hsum[qt] = alpha * (hsum[qt] + dl * lsum[qt]);
      lsum[qt] *= alpha;
    }
    ltil[qt] *= alpha;
    msc[qt] = m;
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        // one tile at a time (the empty statements tie the tile's copies out of and back into the
        // accumulation registers to this place, so they do not pile up beside the loop's registers)
        asm volatile("" : "+a"(oacc[x][qt][ct]));
        scale_acc(oacc[x][qt][ct], alpha);
        asm volatile("" : "+a"(oacc[x][qt][ct]));
        F2_FENCE();
      }
  };
  // A reference has to move: the sub-tile just finished (keys at byte offset `off`; its products are not issued yet) is formed
  // again against new references.
  auto redo = [&](int off, bf16x8 (&pbcur)[Q2][2], int keys_left, int sub) __attribute__((always_inline)) {
    f32x16 s[Q2];
    plain_logits(off, s, sub);
    if (keys_left < 32) mask_tail(s, keys_left);
#pragma unroll
    for (int qt = 0; qt < Q2; ++qt) move_reference(qt, subtile_max(s[qt]) * sc[qt]);
    plain_logits(off, s, sub);  // again: kept meanwhile they would sit beside the copies of the accumulators
    if (keys_left < 32) mask_tail(s, keys_left);
    static_for<0, 8 * Q2>([&](auto kc) {
      score_scale(kc, s);
      score_exp(kc);
      score_sums(kc, pbcur);
    });
    asm volatile("s_nop 1" ::: "memory");
    F2_FENCE();
  };

  // Whether the sub-tile at byte offset `off` holds elements of 2^40 and more (infinities and NaN among them) in a tensor that is multiplied
  auto large_elements = [&](int off) __attribute__((always_inline)) -> bool {
    typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
    typedef __attribute__((address_space(3))) const u32x4* lds_u32x4_ptr;
    typedef __attribute__((__vector_size__(2 * sizeof(uint16_t)))) uint16_t u16x2;
    const unsigned at = lds_base + off + 16 * (threadIdx.x & 63);
    u16x2 largest = {0, 0};
#pragma unroll(TIGHT ? 2 : 4)
    for (int i = 0; i < 32 * ROW_BYTES; i += 1024) {
#pragma unroll
      for (int x = 0; x < NX; ++x) {
        const u32x4 w = *(lds_u32x4_ptr)(unsigned long long)(at + i + (x == XV && OUT_V ? V_OFF : 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) largest = __builtin_elementwise_max(largest, __builtin_bit_cast(u16x2, w[e] & 0x7fff7fffu));
      }
    }
    return __any(max(largest[0], largest[1]) >= 0x5380);  // bf16 bits of 2^40
  };

  // S_OFF / PV_OFF: byte offsets (slot and sub-tile) this step's logits and products read;
  // NS_OFF / NPV_OFF: the same for the step that follows (its first operands are requested here).
  auto step = [&](auto s_c, auto pv_c, auto ns_c, auto npv_c, f32x16 (&scur)[Q2], f32x16 (&snext)[Q2], bf16x8 (&pbprev)[Q2][2],
                  bf16x8 (&pbcur)[Q2][2], int keys_left, int sub) __attribute__((always_inline)) {
    constexpr int S_OFF = decltype(s_c)::value, PV_OFF = decltype(pv_c)::value;
    constexpr int NS_OFF = decltype(ns_c)::value, NPV_OFF = decltype(npv_c)::value;
    if constexpr (NX == 0) F2_MFMA_RESULT_WAIT();  // no products between the logits' last MFMA and here
    F2_FENCE();
    if (keys_left < 32) mask_tail(scur, keys_left);
    if (BIAS != 0) load_kterm(sub + 1);
    F2_FENCE();
    // (with one sub-tile per tile the next step's logits are those of a tile that may still be travelling when this one ends)
    if constexpr (BT == 32) static_for<0, PF>([&](auto gc) { request(gc, S_OFF, PV_OFF); });
    static_for<0, NG>([&](auto gc) {
      constexpr int GI = decltype(gc)::value;
      // request the operand of group GI + PF (of the next step beyond the end of this one)
      if constexpr (GI + PF < NG) {
        request(std::integral_constant<int, GI + PF>{}, S_OFF, PV_OFF);
      } else if constexpr (BT == 64) {
        request(std::integral_constant<int, GI + PF - NG>{}, NS_OFF, NPV_OFF);
      }
      static_for<0, Q2>([&](auto qc) {
        constexpr int SL = Q2 * GI + decltype(qc)::value;
        issue(gc, qc, snext, pbprev);
        // score pairs dealt evenly over the slots: pair k starts in slot floor(k NSL / (8 Q2)), its exponents follow one
        // slot later and its sums two slots later (both clamped to the step's last slot).  Pairs in ascending
        // order, stages in their own order: a pair's stages that meet in one slot stay in sequence, and the sums
        // of pair k come before pair k + 2 reuses its buffers (it starts two slots after pair k; one in the pass without
        // products, whose sums need no exponents).
        static_assert(NSL >= 8 * Q2 || ENT != 1, "the sums of p t find their exponents");
        static_for<0, 8 * Q2>([&](auto kc) {
          constexpr int K = decltype(kc)::value;
          constexpr int S0 = (K * NSL) / (8 * Q2);
          constexpr int S1 = S0 + 1 < NSL ? S0 + 1 : NSL - 1;
          constexpr int S2 = S0 + 2 < NSL ? S0 + 2 : NSL - 1;
          if constexpr (S0 == SL) score_scale(kc, scur);
          if constexpr (S1 == SL) score_exp(kc);
          if constexpr (S2 == SL) score_sums(kc, pbcur);
        });
        F2_FENCE();
      });
    });
#pragma unroll
    for (int qt = 0; qt < Q2; ++qt)
      if (!LSE_ONLY) asm volatile("" : "+v"(pbcur[qt][0]), "+v"(pbcur[qt][1]));
    constexpr float LIMIT = LSE_ONLY ? STEP_MAX2 : STEP_LARGE2;
    if (BIAS != 2 && __any(ltstep[0] > LIMIT || ltstep[Q2 - 1] > LIMIT)) {
      if (LSE_ONLY || __any(ltstep[0] > STEP_MAX2 || ltstep[Q2 - 1] > STEP_MAX2) || large_elements(NPV_OFF)) redo(NPV_OFF, pbcur, keys_left, sub);
    }
#pragma unroll
    for (int qt = 0; qt < Q2; ++qt) {
      ltil[qt] += ltstep[qt];
      if (ENT == 1) {
        lsum[qt] += lstep[qt];
        hsum[qt] += hstep[qt];
      }
    }
  };
  if (ntiles > 0) {
    // Four LDS slots, tile t in slot t & 3: during tile t the products of the last sub-tile of
    // tile t-1 are still outstanding, tile t+1 is resident (its first sub-tile is needed one
    // step ahead) and tile t+2 is in flight.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    f32x16 sA[Q2], sB[Q2];
    bf16x8 pbA[Q2][2], pbB[Q2][2];
    {
      const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int qt = 0; qt < Q2; ++qt)
#pragma unroll
        for (int c = 0; c < 2; ++c) pbB[qt][c] = zero;  // step 0 has no predecessor: it adds P^T = 0
    }
    // A wave whose query rows all lie past the end of the problem (the tail of the last query
    // block) only helps to load the tiles.
    const bool active = qb * BQ2 + wave * (32 * Q2) < P.nq;
    if (active) {
      // logits of sub-tile 0, plain form; their row maxima are the first references
      plain_logits(0, sA, 0);
      if (BIAS != 2) {
        float head[Q2];
        bool sharp = false;
#pragma unroll
        for (int qt = 0; qt < Q2; ++qt) {
          msc[qt] = fmaxf(subtile_max(sA[qt]) * sc[qt], NEG_BIG);
          head[qt] = first_headroom(sA[qt], sc[qt], msc[qt]);
          sharp = sharp || head[qt] >= HEADROOM2;
        }
        // in sharp rows the first 32 logits say little of the rest: the maxima of all keys that are here (252 frames of 1560, d = 128, deviation
        // 30: 462 -> 362 us)
        if (__any(sharp)) {
          const int subs = min(2, ntiles) * (BT / 32);
#pragma unroll 1
          for (int sub = 1; sub < subs; ++sub) {
            plain_logits(sub * 32 * ROW_BYTES, sB, sub);
#pragma unroll
            for (int qt = 0; qt < Q2; ++qt) msc[qt] = fmaxf(msc[qt], subtile_max(sB[qt]) * sc[qt]);
          }
        }
#pragma unroll
        for (int qt = 0; qt < Q2; ++qt) msc[qt] += head[qt];
      }
      // operands of the first groups of the first step (sub-tile 1 of slot 0; products against slot 3)
      if constexpr (BT == 64) static_for<0, PF>([&](auto gc) { request(gc, 32 * ROW_BYTES, 3 * TILE_BYTES + 32 * ROW_BYTES); });
    }
    // Four tiles per trip so that every LDS slot offset is an instruction immediate.
    auto tile_iteration = [&](auto slot_c, int t) __attribute__((always_inline)) {
      constexpr int SLOT = decltype(slot_c)::value;
      if (t > 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();  // tile t+1 has landed for everyone; everyone is done with tile t-2
      }
      if (t + 2 < ntiles) issue_tile(t + 2);
      constexpr int kp = ((SLOT + 3) & 3) * TILE_BYTES;  // tile t-1
      constexpr int kt = SLOT * TILE_BYTES;
      constexpr int kn = ((SLOT + 1) & 3) * TILE_BYTES;
      constexpr int HALF = 32 * ROW_BYTES;  // second sub-tile of a tile
      const int left0 = t == ntiles - 1 ? last_left : BT;
      if (active && BT == 32) {
        // one sub-tile per tile: logits of t+1, products of t-1 [at t = 0: P^T = 0 against the cleared slot 3], softmax of t
        constexpr int k2 = ((SLOT + 2) & 3) * TILE_BYTES;
        step(std::integral_constant<int, kn>{}, std::integral_constant<int, kp>{}, std::integral_constant<int, k2>{},
             std::integral_constant<int, kt>{}, SLOT % 2 ? sB : sA, SLOT % 2 ? sA : sB, SLOT % 2 ? pbA : pbB, SLOT % 2 ? pbB : pbA, left0, t);
      } else if (active) {
        // logits of (t, 1), products of (t-1, 1) [at t = 0: P^T = 0 against the cleared slot 3], softmax of (t, 0);
        // the step after it: logits of (t+1, 0), products of (t, 0)
        step(std::integral_constant<int, kt + HALF>{}, std::integral_constant<int, kp + HALF>{},
             std::integral_constant<int, kn>{}, std::integral_constant<int, kt>{}, sA, sB, pbB, pbA, left0, 2 * t);
        // logits of (t+1, 0), products of (t, 0), softmax of (t, 1); then logits of (t+1, 1), products of (t, 1)
        step(std::integral_constant<int, kn>{}, std::integral_constant<int, kt>{},
             std::integral_constant<int, kn + HALF>{}, std::integral_constant<int, kt + HALF>{}, sB, sA, pbA, pbB, left0 - 32, 2 * t + 1);
      }
    };
    for (int t0_ = 0; t0_ < ntiles; t0_ += 4) {
      tile_iteration(std::integral_constant<int, 0>{}, t0_);
      if (t0_ + 1 < ntiles) tile_iteration(std::integral_constant<int, 1>{}, t0_ + 1);
      if (t0_ + 2 < ntiles) tile_iteration(std::integral_constant<int, 2>{}, t0_ + 2);
      if (t0_ + 3 < ntiles) tile_iteration(std::integral_constant<int, 3>{}, t0_ + 3);
    }
    if (active) {
      // drain: the products of the last sub-tile, (ntiles-1, 1), plain form
      const int pv_off = ((ntiles - 1) & 3) * TILE_BYTES + (BT - 32) * ROW_BYTES;
      // softmax weights of the last sub-tile: the second of a tile, or the only one, whose set goes by the slot
      if (BT == 32 && (ntiles & 1)) {
#pragma unroll
        for (int qt = 0; qt < Q2; ++qt) {
          pbB[qt][0] = pbA[qt][0];
          pbB[qt][1] = pbA[qt][1];
        }
        asm volatile("s_nop 1" ::: "memory");
      }
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int x = 0; x < NX; ++x) {
            const bf16x4 lo = rd_tr(t_off[NTO == 2 ? x : 0][ct][0] + pv_off + (c * 16 * ROW_BYTES + (x == 1 ? V_IMM : 0)));
            const bf16x4 hi = rd_tr(t_off[NTO == 2 ? x : 0][ct][1] + pv_off + (c * 16 * ROW_BYTES + (x == 1 ? V_IMM : 0)));
            const bf16x8 a = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
            for (int qt = 0; qt < Q2; ++qt) mfma_a(oacc[x][qt][ct], a, pbB[qt][c]);
          }
    }
  }
  F2_MFMA_RESULT_WAIT();  // the accumulators are read by plain vector code from here on
#pragma unroll
  for (int x = 0; x < NX; ++x)
#pragma unroll
    for (int qt = 0; qt < Q2; ++qt)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) asm volatile("" : "+a"(oacc[x][qt][ct]));  // ... and not before this line
  F2_FENCE();
  // ---- epilogue ------------------------------------------------------------------------------
  // Normalised rows are staged in LDS (each wave owns the rows it computed, swizzled like the
  // key tiles; the R K rows over the K slots, the R V rows over the V slots) and leave as whole
  // rows, 16 bytes per lane.  Lane-dependent values are derived again from the thread index,
  // behind an opaque copy, so that none of the epilogue's address arithmetic stays live across
  // the key loop.
  __syncthreads();  // every wave is done with the key/value tiles
  int tid_e = threadIdx.x;
  asm volatile("" : "+v"(tid_e));
  const int lane_e = tid_e & 63;
  const int ql_e = lane_e & 31;
  const int g_e = lane_e >> 5;
  const int row_first = qb * BQ2 + wave * (32 * Q2);
  constexpr int STAGE_BYTES = 32 * Q2 * ROW_BYTES;  // per wave and product: W2 of them fill the NSLOT slots exactly
  static_assert(W2 * STAGE_BYTES <= NSLOT * TILE_BYTES, "staged rows fit the slots of their tensor");
#pragma unroll
  for (int qt = 0; qt < Q2; ++qt) {
    F2_FENCE();  // one query tile at a time: both at once need more ordinary registers than the queries leave
    const int qr = row_first + qt * 32 + ql_e;
    const bool qvalid = qr < P.nq;
    const float lt = ltil[qt] + __shfl_xor(ltil[qt], 32);
    const float inv = BIAS == 2 ? 1.0f : lt > 0.f ? 1.0f / lt : 0.f;
    if (!SPLIT) {
      const float l = ENT == 1 ? lsum[qt] + __shfl_xor(lsum[qt], 32) : lt;
      const int r = row_of(qr);
      const long long row = qrow0 + r * rs;
      if (BIAS == 2 && r >= 0 && g_e == 0) P.cl[row] = lt;
      if (BIAS != 2 && P.lse != nullptr && r >= 0 && g_e == 0) P.lse[row] = LN2 * (msc[qt] + __log2f(l));
      if (ENT == 1) {
        // App. B: H = log S - L / S; here in base-2 units, c_L = -H
        const float h = hsum[qt] + __shfl_xor(hsum[qt], 32);
        if (qvalid && g_e == 0) P.cl[row] = LN2 * (h / l - __log2f(l));
      }
      if (ENT == 2) {
        const float mean_t = row_dot<D>(qreg[qt], oacc[0][qt]) * inv * sc[qt];  // sum_l R_l (s_l sc), log2 units
        if (qvalid && g_e == 0) P.cl[row] = LN2 * (mean_t - (msc[qt] + __log2f(l)));
      }
      // lane (q, g) holds channels 32 ct + 8 c + 4 g .. + 3 of query q: 8-byte pieces
#pragma unroll
      for (int x = 0; x < NX; ++x) {
        // one product at a time (as in the rescale above: its copies out of the accumulation registers start here)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) asm volatile("" : "+a"(oacc[x][qt][ct]));
        F2_FENCE();
        char* stage = smem + (x == XV && OUT_V ? V_OFF : 0) + wave * STAGE_BYTES;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            uint2 w;
            w.x = pack_bf16(oacc[x][qt][ct][4 * c + 0] * inv, oacc[x][qt][ct][4 * c + 1] * inv);
            w.y = pack_bf16(oacc[x][qt][ct][4 * c + 2] * inv, oacc[x][qt][ct][4 * c + 3] * inv);
            *reinterpret_cast<uint2*>(stage + (32 * qt + ql_e) * ROW_BYTES + (((4 * ct + c) ^ swz(ql_e)) << 4) + 8 * g_e) = w;
          }
      }
    } else {
      // partial result of this key range: normalised output and log2-sum-exp
      if (qvalid) {
        const long long nprob = P.total_blocks / (P.nqb * P.nsplit);
        const long long prow = ((long long)split * nprob + prob) * P.nq + qr;
        if (g_e == 0) P.part_lse[prow] = lt > 0.f ? msc[qt] + __log2f(lt) : NEG_BIG;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int ch = 32 * ct + 8 * c + 4 * g_e;
            const float4 w = {oacc[NX - 1][qt][ct][4 * c + 0] * inv, oacc[NX - 1][qt][ct][4 * c + 1] * inv,
                              oacc[NX - 1][qt][ct][4 * c + 2] * inv, oacc[NX - 1][qt][ct][4 * c + 3] * inv};
            *reinterpret_cast<float4*>(P.part_o + prow * D + ch) = w;
          }
      }
    }
  }
  if (!SPLIT) {
    // the staged rows are private to the wave: no barrier, only the LDS writes above must land
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int x = 0; x < NX; ++x) {
      const char* stage = smem + (x == XV && OUT_V ? V_OFF : 0) + wave * STAGE_BYTES;
      bf16_t* dst = (x == XV && OUT_V) ? P.outv : P.outk;
#pragma unroll
      for (int ps = 0; ps < 32 * Q2 / RPI; ++ps) {
        const int lr = ps * RPI + lane_e / CH;  // row within the wave's block
        const int pc = lane_e % CH;
        const int lc = pc ^ swz(lr);
        const int r = row_of(row_first + lr);
        if (r >= 0) {
          uint4 w = *reinterpret_cast<const uint4*>(stage + lr * ROW_BYTES + pc * 16);
          uint4* gp = reinterpret_cast<uint4*>(dst + (qrow0 + r * rs) * D + lc * 8);
          if (P.blend) w = average_bf16x8(w, *gp);
          *gp = w;
        }
      }
    }
  }
}

template <int D, bool OUT_K, bool OUT_V, int ENT, bool SPLIT, int Q2, int BIAS>
__global__ void __launch_bounds__(64 * W2, D == 128 && OUT_K && OUT_V && Q2 == 1 ? 2 : 1) flash2_kernel(FlashParams P) {
  flash2_block<D, OUT_K, OUT_V, ENT, SPLIT, Q2, BIAS>(P, blockIdx.x);
}

// A fitting update without values (blocks 0 .. na - 1, na a multiple of 8) and the key ranges of exact rows in one launch.
template <int D>
__global__ void __launch_bounds__(64 * W2, 2) flash2_pair_kernel(FlashParams A, FlashParams B, int na) {
  if ((int)blockIdx.x < na) flash2_block<D, true, false, 1, false, 1, 0, true>(A, blockIdx.x);
  else flash2_block<D, false, true, 0, true, 1, 0, true>(B, blockIdx.x - na);
}

// Block counts of a launch of `problems` problems
hipError_t count_blocks(FlashParams& P, long long problems, int block_rows) {
  P.nqb = (P.nq + block_rows - 1) / block_rows;
  const long long total = problems * P.nqb * P.nsplit;
  if (total > 0x3fffffffLL) return hipErrorInvalidValue;
  P.total_blocks = (int)total;
  P.blocks_per_xcd = (P.total_blocks + 7) / 8;
  return hipSuccess;
}

template <int D, bool OUT_K, bool OUT_V, int ENT, bool SPLIT, int Q2, int BIAS = 0>
hipError_t launch_flash2(FlashParams P, long long problems, hipStream_t st) {
  constexpr int ROWS = 32 * Q2;  // per wave
  // four K slots always (the logits need them), four V slots when values are multiplied: 128 KB at d = 128
  constexpr int BT = tile_rows<D, OUT_V, Q2, BIAS>();
  constexpr int TILE_LDS = (OUT_V ? 2 : 1) * NSLOT * BT * D * 2;
  constexpr int MAX_LDS = TILE_LDS + (BIAS != 0 ? (kMaxBiasedKeys + 32) * 4 : 0);
  static_assert(MAX_LDS <= 160 * 1024 && kMaxBiasedKeys % BT == 0, "a unit's LDS holds the tiles and the longest row of key terms");
  const int lds = TILE_LDS + (BIAS != 0 ? ((P.nk + BT - 1) / BT * BT + 32) * 4 : 0);
  if (lds > MAX_LDS) return hipErrorInvalidValue;
  const hipError_t ec = count_blocks(P, problems, W2 * ROWS);
  if (ec != hipSuccess) return ec;
  auto kern = flash2_kernel<D, OUT_K, OUT_V, ENT, SPLIT, Q2, BIAS>;
  static bool configured = false;  // the attribute is per function, set once per process
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, MAX_LDS);
    if (e != hipSuccess) return e;
    configured = true;
  }
  hipLaunchKernelGGL(kern, dim3(P.blocks_per_xcd * 8), dim3(64 * W2), lds, st, P);
  return hipGetLastError();
}

#undef F2_FENCE
#undef F2_MFMA_RESULT_WAIT

FlashParams exact_rows_params(const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* out, float* lse, float* part_o, float* part_lse,
                              const Dims& dm, int nrows, const int* rows, int ns, int keys_per_split) {
  FlashParams P = {};
  P.q = q; P.k = k; P.v = v; P.outv = out; P.lse = lse; P.part_o = part_o; P.part_lse = part_lse;
  P.q_index = rows;
  P.q_index_limit = (int)dm.N;
  P.q_rows_per_problem = dm.N; P.k_rows_per_problem = dm.N;
  P.nq = nrows;
  P.nk = (int)dm.N;
  P.nsplit = ns;
  P.keys_per_split = keys_per_split;
  P.row_scale = 1.0f / sqrtf((float)dm.d);
  P.cr_min = 0.f;
  return P;
}
FlashParams r_update_params(const bf16_t* aR, const float* cR, const bf16_t* k, const bf16_t* v, bf16_t* aL, float* cL, bf16_t* y,
                            float* lse, const Dims& dm, float row_scale, float cr_min) {
  FlashParams P = {};
  P.q = aR; P.cR = cR; P.k = k; P.v = v; P.outk = aL; P.outv = y; P.cl = cL; P.lse = lse;
  P.q_rows_per_problem = dm.b; P.k_rows_per_problem = dm.b;
  P.nq = dm.b; P.nk = dm.b;
  P.nsplit = 1;
  P.keys_per_split = ((dm.b + BK - 1) / BK) * BK;
  P.row_scale = row_scale; P.cr_min = cr_min;
  return P;
}
}  // namespace

// Exact attention of nrows query rows per head (a contiguous run, or those of a list) over all keys (Sec. 3.3), the keys
// cut into `ns` ranges of keys_per_split (a multiple of 64) whose partial results go to part_o / part_lse
// for the merge (ns == 1: straight to out / lse); query blocks of 128 rows or of 256.
template <int D>
hipError_t launch_exact_rows_flash2(const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* out, float* lse,
                                    float* part_o, float* part_lse, const Dims& dm, int nrows, const int* rows, int ns,
                                    int keys_per_split, bool short_blocks, hipStream_t st) {
  const FlashParams P = exact_rows_params(q, k, v, out, lse, part_o, part_lse, dm, nrows, rows, ns, keys_per_split);
  if (short_blocks)
    return ns > 1 ? launch_flash2<D, false, true, 0, true, 1>(P, dm.BH, st) : launch_flash2<D, false, true, 0, false, 1>(P, dm.BH, st);
  return ns > 1 ? launch_flash2<D, false, true, 0, true, 2>(P, dm.BH, st) : launch_flash2<D, false, true, 0, false, 2>(P, dm.BH, st);
}

// out <- (out + softmax(q K_F1^T / sqrt(d)) V_F1) / 2 (Sec. 4.4): all N queries of a head against its first frame's b keys.
template <int D>
hipError_t launch_sink_average_flash2(const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* out, const Dims& dm,
                                      hipStream_t st) {
  FlashParams P = {};
  P.q = q; P.k = k; P.v = v; P.outv = out;
  P.q_rows_per_problem = dm.N; P.k_rows_per_problem = dm.N;
  P.nq = (int)dm.N;
  P.nk = dm.b;
  P.nsplit = 1;
  P.keys_per_split = ((dm.b + BK - 1) / BK) * BK;
  P.row_scale = 1.0f / sqrtf((float)D);
  P.cr_min = 0.f;
  P.blend = 1;
  // Short blocks always at d = 128, at d = 64 while long ones do not give every compute unit one (short / long, us: d = 128: 12 heads x
  // 21 frames of 1560 312 / 331, 40 x 60 of 100 47.9 / 65.7; d = 64: 4 x 8 of 1000 17.4 / 23.4, 12 x 21 of 300 17.7 / 17.4, of 1560 196
  // / 160; the one-tile kernel of flash.hip 336, 53.0, 23.2, 21.2, 205).
  if constexpr (D == 64)
    if ((P.nq + 255LL) / 256 * dm.BH > compute_units()) return launch_flash2<D, false, true, 0, false, 2>(P, dm.BH, st);
  return launch_flash2<D, false, true, 0, false, 1>(P, dm.BH, st);
}

// The temporal factor through this kernel, for any number of frames T (Eq. L with Eq. alpha_R / c_R, and
// the apply-to-V of App. A).  A problem is one (head, position i); its rows are the T frames of that position, b rows
// apart in the frame-major tensors.  With u[j,k] = q_scale (Q[j] . alpha_L[k]) - c_L[k]:
//   last sweep     one pass, queries Q[j], keys alpha_L[k] with the additive term -c_L[k], values y[k]:
//                  out[j] = sum_k softmax_k(u[j,:])[k] y[k];
//   fitting sweep  pass 1, the same queries and keys without a product: lse[j] = log sum_k exp u[j,k];
//                  pass 2 with the roles exchanged, queries alpha_L[k] (fixed reference c_L[k]), keys Q[j] with the
//                  additive term -lse[j], values Q[j]: the weights exp(u[j,k] - lse[j]) = L[j,k] are final, so
//                  alpha_R[k] = sum_j L[j,k] Q[j] and c_R[k] = sum_j L[j,k] are plain unnormalised sums.
// lse_scratch: BH * N floats (fitting sweep only).
// The pass for the log-sum-exps keeps no products, a key's term is the value its logits' accumulation starts from, and there is no running
// maximum: vector work, which bounds these passes at d = 64 (0.69 .. 0.81 of the cycles), falls by a quarter.  12 x 64 problems of 512
// frames, d = 64: fitting 128 -> 106 us, last 83 -> 71; 8 x 100 of 300 88 -> 66, 55 -> 44, d = 128 173 -> 112, 109 -> 75.
template <int D>
hipError_t launch_l_update_flash2(const bf16_t* q, const bf16_t* aL, const float* cL, const bf16_t* y, bf16_t* aR, float* cR,
                                  bf16_t* out, float* lse_scratch, const Dims& dm, float q_scale, hipStream_t st) {
  if (dm.T > kMaxBiasedKeys) return hipErrorInvalidValue;
  FlashParams P = {};
  P.q_rows_per_problem = dm.N; P.k_rows_per_problem = dm.N;
  P.inner = dm.b; P.row_stride = dm.b;
  P.nq = dm.T; P.nk = dm.T;
  P.nsplit = 1;
  P.keys_per_split = ((dm.T + BK - 1) / BK) * BK;
  P.row_scale = q_scale;
  P.kb_scale = -LOG2E;
  const long long problems = (long long)dm.BH * dm.b;
  const int units = compute_units();
  const bool short_products = temporal_product_short_blocks(D, y != nullptr, problems, dm.T, units);
  if (y != nullptr) {
    P.q = q; P.k = aL; P.v = y; P.outv = out; P.kbias = cL;
    return short_products ? launch_flash2<D, false, true, 0, false, 1, 1>(P, problems, st) : launch_flash2<D, false, true, 0, false, 2, 1>(P, problems, st);
  }
  if (lse_scratch == nullptr) return hipErrorInvalidValue;
  P.q = q; P.k = aL; P.lse = lse_scratch; P.kbias = cL;
  hipError_t e = temporal_lse_short_blocks(D, problems, dm.T, units) ? launch_flash2<D, true, false, 0, false, 1, 1>(P, problems, st)
                                                                     : launch_flash2<D, true, false, 0, false, 2, 1>(P, problems, st);
  if (e != hipSuccess) return e;
  P.q = aL; P.k = q; P.outk = aR; P.cl = cR; P.lse = nullptr;
  P.kbias = lse_scratch;          // natural log, like c_L: the same scale -log2(e) applies
  P.qbias = cL; P.qb_scale = LOG2E;
  if constexpr (D == 64)
    if (!short_products) return launch_flash2<D, true, false, 0, false, 2, 2>(P, problems, st);
  return launch_flash2<D, true, false, 0, false, 1, 2>(P, problems, st);
}

// One R-update: alpha_L, c_L (and lse if not null), plus y when v is given.
template <int D>
hipError_t launch_r_update_flash2(const bf16_t* aR, const float* cR, const bf16_t* k, const bf16_t* v, bf16_t* aL,
                                  float* cL, bf16_t* y, float* lse, const Dims& dm, float row_scale, float cr_min,
                                  int entropy_mode, hipStream_t st) {
  if (dm.d != D || (v == nullptr) != (y == nullptr)) return hipErrorInvalidValue;
  const FlashParams P = r_update_params(aR, cR, k, v, aL, cL, y, lse, dm, row_scale, cr_min);
  const long long problems = (long long)dm.BH * dm.T;
  const bool short_blocks = update_short_blocks(D, v != nullptr, problems, dm.b, compute_units());
  auto launch = [&](auto ent) -> hipError_t {
    constexpr int ENT = decltype(ent)::value;
    if (v == nullptr)
      return short_blocks ? launch_flash2<D, true, false, ENT, false, 1>(P, problems, st) : launch_flash2<D, true, false, ENT, false, 2>(P, problems, st);
    return short_blocks ? launch_flash2<D, true, true, ENT, false, 1>(P, problems, st) : launch_flash2<D, true, true, ENT, false, 2>(P, problems, st);
  };
  return entropy_mode == VMONARCH_ENTROPY_IDENTITY ? launch(std::integral_constant<int, 2>{}) : launch(std::integral_constant<int, 1>{});
}

// The first fitting update and the key ranges of the first frame's exact rows (ns > 1) in one launch, both in blocks of 128 rows.  The
// exact rows need nothing of the sweeps.  In a call as small as this each of the two launches leaves places on the compute units empty and
// takes one block's time all the same; together they take little more than one.  Whole calls of two sweeps, separate / together, us: 13 frames
// of 323, 10 heads, d = 64 64.6 / 57.1; 13 of 400, 4 heads 52.6 / 44.8, d = 128 73.3 / 63.0; 13 of 300, 4 heads, d = 128 62.2 / 51.8.  Only where all
// blocks of both run at once.
template <int D>
bool update_and_first_frame_supported(const Dims& dm, int ns) {
  auto blocks = [&](long long n) -> long long { return n * ((dm.b + 127) / 128); };
  return ns > 1 && blocks((long long)dm.BH * dm.T) + blocks((long long)dm.BH * ns) <= (D == 64 ? 3 : 2) * compute_units();
}

template <int D>
hipError_t launch_update_and_first_frame_flash2(const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* aL, float* cL, float* part_o,
                                                float* part_lse, const Dims& dm, float row_scale, float cr_min, int ns,
                                                int keys_per_split, hipStream_t st) {
  FlashParams A = r_update_params(q, nullptr, k, nullptr, aL, cL, nullptr, nullptr, dm, row_scale, cr_min);
  FlashParams B = exact_rows_params(q, k, v, nullptr, nullptr, part_o, part_lse, dm, dm.b, nullptr, ns, keys_per_split);
  hipError_t e = count_blocks(A, (long long)dm.BH * dm.T, 32 * W2);
  if (e == hipSuccess) e = count_blocks(B, dm.BH, 32 * W2);
  if (e != hipSuccess) return e;
  constexpr int LDS_A = NSLOT * tile_rows<D, false, 1, 0, true>() * D * 2, LDS_B = 2 * NSLOT * tile_rows<D, true, 1, 0, true>() * D * 2;
  constexpr int LDS_BYTES = LDS_A > LDS_B ? LDS_A : LDS_B;
  auto kern = flash2_pair_kernel<D>;
  static bool configured = false;  // the attribute is per function, set once per process
  if (!configured) {
    e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int na = A.blocks_per_xcd * 8;
  hipLaunchKernelGGL(kern, dim3(na + B.blocks_per_xcd * 8), dim3(64 * W2), LDS_BYTES, st, A, B, na);
  return hipGetLastError();
}

// This file is compiled once per head dimension.
template hipError_t launch_exact_rows_flash2<VM_FLASH2_D>(const bf16_t*, const bf16_t*, const bf16_t*, bf16_t*, float*, float*, float*,
                                                          const Dims&, int, const int*, int, int, bool, hipStream_t);
template bool update_and_first_frame_supported<VM_FLASH2_D>(const Dims&, int);
template hipError_t launch_update_and_first_frame_flash2<VM_FLASH2_D>(const bf16_t*, const bf16_t*, const bf16_t*, bf16_t*, float*, float*, float*,
                                                                      const Dims&, float, float, int, int, hipStream_t);
template hipError_t launch_sink_average_flash2<VM_FLASH2_D>(const bf16_t*, const bf16_t*, const bf16_t*, bf16_t*, const Dims&, hipStream_t);
template hipError_t launch_l_update_flash2<VM_FLASH2_D>(const bf16_t*, const bf16_t*, const float*, const bf16_t*, bf16_t*, float*, bf16_t*,
                                                        float*, const Dims&, float, hipStream_t);
template hipError_t launch_r_update_flash2<VM_FLASH2_D>(const bf16_t*, const float*, const bf16_t*, const bf16_t*, bf16_t*, float*,
                                                        bf16_t*, float*, const Dims&, float, float, int, hipStream_t);

}  // namespace vm
