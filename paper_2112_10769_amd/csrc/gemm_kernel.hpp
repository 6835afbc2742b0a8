// 4-bit GEMMs on INT8 MFMA (gfx950): the tile kernel, shared by the backward /
// update GEMMs (gemm.hip) and the forward GEMM (gemm_fwd.hip).
//
//   C[m][n] = (alpha / ns) * s_B * sum_k A[m][k] * B[n][k]
//
// A holds LUQ codes (Section 4 of the paper; ns SMP planes, Section 5.1), B
// INT4 codes (Section 3.3).  Both operands are K-major nibble matrices; the
// quantizers write whichever layout (row-major or transposed) a GEMM needs,
// so the GEMM never transposes.
//
// Carrier: v_mfma_i32_32x32x32_i8 with exact int32 accumulation.  Codes are
// expanded from nibbles to int8 once per workgroup tile, on the way from
// global memory into LDS:
//   LUQ  : two byte lookups (v_perm_b32) and an xor per four codes
//          (luq_value4).  Two SMP planes are expanded to excess-64 bytes and
//          summed with one word add (|sum| <= 64, no carries).
//   INT4 : the nibble is moved to the top of its byte, giving 16*q (signed,
//          two's complement) or 8*q (unsigned) with no further work; the
//          extra power of two is removed exactly in the epilogue.
// The even-k nibbles of a word land in one int8 word and the odd-k nibbles
// in the next.  Both operands use the same order, so the contraction over
// k is unchanged.
//
// The per-tensor scales are applied once to the int32 sums (Appendix A.1):
//   C = fl32( fl32(acc) * fl32( fl32(alpha / ns) * s_B ) * 2^-4|2^-3 ).
// Long reductions are split along K into chunks whose int32 sums cannot
// overflow; chunk sums are added in int64 in a fixed order.
#pragma once

#include <type_traits>

#include "luq_device.hpp"
#include "luq_launch.hpp"

namespace luq {

// Code type of the A operand.
constexpr int kAcLuq = 0;     // LUQ codes, NS planes (Section 4, 5.1)
constexpr int kAcInt4S = 1;   // signed INT4 codes (-7..7)
constexpr int kAcInt4U = 2;   // unsigned INT4 codes (0..15)
constexpr int kAcSum2 = 3;    // int8 sums of two LUQ samples (Section 5.1), one byte per k

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

// Word 3 of a raw buffer descriptor on gfx9 (32-bit data, no swizzle).
constexpr int kBufferFlags = 0x00020000;
// A buffer offset beyond any operand's range: such loads return zeros.
constexpr int kOutOfRange = 0x7FFFFFF0;

// int32-exact reduction lengths: |A| <= 64 (LUQ) or 120 (INT4 as 16q / 8q),
// |B| <= 120: 2^18 * 7680 < 2^31 and 2^17 * 14400 < 2^31
constexpr int64_t kMaxExactK = 1 << 18;
constexpr int64_t kMaxExactKInt4 = 1 << 17;

// ---- nibble -> int8 expansion ------------------------------------------------

// One LUQ code n = (sign, e) per selector byte -> its int8 value, by two byte
// lookups whose out-of-table selectors cancel.  v_perm_b32 gives table byte n
// for a selector below 8, the sign mask of table byte 1, 3, 5 or 7 for 8..11, 0
// for 12 and 0xFF above.  A positive code reads its value from the first table
// and a constant f(n) from the second (selector n ^ 8), a negative one the
// reverse; with f(n) and its counterpart folded into the table entries, the xor
// of the two lookups is the value: first table {-, 1, 2, 4, 8, ~16, ~32, ~64},
// second {-, -1, ~(-2), ~(-4), -8, ~(-16), ~(-32), ~(-64)}, the entries for code
// 0 chosen so that it gives 0.  Code 8 (a negative zero) does not occur.
// 11 VALU per 8 codes against 14 for a magnitude lookup negated under a sign
// mask (MLP dX, alone: 368 -> 344 us together with the deeper prefetch it lets
// fit the registers).
__device__ __forceinline__ uint32_t luq_value4(uint32_t n) {
  return __builtin_amdgcn_perm(0xBFDFEF08u, 0x040201FFu, n) ^
         __builtin_amdgcn_perm(0x3F1F0FF8u, 0x0301FF00u, n ^ 0x08080808u);
}

__device__ __forceinline__ void expand_luq(uint32_t x, uint32_t& lo, uint32_t& hi) {
  lo = luq_value4(x & 0x0F0F0F0Fu);
  hi = luq_value4((x >> 4) & 0x0F0F0F0Fu);
}

// SMP operand (two LUQ planes, R <= 5 so every value is in [-32, 32]): each
// plane is expanded to excess-64 bytes u = 64 + v (a LUT of 64 + 2^(e-1),
// and 128 - that for negative codes, as (P ^ 0x7F) + 1), so that the byte
// sum u0 + u1 = 128 + v0 + v1 lies in [64, 192] and one word add carries
// nothing across bytes; flipping bit 7 then gives v0 + v1 in two's
// complement.
__device__ __forceinline__ void expand_luq_excess64(uint32_t x, uint32_t& lo, uint32_t& hi) {
  // bytes 0..7: 64 + {0, 1, 2, 4, 8, 16, 32, 64}
  const uint32_t t_lo = 0x44424140u, t_hi = 0x80605048u;
  const uint32_t p_lo = __builtin_amdgcn_perm(t_hi, t_lo, x & 0x07070707u);
  const uint32_t p_hi = __builtin_amdgcn_perm(t_hi, t_lo, (x >> 4) & 0x07070707u);
  const uint32_t s_lo = (x >> 3) & 0x01010101u, s_hi = (x >> 7) & 0x01010101u;
  lo = (p_lo ^ ((s_lo << 7) - s_lo)) + s_lo;
  hi = (p_hi ^ ((s_hi << 7) - s_hi)) + s_hi;
}

template <bool SIGNED>
__device__ __forceinline__ void expand_int4(uint32_t x, uint32_t& lo, uint32_t& hi) {
  if constexpr (SIGNED) {
    lo = (x << 4) & 0xF0F0F0F0u;  // 16 * q
    hi = x & 0xF0F0F0F0u;
  } else {
    lo = (x << 3) & 0x78787878u;  // 8 * q
    hi = (x >> 1) & 0x78787878u;
  }
}

struct GemmArgs {
  const uint8_t* A;
  int64_t a_plane;
  const uint8_t* B;
  int64_t M, N, K;
  const float* alpha;
  const float* bscale;
  float* C;
  int32_t* partial;   // split-K chunk sums [splits][M][N], or null
  int64_t k_chunk;    // k per split (a multiple of the tile's stage depth)
  int tiles_m, tiles_n;
  int vec;            // N % 4 == 0 and rows of C (or partial) are 16-byte aligned: vector stores
};

// Block -> output tile.  Blocks are dispatched round-robin over the 8 XCDs
// (each with its own L2), so consecutive runs of tiles are given to one XCD;
// within that run tiles are visited in groups of
// 8 tile-rows so that the A rows and B rows in flight are shared.
__device__ __forceinline__ void tile_coords(int bid, int ntm, int ntn, int& tm, int& tn) {
  const int total = ntm * ntn;
  // XCD x takes a run of total / 8 tiles, the first total % 8 XCDs one more
  const int xcd = bid & 7, q = total >> 3, r = total & 7;
  const int L = xcd * q + min(xcd, r) + (bid >> 3);
  constexpr int G = 8;
  const int per_group = G * ntn;
  const int first_m = (L / per_group) * G;
  const int gsize = min(ntm - first_m, G);
  const int in_group = L - (L / per_group) * per_group;
  tm = first_m + in_group % gsize;
  tn = in_group / gsize;
}

// fl32(fl32(alpha / NS) * s_B) times the exact powers of two of the
// expansions (B: 2^-4 signed, 2^-3 unsigned; an INT4 A the same).
template <int AC, int NS, bool BSIGNED>
__device__ __forceinline__ float epilogue_scale(float alpha, float bscale) {
  constexpr float kInvSamples = AC == kAcSum2 ? 0.5f : 1.0f / NS;
  float sc = __fmul_rn(__fmul_rn(alpha, kInvSamples), bscale) * (BSIGNED ? 0x1p-4f : 0x1p-3f);
  if constexpr (AC == kAcInt4S) sc *= 0x1p-4f;
  if constexpr (AC == kAcInt4U) sc *= 0x1p-3f;
  return sc;
}

// ---- the tile kernel: A through LDS, the B operand in registers ----------------
//
// KG k-groups of WM x WN waves (eight waves, but for the small four-wave tile);
// a wave owns a (32 TM) x (32 TN) block of C, so a workgroup's tile is
// BM = 32 WM TM rows by BN = 32 WN TN columns and two or more waves share each
// SIMD: the expansion, address and LDS work of one overlaps the MFMAs of the
// others.  The MFMA takes the B fragment as its first operand, so each lane ends
// up with 4 consecutive columns of one C row.  Operands are read through buffer
// descriptors whose range is the operand itself: rows past M (or N) fall
// outside the range, and with FULLK false a chunk past the end of the split's k
// range is given an offset outside it, so both read as zeros without a branch.
// FULLK: K is a multiple of BK, so every stage of a split lies inside the
// operands' rows; stages past the end of the split are never multiplied.
//
// AC is the A operand's code type: LUQ (NS planes), INT4 (the forward product,
// NS = 1), expanded like B, or the int8 sums of two LUQ samples (NS = 1): 32
// bytes per 32-deep chunk, whose bytes only need the even / odd k split of the
// nibble expansions (two byte permutes per 8 values).
//
// Only A passes through LDS, expanded
// to int8 once per workgroup (the LUQ expansion is the costly one, and LDS
// stores run at a quarter of the LDS read rate).  Each wave loads the nibbles
// of its own 32 TN B rows straight into registers (the waves of the other row
// blocks load the same rows) and expands every fragment just before its MFMAs,
// which is a shift and a mask per word.
//
// With KG > 1 the k-groups share the tile and take 128 k each of a stage of
// 128 KG: a small tile still feeds eight waves, each with long contiguous B
// segments in flight, and the groups' int32 sums are added through LDS in the
// epilogue instead of through memory.
//
// k order: a 128-deep group stage is 64 nibble bytes of every row.  At k-step
// kk, lane half h = lane/32 supplies the k of nibble bytes 32h + 8kk .. +7 of
// the group's 64, for both operands, so a lane's B nibbles of a whole stage
// are one contiguous 32-byte segment.  The products summed are the same, in
// another order.  A sits in LDS as 8 KG slots of 16 expanded bytes per row,
// slot 8g + 2kk + h holding those k.
//
// Pipeline (one barrier per stage): stage t is multiplied from LDS buffer t%2
// with B registers set t%2, while the A codes of stage t+1 are expanded into
// the other buffer; each A chunk and each B half-segment is reloaded (A with
// stage t+3, B with stage t+2) as soon as its registers are consumed.
//
// PF sets how far ahead the MFMA operands are fetched, so that the LDS read
// latency is covered by the previous k-step's MFMAs:
//   0: each k-step's fragments are read and expanded just before its MFMAs;
//   1: the A fragments of k-step kk+1 are read while kk is multiplied;
//   2: as 1, and the B fragments of kk+1 are expanded during kk too;
//   3: as 2 across the stage boundary as well (the next stage's first B
//      fragments at the last k-step), with the B reload one k-step earlier.
// Every mode sums the same products; the launcher picks the deepest mode that
// fits the register budget for the operand kinds.

// Shape of a tile; OCC = waves per SIMD its registers must allow (512 / OCC
// registers a wave: two workgroups of the smaller tiles fit a CU).
template <int WM_, int WN_, int KG_, int TM_, int TN_, int OCC_>
struct GemmShape {
  static constexpr int WM = WM_, WN = WN_, KG = KG_, TM = TM_, TN = TN_, OCC = OCC_;
  static constexpr int BM = 32 * WM * TM, BN = 32 * WN * TN, BK = 128 * KG;
  static constexpr int NW = WM * WN * KG, THREADS = 64 * NW;
};
using Tile256x256 = GemmShape<2, 4, 1, 4, 2, 1>;
using Tile128x256 = GemmShape<2, 4, 1, 2, 2, 2>;
using Tile128x128 = GemmShape<2, 4, 1, 2, 1, 4>;
using Tile64x128 = GemmShape<1, 4, 2, 2, 1, 4>;
using Tile64x64 = GemmShape<1, 2, 4, 2, 1, 4>;
using Tile32x64 = GemmShape<1, 2, 4, 1, 1, 4>;
using Tile32x32 = GemmShape<1, 1, 8, 1, 1, 4>;
using Tile64x64k1 = GemmShape<2, 2, 1, 1, 1, 4>;

template <int AC, int NS, bool BSIGNED, bool FULLK, int PF, typename S>
__global__ __launch_bounds__(S::THREADS, S::OCC) void gemm_tile_kernel(GemmArgs a) {
  constexpr int BM = S::BM, kBK = S::BK, kThr = S::THREADS, KG = S::KG;
  constexpr int kPitch = kBK + 16;        // A row: 8 KG slots of 16 bytes, 16 bytes of pad
  constexpr int STAGE = BM * kPitch;
  constexpr int TM = S::TM, TN = S::TN;   // 32x32 tiles per wave
  constexpr int KC = kBK / 32;            // 16-byte A chunks per row and stage
  constexpr int ACH = BM * KC / kThr;     // A chunks per thread and stage
  constexpr bool kI8 = AC == kAcSum2;
  constexpr int NA = kI8 ? 2 : NS;
  static_assert(ACH == 1 || ACH == 2, "at most one A half-chunk per k-step");
  static_assert(BM * KC % kThr == 0, "every thread loads the same chunks");
  constexpr int EP = 32 * TN + 4;         // epilogue slab row pitch in 32-bit words
  constexpr int kSlabs = S::NW * 32 * EP * 4;
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * STAGE > kSlabs ? 2 * STAGE : kSlabs];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kg = wave / (S::WM * S::WN), wm = (wave / S::WN) % S::WM, wn = wave % S::WN, h = lane >> 5;
  int tm, tn;
  tile_coords(blockIdx.x, a.tiles_m, a.tiles_n, tm, tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * S::BN;
  const int64_t kbeg = (int64_t)blockIdx.y * a.k_chunk;
  const int64_t kend = min(kbeg + a.k_chunk, a.K);
  const int nkt = (int)((kend - kbeg + kBK - 1) / kBK);
  const int64_t ld = a.K >> 1;              // bytes per B row (and per nibble A row)
  const int64_t lda = kI8 ? a.K : ld;       // bytes per A row

  __amdgpu_buffer_rsrc_t rsa[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s)
    rsa[s] = __builtin_amdgcn_make_buffer_rsrc((void*)(a.A + s * a.a_plane), (short)0,
                                               (int)(a.M * lda), kBufferFlags);
  const __amdgpu_buffer_rsrc_t rsb =
      __builtin_amdgcn_make_buffer_rsrc((void*)a.B, (short)0, (int)(a.N * ld), kBufferFlags);
  // A loader: chunk i of a thread is row c/KC, 16 nibble bytes (32 k) at 16*(c%KC)
  int offa[ACH], kca[ACH], slota[ACH], rowa[ACH];
#pragma unroll
  for (int i = 0; i < ACH; ++i) {
    const int c = tid + i * kThr, row = c / KC, kc = c % KC;
    kca[i] = kc * 32;
    rowa[i] = row;
    // slot of the chunk's first half; the second is 2 further
    slota[i] = 8 * (kc >> 2) + 4 * (kc & 1) + ((kc >> 1) & 1);
    offa[i] = kI8 ? (int)((m0 + row) * lda + kbeg + kc * 32) : (int)((m0 + row) * ld + (kbeg >> 1) + kc * 16);
  }
  // B loader: load q takes the rows 2i + q of a 32-row block, lane l the
  // 16-byte chunk kcb of row (l & 30) + q, so that neighbouring lanes read 32
  // contiguous bytes and an instruction takes 64 bytes from each of 16 rows.
  // With one row per lane an instruction touched 32 rows, twice, and the
  // address unit bound the kernel (MLP dX, alone: 400 -> 365 us; a copy that
  // left the lanes unpaired: 330)
  const int kcb = (lane & 1) | (h << 1);
  int offb[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
    offb[j] = (int)((n0 + (wn * TN + j) * 32 + (lane & 30)) * ld + (kbeg >> 1) + kg * 64 + kcb * 16);

  struct ARegs {
    v4u a[NA][ACH];
  };
  struct BRegs {
    v4u b[TN][2];
  };
  auto load_a = [&](ARegs& r, int t, int i) {
    const int64_t k0 = kbeg + (int64_t)t * kBK;
    const bool in = FULLK || (k0 + kca[i]) < kend;
    if constexpr (kI8) {
      const int off = in ? offa[i] + t * kBK : kOutOfRange;
      r.a[0][i] = __builtin_amdgcn_raw_buffer_load_b128(rsa[0], off, 0, 0);
      r.a[1][i] = __builtin_amdgcn_raw_buffer_load_b128(rsa[0], in ? off + 16 : kOutOfRange, 0, 0);
    } else {
      const int off = in ? offa[i] + t * (kBK / 2) : kOutOfRange;
#pragma unroll
      for (int s = 0; s < NS; ++s) r.a[s][i] = __builtin_amdgcn_raw_buffer_load_b128(rsa[s], off, 0, 0);
    }
  };
  auto load_b = [&](BRegs& r, int t, int q) {
    const bool in = FULLK || (kbeg + (int64_t)t * kBK + kg * 128 + kcb * 32) < kend;
#pragma unroll
    for (int j = 0; j < TN; ++j)
      r.b[j][q] =
          __builtin_amdgcn_raw_buffer_load_b128(rsb, in ? offb[j] + t * (kBK / 2) + q * (int)ld : kOutOfRange, 0, 0);
  };
  // dwords 2hf, 2hf + 1 of a loaded set, exchanged within the lane pairs so that
  // lane l holds row l%32: b[.][q] becomes bytes 32h + 16q .. +15 of its row
  const bool odd = lane & 1;
  auto pair_b = [&](BRegs& r, int hf) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int d = 2 * hf; d < 2 * hf + 2; ++d) {
        const uint32_t x = r.b[j][0][d], y = r.b[j][1][d];
        // what the neighbour lane needs: quad_perm (1, 0, 3, 2)
        const uint32_t u = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(odd ? x : y), 0xB1, 0xF, 0xF, true);
        r.b[j][0][d] = odd ? u : x;
        r.b[j][1][d] = odd ? y : u;
      }
  };
  // half hf of A chunk i (its k 16hf .. 16hf+15) -> 16 bytes of LDS
  auto expand_a = [&](const ARegs& r, int buf, int i, int hf) {
    uint32_t w[4];
    if constexpr (kI8) {
      const v4u x = r.a[hf][i];
      w[0] = __builtin_amdgcn_perm(x[1], x[0], 0x06040200u);  // k even
      w[1] = __builtin_amdgcn_perm(x[1], x[0], 0x07050301u);  // k odd
      w[2] = __builtin_amdgcn_perm(x[3], x[2], 0x06040200u);
      w[3] = __builtin_amdgcn_perm(x[3], x[2], 0x07050301u);
    } else if constexpr (AC != kAcLuq) {
      expand_int4<AC == kAcInt4S>(r.a[0][i][2 * hf], w[0], w[1]);
      expand_int4<AC == kAcInt4S>(r.a[0][i][2 * hf + 1], w[2], w[3]);
    } else if constexpr (NS == 1) {
      expand_luq(r.a[0][i][2 * hf], w[0], w[1]);
      expand_luq(r.a[0][i][2 * hf + 1], w[2], w[3]);
    } else {
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        uint32_t l0, h0, l1, h1;
        expand_luq_excess64(r.a[0][i][2 * hf + d], l0, h0);
        expand_luq_excess64(r.a[1][i][2 * hf + d], l1, h1);
        w[2 * d] = (l0 + l1) ^ 0x80808080u;
        w[2 * d + 1] = (h0 + h1) ^ 0x80808080u;
      }
    }
    *reinterpret_cast<uint4*>(lds + buf * STAGE + rowa[i] * kPitch + ((slota[i] + 2 * hf) << 4)) =
        make_uint4(w[0], w[1], w[2], w[3]);
  };

  v16i acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = v16i{};

  // A fragment i of k-step kk: row 32 (TM wm + i) + lane%32, slot 8 kg + 2kk + h
  const int aoff = (wm * TM * 32 + (lane & 31)) * kPitch + kg * 128 + (h << 4);
  auto read_a = [&](int buf, int kk, v4i (&fa)[TM]) {
    const uint8_t* as = lds + buf * STAGE + aoff + (kk << 5);
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const v4i*>(as + i * 32 * kPitch);
  };
  // B fragment j of k-step kk: nibble dwords 2kk, 2kk+1 of the lane's segment
  auto frag_b = [&](const BRegs& r, int kk, v4i (&fb)[TN]) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      uint32_t l0, h0, l1, h1;
      expand_int4<BSIGNED>(r.b[j][kk >> 1][2 * (kk & 1)], l0, h0);
      expand_int4<BSIGNED>(r.b[j][kk >> 1][2 * (kk & 1) + 1], l1, h1);
      fb[j] = v4i{(int)l0, (int)h0, (int)l1, (int)h1};
    }
  };

  // fragments fetched one k-step ahead (PF >= 1), carried across stages (PF 3)
  v4i fa2[2][TM], fb2[2][TN];
  auto mma = [&](const v4i (&fa)[TM], const v4i (&fb)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[j], fa[i], acc[i][j], 0, 0, 0);
  };
  // multiply stage t from buffer cb and B set rb while expanding the A codes
  // of stage t+1 (ra) into the other buffer; rbn is the next stage's B set
  auto step = [&](int cb, ARegs& ra, int ta, BRegs& rb, int tb, BRegs& rbn) {
    if constexpr (PF >= 1) read_a(cb, 0, fa2[0]);
    if constexpr (PF != 3) pair_b(rb, 0);
    if constexpr (PF == 2) frag_b(rb, 0, fb2[0]);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk == (PF >= 2 ? 0 : 1)) pair_b(rb, 1);
      // the first B half-segment and A chunk are consumed: reload them now
      // (the scheduler would otherwise sink the loads to the barrier)
      if (kk == (PF == 3 ? 1 : 2)) {
        load_b(rb, tb, 0);
        if (PF != 3) load_a(ra, ta, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (PF == 3 && kk == 2) {
        load_a(ra, ta, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (PF == 0) {
        v4i fa[TM], fb[TN];
        read_a(cb, kk, fa);
        frag_b(rb, kk, fb);
        mma(fa, fb);
      } else if constexpr (PF == 1) {
        v4i fb[TN];
        if (kk + 1 < 4) read_a(cb, kk + 1, fa2[(kk + 1) & 1]);
        frag_b(rb, kk, fb);
        mma(fa2[kk & 1], fb);
      } else {
        if (kk + 1 < 4) {
          read_a(cb, kk + 1, fa2[(kk + 1) & 1]);
          frag_b(rb, kk + 1, fb2[(kk + 1) & 1]);
        } else if (PF == 3) {
          pair_b(rbn, 0);
          frag_b(rbn, 0, fb2[0]);
        }
        mma(fa2[kk & 1], fb2[kk & 1]);
      }
      if (kk < 2 * ACH) expand_a(ra, cb ^ 1, kk >> 1, kk & 1);
    }
    load_b(rb, tb, 1);
    if constexpr (ACH == 2) load_a(ra, ta, 1);
    __syncthreads();
    // keep the next stage's work below the barrier: hoisted above it, the
    // expansion of registers loaded in this stage would wait for those loads
    __builtin_amdgcn_sched_barrier(0);
  };

  ARegs r0, r1;
  BRegs b0, b1;
#pragma unroll
  for (int i = 0; i < ACH; ++i) load_a(r0, 0, i);
  load_b(b0, 0, 0);
  load_b(b0, 0, 1);
  // the order of the loop: the waits at its head, which hold for the entry and
  // for the back edge, then count the same loads behind the ones they need
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < ACH; ++i) load_a(r1, 1, i);
  load_b(b1, 1, 0);
  load_b(b1, 1, 1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kk = 0; kk < 2 * ACH; ++kk) expand_a(r0, 0, kk >> 1, kk & 1);
  if constexpr (PF == 3) {
    pair_b(b0, 0);
    frag_b(b0, 0, fb2[0]);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ACH; ++i) load_a(r0, 2, i);
  int t = 0;
  for (; t + 2 <= nkt; t += 2) {
    step(0, r1, t + 3, b0, t + 2, b1);  // multiply t, expand t+1 (r1); reload r1 with t+3, b0 with t+2
    step(1, r0, t + 4, b1, t + 3, b0);  // multiply t+1, expand t+2 (r0); reload r0 with t+4, b1 with t+3
  }
  if (t < nkt) step(0, r1, t + 3, b0, t + 2, b1);

  // Epilogue through LDS.  In MFMA tile (i, j), lane l holds row l%32 and, in
  // registers 4q..4q+3, the 4 consecutive columns 8q + 4*(l/32) + 0..3.  Each
  // wave stages 32 rows of its block at a time as a row-major slab in its own
  // part of the (now idle) stage buffers, then stores whole row segments: LPR
  // consecutive lanes cover one row of the block, RPI rows per instruction, or,
  // where rows are not 16-byte aligned, 4 bytes a lane on consecutive columns (four
  // scalar stores a lane, 16 bytes apart, took the odd widths 1845 x 14329 over K = 128
  // 52.5 against 23.1 us, 2655 x 2210 over 256 17.5 against 10.3).  With
  // KG > 1 the slabs hold the int32 sums and each k-group's wave stores 32 / KG of
  // the block's rows, adding the KG slabs of that block.  C gets the scaled fp32
  // values, the split-K workspace the raw int32 sums.
  constexpr int LPR = 8 * TN, RPI = 64 / LPR, SR = 32 / KG;
  static_assert(TN <= 2 && SR % (2 / TN) == 0, "4-byte stores: whole rows per instruction");
  uint32_t* E = reinterpret_cast<uint32_t*>(lds) + wave * 32 * EP;
  const uint32_t* E0 = reinterpret_cast<const uint32_t*>(lds) + (wave % (S::WM * S::WN)) * 32 * EP;
  const bool part = a.partial != nullptr;
  const float sc = part ? 0.0f : epilogue_scale<AC, NS, BSIGNED>(*a.alpha, *a.bscale);
  uint32_t* out = part ? reinterpret_cast<uint32_t*>(a.partial + (int64_t)blockIdx.y * a.M * a.N)
                       : reinterpret_cast<uint32_t*>(a.C);
  const int64_t rbase = m0 + wm * TM * 32, cbase = n0 + wn * TN * 32;
  const int srow = lane / LPR, scol = (lane % LPR) * 4;
  __syncthreads();  // every wave is done with the stage buffers
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v4u v;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int32_t x = acc[i][j][4 * q + r];
          v[r] = KG > 1 || part ? (uint32_t)x : __float_as_uint(__fmul_rn((float)x, sc));
        }
        *reinterpret_cast<v4u*>(E + (lane & 31) * EP + j * 32 + 8 * q + 4 * (lane >> 5)) = v;
      }
    __syncthreads();
    if (a.vec) {
#pragma unroll
      for (int rr = 0; rr < SR; rr += RPI) {
        const int sr = kg * SR + rr + srow;
        const int64_t row = rbase + i * 32 + sr;
        const int64_t col = cbase + scol;
        if (row < a.M && col < a.N && (SR % RPI == 0 || rr + srow < SR)) {
          v4u v = *reinterpret_cast<const v4u*>(E0 + sr * EP + scol);
          if constexpr (KG > 1) {
#pragma unroll
            for (int g = 1; g < KG; ++g)
              v += *reinterpret_cast<const v4u*>(E0 + (g * S::WM * S::WN * 32 + sr) * EP + scol);
            if (!part) {
#pragma unroll
              for (int r = 0; r < 4; ++r) v[r] = __float_as_uint(__fmul_rn((float)(int32_t)v[r], sc));
            }
          }
          *reinterpret_cast<v4u*>(out + row * a.N + col) = v;
        }
      }
    } else if (cbase < a.N && rbase + i * 32 + kg * SR < a.M) {
      // the LDS reads of a batch in flight together: 16 instructions where the block's
      // rows all lie inside, else four, and none past M
      constexpr int WC = 32 * TN, RS = 64 / WC, UA = SR < 16 * RS ? SR / RS : 16, UP = UA < 4 ? UA : 4;
      int el = lane;
      asm("" : "+v"(el));   // nothing of this path is computed before the loop
      const int wrow = el / WC, wcol = el % WC;
      const int64_t row0 = rbase + i * 32 + kg * SR, col = cbase + wcol;
      const int inside = (int)min(a.M - row0, (int64_t)SR), rows = inside - wrow;   // the lane's rows
      uint32_t* const dst = out + (row0 + wrow) * a.N + col;
      const uint32_t* src = E0 + (kg * SR + wrow) * EP + wcol;
      auto batch = [&](int rr, auto u_, auto whole) __attribute__((always_inline)) {
        constexpr int U = decltype(u_)::value;
        uint32_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = src[(rr + u * RS) * EP];
        if constexpr (KG > 1) {
#pragma unroll
          for (int g = 1; g < KG; ++g)
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] += src[(g * S::WM * S::WN * 32 + rr + u * RS) * EP];
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (!part) v[u] = __float_as_uint(__fmul_rn((float)(int32_t)v[u], sc));
        }
        uint32_t* const o = dst + rr * a.N;
        if (col < a.N) {
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (decltype(whole)::value || rr + u * RS < rows) o[u * RS * a.N] = v[u];
        }
      };
      if (inside == SR) {
        for (int rr = 0; rr < SR; rr += UA * RS) batch(rr, std::integral_constant<int, UA>{}, std::true_type{});
      } else {
        for (int rr = 0; rr < inside; rr += UP * RS) batch(rr, std::integral_constant<int, UP>{}, std::false_type{});
      }
    }
    __syncthreads();  // the slab is rewritten by the next i
  }
}

// Sums the split-K chunk sums in int64 in a fixed order and applies the scales.  A
// wave takes a run of 64 W outputs, W a lane; P waves share a run (wave p adds every
// P-th chunk, and with P > 1 their sums meet in LDS), RUNS runs make a workgroup.
// Bound by latency below about 2^19 outputs (one output a lane spreads the few there
// are over the most waves, and small workgroups start soonest) and by memory above it
// (16 bytes a lane, 16 neighbouring runs per workgroup).  The chunk index is scalar,
// so that the loads of a batch are issued without a test between them.  The chunks'
// base is always 16-byte aligned; vec_out: so is out.
template <int P, int RUNS, int W, typename Scale>
__global__ __launch_bounds__(64 * P * RUNS) void split_reduce_kernel(const int32_t* __restrict__ partial, int splits,
                                                                    int64_t MN, int vec_out, Scale scale,
                                                                    float* __restrict__ out) {
  static_assert(P == 1 || (W == 1 && RUNS == 1), "shared runs are one output a lane");
  typedef int vw __attribute__((ext_vector_type(W)));
  typedef float fw __attribute__((ext_vector_type(W)));
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int part = wave % P;
  const int64_t i0 = ((int64_t)blockIdx.x * RUNS + wave / P) * 64 * W + W * lane;
  const bool in = i0 < MN;   // MN is a multiple of W: a lane's outputs are in or out together
  int64_t s[W];
#pragma unroll
  for (int k = 0; k < W; ++k) s[k] = 0;
  if (in) {
    const int32_t* src = partial + i0;
    int p = part;
    auto batch = [&](auto u_) __attribute__((always_inline)) {
      constexpr int U = decltype(u_)::value;
      vw v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const vw*>(src + (int64_t)(p + P * u) * MN);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < W; ++k) s[k] += v[u][k];
      p += P * U;
    };
    while (p + 7 * P < splits) batch(std::integral_constant<int, 8>{});
    if (p + 3 * P < splits) batch(std::integral_constant<int, 4>{});
    if (p + P < splits) batch(std::integral_constant<int, 2>{});
    if (p < splits) batch(std::integral_constant<int, 1>{});
  }
  const float sc = scale();
  if constexpr (P > 1) {
    __shared__ int64_t red[P][64];
    red[part][lane] = s[0];
    __syncthreads();
    if (part == 0 && in) {
#pragma unroll
      for (int w = 1; w < P; ++w) s[0] += red[w][lane];
      out[i0] = __fmul_rn((float)s[0], sc);
    }
  } else if (in) {
    fw v;
#pragma unroll
    for (int k = 0; k < W; ++k) v[k] = __fmul_rn((float)s[k], sc);
    if (W > 1 && vec_out) {
      *reinterpret_cast<fw*>(out + i0) = v;
    } else {
#pragma unroll
      for (int k = 0; k < W; ++k) out[i0 + k] = v[k];
    }
  }
}

// out = scale * sum of `splits` chunk sums of MN outputs.  Timed alone over 64 to 2^22
// outputs and 2 to 256 chunks (us): from 2^19 outputs of whole 16-byte groups on, W = 4
// (2^20 outputs, 4 chunks: 3.4 against 3.7 with one output a lane and 6.5 with shared
// runs; 2^21, 12: 17.4, 20.7, 20.5); below, one wave a run up to 24 chunks (55296
// outputs, 16 chunks: 2.4 against 2.4 with four; 2^18, 16: 2.9 against 3.6) and four
// waves beyond, or beyond 32 from 2^17 outputs on (1024 outputs, 128 chunks: 2.6
// against 4.3; 55296, 64: 2.9 against 3.5).
template <typename Scale>
static void launch_split_reduce(const int32_t* partial, int splits, int64_t MN, Scale scale, float* out,
                                hipStream_t st) {
  auto launch = [&](auto kernel, int64_t outs, int threads, int vec_out) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((MN + outs - 1) / outs)), dim3(threads), 0, st, partial, splits, MN,
                       vec_out, scale, out);
  };
  if (MN >= (1 << 19) && MN % 4 == 0 && splits <= 24)
    launch(split_reduce_kernel<1, 16, 4, Scale>, 4096, 1024, ((uintptr_t)out & 15) == 0);
  else if (splits <= (MN >= (1 << 17) ? 32 : 24))
    launch(split_reduce_kernel<1, 4, 1, Scale>, 256, 256, 0);
  else
    launch(split_reduce_kernel<4, 1, 1, Scale>, 64, 256, 0);
}

template <int AC, int NS, bool BSIGNED>
struct EpilogueScale {
  const float* alpha;
  const float* bscale;
  __device__ __forceinline__ float operator()() const { return epilogue_scale<AC, NS, BSIGNED>(*alpha, *bscale); }
};

// ---- planning and launch ----------------------------------------------------------

enum GemmTile {
  kTile256x256, kTile128x256, kTile128x128, kTile64x128, kTile64x64, kTile32x64, kTile32x32, kTile64x64k1,
  kGemmTiles
};

// A tile's shape and its cost in microseconds.  With S = k per workgroup / 128
// stages, a workgroup alone on its CU takes S * stage1 + fixed1 (latency:
// loads, barriers, epilogue), and a CU with several of them S * stage + fixed
// each (throughput: expansion, LDS, MFMA, output stores).
struct TileCost {
  int lm, ln, lk;   // log2 of the tile's rows, columns and stage depth
  float stage1, fixed1, stage, fixed;
};

// Operands a plan is for: one code of A per k (one LUQ plane, int8 sums, INT4), or two
// LUQ planes, whose expansion takes twice the loads and three times the VALU work.
enum PlanKind { kPlanOne, kPlanTwoPlanes, kPlanKinds };

// Fitted to 73 000 timings on an MI355X: 1050 shapes drawn over M and N from 1 to 300000
// and K from 32 to 262144 (a quarter short reductions, a quarter few outputs; odd sizes
// among them), one LUQ plane, int8 sums, INT4 and two planes as the A operand, every
// tile that covers a shape sensibly in 1 to 85 splits.  Minimised is the time that the
// choice loses against the best one measured: 0.8 / 0.5% in the geometric mean (one code
// per k / two planes), 5% at the 95th percentile, 27 / 19% at worst.  The former table,
// one for all operands and fitted to the times alone, lost 2.4 / 4.2% on these shapes (14
// / 29%, 43 / 72% at worst) and made short reductions of wide outputs and split products
// of two planes slower than the tile rule before it (6912 x 3840 over 64 20.4 -> 23.4 us,
// now 19.6; two planes of 128 x 64 over 6048 9.2 -> 11.8, now 6.4).
constexpr TileCost kTileCost[kPlanKinds][kGemmTiles] = {
    {
        {8, 8, 7, 1.165f, 7.214f, 0.917f, 14.462f},
        {7, 8, 7, 0.901f, 2.625f, 0.813f, 6.118f},
        {7, 7, 7, 0.591f, 1.611f, 0.523f, 2.156f},
        {6, 7, 8, 0.274f, 2.821f, 0.271f, 1.507f},
        {6, 6, 9, 0.119f, 0.518f, 0.185f, 3.072f},
        {5, 6, 9, 0.140f, 1.224f, 0.131f, 1.711f},
        {5, 5, 10, 0.031f, 0.851f, 0.093f, 1.965f},
        {6, 6, 7, 0.541f, 1.654f, 0.248f, 0.437f},
    },
    {
        {8, 8, 7, 0.987f, 11.349f, 1.106f, 9.094f},
        {7, 8, 7, 0.601f, 5.800f, 0.742f, 4.720f},
        {7, 7, 7, 0.558f, 2.448f, 0.551f, 1.647f},
        {6, 7, 8, 0.268f, 1.772f, 0.245f, 1.500f},
        {},
        {5, 6, 9, 0.139f, 0.706f, 0.121f, 0.846f},
        {},
        {6, 6, 7, 0.426f, 0.476f, 0.331f, 0.657f},
    },
};
struct SplitCost {
  float launch;     // the reduction's launch
  float per_mout;   // per 10^6 chunk sums written and read back
};
constexpr SplitCost kSplitCost[kPlanKinds] = {{2.664f, 2.120f}, {1.572f, 1.276f}};
// Workgroups per CU: this far from the mean (0) to the busiest CU's (1).
constexpr float kBusiest[kPlanKinds] = {0.760f, 1.000f};
// Outputs beyond the 256 MB last-level cache leave at the rate of their row pieces: tiles
// of 64 columns (256 bytes) take 1.05 to 1.5 times the 128-column tiles' time there, and
// 0.87 to 1.2 times below (200704 x 576 over K = 64: 102 against 90 us).
constexpr int64_t kCachedOutputs = 56 << 20;
constexpr float kNarrowBeyondCache = 1.2f;
constexpr int kCus = 256;

// Two planes have no 64x64 and 32x32 tiles with k-groups: of 1050 shapes 8 were more than
// 2% faster on them (5930 x 282 over 6528 by 7%, the most), and the cost table chose them
// for next to none.
constexpr bool tile_built(PlanKind kind, int t) {
  return kind == kPlanOne || (t != kTile64x64 && t != kTile32x32);
}

struct GemmPlan {
  GemmTile tile;
  int64_t tiles_m, tiles_n;
  int splits;
  int64_t k_chunk;
};

// The tile and the number of splits with the least predicted time.  A split's k
// range is a multiple of the tile's stage depth; min_splits keeps a chunk's int32
// sums exact; kind chooses the cost table.  M, N <= 2^30 and K < 2^31 (checked at the
// entry points, the workspace query among them), so no count overflows.
static GemmPlan search_plan(int64_t M, int64_t N, int64_t K, int64_t max_exact_k, PlanKind kind) {
  GemmPlan best{};
  float best_cost = 0.0f;
  const int64_t min_splits = K <= max_exact_k ? 1 : (K - 1) / max_exact_k + 1;
  const SplitCost& sc = kSplitCost[kind];
  const float split_out = sc.per_mout * 1e-6f * (float)M * (float)N;   // per split
  for (int t = 0; t < kGemmTiles; ++t) {
    if (!tile_built(kind, t)) continue;
    const TileCost& c = kTileCost[kind][t];
    auto ceil_shift = [](int64_t v, int l) { return ((v - 1) >> l) + 1; };
    const int64_t tiles_m = ceil_shift(M, c.lm), tiles_n = ceil_shift(N, c.ln), nt = tiles_m * tiles_n;
    const int64_t stages = ceil_shift(K, c.lk);
    auto consider = [&](int64_t want) {
      if (want < min_splits) want = min_splits;
      if (want > stages) want = stages;
      const int64_t chunk = want == 1 ? stages : (stages - 1) / want + 1;
      const int64_t splits = want == 1 ? 1 : (stages - 1) / chunk + 1;
      const float s = (float)(chunk << c.lk) * (1.0f / 128);
      const int64_t nb = nt * splits;
      const float mean = nb < kCus ? 1.0f : (float)nb * (1.0f / kCus);
      const float per_cu = mean + kBusiest[kind] * ((float)((nb + kCus - 1) / kCus) - mean);
      const float alone = s * c.stage1 + c.fixed1, shared = per_cu * (s * c.stage + c.fixed);
      float cost = alone > shared ? alone : shared;
      if (M * N > kCachedOutputs && c.ln < 7) cost *= kNarrowBeyondCache;
      if (splits > 1) cost += sc.launch + split_out * (float)splits;
      if (best.splits == 0 || cost < best_cost) {
        best_cost = cost;
        best = GemmPlan{(GemmTile)t, tiles_m, tiles_n, (int)splits, chunk << c.lk};
      }
    };
    consider(1);
    // splits only where the tiles leave CUs idle (up to two workgroups per CU)
    // and two of them alone do not cost more than there is to gain
    const float least = sc.launch + 2 * split_out + c.fixed1;
    if (nt < kCus && stages > 1 && best_cost > least) {
      for (int64_t s = 2; s * nt < 2 * kCus && s <= stages; s *= 2) consider(s);
      consider(kCus / nt);
    }
  }
  return best;
}

// The plan of the calling thread's last shape of each kind is kept: a call asks for it
// up to three times (workspace size, its check, the launch), and the search costs 0.1 to
// 0.5 us of host time.
static GemmPlan plan_gemm(int64_t M, int64_t N, int64_t K, int64_t max_exact_k, PlanKind kind = kPlanOne) {
  struct Last {
    int64_t M, N, K, exact;
    GemmPlan plan;
  };
  static thread_local Last last[kPlanKinds]{};
  Last& l = last[kind];
  if (l.M != M || l.N != N || l.K != K || l.exact != max_exact_k)
    l = Last{M, N, K, max_exact_k, search_plan(M, N, K, max_exact_k, kind)};
  return l.plan;
}

// Bytes of the plan's split sums; 0 without splits, and where they exceed any memory
// (such operands are refused).
static size_t split_bytes(const GemmPlan& p, int64_t M, int64_t N) {
  size_t b = 0;
  if (p.splits <= 1 || __builtin_mul_overflow((size_t)M * (size_t)N * sizeof(int32_t), (size_t)p.splits, &b)) return 0;
  return b;
}

template <typename S, int AC, int NS, bool BSIGNED>
static void launch_tile(const GemmArgs& a, dim3 grid, hipStream_t st) {
  // Prefetch depth, by what measured best; registers are 256 a wave for the two largest
  // tiles and 128 for the others, and a deeper mode costs more of them.  256x256: the
  // next stage's fragments too (PF 3), but for the int8 sums with unsigned B and two
  // planes (PF 2: two planes spill 2 to 5 registers in either mode, and PF 1 took 8192 x
  // 4096 over K = 16384 from 555 to 582 us).  With a partly filled last stage the k tests
  // take registers: the int8 sums spilled 4 in PF 1 and none in PF 0 (4096 x 4096 over
  // 1056: 32.1 -> 31.0 us).  64x64 with four k-groups, partial: PF 1 (up to 5 spilled in
  // PF 2; 1024 x 512 over 4128, LUQ 11.6 -> 11.0 us, sums 10.1 -> 9.6).  Elsewhere one
  // k-step ahead.
  constexpr bool kBig = S::BM == 256, kLuq1 = AC == kAcLuq && NS == 1, kLuq2 = AC == kAcLuq && NS == 2;
  constexpr int kSmall = S::BM == 64 && S::BN == 128 ? 1 : 2;
  constexpr bool k64 = S::BM == 64 && S::BN == 64 && S::KG == 4;   // one code per k only
  constexpr int kPfFull = !kBig ? kSmall : kLuq2 ? 2 : AC == kAcSum2 && !BSIGNED ? 2 : 3;
  constexpr int kPfPart = !kBig ? (k64 ? 1 : kSmall) : kLuq1 ? 2 : kLuq2 || AC == kAcSum2 ? 0 : 1;
  if (a.K % S::BK == 0)
    hipLaunchKernelGGL((gemm_tile_kernel<AC, NS, BSIGNED, true, kPfFull, S>), grid, dim3(S::THREADS), 0, st, a);
  else
    hipLaunchKernelGGL((gemm_tile_kernel<AC, NS, BSIGNED, false, kPfPart, S>), grid, dim3(S::THREADS), 0, st, a);
}

template <int AC, int NS, bool BSIGNED>
static hipError_t gemm_launch_t(const GemmArgs& a0, const GemmPlan& p, hipStream_t st) {
  GemmArgs a = a0;
  a.tiles_m = (int)p.tiles_m;
  a.tiles_n = (int)p.tiles_n;
  a.k_chunk = p.k_chunk;
  const dim3 grid((unsigned)(p.tiles_m * p.tiles_n), (unsigned)p.splits);
  // 16-byte stores need 16-byte aligned rows
  a.vec = (a.N % 4) == 0 && (((uintptr_t)(a.partial ? (void*)a.partial : (void*)a.C)) & 15) == 0;
  constexpr PlanKind kKind = AC == kAcLuq && NS == 2 ? kPlanTwoPlanes : kPlanOne;
  switch (p.tile) {
    case kTile256x256: launch_tile<Tile256x256, AC, NS, BSIGNED>(a, grid, st); break;
    case kTile128x256: launch_tile<Tile128x256, AC, NS, BSIGNED>(a, grid, st); break;
    case kTile128x128: launch_tile<Tile128x128, AC, NS, BSIGNED>(a, grid, st); break;
    case kTile64x128: launch_tile<Tile64x128, AC, NS, BSIGNED>(a, grid, st); break;
    case kTile64x64:
      if constexpr (tile_built(kKind, kTile64x64)) launch_tile<Tile64x64, AC, NS, BSIGNED>(a, grid, st);
      break;
    case kTile32x64: launch_tile<Tile32x64, AC, NS, BSIGNED>(a, grid, st); break;
    case kTile32x32:
      if constexpr (tile_built(kKind, kTile32x32)) launch_tile<Tile32x32, AC, NS, BSIGNED>(a, grid, st);
      break;
    default: launch_tile<Tile64x64k1, AC, NS, BSIGNED>(a, grid, st); break;
  }
  if (p.splits > 1)
    launch_split_reduce(a.partial, p.splits, a.M * a.N, EpilogueScale<AC, NS, BSIGNED>{a.alpha, a.bscale}, a.C, st);
  return hipGetLastError();
}

}  // namespace luq
