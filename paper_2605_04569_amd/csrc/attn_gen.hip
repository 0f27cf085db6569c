// General matrix-core attention kernel: every dtype, head dimension and block size that the pipelined bf16 D = 128,
// block = 128 kernels do not cover (and those too when they are switched off): exact online-softmax attention (Alg. 2
// Part A), block-wise 0-th order Taylor attention with and without exact sets (Sec. 3, Eq. 3-4; Alg. 2 Parts A+B), dense.
//
// Precision: every number that a plain fp32 evaluation holds in fp32 is held in 24 bits here, down to about 2^-110.
//   fp32 tensors: queries, keys, values, means and weights are cut into three bf16 terms of 8 bits each whose sum is the number, and a
//     product is the sum of six products of terms (v_mfma_f32_16x16x32_bf16).  Left out are middle x low and low x low: the terms are rounded
//     to nearest, so these are at most 2^-24 of the product of the leading bits, of either sign (with terms cut off up to 2^-21, always towards
//     zero).  An item with a number whose terms have lost bits (below about 2^-110) is run again with v_mfma_f32_16x16x4_f32 where these can show:
//     any such query, such keys beside queries of 2^96, such values in results below 2^-108.  A weight that small,
//     against the row's largest, loses less than 2^-133 of that one, unchecked: a part of the result only where the heavier keys' values are 0.
//     Error against 64 bits of dense attention on fp32 matrix instructions / in terms, 2-norm: 2000 random tokens, D = 128, 9.2e-7 / 5.6e-7, D = 64
//     6.6e-7 / 4.8e-7; one massive channel beside random ones 1.1e-5 / 6.0e-6; scores of a single channel's product 1.46e-6 / 1.44e-6 (with
//     terms cut off 2.7e-6), 300 tokens 1.25e-6 / 1.30e-6 (an instruction adds 32 products where one on fp32 adds 4).
//   bf16 tensors: scores of tokens with v_mfma_f32_16x16x32_bf16 (products of bf16 numbers are exact in fp32); the softmax
//     weights and the fp32 block means are cut into three bf16 terms whose sum is the fp32 number (8 bits each), and
//     the product is the sum of the terms' products: 3 matrix instructions for weights x tokens, 3 for queries x means, 8
//     for weights x means (the term low x low, below 2^-30 of the product, is left out; a mean below 2^-110 loses less than 2^-133, unchecked).
//
// Shape.  A workgroup of 4 waves owns 64 QT query rows, QT 16-query tiles per wave (QT = 1 when a launch has so few rows
// that 128 a workgroup would leave compute units idle).  With r = lane % 16, g = lane / 16 the scores are computed
// transposed (S^T = K Q^T): lane (r, g) holds keys 16 kt + 4 g + i of query 16 qt + r, which is the operand layout of the
// second product (O^T = V^T P^T), so the weights never leave their registers; V is read transposed out of its row-major
// tile (ds_read_b64_tr_b16; on fp32 matrix instructions a lane's four channels of a row serve four output tiles).  Tiles of 64
// bf16 (32 fp32) rows go global -> LDS directly, one tile ahead, two stages, 16-byte chunks XOR-swizzled by row.  A stage
// is 256 D bytes either way.  An fp32 tile is taken apart once per workgroup, from its one raw place into the place of the terms, which
// keys and values share (a wave takes apart what it has fetched itself); the raw place is filled again at once.  A launch with few long items cuts their key lists into parts, a workgroup each, and a second kernel adds
// them up, or gives a workgroup two groups of 4 waves that take the tiles in turn (NG = 2).  Groups that share a compute unit, whose softmax
// runs beside each other's matrix instructions (there is no hand-made interleaving here): D = 128, 66 KB each, two; D = 64, 33 KB, three of
// QT = 2 (registers) or four of QT = 1.
//
// What bounds it (measured, 24 heads of 64 channels, 15 600 tokens in blocks of 64, keep 0.5, full 0.25): the vector issue port, which a matrix
// instruction holds too. The exact cut of a weight into three terms takes 1.5 vector instructions and half a matrix instruction: the
// differences are taken by matrix instructions (with 5.5 vector instructions 2 % slower; the bf16 dot instruction is slower still
// and not exact).  A full tile is fetched from scalar addresses, its keys are weighed 64 at a time, and a loop has tiles of one kind only, so
// that the accumulators stay where they are: 131 -> 80 vector instructions per 16 matrix ones, and 40 to 60 registers less.  Counters of that
// launch: vector instructions issuing in 94 -> 70 % of the cycles, matrix pipe busy 42 -> 62 %, no LDS bank conflicts.  Whole call 740 -> 651 us;
// 128 channels 1271 -> 1133, dense attention of 8 such heads 1153 -> 977.  A kernel of one row per four lanes in scalar arithmetic took 11.6 ms.
//
// fp32: six bf16 products in place of eight fp32 ones that take twice as long each: 24 heads of 128 channels, 15 600 tokens, 5.6 -> 3.2 ms a call (1.1
// PFLOP/s of bf16 products), 64 channels in blocks of 64 2.96 -> 1.56 ms; 8 heads of 5280 tokens 301 -> 194 us.  Counters of the first / the last: matrix
// pipe busy 54 / 49 % of the cycles, vector and matrix instructions at their port in 45 / 45 %; of the waves' cycles 40 / 39 % wait for a place there and
// 22 / 25 % for data or at the four barriers of a tile.  With 16 rows a wave the LDS reads take as long as the products, with 32 half of that.
#include <math.h>

#include <type_traits>

#include "attn_mfma.h"

namespace isa {

#define ISA_GEN_FENCE() __builtin_amdgcn_sched_barrier(0)
// a barrier of the workgroup that leaves global loads in flight
#define ISA_GEN_BARRIER() asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory")

namespace {

constexpr float FAST_MAX = 16777216.f;    // 2^24, log2 domain: a maximum below is rounded by half at most

template <int D> constexpr int ITEM_LDS = 512 * D + 2 * 64 * 4;          // two stages of a K and a V tile, weights of mean tiles
template <int D, int QT> constexpr int RESIDENT = D == 128 ? 2 : QT == 1 ? 4 : 3;     // workgroups of a compute unit: LDS, registers (D = 64, QT = 2)
constexpr int MAX_PARTS = 8;

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v* lds_s4_ptr;

// Eight small numbers, one per batch item, in a word (what a launch hands over is copied for every call)
static_assert(ISA_MAX_BATCH <= 8, "four bits a batch item");
__host__ __device__ __forceinline__ int nibble(uint32_t x, int b) { return (x >> (4 * b)) & 15; }

// Work items of `rows` rows of n blocks: two blocks of 64 rows make one of 128, a block of 128 two of 64.
__host__ __device__ __forceinline__ int slots_of(int block, int n, int rows) { return block > rows ? 2 * n : block == rows ? n : (n + 1) / 2; }

struct GenArgs {
  AttnArgs a;
  int slots_long, slots_taylor;     // work items per (batch, head) of the exact branch / of the Taylor branch (batch items alike)
  int per_xcd_long, per_xcd_taylor; // and per XCD, over all (batch, head)s
  // Batch items that differ: an XCD has an equal range of every one's own items, longest key lists first (by_length), as in the heads' order of
  // all of them, with the most items of any, an XCD could get nothing but short ones.  With parts by each one's own list (both, whole
  // calls; before: as many parts as the shortest list can have, or none): bf16, D = 128, blocks of 64, 8 heads of 6000 and 1500 tokens
  // 298 / 144 us, of 5000 and 100 253 / 113, D = 64, 2 heads of 15 600 and 64 297 / 114.
  int ragged; uint32_t by_length, long_items[ISA_MAX_BATCH], taylor_items[ISA_MAX_BATCH];       // items in that order, at most 65535 x 8192
  // A long item of batch item b runs as own_parts(b) workgroups (at most `parts`), each over its share of the listed blocks; if that is more
  // than one, they leave [first_part[b] + item of b * own_parts(b) + part][row][D] their normalised results and {maximum, sum} of the row
  int parts; uint32_t own_parts;
  int first_part[ISA_MAX_BATCH];
  float* part_o; float2* part_ml;
};

__device__ __forceinline__ void dma16(const void* src, uint32_t lds_addr) {      // lane i -> LDS bytes lds_addr + 16 i
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds_addr), "v"(src) : "memory", "m0");
}
__device__ __forceinline__ void dma16(const void* base, uint32_t offset, uint32_t lds_addr) {      // the same from a common base
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds_addr), "v"(offset), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(size_t)(__attribute__((address_space(3))) const void*)p;
}
__device__ __forceinline__ f32x4 mfma_bf(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float bits_f(uint32_t u) { return __uint_as_float(u); }

// Eight fp32 numbers as three bf16 fragments that add up to them: a term is the leading 8 bits of what the terms before it left over, so that the
// differences are exact and the third term ends at bit 24.  ROUND: the first two terms are rounded to nearest instead of cut off: then the middle is at
// most 2^-8 and the low 2^-17 of the leading bit, and of either sign (cut off: 2^-7 and 2^-15, of the number's sign), which is what products
// need that leave out the smallest ones.  Returns a word whose low half is 0 unless a number is so small that its third term has lost bits.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
template <bool ROUND> __device__ __forceinline__ uint32_t lead8(float a, float b) {        // a below, b above
  if constexpr (ROUND) {
    const bf16x2 r = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, r);
  } else {
    return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
  }
}
template <bool ROUND> __device__ __forceinline__ uint32_t split3(const float (&x)[8], bf16x8 (&t)[3]) {
#pragma clang fp contract(off)                         // of the numbers as they are, not of a product they come from
  uint32_t w[3][4], rest = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float a = x[2 * e], b = x[2 * e + 1];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      w[k][e] = lead8<ROUND>(a, b);
      a -= bits_f(ROUND ? w[k][e] << 16 : __float_as_uint(a) & 0xffff0000u);
      b -= bits_f((ROUND ? w[k][e] : __float_as_uint(b)) & 0xffff0000u);
    }
    w[2][e] = lead8<false>(a, b);
    rest |= __float_as_uint(a) | __float_as_uint(b);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) t[k] = __builtin_bit_cast(bf16x8, make_uint4(w[k][0], w[k][1], w[k][2], w[k][3]));
  return rest;
}
// The same of a lane's numbers x[0 .. 3], x[4 .. 7] with the differences taken by matrix instructions: x - term = x + A term, A[4 g + i][8 g + 4 u + i]
// = -1 (u = 0: the first four numbers, u = 1: the others), which is exact like the subtraction.  Two of them take 16 cycles of the vector
// issue port, 16 vector instructions 64.
__device__ __forceinline__ bf16x8 minus_ones(int u, int r16, int g) {
  const uint32_t one = g == (r16 >> 2) ? 0xbf80u << (16 * (r16 & 1)) : 0u;
  const uint32_t lo = r16 & 2 ? 0u : one, hi = r16 & 2 ? one : 0u;
  return __builtin_bit_cast(bf16x8, u ? make_uint4(0u, 0u, lo, hi) : make_uint4(lo, hi, 0u, 0u));
}
template <bool ROUND> __device__ __forceinline__ void split3(f32x4 x0, f32x4 x1, const bf16x8 (&minus)[2], bf16x8 (&t)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a = (e < 2 ? x0 : x1)[2 * (e & 1)], b = (e < 2 ? x0 : x1)[2 * (e & 1) + 1];
      w[e] = k < 2 ? lead8<ROUND>(a, b) : lead8<false>(a, b);
    }
    t[k] = __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
    if (k < 2) {
      x0 = mfma_bf(minus[0], t[k], x0);
      x1 = mfma_bf(minus[1], t[k], x1);
    }
  }
}

}  // namespace

// One work item: 64 QT rows of one query block (QT = 2, block 64: of two neighbours in the list).  FULL32 is the second pass over an item:
// it evaluates the products of fp32 numbers with fp32 matrix instructions instead of bf16 terms, slower, but infinities go
// through them as through a multiplication (a term that is zero turns an infinity into NaN).  Returns whether this wave's results are
// all finite, its maxima in the range of the fast weights and no bits lost that can show; with FULL32 = false nothing is stored if some wave's are not, and the
// caller runs the item again.
//
// A weight is exp2 of the scaled score minus the scaled running maximum.  The fast form of bf16 tensors is one fma, whose
// product is not rounded while the maximum is: all weights of a row share a factor of 2^r with |r| up to half a unit in the
// last place of the maximum, which cancels in the result as long as it is a small number.  From FAST_MAX on the row is left to the
// second pass; it and fp32 tensors (WIDE) subtract the maximum of the scores as they are, so that the largest key's exponent is 0
// whatever they are, and start it at -infinity, M_INIT being a score that a row may lie below.  fp32 scores come scaled (the queries
// are multiplied by the scale when they are loaded), the second pass over bf16 rows multiplies the difference.
//
// The first pass raises a maximum only when a weight would exceed 2^tau, the second at every larger score: its weights are at most 1, where
// 2^tau times a value near the largest number is none.  (A factor of 2^-tau in the first pass's weights cost values near the
// smallest normal number their last eight bits.)
//
// NG = 2: two groups of 4 waves work on the same rows, each with stages of its own, and take the tiles of the sequence in turn;
// the second group hands its running maxima, sums and outputs to the first through LDS at the end.
// PARTS: part >= 0 is the item's part of that number, first_part the place of its first one's results (a template, as whole items have no register to spare for it).  QI: the item's query tiles per wave (the second pass takes its rows 64 at a time).
template <typename T, int D, int QT, bool FULL32, int QI, bool PARTS, int NG>
__device__ __forceinline__ bool attn_gen_item(const GenArgs& ga, unsigned char* const lds_all, int bhid, bool taylor, int slot, const int part, const int first_part) {
  constexpr bool BF = sizeof(T) == 2, WIDE = !BF || FULL32;
  constexpr bool FM = !BF && FULL32, TERMS = !BF && !FULL32;           // fp32 tensors: on fp32 matrix instructions / in bf16 terms
  constexpr int KTOK = BF ? 64 : 32;                   // tokens per tile; tiles of means hold 32
  constexpr int NT = D / 16;                           // 16-channel tiles
  constexpr int TILE = 128 * D;                        // bytes of a K (or V) tile, token or mean
  constexpr int CT = D * (int)sizeof(T) / 16, CM = D / 4;      // 16-byte chunks per row of token / mean tiles
  constexpr int ST = (CT < 16 ? CT : 16) - 1, SM = 15; // swizzle: chunk c of row r sits at c ^ (r & S)
  constexpr int CP = D / 8, SP = CP - 1, PLANE = 64 * D;       // 16-byte chunks per row, swizzle and bytes of a tile's terms of one kind
  constexpr int NI = D / 32;                           // 1 KB loads per wave, tile and tensor
  constexpr int ROWS = 64 * QT;
  const int grp = NG > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8) : 0;
  unsigned char* const lds = lds_all + grp * ITEM_LDS<D>;
  const AttnArgs& a = ga.a;
  float* const wts = reinterpret_cast<float*>(lds + 4 * TILE);         // [stage][block of the item][32]: weights of a mean tile's slots

  const int b = bhid / a.geo.H, h = bhid % a.geo.H;
  const BatchCounts c = a.cnt.b[b];
  const int T_max = a.geo.T_max, block = a.geo.block;
  const long long bh = bhid;
  const int* const kvl = a.dense ? nullptr : a.kv_list + bh * T_max;
  const int n_list_kv = a.dense ? c.T : c.T_new;
  const int kv_lo = !PARTS || part < 0 ? 0 : part * n_list_kv / nibble(ga.own_parts, b);
  const int n_kv = !PARTS || part < 0 ? n_list_kv : (part + 1) * n_list_kv / nibble(ga.own_parts, b);
  const int* const bs = a.blk_start + b * T_max;
  const int* const bn = a.blk_n + b * T_max;
  const long long tbase = (long long)b * a.geo.stride_b + (long long)h * a.geo.stride_h;

  const int tid = NG > 1 ? threadIdx.x & 255 : threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;

  // this wave's query block and rows
  const bool pair = QT == 2 && block == 64;
  const int subs = pair ? 1 : block / ROWS;
  const int n_list = a.dense ? c.T : taylor ? c.n_flat : c.n_full;
  const int entry0 = pair ? 2 * slot : slot / subs;
  const int own = pair ? wave >> 1 : 0;                // which of the item's blocks
  const int entry = entry0 + own;
  const bool active = entry < n_list;
  const int e_use = active ? entry : entry0;
  const int qi = a.dense ? e_use : block_in_range((taylor ? a.flat_list : a.full_list)[bh * T_max + e_use], c.T);
  const int n_q = active ? bn[qi] : 0, q_start = bs[qi];
  const int row0 = pair ? (wave & 1) * 32 : (slot % subs) * ROWS + wave * 16 * QT;
  const bool sets = taylor && a.exact_mask && c.k_exact > 0;
  const uint32_t* const mrow = sets ? a.exact_mask + (bh * T_max + entry0) * a.cnt.mask_words : nullptr;
  const int n_sets = pair && entry0 + 1 < n_list ? 2 : 1;              // bit rows of the item
  auto set_bits = [&](int t) -> int {                  // bit u: kv_list[t] is in the exact set of the item's block u
    int bits = (mrow[t >> 5] >> (t & 31)) & 1;
    if (n_sets == 2) bits |= ((mrow[a.cnt.mask_words + (t >> 5)] >> (t & 31)) & 1) << 1;
    return bits;
  };

  const float cscale = 1.4426950408889634f / sqrtf((float)D);
  // Q fragments: bf16 lane (r, g) holds channels 32 ks + 8 g .. + 7 of query 16 qt + r, fp32 (scaled) channels 16 t + 4 g .. + 3 or, in terms, as bf16
  bf16x8 qb[QT][D / 32];
  f32x4 qf[QT][NT];
  bf16x8 q3[QT][D / 32][3];                            // TERMS: of the scaled queries, channels as in qb
  uint32_t q_lost = 0, lost = 0;                       // TERMS: bits that terms have lost: of queries; of keys (low half) and values (high half)
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    const int row = row0 + 16 * qt + r16;
    const T* qp = (const T*)a.q + tbase + (long long)(q_start + (row < n_q ? row : 0)) * a.geo.stride_t;
    if constexpr (BF) {
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) qb[qt][ks] = *reinterpret_cast<const bf16x8*>(qp + 32 * ks + 8 * g);
    } else if constexpr (TERMS) {
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const f32x4 y = *reinterpret_cast<const f32x4*>(qp + 32 * ks + 8 * g + 4 * u) * cscale;
#pragma unroll
          for (int i = 0; i < 4; ++i) x[4 * u + i] = y[i];
        }
        q_lost |= split3<true>(x, q3[qt][ks]);
      }
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t) qf[qt][t] = *reinterpret_cast<const f32x4*>(qp + 16 * t + 4 * g) * cscale;
    }
  }

  // ---- the sequence of tiles: the tokens of the listed blocks (Taylor: of the blocks of the exact sets), then, for
  // Taylor blocks, the means of the list.  The lanes hold the table rows of 64 list entries at a time.
  int c_start = 0, c_n = 0, c_bits = 0, cbase = kv_lo - 64;
  unsigned long long todo = 0ull;
  struct Tile { int start, nk, bits; bool mean, end; };
  Tile at = {0, 0, 3, false, false};                   // the tile that was described last
  int left = 0;                                        // tokens of its block that come after it
  auto next_tile = [&]() {
    if (!at.mean) {
      if (left > 0) {
        at.start += KTOK;
        at.nk = min(KTOK, left);
        left -= KTOK;
        return;
      }
      while (todo == 0ull && (!taylor || sets) && cbase + 64 < n_kv) {
        cbase += 64;
        const int t = cbase + lane;
        const int j = t < n_kv ? (kvl ? block_in_range(kvl[t], c.T) : t) : 0;
        c_bits = t < n_kv ? (taylor ? set_bits(t) : 3) : 0;
        c_start = bs[j];
        c_n = bn[j];
        todo = __ballot(c_bits != 0);
      }
      if (todo != 0ull) {
        const int l = __builtin_ctzll(todo);
        todo &= todo - 1;
        at.start = __builtin_amdgcn_readlane(c_start, l);
        at.bits = __builtin_amdgcn_readlane(c_bits, l);
        const int n = __builtin_amdgcn_readlane(c_n, l);
        at.nk = min(KTOK, n);
        left = n - KTOK;
        return;
      }
      at.start = -32;
      at.mean = taylor;
      at.end = !taylor;
    }
    at.start += 32;                                    // mean tiles: position in kv_list
    at.nk = min(32, n_kv - at.start);
    at.bits = 3;
    if (at.nk <= 0) at.end = true;
  };
  // Loads of a token tile: load i of a wave fetches RPL rows from (4 i + wave) RPL on.  A full tile's rows are at one offset per lane from
  // scalar addresses: no vector instructions per load
  constexpr int RPL = TERMS ? 64 / CP : 64 / CT, NL = TERMS ? D / 64 : NI;
  const uint32_t lane_off = (uint32_t)((lane / (64 / RPL)) * (int)a.geo.stride_t + (TERMS ? lane % CP * 8 : ((lane % CT) ^ ((wave * RPL + lane / CT) & ST)) * (16 / (int)sizeof(T)))) * (uint32_t)sizeof(T);
  auto is_full = [&](const Tile& t) { return t.nk == KTOK && a.geo.stride_t < (1 << 22); };
  // TERMS: one tensor (v or k) of tile t to its place.  16-byte piece u of eight-channel chunk p at (u * 4 D + p) * 16: a lane takes
  // the same chunks apart again that it has fetched
  auto issue_terms = [&](const Tile& t, const auto mean_c, const bool value) {
    constexpr bool mean = decltype(mean_c)::value;
    const uint32_t dst = lds_addr(lds) + (value ? TILE : 0) + wave * 1024;
    if (!mean && is_full(t)) {
      const float* src = (const float*)(value ? a.v : a.k) + tbase + ((long long)t.start + wave * RPL) * a.geo.stride_t;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        dma16(src, lane_off, dst + i * 4096);
        dma16(src + 4, lane_off, dst + i * 4096 + TILE / 2);
        src += 4 * RPL * a.geo.stride_t;
      }
      return;
    }
    int li = lane;
    asm volatile("" : "+v"(li));
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int row = min((4 * i + wave) * RPL + li / CP, t.nk - 1), ch = li % CP * 8;
      const float* src;
      if constexpr (!mean) src = (const float*)(value ? a.v : a.k) + tbase + (long long)(t.start + row) * a.geo.stride_t + ch;
      else src = (value ? a.vc : a.kc) + (bh * T_max + block_in_range(kvl[t.start + row], c.T)) * D + ch;
      dma16(src, dst + i * 4096);
      dma16(src + 4, dst + i * 4096 + TILE / 2);
    }
  };
  // the weights of a mean tile's slots: slot tid % 32 as block tid / 32 of the item sees it: n_j, or 0
  auto mean_weights = [&](const Tile& t, int stage) {
    if (tid < 64) {
      const int s = t.start + (tid & 31);
      float w = 0.f;
      if ((tid & 31) < t.nk && !(sets && ((set_bits(s) >> (tid >> 5)) & 1))) w = (float)bn[block_in_range(kvl[s], c.T)];
      wts[stage * 64 + tid] = w;
    }
  };
  auto issue = [&](const Tile& t, const auto mean_c, int stage) {
    constexpr bool mean = decltype(mean_c)::value;
    const uint32_t kdst = lds_addr(lds) + stage * 2 * TILE;
    if (BF && !mean && is_full(t)) {
      const long long off = tbase + ((long long)t.start + wave * RPL) * a.geo.stride_t;
      const T *k = (const T*)a.k + off, *v = (const T*)a.v + off;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        dma16(k, lane_off, kdst + (4 * i + wave) * 1024);
        dma16(v, lane_off, kdst + (4 * i + wave) * 1024 + TILE);
        k += 4 * RPL * a.geo.stride_t;
        v += 4 * RPL * a.geo.stride_t;
      }
      return;
    }
    int li = lane;
    asm volatile("" : "+v"(li));                       // worked out for every tile, not kept in registers
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int p = (4 * i + wave) * 64 + li;
      const uint32_t dst = kdst + (4 * i + wave) * 1024;
      if constexpr (!mean) {
        const int row = p / CT, ch = (p % CT) ^ (row & ST);
        const long long off = tbase + (long long)(t.start + min(row, t.nk - 1)) * a.geo.stride_t + ch * (16 / (int)sizeof(T));
        dma16((const T*)a.k + off, dst);
        dma16((const T*)a.v + off, dst + TILE);
      } else {
        const int row = p / CM, ch = (p % CM) ^ (row & SM);
        const int j = block_in_range(kvl[t.start + min(row, t.nk - 1)], c.T);
        const long long off = (bh * T_max + j) * D + ch * 4;
        dma16(a.kc + off, dst);
        dma16(a.vc + off, dst + TILE);
      }
    }
    if (mean) mean_weights(t, stage);
  };

  const bf16x8 minus[2] = {minus_ones(0, r16, g), minus_ones(1, r16, g)};
  f32x4 acc[NT][QT];                                   // element i: channel 16 ct + 4 g + i; on fp32 matrix instructions: see the store
  constexpr float NONE = WIDE ? INFINITY : -M_INIT;    // minus the maximum of no score
  float neg_m[QT], l_run[QT];                          // minus the running maximum (log2 domain; WIDE bf16: as the score is); sums per lane
  // what is added to a score before its weight is formed: while a WIDE row has seen nothing but masked slots, 0, so that their
  // weights are exp2(-infinity), not of a difference of infinities
  auto shift = [&](float nm) { return WIDE && nm == INFINITY ? 0.f : nm; };
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    neg_m[qt] = NONE;
    l_run[qt] = 0.f;
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) acc[ct][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto factor = [&](float diff) { return __builtin_amdgcn_exp2f(WIDE && BF ? diff * cscale : diff); };      // between two maxima, from their difference

  // ---- 16 KT keys from row `r0` of the stage: a half tile, or a whole one of tokens in the first pass over bf16 rows; `nk` of them real; wt: weights of a mean tile's 32 slots.  TERMS: kb and vb are the
  // same place, filled with the terms of the keys and, while `between` runs, with those of the values
  auto half = [&](const unsigned char* kb, const unsigned char* vb, const int r0, const int nk, const auto mean_c, const float* wt, const auto between)
      __attribute__((always_inline)) {
    constexpr bool mean = decltype(mean_c)::value;
    // the lane's coordinates for the reads of mean tiles: opaque, so that their many LDS addresses are worked out where they
    // are used instead of being kept in registers through the loop
    int rm = r16, gm = g;
    if (BF || TERMS) asm volatile("" : "+v"(rm), "+v"(gm));
    constexpr int KT = BF && !FULL32 && !mean ? 4 : 2;
    f32x4 s[KT][QT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) s[kt][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (TERMS) {
      f32x4 small[2][QT];                              // all products but high x high
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) small[kt][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) {
        ISA_GEN_FENCE();
        bf16x8 k3[2][3];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int u = 0; u < 3; ++u)
            k3[kt][u] = *reinterpret_cast<const bf16x8*>(kb + u * PLANE + ((16 * kt + rm) * CP + ((4 * ks + gm) ^ (rm & SP))) * 16);
#pragma unroll
        for (int u = 2; u >= 0; --u)                   // the smallest first
#pragma unroll
          for (int w = 2 - u; w >= 0; --w)
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
              for (int qt = 0; qt < QT; ++qt) {
                f32x4& to = u + w > 0 ? small[kt][qt] : s[kt][qt];
                to = mfma_bf(k3[kt][u], q3[qt][ks][w], to);
              }
      }
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) s[kt][qt] += small[kt][qt];
    } else if constexpr (FM) {
      f32x4 k4[2][2];                                  // [t % 2][kt]: the fragments of a step are read a step ahead
      auto k_load = [&](int t) {
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
          k4[t & 1][kt] = *reinterpret_cast<const f32x4*>(kb + ((16 * kt + r16) * CM + ((4 * t + g) ^ r16)) * 16);
      };
      k_load(0);
      // every other group of four channels adds up here, in two chains of half the length.  Error against 64 bits of dense attention over
      // 1000 / 5280 tokens with one chain and with two, 128 channels: 1.15e-6 / 2.31e-6, 7.4e-7 / 1.99e-6 (four partial sums in scalar
      // arithmetic: 1.08e-6 / 5.87e-6), 64 channels 9.0e-7 / 1.47e-6, 6.3e-7 / 1.26e-6
      f32x4 s_odd[2][QT];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) s_odd[kt][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        ISA_GEN_FENCE();
        if (t + 1 < NT) k_load(t + 1);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) {
              f32x4& to = i & 1 ? s_odd[kt][qt] : s[kt][qt];
              to = mfma_f(k4[t & 1][kt][i], qf[qt][t][i], to);
            }
      }
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) s[kt][qt] += s_odd[kt][qt];
    } else if constexpr (!mean) {
      if constexpr (BF && D == 64) __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks)
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
          const bf16x8 k8 = *reinterpret_cast<const bf16x8*>(kb + ((r0 + 16 * kt + r16) * CT + ((4 * ks + g) ^ (r16 & ST))) * 16);
#pragma unroll
          for (int qt = 0; qt < QT; ++qt) s[kt][qt] = mfma_bf(k8, qb[qt][ks], s[kt][qt]);
        }
    } else {
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
          ISA_GEN_FENCE();
          float x[8];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const f32x4 k4 = *reinterpret_cast<const f32x4*>(kb + ((16 * kt + rm) * CM + ((8 * ks + 2 * gm + u) ^ rm)) * 16);
#pragma unroll
            for (int i = 0; i < 4; ++i) x[4 * u + i] = k4[i];
          }
          if constexpr (FULL32) {
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) {
              uint4 qw = __builtin_bit_cast(uint4, qb[qt][ks]);          // converted here, not kept as fp32
              asm volatile("" : "+v"(qw.x), "+v"(qw.y), "+v"(qw.z), "+v"(qw.w));
              const uint32_t q2[4] = {qw.x, qw.y, qw.z, qw.w};
#pragma unroll
              for (int e = 0; e < 8; ++e)
                s[kt][qt] = mfma_f(x[e], bits_f(e & 1 ? q2[e >> 1] & 0xffff0000u : q2[e >> 1] << 16), s[kt][qt]);
            }
          } else {
            bf16x8 k3[3];
            split3<false>(x, k3);
#pragma unroll
            for (int u = 2; u >= 0; --u)
#pragma unroll
              for (int qt = 0; qt < QT; ++qt) s[kt][qt] = mfma_bf(k3[u], qb[qt][ks], s[kt][qt]);
          }
        }
    }
    if constexpr (BF && D == 64) __builtin_amdgcn_s_setprio(0);
    // masks: slots past the end, mean slots with weight 0
    f32x4 w4[2];
    if constexpr (mean) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        w4[kt] = *reinterpret_cast<const f32x4*>(wt + 16 * kt + 4 * g);
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
#pragma unroll
          for (int i = 0; i < 4; ++i) s[kt][qt][i] = w4[kt][i] > 0.f ? s[kt][qt][i] : -INFINITY;
      }
    } else if (nk < 16 * KT) {
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
#pragma unroll
          for (int i = 0; i < 4; ++i) s[kt][qt][i] = 16 * kt + 4 * g + i < nk ? s[kt][qt][i] : -INFINITY;
      asm volatile("");                                // a branch around all of it, not selects in every full tile
    }
    // running maxima, raised only when a score exceeds one by more than 2^tau
    float mx[QT];
    unsigned long long raise = 0ull;
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      mx[qt] = s[0][qt][0];
#pragma unroll
      for (int e = 1; e < 4 * KT - 1; e += 2) mx[qt] = fmaxf(fmaxf(mx[qt], s[e >> 2][qt][e & 3]), s[(e + 1) >> 2][qt][(e + 1) & 3]);
      mx[qt] = fmaxf(mx[qt], s[KT - 1][qt][3]) * (WIDE ? 1.f : cscale);
      raise |= __ballot((mx[qt] + neg_m[qt]) * (WIDE && BF ? cscale : 1.f) > (FULL32 ? 0.f : RESCALE_TAU));
    }
    if (raise != 0ull) {
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        float m = fmaxf(mx[qt], __shfl_xor(mx[qt], 16, 64));
        m = fmaxf(m, __shfl_xor(m, 32, 64));
        m = fmaxf(m, -neg_m[qt]);
        const float alpha = factor(shift(-m) - neg_m[qt]);
        neg_m[qt] = -m;
        l_run[qt] *= alpha;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) acc[ct][qt] *= alpha;
      }
    }
#pragma unroll
    for (int k0 = 0; k0 < KT; k0 += 2) {
      f32x4 p[QT][2];                                    // [kt % 2]
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        const float sh = shift(neg_m[qt]);
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            p[qt][kt][i] = __builtin_amdgcn_exp2f(WIDE ? (s[k0 + kt][qt][i] + sh) * (BF ? cscale : 1.f) : fmaf(s[k0 + kt][qt][i], cscale, sh));
      }
      if constexpr (mean) {                              // Eq. 4: a mean key weighs its block's token count
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
#pragma unroll
          for (int kt = 0; kt < 2; ++kt) p[qt][kt] *= w4[kt];
      }
#pragma unroll
      for (int qt = 0; qt < QT; ++qt)
#pragma unroll
        for (int e = 0; e < 8; ++e) l_run[qt] += p[qt][e >> 2][e & 3];
      // O^T += V^T P^T
      if constexpr (TERMS) {
        bf16x8 p3[QT][3];
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
          split3<true>(p[qt][0], p[qt][1], minus, p3[qt]);
          asm volatile("" : "+v"(p3[qt][0]), "+v"(p3[qt][1]), "+v"(p3[qt][2]), "+v"(l_run[qt]));      // before the barriers, not where they are used
        }
        ISA_GEN_FENCE();
        between();
        asm volatile("" : "+v"(rm), "+v"(gm));
        const int tr_row = 4 * gm + (rm >> 2);
        constexpr int GR = 2;                            // (one at a time 4 % slower, four alike)
#pragma unroll
        for (int c0 = 0; c0 < NT; c0 += GR) {
          ISA_GEN_FENCE();
          bf16x8 v3[GR][3];
#pragma unroll
          for (int n = 0; n < GR; ++n)
#pragma unroll
            for (int u = 0; u < 3; ++u) {
              const unsigned char* src = vb + u * PLANE + (tr_row * CP + ((2 * (c0 + n) + ((rm & 3) >> 1)) ^ (tr_row & SP))) * 16 + (rm & 1) * 8;
              const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(src));
              const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(src + 16 * CP * 16));
              v3[n][u] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
#pragma unroll
          for (int u = 2; u >= 0; --u)
#pragma unroll
            for (int w = 2 - u; w >= 0; --w)
#pragma unroll
              for (int n = 0; n < GR; ++n)
#pragma unroll
                for (int qt = 0; qt < QT; ++qt) acc[c0 + n][qt] = mfma_bf(v3[n][u], p3[qt][w], acc[c0 + n][qt]);
        }
      } else if constexpr (FM) {
        f32x4 v4[2][NT / 4];                             // tiles 4 u + e: output row m is channel 64 u + 4 m + e
        auto v_load = [&](int n) {                       // key slot 16 kt + 4 g + i, n = 4 kt + i
          const int row = 4 * (n & 4) + 4 * g + (n & 3);
#pragma unroll
          for (int u = 0; u < NT / 4; ++u) {
            v4[n & 1][u] = *reinterpret_cast<const f32x4*>(vb + (row * CM + ((16 * u + r16) ^ (row & SM))) * 16);
            if (mean ? w4[n >> 2][n & 3] == 0.f : nk < 32 && row >= nk) v4[n & 1][u] = f32x4{0.f, 0.f, 0.f, 0.f};      // what is masked may hold anything
          }
        };
        v_load(0);
#pragma unroll
        for (int n = 0; n < 8; ++n) {
          ISA_GEN_FENCE();
          if (n + 1 < 8) v_load(n + 1);
#pragma unroll
          for (int u = 0; u < NT / 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
              for (int qt = 0; qt < QT; ++qt) acc[4 * u + e][qt] = mfma_f(v4[n & 1][u][e], p[qt][n >> 2][n & 3], acc[4 * u + e][qt]);
        }
      } else if constexpr (FULL32) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          asm volatile("" : "+v"(rm), "+v"(gm));
          const int row = (e & 4) * 4 + 4 * gm + (e & 3);
#pragma unroll
          for (int ct = 0; ct < NT; ++ct) {
            ISA_GEN_FENCE();
            float v;
            if constexpr (mean) v = *reinterpret_cast<const float*>(vb + (row * CM + ((4 * ct + (rm >> 2)) ^ (row & SM))) * 16 + (rm & 3) * 4);
            else v = bits_f((uint32_t)*reinterpret_cast<const uint16_t*>(vb + ((r0 + row) * CT + ((2 * ct + (rm >> 3)) ^ (row & ST))) * 16 + (rm & 7) * 2) << 16);
            if (mean ? w4[e >> 2][e & 3] == 0.f : row >= nk) v = 0.f;
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) acc[ct][qt] = mfma_f(v, p[qt][e >> 2][e & 3], acc[ct][qt]);
          }
        }
      } else {
        bf16x8 p3[QT][3];
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) split3<false>(p[qt][0], p[qt][1], minus, p3[qt]);
        if constexpr (!mean) {
          const int tr_row = 4 * g + (r16 >> 2);         // see the transposed reads of the backward kernel
          if constexpr (D == 64) __builtin_amdgcn_s_setprio(1);
          constexpr int GR = 4;                          // output tiles whose V^T fragments are held at a time
#pragma unroll
          for (int c0 = 0; c0 < NT; c0 += GR) {
            bf16x8 v8[GR];
#pragma unroll
            for (int n = 0; n < GR; ++n) {
              const unsigned char* src = vb + ((r0 + 16 * k0 + tr_row) * CT + ((2 * (c0 + n) + ((r16 & 3) >> 1)) ^ (tr_row & ST))) * 16 + (r16 & 1) * 8;
              const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(src));
              const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(src + 16 * CT * 16));
              v8[n] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
#pragma unroll
            for (int u = 2; u >= 0; --u)                 // the small terms first
#pragma unroll
              for (int n = 0; n < GR; ++n)
#pragma unroll
                for (int qt = 0; qt < QT; ++qt) acc[c0 + n][qt] = mfma_bf(v8[n], p3[qt][u], acc[c0 + n][qt]);
          }
          if constexpr (D == 64) __builtin_amdgcn_s_setprio(0);
        } else {
#pragma unroll
          for (int ct = 0; ct < NT; ++ct) {
            ISA_GEN_FENCE();
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const int row = (e & 4) * 4 + 4 * gm + (e & 3);
              x[e] = *reinterpret_cast<const float*>(vb + (row * CM + ((4 * ct + (rm >> 2)) ^ (row & SM))) * 16 + (rm & 3) * 4);
            }
            bf16x8 v3[3];
            split3<false>(x, v3);
#pragma unroll
            for (int u = 2; u >= 0; --u)
#pragma unroll
              for (int w = 2; w >= 0; --w)
                if (u + w < 4) {
#pragma unroll
                  for (int qt = 0; qt < QT; ++qt) acc[ct][qt] = mfma_bf(v3[u], p3[qt][w], acc[ct][qt]);
                }
          }
        }
      }
    }
  };

  // ---- the loop: the loads of a group's next tile fly while its current one is multiplied
  int n_first = 0, n_mine = 0;                         // tiles of the first group / of this one among those described
  auto next_mine = [&]() -> Tile {
    if constexpr (NG == 1) {
      next_tile();
      return at;
    }
    Tile mine = at;
#pragma unroll
    for (int u = 0; u < NG; ++u) {
      if (!at.end) next_tile();
      if (u == 0) n_first += at.end ? 0 : 1;
      if (u == grp) mine = at;
    }
    return mine;
  };
  Tile cur = next_mine();
  // Queries whose terms have lost bits: at once.  (Here, as the first tables are read while the queries are: 0.3 us of a call of 24, further up 0.6.)
  if constexpr (TERMS)
    if (__syncthreads_or(q_lost & 0xffffu)) return false;
  int stage = 0;
  // TERMS: this wave's share of a tile of keys or values, which it has fetched itself, taken apart into the common place
  auto take_apart = [&](const bool value) {
    const unsigned char* const src = lds + (value ? TILE : 0);
    int li = lane;
    asm volatile("" : "+v"(li));
#pragma unroll
    for (int i = 0; i < D / 64; ++i) {
      ISA_GEN_FENCE();
      const int p = (4 * i + wave) * 64 + li, row = p / CP;
      float x[8];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const f32x4 y = *reinterpret_cast<const f32x4*>(src + u * (TILE / 2) + p * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * u + e] = y[e];
      }
      bf16x8 t[3];
      const uint32_t rest = split3<true>(x, t);
      lost |= value ? rest << 16 : rest & 0xffffu;
      asm volatile("" : "+v"(lost));                   // here, not where it is read
#pragma unroll
      for (int u = 0; u < 3; ++u) *reinterpret_cast<bf16x8*>(lds + 2 * TILE + u * PLANE + (row * CP + ((p % CP) ^ (row & SP))) * 16) = t[u];
    }
  };
  auto tiles = [&](const auto mean_c) __attribute__((always_inline)) {
    constexpr bool mean = decltype(mean_c)::value;
    if constexpr (TERMS) {
      // The keys' raw tile, then the values', become terms in one place; each raw place is filled again as soon as its wave has read it
      // (with the same tile where there is no next one: with branches around the loads, and tiles of both kinds in one loop, the compiler
      // keeps the accumulators twice and spills 80 registers).  Loads end in order: when no more than one tensor's are in flight,
      // those of the tensor before it are there.
      if (cur.end || cur.mean != mean) return;
      if (mean) mean_weights(cur, stage);
      issue_terms(cur, mean_c, false);
      issue_terms(cur, mean_c, true);
      for (bool more = true; more; stage ^= 1) {
        const Tile nxt = next_mine();
        more = !nxt.end && nxt.mean == mean;
        const Tile load = more ? nxt : cur;
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NI) : "memory");
        ISA_GEN_BARRIER();                             // everybody has left the values of the tile before
        take_apart(false);
        if (mean) mean_weights(load, stage ^ 1);
        issue_terms(load, mean_c, false);
        ISA_GEN_BARRIER();
        __builtin_amdgcn_s_setprio(1);
        auto values = [&]() __attribute__((always_inline)) {
          asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NI) : "memory");
          ISA_GEN_BARRIER();                           // everybody has left the keys
          __builtin_amdgcn_s_setprio(0);
          take_apart(true);
          issue_terms(load, mean_c, true);
          ISA_GEN_BARRIER();
          __builtin_amdgcn_s_setprio(1);
        };
        // a tile of the other block's exact set has no keys for this wave
        half(lds + 2 * TILE, lds + 2 * TILE, 0, (cur.bits >> own) & 1 ? cur.nk : 0, mean_c, wts + stage * 64 + own * 32, values);
        __builtin_amdgcn_s_setprio(0);
        cur = nxt;
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      ISA_GEN_BARRIER();                               // everybody has left the weights of the last tile
      return;
    }
    if (cur.end || cur.mean != mean) return;
    issue(cur, mean_c, stage);
    for (bool more = true; more; stage ^= 1) {
      const Tile nxt = next_mine();                    // its table reads wait together with the tile loads
      more = !nxt.end && nxt.mean == mean;
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();                                 // the tile is complete; everybody has left the one before, whose stage is filled next
      if (more) issue(nxt, mean_c, stage ^ 1);
      const unsigned char* kb = lds + stage * 2 * TILE;
      const int n_own = (cur.bits >> own) & 1 ? cur.nk : 0;      // a tile of the other block's exact set has no keys for this wave
      if constexpr (BF && !FULL32) {
        if (n_own > 0) half(kb, kb + TILE, 0, n_own, mean_c, wts + stage * 64 + own * 32, [] {});
      } else {
#pragma unroll 1
        for (int r0 = 0; r0 < n_own; r0 += 32) half(kb, kb + TILE, r0, n_own - r0, mean_c, wts + stage * 64 + own * 32, [] {});
      }
      cur = nxt;
      ++n_mine;
    }
  };
  // two loops: the kinds of tile share no code path through which the accumulators would have to be moved
  tiles(std::false_type{});
  tiles(std::true_type{});
  if (NG > 1 && n_mine < n_first) __syncthreads();     // the first group has had one tile, and one barrier, more
  __syncthreads();                                     // nobody reads LDS any more: the caller may start another pass

  // ---- the second group's part (the merge step of the online softmax)
  if constexpr (NG > 1) {
    constexpr int W = QT * (4 * NT + 2);               // floats of a lane
    float* const hand = reinterpret_cast<float*>(lds_all + ITEM_LDS<D>) + wave * W * 64 + lane;
    if (grp == 1) {
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        hand[(qt * (4 * NT + 2)) * 64] = neg_m[qt];
        hand[(qt * (4 * NT + 2) + 1) * 64] = l_run[qt];
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
          for (int i = 0; i < 4; ++i) hand[(qt * (4 * NT + 2) + 2 + 4 * ct + i) * 64] = acc[ct][qt][i];
      }
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        const float other = hand[(qt * (4 * NT + 2)) * 64];
        const float nm = fminf(neg_m[qt], other);      // minus the larger maximum
        const float mine = factor(shift(nm) - neg_m[qt]), theirs = factor(shift(nm) - other);
        neg_m[qt] = nm;
        l_run[qt] = l_run[qt] * mine + hand[(qt * (4 * NT + 2) + 1) * 64] * theirs;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[ct][qt][i] = acc[ct][qt][i] * mine + hand[(qt * (4 * NT + 2) + 2 + 4 * ct + i) * 64] * theirs;
      }
    }
    __syncthreads();                                   // read before the caller's next pass fills the stages again
  }

  // ---- normalise, check, store
  float inv[QT];
  bool ok = true;
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    float l = l_run[qt];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    inv[qt] = 1.0f / l;
    if (grp == 0 && row0 + 16 * qt + r16 < n_q) {
      if (!WIDE) ok = ok && fabsf(neg_m[qt]) < FAST_MAX;
#pragma unroll
      for (int ct = 0; ct < NT; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i) ok = ok && fabsf(acc[ct][qt][i] * inv[qt]) < INFINITY;
    }
  }
  if constexpr (TERMS) {
    // Lost bits of keys (less than 2^-133 each) change a score of queries below 2^96 by less than 2^-29, those of values a result by less than
    // 2^-133, 2^-25 of one of 2^-108: the item is run again where queries or results are beyond.  8 heads of 5280 tokens, us, fp32 instructions
    // alone / in terms, none such / one value or key of 2^-120 a head, always run again / now: 287 / 183 / 301 / 180; 24 heads of 64 channels 390 / 285 / 618 / 287; a
    // query in every block 292 / - / 445 / 321; nothing but such values, both passes: 291 / - / 447 / 447
    if (__syncthreads_or(!ok || lost != 0)) {
      const bool keys = __syncthreads_or(lost & 0xffffu), values = __syncthreads_or(lost >> 16);
      uint32_t q_max = 0;                              // of the leading terms, sign off
      float o_min = INFINITY;
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks) {
          const uint4 w = __builtin_bit_cast(uint4, q3[qt][ks][0]);
          q_max = max(q_max, max(max(w.x << 1, w.y << 1), max(w.z << 1, w.w << 1)));
          q_max = max(q_max, max(max(w.x << 17, w.y << 17), max(w.z << 17, w.w << 17)));
        }
        if (row0 + 16 * qt + r16 < n_q)
#pragma unroll
          for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int i = 0; i < 4; ++i) o_min = fminf(o_min, fabsf(acc[ct][qt][i] * inv[qt]));
      }
      if (__syncthreads_or(!ok || (keys && q_max >= __float_as_uint(0x1p96f) << 1) || (values && o_min < 0x1p-108f))) return false;
    }
  } else if constexpr (!FULL32) {
    if (__syncthreads_or(!ok)) return false;
  }
  if (grp != 0) return true;
  if (PARTS && part >= 0) {
    const long long part_row = (long long)(first_part + part) * (64 * QI) + (FULL32 ? 64 * (slot % QI) : 0);
    // normalised; the maximum in the units it was subtracted in: a minus in the sum's
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {                  // sign bit: of the score as it is (WIDE, bf16), else in the log2 domain
      float l = l_run[qt];
      l += __shfl_xor(l, 16, 64);
      l += __shfl_xor(l, 32, 64);
      const long long row = part_row + wave * 16 * QT + 16 * qt + r16;
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        f32x4 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = (FM ? acc[4 * (n >> 2) + i][qt][n & 3] : acc[n][qt][i]) * inv[qt];
        *reinterpret_cast<f32x4*>(ga.part_o + row * D + (FM ? 64 * (n >> 2) + 16 * g + 4 * (n & 3) : 16 * n + 4 * g)) = r;
      }
      if (g == 0) ga.part_ml[row] = make_float2(-neg_m[qt], WIDE && BF ? -l : l);
    }
    return true;
  }
  // coarse residual (Alg. 1 Stage 5): the block's row of O_coarse, the same for all of its tokens
  const float* const oc = (a.ocoarse && !a.dense) ? a.ocoarse + (bh * T_max + qi) * D : nullptr;
#pragma unroll
  for (int qt = 0; qt < QT; ++qt) {
    const int row = row0 + 16 * qt + r16;
    if (row >= n_q) continue;
    T* op = (T*)a.out + tbase + (long long)(q_start + row) * a.geo.stride_t;
#pragma unroll
    for (int n = 0; n < NT; ++n) {                     // four consecutive channels at a time
      float r[4];
      const int ch = FM ? 64 * (n >> 2) + 16 * g + 4 * (n & 3) : 16 * n + 4 * g;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        r[i] = (FM ? acc[4 * (n >> 2) + i][qt][n & 3] : acc[n][qt][i]) * inv[qt];
        if (oc) r[i] = fmaf(a.gamma, oc[ch + i], r[i]);
      }
      if constexpr (BF) {
        *reinterpret_cast<uint2*>(op + ch) = make_uint2(f2bf(r[0]) | ((uint32_t)f2bf(r[1]) << 16), f2bf(r[2]) | ((uint32_t)f2bf(r[3]) << 16));
      } else {
        *reinterpret_cast<float4*>(op + ch) = make_float4(r[0], r[1], r[2], r[3]);
      }
    }
  }
  return true;
}

// (the launch bounds' second number is wavefronts per SIMD: the same for one and for two groups)
template <typename T, int D, int QT, bool PARTS, int NG>
__global__ __launch_bounds__(256 * NG, (RESIDENT<D, QT>)) void k_attn_gen(GenArgs ga) {
  static_assert(NG == 1 || (QT == 1 && !PARTS), "what is launched");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NG * ITEM_LDS<D>];
  // Workgroup ids go round-robin over the 8 XCDs; each has its range of the items of all (batch, head)s, the long ones
  // (exact branch) first: all items' first parts, then their second ones (what runs together reads the same keys).
  const int xcd = blockIdx.x & 7, n_bh = ga.a.geo.B * ga.a.geo.H;
  int j = blockIdx.x >> 3, bhid = -1, slot = 0, part = -1, first_part = 0;
  bool taylor = false;
  if (!ga.ragged) {
    const int n_long = ga.per_xcd_long * (PARTS ? ga.parts : 1);
    taylor = j >= n_long;
    if (taylor) j -= n_long;
    else if (PARTS) { part = j / ga.per_xcd_long; j %= ga.per_xcd_long; }
    const int slots = taylor ? ga.slots_taylor : ga.slots_long;
    const long long total = (long long)n_bh * slots;
    const int idx = xcd_first(total, xcd) + j;
    if (idx >= xcd_first(total, xcd + 1)) return;
    bhid = head_at(idx / slots, n_bh);
    slot = idx % slots;
  } else {
    uint32_t first = 0, n = 0;
    int found = -1, parts = 1;
#pragma unroll
    for (int i = 0; i < 2 * ISA_MAX_BATCH; ++i) {      // unrolled: the arguments are loaded together
      const int k = i % ISA_MAX_BATCH;
      const uint32_t total = i < ISA_MAX_BATCH ? ga.long_items[k] : ga.taylor_items[k];
      if (found >= 0) continue;
      first = total * xcd >> 3;                        // x 8 is below 2^32
      n = (total * (xcd + 1) >> 3) - first;
      parts = PARTS && i < ISA_MAX_BATCH ? nibble(ga.own_parts, nibble(ga.by_length, k)) : 1;
      if (j < (int)n * parts) found = i;
      else j -= (int)n * parts;
    }
    if (found < 0) return;
    taylor = found >= ISA_MAX_BATCH;
    const int b = nibble(ga.by_length, found % ISA_MAX_BATCH);
    const int slots = slots_of(ga.a.geo.block, ga.a.dense ? ga.a.cnt.b[b].T : taylor ? ga.a.cnt.b[b].n_flat : ga.a.cnt.b[b].n_full, 64 * QT);
    part = parts > 1 ? j / (int)n : -1;
    const int item = (int)first + j % (int)n;
    bhid = b * ga.a.geo.H + head_at(item / slots, ga.a.geo.H);
    slot = item % slots;
  }
  bhid = __builtin_amdgcn_readfirstlane(bhid);
  slot = __builtin_amdgcn_readfirstlane(slot);
  part = PARTS ? __builtin_amdgcn_readfirstlane(part) : -1;
  taylor = __builtin_amdgcn_readfirstlane(taylor ? 1 : 0) != 0;
  const int b = bhid / ga.a.geo.H;
  const BatchCounts c = ga.a.cnt.b[b];
  const int n_list = ga.a.dense ? c.T : taylor ? c.n_flat : c.n_full;
  if (PARTS && part >= 0)
    first_part = ga.first_part[b] + (bhid % ga.a.geo.H * slots_of(ga.a.geo.block, n_list, 64 * QT) + slot) * nibble(ga.own_parts, b);
  // QT-tile slot n of a list: rows 64 QT n .. of a 128-row block's sequence of rows, or block n / blocks 2 n, 2 n + 1 of 64 rows
  auto first_entry = [&](int qt, int n) { return ga.a.geo.block == 64 ? qt * n : n * qt / 2; };
  if (attn_gen_item<T, D, QT, false, QT, PARTS, NG>(ga, lds, bhid, taylor, slot, part, first_part)) return;
#pragma unroll 1
  for (int n = QT * slot; n < QT * (slot + 1); ++n)    // again, 64 rows at a time
    if (first_entry(1, n) < n_list) attn_gen_item<T, D, 1, true, QT, PARTS, NG>(ga, lds, bhid, taylor, n, part, first_part);
}

// Adds up the parts of the long items: out = sum_p o_p l_p 2^(m_p - m) / sum_p l_p 2^(m_p - m) with m = max_p m_p (the merge step
// of the online softmax).  The parts' results are normalised, so that no sum of them leaves the range; a part that has seen nothing but
// masked keys (l_p = 0) has none.  Maxima of the two passes over bf16 rows meet in double precision: a difference of theirs must not carry
// the rounding of a large score.  One workgroup per item and 1024 / D rows, 4 channels a thread.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_gen_merge(GenArgs ga, int rows) {
  constexpr int RW = 1024 / D;                         // rows of a workgroup
  const AttnArgs& a = ga.a;
  const int per_item = rows / RW, idx = blockIdx.x / per_item;
  const int row = blockIdx.x % per_item * RW + threadIdx.x / (D / 4), ch = threadIdx.x % (D / 4) * 4;
  const int n_bh = a.geo.B * a.geo.H, slots = ga.slots_long;
  const int bhid = head_at(idx / slots, n_bh), slot = idx % slots, b = bhid / a.geo.H, h = bhid % a.geo.H;
  const BatchCounts c = a.cnt.b[b];
  const int parts = nibble(ga.own_parts, b), n_list = a.dense ? c.T : c.n_full;
  if (parts == 1) return;
  const bool pair = rows == 128 && a.geo.block == 64;
  const int subs = pair ? 1 : a.geo.block / rows;
  const int entry = pair ? 2 * slot + row / 64 : slot / subs;
  if (entry >= n_list) return;
  const int qi = a.dense ? entry : block_in_range(a.full_list[(long long)bhid * a.geo.T_max + entry], c.T);
  const int in_block = pair ? row % 64 : slot % subs * rows + row;
  if (in_block >= a.blk_n[b * a.geo.T_max + qi]) return;
  const long long first = (long long)(ga.first_part[b] + (h * slots_of(a.geo.block, n_list, rows) + slot) * parts) * rows + row;
  const double cs = 1.4426950408889634f / sqrtf((float)D);       // the factor of the passes, rounded as there: another is 1e-8 of a large score off
  auto log2_max = [&](const float2 ml) { return sizeof(T) == 2 && (__float_as_uint(ml.y) >> 31) ? (double)ml.x * cs : (double)ml.x; };
  // all parts' loads in flight at once (a part past the last repeats it, with weight 0)
  float2 ml[MAX_PARTS];
  float4 o[MAX_PARTS];
#pragma unroll
  for (int p = 0; p < MAX_PARTS; ++p) {
    const long long at = first + (long long)min(p, parts - 1) * rows;
    ml[p] = ga.part_ml[at];
    o[p] = *reinterpret_cast<const float4*>(ga.part_o + at * D + ch);
  }
  double m = -INFINITY;
#pragma unroll
  for (int p = 0; p < MAX_PARTS; ++p)
    if (ml[p].y != 0.f) m = fmax(m, log2_max(ml[p]));  // (a NaN sum makes the result NaN below)
  float w[MAX_PARTS], l = 0.f;
#pragma unroll
  for (int p = 0; p < MAX_PARTS; ++p) {
    w[p] = p < parts && ml[p].y != 0.f ? fabsf(ml[p].y) * __builtin_amdgcn_exp2f((float)(log2_max(ml[p]) - m)) : 0.f;
    l += w[p];
  }
  const float inv = 1.0f / l;
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int p = 0; p < MAX_PARTS; ++p) {
    if (p >= parts || ml[p].y == 0.f) continue;
    const float x = w[p] * inv;
    sum.x = fmaf(x, o[p].x, sum.x); sum.y = fmaf(x, o[p].y, sum.y); sum.z = fmaf(x, o[p].z, sum.z); sum.w = fmaf(x, o[p].w, sum.w);
  }
  if (l == 0.f) sum = make_float4(NAN, NAN, NAN, NAN);                   // no key at all that is not masked
  if (a.ocoarse && !a.dense) {
    const float4 oc = *reinterpret_cast<const float4*>(a.ocoarse + ((long long)bhid * a.geo.T_max + qi) * D + ch);
    sum.x = fmaf(a.gamma, oc.x, sum.x); sum.y = fmaf(a.gamma, oc.y, sum.y); sum.z = fmaf(a.gamma, oc.z, sum.z); sum.w = fmaf(a.gamma, oc.w, sum.w);
  }
  T* op = (T*)a.out + (long long)b * a.geo.stride_b + (long long)h * a.geo.stride_h + (long long)(a.blk_start[b * a.geo.T_max + qi] + in_block) * a.geo.stride_t + ch;
  if constexpr (sizeof(T) == 2) *reinterpret_cast<uint2*>(op) = make_uint2(f2bf(sum.x) | ((uint32_t)f2bf(sum.y) << 16), f2bf(sum.z) | ((uint32_t)f2bf(sum.w) << 16));
  else *reinterpret_cast<float4*>(op) = sum;
}

// The long items cut: those of the batch item with the longest key list into p parts, the others into parts of about the same length (of
// at least a block, bf16: 256 tokens).  cut.slots (long items of a (batch, head)) is there; false if p parts are too many or the partial
// results have no room.
struct Cut { int slots[ISA_MAX_BATCH], parts[ISA_MAX_BATCH], first[ISA_MAX_BATCH]; };
static bool cut_long_items(const Problem& pr, bool dense, int rows, int p, Cut& cut) {
  int longest = 1;
  for (int b = 0; b < pr.p.B; ++b)
    if (cut.slots[b] > 0) longest = max(longest, dense ? pr.cnt.b[b].T : pr.cnt.b[b].T_new);
  const int least = pr.p.dtype == ISA_BF16 ? 256 / pr.p.block : 1;          // blocks of a part
  if (p > 1 && longest < p * least) return false;
  long long n = 0;
  for (int b = 0; b < pr.p.B; ++b) {
    const int list = dense ? pr.cnt.b[b].T : pr.cnt.b[b].T_new;             // at most 4096
    cut.parts[b] = list == longest ? p : max(1, min(min(list / least, p), (2 * list * p + longest) / (2 * longest)));
    cut.first[b] = (int)n;
    if (cut.parts[b] > 1) n += (long long)pr.p.H * cut.slots[b] * cut.parts[b];
  }
  return n * rows * pr.p.D <= GEN_PARTIAL_ELEMENTS;
}

// Dense attention has the longest lists and the most long items; a workgroup of 128 rows holds one block of 64 at worst.
long long gen_partial_rows(const Problem& pr) {
  const int least = pr.p.dtype == ISA_BF16 ? 256 / pr.p.block : 1;
  long long rows = 0;
  for (int b = 0; b < pr.p.B; ++b) {
    const int T = pr.cnt.b[b].T, parts = min(MAX_PARTS, T / least);
    if (parts > 1) rows += (long long)pr.p.H * slots_of(pr.p.block, T, 128) * max(128, pr.p.block) * parts;
  }
  return min(rows, GEN_PARTIAL_ELEMENTS / pr.p.D);
}

hipError_t launch_attn_gen(const Problem& pr, const Workspace& ws, const AttnArgs& a, hipStream_t st) {
  GenArgs ga = {};
  ga.a = a;
  int n_long = 0, n_taylor = 0;
  long long taylor_128 = 0;                            // Taylor items of 128 rows
  double set_share = 0.0;                              // of a long item's tokens, those a Taylor item reads for its exact set
  for (int b = 0; b < pr.p.B; ++b) {
    const BatchCounts& c = pr.cnt.b[b];
    if (!a.dense && a.exact_mask && c.n_flat > 0) set_share = fmax(set_share, (double)c.k_exact / c.T_new);
    const int f = a.dense ? c.T : c.n_full, t = a.dense ? 0 : c.n_flat;
    n_long = f > n_long ? f : n_long;
    n_taylor = t > n_taylor ? t : n_taylor;
    taylor_128 += pr.p.H * slots_of(pr.p.block, t, 128);
  }
  const long long bh = (long long)pr.p.B * pr.p.H;
  const bool d64 = pr.p.D == 64, bf = pr.p.dtype == ISA_BF16;
  const double chip = (double)N_XCD * cus_per_xcd();
  // The form of a workgroup (64 rows; 128, which read every LDS fragment once for two query tiles; bf16 also 64 in two groups of waves) and the parts per long item,
  // chosen together by a model of the call's time: with k workgroups per compute unit a block of 64 tokens takes each of them pace[k - 1]
  // us (k beyond what fits a compute unit: further rounds), and a workgroup spends `start` tokens' time on its start.  The merge of partial
  // results is `merge` us more, and they are written and read at `rate` TB/s.  A Taylor item counts for `taylor` of a long one of the same
  // rows, plus its exact set's share (x `shared` in two groups); Taylor items fill what the long ones leave idle, so the time is that of the
  // long items' rounds or that of all items with the chip full, whichever is longer; not so beside two groups, which leave little idle.  A bf16
  // part has at least 256 tokens, an fp32 one may be a single block (D = 128, 1 head, 300 tokens: 46 whole, 35 in parts).
  // The numbers are fitted to 1200 calls (1 to 40 heads, 300 to 15 600 tokens, dense and sparse, ragged batches) with every form and number of
  // parts measured: the choice costs 0.7 to 1.5 % more than the best one on the geometric average.  Measured, whole calls, us, keep 0.5, full 0.25, whole
  // items of 128 rows / of 64 / in two groups / as chosen: bf16, 15 600 tokens, blocks of 64: D = 64, 1 head 325 / 247 / 203 / 77, 4 heads 340 / 266 /
  // 212 / 150, 8 349 / 282 / 295 / 250, 12 391 / 383 / 419 / 355, 16 442 / 482 / 545 / 442; D = 128: 2 heads 491 / 342 / 281 / 163, 4 505 / 353 / 358 / 253, 8
  // 513 / 477 / 671 / 428, 12 659 / 709 / 952 / 658 (the partial results have no room), 16 772 / 901 / 1257 / 770; dense, 1980 tokens, 8 heads: D = 64
  // 55 / 42 / 36 / 36, D = 128 84 / 56 / 51 / 52.  fp32, 64 rows / 128 / as chosen: 4800 tokens, D = 128, 4 heads 341 / 434 / 109, 12 351 / 448 / 192, D = 64, 4 heads 213 / 269 / 75.
  struct Form { int rows, groups, resident; double pace[4], start; };
  struct Kind { double taylor, shared, merge, rate; Form form[3]; };
  static const Kind kinds[2][2] = {                    // [bf16][D = 64]
      {{.0086, 1, 6.3, 4.7, {{64, 1, 2, {4.1, 4.8}, 40}, {128, 1, 2, {5.13, 6.52}, 30}}},
       {.013, 1, 3.7, 4.3, {{64, 1, 4, {2.15, 2.6, 3.04, 4.75}, 16}, {128, 1, 3, {3.15, 3.27, 5.25}, 14.5}}}},
      {{.075, 1.4, 6.0, 5.4, {{64, 1, 2, {1.63, 2.52}, 185}, {128, 1, 2, {2.67, 3.87}, 180}, {64, 2, 1, {2.77}, 145}}},
       {.0436, 1.68, 5.75, 3.7, {{64, 1, 4, {1.285, 1.57, 2.13, 3.04}, 257}, {128, 1, 3, {1.73, 2.5, 3.29}, 349}, {64, 2, 2, {1.85, 3.58}, 209}}}}};
  const Kind& kind = kinds[bf][d64];
  bool two = false, groups = false;
  Cut chosen = {};
  ga.parts = 1;
  if (n_long == 0) {
    // Taylor items alone, 128 rows / 64, us by items of 128 rows: bf16, D = 64: 2928 179 / 219, 912 53 / 57, 304 35.7 / 35.4; D = 128: 2928
    // 341 / 457, 304 50 / 57, 288 33 / 37, 244 79 / 78; fp32, D = 64: 2928 202 / 221, 912 60.3 / 60.4, 304 39.4 / 38.8; D = 128: 2928 430 / 524,
    // 288 39 / 41, 244 63 / 61; every batch item's own: 2 heads of 4977, 86 and 6481 tokens, bf16, D = 128, 182 items (306 if all were as long) 73 / 69.  With exact sets a pair of blocks of 64 reads both blocks' sets: bf16, 2928: D = 64 496 / 452, D = 128
    // 958 / 900; fp32 1207 / 885, 2424 / 1946.
    two = !(set_share > 0.0 && pr.p.block == 64) && taylor_128 >= chip * (bf ? (d64 ? 1.75 : 1.0) : d64 ? 3.5 : 1.0);
  } else {
    double best = INFINITY;
    for (int f = 0; f < (bf ? 3 : 2); ++f) {
      const Form& form = kind.form[f];
      // per workgroup with the chip full; a pair of blocks of 64 reads both blocks' exact sets
      const Form& one = kind.form[form.rows == 128];
      const double full = one.pace[one.resident - 1] / one.resident / chip;
      Cut cut;
      double taylor = 0.0;                             // the Taylor items, in tokens (as all below)
      for (int b = 0; b < pr.p.B; ++b) {
        const BatchCounts& c = pr.cnt.b[b];
        cut.slots[b] = slots_of(pr.p.block, a.dense ? c.T : c.n_full, form.rows);
        if (a.dense) continue;
        const double set = a.exact_mask && c.n_flat > 0 ? (double)c.k_exact / c.T_new : 0.0;
        taylor += (double)pr.p.H * slots_of(pr.p.block, c.n_flat, form.rows) * (kind.taylor + set * (form.rows > pr.p.block ? 2 : 1)) * c.T_new * pr.p.block;
      }
      for (int p = 1; p <= MAX_PARTS && (p == 1 || (ws.split_o && form.groups == 1)) && cut_long_items(pr, a.dense, form.rows, p, cut); ++p) {
        double work = 0.0, each = 0.0, partial = 0.0;  // all long items; the longest part; rows of partial results
        for (int b = 0; b < pr.p.B; ++b) {
          if (cut.slots[b] == 0) continue;
          const double tokens = (double)(a.dense ? pr.cnt.b[b].T : pr.cnt.b[b].T_new) * pr.p.block, own = tokens / (cut.parts[b] * form.groups) + form.start;
          work += (double)pr.p.H * cut.slots[b] * cut.parts[b] * own;
          each = fmax(each, own);
          if (cut.parts[b] > 1) partial += (double)pr.p.H * cut.slots[b] * cut.parts[b] * form.rows;
        }
        const int k = (int)ceil(work / (each * chip) - 1e-9), rounds = (k - 1) / form.resident;      // as many as if all were as long as the longest
        const double pace = rounds * form.pace[form.resident - 1] + form.pace[(k - 1) % form.resident];
        const double us = (form.groups > 1 ? pace * each + kind.shared * taylor * full : fmax(pace * each, (work + taylor) * full)) / 64;
        const double cost = us + (p > 1 ? kind.merge + partial * pr.p.D * 8e-6 / kind.rate : 0.0);
        if (cost < best) { best = cost; two = form.rows == 128; groups = form.groups > 1; ga.parts = p; chosen = cut; }
        if (p == 1 && best <= (work + taylor) * full / 64 + kind.merge) break;       // no number of parts can be quicker: they add starts and a merge
      }
    }
  }
  ga.part_o = ws.split_o; ga.part_ml = (float2*)ws.split_ml;
  const int rows = two ? 128 : 64;
  ga.slots_long = slots_of(pr.p.block, n_long, rows);
  ga.slots_taylor = slots_of(pr.p.block, n_taylor, rows);
  ga.per_xcd_long = (int)((bh * ga.slots_long + N_XCD - 1) / N_XCD);
  ga.per_xcd_taylor = (int)((bh * ga.slots_taylor + N_XCD - 1) / N_XCD);
  int wgs = ga.per_xcd_long * ga.parts + ga.per_xcd_taylor;               // of an XCD
  for (int b = 0; b < pr.p.B; ++b) {
    const BatchCounts &c = pr.cnt.b[b], &d = pr.cnt.b[0];
    ga.ragged |= a.dense ? c.T != d.T : c.T_new != d.T_new || c.n_full != d.n_full || c.n_flat != d.n_flat;
  }
  for (int b = 0; b < pr.p.B; ++b) {
    ga.first_part[b] = chosen.first[b];
    ga.own_parts |= (uint32_t)(ga.parts > 1 ? chosen.parts[b] : 1) << (4 * b);
  }
  if (ga.ragged) {
    wgs = 0;
    int order[ISA_MAX_BATCH];                          // longest key lists first, ties in order
    for (int b = 0; b < pr.p.B; ++b) {
      const BatchCounts& c = pr.cnt.b[b];
      int at = b;
      for (; at > 0 && (a.dense ? pr.cnt.b[order[at - 1]].T < c.T : pr.cnt.b[order[at - 1]].T_new < c.T_new); --at) order[at] = order[at - 1];
      order[at] = b;
    }
    for (int i = 0; i < pr.p.B; ++i) {
      const BatchCounts& c = pr.cnt.b[order[i]];
      ga.by_length |= (uint32_t)order[i] << (4 * i);
      ga.long_items[i] = (uint32_t)pr.p.H * slots_of(pr.p.block, a.dense ? c.T : c.n_full, rows);
      ga.taylor_items[i] = a.dense ? 0u : (uint32_t)pr.p.H * slots_of(pr.p.block, c.n_flat, rows);
      wgs += (int)((ga.long_items[i] + N_XCD - 1) / N_XCD) * nibble(ga.own_parts, order[i]) + (int)((ga.taylor_items[i] + N_XCD - 1) / N_XCD);
    }
  }
  if (ga.slots_long == 0) ga.slots_long = 1;           // divisors in the kernel; a branch without work gets no workgroups
  if (ga.slots_taylor == 0) ga.slots_taylor = 1;
  const dim3 grid((unsigned)(N_XCD * wgs));
#define ISA_GEN(T, D, QT)                                                                                  \
  do {                                                                                                     \
    if (ga.parts > 1) hipLaunchKernelGGL((k_attn_gen<T, D, QT, true, 1>), grid, dim3(256), 0, st, ga);      \
    else hipLaunchKernelGGL((k_attn_gen<T, D, QT, false, 1>), grid, dim3(256), 0, st, ga);                  \
  } while (0)
  if (groups && d64) hipLaunchKernelGGL((k_attn_gen<uint16_t, 64, 1, false, 2>), grid, dim3(512), 0, st, ga);
  else if (groups) hipLaunchKernelGGL((k_attn_gen<uint16_t, 128, 1, false, 2>), grid, dim3(512), 0, st, ga);
  else if (bf && d64) { if (two) ISA_GEN(uint16_t, 64, 2); else ISA_GEN(uint16_t, 64, 1); }
  else if (bf) { if (two) ISA_GEN(uint16_t, 128, 2); else ISA_GEN(uint16_t, 128, 1); }
  else if (d64) { if (two) ISA_GEN(float, 64, 2); else ISA_GEN(float, 64, 1); }
  else if (two) ISA_GEN(float, 128, 2);
  else ISA_GEN(float, 128, 1);
  if (ga.parts > 1) {
    const dim3 merge((unsigned)(bh * ga.slots_long * (rows * pr.p.D / 1024)));      // (slots_long: the most of a batch item)
    if (bf) {
      if (d64) hipLaunchKernelGGL((k_gen_merge<uint16_t, 64>), merge, dim3(256), 0, st, ga, rows);
      else hipLaunchKernelGGL((k_gen_merge<uint16_t, 128>), merge, dim3(256), 0, st, ga, rows);
    } else {
      if (d64) hipLaunchKernelGGL((k_gen_merge<float, 64>), merge, dim3(256), 0, st, ga, rows);
      else hipLaunchKernelGGL((k_gen_merge<float, 128>), merge, dim3(256), 0, st, ga, rows);
    }
  }
#undef ISA_GEN
  return hipGetLastError();
}

}  // namespace isa
