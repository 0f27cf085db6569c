// Backward pass of In-Context Sparse Attention for bf16, D = 128, block = 128 on gfx950 (the paper states that the
// operator is trainable, Sec. 4 "Implementation Detail and Analysis", and gives no formulas: these are the analytic
// gradients of Alg. 1 Stages 4-5 with the index decisions of Stages 2 and 3 held fixed).
//
// With P = softmax weights of a query row (exact branch: over the tokens of the kept blocks; Taylor branch, Eq. 4: over
// the kept blocks' mean keys, each weighted with its token count n_j, and, with exact sets, Alg. 2 Part A, over the
// tokens of the block's exact set instead of their means), delta = rowsum(dO * O) and dP = dO V^T:
//     dS = P * (dP - delta),   dQ = dS K / sqrt(D),   dK = dS^T Q / sqrt(D),   dV = P^T dO,
// and the gradient of a block mean is spread evenly over the block's tokens (dK[t] += dKc[j] / n_j, same for V).
// The coarse residual gamma * O_coarse (Stages 1 and 5) adds the gradient of a small T x T attention over the block
// means (kernels at the end of this file), which enters the big launches through their epilogues.
//
// One kernel body does these products (dK and dV have a kernel of their own, attn_bwd_kv.hip).  A workgroup (8 waves)
// keeps 2 x 128 "stationary" rows in registers and streams 64-row tiles of the other side through LDS; per tile it forms
// T1 = Y1 X1^T (the scores) and, for dS (all but dVc), T2 = Y2 X2^T (dP), turns them into W = P or dS in registers and accumulates acc^T += Yt W^T, where Yt is the
// transpose of a streamed tile: its fragments are read out of the row-major tile in LDS with ds_read_b64_tr_b16, in the
// key order of the 16x16x32 accumulators, so no transposed copy of any tensor exists.  Three kinds of items, one launch:
//     dQ, exact branch : stationary (Q, dO) of the full-attention blocks,  streamed K, V of the kept tokens (Yt = K^T)
//     dQ, Taylor branch: stationary (Q, dO) of the Taylor blocks,          streamed Kc, Vc (block means), after the
//                        K, V tiles of the blocks' exact sets
//     dKc, dVc         : stationary (Kc, Vc) / Kc rows,                    streamed Q, dO of the Taylor blocks (Yt = Q^T / dO^T),
//                        half of the workgroups each
// Every output element is written by exactly one workgroup: no atomics, results are reproducible.
//
// The additive terms of a weight ride in the MFMA accumulators: T1 starts at b_x / c (minus the log-sum-exp of a
// stationary query row, log2 n_j of a stationary mean), T2 at minus delta: of the stationary rows when those are queries,
// of the streamed rows when these are (read from the tile's side array as the C operand of the first T2 MFMA), so that
// a weight costs an fma, an exp2, a multiplication and half a packed conversion.  Matrix and vector instructions issue
// through one port on this chip and a sub-tile's weights take about as long as its MFMAs, so the weights are issued in
// slices between the MFMAs of the following sub-tile, with the LDS fragments requested two steps ahead (one with exact sets).
// dQ of the exact branch at 480p with the paper's ratios: matrix pipe busy 64 % of the cycles, 2 cycles of bank conflicts per transposed
// read (1.5e9 of 6.4e9 LDS cycles; another swizzle: see attn_bwd_kv.hip).
#include "attn_mfma.h"

namespace isa {

#define ISA_BWD_FENCE() __builtin_amdgcn_sched_barrier(0)

namespace {

constexpr int STAGE = 2 * K_TILE;                    // bf16 elements of one LDS stage: the Y1 and Y2 tiles
constexpr int SIDE_BYTES = 1024;                      // per stage: 64 exponent terms, then 64 minus-deltas, of the streamed rows (512 B used)

// 16 bytes per lane from global memory straight into LDS (lane i -> LDS bytes lds_addr + 16 i); inline assembly so
// that the only wait for these loads is the explicit one at the top of the loop.
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff_bytes, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_addr), "v"(voff_bytes), "s"(sbase) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(size_t)(__attribute__((address_space(3))) const void*)p;
}
// A pointer that is wave-uniform by construction, moved to scalar registers explicitly.
__device__ __forceinline__ const char* uniform_ptr(const void* p) {
  const uint64_t u = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return reinterpret_cast<const char*>((uintptr_t)(((uint64_t)hi << 32) | lo));
}
typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v* lds_s4_ptr;
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

}  // namespace

// One phase of the streamed side of a launch: token tiles of the blocks of a list, or tiles of gathered block means.
struct BwdStream {
  const uint16_t* y1; const uint16_t* y2;     // row-major rows for the scores / for dP; the accumulation product reads
                                              // the transpose of y1 (launches that need dS) or of y2 (the others: dO)
  const uint16_t* y3;                         // EX == 2, mean tiles: rows whose transpose the accumulation product reads instead of
                                              // y1's (the mean keys without the subtraction of Kc_0); null otherwise
  const int4* tab;                            // token tiles: [bh][T_max] {token offset, tokens, block id} per list entry; null: mean tiles
  const float2* ybd;                          // per tile of 64 streamed positions: 64 additive exponent terms (-inf: masked), then 64 minus-deltas
  bool flat;                                  // token tiles: the list's entries are the Taylor blocks, otherwise the kept blocks
  int masked;                                 // exact sets (Alg. 2 Part A): 0 none; 1 token tiles of the entries whose bit is set for the
                                              // stationary entry, others skipped; 2 mean tiles, positions whose bit is set are masked;
                                              // 3 (mean rows stationary) entries whose bit is set for the lane's row are masked
};

struct BwdArgs {
  // stationary rows: token tensors (strides of `geo`, blocks taken from `stat_list`) or gathered mean rows [bh][Tn_pad][128]
  const uint16_t* x1; const uint16_t* x2;
  const int* stat_list;                       // [bh][T_max] block ids; unused for mean rows
  bool stat_flat;                             // they are the Taylor blocks, otherwise the full-attention blocks
  const float* bx; const float* dx;           // per stationary row: additive exponent term / delta ([bh][S_max] or [bh][Tn_pad]; dx null: 0)
  // EX == 2 only (stationary Taylor queries; the streamed gathered mean keys are stored minus the mean key of block 0):
  // rx [bh][S_max] = q . Kc_0 of every stationary row in raw score units, added to its scores against mean tiles
  const float* rx;
  BwdStream s[2];
  int n_phases;
  // exact sets: bit matrix [bh][T_max][mask_words] whose row is a stationary entry (token blocks) or a stationary mean row,
  // and whose bit index is a streamed list entry / mean position
  const uint32_t* bits; int mask_words;
  // outputs
  uint16_t* out_bf; float* out_f32;           // token rows (bf16, strides of `geo`) or mean rows (fp32 [bh][Tn_pad][128])
  const float* add_rows;                      // token rows: null, or fp32 [bh][T_max][128] by block id: a row's share, divided by the block's
                                              // tokens, is added
  float oscale;
  const int* blk_start; const int* blk_n;
  Geometry geo; Counts cnt;
  int Tn_pad, S_max;
  int items;                                  // work items (pairs of stationary blocks) per (batch, head) in this launch
  // mean rows only: every item runs as `parts` workgroups, each over its share of the streamed entries, and writes its
  // partial sums to out_f32 + part * part_stride (k_bwd_merge adds them up)
  int parts; long long part_stride;
  // token rows: the last tail_items items of every XCD (its last, incomplete round over the compute
  // units) run as tail_parts workgroups each, every one over its share of the streamed entries of each phase; they leave their
  // unscaled fp32 sums in tail_scratch [XCD][tail item][part][256 rows][128] and k_bwd_merge writes the rows
  int items_xcd, tail_items, tail_parts;
  float* tail_scratch;
  // token rows: null, or a counter (0 when the launch starts) from which every workgroup takes the number of its item,
  // numbered over all (batch, head)s: the launch then has more workgroups than items, and an XCD that gets through its
  // workgroups sooner takes more of the items (the XCDs of a chip are not equally fast)
  int* dyn_ctr;
  int dyn_whole, dyn_total;                   // the first dyn_whole of them are whole items, the others tail_parts parts of an item each
};

// SM: stationary rows are block means and the streamed rows are queries, which carry the deltas; otherwise the stationary rows
// are queries.  T2: W = P * (T2 - delta), else (dVc) W = P.  EX: exact-set bits are in play: 1 (SM) stationary rows masked for a
// streamed block; 2 (queries) streamed tiles masked or not for a stationary block, and single positions of a tile of gathered means.
template <bool SM, bool T2, int EX>
__device__ __forceinline__ void attn_bwd(const BwdArgs& a, uint16_t* const lds, const int wg, float* const out_f32, const float oscale) {
  static_assert(SM ? EX == 0 || EX == 1 : T2 && (EX == 0 || EX == 2), "what the launch uses");
  constexpr bool YD = SM && T2;                              // minus-deltas of the streamed rows start T2
  constexpr int STG = EX == 2 ? STAGE + K_TILE : STAGE;      // EX == 2: a third tile per stage (see BwdStream::y3)
  // Workgroup ids go round-robin over the 8 XCDs: XCD x has its range of the items of all (batch, head)s (xcd_first, head_at) and
  // works through it one head after the other, so that the workgroups that run together on an XCD (and share its L2)
  // stream the same rows.
  const int xcd = wg & 7, jj = wg >> 3;
  const int n_bh = a.geo.B * a.geo.H;
  int parts = 1, part = 0, item, bhid, tail_slot = -1;
  if (SM) {
    parts = a.parts;
    const int per_head = a.items * parts;
    const int idx = xcd_first((long long)n_bh * per_head, xcd) + jj;
    if (idx >= xcd_first((long long)n_bh * per_head, xcd + 1)) return;
    const int item_all = idx % per_head;
    bhid = head_at(idx / per_head, n_bh);
    item = item_all / parts;
    part = item_all - item * parts;
  } else {
    if (a.dyn_ctr) {
      __shared__ int taken;
      if (threadIdx.x == 0) taken = atomicAdd(a.dyn_ctr, 1);
      __syncthreads();
      int idx = __builtin_amdgcn_readfirstlane(taken);
      if (idx >= a.dyn_total) return;                     // the launch has more workgroups than items
      if (idx >= a.dyn_whole) {
        tail_slot = (idx - a.dyn_whole) / a.tail_parts;
        part = (idx - a.dyn_whole) % a.tail_parts;
        parts = a.tail_parts;
        idx = a.dyn_whole + tail_slot;
      }
      item = idx % a.items;
      bhid = idx / a.items;
    } else {
      const int n_reg = a.items_xcd - a.tail_items;       // items_xcd = items of an XCD (some have one fewer); no tail: jj itself
      int idx = jj;
      if (jj >= n_reg) {
        const int u = jj - n_reg;
        tail_slot = u / a.tail_parts;
        part = u - tail_slot * a.tail_parts;
        parts = a.tail_parts;
        idx = n_reg + tail_slot;
      }
      idx += xcd_first((long long)n_bh * a.items, xcd);
      if (idx >= xcd_first((long long)n_bh * a.items, xcd + 1)) return;
      item = idx % a.items;
      bhid = head_at(idx / a.items, n_bh);
    }
  }
  const int h = bhid % a.geo.H, b = bhid / a.geo.H;
  const int T_new = a.cnt.b[b].T_new, n_full = a.cnt.b[b].n_full, n_flat = a.cnt.b[b].n_flat;
  const int T_max = a.geo.T_max;
  const long long bh = bhid;
  const int n_stat = SM ? (T_new + 127) / 128 : a.stat_flat ? n_flat : n_full;
  if (2 * item >= n_stat) return;
  const long long tbase = (long long)b * a.geo.stride_b + (long long)h * a.geo.stride_h;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2, wq = wave & 3;
  const int r16 = lane & 15, q = lane >> 4;

  // ---- stationary rows of this wave: 32 rows of block `entry` (the second group idles on block 0 in the last pair of
  // an odd list: computes, stores nothing)
  const int entry = 2 * item + grp;
  const bool active = entry < n_stat;
  const int e_use = active ? entry : 0;
  int n_x, x_start = 0, x_blk = 0;
  const uint16_t *xb1, *xb2;
  long long xstride;
  long long bx_base;
  if (SM) {
    n_x = active ? min(128, T_new - entry * 128) : 0;
    xb1 = a.x1 + (bh * a.Tn_pad + (long long)e_use * 128) * MD;
    xb2 = T2 ? a.x2 + (bh * a.Tn_pad + (long long)e_use * 128) * MD : nullptr;
    xstride = MD;
    bx_base = bh * a.Tn_pad + (long long)e_use * 128;
  } else {
    const int blk = block_in_range(a.stat_list[bh * T_max + e_use], a.cnt.b[b].T);
    x_blk = blk;
    n_x = active ? a.blk_n[b * T_max + blk] : 0;
    x_start = a.blk_start[b * T_max + blk];
    xb1 = a.x1 + tbase + (long long)x_start * a.geo.stride_t;
    xb2 = a.x2 + tbase + (long long)x_start * a.geo.stride_t;
    xstride = a.geo.stride_t;
    bx_base = bh * a.S_max + x_start;
  }
  int rowq[2];
  bool row_ok[2];
  bf16x8 x1f[2][4], x2f[2][4];
  float bxv[2], dxv[2], rxv[2] = {0.f, 0.f};
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    rowq[qt] = wq * 32 + 16 * qt + r16;
    row_ok[qt] = rowq[qt] < n_x;
    const long long ro = (long long)(row_ok[qt] ? rowq[qt] : 0) * xstride + 8 * q;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      x1f[qt][ks] = *reinterpret_cast<const bf16x8*>(xb1 + ro + 32 * ks);
      if (T2) x2f[qt][ks] = *reinterpret_cast<const bf16x8*>(xb2 + ro + 32 * ks);
    }
    bxv[qt] = row_ok[qt] ? a.bx[bx_base + rowq[qt]] : 0.f;
    dxv[qt] = (a.dx && row_ok[qt]) ? a.dx[bx_base + rowq[qt]] : 0.f;
    if (EX == 2) rxv[qt] = (a.rx && row_ok[qt]) ? a.rx[bx_base + rowq[qt]] : 0.f;
  }
  // Exact-set bits of the stationary token blocks: lane L holds word L of the row of this wave's own entry and of the
  // pair's other entry (zeros for an entry that does not exist); handed out with readlane.
  uint32_t bits_own = 0u, bits_other = 0u, bits_own_hi = 0u, bits_other_hi = 0u;     // words L and 64 + L
  if (EX && !SM) {
    const int e_other = 2 * item + (1 - grp);
    if (active && lane < a.mask_words) bits_own = a.bits[(bh * T_max + entry) * a.mask_words + lane];
    if (active && lane + 64 < a.mask_words) bits_own_hi = a.bits[(bh * T_max + entry) * a.mask_words + lane + 64];
    if (e_other < n_stat && lane < a.mask_words) bits_other = a.bits[(bh * T_max + e_other) * a.mask_words + lane];
    if (e_other < n_stat && lane + 64 < a.mask_words) bits_other_hi = a.bits[(bh * T_max + e_other) * a.mask_words + lane + 64];
  }
  const uint32_t bits_any = bits_own | bits_other, bits_any_hi = bits_own_hi | bits_other_hi;
  // word w (0..127) of a bit row held as (lo, hi)
  auto word_of = [&](uint32_t lo, uint32_t hi, int w) __attribute__((always_inline)) -> uint32_t {
    return w < 64 ? (uint32_t)__builtin_amdgcn_readlane((int)lo, w) : (uint32_t)__builtin_amdgcn_readlane((int)hi, min(w - 64, 63));
  };
  // consume the prologue loads here: the waits the compiler places inside the loop must not cover them
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      asm volatile("" : "+v"(x1f[qt][ks]));
      if (T2) asm volatile("" : "+v"(x2f[qt][ks]));
    }
    asm volatile("" : "+v"(bxv[qt]), "+v"(dxv[qt]));
    if (EX == 2) asm volatile("" : "+v"(rxv[qt]));
  }
  if (EX) asm volatile("" : "+v"(bits_own), "+v"(bits_other), "+v"(bits_own_hi), "+v"(bits_other_hi));

  // ---- tile loads: global -> LDS, 16 bytes per lane, rows XOR-swizzled on the source side (the row-major layout of
  // the forward kernel: tiles of 64 rows x 256 B, chunk c of row r at c ^ (r & 15))
  const int l16 = lane >> 4;
  uint32_t nchunk_b[2];
  int nrow_l[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    nrow_l[i] = 8 * wave + 4 * i + l16;
    nchunk_b[i] = (uint32_t)((((lane & 15) ^ (nrow_l[i] & 15)) * 8) * 2);
  }

  // ---- the sequence of streamed tiles: phase p, tile T of the phase (token tiles: entry T / 2, half T % 2).
  // Everything the loop needs to know about the two phases is copied into plain variables here and selected by value:
  // indexing the kernel argument (or a closure) with a run-time phase number would move it to scratch memory.
  struct Cursor { int p, T; };
  const int n_phases = a.n_phases;
  const int ph_ent0 = a.s[0].flat ? n_flat : T_new;
  const int ph_ent1 = a.s[1].flat ? n_flat : T_new;
  const int4* const ph_tab0 = a.s[0].tab;
  const int4* const ph_tab1 = a.s[1].tab;
  // this part's share of each phase: tiles [lo, hi), cut between entries (token tiles) or between tiles of means
  auto share = [&](bool tokens, int entries, int p) __attribute__((always_inline)) -> int {
    const int units = tokens ? entries : (T_new + KT - 1) / KT;
    const int u = parts > 1 ? (int)((long long)p * units / parts) : p * units;
    return tokens ? 2 * u : u;
  };
  const int ph_lo0 = share(ph_tab0 != nullptr, ph_ent0, part), ph_tiles0 = share(ph_tab0 != nullptr, ph_ent0, part + 1);
  const int ph_lo1 = share(ph_tab1 != nullptr, ph_ent1, part), ph_tiles1 = share(ph_tab1 != nullptr, ph_ent1, part + 1);
  const int ph_masked0 = a.s[0].masked, ph_masked1 = a.s[1].masked;
  const uint16_t* const ph_y1_0 = a.s[0].y1; const uint16_t* const ph_y1_1 = a.s[1].y1;
  const uint16_t* const ph_y2_0 = a.s[0].y2; const uint16_t* const ph_y2_1 = a.s[1].y2;
  const uint16_t* const ph_y3_0 = a.s[0].y3; const uint16_t* const ph_y3_1 = a.s[1].y3;
  const float2* const ph_ybd_0 = a.s[0].ybd; const float2* const ph_ybd_1 = a.s[1].ybd;
#define PH(p, x0, x1) ((p) == 0 ? (x0) : (x1))
  auto tiles_of = [&](int p) __attribute__((always_inline)) -> int { return PH(p, ph_tiles0, ph_tiles1); };
  // first entry >= e0 of the phase whose bit is set for either stationary entry of the pair (n_ent if none)
  auto next_linked = [&](int e0, int n_ent) __attribute__((always_inline)) -> int {
    int w = e0 >> 5;
    if (e0 >= n_ent) return n_ent;
    uint32_t word = word_of(bits_any, bits_any_hi, w) & (~0u << (e0 & 31));
    const int nw = (n_ent + 31) >> 5;
    while (word == 0u && ++w < nw) word = word_of(bits_any, bits_any_hi, w);
    if (word == 0u) return n_ent;
    return min(n_ent, w * 32 + __builtin_ctz(word));
  };
  // normalises a cursor: skips unlinked entries of a masked token phase and moves on to the next phase at the end
  auto settle = [&](Cursor c) __attribute__((always_inline)) -> Cursor {
    while (c.p < n_phases) {
      const int nt = tiles_of(c.p);
      if (EX && !SM && PH(c.p, ph_masked0, ph_masked1) == 1 && (c.T & 1) == 0 && c.T < nt) c.T = 2 * next_linked(c.T >> 1, nt >> 1);
      if (c.T < nt) break;
      c.p += 1;
      c.T = ph_lo1;
    }
    return c;
  };
  auto advance = [&](Cursor c) __attribute__((always_inline)) -> Cursor { c.T += 1; return settle(c); };
  // The table row of a tile is fetched one iteration before the tile's loads are issued, so that its latency is not
  // waited for inside the loop.
  auto row_of = [&](Cursor c) __attribute__((always_inline)) -> int4 {
    const int4* const tab = PH(c.p, ph_tab0, ph_tab1);
    if (c.p >= n_phases || !tab) return make_int4(0, 0, 0, 0);
    return tab[bh * T_max + (c.T >> 1)];
  };
  auto issue_tile = [&](Cursor c, int stage, const int4 ent) __attribute__((always_inline)) {
    const bool means = PH(c.p, ph_tab0, ph_tab1) == nullptr;
    const uint16_t* const ph_y1 = PH(c.p, ph_y1_0, ph_y1_1);
    const uint16_t* const ph_y2 = PH(c.p, ph_y2_0, ph_y2_1);
    const float2* const ph_ybd = PH(c.p, ph_ybd_0, ph_ybd_1);
    const int T = c.T;
    uint32_t y_off, bd_off, ystride_b;
    int nk;
    const char *y1_head, *y2_head, *ybd_head;
    if (means) {
      ystride_b = (uint32_t)MD * 2u;
      y1_head = reinterpret_cast<const char*>(ph_y1 + bh * a.Tn_pad * MD);
      y2_head = reinterpret_cast<const char*>(ph_y2 + bh * a.Tn_pad * MD);
      ybd_head = reinterpret_cast<const char*>(ph_ybd + bh * a.Tn_pad);
      y_off = (uint32_t)T * (uint32_t)(KT * MD * 2);
      bd_off = (uint32_t)T * (uint32_t)(KT * 8);
      nk = KT;                                            // the gathered mean arrays are padded to whole tiles
    } else {
      ystride_b = (uint32_t)a.geo.stride_t * 2u;
      y1_head = reinterpret_cast<const char*>(ph_y1 + tbase);
      y2_head = reinterpret_cast<const char*>(ph_y2 + tbase);
      ybd_head = reinterpret_cast<const char*>(ph_ybd + bh * T_max * 128);
      const int sub = T & 1;
      const bool empty = ent.y <= sub * KT;               // second tile of a short block: masked, reads the block's first rows
      y_off = (uint32_t)(ent.x + (empty ? 0 : sub * KT)) * ystride_b;
      bd_off = (uint32_t)((T >> 1) * 128 + sub * KT) * 8u;
      nk = empty ? 1 : min(KT, ent.y - sub * KT);
    }
    // wave-uniform by construction; made scalar explicitly so that the bases of the loads live in scalar registers
    y_off = __builtin_amdgcn_readfirstlane(y_off);
    bd_off = __builtin_amdgcn_readfirstlane(bd_off);
    nk = __builtin_amdgcn_readfirstlane(nk);
    ystride_b = __builtin_amdgcn_readfirstlane(ystride_b);
    const char* const y1_tile = uniform_ptr(y1_head + y_off);
    const char* const y2_tile = uniform_ptr(y2_head + y_off);
    const char* const ybd_tile = uniform_ptr(ybd_head + bd_off);
    uint16_t* sb = lds + stage * STG;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t ro = (uint32_t)min(nrow_l[i], nk - 1) * ystride_b + nchunk_b[i];     // rows past the end re-read the last one
      dma16(y1_tile, ro, lds_addr(sb + (wave * 2 + i) * 512));
      dma16(y2_tile, ro, lds_addr(sb + K_TILE + (wave * 2 + i) * 512));
    }
    if (EX == 2 && means) {                                // the mean keys as they are, for the transposed read
      const char* const y3_tile = uniform_ptr(reinterpret_cast<const char*>(PH(c.p, ph_y3_0, ph_y3_1) + bh * a.Tn_pad * MD) + y_off);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        dma16(y3_tile, (uint32_t)nrow_l[i] * ystride_b + nchunk_b[i], lds_addr(sb + 2 * K_TILE + (wave * 2 + i) * 512));
    }
    if (wave == 0)                                         // {bias, delta} of the 64 rows: 512 B, lanes 32..63 repeat lanes 0..31
      dma16(ybd_tile, (uint32_t)(lane & 31) * 16u, lds_addr(lds + 2 * STG + stage * (SIDE_BYTES / 2)));
  };

  // per-lane fragment offsets (bf16 elements), as in the forward kernel
  int koff[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) koff[ks] = r16 * MD + (((4 * ks + q) ^ r16) * 8);
  // Transposed fragments of the accumulation product (A operand: 16 channels x 32 streamed rows) come straight out of
  // a row-major tile with ds_read_b64_tr_b16: in every group of 16 lanes, lane s points at 4 consecutive channels
  // 16 ct + 4 (s & 3) .. of row 4 q + (s >> 2) of a 16-row sub-tile, and lane l receives, for i = 0..3, channel 16 ct + l
  // of row 4 q + i -- the four rows whose weights the lane group holds in elements 4 kt + i of its W fragment.
  const int tr_row = 4 * q + (r16 >> 2);
  int tr_base[2];                              // sub-tile kt: row offset plus the lane's half of a 16-byte chunk
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) tr_base[kt] = (16 * kt + tr_row) * MD + 4 * (r16 & 1);
  int tr_pos[8];                               // channel tile ct: swizzled position of the lane's chunk in its row
#pragma unroll
  for (int ct = 0; ct < 8; ++ct) tr_pos[ct] = ((2 * ct + ((r16 & 3) >> 1)) ^ (tr_row & 15)) * 8;

  f32x4 acc[8][2];
#pragma unroll
  for (int ct = 0; ct < 8; ++ct)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) acc[ct][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float cscale = 1.4426950408889634f / sqrtf((float)MD);       // log2(e) / sqrt(D)
  f32x4 t1_init[2], t2_init[2];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const float b0 = bxv[qt] / cscale;
    t1_init[qt] = f32x4{b0, b0, b0, b0};
    t2_init[qt] = f32x4{-dxv[qt], -dxv[qt], -dxv[qt], -dxv[qt]};
  }

  // cur: tile being multiplied; nxt: tile whose loads are in flight; nn: tile whose table row is being fetched
  Cursor cur = settle(Cursor{0, ph_lo0});
  Cursor nxt = cur.p < n_phases ? advance(cur) : cur;
  int4 ent_nxt = row_of(cur);
  if (cur.p < n_phases) issue_tile(cur, 0, ent_nxt);
  ent_nxt = row_of(nxt);
  uint32_t sm_word[2] = {0u, 0u};             // masked == 3: word (entry / 32) of the bit rows of the lane's two mean rows
  int sm_word_of = -1;
  for (int it = 0; cur.p < n_phases; ++it) {
    // this wave's loads of the current tile have landed; after the barrier everybody's have, and everybody has finished
    // reading the other stage (the previous tile), which the loads of the next tile now overwrite
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const uint16_t* sb = lds + (it & 1) * STG;
    const float* side = reinterpret_cast<const float*>(lds + 2 * STG + (it & 1) * (SIDE_BYTES / 2));   // 64 terms, 64 minus-deltas
    const bool mean_tile = EX == 2 && PH(cur.p, ph_tab0, ph_tab1) == nullptr;     // wave-uniform
    f32x4 nd[2];                              // YD: minus delta of the streamed rows of the sub-tile whose T steps are next
    auto load_delta = [&](int hh, int kt) {
      if (T2 && YD) nd[kt] = *reinterpret_cast<const f32x4*>(side + 64 + 32 * hh + 16 * kt + 4 * q);
    };
    // LDS fragments are requested PF steps before the MFMAs that read them (a step is 64 or 32 cycles of matrix pipe,
    // an LDS read takes longer than one of them), in PF + 1 rotating register sets
    constexpr int PF = EX == 2 ? 1 : 2, NB = PF + 1;        // (EX == 2: one step ahead, its registers are all spoken for)
    bf16x8 fa[NB], fb[NB];                    // Y1 / Y2 fragments of T steps n .. n + PF
    bf16x8 fc[NB];                            // Yt fragments of C steps
    auto t_load = [&](int n) {                // fragments of T step n (sub-tile n / 4, k-slice n % 4)
      const int s2 = n >> 2, ks2 = n & 3;
      const uint16_t* rowp = sb + (32 * (s2 >> 1) + 16 * (s2 & 1)) * MD + koff[ks2];
      fa[n % NB] = *reinterpret_cast<const bf16x8*>(rowp);
      if (T2) fb[n % NB] = *reinterpret_cast<const bf16x8*>(rowp + K_TILE);
    };
    auto c_load = [&](int n) {                // fragment of C step n (half n / 8, channel tile n % 8)
      // the tile whose transpose is Yt
      const uint16_t* src = sb + (T2 ? ((EX == 2 && mean_tile) ? 2 * K_TILE : 0) : K_TILE) + (n >> 3) * 32 * MD + tr_pos[n & 7];
      const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(src + tr_base[0]));
      const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(src + tr_base[1]));
      fc[n % NB] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
#pragma unroll
    for (int n = 0; n < PF; ++n) t_load(n);
    load_delta(0, 0);
    // the first fragments are on their way from LDS while the next tile's loads are set up and issued
    if (nxt.p < n_phases) issue_tile(nxt, (it + 1) & 1, ent_nxt);
    const Cursor nn = nxt.p < n_phases ? advance(nxt) : nxt;
    ent_nxt = row_of(nn);
    // exact sets: what of this tile is masked for this wave's stationary rows
    float gm_tile[2] = {0.f, 0.f};            // per stationary 16-row tile of the wave
    uint32_t pos_w0 = 0u, pos_w1 = 0u;        // masked == 2: bits of the tile's 64 positions (set = masked)
    bool dead = false;                        // the whole tile is masked for all stationary rows of this wave
    if (EX) {
      const int masked = PH(cur.p, ph_masked0, ph_masked1);
      if (!SM && masked == 1) {
        const int e = cur.T >> 1;
        const bool linked = (word_of(bits_own, bits_own_hi, e >> 5) >> (e & 31)) & 1u;
        gm_tile[0] = gm_tile[1] = linked ? 0.f : -INFINITY;
        dead = !linked;                       // streamed for the other block of the pair only: every weight would be 0
      } else if (EX == 2 && !SM && masked == 2) {
        pos_w0 = word_of(bits_own, bits_own_hi, 2 * cur.T);
        pos_w1 = word_of(bits_own, bits_own_hi, 2 * cur.T + 1);
      } else if (SM && masked == 3) {
        const int e = cur.T >> 1;
        if ((e >> 5) != sm_word_of) {
          sm_word_of = e >> 5;
#pragma unroll
          for (int qt = 0; qt < 2; ++qt)
            sm_word[qt] = row_ok[qt] ? a.bits[(bh * T_max + entry * 128 + rowq[qt]) * a.mask_words + sm_word_of] : 0u;
        }
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) gm_tile[qt] = ((sm_word[qt] >> (e & 31)) & 1u) ? -INFINITY : 0.f;
      }
    }
    // One tile = two halves (hh) of 32 streamed rows, each of two 16-row sub-tiles (kt).  Per sub-tile: the T products
    // (4 steps of 4 MFMAs, 2 without T2) and then 8 weights per lane on the vector ALU (exp2 runs at half the
    // vector rate, so a sub-tile's weights cost about as much as its MFMAs); per half: the C product (8 steps of 2 MFMAs)
    // once all 16 weights exist.  Back to back these would take turns on the two pipes; instead the weights of a
    // sub-tile are issued in slices between the MFMAs of the next sub-tile's T steps, and those of the last sub-tile
    // between the MFMAs of the first half's C steps:
    //   T(0,0) | T(0,1) + W(0,0) | T(1,0) + W(0,1) | T(1,1) + W(1,0) | C(0) + W(1,1) | C(1)
    if (!(EX && dead)) {                      // wave-uniform
    f32x4 t1[2][2], t2[2][2];                 // [kt][qt]
    bf16x8 w[2][2];                           // [hh][qt]; element 4 kt + i = streamed row 32 hh + 16 kt + 4 q + i
    f32x4 c1[2];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
      c1[qt] = EX ? t1_init[qt] + f32x4{gm_tile[qt], gm_tile[qt], gm_tile[qt], gm_tile[qt]} : t1_init[qt];
    if (EX == 2 && mean_tile) {               // the gathered mean keys are stored minus Kc_0: q . Kc_0 goes back onto the scores
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) c1[qt] += f32x4{rxv[qt], rxv[qt], rxv[qt], rxv[qt]};
    }
    f32x4 bt[2];                              // exponent terms of the sub-tile whose weights are in progress, [kt]
    auto load_side = [&](int hh, int kt) {
      const uint32_t pos_w = hh ? pos_w1 : pos_w0;
      bt[kt] = *reinterpret_cast<const f32x4*>(side + 32 * hh + 16 * kt + 4 * q);
      if (EX == 2) {                          // only the launch that streams gathered means under exact sets has such bits
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if ((pos_w >> (16 * kt + 4 * q + i)) & 1u) bt[kt][i] = -INFINITY;
      }
    };
    auto weight2 = [&](int hh, int kt, int tp) {          // weights 2 tp and 2 tp + 1 of sub-tile (hh, kt): tile qt = tp / 2
      const int qt = tp >> 1, i0 = (2 * tp) & 3;
      float val[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float pw = __builtin_amdgcn_exp2f(fmaf(t1[kt][qt][i0 + j], cscale, bt[kt][i0 + j]));
        val[j] = T2 ? pw * t2[kt][qt][i0 + j] : pw;       // T2 started at minus the deltas: it already is dP - delta
      }
      w[hh][qt][4 * kt + i0] = (__bf16)val[0];
      w[hh][qt][4 * kt + i0 + 1] = (__bf16)val[1];
    };
#pragma unroll
    for (int s = 0; s < 4; ++s) {             // sub-tile (hh, kt) = (s / 2, s % 2)
      const int kt = s & 1;
      if (s > 0) load_side((s - 1) >> 1, (s - 1) & 1);
      if (s < 3) load_delta((s + 1) >> 1, (s + 1) & 1);   // read by the first MFMAs of the next sub-tile
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int n = 4 * s + ks, cb = n % NB;
        ISA_BWD_FENCE();
        if (n + PF < 16) t_load(n + PF);
        else c_load(n + PF - 16);
        t1[kt][0] = mfma16(fa[cb], x1f[0][ks], ks == 0 ? c1[0] : t1[kt][0]);
        t1[kt][1] = mfma16(fa[cb], x1f[1][ks], ks == 0 ? c1[1] : t1[kt][1]);
        if (T2) {
          t2[kt][0] = mfma16(fb[cb], x2f[0][ks], ks == 0 ? (YD ? nd[kt] : t2_init[0]) : t2[kt][0]);
          t2[kt][1] = mfma16(fb[cb], x2f[1][ks], ks == 0 ? (YD ? nd[kt] : t2_init[1]) : t2[kt][1]);
        }
        if (s > 0) weight2((s - 1) >> 1, (s - 1) & 1, ks);
      }
    }
    load_side(1, 1);
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) {
        const int n = 8 * hh + ct, cb = n % NB;
        ISA_BWD_FENCE();
        if (n + PF < 16) c_load(n + PF);
        acc[ct][0] = mfma16(fc[cb], w[hh][0], acc[ct][0]);
        acc[ct][1] = mfma16(fc[cb], w[hh][1], acc[ct][1]);
        if (hh == 0 && (ct & 1)) weight2(1, 1, ct >> 1);
      }
    }
    ISA_BWD_FENCE();
    cur = nxt;
    nxt = nn;
  }

#undef PH
  if (!SM && tail_slot >= 0) {                // a part of a tail item: unscaled sums to scratch, the merge kernel does the rest
    float* dst = a.tail_scratch + (((long long)((a.dyn_ctr ? 0 : xcd * a.tail_items) + tail_slot) * parts + part) * 256 + grp * 128) * MD;
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
      for (int ct = 0; ct < 8; ++ct)
        *reinterpret_cast<f32x4*>(dst + rowq[qt] * MD + 16 * ct + 4 * q) = acc[ct][qt];
    return;
  }
  // ---- store: element i of acc[ct][qt] is channel 16 ct + 4 q + i of stationary row 16 qt + r
  const float inv_n = n_x > 0 ? 1.0f / (float)n_x : 0.f;
  const float* addp = SM || !a.add_rows ? nullptr : a.add_rows + (bh * T_max + x_blk) * MD + 4 * q;
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    if (!row_ok[qt]) continue;
    const int row = rowq[qt];
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
      float4 r = make_float4(acc[ct][qt][0] * oscale, acc[ct][qt][1] * oscale, acc[ct][qt][2] * oscale,
                             acc[ct][qt][3] * oscale);
      if (addp) {
        const float4 m4 = *reinterpret_cast<const float4*>(addp + 16 * ct);
        r.x = fmaf(m4.x, inv_n, r.x); r.y = fmaf(m4.y, inv_n, r.y);
        r.z = fmaf(m4.z, inv_n, r.z); r.w = fmaf(m4.w, inv_n, r.w);
      }
      if (SM) {
        *reinterpret_cast<float4*>(out_f32 + part * a.part_stride + (bh * a.Tn_pad + (long long)entry * 128 + row) * MD + 16 * ct + 4 * q) = r;
      } else {
        bf16x2 lo = {(__bf16)r.x, (__bf16)r.y};
        bf16x2 hi = {(__bf16)r.z, (__bf16)r.w};
        uint2 o;
        o.x = *reinterpret_cast<uint32_t*>(&lo);
        o.y = *reinterpret_cast<uint32_t*>(&hi);
        *reinterpret_cast<uint2*>(a.out_bf + tbase + (long long)(x_start + row) * a.geo.stride_t + 16 * ct + 4 * q) = o;
      }
    }
  }
}

// dQ of both branches and the mean-row launch (dKc, then dVc) in one launch: workgroups 0 .. wgs_full - 1 take the exact branch's items (the
// longest), then come wgs_means for each of dKc and dVc, then the Taylor branch's; all three counts are multiples of the XCDs.
// None reads what another writes, and each alone leaves compute units idle at its end (all of the time, if it is small).  Measured, three
// launches / one, a training step of 12 heads of 1564 tokens 211 / 190 us (78 / 33 of them in these launches and their merges); steps of 15 600
// and 65 520 tokens gain less than 1 %, no more than runs and boxes differ.
struct BwdTokensArgs { BwdArgs full, flat, means; float* dvc; int wgs_full, wgs_flat, wgs_means; };
template <int EX>
__global__ __launch_bounds__(512, 1) void k_attn_bwd(BwdTokensArgs p) {
  __shared__ __attribute__((aligned(1024))) uint16_t lds[2 * (EX ? STAGE + K_TILE : STAGE) + 2 * SIDE_BYTES / 2];
  int wg = blockIdx.x;
  if (wg < p.wgs_full) {
    attn_bwd<false, true, 0>(p.full, lds, wg, nullptr, p.full.oscale);
  } else if ((wg -= p.wgs_full) < p.wgs_means) {
    attn_bwd<true, true, EX>(p.means, lds, wg, p.means.out_f32, p.means.oscale);
  } else if ((wg -= p.wgs_means) < p.wgs_means) {
    attn_bwd<true, false, EX>(p.means, lds, wg, p.dvc, 1.0f);
  } else {
    attn_bwd<false, true, EX ? 2 : 0>(p.flat, lds, wg - p.wgs_means, nullptr, p.flat.oscale);
  }
}

// What the launches need before they start, in one launch of 256 threads a workgroup, blockIdx = {block or list entry, head, task * B + batch
// item}: the arrays over the padded means are a thread's work each.  (As a workgroup's each they had 128 workgroups and more per head start
// beside the one of a single block: training steps of 100 heads of 128 tokens 103 / 68 us, 8 x 40 heads of 500 + 100 tokens 666 / 437.)  Tasks: the lists of
// the kept, the full-attention and the Taylor blocks (bwd_rows), with exact sets the transposed bits (bwd_tmask): none reads what another
// writes, and none writes a gradient: `out` is read here for the last time, and its buffer may be that of one of them.  Delta belongs to the blocks' rows and is worked out where their terms are: as a launch of its own it
// was one more wait and another 4 us of the host's time (a training step of 12 heads of 1564 tokens 183 / 177 us, two runs where the host
// bounds it; 65 520 tokens at the paper's ratios equal).
struct PrepArgs {
  int B, H, Tn_pad, S_max;
  const int* list[3]; int4* tab[3]; float2* ybd[3];          // kept, full-attention, Taylor blocks
  const float* rq; float2* ybd_flatm;                        // exact sets: the Taylor rows' terms a second time (null: none)
  const int4* btab; const float* nlse; float rq_scale;
  const uint16_t *o, *olo, *d_o;                             // o null: delta is there already (k_bwd_delta_residual)
  float* delta; int* ctr;
  float2* ybd_mean; float* bx_mean;
  const uint32_t* mask; uint32_t* mask_t;
  Geometry geo; Counts cnt;
};

// Per list entry: the table row of its block and the {exponent term, minus delta} pair of each of its 128 row positions
// (masked positions: -inf, 0), stored per tile of 64 positions as 64 terms followed by 64 minus-deltas.  kind 0: kept blocks as streamed
// keys (term 0), plus the per-mean arrays of the Taylor branch (log2 n_j per gathered mean, -inf for the padding); kinds 1, 2:
// full-attention / Taylor blocks as streamed queries (term = minus the row's log-sum-exp in the log2 domain, delta of the row); for scores
// against the gathered means under exact sets, which are stored minus Kc_0, the Taylor rows a second time with their q . Kc_0, scaled
// to the log2 domain, added to the term.
// delta = sum_d dO * O (fp32); 16 lanes per token row, 16 bytes per lane and tensor.  O is taken as out + olo: the bf16 output plus
// what its rounding cut off, which the forward kernels keep for this purpose.  With the bf16 output alone, delta carries that rounding
// (2^-9 |dO||O|) into dS = P (dP - delta), which for a query that attends almost one-hot is a difference of nearly equal numbers.
__device__ __forceinline__ void bwd_rows(const PrepArgs& p, int kind, int b) {
  __shared__ float dl[128];
  const int e = blockIdx.x, h = blockIdx.y;
  const Counts& cnt = p.cnt;
  const int* const list = p.list[kind];
  const int T_max = cnt.T_max;
  const long long bh = (long long)b * p.H + h;
  const int n_list = kind == 0 ? cnt.b[b].T_new : kind == 1 ? cnt.b[b].n_full : cnt.b[b].n_flat;
  if (kind == 0)
    for (int t = e * 256 + threadIdx.x; t < p.Tn_pad; t += T_max * 256) {
      float l2 = -INFINITY;
      if (t < n_list) l2 = log2f((float)p.btab[b * T_max + block_in_range(list[bh * T_max + t], cnt.b[b].T)].y);
      const long long m = bh * p.Tn_pad + t;                  // planar per 64 positions: 64 terms, then 64 deltas
      float* ym = reinterpret_cast<float*>(p.ybd_mean);
      ym[(m >> 6) * 128 + (m & 63)] = l2;
      ym[(m >> 6) * 128 + 64 + (m & 63)] = 0.f;
      p.bx_mean[m] = t < n_list ? l2 : 0.f;
    }
  if (e >= n_list) return;
  const int4 ent = p.btab[b * T_max + block_in_range(list[bh * T_max + e], cnt.b[b].T)];
  if (threadIdx.x == 0) p.tab[kind][bh * T_max + e] = ent;
  if (kind > 0 && p.o) {
    const int c16 = threadIdx.x & 15, rg = threadIdx.x >> 4;
    const long long base = (long long)b * p.geo.stride_b + (long long)h * p.geo.stride_h + (long long)ent.x * p.geo.stride_t + 8 * c16;
    uint4 uo[8], ud[8], ul[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = rg + 16 * i;
      uo[i] = ud[i] = ul[i] = make_uint4(0u, 0u, 0u, 0u);
      if (r < ent.y) {
        uo[i] = *reinterpret_cast<const uint4*>(p.o + base + (long long)r * p.geo.stride_t);
        ud[i] = *reinterpret_cast<const uint4*>(p.d_o + base + (long long)r * p.geo.stride_t);
        if (p.olo) ul[i] = *reinterpret_cast<const uint4*>(p.olo + (bh * p.S_max + ent.x + r) * MD + 8 * c16);
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = rg + 16 * i;
      const uint32_t wo[4] = {uo[i].x, uo[i].y, uo[i].z, uo[i].w}, wd[4] = {ud[i].x, ud[i].y, ud[i].z, ud[i].w},
                     wl[4] = {ul[i].x, ul[i].y, ul[i].z, ul[i].w};
      float s = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        s += (__uint_as_float(wo[k] << 16) + __uint_as_float(wl[k] << 16)) * __uint_as_float(wd[k] << 16) +
             (__uint_as_float(wo[k] & 0xffff0000u) + __uint_as_float(wl[k] & 0xffff0000u)) * __uint_as_float(wd[k] & 0xffff0000u);
#pragma unroll
      for (int m = 8; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
      if (c16 == 0) {
        dl[r] = s;
        if (r < ent.y) p.delta[bh * p.S_max + ent.x + r] = s;
      }
    }
    __syncthreads();
  }
  const int r = threadIdx.x;
  if (r >= 128) return;
  float2 v = make_float2(-INFINITY, 0.f);
  float vm = -INFINITY;
  if (r < ent.y) {
    if (kind == 0) {
      v.x = 0.f;
    } else {
      const long long row = bh * p.S_max + ent.x + r;
      v = make_float2(p.nlse[row], -(p.o ? dl[r] : p.delta[row]));
      if (kind == 2 && p.rq) vm = v.x + p.rq_scale * p.rq[row];
    }
  }
  const long long pos = (bh * T_max + e) * 128 + r, at = (pos >> 6) * 128 + (pos & 63);
  float* yf = reinterpret_cast<float*>(p.ybd[kind]);
  yf[at] = v.x;
  yf[at + 64] = v.y;
  if (kind == 2 && p.rq) {
    yf = reinterpret_cast<float*>(p.ybd_flatm);
    yf[at] = vm;
    yf[at + 64] = v.y;
  }
}

// Rows of dK and dV that no later launch writes (keys and values of blocks that were not kept): zero, or, with the
// coarse residual, the block's share `rows[block] / n` of the gradient of its mean.  The launches over the kept blocks write
// theirs, so those are left alone (480p at the paper's ratios, half the blocks kept: 220 us for all rows of both -> 79).
struct Fill { uint16_t *dk, *dv; const float *rows_k, *rows_v; const int* kv_list; const int4* btab; };
__device__ __forceinline__ void bwd_fill(const Fill& f, int wg, const Geometry& g, const Counts& cnt) {
  const int blk = wg % cnt.T_max, h = wg / cnt.T_max % g.H, b = wg / cnt.T_max / g.H;
  const int T = cnt.b[b].T, T_new = cnt.b[b].T_new;
  if (blk >= T) return;
  const long long bh = (long long)b * g.H + h;
  int kept = 0;
  for (int t = threadIdx.x; t < T_new; t += 256) kept |= block_in_range(f.kv_list[bh * cnt.T_max + t], T) == blk ? 1 : 0;
  if (__syncthreads_or(kept)) return;
  const int4 ent = f.btab[b * cnt.T_max + blk];
  const int c16 = threadIdx.x & 15;
  const float inv = 1.0f / (float)ent.y;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const float* rows = t ? f.rows_v : f.rows_k;
    uint4 val = make_uint4(0, 0, 0, 0);
    if (rows) {
      const float* rp = rows + (bh * cnt.T_max + blk) * MD + 8 * c16;
      uint32_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = f2bf(rp[2 * i] * inv) | ((uint32_t)f2bf(rp[2 * i + 1] * inv) << 16);
      val = make_uint4(w[0], w[1], w[2], w[3]);
    }
    uint16_t* x = (t ? f.dv : f.dk) + (long long)b * g.stride_b + (long long)h * g.stride_h + (long long)ent.x * g.stride_t + 8 * c16;
    for (int r = threadIdx.x >> 4; r < ent.y; r += 16) *reinterpret_cast<uint4*>(x + (long long)r * g.stride_t) = val;
  }
}

// Transposed exact-set bits: bit r of word r / 32 of row t is bit t of row r of `mask` (r: position in the Taylor list,
// t: position in the kept list), so that a kept block finds the Taylor blocks that attend to its tokens.
__device__ __forceinline__ void bwd_tmask(const uint32_t* __restrict__ mask, uint32_t* __restrict__ mask_t, int b, const Counts& cnt, int H) {
  const int t = blockIdx.x, h = blockIdx.y, w = threadIdx.x;
  const int T_max = cnt.T_max, mw = cnt.mask_words;
  if (w >= mw || t >= T_max) return;
  const long long bh = (long long)b * H + h;
  uint32_t out = 0u;
  if (t < cnt.b[b].T_new)
    for (int i = 0; i < 32; ++i) {
      const int r = 32 * w + i;
      if (r < cnt.b[b].n_flat) out |= ((mask[(bh * T_max + r) * mw + (t >> 5)] >> (t & 31)) & 1u) << i;
    }
  mask_t[(bh * T_max + t) * mw + w] = out;
}

__global__ __launch_bounds__(256) void k_bwd_prepare(PrepArgs p) {
  const int task = blockIdx.z / p.B, b = blockIdx.z % p.B;
  // the item counters of the launches that follow start at zero (ordinary stores: the call can be captured in a graph)
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x < 8) p.ctr[threadIdx.x] = 0;
  if (task < 3) bwd_rows(p, task, b);
  else bwd_tmask(p.mask, p.mask_t, b, p.cnt, p.H);
}

// ---- coarse residual (Alg. 1 Stage 1 and Stage 5): out += gamma * O_coarse[block], O_coarse = softmax(Qc Kc^T / sqrt D) Vc.
// Its gradient: dOc[i] = gamma * (sum of dO over block i); dVc = S^T dOc; dS = dOc Vc^T; dZ = S * (dS - rowsum(dS * S));
// dQc = dZ Kc / sqrt D; dKc = dZ^T Qc / sqrt D; each mean's gradient is spread evenly over its block's tokens.

// One workgroup per (block, head): delta without the residual's share (the attention branches' delta
// is rowsum(dO * (out - gamma * O_coarse[block]))), and doc[block] = gamma * column sums of the block's dO rows, from one
// read of dO.  HBM-bound: 40 heads of 15 600 tokens 97 + 60 us in two kernels -> 114.
__global__ __launch_bounds__(256) void k_bwd_delta_residual(const uint16_t* __restrict__ o, const uint16_t* __restrict__ olo,
                                                            const uint16_t* __restrict__ d_o, const float* __restrict__ ocoarse,
                                                            float gamma, float* __restrict__ delta, float* __restrict__ doc,
                                                            const int4* __restrict__ btab, Geometry g,
                                                            Counts cnt, int S_max) {
  __shared__ float red[16][MD];
  const int blk = blockIdx.x, h = blockIdx.y, b = blockIdx.z, c16 = threadIdx.x & 15, rg = threadIdx.x >> 4;
  if (blk >= cnt.b[b].T) return;
  const int4 ent = btab[b * cnt.T_max + blk];
  const long long bh = (long long)b * g.H + h;
  const long long base = (long long)b * g.stride_b + (long long)h * g.stride_h + (long long)ent.x * g.stride_t + 8 * c16;
  const float* op = ocoarse + (bh * cnt.T_max + blk) * MD + 8 * c16;
  const float4 oc0 = *reinterpret_cast<const float4*>(op), oc1 = *reinterpret_cast<const float4*>(op + 4);
  const float oc[8] = {oc0.x, oc0.y, oc0.z, oc0.w, oc1.x, oc1.y, oc1.z, oc1.w};
  uint4 uo[8], ud[8], ul[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = rg + 16 * i;
    uo[i] = ud[i] = ul[i] = make_uint4(0u, 0u, 0u, 0u);
    if (r < ent.y) {
      uo[i] = *reinterpret_cast<const uint4*>(o + base + (long long)r * g.stride_t);
      ud[i] = *reinterpret_cast<const uint4*>(d_o + base + (long long)r * g.stride_t);
      if (olo) ul[i] = *reinterpret_cast<const uint4*>(olo + (bh * S_max + ent.x + r) * MD + 8 * c16);
    }
  }
  float col[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = rg + 16 * i;
    const uint32_t wo[4] = {uo[i].x, uo[i].y, uo[i].z, uo[i].w}, wd[4] = {ud[i].x, ud[i].y, ud[i].z, ud[i].w},
                   wl[4] = {ul[i].x, ul[i].y, ul[i].z, ul[i].w};
    float s = 0.f, dot = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float d0 = __uint_as_float(wd[e] << 16), d1 = __uint_as_float(wd[e] & 0xffff0000u);
      s += (__uint_as_float(wo[e] << 16) + __uint_as_float(wl[e] << 16)) * d0 +
           (__uint_as_float(wo[e] & 0xffff0000u) + __uint_as_float(wl[e] & 0xffff0000u)) * d1;
      dot = fmaf(d1, oc[2 * e + 1], fmaf(d0, oc[2 * e], dot));
      col[2 * e] += d0;
      col[2 * e + 1] += d1;
    }
#pragma unroll
    for (int m = 8; m >= 1; m >>= 1) {
      s += __shfl_xor(s, m, 64);
      dot += __shfl_xor(dot, m, 64);
    }
    if (r < ent.y && c16 == 0) delta[bh * S_max + ent.x + r] = fmaf(-gamma, dot, s);
  }
#pragma unroll
  for (int e = 0; e < 8; e += 4) *reinterpret_cast<float4*>(&red[rg][8 * c16 + e]) = make_float4(col[e], col[e + 1], col[e + 2], col[e + 3]);
  __syncthreads();
  if (threadIdx.x < MD) {
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) sum += red[r][threadIdx.x];
    doc[(bh * cnt.T_max + blk) * MD + threadIdx.x] = gamma * sum;
  }
}

// ROWS rows of the pooled map (COLS: ROWS columns): with x the rows' own means and y the other side's,
//     Z = x1 . y1 / sqrt D and dS = x2 . y2 of all pairs, then
//   rows    (x = Qc, dOc; y = Kc, Vc): softmax statistics {max, sum, rowsum(dS * S)} of every row, out1 = dQc = dZ Kc / sqrt D;
//   columns (x = Kc, Vc; y = Qc, dOc): S and dZ from the rows' statistics, out1 = dKc = dZ^T Qc / sqrt D, out2 = dVc = S^T dOc.
// All products on fp32 matrix instructions (v_mfma_f32_16x16x4_f32, operands as in k_coarse): one thread per pair, each
// walking its own row of 512 bytes, took 137 + 111 us for 40 heads of 122 blocks; this takes 22 + 23.  Both T-wide arrays of the
// workgroup's rows sit in LDS: 16 rows up to 1088 blocks, 4 above.
template <int ROWS, bool COLS>
__global__ __launch_bounds__(256) void k_bwd_coarse(const float* __restrict__ x1, const float* __restrict__ x2,
                                                    const float* __restrict__ y1, const float* __restrict__ y2,
                                                    float4* __restrict__ stats, float* __restrict__ out1, float* __restrict__ out2,
                                                    Counts cnt, int n_bh, int H, int stride, int row_tiles) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  float* const zs = sm;                                 // [ROWS][stride]: Z, in the end S
  float* const ds = sm + ROWS * stride;                 // [ROWS][stride]: dS, in the end dZ
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;             // an XCD works through one head after the other (see k_coarse)
  const int bhid = (slot / row_tiles) * 8 + xcd;
  if (bhid >= n_bh) return;
  const int T = cnt.b[bhid / H].T, i0 = (slot % row_tiles) * ROWS;
  if (i0 >= T) return;
  const long long row0 = (long long)bhid * cnt.T_max;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
  const float scale = 1.0f / sqrtf((float)MD);
  const int n_ct = (T + 15) / 16;
  {
    float4 bx1[8], bx2[8];
    const long long xr = (row0 + min(i0 + l16, T - 1)) * MD + 4 * g;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      bx1[t] = *reinterpret_cast<const float4*>(x1 + xr + 16 * t);
      bx2[t] = *reinterpret_cast<const float4*>(x2 + xr + 16 * t);
    }
    for (int jt = wave; jt < n_ct; jt += 4) {
      const long long yr = (row0 + min(jt * 16 + l16, T - 1)) * MD + 4 * g;
      float4 a1[8], a2[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        a1[t] = *reinterpret_cast<const float4*>(y1 + yr + 16 * t);
        a2[t] = *reinterpret_cast<const float4*>(y2 + yr + 16 * t);
      }
      f32x4 z = {0.f, 0.f, 0.f, 0.f}, d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        z = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[t].x, bx1[t].x, z, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(a2[t].x, bx2[t].x, d, 0, 0, 0);
        z = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[t].y, bx1[t].y, z, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(a2[t].y, bx2[t].y, d, 0, 0, 0);
        z = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[t].z, bx1[t].z, z, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(a2[t].z, bx2[t].z, d, 0, 0, 0);
        z = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[t].w, bx1[t].w, z, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(a2[t].w, bx2[t].w, d, 0, 0, 0);
      }
      // lane (l16, g) holds y = 16 jt + 4 g .. + 3 of x row l16
      float zv[4], dv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int y = jt * 16 + 4 * g + i;
        zv[i] = z[i] * scale;
        dv[i] = d[i];
        if (COLS) {
          const float4 st = stats[row0 + min(y, T - 1)];
          zv[i] = __expf(zv[i] - st.x) / st.y;
          dv[i] = zv[i] * (dv[i] - st.z);
        }
        if (y >= T) zv[i] = dv[i] = 0.f;
      }
      if (l16 < ROWS) {
        *reinterpret_cast<float4*>(zs + l16 * stride + jt * 16 + 4 * g) = make_float4(zv[0], zv[1], zv[2], zv[3]);
        *reinterpret_cast<float4*>(ds + l16 * stride + jt * 16 + 4 * g) = make_float4(dv[0], dv[1], dv[2], dv[3]);
      }
    }
  }
  __syncthreads();
  if (!COLS) {
    auto all = [](float x, bool take_max) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const float y = __shfl_xor(x, o, 64);
        x = take_max ? fmaxf(x, y) : x + y;
      }
      return x;
    };
    for (int r = wave; r < ROWS; r += 4) {              // one wave per row: nothing to synchronise between the passes
      if (i0 + r >= T) break;
      float* const zr = zs + r * stride;
      float* const dr = ds + r * stride;
      float m = -INFINITY, l = 0.f, rd = 0.f;
      for (int j = lane; j < T; j += 64) m = fmaxf(m, zr[j]);
      m = all(m, true);
      for (int j = lane; j < T; j += 64) l += (zr[j] = __expf(zr[j] - m));
      l = all(l, false);
      for (int j = lane; j < T; j += 64) rd += (zr[j] /= l) * dr[j];
      rd = all(rd, false);
      for (int j = lane; j < T; j += 64) dr[j] = zr[j] * (dr[j] - rd);
      if (lane == 0) stats[row0 + i0 + r] = make_float4(m, l, rd, 0.f);
    }
    __syncthreads();
  }
  // out^T[channel][row] += y^T[channel][j] dZ[row][j]: a wave takes two tiles of 16 channels, 16 j at a time
  f32x4 acc1[2], acc2[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) acc1[u] = acc2[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int lr = l16 < ROWS ? l16 : 0;
  for (int jt = 0; jt < n_ct; ++jt) {
    float a1[4][2], a2[4][2];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const long long yr = (row0 + min(jt * 16 + 4 * k + g, T - 1)) * MD + 32 * wave + l16;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        a1[k][u] = y1[yr + 16 * u];
        if (COLS) a2[k][u] = y2[yr + 16 * u];
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float bd = ds[lr * stride + jt * 16 + 4 * k + g];
      const float bs = COLS ? zs[lr * stride + jt * 16 + 4 * k + g] : 0.f;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        acc1[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[k][u], bd, acc1[u], 0, 0, 0);
        if (COLS) acc2[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a2[k][u], bs, acc2[u], 0, 0, 0);
      }
    }
  }
  if (l16 < ROWS && i0 + l16 < T) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const long long to = (row0 + i0 + l16) * MD + 32 * wave + 16 * u + 4 * g;
      *reinterpret_cast<float4*>(out1 + to) = make_float4(acc1[u][0] * scale, acc1[u][1] * scale, acc1[u][2] * scale, acc1[u][3] * scale);
      if (COLS) *reinterpret_cast<float4*>(out2 + to) = make_float4(acc2[u][0], acc2[u][1], acc2[u][2], acc2[u][3]);
    }
  }
}

template <int ROWS, bool COLS>
static hipError_t launch_bwd_coarse(const Problem& pr, const Workspace& ws, hipStream_t st) {
  const int T_max = pr.cnt.T_max, n_bh = pr.p.B * pr.p.H;
  const int stride = (T_max + 15) / 16 * 16 + 4, row_tiles = (T_max + ROWS - 1) / ROWS;      // + 4 spreads the rows over the banks
  const size_t lds = (size_t)2 * ROWS * stride * sizeof(float);
  if (lds > 64 * 1024) {                                // beyond the default limit of dynamic LDS: ask for it
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bwd_coarse<ROWS, COLS>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_bwd_coarse<ROWS, COLS>), dim3((unsigned)(N_XCD * ((n_bh + N_XCD - 1) / N_XCD) * row_tiles)), dim3(256), lds, st,
                     COLS ? ws.kc : ws.qc, COLS ? ws.vc : ws.doc, COLS ? ws.qc : ws.kc, COLS ? ws.doc : ws.vc, ws.cstats,
                     COLS ? ws.cdk : ws.cdq, COLS ? ws.cdv : (float*)nullptr, pr.cnt, n_bh, pr.p.H, stride, row_tiles);
  return hipGetLastError();
}

// Gradients of the gathered means, dKc and dVc: the partial sums of the `parts` parts of the launch over the mean rows (0: there was
// none) plus, with the coarse residual, its gradient of the same mean (coarse, by block id), into part 0.  Two gathered mean rows per
// workgroup, 128 threads each; workgroups: {row pair} x H x {2 * batch item + which}.
struct MeanSums { float *dkc, *dvc; const float *coarse_k, *coarse_v; const int* kv_list; int parts, rows2; long long part_stride; };
__device__ __forceinline__ void bwd_mean_sums(const MeanSums& m, int wg, const Counts& cnt, int H, int Tn_pad) {
  const int e = wg % m.rows2 * 2 + (threadIdx.x >> 7), d = threadIdx.x & 127;
  wg /= m.rows2;
  const int h = wg % H, b = wg / H >> 1;
  const bool dv = wg / H & 1;
  if (e >= cnt.b[b].T_new) return;
  float* const g = dv ? m.dvc : m.dkc;
  const float* const coarse = dv ? m.coarse_v : m.coarse_k;
  const long long bh = (long long)b * H + h, i = (bh * Tn_pad + e) * MD + d;
  float sum = m.parts > 0 ? g[i] : 0.f;
  for (int p = 1; p < m.parts; ++p) sum += g[p * m.part_stride + i];
  if (coarse) sum += coarse[(bh * cnt.T_max + block_in_range(m.kv_list[bh * cnt.T_max + e], cnt.b[b].T)) * MD + d];
  g[i] = sum;
}

// Adds up the parts of the tail items of a token-row launch and writes their rows: what the attention kernel's own store
// does for whole items.  One workgroup per (XCD, tail item, block of the pair, 8 rows); 32 threads per row, 4 channels each.
__device__ __forceinline__ void bwd_tail_merge(const BwdArgs& a, int wg) {
  const int rows8 = wg & 15, grp = (wg >> 4) & 1;
  const int slot = wg >> 5, n_bh = a.geo.B * a.geo.H;
  int item, bhid;
  if (a.dyn_ctr) {
    item = (a.dyn_whole + slot) % a.items;
    bhid = (a.dyn_whole + slot) / a.items;
  } else {
    const int xcd = slot / a.tail_items;
    const long long n_items = (long long)a.items * n_bh;
    const int idx = xcd_first(n_items, xcd) + a.items_xcd - a.tail_items + slot % a.tail_items;
    if (idx >= xcd_first(n_items, xcd + 1)) return;
    item = idx % a.items;
    bhid = head_at(idx / a.items, n_bh);
  }
  const int h = bhid % a.geo.H, b = bhid / a.geo.H;
  const long long bh = bhid;
  const int T_max = a.geo.T_max;
  const int n_stat = a.stat_flat ? a.cnt.b[b].n_flat : a.cnt.b[b].n_full;
  const int entry = 2 * item + grp;
  if (entry >= n_stat) return;
  const int blk = block_in_range(a.stat_list[bh * T_max + entry], a.cnt.b[b].T);
  const int n_x = a.blk_n[b * T_max + blk], x_start = a.blk_start[b * T_max + blk];
  const int row = rows8 * 8 + (threadIdx.x >> 5), ch = (threadIdx.x & 31) * 4;
  if (row >= n_x) return;
  const float* src = a.tail_scratch + ((long long)slot * a.tail_parts * 256 + grp * 128 + row) * MD + ch;
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int p0 = 0; p0 < a.tail_parts; p0 += 4) {        // four parts' loads in flight
    float4 o[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = *reinterpret_cast<const float4*>(src + (long long)min(p0 + u, a.tail_parts - 1) * 256 * MD);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (p0 + u >= a.tail_parts) break;
      sum.x += o[u].x; sum.y += o[u].y; sum.z += o[u].z; sum.w += o[u].w;
    }
  }
  sum.x *= a.oscale; sum.y *= a.oscale; sum.z *= a.oscale; sum.w *= a.oscale;
  if (a.add_rows) {
    const float inv_n = 1.0f / (float)n_x;
    const float4 m4 = *reinterpret_cast<const float4*>(a.add_rows + (bh * T_max + blk) * MD + ch);
    sum.x = fmaf(m4.x, inv_n, sum.x); sum.y = fmaf(m4.y, inv_n, sum.y);
    sum.z = fmaf(m4.z, inv_n, sum.z); sum.w = fmaf(m4.w, inv_n, sum.w);
  }
  bf16x2 lo = {(__bf16)sum.x, (__bf16)sum.y};
  bf16x2 hi = {(__bf16)sum.z, (__bf16)sum.w};
  uint2 o;
  o.x = *reinterpret_cast<uint32_t*>(&lo);
  o.y = *reinterpret_cast<uint32_t*>(&hi);
  const long long tbase = (long long)b * a.geo.stride_b + (long long)h * a.geo.stride_h;
  *reinterpret_cast<uint2*>(a.out_bf + tbase + (long long)(x_start + row) * a.geo.stride_t + ch) = o;
}

// Both, behind the launch whose parts they add up, and the fill: the first wgs_full workgroups merge the exact branch's cut items, the next
// wgs_flat the Taylor branch's, wgs_sums sum the means' gradients, the rest (a block of a head each) fill the rows of blocks that were not
// kept.
struct BwdMergeArgs { BwdArgs full, flat; MeanSums means; Fill fill; int wgs_full, wgs_flat, wgs_sums; };
__global__ __launch_bounds__(256) void k_bwd_merge(BwdMergeArgs p) {
  int wg = blockIdx.x;
  if (wg < p.wgs_full) bwd_tail_merge(p.full, wg);
  else if ((wg -= p.wgs_full) < p.wgs_flat) bwd_tail_merge(p.flat, wg);
  else if ((wg -= p.wgs_flat) < p.wgs_sums) bwd_mean_sums(p.means, wg, p.full.cnt, p.full.geo.H, p.full.Tn_pad);
  else bwd_fill(p.fill, wg - p.wgs_sums, p.full.geo, p.full.cnt);
}

// Distribution of the dQ items of one branch: sets the fields of `a` that say which items are cut and returns the number of workgroups
// (a multiple of the XCDs).  split_units: into how many parts the streamed side can be cut (list entries or tiles of means); one_round: 0,
// or the parts every item is cut into; n_sub: sub-items that the partial-result area already holds; n_merge: cut items.
static int plan_dq(BwdArgs& a, int B, int H, int split_units, int* dyn_ctr, int min_dyn, int one_round, int& n_sub, int& n_merge) {
  n_merge = 0;
  a.dyn_ctr = nullptr; a.items_xcd = 0; a.tail_items = 0; a.tail_parts = 1; a.dyn_whole = a.dyn_total = 0;
  if (a.items <= 0) { a.items = 0; return 0; }
  const int cus = cus_per_xcd(), room = SPLIT_MAX_SUB - n_sub;
  a.tail_scratch += (long long)n_sub * 256 * MD;
  a.items_xcd = (int)(((long long)a.items * B * H + N_XCD - 1) / N_XCD);
  // items from a counter only where an XCD has min_dyn of them: fewer are cut into parts instead
  a.dyn_ctr = one_round || a.items_xcd < min_dyn ? nullptr : dyn_ctr;
  if (!a.dyn_ctr && split_units > 1) {
    // the last round of an XCD's 32 compute units: if at most half of them would have an item, cut those items
    const int t = one_round ? a.items_xcd : a.items_xcd % cus;
    if (t > 0 && (one_round || t <= cus / 2)) {
      int parts = one_round ? one_round : cus / t > 8 ? 8 : cus / t;
      if (parts > split_units) parts = split_units;
      while (parts > 1 && N_XCD * t * parts > room) --parts;       // the partial-result area holds SPLIT_MAX_SUB sub-items
      if (parts > 1) { a.tail_items = t; a.tail_parts = parts; }
    }
  }
  // A counted launch of 8 rounds or more runs its last 32 items in 8 parts each, so that it ends within an eighth of an item of
  // the ideal.  dQ of the exact branch at 480p with the paper's ratios, 20 rounds, and dK / dV
  // likewise: training step 101.35 -> 100.85 ms, at keep 0.5, full 0.2 52.3 -> 51.9.
  a.dyn_whole = a.items * B * H;
  a.dyn_total = a.dyn_whole;
  n_merge = N_XCD * a.tail_items;
  if (a.dyn_ctr && a.items_xcd >= 8 * cus && split_units >= 16 && room == SPLIT_MAX_SUB) {
    a.tail_parts = 8;
    n_merge = SPLIT_MAX_SUB / a.tail_parts;
    a.dyn_whole -= n_merge;
    a.dyn_total += n_merge * (a.tail_parts - 1);
  }
  n_sub += n_merge * a.tail_parts;
  // dynamic items: an eighth more workgroups than items and one round of the chip, so that the faster XCDs do not run out
  // of workgroups before the items run out
  const long long n_dyn = a.dyn_total;
  const long long dyn_wgs = ((n_dyn + n_dyn / 8) / N_XCD + cus + 1) * N_XCD;
  return (int)(a.dyn_ctr ? dyn_wgs : (a.items_xcd - a.tail_items + a.tail_items * a.tail_parts) * N_XCD);
}

hipError_t launch_attn_bwd(const Problem& pr, const Workspace& ws, const void* q, const void* k, const void* v,
                           const void* out, const void* d_out, const int* kv_list, const int* full_list,
                           const int* flat_list, const uint32_t* exact_mask, void* dq, void* dk, void* dv,
                           hipStream_t st) {
  const float gamma = (float)pr.p.gamma;
  const bool resid = pr.p.gamma != 0.0;               // ws.ocoarse holds O_coarse (recomputed by the caller of this function)
  const int B = pr.p.B, H = pr.p.H, T_max = pr.cnt.T_max;
  int S_max = pr.S_max, sf = 0, sl = 0, sk = 0, min_kept = 1 << 30;
  for (int b = 0; b < B; ++b) {
    const BatchCounts& c = pr.cnt.b[b];
    sf = c.n_full > sf ? c.n_full : sf;
    sl = c.n_flat > sl ? c.n_flat : sl;
    sk = c.T_new > sk ? c.T_new : sk;
    min_kept = c.T_new < min_kept ? c.T_new : min_kept;
  }
  // The forward ran its 4-wave kernel (exact sets, possibly empty ones when exact_frac is too small for the list): token
  // keys and mean keys in one softmax, the mean keys stored minus Kc_0 and q . Kc_0 kept per Taylor row (ws.rq).
  const bool ex = pr.p.exact_frac > 0.0 && sl > 0 && exact_mask != nullptr;
#define ISA_BWD_CHECK()                           \
  do {                                            \
    hipError_t e__ = hipGetLastError();           \
    if (e__ != hipSuccess) return e__;            \
  } while (0)
  // delta, per-list tables and row terms
  if (resid) {
    // delta without the residual's share; gradient of the coarse residual with respect to the block means (all blocks, by
    // block id)
    hipLaunchKernelGGL(k_bwd_delta_residual, dim3(T_max, H, B), dim3(256), 0, st, (const uint16_t*)out, ws.olo, (const uint16_t*)d_out,
                       ws.ocoarse, gamma, ws.delta, ws.doc, ws.btab, pr.geo, pr.cnt, S_max);
    ISA_BWD_CHECK();
    const bool wide = T_max <= 1088;
    hipError_t ec = wide ? launch_bwd_coarse<16, false>(pr, ws, st) : launch_bwd_coarse<4, false>(pr, ws, st);
    if (ec == hipSuccess) ec = wide ? launch_bwd_coarse<16, true>(pr, ws, st) : launch_bwd_coarse<4, true>(pr, ws, st);
    if (ec != hipSuccess) return ec;
  }
  PrepArgs pa = {B, H, pr.Tn_pad, S_max, {kv_list, full_list, flat_list}, {ws.ktab, ws.ftab, ws.ltab}, {ws.ybd_kv, ws.ybd_full, ws.ybd_flat},
                 ex ? ws.rq : nullptr, ws.ybd_flatm, ws.btab, ws.nlse, 1.4426950408889634f / sqrtf((float)MD) /* raw score -> log2 domain */,
                 resid ? nullptr : (const uint16_t*)out, ws.olo, (const uint16_t*)d_out, ws.delta, ws.bwd_ctr, ws.ybd_mean, ws.bx_mean,
                 exact_mask, ws.mask_t, pr.geo, pr.cnt};
  hipLaunchKernelGGL(k_bwd_prepare, dim3(T_max, H, B * (ex ? 4 : 3)), dim3(256), 0, st, pa);
  ISA_BWD_CHECK();

  BwdArgs a;
  a.blk_start = ws.blk_start; a.blk_n = ws.blk_n;
  a.geo = pr.geo; a.cnt = pr.cnt; a.Tn_pad = pr.Tn_pad; a.S_max = S_max;
  a.mask_words = pr.cnt.mask_words;
  a.parts = 1; a.part_stride = 0;
  a.items_xcd = 0; a.tail_items = 0; a.tail_parts = 1; a.tail_scratch = ws.split_o;   // the forward's partial-result area: 256 x 256 x 128 floats
  const float scale = 1.0f / sqrtf((float)MD);
  const uint16_t *Q = (const uint16_t*)q, *K = (const uint16_t*)k, *V = (const uint16_t*)v, *DO = (const uint16_t*)d_out;
  const BwdStream none = {nullptr, nullptr, nullptr, nullptr, nullptr, false, 0};
  hipError_t e;

  // ---- dQ: exact branch over the kept tokens; Taylor branch over the tokens of each block's exact
  // set and the means of the other kept blocks
  BwdMergeArgs mg;
  BwdTokensArgs tk;
  const BwdStream kept_tokens = {K, V, nullptr, ws.ktab, ws.ybd_kv, false, 0};
  const uint16_t* mean_keys = ws.kcn;             // stored minus the mean key of block 0
  const BwdStream kept_means = {mean_keys, ws.vcn, ex ? ws.kcnb : nullptr, nullptr, ws.ybd_mean, false, 0};
  a.x1 = Q; a.x2 = DO; a.bx = ws.nlse; a.dx = ws.delta; a.rx = nullptr;
  a.out_bf = (uint16_t*)dq; a.out_f32 = nullptr; a.oscale = scale;
  a.add_rows = resid ? ws.cdq : nullptr;          // every query block's share of dQc
  a.stat_list = full_list; a.stat_flat = false; a.items = (sf + 1) / 2;
  a.s[0] = kept_tokens; a.s[1] = none; a.n_phases = 1; a.bits = nullptr;
  tk.full = a;
  a.stat_list = flat_list; a.stat_flat = true; a.items = (sl + 1) / 2;
  if (ex) {
    a.s[0] = kept_tokens; a.s[0].masked = 1;
    a.s[1] = kept_means; a.s[1].masked = 2;
    a.n_phases = 2; a.bits = exact_mask;
    a.rx = ws.rq;
  } else {
    a.s[0] = kept_means; a.n_phases = 1;
  }
  tk.flat = a;
  // ---- dKc, dVc: gradients of the gathered means (streamed Q, dO of every Taylor block, minus its exact set)
  // dKc: W = dS, read Q transposed; dVc: W = P, dO transposed.
  const int n_mean_pairs = sl > 0 && sk > 0 ? ((sk + 127) / 128 + 1) / 2 : 0;
  a.x1 = mean_keys; a.x2 = ws.vcn; a.stat_list = nullptr; a.bx = ws.bx_mean; a.dx = nullptr; a.rx = nullptr;
  a.s[0] = {Q, DO, nullptr, ws.ltab, ex ? ws.ybd_flatm : ws.ybd_flat, true, ex ? 3 : 0};      // scored against gathered means
  a.s[1] = none; a.n_phases = 1; a.bits = ws.mask_t;
  a.out_bf = nullptr; a.out_f32 = ws.dkc; a.add_rows = nullptr; a.items = n_mean_pairs;
  a.part_stride = (long long)B * H * pr.Tn_pad * MD;
  a.dyn_ctr = nullptr;
  tk.means = a; tk.dvc = ws.dvc;
  // The mean rows have few items (two per 256 gathered means and head): each is cut into up to BWD_MEAN_PARTS parts along the streamed
  // entries, as many as make their rounds over the compute units shortest.  Where all three kinds of items fit one round, the
  // exact branch's and the means' parts are those with which the launch ends first by a model of it, in streamed blocks (a start counts for
  // one): the longest part, or all of them shared evenly and, past a round, the last of the short Taylor items behind them.
  // (Parts only as far as they fit the round left an exact branch's item almost whole where the Taylor items filled the rest: training steps of
  // 8 heads of 6000 tokens 355 / 272 us, of 6100 394 / 299, 3 heads of 15 600 with the residual 805 / 688, 40 heads of 1024 139 / 125.)
  const int cus = cus_per_xcd();
  int mean_parts = 0, one_round = 0;
  const auto per_xcd = [&](int items) { return (int)(((long long)items * B * H + N_XCD - 1) / N_XCD); };
  const int e_xcd = per_xcd(tk.full.items), l_xcd = per_xcd(tk.flat.items), m_xcd = per_xcd(n_mean_pairs);
  if (n_mean_pairs > 0) {
    double best = 1e30;
    for (int p = 1; p <= BWD_MEAN_PARTS; ++p) {
      const long long chip = (long long)cus * N_XCD, wgs = 2ll * n_mean_pairs * B * H * p;
      const double rounds = (double)((wgs + chip - 1) / chip) / p;
      if (rounds < best - 1e-9) { best = rounds; mean_parts = p; }
    }
  }
  if (e_xcd > 0 && e_xcd + l_xcd + 2 * m_xcd <= cus) {
    int k_exact = 0;
    for (int b = 0; b < B; ++b) k_exact = ex && pr.cnt.b[b].k_exact > k_exact ? pr.cnt.b[b].k_exact : k_exact;
    const double taylor = 1.0 + 0.5 * ((sk + KT - 1) / KT) + 2.0 * k_exact;
    double best = INFINITY;
    for (int pe = 1; pe <= 8 && pe <= min_kept && (pe == 1 || N_XCD * e_xcd * pe <= SPLIT_MAX_SUB); ++pe)
      for (int pm = n_mean_pairs > 0 ? 1 : 0; pm <= (n_mean_pairs > 0 ? BWD_MEAN_PARTS : 0); ++pm) {
        const int n_e = e_xcd * pe, n_m = 2 * per_xcd(n_mean_pairs * pm);
        const double exact = 1.0 + (sk + pe - 1) / pe, mean = pm > 0 ? 1.0 + (sl + pm - 1) / pm : 0.0;
        const double even = (n_e * exact + n_m * mean + l_xcd * taylor) / cus + (n_e + n_m + l_xcd > cus ? taylor : 0.0);
        const double cost = fmax(fmax(exact, mean), fmax(l_xcd > 0 ? taylor : 0.0, even));
        if (cost < best - 0.01) { best = cost; one_round = pe; mean_parts = pm; }
      }
  }
  tk.means.parts = mean_parts > 0 ? mean_parts : 1;
  int n_sub = 0, n_merge_full = 0, n_merge_flat = 0;
  tk.wgs_full = plan_dq(tk.full, B, H, min_kept, ws.bwd_ctr + 2, 8 * cus, one_round, n_sub, n_merge_full);
  // (the surplus workgroups of a counted launch would keep the rest of a single round waiting)
  const int flat_units = one_round ? 1 : (min_kept + KT - 1) / KT, flat_dyn = one_round ? 1 << 30 : min_kept > KT ? cus / 2 + 1 : 0;
  tk.wgs_flat = plan_dq(tk.flat, B, H, flat_units, ws.bwd_ctr + 0, flat_dyn, 0, n_sub, n_merge_flat);
  tk.wgs_means = n_mean_pairs > 0 ? N_XCD * per_xcd(n_mean_pairs * mean_parts) : 0;
  const int wgs = tk.wgs_full + tk.wgs_flat + 2 * tk.wgs_means;
  if (wgs > 0) {
    if (ex) hipLaunchKernelGGL((k_attn_bwd<1>), dim3((unsigned)wgs), dim3(512), 0, st, tk);
    else hipLaunchKernelGGL((k_attn_bwd<0>), dim3((unsigned)wgs), dim3(512), 0, st, tk);
    ISA_BWD_CHECK();
  }
  mg.full = tk.full; mg.flat = tk.flat;
  mg.wgs_full = n_merge_full * 32; mg.wgs_flat = n_merge_flat * 32;
  mg.means = {ws.dkc, ws.dvc, resid ? ws.cdk : nullptr, resid ? ws.cdv : nullptr, kv_list, mean_parts, (sk + 1) / 2, tk.means.part_stride};
  mg.wgs_sums = sk > 0 && (mean_parts > 1 || resid) ? mg.means.rows2 * H * 2 * B : 0;
  mg.fill = {(uint16_t*)dk, (uint16_t*)dv, resid ? ws.cdk : nullptr, resid ? ws.cdv : nullptr, kv_list, ws.btab};
  bool all_kept = true;
  for (int b = 0; b < B; ++b) all_kept = all_kept && pr.cnt.b[b].T_new == pr.cnt.b[b].T;
  const int wgs_fill = all_kept ? 0 : T_max * H * B, wgs_merge = mg.wgs_full + mg.wgs_flat + mg.wgs_sums + wgs_fill;
  if (wgs_merge > 0) {
    hipLaunchKernelGGL(k_bwd_merge, dim3((unsigned)wgs_merge), dim3(256), 0, st, mg);
    ISA_BWD_CHECK();
  }
  // ---- dK, dV of the kept tokens: every full-attention block, the Taylor blocks whose exact set holds the block, and
  // the block's share of its mean's gradient
  if ((e = launch_bwd_kv(pr, ws, q, k, v, d_out, ex, sl > 0 || resid, dk, dv, st)) != hipSuccess) return e;
#undef ISA_BWD_CHECK
  return hipSuccess;
}

}  // namespace isa
