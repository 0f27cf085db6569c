// dK and dV of the backward pass in one launch (bf16, D = 128, block = 128 on gfx950; see attn_bwd.hip for the formulas):
// the scores and dP of a kept key block against the streamed queries are formed once and feed both accumulations, four matrix
// products per query-key pair.
//
// Shape.  A workgroup is one kept block and 4 waves, one per SIMD: a wave keeps its 32 rows of K and V (64 registers) and
// both accumulators (128) beside a tile's state, which takes the 512 registers a wave has when it is alone on its SIMD
// (two waves per SIMD have 256 each: with them dK and dV were two launches of five products).  The streamed tiles, 64 rows of
// Q and dO, come global -> LDS two tiles ahead, in four stages.  An iteration of a wave is 128 MFMAs (2048 cycles of the
// matrix pipe); each of its 64 KB of fragments feeds two of them, so the four waves together read at the LDS's full rate
// meanwhile, and the 32 weights per lane (fma, exp2, two products' roundings) are issued between the MFMAs of the next
// sub-tile.
//
// Measured at 480p with the paper's ratios (40 heads, 288 kept and 256 full-attention blocks each): 56.0 ms in two launches of 8
// waves -> 47.2 in this one, 45.1 with the tile set-up, the barrier and the first fragments of the next tile moved into the
// shadows of matrix instructions.  Matrix pipe busy 52 % of 4000 cycles an iteration at 2.2 GHz; a wave waits 20 % of
// them for LDS or the barrier and 28 % for the pipe.  Every transposed read costs 2 cycles of bank conflicts (the eight rows it takes
// 32 bytes of at a time meet four places of the swizzle): 3.2e9 of 1.04e10 LDS cycles.  Without effect (within 1 %): fragments 5 or 7
// steps ahead instead of 3, vector instructions placed one by one behind every matrix instruction, chunk c of row r at
// c ^ (((r & 7) << 1) | ((r >> 3) & 1)), which frees the transposed reads of conflicts and gives every row read 4 cycles of them.
//
// Layouts as in attn_bwd.hip: with r = lane % 16, q = lane / 16, T1 = Q K^T and T2 = dO V^T - delta of a 16-row sub-tile give lane
// (r, q) streamed rows 4 q + i of key 16 qt + r; the weights P and dS of two sub-tiles are the B operands of dV^T += dO^T P
// and dK^T += Q^T dS, whose A operands are read transposed out of the row-major tiles (ds_read_b64_tr_b16).
#include "attn_mfma.h"

namespace isa {

#define ISA_KV_FENCE() __builtin_amdgcn_sched_barrier(0)

namespace {

constexpr int NST = 4;                                // LDS stages; two tiles are in flight (see the loop)
constexpr int STAGE_B = 2 * K_TILE * 2 + 1024;        // bytes of a stage: the Q and dO tiles, then 64 exponent terms and 64 minus-deltas
constexpr int TILE_LOADS = 9;                         // load instructions of a wave per tile

__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff_bytes, uint32_t lds_addr) {   // lane i -> LDS bytes lds_addr + 16 i
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_addr), "v"(voff_bytes), "s"(sbase) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(size_t)(__attribute__((address_space(3))) const void*)p;
}
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
// acc += a b with the accumulator in accumulation registers.  Written as inline assembly because the compiler gives all matrix
// instructions of a function one kind of destination: with accumulation registers for the scores and dP as well, every
// one of their values is copied there and back (132 moves per tile).  Nothing but these instructions touches the
// accumulators inside the loop, and the next one to touch the same accumulator is 32 matrix instructions away; `settle` keeps the
// first read after the loop behind the last write.
__device__ __forceinline__ void mfma16_acc(bf16x8 a, bf16x8 b, f32x4& acc) {
  asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void settle(f32x4& acc) { asm volatile("s_nop 15" : "+a"(acc)); }

struct KvArgs {
  const uint16_t *q, *k, *v, *d_o;
  const int4* ktab;                          // [bh][T_max] {token offset, tokens, block} of the kept blocks
  const int4* qtab[2];                       // the same of the full-attention blocks / of the Taylor blocks
  const float2* qside[2];                    // per 64 list positions: 64 exponent terms (-inf: masked), 64 minus-deltas
  const uint32_t* bits;                      // [bh][T_max][mask_words] per kept block: the Taylor blocks whose exact set holds it; null: none
  const float *mean_k, *mean_v;              // null, or [bh][Tn_pad][128]: a row's share (divided by the block's tokens) is added
  uint16_t *dk, *dv;
  float scale;
  Geometry geo; Counts cnt;
  int Tn_pad;
  int items;                                 // kept blocks per (batch, head) (largest of the batch)
  // distribution as in k_attn_bwd: a counter, or equal ranges per XCD whose last tail_items run as tail_parts parts each
  int* dyn_ctr;
  int dyn_whole, dyn_total;
  int items_xcd, tail_items, tail_parts;
  float* tail_scratch;                       // [XCD][tail item][part][dK, dV][128][128]
};

__device__ __forceinline__ uint2 bf16x4_of(const float4 r) {
  const bf16x2 lo = {(__bf16)r.x, (__bf16)r.y}, hi = {(__bf16)r.z, (__bf16)r.w};
  return make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
}

}  // namespace

__global__ __launch_bounds__(256, 1) void k_bwd_kv(KvArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NST * STAGE_B];
  __shared__ int taken;
  const int xcd = blockIdx.x & 7, jj = blockIdx.x >> 3;
  const int n_bh = a.geo.B * a.geo.H;
  int parts = 1, part = 0, tail_slot = -1, idx;
  if (a.dyn_ctr) {
    if (threadIdx.x == 0) taken = atomicAdd(a.dyn_ctr, 1);
    __syncthreads();
    idx = __builtin_amdgcn_readfirstlane(taken);
    if (idx >= a.dyn_total) return;                    // the launch has more workgroups than items
    if (idx >= a.dyn_whole) {
      tail_slot = (idx - a.dyn_whole) / a.tail_parts;
      part = (idx - a.dyn_whole) % a.tail_parts;
      parts = a.tail_parts;
      idx = a.dyn_whole + tail_slot;
    }
  } else {
    const int n_reg = a.items_xcd - a.tail_items;
    idx = jj;
    if (jj >= n_reg) {
      const int u = jj - n_reg;
      tail_slot = u / a.tail_parts;
      part = u - tail_slot * a.tail_parts;
      parts = a.tail_parts;
      idx = n_reg + tail_slot;
    }
    idx += xcd_first((long long)n_bh * a.items, xcd);
    if (idx >= xcd_first((long long)n_bh * a.items, xcd + 1)) return;
  }
  const int entry = idx % a.items;
  const int bhid = a.dyn_ctr ? idx / a.items : head_at(idx / a.items, n_bh);
  const int h = bhid % a.geo.H, b = bhid / a.geo.H;
  const BatchCounts c = a.cnt.b[b];
  if (entry >= c.T_new) return;
  const int T_max = a.geo.T_max;
  const long long bh = bhid;
  const long long tbase = (long long)b * a.geo.stride_b + (long long)h * a.geo.stride_h;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, q = lane >> 4;

  // ---- the stationary rows: 32 of the kept block's
  const int4 own = a.ktab[bh * T_max + entry];
  const int x_start = __builtin_amdgcn_readfirstlane(own.x), n_x = __builtin_amdgcn_readfirstlane(own.y);
  bf16x8 kf[2][4], vf[2][4];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int row = wave * 32 + 16 * qt + r16;
    const long long off = tbase + (long long)(x_start + (row < n_x ? row : 0)) * a.geo.stride_t + 8 * q;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      kf[qt][ks] = *reinterpret_cast<const bf16x8*>(a.k + off + 32 * ks);
      vf[qt][ks] = *reinterpret_cast<const bf16x8*>(a.v + off + 32 * ks);
    }
  }
  // consumed here: the waits the compiler places for them must not land inside the loop, where they would cover the tile loads
#pragma unroll
  for (int qt = 0; qt < 2; ++qt)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) asm volatile("" : "+v"(kf[qt][ks]), "+v"(vf[qt][ks]));

  // ---- the sequence of streamed tiles: the full-attention blocks, then the Taylor blocks linked to this block; a part takes
  // its share of both lists.  Lane L holds the table row of list entry cbase + L.
  const uint32_t* const bits = a.bits ? a.bits + (bh * T_max + entry) * a.cnt.mask_words : nullptr;
  auto cut = [&](int n, int p) { return parts > 1 ? (int)((long long)p * n / parts) : p * n; };
  int phase = 0, cbase = cut(c.n_full, part) - 64, hi = cut(c.n_full, part + 1);
  int c_start = 0, c_n = 0;
  unsigned long long todo = 0ull;
  struct Tile { int start, nk, pos; };                  // first row, rows, list position of the first row (entries are 128 apart)
  Tile at = {0, 1, 0};                                  // (an empty sequence loads row 0 and multiplies nothing)
  bool end = false;                                     // `at` was the last one
  int rest = 0;                                         // rows of its block behind the tile described last
  auto next_tile = [&]() __attribute__((always_inline)) {
    if (rest > 0) {
      at.start += KT;
      at.pos += KT;
      at.nk = rest;
      rest = 0;
      return;
    }
    while (todo == 0ull) {
      if (cbase + 64 >= hi) {
        if (phase == 1 || !bits) { end = true; return; }
        phase = 1;
        cbase = cut(c.n_flat, part) - 64;
        hi = cut(c.n_flat, part + 1);
        continue;
      }
      cbase += 64;
      const int t = cbase + lane;
      bool ok = t < hi;
      if (ok && phase == 1) ok = (bits[t >> 5] >> (t & 31)) & 1u;
      const int4 row = (phase == 0 ? a.qtab[0] : a.qtab[1])[bh * T_max + (ok ? t : 0)];
      c_start = row.x;
      c_n = row.y;
      asm volatile("" : "+v"(c_start), "+v"(c_n));
      todo = __ballot(ok);
    }
    const int l = __builtin_ctzll(todo);
    todo &= todo - 1;
    at.start = __builtin_amdgcn_readlane(c_start, l);
    const int n = __builtin_amdgcn_readlane(c_n, l);
    at.nk = min(KT, n);
    rest = n - KT;
    at.pos = (cbase + l) * 128;
  };
  const uint32_t stride_b = (uint32_t)a.geo.stride_t * 2u;
  const char* const q_head = reinterpret_cast<const char*>(a.q + tbase);
  const char* const o_head = reinterpret_cast<const char*>(a.d_o + tbase);
  const int l16 = lane >> 4;
  // The loads of a tile in four slices: 0 describes the tile and works its addresses out, 1 to 3 issue the loads.  A
  // sequence that has ended loads its last tile again: the number of loads in flight stays the same.
  uint32_t row_off[4];                                  // bytes from the tile's first row: row 16 wave + 4 i + lane / 16, swizzled chunk
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 16 * wave + 4 * i + l16;            // chunk ch of row r sits at ch ^ (r & 15)
    row_off[i] = (uint32_t)row * stride_b + (uint32_t)(((lane & 15) ^ (row & 15)) * 16);
  }
  const char *q_tile = nullptr, *o_tile = nullptr, *side_tile = nullptr;
  uint32_t dst = 0, ro[4];
  int in_stage = 0;                                     // where the next tile goes
  auto issue_slice = [&](int f) __attribute__((always_inline)) {
    if (f == 0) {
      next_tile();
      const uint32_t off = (uint32_t)at.start * stride_b;
      q_tile = uniform_ptr(q_head + off);
      o_tile = uniform_ptr(o_head + off);
      side_tile = uniform_ptr(reinterpret_cast<const char*>((phase == 0 ? a.qside[0] : a.qside[1]) + bh * T_max * 128 + at.pos));
      dst = __builtin_amdgcn_readfirstlane(lds_addr(lds) + (uint32_t)in_stage * STAGE_B);
      in_stage = (in_stage + 1) & (NST - 1);
#pragma unroll
      for (int i = 0; i < 4; ++i) ro[i] = row_off[i];
      if (__builtin_expect(at.nk < KT, 0)) {            // rows past the end repeat the last one
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = 16 * wave + 4 * i + l16;
          ro[i] = (uint32_t)min(row, at.nk - 1) * stride_b + (uint32_t)(((lane & 15) ^ (row & 15)) * 16);
        }
      }
    } else if (f < 3) {
#pragma unroll
      for (int i = 2 * (f - 1); i < 2 * f; ++i) {
        dma16(q_tile, ro[i], dst + (uint32_t)wave * 4096u + i * 1024);
        dma16(o_tile, ro[i], dst + (uint32_t)wave * 4096u + K_TILE * 2 + i * 1024);
      }
    } else {
      // 512 B, lanes 32..63 repeat lanes 0..31; every wave loads them, so that all waves have the same number of loads in flight
      dma16(side_tile, (uint32_t)(lane & 31) * 16u, dst + 4u * K_TILE);
    }
  };

  // per-lane fragment offsets in bytes (attn_bwd.hip has the layouts)
  int koff[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) koff[ks] = (r16 * MD + (((4 * ks + q) ^ r16) * 8)) * 2;
  const int tr_row = 4 * q + (r16 >> 2);
  const int tr_base = (tr_row * MD + 4 * (r16 & 1)) * 2;
  int tr_pos[8];
#pragma unroll
  for (int ct = 0; ct < 8; ++ct) tr_pos[ct] = tr_base + ((2 * ct + ((r16 & 3) >> 1)) ^ (tr_row & 15)) * 16;

  f32x4 ak[8][2], av[8][2];
#pragma unroll
  for (int ct = 0; ct < 8; ++ct)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) ak[ct][qt] = av[ct][qt] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float cscale = 1.4426950408889634f / sqrtf((float)MD);       // log2(e) / sqrt(D)
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};

  constexpr int PF = 3, NB = 4;                         // fragments are requested PF steps ahead, in NB rotating sets
  bf16x8 fa[NB], fb[NB];                                // T steps: Q, dO rows; C steps: Q^T, dO^T
  f32x4 nd[2], bt[2];                                   // minus deltas / exponent terms of the rows of a sub-tile, [kt]
  // steps 0..15 of a tile: T (sub-tile n / 4, k-slice n % 4); 16..31: C (half, channel tile)
  auto load = [&](const unsigned char* sb, int n) __attribute__((always_inline)) {
    if (n < 16) {
      const unsigned char* p = sb + (n >> 2) * 16 * MD * 2 + koff[n & 3];
      fa[n % NB] = *reinterpret_cast<const bf16x8*>(p);
      fb[n % NB] = *reinterpret_cast<const bf16x8*>(p + K_TILE * 2);
    } else {
      const unsigned char* p = sb + ((n - 16) >> 3) * 32 * MD * 2 + tr_pos[n & 7];
      auto tr = [](const unsigned char* x) __attribute__((always_inline)) {
        const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)x);
        const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(x + 16 * MD * 2));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      };
      fa[n % NB] = tr(p);
      fb[n % NB] = tr(p + K_TILE * 2);
    }
  };
  auto load_delta = [&](const unsigned char* sb, int s) __attribute__((always_inline)) {
    nd[s & 1] = *reinterpret_cast<const f32x4*>(sb + 4 * K_TILE + 256 + (16 * s + 4 * q) * 4);
  };
  auto load_term = [&](const unsigned char* sb, int s) __attribute__((always_inline)) {
    bt[s & 1] = *reinterpret_cast<const f32x4*>(sb + 4 * K_TILE + (16 * s + 4 * q) * 4);
  };

  // ---- loop over the tiles; iteration n:
  //   T products of tile n, with the set-up and the loads of tile n + 2 in the shadows of its first four steps (which have no weights
  //   to issue); the first half's C products;
  //   wait for this wave's loads of tile n + 1 (all but the last tile's, loads complete in the order of their issue); barrier:
  //   tile n + 1 is complete for everybody, and everybody is through tile n - 1, whose stage tile n + 3 will fill;
  //   the second half's C products, with the first fragments of tile n + 1 requested in their shadows.
  // A wave is alone on its SIMD: what it waits for, or works out with no matrix instruction in flight, nothing hides.
  int live = 0;                                         // tiles described and not yet multiplied
  auto describe = [&](int f) __attribute__((always_inline)) {
    issue_slice(f);
    if (f == 0) live += end ? 0 : 1;
  };
#pragma unroll
  for (int f = 0; f < 4; ++f) describe(f);
  if (live > 0) {
#pragma unroll
  for (int f = 0; f < 4; ++f) describe(f);
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(TILE_LOADS) : "memory");
  __syncthreads();
#pragma unroll
  for (int n = 0; n < PF; ++n) load(lds, n);
  load_delta(lds, 0);
  for (int stage = 0;;) {
    const unsigned char* const sb = lds + stage * STAGE_B;
    stage = (stage + 1) & (NST - 1);
    const unsigned char* const sb_next = lds + stage * STAGE_B;
    f32x4 t1[2][2], t2[2][2];                           // [kt][qt]
    bf16x8 wp[2][2], ws[2][2];                          // [half][qt]: P and dS; element 4 kt + i = streamed row 32 half + 16 kt + 4 q + i
    auto weight2 = [&](int s, int tp) __attribute__((always_inline)) {      // weights 2 tp, 2 tp + 1 of sub-tile s: key tile tp / 2
      const int hh = s >> 1, kt = s & 1, qt = tp >> 1, i0 = (2 * tp) & 3;
      float p[2], ds[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        p[j] = __builtin_amdgcn_exp2f(fmaf(t1[kt][qt][i0 + j], cscale, bt[kt][i0 + j]));
        ds[j] = p[j] * t2[kt][qt][i0 + j];
      }
      wp[hh][qt][4 * kt + i0] = (__bf16)p[0];
      wp[hh][qt][4 * kt + i0 + 1] = (__bf16)p[1];
      ws[hh][qt][4 * kt + i0] = (__bf16)ds[0];
      ws[hh][qt][4 * kt + i0 + 1] = (__bf16)ds[1];
    };
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int kt = s & 1;
      if (s > 0) load_term(sb, s - 1);
      if (s < 3) load_delta(sb, s + 1);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int n = 4 * s + ks, cb = n % NB;
        ISA_KV_FENCE();
        load(sb, n + PF);
        t1[kt][0] = mfma16(fa[cb], kf[0][ks], ks == 0 ? zero4 : t1[kt][0]);
        t1[kt][1] = mfma16(fa[cb], kf[1][ks], ks == 0 ? zero4 : t1[kt][1]);
        t2[kt][0] = mfma16(fb[cb], vf[0][ks], ks == 0 ? nd[kt] : t2[kt][0]);
        t2[kt][1] = mfma16(fb[cb], vf[1][ks], ks == 0 ? nd[kt] : t2[kt][1]);
        if (s > 0) weight2(s - 1, ks);
        else describe(ks);
      }
    }
    load_term(sb, 3);
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      if (hh == 1) {
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(TILE_LOADS) : "memory");
        __builtin_amdgcn_s_barrier();                   // the fragments in flight are of this tile, whose stage nobody fills yet
        asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) {
        const int n = 16 + 8 * hh + ct, cb = n % NB;
        ISA_KV_FENCE();
        load(n + PF < 32 ? sb : sb_next, (n + PF) % 32);
        if (n == 31) load_delta(sb_next, 0);
        mfma16_acc(fa[cb], ws[hh][0], ak[ct][0]);
        mfma16_acc(fa[cb], ws[hh][1], ak[ct][1]);
        mfma16_acc(fb[cb], wp[hh][0], av[ct][0]);
        mfma16_acc(fb[cb], wp[hh][1], av[ct][1]);
        if (hh == 0 && ct < 7 && !(ct & 1)) weight2(3, ct >> 1);
      }
    }
    ISA_KV_FENCE();
    if (--live == 0) break;
  }
  }
  // the loads past the end still target this workgroup's LDS: let them land before the waves end
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int ct = 0; ct < 8; ++ct)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) { settle(ak[ct][qt]); settle(av[ct][qt]); }
  // ---- element i of ak / av[ct][qt] is channel 16 ct + 4 q + i of row 16 qt + r
  if (tail_slot >= 0) {                                 // a part: unscaled sums, k_bwd_kv_merge does the rest
    float* dst = a.tail_scratch + ((long long)((a.dyn_ctr ? 0 : xcd * a.tail_items) + tail_slot) * parts + part) * 2 * 128 * MD;
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) {
        float* p = dst + (wave * 32 + 16 * qt + r16) * MD + 16 * ct + 4 * q;
        *reinterpret_cast<f32x4*>(p) = ak[ct][qt];
        *reinterpret_cast<f32x4*>(p + 128 * MD) = av[ct][qt];
      }
    return;
  }
  const float inv_n = 1.0f / (float)n_x;
  const long long mean = (bh * a.Tn_pad + entry) * MD + 4 * q;
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int row = wave * 32 + 16 * qt + r16;
    if (row >= n_x) continue;
    const long long off = tbase + (long long)(x_start + row) * a.geo.stride_t + 4 * q;
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
      float4 rk = make_float4(ak[ct][qt][0] * a.scale, ak[ct][qt][1] * a.scale, ak[ct][qt][2] * a.scale, ak[ct][qt][3] * a.scale);
      float4 rv = make_float4(av[ct][qt][0], av[ct][qt][1], av[ct][qt][2], av[ct][qt][3]);
      if (a.mean_k) {
        const float4 mk = *reinterpret_cast<const float4*>(a.mean_k + mean + 16 * ct);
        const float4 mv = *reinterpret_cast<const float4*>(a.mean_v + mean + 16 * ct);
        rk.x = fmaf(mk.x, inv_n, rk.x); rk.y = fmaf(mk.y, inv_n, rk.y); rk.z = fmaf(mk.z, inv_n, rk.z); rk.w = fmaf(mk.w, inv_n, rk.w);
        rv.x = fmaf(mv.x, inv_n, rv.x); rv.y = fmaf(mv.y, inv_n, rv.y); rv.z = fmaf(mv.z, inv_n, rv.z); rv.w = fmaf(mv.w, inv_n, rv.w);
      }
      *reinterpret_cast<uint2*>(a.dk + off + 16 * ct) = bf16x4_of(rk);
      *reinterpret_cast<uint2*>(a.dv + off + 16 * ct) = bf16x4_of(rv);
    }
  }
}

// Adds up the parts of the tail items in a fixed order and writes their rows.  One workgroup per (XCD, tail item, tensor, 8 rows);
// 32 threads per row, 4 channels each.
__global__ __launch_bounds__(256) void k_bwd_kv_merge(KvArgs a) {
  const int rows8 = blockIdx.x & 15, which = (blockIdx.x >> 4) & 1;
  const int slot = blockIdx.x >> 5, n_bh = a.geo.B * a.geo.H;
  int entry, bhid;
  if (a.dyn_ctr) {
    entry = (a.dyn_whole + slot) % a.items;
    bhid = (a.dyn_whole + slot) / a.items;
  } else {
    const int xcd = slot / a.tail_items;
    const long long n_items = (long long)a.items * n_bh;
    const int idx = xcd_first(n_items, xcd) + a.items_xcd - a.tail_items + slot % a.tail_items;
    if (idx >= xcd_first(n_items, xcd + 1)) return;
    entry = idx % a.items;
    bhid = head_at(idx / a.items, n_bh);
  }
  const int h = bhid % a.geo.H, b = bhid / a.geo.H;
  if (entry >= a.cnt.b[b].T_new) return;
  const int4 own = a.ktab[(long long)bhid * a.geo.T_max + entry];
  const int row = rows8 * 8 + (threadIdx.x >> 5), ch = (threadIdx.x & 31) * 4;
  if (row >= own.y) return;
  const float* src = a.tail_scratch + ((long long)slot * a.tail_parts * 2 + which) * 128 * MD + row * MD + ch;
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int p0 = 0; p0 < a.tail_parts; p0 += 4) {        // four parts' loads in flight
    float4 o[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = *reinterpret_cast<const float4*>(src + (long long)min(p0 + u, a.tail_parts - 1) * 2 * 128 * MD);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (p0 + u >= a.tail_parts) break;
      sum.x += o[u].x; sum.y += o[u].y; sum.z += o[u].z; sum.w += o[u].w;
    }
  }
  if (!which) { sum.x *= a.scale; sum.y *= a.scale; sum.z *= a.scale; sum.w *= a.scale; }
  if (a.mean_k) {
    const float inv_n = 1.0f / (float)own.y;
    const float4 m = *reinterpret_cast<const float4*>((which ? a.mean_v : a.mean_k) + ((long long)bhid * a.Tn_pad + entry) * MD + ch);
    sum.x = fmaf(m.x, inv_n, sum.x); sum.y = fmaf(m.y, inv_n, sum.y); sum.z = fmaf(m.z, inv_n, sum.z); sum.w = fmaf(m.w, inv_n, sum.w);
  }
  const long long off = (long long)b * a.geo.stride_b + (long long)h * a.geo.stride_h + (long long)(own.x + row) * a.geo.stride_t + ch;
  *reinterpret_cast<uint2*>((which ? a.dv : a.dk) + off) = bf16x4_of(sum);
}

hipError_t launch_bwd_kv(const Problem& pr, const Workspace& ws, const void* q, const void* k, const void* v, const void* d_out,
                         bool exact_sets, bool mean_grads, void* dk, void* dv, hipStream_t st) {
  const int B = pr.p.B, H = pr.p.H, cus = cus_per_xcd();
  int sk = 0, min_full = 1 << 30;
  for (int b = 0; b < B; ++b) {
    const BatchCounts& c = pr.cnt.b[b];
    sk = c.T_new > sk ? c.T_new : sk;
    min_full = c.n_full < min_full ? c.n_full : min_full;
  }
  KvArgs a;
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v; a.d_o = (const uint16_t*)d_out;
  a.ktab = ws.ktab;
  a.qtab[0] = ws.ftab; a.qtab[1] = ws.ltab;
  a.qside[0] = ws.ybd_full; a.qside[1] = ws.ybd_flat;
  a.bits = exact_sets ? ws.mask_t : nullptr;
  a.mean_k = mean_grads ? ws.dkc : nullptr; a.mean_v = mean_grads ? ws.dvc : nullptr;
  a.dk = (uint16_t*)dk; a.dv = (uint16_t*)dv;
  a.scale = 1.0f / sqrtf((float)MD);
  a.geo = pr.geo; a.cnt = pr.cnt; a.Tn_pad = pr.Tn_pad;
  a.items = sk;
  a.items_xcd = (int)(((long long)sk * B * H + N_XCD - 1) / N_XCD);
  a.tail_items = 0; a.tail_parts = 1; a.tail_scratch = ws.split_o;
  // Items from a counter (an XCD that gets through its workgroups sooner takes more of them) where there is more than half a
  // round of them; fewer are cut into parts along the streamed lists instead.
  a.dyn_ctr = ws.bwd_ctr + 1;
  if (a.items_xcd <= cus / 2 && min_full > 1) {
    int parts = cus / a.items_xcd > 8 ? 8 : cus / a.items_xcd;
    if (parts > min_full) parts = min_full;
    while (parts > 1 && N_XCD * a.items_xcd * parts > SPLIT_MAX_SUB) --parts;       // the partial-result area holds SPLIT_MAX_SUB sub-items
    if (parts > 1) { a.dyn_ctr = nullptr; a.tail_items = a.items_xcd; a.tail_parts = parts; }
  }
  // 8 rounds or more: the last 32 items run in 8 parts each, so that the launch ends within an eighth of an item of the ideal.
  a.dyn_whole = sk * B * H;
  a.dyn_total = a.dyn_whole;
  int n_merge = N_XCD * a.tail_items;
  if (a.dyn_ctr && a.items_xcd >= 8 * cus && min_full >= 16) {
    a.tail_parts = 8;
    n_merge = SPLIT_MAX_SUB / a.tail_parts;
    a.dyn_whole -= n_merge;
    a.dyn_total += n_merge * (a.tail_parts - 1);
  }
  // an eighth more workgroups than items and one round of the chip, so that the faster XCDs do not run out of workgroups
  const long long n_dyn = a.dyn_total;
  const long long wgs = a.dyn_ctr ? (n_dyn + n_dyn / 8) / N_XCD + cus + 1 : (long long)a.tail_items * a.tail_parts;
  hipLaunchKernelGGL(k_bwd_kv, dim3((unsigned)(wgs * N_XCD)), dim3(256), 0, st, a);
  if (n_merge > 0) hipLaunchKernelGGL(k_bwd_kv_merge, dim3((unsigned)(n_merge * 32)), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace isa
