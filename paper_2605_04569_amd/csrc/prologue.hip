// Prologue of the operator: tile-order flattening (Sec. 2 "Block Sparse Attention": spatiotemporal tiles are formed
// first and flattened in tile order, then the sequence is cut into blocks) and the decoupled rotary embedding (Sec. 4:
// applied to the source and to every context reference independently, coordinates counted from zero in each), fused
// with the block means of Alg. 1 Stage 1 into one streaming pass over Q, K and V.
//
// Input tokens of a segment arrive row-major over its (t, h, w) grid, w fastest.  Output position p of a segment holds
// the p-th token in tile order: tiles row-major over tile coordinates, tokens row-major inside a tile, tiles clipped at
// the far edges of the grid.  Q and K are rotated on interleaved channel pairs (2i, 2i+1): the first rope_dims[0]
// channels by the frame coordinate, the next rope_dims[1] by the row, the next rope_dims[2] by the column; pair j of an
// axis with d channels turns by coordinate * theta^(-2j/d) radians.  V is only reordered.
//
// HBM-bound: one workgroup owns one output block (<= 128 tokens) of a few heads, reads every token row once with 16-byte
// loads (a row is D contiguous elements wherever it comes from, so the gather costs nothing in coalescing), rotates in
// registers (the sines and cosines of a thread's pairs are computed once and reused for every head and for Q and K),
// writes the row once and keeps the running sums for the block means.  The rows of the next (head, tensor) pass are
// loaded into a second set of registers while the current pass is rotated and stored.
#include <math.h>
#include <string.h>

#include "isa_internal.h"

namespace isa {

constexpr int PBLOCK = 128;   // largest block
constexpr int ENTRIES = 4096; // sines and cosines that a workgroup has room for

struct GridDesc {             // passed to kernels by value
  int grid[ISA_MAX_SEGMENTS][3];
  int tile[3];
  int rope_dims[3];
  double log2_theta;
};

struct BlockPos { int n, start, seg_start, p0, t, h, w; };

// Block j of batch item b: its real tokens n (0 if there is no such block), first token `start` inside the batch item,
// the first token of its segment, its offset p0 inside the segment and the segment's grid.  Static indices only.
__device__ inline BlockPos locate_block(const SegDesc& seg, const GridDesc& gd, int b, int j, int block) {
  int s0 = 0, s1 = 0;
#pragma unroll
  for (int i = 0; i < ISA_MAX_BATCH; ++i)
    if (i == b) { s0 = seg.seg_ptr[i]; s1 = seg.seg_ptr[i + 1]; }
  BlockPos r = {0, 0, 0, 0, 1, 1, 1};
  int blocks = 0, tok = 0;
  bool found = false;
#pragma unroll
  for (int s = 0; s < ISA_MAX_SEGMENTS; ++s) {
    if (s >= s0 && s < s1) {
      const int len = seg.seg_len[s];
      const int nb = (len + block - 1) / block;
      if (!found && j < blocks + nb) {
        found = true;
        r.p0 = (j - blocks) * block;
        r.n = min(block, len - r.p0);
        r.seg_start = tok;
        r.start = tok + r.p0;
        r.t = gd.grid[s][0]; r.h = gd.grid[s][1]; r.w = gd.grid[s][2];
      }
      blocks += nb;
      tok += len;
    }
  }
  return r;
}

// Coordinates of the token at position p of a segment's tile order.
__device__ inline void tile_coords(int p, int t, int h, int w, int tt, int th, int tw, int* ct, int* ch, int* cw) {
  tt = min(tt, t); th = min(th, h); tw = min(tw, w);
  const int a = p / (tt * h * w);                  // all tiles before tile plane a cover tt whole frames each
  p -= a * tt * h * w;
  const int st = min(tt, t - a * tt);
  const int bq = p / (st * th * w);                // inside the plane: tile rows cover th whole rows of st frames
  p -= bq * st * th * w;
  const int sh = min(th, h - bq * th);
  const int c = p / (st * sh * tw);
  p -= c * st * sh * tw;
  const int sw = min(tw, w - c * tw);
  const int lt = p / (sh * sw);
  p -= lt * sh * sw;
  const int lh = p / sw;
  *ct = a * tt + lt;
  *ch = bq * th + lh;
  *cw = c * tw + (p - lh * sw);
}

// Rows of long calls are streamed (nontemporal): loads of more than the last-level cache holds, and stores of so much that little of it is found
// there by what reads it next.  Chains, us, cached / streamed stores: copy into q, k, v - isa_prologue - isa_attention - isa_untile - copy of its
// output, 40 heads of 3168 tokens (32 MB a tensor) 222 / 229, 24 of 10 400 (64) 543 / 542, 20 of 15 600 (80) 800 / 794, 40 of 15 600 (160)
// 1540 / 1501; the same with inputs from memory 183 / 190, 464 / 480, 703 / 711, 1365 / 1334.  The three calls over and over on the same
// buffers, whose outputs nothing reads: 20 of 6240 (32 MB) 83 / 79, 20 of 15 600 215 / 182, with streamed loads as well 198; 40 of 39 680 (1.2 GB of q, k, v)
// 1030 / 1003 / 926.
constexpr long long CACHE_BYTES = 256ll << 20;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <bool STREAM> __device__ __forceinline__ void store16(void* p, uint32_t x, uint32_t y, uint32_t z, uint32_t w) {
  if constexpr (STREAM) __builtin_nontemporal_store(u32x4{x, y, z, w}, reinterpret_cast<u32x4*>(p));
  else *reinterpret_cast<u32x4*>(p) = u32x4{x, y, z, w};
}
template <bool STREAM> __device__ __forceinline__ uint4 load16(const void* p) {
  const u32x4* const q = reinterpret_cast<const u32x4*>(p);
  u32x4 r;
  if constexpr (STREAM) r = __builtin_nontemporal_load(q);
  else r = *q;
  return make_uint4(r.x, r.y, r.z, r.w);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
template <typename T> struct Row16;      // 16 bytes of a token row
template <> struct Row16<float> {
  static constexpr int N = 4;
  __device__ static void unpack(const uint4& v, float* o) {
    o[0] = __uint_as_float(v.x); o[1] = __uint_as_float(v.y); o[2] = __uint_as_float(v.z); o[3] = __uint_as_float(v.w);
  }
  template <bool STREAM> __device__ static void store(float* p, float* o) {       // o is left holding the stored values
    store16<STREAM>(p, __float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3]));
  }
};
template <> struct Row16<uint16_t> {   // bf16 storage
  static constexpr int N = 8;
  __device__ static void unpack(const uint4& v, float* o) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  template <bool STREAM> __device__ static void store(uint16_t* p, float* o) {    // o is left holding the rounded values
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bf16x2 r = {(__bf16)o[2 * i], (__bf16)o[2 * i + 1]};         // one instruction, to nearest even
      w[i] = __builtin_bit_cast(uint32_t, r);
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
    store16<STREAM>(p, w[0], w[1], w[2], w[3]);
  }
};

// Loads the thread's 16-byte piece of TPT token rows (all in flight together).
template <typename T, int TPT, bool STREAM>
__device__ __forceinline__ void load_rows(uint4 (&raw)[TPT], const T* ip, const int (&src)[TPT], long long stride_t) {
#pragma unroll
  for (int tk = 0; tk < TPT; ++tk) raw[tk] = load16<STREAM>(ip + (long long)src[tk] * stride_t);
}

// Rotates (if asked), stores and sums the rows that load_rows brought in; acc receives the column sums of what was stored.
template <typename T, int TPT, int NP, bool STREAM>
__device__ __forceinline__ void finish_rows(const uint4 (&raw)[TPT], const float (&cs)[TPT][NP], const float (&sn)[TPT][NP],
                                            bool rotate, unsigned valid, T* op, const int (&dst)[TPT], long long stride_t,
                                            float (&acc)[2 * NP]) {
#pragma unroll
  for (int i = 0; i < 2 * NP; ++i) acc[i] = 0.f;
#pragma unroll
  for (int tk = 0; tk < TPT; ++tk) {
    float x[2 * NP];
    Row16<T>::unpack(raw[tk], x);
    if (rotate) {      // uniform
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const float a0 = x[2 * i], a1 = x[2 * i + 1];
        x[2 * i] = a0 * cs[tk][i] - a1 * sn[tk][i];
        x[2 * i + 1] = a0 * sn[tk][i] + a1 * cs[tk][i];
      }
    }
    if (valid >> tk & 1) {
      Row16<T>::template store<STREAM>(op + (long long)dst[tk] * stride_t, x);
#pragma unroll
      for (int i = 0; i < 2 * NP; ++i) acc[i] += x[i];
    }
  }
}

// The smallest / largest of a wave's 64 numbers, in every lane.
template <bool MAX>
__device__ __forceinline__ int wave_extreme(int x) {
  auto both = [](int a, int b) { return MAX ? max(a, b) : min(a, b); };
  const auto s = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  x = both(s[0], s[1]);
  const auto t = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = both(t[0], t[1]);
  x = both(x, __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, true));         // row_ror 8, 4, 2, 1
  x = both(x, __builtin_amdgcn_update_dpp(0, x, 0x124, 0xf, 0xf, true));
  x = both(x, __builtin_amdgcn_update_dpp(0, x, 0x122, 0xf, 0xf, true));
  return both(x, __builtin_amdgcn_update_dpp(0, x, 0x121, 0xf, 0xf, true));
}

// A long launch is HBM-bound (see the top), a short one waits for a workgroup's own chain: coordinates, frequencies, sines and cosines, then
// a pass per tensor.
// TABLE: a block's tokens have few coordinates (a tile of 2 x 8 x 8: 2 frames, 8 rows, 8 columns), so the workgroup works the sines and
// cosines of each coordinate out once, one channel pair a thread, and hands them out through LDS: 380 in place of 8192, and 11 KB less
// code to fetch.  Without: a thread works out its own, for grids whose coordinates have no room and where it has 8 (D = 64, blocks of 64).
// SPLIT: a workgroup takes one of the three tensors.  PB: the block, so that a thread has no rows that a block of 64 has not.
// All three, and roundings of one instruction, us (isa_prologue; before / after): bf16, 5 heads of 440 tokens 19.3 / 9.7, 16 of 1848 22.1 /
// 15.9, 8 of 15 600 47 / 35.5; blocks of 64, 12 of 2704 28 / 17, D = 64 12 of 7920 25 / 19; fp32, 4 of 39 680 117 / 101.
// LOADS, STORES: streamed, see load16 and store16.
template <typename T, int D, int PB, bool TABLE, bool SPLIT, bool LOADS, bool STORES>
__global__ __launch_bounds__(256) void k_prologue(const T* __restrict__ q_in, const T* __restrict__ k_in,
                                                  const T* __restrict__ v_in, T* __restrict__ q_out,
                                                  T* __restrict__ k_out, T* __restrict__ v_out,
                                                  float* __restrict__ qc, float* __restrict__ kc,
                                                  float* __restrict__ vc, SegDesc seg, GridDesc gd, Geometry g, int hpw,
                                                  int inverse) {
  constexpr int VEC = Row16<T>::N;
  constexpr int CH = D / VEC;            // 16-byte chunks per row
  constexpr int RP = 256 / CH;           // rows covered per pass
  constexpr int TPT = PB / RP;           // rows per thread
  constexpr int NP = VEC / 2;            // channel pairs per thread
  __shared__ int s_src[PB];
  __shared__ int s_pos[PB][3];
  constexpr int RED = 2 * RP * D, SHARED = TABLE && 2 * ENTRIES > RED ? 2 * ENTRIES : RED;
  __shared__ __attribute__((aligned(16))) float shared[SHARED];
  float (&red)[2][RP][D] = *reinterpret_cast<float (*)[2][RP][D]>(shared);
  float2* const table = reinterpret_cast<float2*>(shared);             // until the passes begin
  __shared__ int s_lo[4][3], s_hi[4][3];
  const int j = blockIdx.x, b = blockIdx.z, h0 = SPLIT ? blockIdx.y / 3 : blockIdx.y * hpw;
  const BlockPos bp = locate_block(seg, gd, b, j, g.block);
  if (bp.n == 0) return;
  if (TABLE || threadIdx.x < bp.n) {
    int co[3];
    const int i = min((int)threadIdx.x, bp.n - 1);     // (the others repeat the last token's)
    tile_coords(bp.p0 + i, bp.t, bp.h, bp.w, gd.tile[0], gd.tile[1], gd.tile[2], &co[0], &co[1], &co[2]);
    if (threadIdx.x < bp.n) {
      s_src[i] = bp.seg_start + (co[0] * bp.h + co[1]) * bp.w + co[2];
#pragma unroll
      for (int a = 0; a < 3; ++a) s_pos[i][a] = co[a];
    }
    if constexpr (TABLE) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        s_lo[threadIdx.x >> 6][a] = wave_extreme<false>(co[a]);
        s_hi[threadIdx.x >> 6][a] = wave_extreme<true>(co[a]);
      }
    }
  }
  __syncthreads();

  const int c = threadIdx.x % CH, rg = threadIdx.x / CH;
  // the thread's rows: where each is read and where it is written (rows past the block's end re-read the block's first
  // row and are dropped).  Forward: gathered from the row-major place, written at the tile-order place; the inverse
  // direction (the transpose, used for gradients) swaps the two.
  int src[TPT], dst[TPT];
  unsigned valid = 0;
#pragma unroll
  for (int tk = 0; tk < TPT; ++tk) {
    const int r = rg + tk * RP, rc = r < bp.n ? r : 0;
    const int raster = s_src[rc], tiled = bp.start + rc;
    src[tk] = inverse ? tiled : raster;
    dst[tk] = inverse ? raster : tiled;
    valid |= (r < bp.n ? 1u : 0u) << tk;
  }
  // (head, tensor) passes of this workgroup: q, k, v of a head in turn, or one of them
  const int first_it = SPLIT ? blockIdx.y % 3 : 0, n_it = SPLIT ? first_it + 1 : 3 * min(hpw, g.H - h0);
  const long long base0 = (long long)b * g.stride_b + (long long)h0 * g.stride_h + c * VEC;

  // Two sets of landing registers: the rows of pass it + 1 are in flight while pass it is rotated and stored.
  uint4 raw0[TPT], raw1[TPT];
#define ISA_IN_PTR(it) ((((it) % 3) == 0 ? q_in : ((it) % 3) == 1 ? k_in : v_in) + base0 + (long long)((it) / 3) * g.stride_h)
  load_rows<T, TPT, LOADS>(raw0, ISA_IN_PTR(first_it), src, g.stride_t);

  // the thread's channel pairs: which coordinate turns them, and how fast; then the sines and cosines of its rows
  // (computed while the first rows are on their way)
  float cs[TPT][NP], sn[TPT][NP];
  auto pair_axis = [&](int& pr) {                        // pr: from channel pair to pair of its axis
    if (pr < gd.rope_dims[0] / 2) return 0;
    if ((pr -= gd.rope_dims[0] / 2) < gd.rope_dims[1] / 2) return 1;
    if ((pr -= gd.rope_dims[1] / 2) < gd.rope_dims[2] / 2) return 2;
    return -1;
  };
  auto pick = [](int axis, int x0, int x1, int x2) { return axis == 0 ? x0 : axis == 1 ? x1 : x2; };
  auto pair_freq = [&](int axis, int pr) {
    return axis < 0 ? 0.0 : exp2(-2.0 * (double)pr / (double)pick(axis, gd.rope_dims[0], gd.rope_dims[1], gd.rope_dims[2]) * gd.log2_theta);
  };
  auto turn = [&](int pos, double freq, float* sine, float* cosine) {
    double turns = (double)pos * freq * 0.1591549430918953357689;                  // angle / 2 pi
    turns -= rint(turns);                                                          // into [-1/2, 1/2]
    sincospif((float)(2.0 * turns), sine, cosine);
    if (inverse) *sine = -*sine;                                                   // turn back
  };
  if constexpr (TABLE) {
    int lo[3], n[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = min(min(s_lo[0][a], s_lo[1][a]), min(s_lo[2][a], s_lo[3][a]));
      n[a] = max(max(s_hi[0][a], s_hi[1][a]), max(s_hi[2][a], s_hi[3][a])) - lo[a] + 1;
    }
    const int p0 = gd.rope_dims[0] / 2, p1 = gd.rope_dims[1] / 2, p2 = gd.rope_dims[2] / 2;
    const bool rotates = !SPLIT || first_it < 2;
    if (rotates) {
      int pr = threadIdx.x % (D / 2);
      const int axis = pair_axis(pr);
      if (axis >= 0) {
        const double freq = pair_freq(axis, pr);
        const int count = pick(axis, n[0], n[1], n[2]), from = pick(axis, lo[0], lo[1], lo[2]), pairs = pick(axis, p0, p1, p2);
        float2* const out = table + pick(axis, 0, n[0] * p0, n[0] * p0 + n[1] * p1) + pr;
#pragma unroll 1
        for (int k = threadIdx.x / (D / 2); k < count; k += 256 / (D / 2)) {
          float2 t;
          turn(from + k, freq, &t.x, &t.y);
          out[k * pairs] = t;
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      int pr = c * NP + i;
      const int axis = pair_axis(pr);
      const bool turned = rotates && axis >= 0;
      const int pairs = pick(axis, p0, p1, p2), a = max(axis, 0);
      const int at = pick(axis, 0, n[0] * p0, n[0] * p0 + n[1] * p1) + pr - pick(axis, lo[0], lo[1], lo[2]) * pairs;
#pragma unroll
      for (int tk = 0; tk < TPT; ++tk) {
        const int r = rg + tk * RP;
        const float2 t = table[turned ? at + s_pos[r < bp.n ? r : 0][a] * pairs : 0];
        sn[tk][i] = turned ? t.x : 0.f;
        cs[tk][i] = turned ? t.y : 1.f;
      }
    }
    if (rotates) __syncthreads();                        // from here on the place is the block means'
  } else {
    int axis[NP];
    double freq[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      int pr = c * NP + i;
      axis[i] = pair_axis(pr);
      freq[i] = pair_freq(axis[i], pr);
    }
#pragma unroll
    for (int tk = 0; tk < TPT; ++tk) {
      const int r = rg + tk * RP;
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        cs[tk][i] = 1.f; sn[tk][i] = 0.f;
        if (r < bp.n && axis[i] >= 0) turn(pick(axis[i], s_pos[r][0], s_pos[r][1], s_pos[r][2]), freq[i], &sn[tk][i], &cs[tk][i]);
      }
    }
  }

  const float inv_n = 1.0f / (float)bp.n;
  const bool means = qc != nullptr;
  // the second half of a pass: the block means of what was just stored.  red[B] is next written two passes later,
  // behind the barrier of the pass in between.
#define ISA_PASS(RAW, B, it)                                                                                          \
  {                                                                                                                   \
    const int t_ = (it) % 3, hh_ = (it) / 3;                                                                          \
    float acc_[VEC];                                                                                                  \
    finish_rows<T, TPT, NP, STORES>(RAW, cs, sn, t_ < 2, valid,                                                       \
                            (t_ == 0 ? q_out : t_ == 1 ? k_out : v_out) + base0 + (long long)hh_ * g.stride_h,         \
                            dst, g.stride_t, acc_);                                                                    \
    if (means) {                                                                                                      \
      _Pragma("unroll") for (int i = 0; i < VEC; ++i) red[B][rg][c * VEC + i] = acc_[i];                              \
      __syncthreads();                                                                                                \
      if (threadIdx.x < D) {                                                                                          \
        float sum_ = 0.f;                                                                                             \
        _Pragma("unroll") for (int r = 0; r < RP; ++r) sum_ += red[B][r][threadIdx.x];                                \
        float* mp_ = t_ == 0 ? qc : t_ == 1 ? kc : vc;                                                                \
        mp_[(((long long)b * g.H + h0 + hh_) * g.T_max + j) * D + threadIdx.x] = sum_ * inv_n;                        \
      }                                                                                                               \
    }                                                                                                                 \
  }
  for (int it = first_it; it < n_it; it += 2) {
    if (it + 1 < n_it) load_rows<T, TPT, LOADS>(raw1, ISA_IN_PTR(it + 1), src, g.stride_t);
    ISA_PASS(raw0, 0, it)
    if (it + 1 < n_it) {
      if (it + 2 < n_it) load_rows<T, TPT, LOADS>(raw0, ISA_IN_PTR(it + 2), src, g.stride_t);
      ISA_PASS(raw1, 1, it + 1)
    }
  }
#undef ISA_PASS
#undef ISA_IN_PTR
}

// Inverse reordering of one tensor: token p of the tile order goes back to its row-major place.
template <typename T, int D, int PB, bool LOADS, bool STORES>
__global__ __launch_bounds__(256) void k_untile(const T* __restrict__ x_tiled, T* __restrict__ x_raster, SegDesc seg,
                                                GridDesc gd, Geometry g, int hpw) {
  constexpr int VEC = Row16<T>::N;
  constexpr int CH = D / VEC;
  constexpr int RP = 256 / CH;
  constexpr int TPT = PB / RP;
  __shared__ int s_src[PB];
  const int j = blockIdx.x, b = blockIdx.z, h0 = blockIdx.y * hpw;
  const BlockPos bp = locate_block(seg, gd, b, j, g.block);
  if (bp.n == 0) return;
  if (threadIdx.x < bp.n) {
    int ct, ch, cw;
    tile_coords(bp.p0 + threadIdx.x, bp.t, bp.h, bp.w, gd.tile[0], gd.tile[1], gd.tile[2], &ct, &ch, &cw);
    s_src[threadIdx.x] = bp.seg_start + (ct * bp.h + ch) * bp.w + cw;
  }
  __syncthreads();
  const int c = threadIdx.x % CH, rg = threadIdx.x / CH;
  int src[TPT];
#pragma unroll
  for (int tk = 0; tk < TPT; ++tk) src[tk] = rg + tk * RP < bp.n ? s_src[rg + tk * RP] : -1;
  for (int hh = 0; hh < hpw; ++hh) {
    const int h = h0 + hh;
    if (h >= g.H) break;
    const long long base = (long long)b * g.stride_b + (long long)h * g.stride_h + c * VEC;
    uint4 x[TPT];
#pragma unroll
    for (int tk = 0; tk < TPT; ++tk) {      // rows past the block's end re-read its first row and are not stored
      const int row = src[tk] >= 0 ? bp.start + rg + tk * RP : bp.start;
      x[tk] = load16<LOADS>(x_tiled + base + (long long)row * g.stride_t);
    }
#pragma unroll
    for (int tk = 0; tk < TPT; ++tk)
      if (src[tk] >= 0) store16<STORES>(x_raster + base + (long long)src[tk] * g.stride_t, x[tk].x, x[tk].y, x[tk].z, x[tk].w);
  }
}

// Heads per workgroup: as many as still leave about eight workgroups per compute unit (the per-block set-up, the sines
// and cosines above all, is paid once per workgroup).
static int heads_per_wg(const Problem& pr) {
  const long long blocks = (long long)pr.cnt.T_max * pr.p.B;
  long long hpw = blocks * pr.p.H / 2048;
  if (hpw < 1) hpw = 1;
  if (hpw > pr.p.H) hpw = pr.p.H;
  return (int)hpw;
}

// Stores are streamed from tensors of 64 MB on (see store16)
constexpr int STORE_TENSORS = 4;
// Whether `tensors` of the problem's tensors have more bytes than the last-level cache.
static bool exceeds_cache(const Problem& pr, int tensors) {
  long long rows = 0;
  for (int b = 0; b < pr.p.B; ++b) rows += pr.cnt.b[b].S;
  return tensors * rows * pr.p.H * pr.p.D * (pr.p.dtype == ISA_BF16 ? 2 : 4) >= CACHE_BYTES;
}

static GridDesc make_desc(const Problem& pr, const isa_grid* gr) {
  GridDesc gd;
  memset(&gd, 0, sizeof(gd));
  const int n_seg = pr.seg.seg_ptr[pr.p.B];
  for (int s = 0; s < n_seg; ++s)
    for (int a = 0; a < 3; ++a) gd.grid[s][a] = gr->seg_grid[3 * s + a];
  for (int a = 0; a < 3; ++a) { gd.tile[a] = gr->tile[a]; gd.rope_dims[a] = gr->rope_dims[a]; }
  gd.log2_theta = log2(gr->rope_theta);
  return gd;
}

// Whether the coordinates of every block have room in the table.  A block is at most 128 consecutive tokens of the tile order: they may
// have any row and column of the grid, and the frames of the tile planes they lie in.
static bool table_fits(const Problem& pr, const isa_grid* gr) {
  const int n_seg = pr.seg.seg_ptr[pr.p.B];
  for (int s = 0; s < n_seg; ++s) {
    const long long t = gr->seg_grid[3 * s], h = gr->seg_grid[3 * s + 1], w = gr->seg_grid[3 * s + 2];
    if (t == 0 || h == 0 || w == 0) continue;
    const long long tt = gr->tile[0] < t ? gr->tile[0] : t, planes = (PBLOCK - 1) / (tt * h * w) + 2;
    const long long frames = planes * tt < t ? planes * tt : t;
    if (frames * (gr->rope_dims[0] / 2) + h * (gr->rope_dims[1] / 2) + w * (gr->rope_dims[2] / 2) > ENTRIES) return false;
  }
  return true;
}

hipError_t launch_prologue(const Problem& pr, const isa_grid* gr, const void* q_in, const void* k_in, const void* v_in,
                           void* q_out, void* k_out, void* v_out, float* qc, float* kc, float* vc, bool inverse,
                           hipStream_t st) {
  const GridDesc gd = make_desc(pr, gr);
  const bool loads = exceeds_cache(pr, 3), stores = exceeds_cache(pr, STORE_TENSORS);
  const int hpw = heads_per_wg(pr);
  // one tensor a workgroup as long as all of them run at once (an fp32 row of 128 channels takes a whole compute unit's registers): 8 heads of
  // 2400 tokens (160 workgroups) 14.7 / 13.6 us, 16 of 1848 (256) 15.9 / 21.1; fp32, 12 of 1564 (168) 18.4 / 22.8
  const long long resident = pr.p.dtype == ISA_F32 && pr.p.D == 128 && pr.p.block == 128 ? 1 : 2;
  const bool split = 3ll * pr.cnt.T_max * pr.p.B * pr.p.H <= resident * N_XCD * cus_per_xcd(), table = table_fits(pr, gr);
  const dim3 grid(pr.cnt.T_max, split ? 3 * pr.p.H : (pr.p.H + hpw - 1) / hpw, pr.p.B), blk(256);
#define ISA_PRO2(T, D, PB, TABLE, SPLIT, LOADS, STORES)                                                               \
  hipLaunchKernelGGL((k_prologue<T, D, PB, TABLE, SPLIT, LOADS, STORES>), grid, blk, 0, st, (const T*)q_in, (const T*)k_in,   \
                     (const T*)v_in, (T*)q_out, (T*)k_out, (T*)v_out, qc, kc, vc, pr.seg, gd, pr.geo, hpw, inverse ? 1 : 0)
#define ISA_PRO1(T, D, PB, TABLE)                                                                                     \
  do {                                                                                                                \
    if (split) ISA_PRO2(T, D, PB, TABLE, true, false, false);                                                         \
    else if (loads) ISA_PRO2(T, D, PB, TABLE, false, true, true);                                                     \
    else if (stores) ISA_PRO2(T, D, PB, TABLE, false, false, true);                                                   \
    else ISA_PRO2(T, D, PB, TABLE, false, false, false);                                                              \
  } while (0)
#define ISA_PRO(T, D)                                                                                                \
  do {                                                                                                               \
    if (pr.p.block == 128) { if (table) ISA_PRO1(T, D, 128, true); else ISA_PRO1(T, D, 128, false); }                \
    else if (D == 128 && table) ISA_PRO1(T, D, 64, (D == 128));                                                      \
    else ISA_PRO1(T, D, 64, false);                                                                                  \
  } while (0)
  if (pr.p.dtype == ISA_BF16) {
    if (pr.p.D == 128) ISA_PRO(uint16_t, 128); else ISA_PRO(uint16_t, 64);
  } else {
    if (pr.p.D == 128) ISA_PRO(float, 128); else ISA_PRO(float, 64);
  }
#undef ISA_PRO
#undef ISA_PRO1
#undef ISA_PRO2
  return hipGetLastError();
}

hipError_t launch_untile(const Problem& pr, const isa_grid* gr, const void* x_tiled, void* x_raster, hipStream_t st) {
  const GridDesc gd = make_desc(pr, gr);
  const bool loads = exceeds_cache(pr, 1), stores = exceeds_cache(pr, STORE_TENSORS);
  const int hpw = heads_per_wg(pr);
  const dim3 grid(pr.cnt.T_max, (pr.p.H + hpw - 1) / hpw, pr.p.B), blk(256);
#define ISA_UNT2(T, D, PB, LOADS, STORES) \
  hipLaunchKernelGGL((k_untile<T, D, PB, LOADS, STORES>), grid, blk, 0, st, (const T*)x_tiled, (T*)x_raster, pr.seg, gd, pr.geo, hpw)
#define ISA_UNT1(T, D, PB)                                                                                           \
  do {                                                                                                               \
    if (loads) ISA_UNT2(T, D, PB, true, true);                                                                       \
    else if (stores) ISA_UNT2(T, D, PB, false, true);                                                                \
    else ISA_UNT2(T, D, PB, false, false);                                                                           \
  } while (0)
#define ISA_UNT(T, D)                                                                                                \
  do {                                                                                                               \
    if (pr.p.block == 64) ISA_UNT1(T, D, 64); else ISA_UNT1(T, D, 128);                                              \
  } while (0)
  if (pr.p.dtype == ISA_BF16) {
    if (pr.p.D == 128) ISA_UNT(uint16_t, 128); else ISA_UNT(uint16_t, 64);
  } else {
    if (pr.p.D == 128) ISA_UNT(float, 128); else ISA_UNT(float, 64);
  }
#undef ISA_UNT
#undef ISA_UNT1
#undef ISA_UNT2
  return hipGetLastError();
}

}  // namespace isa
