// The small stages of ISA: block table, block means (Alg. 1 Stage 1), pooled attention scores with
// context saliency (Sec. 3, Eq. 1) and sharpness (Alg. 1 Stage 3), and the integer selection work
// (Eq. 2, Alg. 1 Stage 3 split, Alg. 2 Stage 2).  All reductions run in a fixed order, so results
// are reproducible from run to run.
#include <hip/hip_bf16.h>

#include "gather.h"

namespace isa {

// ------------------------------------------------------------------------------------------
// helpers
// ------------------------------------------------------------------------------------------
// Reductions over the 64 lanes of a wave, every lane gets the result: partners 32, 16, 8, 4, 2, 1 lanes away in turn.  The halves and the rows
// of 16 lanes meet through the two swap instructions, the lanes of a row by rotating it (by 8, 4, 2, 1: by then the lanes 8, 4, 2
// further on hold the same value, so the rotated lane stands for the exchanged one).  All on the vector unit: through the LDS (ds_bpermute), 16
// waves' reductions of 64-bit numbers were what k_plan spent its time on (whole calls, 5 heads of 9 blocks 38.9 -> 38.1 us, 10 heads of
// 62 blocks 92.8 -> 90.2).
template <int O> __device__ __forceinline__ void partners(uint32_t x, uint32_t& a, uint32_t& b) {
  if constexpr (O == 32) {
    const auto s = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    a = s[0]; b = s[1];
  } else if constexpr (O == 16) {
    const auto s = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    a = s[0]; b = s[1];
  } else {
    a = x;
    b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x120 + O, 0xf, 0xf, true);           // row_ror
  }
}
template <int O> __device__ __forceinline__ float lanes_max(float x) {
  uint32_t a, b;
  partners<O>(__float_as_uint(x), a, b);
  return fmaxf(__uint_as_float(a), __uint_as_float(b));
}
template <int O> __device__ __forceinline__ double lanes_add(double x) {
  uint32_t a0, b0, a1, b1;
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  partners<O>((uint32_t)u, a0, b0);
  partners<O>((uint32_t)(u >> 32), a1, b1);
  return __longlong_as_double((long long)(((unsigned long long)a1 << 32) | a0)) + __longlong_as_double((long long)(((unsigned long long)b1 << 32) | b0));
}
__device__ __forceinline__ double wave_sum(double x) {
  return lanes_add<1>(lanes_add<2>(lanes_add<4>(lanes_add<8>(lanes_add<16>(lanes_add<32>(x))))));
}
__device__ __forceinline__ float wave_max(float x) {
  return lanes_max<1>(lanes_max<2>(lanes_max<4>(lanes_max<8>(lanes_max<16>(lanes_max<32>(x))))));
}

__device__ inline float bf16_bits_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// ------------------------------------------------------------------------------------------
// Block table: token offset and real token count of every block of every batch item.
// ------------------------------------------------------------------------------------------
__global__ void k_layout(SegDesc seg, int block, int T_max, int* blk_start, int* blk_n, int4* btab) {
  const int b = blockIdx.x;
  for (int j = threadIdx.x; j < T_max; j += blockDim.x) {
    int start, n;
    block_place(seg, block, b, j, start, n);
    blk_start[b * T_max + j] = start;
    blk_n[b * T_max + j] = n;
    btab[b * T_max + j] = make_int4(start, n, j, 0);
  }
}

hipError_t launch_layout(const Problem& pr, const Workspace& ws, hipStream_t st) {
  hipLaunchKernelGGL(k_layout, dim3(pr.p.B), dim3(256), 0, st, pr.seg, pr.p.block, pr.cnt.T_max, ws.blk_start, ws.blk_n, ws.btab);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Block means, and the block table (the workgroups of head 0 write it: a launch less than with k_layout in front).  One workgroup per
// (block, head, batch); q, k and v in turn.
// A thread owns VEC consecutive channels (one 16-byte load) of every RP-th row.
// ------------------------------------------------------------------------------------------
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int N = 4;
  __device__ static void load(const float* p, float* o) {
    const float4 v = *reinterpret_cast<const float4*>(p);
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
  }
};
template <> struct Vec16<uint16_t> {   // bf16 storage
  static constexpr int N = 8;
  __device__ static void load(const uint16_t* p, float* o) {
    const uint4 v = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};

template <typename T, int D>
__global__ __launch_bounds__(256) void k_block_means(const T* __restrict__ q, const T* __restrict__ k,
                                                     const T* __restrict__ v, float* __restrict__ qc,
                                                     float* __restrict__ kc, float* __restrict__ vc,
                                                     int* __restrict__ blk_start, int* __restrict__ blk_n,
                                                     int4* __restrict__ btab, SegDesc seg, Geometry g) {
  constexpr int VEC = Vec16<T>::N;
  constexpr int CH = D / VEC;          // 16-byte chunks per row
  constexpr int RP = 256 / CH;         // rows covered per pass
  __shared__ float red[RP][D];
  const int j = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  int start, n;
  block_place(seg, g.block, b, j, start, n);
  if (h == 0 && threadIdx.x == 0) {
    blk_start[b * g.T_max + j] = start;
    blk_n[b * g.T_max + j] = n;
    btab[b * g.T_max + j] = make_int4(start, n, j, 0);
  }
  if (n == 0) return;
  const int c = threadIdx.x % CH, rg = threadIdx.x / CH;
  const long long base = (long long)b * g.stride_b + (long long)h * g.stride_h + (long long)start * g.stride_t + c * VEC;
  const long long obase = (((long long)b * g.H + h) * g.T_max + j) * D;
  const T* src[3] = {q, k, v};
  float* dst[3] = {qc, kc, vc};
  for (int t = 0; t < 3; ++t) {
    float acc[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
    for (int r = rg; r < n; r += RP) {
      float x[VEC];
      Vec16<T>::load(src[t] + base + (long long)r * g.stride_t, x);
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] += x[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < VEC; ++i) red[rg][c * VEC + i] = acc[i];
    __syncthreads();
    if (threadIdx.x < D) {
      float s = 0.f;
#pragma unroll
      for (int r = 0; r < RP; ++r) s += red[r][threadIdx.x];
      dst[t][obase + threadIdx.x] = s / (float)n;
    }
  }
}

hipError_t launch_block_means(const Problem& pr, const Workspace& ws, const void* q, const void* k, const void* v,
                              float* qc, float* kc, float* vc, hipStream_t st) {
  const dim3 grid(pr.cnt.T_max, pr.p.H, pr.p.B), blk(256);
#define ISA_MEANS(T, D)                                                                                        \
  hipLaunchKernelGGL((k_block_means<T, D>), grid, blk, 0, st, (const T*)q, (const T*)k, (const T*)v, qc, kc, vc, \
                     ws.blk_start, ws.blk_n, ws.btab, pr.seg, pr.geo)
  if (pr.p.dtype == ISA_BF16) {
    if (pr.p.D == 128) ISA_MEANS(uint16_t, 128); else ISA_MEANS(uint16_t, 64);
  } else {
    if (pr.p.D == 128) ISA_MEANS(float, 128); else ISA_MEANS(float, 64);
  }
#undef ISA_MEANS
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Pooled attention: rows of S_coarse = softmax_j(qc_i . kc_j / sqrt(D)) (Alg. 1 Stage 1).
// One workgroup computes ROWS rows; it writes the context columns of the source rows to pctx (for
// the column means of Eq. 1) and the sharpness of every row (Alg. 1 Stage 3).
//
// Logits: fp32 matrix instructions (v_mfma_f32_16x16x4_f32), transposed: the 16 rows of the A operand are 16 mean
// keys, the 16 columns of the B operand the workgroup's mean queries, so that a lane ends up with four consecutive
// columns of one row of S_coarse (one 16-byte LDS store).  With l = lane % 16 and g = lane / 16, lane (l, g) feeds
// channel 16 t + 4 g + i of key / query l into step (t, i): one 16-byte load per lane covers four steps.  The mean
// queries stay in registers for the whole workgroup; the four waves take pairs of 16-column tiles in turn.
// Workgroup ids go round-robin over the XCDs, so XCD x sees ids x, x + 8, ...; each XCD owns every 8th
// (batch, head) and works through its heads one after the other: the workgroups that run together read the same
// head's mean keys out of that XCD's L2.
// ------------------------------------------------------------------------------------------
typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int D, int ROWS>
__global__ __launch_bounds__(256) void k_coarse(const float* __restrict__ qc, const float* __restrict__ kc,
                                                float* __restrict__ pctx, float* __restrict__ sharp,
                                                float* __restrict__ z_out, const float* __restrict__ vc,
                                                float* __restrict__ ocoarse, Counts cnt, int B, int H, int Tsrc_max,
                                                int Tctx_max, int zs_stride, int row_tiles) {
  static_assert(ROWS == 8 || ROWS == 16, "a row tile is half or all of the matrix instruction's 16 columns");
  extern __shared__ __attribute__((aligned(16))) float zs[];      // [ROWS][zs_stride]
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int bhid = (slot / row_tiles) * 8 + xcd;
  if (bhid >= B * H) return;
  const int b = bhid / H, i0 = (slot % row_tiles) * ROWS;
  const int T = cnt.b[b].T, T_src = cnt.b[b].T_src, T_max = cnt.T_max;
  if (i0 >= T) return;
  const long long bh = bhid;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l16 = lane & 15, g = lane >> 4;
  const float scale = 1.0f / sqrtf((float)D);
  constexpr int NT = D / 16;                                       // 16-byte loads per lane and row
  __shared__ float rowmax[4][16];
  {
    // mean queries: rows past the batch item's last block repeat it (their logits are never read)
    float4 bq[NT];
    const float* qrow = qc + (bh * T_max + min(i0 + l16, T - 1)) * D + 4 * g;
#pragma unroll
    for (int t = 0; t < NT; ++t)
      bq[t] = (ROWS == 16 || l16 < ROWS) ? *reinterpret_cast<const float4*>(qrow + 16 * t) : make_float4(0.f, 0.f, 0.f, 0.f);
    const int n_ct = (T + 15) / 16;
    // mean keys of the column tiles jt, jt + 1; columns past the last block repeat it, so they change no maximum
    auto load_pair = [&](int jt, float4 (&ak)[2][NT]) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const float* krow = kc + (bh * T_max + min((jt + u) * 16 + l16, T - 1)) * D + 4 * g;
#pragma unroll
        for (int t = 0; t < NT; ++t) ak[u][t] = *reinterpret_cast<const float4*>(krow + 16 * t);
      }
    };
    float rmax = -INFINITY;                                         // over this lane's columns of row l16
    float4 ak[2][NT], ak_next[2][NT];
    load_pair(2 * wave, ak);
    for (int jt = 2 * wave; jt < n_ct; jt += 8) {
      load_pair(jt + 8, ak_next);                                   // the next pair's loads fly under this pair's products
      f32x4_t acc[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(ak[u][t].x, bq[t].x, acc[u], 0, 0, 0);
          acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(ak[u][t].y, bq[t].y, acc[u], 0, 0, 0);
          acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(ak[u][t].z, bq[t].z, acc[u], 0, 0, 0);
          acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(ak[u][t].w, bq[t].w, acc[u], 0, 0, 0);
        }
      // lane (l16, g) holds columns 16 jt + 4 g .. + 3 of row l16; zs_stride covers whole column tiles
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const float4 zv = make_float4(acc[u][0] * scale, acc[u][1] * scale, acc[u][2] * scale, acc[u][3] * scale);
        rmax = fmaxf(fmaxf(rmax, fmaxf(zv.x, zv.y)), fmaxf(zv.z, zv.w));
        if ((ROWS == 16 || l16 < ROWS) && jt + u < n_ct) *reinterpret_cast<float4*>(zs + l16 * zs_stride + (jt + u) * 16 + 4 * g) = zv;
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int t = 0; t < NT; ++t) ak[u][t] = ak_next[u][t];
    }
    rmax = fmaxf(rmax, __shfl_xor(rmax, 16, 64));
    rmax = fmaxf(rmax, __shfl_xor(rmax, 32, 64));
    if (g == 0) rowmax[wave][l16] = rmax;
  }
  __syncthreads();
  // softmax, context columns and sharpness of a row: one wave per row (waves take rows wave, wave + 4, ...), a lane
  // owns the columns lane, lane + 64, ... from here on, so that nothing has to be synchronised between the passes
  // over a row.  Sums in double precision: the variance of a softmax row over hundreds of columns cancels badly in
  // single precision.
  for (int r = wave; r < ROWS; r += 4) {
    const int i = i0 + r;
    if (i >= T) break;                                  // uniform over the wave
    float* zr = zs + r * zs_stride;
    if (z_out)
      for (int j = lane; j < T; j += 64) z_out[(bh * T_max + i) * T_max + j] = zr[j];
    const float m = fmaxf(fmaxf(rowmax[0][r], rowmax[1][r]), fmaxf(rowmax[2][r], rowmax[3][r]));
    // one pass: e = exp(z - m) with the sums of e over all columns, and of e and e^2 over the source columns
    double l = 0.0, l_src = 0.0, q_src = 0.0;
#pragma unroll 4
    for (int j = lane; j < T; j += 64) {
      const float e = expf(zr[j] - m);
      zr[j] = e;
      const double ed = (double)e;
      l += ed;
      if (j < T_src) {
        l_src += ed;
        q_src = fma(ed, ed, q_src);
      }
    }
    l = wave_sum(l);
    l_src = wave_sum(l_src);
    q_src = wave_sum(q_src);
    // sharpness: variance of the row's softmax weights p = e / l over the source columns, E[p^2] - E[p]^2
    const double mu = l_src / l / (double)T_src;
    const double var = q_src / (l * l) / (double)T_src - mu * mu;
    if (lane == 0) sharp[bh * T_max + i] = (float)fmax(var, 0.0);
    const float inv = (float)(1.0 / l);
    // the weights themselves: the context columns of a source row go to pctx (Eq. 1); all of them stay in LDS for
    // the coarse output
    const int j_lo = ocoarse ? 0 : T_src;
    if (ocoarse || i < T_src) {
#pragma unroll 4
      for (int j = j_lo + lane; j < T; j += 64) {
        const float pw = zr[j] * inv;
        zr[j] = pw;
        if (j >= T_src && i < T_src) pctx[(bh * Tsrc_max + i) * Tctx_max + (j - T_src)] = pw;
      }
    }
  }
  // O_coarse = S_coarse V^c (Alg. 1 Stage 1), only when the caller wants the coarse residual: the rows of
  // S_coarse of this workgroup's query blocks are in LDS; one thread per (row, channel), channels fastest
  if (ocoarse) {
    __syncthreads();
    for (int x = threadIdx.x; x < ROWS * D; x += 256) {
      const int r = x / D, ch = x % D;
      if (i0 + r >= T) continue;
      const float* pr = zs + r * zs_stride;
      const float* vcol = vc + bh * T_max * D + ch;
      double acc = 0.0;
      for (int j = 0; j < T; ++j) acc += (double)pr[j] * (double)vcol[(long long)j * D];
      ocoarse[(bh * T_max + i0 + r) * D + ch] = (float)acc;
    }
  }
}

// Eq. 1: mean over the source query blocks of each context column.  64 columns per workgroup; the four waves each add a
// quarter of the rows, and the quarters are added in a fixed order.
__global__ __launch_bounds__(256) void k_colmean(const float* __restrict__ pctx, float* __restrict__ s_ctx, Counts cnt,
                                                 int H, int Tsrc_max, int Tctx_max) {
  __shared__ double part[4][64];
  const int b = blockIdx.z, h = blockIdx.y, lane = threadIdx.x & 63, quarter = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + lane;
  const int T_src = cnt.b[b].T_src, T_ctx = cnt.b[b].T_ctx;
  const long long bh = (long long)b * H + h;
  const int per = (T_src + 3) / 4, i_lo = quarter * per, i_hi = min(T_src, i_lo + per);
  double acc = 0.0;
  if (j < T_ctx)
    for (int i = i_lo; i < i_hi; ++i) acc += (double)pctx[(bh * Tsrc_max + i) * Tctx_max + j];
  part[quarter][lane] = acc;
  __syncthreads();
  if (quarter == 0 && j < T_ctx)
    s_ctx[bh * cnt.T_max + j] = (float)((((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane]) / (double)T_src);
}

template <int D, int ROWS>
static hipError_t launch_coarse_rows(const Problem& pr, const Workspace& ws, const float* qc, const float* kc, float* sharp,
                                     float* z, const float* vc, float* ocoarse, hipStream_t st) {
  const int T_max = pr.cnt.T_max;
  const int zs_stride = ((T_max + 15) / 16) * 16 + 4;          // whole column tiles; + 4 spreads the rows over the banks
  const int row_tiles = (T_max + ROWS - 1) / ROWS;
  const size_t lds = (size_t)ROWS * zs_stride * sizeof(float);
  if (lds > 64 * 1024) {                                        // beyond the default limit of dynamic LDS: ask for it
    hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_coarse<D, ROWS>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (ea != hipSuccess) return ea;
  }
  const int bh = pr.p.B * pr.p.H;
  const unsigned grid = (unsigned)(N_XCD * ((bh + N_XCD - 1) / N_XCD) * row_tiles);
  hipLaunchKernelGGL((k_coarse<D, ROWS>), dim3(grid), dim3(256), lds, st, qc, kc, ws.pctx, sharp, z, vc, ocoarse, pr.cnt,
                     pr.p.B, pr.p.H, pr.Tsrc_max, pr.Tctx_max, zs_stride, row_tiles);
  return hipGetLastError();
}

hipError_t launch_coarse(const Problem& pr, const Workspace& ws, const float* qc, const float* kc, float* s_ctx,
                         float* sharp, float* z, const float* vc, float* ocoarse, hipStream_t st, bool columns) {
  // 16 rows per workgroup (every column of the matrix instruction's B operand in use) while two such workgroups fit
  // a compute unit's LDS; 8 rows for longer rows (up to ISA_MAX_BLOCKS columns: 131 KB)
  const bool wide = (size_t)16 * (((pr.cnt.T_max + 15) / 16) * 16 + 4) * sizeof(float) <= 80 * 1024;
  hipError_t e;
  if (pr.p.D == 128) e = wide ? launch_coarse_rows<128, 16>(pr, ws, qc, kc, sharp, z, vc, ocoarse, st)
                              : launch_coarse_rows<128, 8>(pr, ws, qc, kc, sharp, z, vc, ocoarse, st);
  else e = wide ? launch_coarse_rows<64, 16>(pr, ws, qc, kc, sharp, z, vc, ocoarse, st)
                : launch_coarse_rows<64, 8>(pr, ws, qc, kc, sharp, z, vc, ocoarse, st);
  if (e != hipSuccess || !columns) return e;
  hipLaunchKernelGGL(k_colmean, dim3((pr.Tctx_max + 63) / 64, pr.p.H, pr.p.B), dim3(256), 0, st, ws.pctx, s_ctx, pr.cnt,
                     pr.p.H, pr.Tsrc_max, pr.Tctx_max);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Selection.  One workgroup of 1024 threads per (head, batch, list kind): the kept context blocks (Eq. 2), or the
// split of the query blocks by sharpness (Alg. 1 Stage 3).  Rank of an entry = number of entries that beat it
// (larger score, or equal score and lower index); entries of rank < k are chosen.  Chosen and unchosen indices are
// compacted in ascending order with a block-wide scan.
// ------------------------------------------------------------------------------------------
__device__ inline bool beats(float sa, int ia, float sb, int ib) { return sa > sb || (sa == sb && ia < ib); }

constexpr int SEL_THREADS = 1024;
constexpr int SEL_PARTS = 16;        // lanes that share the count of an entry's rank, each over every 16th of the peers
constexpr int SEL_EACH = 4;          // entries whose ranks a lane counts at once, against the same peers

// flags[j] = 1 for the entries of sc[0..n) that fewer than k others beat.  Integer counts: the result does not depend
// on how the peers are divided among the lanes.  The 16 lanes of an entry read 16 consecutive peers (a contiguous 16th of
// the peers each put them on few LDS banks, on one where n / 16 is a multiple of 32: 40 heads of 512 blocks 68 -> 17 us).
__device__ void rank_flags(const float* sc, int n, int k, int* flags) {
  const int part = threadIdx.x % SEL_PARTS, first = threadIdx.x / SEL_PARTS;
  constexpr int GROUPS = SEL_THREADS / SEL_PARTS;
  for (int j0 = 0; j0 < n; j0 += GROUPS * SEL_EACH) {                // the same trip count for every thread
    int rank[SEL_EACH];
    float s[SEL_EACH];
#pragma unroll
    for (int u = 0; u < SEL_EACH; ++u) {
      rank[u] = 0;
      s[u] = sc[min(j0 + first + u * GROUPS, n - 1)];
    }
#pragma unroll 4
    for (int x = part; x < n; x += SEL_PARTS) {
      const float v = sc[x];
#pragma unroll
      for (int u = 0; u < SEL_EACH; ++u) rank[u] += beats(v, x, s[u], j0 + first + u * GROUPS) ? 1 : 0;
    }
#pragma unroll
    for (int u = 0; u < SEL_EACH; ++u) {
      const int j = j0 + first + u * GROUPS;
#pragma unroll
      for (int o = SEL_PARTS / 2; o > 0; o >>= 1) rank[u] += __shfl_xor(rank[u], o, 64);
      if (j < n && part == 0) flags[j] = rank[u] < k ? 1 : 0;
    }
  }
}

// flags[0..n) -> ascending indices of flagged entries to out_yes (offset add), of the others to out_no.
__device__ void compact(const int* flags, int n, int add, int* out_yes, int* out_no, int* wsum /* [SEL_THREADS / 64] LDS */) {
  const int chunk = (n + SEL_THREADS - 1) / SEL_THREADS;
  const int lo = min(n, (int)threadIdx.x * chunk), hi = min(n, lo + chunk);
  int c = 0;
  for (int x = lo; x < hi; ++x) c += flags[x];
  // exclusive scan of c over the workgroup: inside a wave with shuffles, then the sums of the waves before this one
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = c;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  __syncthreads();
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  int yes = inc - c;
  for (int w = 0; w < wave; ++w) yes += wsum[w];
  int no = lo - yes;
  for (int x = lo; x < hi; ++x) {
    if (flags[x]) out_yes[yes++] = x + add;
    else if (out_no) out_no[no++] = x + add;
  }
  __syncthreads();
}

// Short problems (SMALL: at most 256 source and 256 context blocks, 256 kept ones): the workgroup of the context blocks also
// takes the column means of Eq. 1 from pctx (in the order of k_colmean) before it selects, and gathers the means of the
// blocks it kept (four tiles, 256 threads each) afterwards.  One launch instead of three, each of which is all latency there: 5 heads of
// 9 blocks 2.1 + 4.9 + 6.5 us and two launches -> 9.9.
constexpr int SMALL_BLOCKS = 256;
struct SelectSmall {
  const float* pctx; float* s_ctx; int Tsrc_max, Tctx_max;
  int* taylor_ctr;
  GatherArgs g;
};

template <bool SMALL>
__global__ __launch_bounds__(SEL_THREADS) void k_select(const float* s_ctx, const float* __restrict__ sharp,      // s_ctx and kv_list: x has them too
                                                        int* kv_list, int* __restrict__ full_list,
                                                        int* __restrict__ flat_list, Counts cnt, int H, SelectSmall x) {
  extern __shared__ float sm[];
  float* sc = sm;                                   // [T_max]
  int* flags = reinterpret_cast<int*>(sm + cnt.T_max);   // [T_max]
  __shared__ int wsum[SEL_THREADS / 64];
  const int h = blockIdx.x, b = blockIdx.y;
  const BatchCounts c = cnt.b[b];
  const long long bh = (long long)b * H + h, off = bh * cnt.T_max;

  if (blockIdx.z == 0) {       // context blocks by saliency: kv_list = all source blocks, then the kept context blocks
    if constexpr (SMALL) {
      __shared__ double sums[4][SMALL_BLOCKS];
      const int j = threadIdx.x % SMALL_BLOCKS, quarter = threadIdx.x / SMALL_BLOCKS;
      const int per = (c.T_src + 3) / 4, i_lo = quarter * per, i_hi = min(c.T_src, i_lo + per);
      double acc = 0.0;
      if (j < c.T_ctx) {
#pragma unroll 8
        for (int i = i_lo; i < i_hi; ++i) acc += (double)x.pctx[(bh * x.Tsrc_max + i) * x.Tctx_max + j];
      }
      sums[quarter][j] = acc;
      __syncthreads();
      if (quarter == 0 && j < c.T_ctx) {
        sc[j] = (float)((((sums[0][j] + sums[1][j]) + sums[2][j]) + sums[3][j]) / (double)c.T_src);
        x.s_ctx[off + j] = sc[j];
      }
      if (threadIdx.x == 0 && h == 0 && b == 0) *x.taylor_ctr = 0;     // see k_gather_means
    } else {
      for (int j = threadIdx.x; j < c.T_ctx; j += SEL_THREADS) sc[j] = s_ctx[off + j];
    }
    for (int j = threadIdx.x; j < cnt.T_max; j += SEL_THREADS) kv_list[off + j] = j < c.T_src ? j : -1;
    __syncthreads();
    rank_flags(sc, c.T_ctx, c.k_keep, flags);
    __syncthreads();
    compact(flags, c.T_ctx, c.T_src, kv_list + off + c.T_src, nullptr, wsum);
    if constexpr (SMALL) {
      __shared__ GatherLds tiles[SMALL_BLOCKS / KT];
      __threadfence_block();                         // the list as the other threads of this workgroup have just written it
      __syncthreads();
      const int tile = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
      gather_tile(x.g, tiles[tile], kv_list + off, threadIdx.x & 255, tile, h, b, tile < x.g.Tn_pad / KT);
    }
  } else {                     // query blocks by sharpness
    for (int i = threadIdx.x; i < c.T; i += SEL_THREADS) sc[i] = sharp[off + i];
    for (int i = threadIdx.x; i < cnt.T_max; i += SEL_THREADS) {
      full_list[off + i] = -1;
      flat_list[off + i] = -1;
    }
    __syncthreads();
    rank_flags(sc, c.T, c.n_full, flags);
    __syncthreads();
    compact(flags, c.T, 0, full_list + off, flat_list + off, wsum);
  }
}

bool select_is_small(const Problem& pr) {
  return pr.mfma_shape && pr.Tsrc_max <= SMALL_BLOCKS && pr.Tctx_max <= SMALL_BLOCKS && pr.Tn_pad <= SMALL_BLOCKS;
}

// Alg. 2 Stage 2: for the Taylor query block at position r of flat_list, mark the k_exact positions of kv_list with the
// largest coarse logit (ties to the lower position): every entry that fewer than k_exact others beat.
//
// One wave per row, NV entries of the list per lane (position lane + 64 u) as unsigned keys that order like the logits.
// The k-th largest key is found bit by bit, counting with ballots the keys that are not below a candidate: 32 steps of NV
// compares, where counting every entry's rank against all others takes T_new of them.  40 heads of 256 Taylor blocks, 288 kept
// blocks: 133 -> 26 us.  A NaN beats nothing and nothing beats it: it is marked whenever k_exact > 0 and takes nobody's place.
template <int NV>
__device__ __forceinline__ void exact_set(const float* zr, const int* kv, uint32_t* mrow, const BatchCounts& c, int mask_words, int lane) {
  uint32_t key[NV];                                  // 0: past the list, or NaN (every number's key is larger)
  unsigned long long nan[NV];
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const int t = lane + 64 * u;
    const int j = t < c.T_new ? block_in_range(kv[t], c.T) : -1;
    const float x = j >= 0 ? zr[j] + 0.0f : 0.f;     // -0 and 0 tie
    const uint32_t bits = __float_as_uint(x);
    const bool is_nan = x != x;
    key[u] = j < 0 || is_nan ? 0u : (bits & 0x80000000u) ? ~bits : bits | 0x80000000u;
    nan[u] = __ballot(is_nan);
  }
  auto count = [&](uint32_t at_least) {
    int n = 0;
#pragma unroll
    for (int u = 0; u < NV; ++u) n += __popcll(__ballot(key[u] >= at_least));
    return n;
  };
  uint32_t kth = 0u;                                 // the k_exact-th largest key (0: there are fewer numbers)
  for (uint32_t bit = 0x80000000u; bit != 0u; bit >>= 1)
    if (count(kth | bit) >= c.k_exact) kth |= bit;
  // all larger keys, and the first of the equal ones
  int equal = c.k_exact - (kth == 0xffffffffu ? 0 : count(kth + 1u));
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    if (2 * u >= mask_words) break;
    const unsigned long long eq = __ballot(kth != 0u && key[u] == kth);
    const int before = __popcll(eq & ((1ull << lane) - 1ull));
    unsigned long long set = __ballot(key[u] > kth || (kth != 0u && key[u] == kth && before < equal));
    equal -= __popcll(eq);
    if (c.k_exact > 0) set |= nan[u];
    if (lane == 0) mrow[2 * u] = (uint32_t)set;
    if (lane == 1 && 2 * u + 1 < mask_words) mrow[2 * u + 1] = (uint32_t)(set >> 32);
  }
}
template <int NV>
__global__ __launch_bounds__(256) void k_exact_sets(const float* __restrict__ z, const int* __restrict__ kv_list,
                                                    const int* __restrict__ flat_list, uint32_t* __restrict__ mask,
                                                    Counts cnt, int H) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, h = blockIdx.y, b = blockIdx.z;
  const BatchCounts c = cnt.b[b];
  if (r >= c.n_flat) return;                         // uniform over the wave; nothing below synchronises waves
  const long long row0 = ((long long)b * H + h) * cnt.T_max;
  const int i = block_in_range(flat_list[row0 + r], c.T);
  exact_set<NV>(z + (row0 + i) * cnt.T_max, kv_list + row0, mask + (row0 + r) * cnt.mask_words, c, cnt.mask_words, lane);
}

// Everything between the block means and the attention launch for a (batch, head) of at most 64 blocks, in one workgroup of 16 waves: the
// pooled map with its softmax, column means and sharpness (as k_coarse and k_colmean, in the same order of additions), both
// selections (a wave each: a lane per block, ranks by comparing with every other lane, lists by the bits of a ballot), then the gathered means (GATHER:
// the pipelined kernels) beside the exact sets.  All latency at these sizes: 5 heads of 9 blocks k_coarse 6.7 + k_select 10.8 us and the
// launch between them -> 9.9; whole call 44.8 -> 38.1 us.
constexpr int PLAN_BLOCKS = 64;
struct PlanArgs {
  const float *qc, *kc;
  float *s_ctx, *sharp;
  int *kv_list, *full_list, *flat_list;
  uint32_t* exact_mask;                              // null: no exact sets
  int* taylor_ctr;
  GatherArgs g;
  Counts cnt;
  int H;
};

template <int D, bool GATHER>
__global__ __launch_bounds__(1024) void k_plan(PlanArgs a) {
  constexpr int ZS = PLAN_BLOCKS + 4, NT = D / 16;
  __shared__ __attribute__((aligned(16))) float zs[PLAN_BLOCKS * ZS];          // logits
  __shared__ float ps[PLAN_BLOCKS * ZS];                                       // softmax weights of the source rows' context columns
  __shared__ double sums[4][PLAN_BLOCKS];
  __shared__ float sh[PLAN_BLOCKS];
  __shared__ int kvs[PLAN_BLOCKS], flat[PLAN_BLOCKS];
  __shared__ GatherLds tile;
  const int h = blockIdx.x, b = blockIdx.y, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const BatchCounts c = a.cnt.b[b];
  const int T = c.T, T_src = c.T_src;
  const long long row0 = ((long long)b * a.H + h) * a.cnt.T_max;
  if (GATHER && threadIdx.x == 0 && h == 0 && b == 0) *a.taylor_ctr = 0;       // see k_gather_means
  {                                                  // a 16 x 16 tile of the map per wave; operands as in k_coarse
    const int it = wave >> 2, jt = wave & 3, l16 = lane & 15, g = lane >> 4;
    if (it * 16 < T && jt * 16 < T) {
      const float* qrow = a.qc + (row0 + min(it * 16 + l16, T - 1)) * D + 4 * g;
      const float* krow = a.kc + (row0 + min(jt * 16 + l16, T - 1)) * D + 4 * g;
      float4 bq[NT], ak[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        bq[t] = *reinterpret_cast<const float4*>(qrow + 16 * t);
        ak[t] = *reinterpret_cast<const float4*>(krow + 16 * t);
      }
      f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ak[t].x, bq[t].x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ak[t].y, bq[t].y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ak[t].z, bq[t].z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ak[t].w, bq[t].w, acc, 0, 0, 0);
      }
      const float scale = 1.0f / sqrtf((float)D);
      *reinterpret_cast<float4*>(zs + (it * 16 + l16) * ZS + jt * 16 + 4 * g) = make_float4(acc[0] * scale, acc[1] * scale, acc[2] * scale, acc[3] * scale);
    }
  }
  __syncthreads();
  // a row of at most 64 columns per wave, two rows' reductions side by side
  for (int i0 = wave; i0 < T; i0 += 32) {
    float e[2];
    double l[2], l_src[2], q_src[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float zv = lane < T ? zs[min(i0 + 16 * u, T - 1) * ZS + lane] : -INFINITY;
      e[u] = zv - wave_max(zv);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      e[u] = lane < T ? expf(e[u]) : 0.f;
      l[u] = (double)e[u];
      l_src[u] = lane < T_src ? l[u] : 0.0;
      q_src[u] = l_src[u] * l_src[u];
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      l[u] = wave_sum(l[u]);
      l_src[u] = wave_sum(l_src[u]);
      q_src[u] = wave_sum(q_src[u]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int i = i0 + 16 * u;
      if (i >= T) break;
      const double mu = l_src[u] / l[u] / (double)T_src;
      const double var = q_src[u] / (l[u] * l[u]) / (double)T_src - mu * mu;
      if (lane == 0) {
        sh[i] = (float)fmax(var, 0.0);
        a.sharp[row0 + i] = sh[i];
      }
      if (i < T_src && lane >= T_src && lane < T) ps[i * ZS + lane - T_src] = e[u] * (float)(1.0 / l[u]);
    }
  }
  __syncthreads();
  if (wave < 4) {                                    // Eq. 1, a quarter of the source rows per wave (see k_colmean)
    const int per = (T_src + 3) / 4, i_lo = wave * per, i_hi = min(T_src, i_lo + per);
    double acc = 0.0;
    if (lane < c.T_ctx) {
#pragma unroll 8
      for (int i = i_lo; i < i_hi; ++i) acc += (double)ps[i * ZS + lane];
    }
    sums[wave][lane] = acc;
  }
  __syncthreads();
  if (wave < 2) {                                    // wave 0: context blocks by saliency; wave 1: query blocks by sharpness
    const int n = wave == 0 ? c.T_ctx : T, k = wave == 0 ? c.k_keep : c.n_full;
    float s = 0.f;
    if (lane < n) {
      if (wave == 0) {
        s = (float)((((sums[0][lane] + sums[1][lane]) + sums[2][lane]) + sums[3][lane]) / (double)T_src);
        a.s_ctx[row0 + lane] = s;
      } else {
        s = sh[lane];
      }
    }
    int rank = 0;
#pragma unroll 8
    for (int x = 0; x < n; ++x) rank += beats(__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(s), x)), x, s, lane) ? 1 : 0;
    const unsigned long long yes = __ballot(lane < n && rank < k), below = (1ull << lane) - 1ull;
    const int at_yes = __popcll(yes & below), at_no = lane - at_yes;
    const bool chosen = (yes >> lane) & 1ull;
    if (wave == 0) {
      if (lane < T_src) kvs[lane] = lane;
      if (chosen) kvs[T_src + at_yes] = T_src + lane;
      // (the same wave reads what it has just written)
      __builtin_amdgcn_wave_barrier();
      if (lane < a.cnt.T_max) a.kv_list[row0 + lane] = lane < T_src + __popcll(yes) ? kvs[lane] : -1;      // (NaN scores: more than k of them)
    } else if (lane < a.cnt.T_max) {
      const int n_yes = __popcll(yes);
      flat[lane] = -1;
      if (lane >= n_yes) a.full_list[row0 + lane] = -1;
      if (lane >= T - n_yes) a.flat_list[row0 + lane] = -1;
      if (lane < T) {
        (chosen ? a.full_list : a.flat_list)[row0 + (chosen ? at_yes : at_no)] = lane;
        if (!chosen) flat[at_no] = lane;
      }
    }
  }
  __syncthreads();
  if (a.exact_mask && wave >= 4)
    for (int r = wave - 4; r < c.n_flat; r += 12) exact_set<1>(zs + block_in_range(flat[r], T) * ZS, kvs, a.exact_mask + (row0 + r) * a.cnt.mask_words, c, a.cnt.mask_words, lane);
  if (GATHER) gather_tile(a.g, tile, kvs, threadIdx.x & 255, 0, h, b, wave < 4);
}

// One workgroup has all rows of a head to itself, which stops paying off towards 64 blocks unless the exact sets' launch is saved as well.  Whole
// calls, separate launches / one: 10 heads of 33, 48, 62 blocks 66.2 / 61.8, 76.0 / 74.7, 88.5 / 90.2 us, with exact sets 33, 62 blocks 91.7 /
// 77.6, 133.6 / 131.3.  Sources without context have the most rows to add up: 1, 3, 8 heads of 48 blocks 57.5 / 59.7, 63.5 / 65.6, 92.8 / 94.6, of 44
// 57.5 / 58.1, 62.8 / 63.2, 89.6 / 90.3 (half of them context: 59.1 / 58.0, 63.5 / 61.3, 85.6 / 83.3).
bool plan_is_small(const Problem& pr) { return pr.cnt.T_max <= (pr.p.exact_frac > 0.0 ? PLAN_BLOCKS : 44) && pr.p.gamma == 0.0; }

hipError_t launch_plan(const Problem& pr, const Workspace& ws, bool gather, hipStream_t st) {
  PlanArgs a = {ws.qc, ws.kc, ws.s_ctx, ws.sharp, ws.kv_list, ws.full_list, ws.flat_list, pr.p.exact_frac > 0.0 ? ws.exact_mask : nullptr,
                ws.taylor_ctr, {}, pr.cnt, pr.p.H};
  const dim3 grid(pr.p.H, pr.p.B);
  if (gather) {
    a.g = gather_args(pr, ws, ws.kc, ws.vc, ws.kv_list);
    hipLaunchKernelGGL((k_plan<128, true>), grid, dim3(1024), 0, st, a);
  } else if (pr.p.D == 128) {
    hipLaunchKernelGGL((k_plan<128, false>), grid, dim3(1024), 0, st, a);
  } else {
    hipLaunchKernelGGL((k_plan<64, false>), grid, dim3(1024), 0, st, a);
  }
  return hipGetLastError();
}

hipError_t launch_select(const Problem& pr, const Workspace& ws, const float* s_ctx, const float* sharp, const float* z,
                         int* kv_list, int* full_list, int* flat_list, uint32_t* exact_mask, hipStream_t st, bool small) {
  const size_t lds = (size_t)pr.cnt.T_max * 8;
  const dim3 sel_grid(pr.p.H, pr.p.B, 2);
  if (small) {
    const SelectSmall x = {ws.pctx, ws.s_ctx, pr.Tsrc_max, pr.Tctx_max, ws.taylor_ctr, gather_args(pr, ws, ws.kc, ws.vc, kv_list)};
    hipLaunchKernelGGL(k_select<true>, sel_grid, dim3(SEL_THREADS), lds, st, s_ctx, sharp, kv_list, full_list, flat_list, pr.cnt,
                       pr.p.H, x);
  } else {
    hipLaunchKernelGGL(k_select<false>, sel_grid, dim3(SEL_THREADS), lds, st, s_ctx, sharp, kv_list, full_list, flat_list, pr.cnt,
                       pr.p.H, SelectSmall{});
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !(pr.p.exact_frac > 0.0)) return e;
  int nflat_max = 0;
  for (int b = 0; b < pr.p.B; ++b) nflat_max = pr.cnt.b[b].n_flat > nflat_max ? pr.cnt.b[b].n_flat : nflat_max;
  if (nflat_max == 0) return hipSuccess;
  const dim3 grid((nflat_max + 3) / 4, pr.p.H, pr.p.B);
  // the list entries a lane holds: enough for T_max, which bounds the mask row as well
#define ISA_SETS(NV) hipLaunchKernelGGL((k_exact_sets<NV>), grid, dim3(256), 0, st, z, kv_list, flat_list, exact_mask, pr.cnt, pr.p.H)
  if (pr.cnt.T_max <= 256) ISA_SETS(4);
  else if (pr.cnt.T_max <= 512) ISA_SETS(8);
  else if (pr.cnt.T_max <= 1024) ISA_SETS(16);
  else if (pr.cnt.T_max <= 2048) ISA_SETS(32);
  else ISA_SETS(64);
#undef ISA_SETS
  return hipGetLastError();
}

}  // namespace isa
