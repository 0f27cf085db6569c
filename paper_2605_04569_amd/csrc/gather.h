// Gathers the block means of one tile of 64 list entries for the attention kernels and the backward pass.
#pragma once

#include "attn_mfma.h"

namespace isa {

struct GatherArgs {
  const float* kc; const float* vc;          // block means, [bh][T_max][128]
  const int* kv_list; const int4* btab;
  uint16_t *kcn, *kcnb, *vcn, *vcnt;         // kcnb, vcn may be null
  float* biasn; int* tflag; int4* ktab;
  Counts cnt;
  int H, Tn_pad, block;
  bool sets;                                 // the problem has exact sets (exact_frac > 0)
};
struct GatherLds { uint16_t vtile[KT][MD + 2]; int ids[KT]; };

// Mean keys (without exact sets: minus the mean key of block 0) / values gathered in kv_list order, rounded to bf16, in the
// layouts the attention kernel reads:
// kcn[bh][t][d], vcn[bh][t][d]; vcnt[bh][t/64][d][pos] with the list position t%64 = key_of_pos16(pos); biasn[bh][t] = ln(n_j) sqrt(D), -inf past T_new.
// `list`: the (batch, head)'s kept blocks.  Called by 256 threads (tid 0..255, the first 64 of them one wave); every thread of the workgroup calls it together (it has two
// barriers), those whose tile does not exist with on = false.
__device__ __forceinline__ void gather_tile(const GatherArgs& a, GatherLds& sm, const int* list, const int tid, const int tile, const int h,
                                            const int b, const bool on) {
  uint16_t (&vtile)[KT][MD + 2] = sm.vtile;
  int (&ids)[KT] = sm.ids;
  const float* const kc = a.kc; const float* const vc = a.vc;
  const Counts& cnt = a.cnt;
  const int Tn_pad = a.Tn_pad, block = a.block, H = a.H;
  const bool sets = a.sets;
  uint16_t* const kcn = a.kcn; uint16_t* const kcnb = a.kcnb; uint16_t* const vcn = a.vcn;
  const int T_new = cnt.b[b].T_new, T_max = cnt.T_max;
  const long long bh = (long long)b * H + h;
  const int t0 = tile * KT;
  if (on && tid < KT) {               // one wave
    const int t = t0 + tid;
    const int j = t < T_new ? block_in_range(list[t], cnt.b[b].T) : -1;
    ids[tid] = j;
    int4 row = make_int4(0, 0, 0, 0);
    if (j >= 0) {
      row = a.btab[b * T_max + j];
      a.ktab[bh * T_max + t] = row;
    }
    // ln(n_j) * sqrt(D): added to the raw score q.k, it becomes ln(n_j) after the 1/sqrt(D) scaling.  Without exact sets
    // (no token keys beside the mean keys) a common factor of the weights cancels in the softmax: ln(n_j / block) is
    // stored instead, which is exactly 0 for full blocks, and tiles of nothing but full blocks take the kernel's plain path
    // (the log-sum-exp the forward hands to the backward is then short of ln(block); the backward uses the same terms).
    const int n_j = row.y;
    const float shift = sets ? 0.f : logf((float)block);
    a.biasn[bh * Tn_pad + t] = j >= 0 ? (n_j == block && !sets ? 0.f : (logf((float)n_j) - shift) * sqrtf((float)MD)) : -INFINITY;
    // every mean key of the tile exists and stands for a full block
    const unsigned long long plain = __ballot(n_j == block);
    if (tid == 0) a.tflag[bh * (Tn_pad / KT) + tile] = !sets && plain == ~0ull ? 0 : 1;
  }
  __syncthreads();
  // A vector common to all keys of a softmax changes nothing, so the mean key of block 0 (a source block, always
  // kept) is subtracted before the rounding to bf16: a component common to all keys (an offset of many standard
  // deviations costs 2^-9 of itself per channel otherwise) then does not eat the precision of what distinguishes
  // them.  Without exact sets the mean keys are the only keys of a Taylor row and nothing else is needed.  With exact
  // sets they share a softmax with token keys: the 4-wave kernel and the backward kernels add each query's product
  // with the subtracted vector (q . Kc_0, kept per query row) back onto its mean-key scores; kcnb is the copy without
  // the subtraction, which the backward's dQ multiplies dS with.
  //
  // Latency-bound (a workgroup's chain is list entry -> block row -> mean rows -> transposed store): a thread has its
  // loads of all four rows in flight at once, 8 channels of a row each.  40 heads of 288 kept blocks, exact sets: 37 -> 13 us; one
  // tile of means: 12.8 -> 7.5 us
  if (on) {
  const int c8 = tid & 15, r0 = tid >> 4;          // 8 channels; rows r0, r0 + 16, r0 + 32, r0 + 48
  float kz[8], kr[4][8], vr[4][8];
  auto load8 = [](const float* p, float (&o)[8]) {
    const float4 lo = *reinterpret_cast<const float4*>(p), hi = *reinterpret_cast<const float4*>(p + 4);
    o[0] = lo.x; o[1] = lo.y; o[2] = lo.z; o[3] = lo.w;
    o[4] = hi.x; o[5] = hi.y; o[6] = hi.z; o[7] = hi.w;
  };
  load8(kc + bh * T_max * MD + 8 * c8, kz);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const long long at = (bh * T_max + max(ids[r0 + 16 * i], 0)) * MD + 8 * c8;      // padding reads block 0, writes zeros
    load8(kc + at, kr[i]);
    load8(vc + at, vr[i]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + 16 * i;
    const bool real = ids[r] >= 0;
    uint32_t kd[4], kw[4], vw[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      auto pack = [&](float x, float y) { return real ? f2bf(x) | ((uint32_t)f2bf(y) << 16) : 0u; };
      kd[e] = pack(kr[i][2 * e] - kz[2 * e], kr[i][2 * e + 1] - kz[2 * e + 1]);
      kw[e] = pack(kr[i][2 * e], kr[i][2 * e + 1]);
      vw[e] = pack(vr[i][2 * e], vr[i][2 * e + 1]);
      *reinterpret_cast<uint32_t*>(&vtile[r][8 * c8 + 2 * e]) = vw[e];
    }
    const long long to = (bh * Tn_pad + t0 + r) * MD + 8 * c8;
    *reinterpret_cast<uint4*>(kcn + to) = make_uint4(kd[0], kd[1], kd[2], kd[3]);
    if (kcnb) *reinterpret_cast<uint4*>(kcnb + to) = make_uint4(kw[0], kw[1], kw[2], kw[3]);
    if (vcn) *reinterpret_cast<uint4*>(vcn + to) = make_uint4(vw[0], vw[1], vw[2], vw[3]);       // the backward pass streams them
  }
  }
  __syncthreads();
  if (!on) return;
  const long long out_off = (bh * (Tn_pad / KT) + tile) * (MD * KT);
#pragma unroll
  for (int x = tid; x < MD * 8; x += 256) {                // 16 bytes: 8 positions of one channel
    const int d = x >> 3, p8 = (x & 7) * 8;
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = vtile[key_of_pos16(p8 + 2 * e)][d] | ((uint32_t)vtile[key_of_pos16(p8 + 2 * e + 1)][d] << 16);
    *reinterpret_cast<uint4*>(a.vcnt + out_off + d * KT + p8) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// the arguments of the gather for `pr` (attn_mfma.hip)
GatherArgs gather_args(const Problem& pr, const Workspace& ws, const float* kc, const float* vc, const int* kv_list);

}  // namespace isa
