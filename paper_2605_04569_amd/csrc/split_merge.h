// The work items of the exact branch (k_attn_sp) that several kernels need to find, and the merge of those that ran as several key ranges.
#pragma once

#include "attn_mfma.h"

namespace isa {

// The `item`-th of an XCD's long items: its (batch, head) and pair; false past the last.  Batch items alike: the XCD's range of all pairs
// in the order of xcd_first and head_at.  A ragged batch: an equal range of every batch item's own pairs, longest key lists first, as
// nothing levels the end of a launch that starts a long item late.  (Through the heads of all batch items as they come, dense attention of
// 12 heads, items of 3000, 100 and 1620 tokens in this order / the longest last, took 146 / 144 us and takes 96 / 95; 3 heads of 6000 and
// 1500 tokens 151 -> 98, 19 heads 482 -> 375; every eighth head an XCD's took 135 / 104, 154, 483.)
__device__ __forceinline__ bool long_item_at(const MfmaArgs& a, int xcd, int item, int& bhid, int& slot) {
  const int H = a.geo.H, n_bh = a.geo.B * H;
  if (!a.ragged) {
    const long long total = (long long)n_bh * a.slots_first;
    const int at = xcd_first(total, xcd) + item;
    if (at >= xcd_first(total, xcd + 1)) return false;
    bhid = head_at(at / a.slots_first, n_bh);
    slot = at % a.slots_first;
    return true;
  }
  int at = -1, pairs = 1, b = 0;
#pragma unroll
  for (int i = 0; i < ISA_MAX_BATCH; ++i) {                     // unrolled: the arguments are loaded together
    if (i >= a.geo.B || at >= 0) break;
    const int total = H * a.own_pairs[i], first = total * xcd / N_XCD, last = total * (xcd + 1) / N_XCD;      // at most 8 x 65535 x 2048
    if (item < last - first) {
      at = first + item;
      pairs = a.own_pairs[i];
      b = a.by_length[i];
    }
    item -= last - first;
  }
  if (at < 0) return false;
  bhid = b * H + head_at(at / pairs, H);
  slot = at % pairs;
  return true;
}

// Combines the partial results of the split work items: out = sum_p O_p 2^(m_p - m) / sum_p l_p 2^(m_p - m) with
// m = max_p m_p (the merge step of the online softmax, Alg. 2 Part A).  One workgroup of 256 threads per (XCD, split item, block of the
// pair, RM x 8 query rows); 32 threads per row, 4 channels each.
template <int RM>
__device__ __forceinline__ void split_merge(const MfmaArgs& a, const int wg) {
  constexpr int PER = 16 / RM;
  const int grp = wg / PER & 1, split_slot = wg / (2 * PER);
  int slot, bhid;
  if (a.long_ctr) {
    const int item = a.ctr_whole + split_slot;
    slot = item % a.slots_first;
    bhid = item / a.slots_first;
  } else {
    const int r = split_slot % a.n_split, xcd = split_slot / a.n_split;
    if (!long_item_at(a, xcd, a.n_long - a.n_split + r, bhid, slot)) return;
  }
  const int h = bhid % a.geo.H, b = bhid / a.geo.H;
  const BatchCounts c = a.cnt.b[b];
  const int T_max = a.geo.T_max;
  const int n_blocks = a.dense ? c.T : c.n_full;
  const int entry = 2 * slot + grp;
  if (entry >= n_blocks) return;
  const int qi = a.dense ? entry : block_in_range(a.full_list[(long long)bhid * T_max + entry], c.T);
  const int n_q = a.blk_n[b * T_max + qi], q_start = a.blk_start[b * T_max + qi];
  const int ch = (threadIdx.x & 31) * 4;
#pragma unroll
  for (int s = 0; s < RM; ++s) {
  const int row = (wg % PER * RM + s) * 8 + (threadIdx.x >> 5);
  if (row >= n_q) continue;
  const long long sid0 = (long long)split_slot * a.parts * 2 + grp;                    // part p is at sid0 + 2p
  // four parts' loads at a time in flight (a part past the last repeats it, with weight 0)
  float m = M_INIT;
  for (int p0 = 0; p0 < a.parts; p0 += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) m = fmaxf(m, a.split_ml[((sid0 + 2 * min(p0 + u, a.parts - 1)) * 128 + row) * 2]);
  }
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  float l = 0.f;
  for (int p0 = 0; p0 < a.parts; p0 += 4) {
    float2 ml[4];
    float4 o[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long long at = (sid0 + 2 * min(p0 + u, a.parts - 1)) * 128 + row;
      ml[u] = *reinterpret_cast<const float2*>(a.split_ml + at * 2);
      o[u] = *reinterpret_cast<const float4*>(a.split_o + at * MD + ch);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (p0 + u >= a.parts) break;
      const float w = __builtin_amdgcn_exp2f(ml[u].x - m);
      acc.x += w * o[u].x; acc.y += w * o[u].y; acc.z += w * o[u].z; acc.w += w * o[u].w;
      l += w * ml[u].y;
    }
  }
  const float inv = 1.0f / l;
  const long long tbase = (long long)b * a.geo.stride_b + (long long)h * a.geo.stride_h;
  if (a.nlse && ch == 0) a.nlse[(long long)bhid * a.S_max + q_start + row] = -m - __log2f(l);
  acc.x *= inv; acc.y *= inv; acc.z *= inv; acc.w *= inv;
  if (a.ocoarse) {                                           // coarse residual, as in the attention kernel's own store
    const float4 c4 = *reinterpret_cast<const float4*>(a.ocoarse + ((long long)bhid * T_max + qi) * MD + ch);
    acc.x = fmaf(a.gamma, c4.x, acc.x); acc.y = fmaf(a.gamma, c4.y, acc.y);
    acc.z = fmaf(a.gamma, c4.z, acc.z); acc.w = fmaf(a.gamma, c4.w, acc.w);
  }
  uint2 o, cut;
  split_bf16x4(acc, o, cut);
  *reinterpret_cast<uint2*>(a.out + tbase + (long long)(q_start + row) * a.geo.stride_t + ch) = o;
  if (a.olo) *reinterpret_cast<uint2*>(a.olo + ((long long)bhid * a.S_max + q_start + row) * MD + ch) = cut;
  }
}

}  // namespace isa
