// The importance of a head's candidates (Eq. 3-4) as extra workgroups of the similarity pass's launch.  It needs the pre-pass
// only, and where a launch of the finalize kernel has no more than one workgroup per compute unit its importance stage is a chain of
// latencies on the critical path.  Beside the similarity pass it fills what that launch leaves idle, and lengthens it where it leaves
// nothing: its workgroups come last in the grid, take the LDS of a scan each and read the logits through the same L2s.
// A step, us, formed by the finalize kernel / here, repeated text at T = 0.5: 2 heads of n = 292 20.7 / 17.8; 8 of n = 1144 26.7 / 23.9, of
// n = 32760 376 / 334; 64 of n = 1144 60.1 / 57.0; 128 of n = 4216 209.5 / 205.8; 256 of n = 1144 107.0 / 103.4.  Where a step streams its
// keys from memory several times nothing is left to gain: 256 heads of n = 2168 201.4 / 200.9, of n = 4216 407.0 / 406.2 (the scan's launch
// 12 longer, the finalize kernel 14 shorter), of n = 8312 1007 / 1008; 224 of n = 4216 353 / 355; 64 of n = 32760 1621 / 1635.
// Noisy copies at T = 0.95, a long scan: 256 of n = 4216 1105 / 1094, of n = 8312 3734 / 3718.  (With thousands of heads the finalize
// kernel's 32 waves a compute unit read the logits faster than the eight that fit beside the similarity pass.)
#pragma once

#include "rkv_internal.h"

namespace rkv {

struct ImportanceArgs {
  const float* logit;    // [heads][8][n_pad]
  const float* stats;    // [heads][groups][8][2]
  float* out;            // [heads][n_pad]
  int groups, n, n_pad;
  int first, per_head;   // first workgroup of the launch that does this (0: none does), workgroups per head
};

constexpr int kImportanceThreads = 256;                  // of a workgroup of the similarity pass, four candidates each

// Default readings with alpha = 8 and W = 4, the operations and their order as in the finalize kernel.  `shared`: 64 bytes of LDS.
__device__ __forceinline__ void importance_block(const ImportanceArgs& a, int block, float* shared) {
  constexpr int A = 8;
  const int t = threadIdx.x, lane = t & 63;
  const int head = block / a.per_head, g = (block - head * a.per_head) * kImportanceThreads + t;
  // the softmax over all candidates, completed from the pre-pass's groups: one wave per window slot, lanes over the groups
  for (int j = t >> 6; j < A; j += kImportanceThreads / 64) {
    const float* st = a.stats + ((int64_t)head * a.groups * A + j) * 2;
    float m = -INFINITY;
    for (int c = lane; c < a.groups; c += 64) m = fmaxf(m, st[(int64_t)c * A * 2]);
    m = full_wave_max(m);
    float den = 0.f;
    for (int c = lane; c < a.groups; c += 64)
      den += st[(int64_t)c * A * 2 + 1] * __expf(st[(int64_t)c * A * 2] - m);
    den = full_wave_sum(den);
    if (lane == 0) {
      shared[j] = m;
      shared[A + j] = 1.0f / (den * (float)A);
    }
  }
  // candidates 4 g .. 4 g + 3 need columns 4 g - 4 .. 4 g + 6 (the last of twelve is not used)
  const float* lg = a.logit + (int64_t)head * A * a.n_pad;
  float x[A][12];
  const bool any = 4 * g < a.n;
#pragma unroll
  for (int j = 0; j < A; ++j)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int col = 4 * g - 4 + 4 * q;
      float4 v = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      if (any && col >= 0 && col < a.n) v = *reinterpret_cast<const float4*>(lg + (int64_t)j * a.n_pad + col);
      x[j][4 * q] = v.x;
      x[j][4 * q + 1] = col + 1 < a.n ? v.y : -INFINITY;
      x[j][4 * q + 2] = col + 2 < a.n ? v.z : -INFINITY;
      x[j][4 * q + 3] = col + 3 < a.n ? v.w : -INFINITY;
    }
  __syncthreads();
  if (!any) return;
  float imp[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < A; ++j) {
    float inner = x[j][3];                                 // entries 3 .. 7 belong to all four windows
#pragma unroll
    for (int c = 4; c < 8; ++c) inner = fmaxf(inner, x[j][c]);
    const float o0 = fmaxf(fmaxf(inner, x[j][0]), fmaxf(x[j][1], x[j][2]));
    const float o1 = fmaxf(fmaxf(inner, x[j][1]), fmaxf(x[j][2], x[j][8]));
    const float o2 = fmaxf(fmaxf(inner, x[j][2]), fmaxf(x[j][8], x[j][9]));
    const float o3 = fmaxf(fmaxf(inner, x[j][8]), fmaxf(x[j][9], x[j][10]));
    const float gm = shared[j], gi = shared[A + j];
    imp[0] += __expf(o0 - gm) * gi;
    imp[1] += __expf(o1 - gm) * gi;
    imp[2] += __expf(o2 - gm) * gi;
    imp[3] += __expf(o3 - gm) * gi;
  }
  *reinterpret_cast<float4*>(a.out + (int64_t)head * a.n_pad + 4 * g) = make_float4(imp[0], imp[1], imp[2], imp[3]);
}

// Workgroups that a launch of `gram_blocks` similarity workgroups is followed by.
inline ImportanceArgs importance_args(const Plan& pl, char* ws, bool with, unsigned gram_blocks) {
  ImportanceArgs a = {};
  if (!with) return a;
  a.logit = reinterpret_cast<const float*>(ws + pl.off_logit);
  a.stats = reinterpret_cast<const float*>(ws + pl.off_stats);
  a.out = reinterpret_cast<float*>(ws + pl.off_imp);
  a.groups = pl.chunks * (prepass_register_path(pl) ? 4 : 1);
  a.n = pl.n; a.n_pad = pl.n_pad;
  a.first = (int)gram_blocks;
  a.per_head = (pl.n + 4 * kImportanceThreads - 1) / (4 * kImportanceThreads);
  return a;
}
inline unsigned importance_blocks(const Plan& pl, const ImportanceArgs& a) { return (unsigned)(pl.heads * a.per_head); }

}  // namespace rkv
