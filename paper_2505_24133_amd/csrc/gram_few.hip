// The similarity pass of few heads (one layer a call, small set-ups): a workgroup takes 128 rows against ONE column tile of 128
// keys, so that what a call waits for is one memory latency and four MFMA chains a wave instead of a block of 384 rows with its two
// latencies and twelve chains.  Every row reports the similarity to its most recent partner in the tile (0: none); the
// finalize kernel keeps the most recent tile's.  The products and their order are those of gram.hip.
// Bound: latency.
#include "importance.h"
#include "rkv_internal.h"

namespace rkv {

namespace {

struct FewArgs {
  const uint16_t* k;
  const float* rnorm;
  const float* upart;
  float* sbar;                  // closed-form row sums, by the newest tile's workgroups
  float* part_pre;              // [heads][tiles][n_pad]
  int H, heads, n, n_pad, tiles;
  int64_t ksp, ksh, kst;
  float T, eps;
  ImportanceArgs imp;
};

constexpr int kFewThreads = 256;
static_assert(kFewThreads == kImportanceThreads, "one launch");

__global__ __launch_bounds__(kFewThreads, 4) void gram_few_kernel(FewArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kPseudoBytes + kGramTile * kRowBytes];
  __shared__ float rjs[kGramTile];
  __shared__ float usum[kFewThreads];
  if (a.imp.first != 0 && blockIdx.x >= a.imp.first) {
    importance_block(a.imp, blockIdx.x - a.imp.first, usum);
    return;
  }
  // whole heads per XCD
  const int xcd = blockIdx.x & 7;
  const int q = blockIdx.x >> 3;
  const int per_head = a.tiles * a.tiles;
  const int head = (q / per_head) * 8 + xcd;
  if (head >= a.heads) return;
  const int rem = q % per_head, rb = rem / a.tiles, ct = rem - rb * a.tiles;
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lrow = lane & 31;
  const int half = lane >> 5;
  const int p = head / a.H, n = a.n;
  const uint16_t* kbase = a.k + p * a.ksp + (head - p * a.H) * a.ksh;
  const float* rn = a.rnorm + (int64_t)head * a.n_pad;
  const uint32_t lds0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)lds);
  const uint32_t row_bytes = (uint32_t)a.kst * 2u;
  const bool closing = ct == a.tiles - 1;

  // everything that comes from memory is requested at once
  unsigned char* tile = lds + kPseudoBytes;
#pragma unroll
  for (int jj = 0; jj < 8; ++jj) {
    const int row0 = wave * 4 + jj * 16;
    const int lane_chunk = (lane & 15) ^ ((row0 + (lane >> 4)) & 15);
    dma16(kbase, (uint32_t)gram_copy_row_clamped(ct, kGramTile, row0, lane, n) * row_bytes + (uint32_t)lane_chunk * 16u,
          lds0 + (uint32_t)(kPseudoBytes + row0 * kRowBytes));
  }
  const int row = rb * kGramTile + wave * 32 + lrow, rowc = gram_own_row(row - lrow, lrow, n);
  bf16x8 res[8];
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) {
    const uint4 x = *reinterpret_cast<const uint4*>(kbase + (int64_t)rowc * a.kst + kk * 16 + half * 8);
    __builtin_memcpy(&res[kk], &x, 16);
  }
  const float r = rn[rowc];
  if (t < kGramTile) rjs[t] = rn[ct * kGramTile + t];
  if (closing) {
    // u = sum of the pre-pass's per-chunk partials, grouped as in gram.hip (at most 16 of them)
    const float* up = a.upart + (int64_t)head * a.tiles * kHeadDim + (t & (kHeadDim - 1));
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int c = (t >> 7) + 2 * i;
      x[i] = up[(int64_t)min(c, a.tiles - 1) * kHeadDim];
      x[i] = c < a.tiles ? x[i] : 0.f;
    }
    usum[t] = ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  auto read_k = [&](bf16x8 (&kf)[8], const unsigned char* from, int s) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) kf[kk] = *reinterpret_cast<const bf16x8*>(from + slot_offset(s * 32 + lrow, kk * 2 + half));
  };
  auto chain = [&](const bf16x8 (&kf)[8]) -> f32x16 {
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], res[kk], acc, 0, 0, 0);
    return acc;
  };
  bf16x8 kf[8];
  if (closing) {
    if (t < kHeadDim) {
      float u = usum[t] + usum[t + kHeadDim];
#pragma unroll
      for (int piece = 0; piece < 3; ++piece) {
        uint32_t bits = __float_as_uint(u);
        bits += 0x7fffu + ((bits >> 16) & 1u);                  // round to nearest even bf16
        const uint16_t hb = (uint16_t)(bits >> 16);
        u -= __uint_as_float((uint32_t)hb << 16);               // exact remainder
        *reinterpret_cast<uint16_t*>(lds + slot_offset(piece, t >> 3) + (t & 7) * 2) = hb;
      }
    }
    __syncthreads();
    // K_i . u = the three pseudo-keys' products (elements 0 .. 2 of the lower half of the wave)
    read_k(kf, lds, 0);
    const f32x16 acc = chain(kf);
    if (half == 0 && row < n) a.sbar[(int64_t)head * a.n_pad + row] = mean_sim_closed(r, (acc[2] + acc[1]) + acc[0], a.eps);
  }
  const float thr = row < n ? a.T / r : INFINITY;
  float found = 0.f;
#pragma unroll
  for (int s = 3; s >= 0; --s) {
    read_k(kf, tile, s);
    const f32x16 acc = chain(kf);
    // keys in ascending order within a lane: the last hit met is the most recent; the upper half's rows of four keys lie behind
    // the lower half's, so the two lanes of a row compare keys
    int self = row - (ct * kGramTile + s * 32) - 4 * half;
    asm volatile("" : "+v"(self));
    float best = 0.f;
    int at = -1;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 rj = *reinterpret_cast<const float4*>(rjs + s * 32 + g * 8 + half * 4);
      const float r4[4] = {rj.x, rj.y, rj.z, rj.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = acc[4 * g + i] * r4[i];
        const bool hit = v > thr && 8 * g + i != self;
        best = hit ? v : best;
        at = hit ? 8 * g + i : at;
      }
    }
    const int mine = at < 0 ? -1 : at + 4 * half;
    const auto cols = __builtin_amdgcn_permlane32_swap((unsigned)mine, (unsigned)mine, false, false);
    const auto vals = __builtin_amdgcn_permlane32_swap(__float_as_uint(best), __float_as_uint(best), false, false);
    const bool low = (int)cols[0] > (int)cols[1];
    const float v = __uint_as_float(low ? vals[0] : vals[1]);
    found = found != 0.f ? found : v;                    // a hit exceeds T >= 0
  }
  if (half == 0 && row < n) a.part_pre[((int64_t)head * a.tiles + ct) * a.n_pad + row] = found;
}

}  // namespace

hipError_t launch_gram_few(const Plan& pl, const void* k, char* ws, bool importance, hipStream_t stream) {
  FewArgs a;
  a.k = static_cast<const uint16_t*>(k);
  a.rnorm = reinterpret_cast<const float*>(ws + pl.off_rnorm);
  a.upart = reinterpret_cast<const float*>(ws + pl.off_upart);
  a.sbar = reinterpret_cast<float*>(ws + pl.off_sbar);
  a.part_pre = reinterpret_cast<float*>(ws + pl.off_ppre);
  a.H = pl.H; a.heads = pl.heads; a.n = pl.n; a.n_pad = pl.n_pad; a.tiles = pl.chunks;
  a.ksp = pl.ksp; a.ksh = pl.ksh; a.kst = pl.kst;
  if (pl.paged) {
    // paged cache: the pre-pass left a dense copy of the candidate keys in the workspace
    a.k = reinterpret_cast<const uint16_t*>(ws + pl.off_kdense);
    a.kst = kHeadDim; a.ksh = (int64_t)pl.n_pad * kHeadDim; a.ksp = a.ksh * pl.H;
  }
  a.T = pl.T; a.eps = pl.eps;
  const unsigned blocks = (unsigned)((pl.heads + 7) / 8 * 8 * a.tiles * a.tiles);
  a.imp = importance_args(pl, ws, importance, blocks);
  hipLaunchKernelGGL(gram_few_kernel, dim3(blocks + importance_blocks(pl, a.imp)), dim3(kFewThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace rkv
