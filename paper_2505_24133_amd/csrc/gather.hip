// Compaction (Alg. 1, gather + concatenate): out[head][r][:] = in[head][kept[head][r]][:] for K and V
// in one launch (the largest in several).  A row is 256 bytes = 16 lanes x 16 bytes; each thread moves one such piece of K and of V, and what is
// in flight on a compute unit are its 32 waves.  Pure HBM traffic; the stores are non-temporal (the
// compacted rows are not read again by this step, and keeping them out of the caches is worth 15 % of
// the kernel's time).
// One row a thread instead of four whose indices (and pages) were asked for one after the other, us of the gather alone: 256 heads,
// budget 1024 39.1 -> 38.8, 4096 180 -> 177, paged 2048 121 -> 92, 2 heads of 256 4.6 -> 2.8; two or four rows with all indices
// first lie between.  In a step, with the orders and loads of gather_index.h: 38.3, 144 and 80.
#include <algorithm>

#include "gather_index.h"
#include "rkv_internal.h"

namespace rkv {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // a type the non-temporal builtins accept

constexpr int kGatherThreads = 256;
constexpr int kRowsPerBlock = kGatherThreads / 16;
// A launch takes fewer than 2^32 work items in a dimension.  Calls with more blocks are made in several launches, each of a multiple
// of 8 workgroups so that the next one's begin at the same XCD, up to the number of rows that one launch of 64 rows a block takes (2^30,
// 512 GB of outputs).
constexpr int64_t kMaxBlocks = (1ll << 32) / kGatherThreads - 8;
constexpr int64_t kMaxBlocksOf64 = (1ll << 32) / kGatherThreads - 1;

struct GatherArgs {
  const uint16_t* k;
  const uint16_t* v;
  const int32_t* kept;
  uint16_t* k_out;
  uint16_t* v_out;
  int heads, H, N, budget;
  uint32_t blocks_per_head, eights, run, step;
  uint32_t first;              // block of the whole call that this launch begins with
  KvLayout kl, vl;
  int64_t osp, osh, ost;
};

template <bool PAGED, bool STREAM>
__global__ __launch_bounds__(kGatherThreads) void gather_kernel(GatherArgs a) {
  int head, blk;
  gather_piece(a.first + blockIdx.x, a.blocks_per_head, a.eights, a.run, a.step, head, blk);
  if (head >= a.heads) return;
  const int p = head / a.H;
  const int h = head - p * a.H;
  const int c16 = threadIdx.x & 15;
  const int row = blk * kRowsPerBlock + (threadIdx.x >> 4);
  if (row >= a.budget) return;
  const int src = min(max(a.kept[(int64_t)head * a.budget + row], 0), a.N - 1);
  int64_t ko, vo;
  if constexpr (PAGED) {
    const int64_t page = a.kl.table[(int64_t)p * a.kl.table_stride + (src >> a.kl.page_shift)];
    const int64_t in_page = src & ((1 << a.kl.page_shift) - 1);
    ko = page * a.kl.spage + h * a.kl.sh + in_page * a.kl.st;
    vo = page * a.vl.spage + h * a.vl.sh + in_page * a.vl.st;
  } else {
    ko = p * a.kl.sp + h * a.kl.sh + (int64_t)src * a.kl.st;
    vo = p * a.vl.sp + h * a.vl.sh + (int64_t)src * a.vl.st;
  }
  const u32x4* kp = reinterpret_cast<const u32x4*>(a.k + ko + c16 * 8);
  const u32x4* vp = reinterpret_cast<const u32x4*>(a.v + vo + c16 * 8);
  const u32x4 kr = STREAM ? __builtin_nontemporal_load(kp) : *kp;
  const u32x4 vr = STREAM ? __builtin_nontemporal_load(vp) : *vp;
  const int64_t o = p * a.osp + h * a.osh + (int64_t)row * a.ost + c16 * 8;
  __builtin_nontemporal_store(kr, reinterpret_cast<u32x4*>(a.k_out + o));
  __builtin_nontemporal_store(vr, reinterpret_cast<u32x4*>(a.v_out + o));
}

}  // namespace

hipError_t launch_gather(const Plan& pl, const void* k, const void* v, const int32_t* kept_idx,
                         void* k_out, void* v_out, hipStream_t stream) {
  GatherArgs a;
  a.k = static_cast<const uint16_t*>(k);
  a.v = static_cast<const uint16_t*>(v);
  a.kept = kept_idx;
  a.k_out = static_cast<uint16_t*>(k_out);
  a.v_out = static_cast<uint16_t*>(v_out);
  a.heads = pl.heads; a.H = pl.H; a.N = pl.N; a.budget = pl.budget;
  a.blocks_per_head = (uint32_t)(((int64_t)pl.budget + kRowsPerBlock - 1) / kRowsPerBlock);
  a.kl = k_layout(pl); a.vl = v_layout(pl);
  a.osp = pl.osp; a.osh = pl.osh; a.ost = pl.ost;
  if (pl.heads * (((int64_t)pl.budget + 63) / 64) > kMaxBlocksOf64) return hipErrorInvalidConfiguration;
  const GatherOrder order = gather_order(pl.heads, a.blocks_per_head, gather_cache_bytes(pl.heads, pl.N));
  a.eights = order.eights; a.run = order.run; a.step = order.step;
  auto launch = [&](auto kernel) {
    hipError_t e = hipSuccess;
    for (int64_t first = 0; first < order.blocks && e == hipSuccess; first += kMaxBlocks) {
      a.first = (uint32_t)first;
      hipLaunchKernelGGL(kernel, dim3((unsigned)std::min(order.blocks - first, kMaxBlocks)), dim3(kGatherThreads), 0, stream, a);
      e = hipGetLastError();
    }
    return e;
  };
  if (gather_streams(pl.heads, pl.N, pl.budget, pl.paged)) return launch(pl.paged ? gather_kernel<true, true> : gather_kernel<false, true>);
  return launch(pl.paged ? gather_kernel<true, false> : gather_kernel<false, false>);
}

}  // namespace rkv
