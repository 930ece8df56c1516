// The launches that the gather of kept rows asks for, recorded instead of made: this program defines the runtime's launch entry itself, so
// that the library's calls end here and no GPU is needed.  A launch may hold fewer than 2^32 work items in a dimension.
// Usage: launch_record problems kv_heads n_tokens budget page_size.  Prints "status <s> launches <n> workgroups <sum> largest <most>".
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "rkv.h"

static long long launches = 0, workgroups = 0, largest = 0;
static hipError_t last = hipSuccess;
static dim3 grid_of, block_of;

extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
  grid_of = grid; block_of = block;
  return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = grid_of; *block = block_of; *shared = 0; *stream = nullptr;
  return hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
  if ((unsigned long long)grid.x * block.x >= 1ull << 32 || grid.x == 0 || grid.y != 1 || grid.z != 1) return last = hipErrorInvalidConfiguration;
  ++launches;
  workgroups += grid.x;
  if (grid.x > largest) largest = grid.x;
  return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  rkv_params p;
  std::memset(&p, 0, sizeof p);
  p.num_problems = std::atoi(argv[1]); p.kv_heads = p.q_heads = std::atoi(argv[2]); p.n_tokens = std::atoi(argv[3]); p.budget = std::atoi(argv[4]);
  p.head_dim = 128; p.alpha = 8; p.pool_w = 4; p.beta = 1; p.sim_threshold = 0.5f; p.lambda = 0.1f; p.eps = 1e-8f;
  if ((p.page_size = std::atoi(argv[5])) != 0) {
    p.table_stride = p.n_tokens / p.page_size + 1;
    p.block_table = reinterpret_cast<const int32_t*>(0x1000);
    p.k_stride_token = p.v_stride_token = 128;
    p.k_stride_head = p.v_stride_head = 128 * p.page_size;
    p.k_stride_page = p.v_stride_page = p.k_stride_head * p.kv_heads;
  }
  void* fake = reinterpret_cast<void*>(0x1000);
  const rkv_status s = rkv_compact(&p, fake, fake, static_cast<const int32_t*>(fake), fake, fake, nullptr);
  std::printf("status %d launches %lld workgroups %lld largest %lld\n", (int)s, launches, workgroups, largest);
  return 0;
}
