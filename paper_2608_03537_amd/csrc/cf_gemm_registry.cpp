// Registry of the compiled GEMM kernels and their launcher.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <mutex>
#include <vector>

#include "cf_internal.h"

namespace cf {

// Every compiled kernel, and its index by (fp32 input, tile rows, tile columns,
// main loop, epilogue, pair): planning a call looks up about twenty candidates, which
// a search of the table made a noticeable part of a short call's host time.
namespace {
struct Registry {
  std::vector<GemmKernel> all;
  std::array<int16_t, 2 * 2 * 4 * 8 * 3 * 4> index;
  static int key(int in_f32, int tm, int tn, int loop, int epi, int pair) {
    const int r = tm == 32 ? 0 : tm == 64 ? 1 : tm == 128 ? 2 : tm == 256 ? 3 : -1;
    const int c = tn == 32 ? 0 : tn == 64 ? 1 : tn == 128 ? 2 : tn == 192 ? 3 : tn == 256 ? 4 : tn == 384 ? 5
                  : tn == 512 ? 6 : tn == 768 ? 7 : -1;
    if (r < 0 || c < 0 || loop < 0 || loop > 2 || epi < 0 || epi > 3) return -1;
    return ((((pair * 2 + (in_f32 != 0)) * 4 + r) * 8 + c) * 3 + loop) * 4 + epi;
  }
  Registry() {
    index.fill(-1);
    for (auto get : {gemm_kernels_v2, gemm_kernels_v1, gemm_kernels_wr, gemm_kernels_split, gemm_kernels_kn,
                     gemm_kernels_big, gemm_kernels_small}) {
      int n = 0;
      const GemmKernel* k = get(&n);
      all.insert(all.end(), k, k + n);
    }
    for (size_t i = 0; i < all.size(); ++i) {
      const int q = key(all[i].in_f32, all[i].tm, all[i].tn, all[i].loop, all[i].epi, all[i].pair);
      if (q >= 0 && index[q] < 0) index[q] = (int16_t)i;
    }
  }
};
const Registry& registry() {
  static const Registry r;
  return r;
}
const std::vector<GemmKernel>& table() { return registry().all; }
}  // namespace

int find_gemm_kernel(int in_f32, int tm, int tn, int loop, int epi, int pair) {
  const int q = Registry::key(in_f32, tm, tn, loop, epi, pair);
  return q < 0 ? -1 : registry().index[q];
}

const GemmKernel& gemm_kernel(int idx) { return table()[idx]; }

int resident_wgs(int idx) {
  static std::mutex mu;
  static std::vector<int> cache;
  std::lock_guard<std::mutex> lock(mu);
  if (cache.empty()) cache.assign(table().size(), 0);
  if (idx < 0 || idx >= (int)cache.size()) return 0;
  if (cache[idx]) return cache[idx];
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  const GemmKernel& k = table()[idx];
  // Both forms must fit: the one-tile form runs when the grid is not capped.
  int per_cu_persist = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k.fn, k.threads, 0) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_persist, k.fn_persist, k.threads, 0) != hipSuccess)
    return 0;
  cache[idx] = cus * std::min(per_cu, per_cu_persist);
  return cache[idx];
}

hipError_t launch_gemm_rows(const GemmRowsParams& p, int idx, hipStream_t st) {
  const GemmKernel& k = table()[idx];
  // 256-row tiles and small tiles without row clusters have one workgroup per
  // tile, the others a whole number of row-block slots.
  unsigned wgs = (unsigned)(8 * p.slots * p.cn);
  if (k.tm == 256 || (k.epi == 3 && p.mode != ROWS_CLUSTER)) wgs = (unsigned)(p.num_rb * p.cn);
  dim3 grid(wgs, (unsigned)p.batch);
  dim3 block((unsigned)k.threads);
  void* args[] = {const_cast<GemmRowsParams*>(&p)};
  // Without row clusters every tile has a workgroup of its own (grouped
  // order); with them, workgroups loop only when the grid was capped below
  // one slot per row block of each XCD.
  const bool persist = p.mode == ROWS_CLUSTER && (int64_t)p.slots * 8 < (int64_t)p.num_rb;
  return hipLaunchKernel(persist ? k.fn_persist : k.fn, grid, block, args, 0, st);
}

}  // namespace cf
