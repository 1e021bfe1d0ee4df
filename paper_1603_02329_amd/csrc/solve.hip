// Host side of the resident solves (passes_solve.h).
#include "passes_common.h"
#include "solve.h"

namespace pat {

hipError_t launch_solve_fwd_32(int nx, int lossy, const SolveArgs& a, hipStream_t st);
hipError_t launch_solve_adj_32(int nx, int lossy, const SolveArgs& a, hipStream_t st);
hipError_t launch_solve_fwd_64(int nx, int lossy, const SolveArgs& a, hipStream_t st);
hipError_t launch_solve_adj_64(int nx, int lossy, const SolveArgs& a, hipStream_t st);
hipError_t launch_solve_fwd_128(int nx, int lossy, const SolveArgs& a, hipStream_t st);
hipError_t launch_solve_adj_128(int nx, int lossy, const SolveArgs& a, hipStream_t st);
hipError_t launch_solve_fwd_256(int nx, int lossy, const SolveArgs& a, hipStream_t st);
hipError_t launch_solve_adj_256(int nx, int lossy, const SolveArgs& a, hipStream_t st);
hipError_t launch_solve_fwd_512(int nx, int lossy, const SolveArgs& a, hipStream_t st);
hipError_t launch_solve_adj_512(int nx, int lossy, const SolveArgs& a, hipStream_t st);

// clears the control block, a few thousand words, and marks the instances
__global__ void __launch_bounds__(256) k_solve_clear(uint32_t* w, int n, const DevPlan* const* list, int count,
                                                     int32_t* open) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  for (int i = t; i < n; i += gridDim.x * 256) w[i] = 0;
  if (!list) {
    if (t == 0) *open = (int32_t)kSolveOpen;
  } else {
    for (int i = t; i < count; i += gridDim.x * 256) list[i]->bad[kBadOpen] = (int32_t)kSolveOpen;
  }
}

namespace {
constexpr int kMaxDevices = 64;
const Tw* g_table[kMaxDevices];  // the twiddle table's address, per device
}  // namespace

hipError_t launch_solve(int nx, int ny, int dir, int lossy, SolveArgs a, int32_t* open, hipStream_t st) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices || !g_table[dev]) return hipErrorNotInitialized;
  a.tw = g_table[dev];
  const int words = (int)(solve_ctl_bytes(a.domains) / 4);
  hipLaunchKernelGGL(k_solve_clear, dim3((words + 1023) / 1024), dim3(256), 0, st, (uint32_t*)a.ctl, words,
                     a.list, a.first[kSolveXcds], open);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  switch (ny) {
    case 32: return dir == 0 ? launch_solve_fwd_32(nx, lossy, a, st) : launch_solve_adj_32(nx, lossy, a, st);
    case 64: return dir == 0 ? launch_solve_fwd_64(nx, lossy, a, st) : launch_solve_adj_64(nx, lossy, a, st);
    case 128: return dir == 0 ? launch_solve_fwd_128(nx, lossy, a, st) : launch_solve_adj_128(nx, lossy, a, st);
    case 256: return dir == 0 ? launch_solve_fwd_256(nx, lossy, a, st) : launch_solve_adj_256(nx, lossy, a, st);
    case 512: return dir == 0 ? launch_solve_fwd_512(nx, lossy, a, st) : launch_solve_adj_512(nx, lossy, a, st);
    default: return hipErrorInvalidValue;
  }
}

// (under the caller's lock, before the first plan of a device exists)
hipError_t upload_twiddles_solve(const Tw* host) {
  int dev = 0;
  void* p = nullptr;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess && (dev < 0 || dev >= kMaxDevices)) e = hipErrorInvalidDevice;
  if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(g_tw), host, sizeof(Tw) * TWN, 0, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_tw));
  if (e == hipSuccess) g_table[dev] = (const Tw*)p;
  return e;
}

}  // namespace pat
