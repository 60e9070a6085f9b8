// The binomial payload's call form (BinomialCallTile) in the engine's
// persistent and plain kernels (its long tiles are always dealt by tickets, so
// the direct kernel never runs it). A translation unit of its own: its unrolled levels are most of the
// library's device code.
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "device_atomics.hpp"
#include "device_tiles.hpp"
#include "kernels.hpp"
#include "sched_device.hpp"

namespace ce {

namespace {
BinomialCallTile make_call(const KernelArgs& a) {
  return BinomialCallTile{a.bin, (const float4*)a.in0, (const float*)a.in1, (float4*)a.out};
}
}  // namespace

uint32_t binomial_call_tiles(const KernelArgs& a, uint64_t g0, uint64_t g1) { return make_call(a).ntiles(g0, g1); }

hipError_t binomial_call_blocks_per_cu(int* blocks) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_persistent<BinomialCallTile>, kBlockThreads, 0);
}

void launch_binomial_call_persistent(const KernelArgs& a, const SchedArgs& s, uint32_t grid, hipStream_t st) {
  hipLaunchKernelGGL(k_persistent<BinomialCallTile>, dim3(grid), dim3(kBlockThreads), 0, st, make_call(a), s);
}

void launch_binomial_call_bare(const KernelArgs& a, uint64_t G, uint32_t tiles, hipStream_t st) {
  hipLaunchKernelGGL(k_bare<BinomialCallTile>, dim3(tiles), dim3(kBlockThreads), 0, st, make_call(a), G);
}

}  // namespace ce
