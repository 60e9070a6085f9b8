// Batched escape-time kernel for gfx950: one launch of as many workgroups as are
// resident runs every job of a batch. The jobs' tiles are concatenated in job
// order and dealt to the workgroups in packages of `pkg_tiles` consecutive tiles
// (dealing.hpp: a dynamic schedule inside the GPU), and each wave takes its parts
// of tiles by itself, without a barrier. A tile's job is found by binary search
// over the jobs' first tiles, kept in LDS, unless it is the wave's last one. The
// per-pixel arithmetic is the same escape_count as the single-job kernels.
// Bound by FP32 issue: 256 jobs of 157 million pixels take 2.5 cycles per vector
// instruction and SIMD, where 2.3 is what eight waves reach.
#include <hip/hip_runtime.h>

#include "batch.hpp"
#include "common.hpp"
#include "device_payloads.hpp"

namespace ce {

template <uint32_t TR>
__global__ __launch_bounds__(kBlockThreads) void k_batch_escape(BatchArgs a) {
  constexpr uint32_t TC = kBlockThreads / TR, kWaves = kBlockThreads / 64;
  // a wave's part of a tile: 16 x 4 pixels, whose orbits are alike in length,
  // or as near to it as the tile's rows allow (256 jobs, tiles of 4 rows: 4.16 ms
  // with 64 pixels of a row, 2.48 so)
  constexpr uint32_t kRows = TR < 4 ? TR : 4, kCols = 64 / kRows, kAcross = TC / kCols;
  extern __shared__ uint64_t sh_base[];  // first tile of each job (n_jobs entries)
  __shared__ DealState deal;
  for (uint32_t j = threadIdx.x; j < a.n_jobs; j += kBlockThreads) sh_base[j] = a.jobs[j].tile_base;
  deal_begin(a.deal, deal);
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t job = 0, part;  // job of this wave's tile, and often of its next
  uint64_t package;
  while (deal_next(a.deal, deal, &package, &part)) {
    const uint64_t t = package * a.pkg_tiles + part / kWaves;
    if (t < sh_base[job] || (job + 1 < a.n_jobs && sh_base[job + 1] <= t)) {
      uint32_t l = 0, h = a.n_jobs;  // sh_base[l] <= t < sh_base[h] (sh_base[n_jobs] = end)
      while (h - l > 1) {
        const uint32_t m = (l + h) >> 1;
        if (sh_base[m] <= t) l = m; else h = m;
      }
      job = __builtin_amdgcn_readfirstlane(l);
    }
    const BatchJob& J = a.jobs[job];
    const uint64_t local = t - J.tile_base;
    uint32_t tx, ty;
    if (local >> 32 == 0) {
      ty = Divisor{J.tiles_x, J.tiles_x_reciprocal}.split((uint32_t)local, &tx);
    } else {
      ty = (uint32_t)(local / J.tiles_x);
      tx = (uint32_t)(local % J.tiles_x);
    }
    const uint32_t w = part % kWaves;
    const uint32_t r = ty * TR + w / kAcross * kRows + lane / kCols, c = tx * TC + w % kAcross * kCols + lane % kCols;
    if (r < J.p.h && c < J.p.w) {
      const float cr = J.p.x0 + (float)c * J.p.dx;
      const float ci = J.p.y0 + (float)r * J.p.dy;
      J.out[(size_t)r * J.p.w + c] = escape_count(cr, ci, J.p.max_iter);
    }
  }
  deal_end(a.deal);
}

uint32_t batch_shape_cols(int shape) { return kBlockThreads / kBatchShapeRows[shape]; }

hipError_t batch_blocks_per_cu(int shape, size_t lds, int* blocks) {
  switch (shape) {
    case 0: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_batch_escape<1>, kBlockThreads, lds);
    case 1: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_batch_escape<2>, kBlockThreads, lds);
    case 2: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_batch_escape<4>, kBlockThreads, lds);
    case 3: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_batch_escape<8>, kBlockThreads, lds);
    case 4: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_batch_escape<16>, kBlockThreads, lds);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_batch(int shape, const BatchArgs& a, uint32_t grid, hipStream_t st) {
  const dim3 g(grid), b(kBlockThreads);
  const size_t lds = (size_t)a.n_jobs * sizeof(uint64_t);
  switch (shape) {
    case 0: hipLaunchKernelGGL(k_batch_escape<1>, g, b, lds, st, a); break;
    case 1: hipLaunchKernelGGL(k_batch_escape<2>, g, b, lds, st, a); break;
    case 2: hipLaunchKernelGGL(k_batch_escape<4>, g, b, lds, st, a); break;
    case 3: hipLaunchKernelGGL(k_batch_escape<8>, g, b, lds, st, a); break;
    case 4: hipLaunchKernelGGL(k_batch_escape<16>, g, b, lds, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace ce
