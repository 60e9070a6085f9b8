// GPU side of the co-execution engine for gfx950 (CDNA4).
//
// One persistent kernel per payload pulls packages of the index space from a
// two-level dispenser (section 5.3 schedulers, section 4.2 architecture):
//  - level 1 lives in host-coherent pinned memory and is shared with the host
//    worker pool; the GPU reaches it with system-scope atomics over PCIe;
//  - level 2 lives in HBM: a ticket counter hands the tiles of the GPU's
//    current package to its workgroups with device-scope atomics.
// The workgroup whose ticket is the first one past the published tiles is the
// only one that claims the next level-1 package, so the GPU acts as a single
// device towards the scheduler while all its workgroups share each package.
//
// Payload arithmetic is written one FP32 operation at a time and compiled
// with -ffp-contract=off, so every work-item gets the same bits as on the
// host workers.
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "device_payloads.hpp"
#include "device_atomics.hpp"
#include "device_divide.hpp"
#include "device_tiles.hpp"
#include "kernels.hpp"
#include "rt_tile.hpp"
#include "sched_device.hpp"

namespace ce {

__global__ void k_calibrate(L1State* l1, uint32_t rounds, uint64_t spin_limit) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  for (uint32_t i = 1; i <= rounds; ++i) {
    uint64_t spins = 0;
    while (sys_load(&l1->ping) != i) {
      if (++spins > spin_limit) return;
      __builtin_amdgcn_s_sleep(1);
    }
    const uint64_t t = now_tick();
    sys_store(&l1->tick, t);
    sys_store(&l1->pong, i);
  }
}

// Escape-time over one package, the GPU alone: no tiles. Workgroup t of T owns
// every T-th of the package's blocks (as EscapeTile spreads a tile's), and its
// waves take them one at a time from a counter in LDS, so that no wave waits
// for another before the workgroup's end. T is the sweepers of the launch; a
// workgroup beyond them has no pixels.
struct SweepArgs {
  uint32_t blocks;  // of the package
  uint32_t bits;    // their columns, as a power of two
  uint32_t turn;    // blocks the assignment is rotated by from one round of T blocks to the next, below T
  Divisor per_row;  // blocks side by side
  Divisor round;    // T
};

__global__ __launch_bounds__(kBlockThreads, EscapeTile::kMinBlocksPerCu) void k_sweep_escape(EscapeTile pay, DirectArgs d,
                                                                                            SweepArgs s) {
  __shared__ uint32_t next;
  const bool first = threadIdx.x == 0;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
  if (first) {
    next = kBlockThreads / 64;
    if (blockIdx.x == 0) {
      const uint64_t tp = now_tick();
      dev_store(&d.pkgs[0].t_claim, tp);
      sys_store(&d.l1->gpu_t_first, tp);
    }
  }
  __syncthreads();
  const bool sweeps = blockIdx.x < s.round.d;
  for (uint32_t i = w; sweeps;) {
    const uint32_t base = i * s.round.d;
    if (base >= s.blocks) break;
    uint32_t place, bx;
    s.round.split(blockIdx.x + i * s.turn, &place);
    const uint32_t b = base + place;
    if (b < s.blocks) {
      const uint32_t by = s.per_row.split(b, &bx);
      pay.pixel(d.g0, d.g1, by, bx, s.bits, lane);
    }
    uint32_t taken = 0;
    if (lane == 0) taken = __hip_atomic_fetch_add(&next, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    i = __builtin_amdgcn_readfirstlane(taken);
  }
  __syncthreads();
  if (first && sweeps) sys_store(&d.wg_end[blockIdx.x], now_tick());
}

// N-body tiles of 64 that do not fill the GPU: eight waves per group of 64 bodies
// and chunks of 48, one workgroup of 256 registers per compute unit. There the
// chain of the sums bounds the run (15.4 cycles of issue per interaction and
// about 250 to hand the sums on, per chunk), so longer chunks and more waves
// that work out terms pay; where several tiles share a compute unit, other
// tiles fill the waits, and the four waves of 24 keep more of them resident.
// 16,384 bodies, strict: 139 us against 245; 30,001
// (469 tiles) with the hardware 1/sqrt: 428 against 365.
constexpr uint32_t kWideThreads = 512;
constexpr uint32_t kWideChunk = 48;
constexpr uint32_t kWideMaxTiles = 256;  // compute units of the GPU

// d.wg_end null: a plain launch, which leaves no ticks
template <class T>
__global__ __launch_bounds__(kWideThreads, 2) void k_wide(T pay, DirectArgs d) {
  if (d.wg_end && blockIdx.x == 0 && threadIdx.x == 0) {
    const uint64_t tp = now_tick();
    dev_store(&d.pkgs[0].t_claim, tp);
    sys_store(&d.l1->gpu_t_first, tp);
  }
  for (uint32_t t = blockIdx.x; t < d.ntiles; t += gridDim.x)
    pay.template run_group<kWideThreads / 64, kWideChunk>(d.g0, t);
  if (!d.wg_end) return;
  __syncthreads();
  if (threadIdx.x == 0) sys_store(&d.wg_end[blockIdx.x], now_tick());
}

// N-body tiles of 16 bodies with seven waves that work out terms: two waves per
// SIMD keep ahead of the adding wave (4,096 bodies, strict, kernel alone: 26 us
// against 36 with the three of a 256-thread workgroup, hardware 1/sqrt 24
// against 28).
constexpr uint32_t kFeedThreads = 512;
constexpr uint32_t kFeedChunk = 8;

template <class T>
__global__ __launch_bounds__(kFeedThreads, 4) void k_feed(T pay, DirectArgs d) {
  if (d.wg_end && blockIdx.x == 0 && threadIdx.x == 0) {
    const uint64_t tp = now_tick();
    dev_store(&d.pkgs[0].t_claim, tp);
    sys_store(&d.l1->gpu_t_first, tp);
  }
  for (uint32_t t = blockIdx.x; t < d.ntiles; t += gridDim.x)
    pay.template run_feed<kFeedThreads / 64, kFeedChunk>(d.g0, t);
  if (!d.wg_end) return;
  __syncthreads();
  if (threadIdx.x == 0) sys_store(&d.wg_end[blockIdx.x], now_tick());
}

// ------------------------------------------------------------ host helpers
namespace {
// k_wide takes tiles of 64 bodies only: a small share of a space of whole
// granules has few tiles too.
template <class T>
bool nbody_wide(const T& pay, uint32_t tiles) {
  return pay.form() == NbodyForm::kGroups && tiles <= kWideMaxTiles;
}
template <class T>
void launch_nbody_direct(const T& pay, const DirectArgs& d, uint32_t grid, hipStream_t st) {
  if (pay.form() == NbodyForm::kFed)
    hipLaunchKernelGGL(k_feed<T>, dim3(grid), dim3(kFeedThreads), 0, st, pay, d);
  else if (nbody_wide(pay, d.ntiles))
    hipLaunchKernelGGL(k_wide<T>, dim3(grid), dim3(kWideThreads), 0, st, pay, d);
  else
    hipLaunchKernelGGL(k_direct<T>, dim3(grid), dim3(kBlockThreads), 0, st, pay, d);
}
template <class T>
void launch_nbody_bare(const T& pay, uint64_t G, uint32_t tiles, hipStream_t st) {
  DirectArgs d{};
  d.g1 = G;
  d.ntiles = tiles;
  if (pay.form() == NbodyForm::kFed) {
    hipLaunchKernelGGL(k_feed<T>, dim3(tiles), dim3(kFeedThreads), 0, st, pay, d);
  } else if (nbody_wide(pay, tiles)) {
    hipLaunchKernelGGL(k_wide<T>, dim3(tiles), dim3(kWideThreads), 0, st, pay, d);
  } else {
    hipLaunchKernelGGL(k_bare<T>, dim3(tiles), dim3(kBlockThreads), 0, st, pay, G);
  }
}
EscapeTile make_escape(const KernelArgs& a) { return EscapeTile(a.esc, (uint32_t*)a.out, a.host_memory); }
Blur5Tile make_blur(const KernelArgs& a) {
  return Blur5Tile{a.blur, (const float*)a.in0, (const float*)a.in1, (float*)a.out, blur_tile_row_bits(a.blur.w, a.blur.h, a.host_memory), {}};
}
template <bool S>
NbodyTile<S> make_nbody(const KernelArgs& a) {
  return NbodyTile<S>{a.nb, (const float4*)a.in0, (float4*)a.out};
}
BinomialTile make_binomial(const KernelArgs& a) {
  return BinomialTile{a.bin, (const float4*)a.in0, (const float*)a.in1, (float4*)a.out};
}
template <bool S>
NbodyStepTile<S> make_nbody_step(const KernelArgs& a) {
  return NbodyStepTile<S>{a.nbs, (const float4*)a.in0, (const float4*)a.in1, (float4*)a.out, (float4*)a.out1};
}
RtTile make_rt(const KernelArgs& a) { return RtTile{a.rt, a.rt_items, a.rt_lws, rt_tile_items(a.rt_items)}; }
}  // namespace

uint64_t gpu_granules(const KernelArgs& a) {
  switch (a.kernel_id) {
    case CE_KERNEL_ESCAPE: return make_escape(a).granules();
    case CE_KERNEL_BLUR5: return make_blur(a).granules();
    case CE_KERNEL_NBODY_ACC: return make_nbody<true>(a).granules();
    case CE_KERNEL_NBODY_STEP: return make_nbody_step<true>(a).granules();
    case CE_KERNEL_BINOMIAL: return make_binomial(a).granules();
    case CE_KERNEL_RUNTIME: return make_rt(a).granules();
  }
  return 0;
}

uint32_t gpu_tiles(const KernelArgs& a, uint64_t g0, uint64_t g1) {
  switch (a.kernel_id) {
    case CE_KERNEL_ESCAPE: return make_escape(a).ntiles(g0, g1);
    case CE_KERNEL_BLUR5: return make_blur(a).ntiles(g0, g1);
    case CE_KERNEL_NBODY_ACC:
      return a.strict ? make_nbody<true>(a).ntiles(g0, g1) : make_nbody<false>(a).ntiles(g0, g1);
    case CE_KERNEL_NBODY_STEP:
      return a.strict ? make_nbody_step<true>(a).ntiles(g0, g1) : make_nbody_step<false>(a).ntiles(g0, g1);
    case CE_KERNEL_BINOMIAL: return a.bin_call ? binomial_call_tiles(a, g0, g1) : make_binomial(a).ntiles(g0, g1);
    case CE_KERNEL_RUNTIME: return make_rt(a).ntiles(g0, g1);
  }
  return 0;
}

hipError_t persistent_blocks_per_cu(const KernelArgs& a, int* blocks) {
  switch (a.kernel_id) {
    case CE_KERNEL_ESCAPE:
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_persistent<EscapeTile>, kBlockThreads, 0);
    case CE_KERNEL_BLUR5:
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_persistent<Blur5Tile>, kBlockThreads, 0);
    case CE_KERNEL_NBODY_ACC:
      return a.strict ? hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_persistent<NbodyTile<true>>,
                                                                     kBlockThreads, 0)
                      : hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_persistent<NbodyTile<false>>,
                                                                     kBlockThreads, 0);
    case CE_KERNEL_NBODY_STEP:
      return a.strict ? hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_persistent<NbodyStepTile<true>>,
                                                                     kBlockThreads, 0)
                      : hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_persistent<NbodyStepTile<false>>,
                                                                     kBlockThreads, 0);
    case CE_KERNEL_BINOMIAL:
      if (a.bin_call) return binomial_call_blocks_per_cu(blocks);
      return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_persistent<BinomialTile>, kBlockThreads, 0);
    case CE_KERNEL_RUNTIME:
      if (!a.rt_fn_persistent) return hipErrorInvalidValue;
      return hipModuleOccupancyMaxActiveBlocksPerMultiprocessor(blocks, (hipFunction_t)a.rt_fn_persistent,
                                                                kBlockThreads, 0);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_persistent(const KernelArgs& a, const SchedArgs& s, uint32_t grid, hipStream_t st) {
  const dim3 g(grid), b(kBlockThreads);
  switch (a.kernel_id) {
    case CE_KERNEL_ESCAPE: hipLaunchKernelGGL(k_persistent<EscapeTile>, g, b, 0, st, make_escape(a), s); break;
    case CE_KERNEL_BLUR5: hipLaunchKernelGGL(k_persistent<Blur5Tile>, g, b, 0, st, make_blur(a), s); break;
    case CE_KERNEL_NBODY_ACC:
      if (a.strict)
        hipLaunchKernelGGL(k_persistent<NbodyTile<true>>, g, b, 0, st, make_nbody<true>(a), s);
      else
        hipLaunchKernelGGL(k_persistent<NbodyTile<false>>, g, b, 0, st, make_nbody<false>(a), s);
      break;
    case CE_KERNEL_NBODY_STEP:
      if (a.strict)
        hipLaunchKernelGGL(k_persistent<NbodyStepTile<true>>, g, b, 0, st, make_nbody_step<true>(a), s);
      else
        hipLaunchKernelGGL(k_persistent<NbodyStepTile<false>>, g, b, 0, st, make_nbody_step<false>(a), s);
      break;
    case CE_KERNEL_BINOMIAL:
      if (a.bin_call)
        launch_binomial_call_persistent(a, s, grid, st);
      else
        hipLaunchKernelGGL(k_persistent<BinomialTile>, g, b, 0, st, make_binomial(a), s);
      break;
    case CE_KERNEL_RUNTIME: {
      if (!a.rt_fn_persistent) return hipErrorInvalidValue;
      RtTile pay = make_rt(a);
      SchedArgs sa = s;
      void* params[] = {&pay, &sa};
      return hipModuleLaunchKernel((hipFunction_t)a.rt_fn_persistent, grid, 1, 1, kBlockThreads, 1, 1, 0, st, params,
                                   nullptr);
    }
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_direct(const KernelArgs& a, const DirectArgs& d, uint32_t grid, hipStream_t st) {
  const dim3 g(grid), b(kBlockThreads);
  switch (a.kernel_id) {
    case CE_KERNEL_ESCAPE: {
      const uint32_t bits = escape_block_bits(d.g1 - d.g0, escape_least_bits(a.esc.w, a.esc.h, a.esc.max_iter, a.host_memory));
      const uint64_t per_row = escape_blocks_across(a.esc.w, bits), blocks = per_row * escape_blocks_down(d.g1 - d.g0, bits);
      if (blocks >= (1ull << 30)) {
        hipLaunchKernelGGL(k_direct<EscapeTile>, g, b, 0, st, make_escape(a), d);
        break;
      }
      const uint32_t T = d.sweepers;
      if (T == 0 || T > grid) return hipErrorInvalidValue;
      const SweepArgs s{(uint32_t)blocks, bits, ((uint32_t)(per_row * 5 / 8) | 1u) % T, Divisor((uint32_t)per_row), Divisor(T)};
      hipLaunchKernelGGL(k_sweep_escape, g, b, 0, st, make_escape(a), d, s);
      break;
    }
    case CE_KERNEL_BLUR5: hipLaunchKernelGGL(k_direct<Blur5Tile>, g, b, 0, st, make_blur(a), d); break;
    case CE_KERNEL_NBODY_ACC:
      if (a.strict)
        launch_nbody_direct(make_nbody<true>(a), d, grid, st);
      else
        launch_nbody_direct(make_nbody<false>(a), d, grid, st);
      break;
    case CE_KERNEL_NBODY_STEP:
      if (a.strict)
        launch_nbody_direct(make_nbody_step<true>(a), d, grid, st);
      else
        launch_nbody_direct(make_nbody_step<false>(a), d, grid, st);
      break;
    case CE_KERNEL_BINOMIAL:
      if (a.bin_call) return hipErrorInvalidValue;  // dealt by tickets
      hipLaunchKernelGGL(k_direct<BinomialTile>, g, b, 0, st, make_binomial(a), d);
      break;
    case CE_KERNEL_RUNTIME: {
      if (!a.rt_fn_direct) return hipErrorInvalidValue;
      RtTile pay = make_rt(a);
      DirectArgs da = d;
      void* params[] = {&pay, &da};
      return hipModuleLaunchKernel((hipFunction_t)a.rt_fn_direct, grid, 1, 1, kBlockThreads, 1, 1, 0, st, params,
                                   nullptr);
    }
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_bare(const KernelArgs& a, hipStream_t st) {
  const uint64_t G = gpu_granules(a);
  const uint32_t tiles = gpu_tiles(a, 0, G);
  if (tiles == 0) return hipSuccess;
  const dim3 g(tiles), b(kBlockThreads);
  switch (a.kernel_id) {
    case CE_KERNEL_ESCAPE: hipLaunchKernelGGL(k_bare<EscapeTile>, g, b, 0, st, make_escape(a), G); break;
    case CE_KERNEL_BLUR5: hipLaunchKernelGGL(k_bare<Blur5Tile>, g, b, 0, st, make_blur(a), G); break;
    case CE_KERNEL_NBODY_ACC:
      if (a.strict)
        launch_nbody_bare(make_nbody<true>(a), G, tiles, st);
      else
        launch_nbody_bare(make_nbody<false>(a), G, tiles, st);
      break;
    case CE_KERNEL_NBODY_STEP:
      if (a.strict)
        launch_nbody_bare(make_nbody_step<true>(a), G, tiles, st);
      else
        launch_nbody_bare(make_nbody_step<false>(a), G, tiles, st);
      break;
    case CE_KERNEL_BINOMIAL:
      if (a.bin_call)
        launch_binomial_call_bare(a, G, tiles, st);
      else
        hipLaunchKernelGGL(k_bare<BinomialTile>, g, b, 0, st, make_binomial(a), G);
      break;
    case CE_KERNEL_RUNTIME: {
      if (!a.rt_fn_bare) return hipErrorInvalidValue;
      RtTile pay = make_rt(a);
      uint64_t g_arg = G;
      void* params[] = {&pay, &g_arg};
      return hipModuleLaunchKernel((hipFunction_t)a.rt_fn_bare, tiles, 1, 1, kBlockThreads, 1, 1, 0, st, params,
                                   nullptr);
    }
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Streaming copy, the achievable-bandwidth reference for the HBM-bound
// payloads: one 16-byte non-temporal load and store per thread, one
// workgroup per 4 KiB (the fastest of the shapes measured on this GPU:
// 1, 2, 4 or 8 vectors per thread, temporal or not, one-shot or grid-stride).
__global__ __launch_bounds__(kBlockThreads) void k_stream_copy(f32x4* __restrict__ dst, const f32x4* __restrict__ src,
                                                               uint64_t n16) {
  const uint64_t i = (uint64_t)blockIdx.x * kBlockThreads + threadIdx.x;
  if (i < n16) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

hipError_t launch_stream_copy(void* dst, const void* src, uint64_t n16, hipStream_t st) {
  if (n16 == 0) return hipSuccess;
  const uint64_t blocks = (n16 + kBlockThreads - 1) / kBlockThreads;
  if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_stream_copy, dim3((uint32_t)blocks), dim3(kBlockThreads), 0, st, (f32x4*)dst,
                     (const f32x4*)src, n16);
  return hipGetLastError();
}

hipError_t launch_calibrate(L1State* l1, uint32_t rounds, uint64_t spin_limit, hipStream_t st) {
  hipLaunchKernelGGL(k_calibrate, dim3(1), dim3(64), 0, st, l1, rounds, spin_limit);
  return hipGetLastError();
}

}  // namespace ce
