// Tile payloads for gfx950: how a workgroup of 256 threads computes one tile
// of each payload. Shared by the persistent, plain and serving kernels so
// every form runs the same per-item FP32 operation sequence.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/coexec.h"
#include "common.hpp"
#include "device_divide.hpp"
#include "device_payloads.hpp"

namespace ce {

// This thread's index, opaque to the compiler: what a tile works out from it
// is otherwise kept in registers over the tile loop, which has none to spare.
__device__ __forceinline__ uint32_t thread_index() {
  uint32_t t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

struct EscapeTile {
  // workgroups per CU the persistent kernel is compiled for: eight, the
  // residency of the plain launch, so that the 2048 tiles of a 1024 x 1024
  // grid run in one round
  static constexpr int kMinBlocksPerCu = 8;
  static constexpr int kMaxBlocksPerCu = 8;
  static constexpr bool kWavesAlone = true;  // a tile's parts need no barrier between them
  ce_escape_params p;
  uint32_t* out;
  Divisor across;       // the blocks side by side where they are 16 x 4
  uint32_t least_bits;  // of a block's columns
  __host__ __device__ EscapeTile(const ce_escape_params& params, uint32_t* o, bool host_memory)
      : p(params), out(o), across(escape_blocks_across(params.w, 4)),
        least_bits(escape_least_bits(params.w, params.h, params.max_iter, host_memory)) {}
  __device__ void load_constants() {}
  __host__ __device__ uint32_t ncb() const { return (uint32_t)ceil_div(p.w, kEscapeTileCols); }
  __host__ __device__ uint64_t granules() const { return p.h; }
  __host__ __device__ uint32_t ntiles(uint64_t g0, uint64_t g1) const {
    return (uint32_t)(ceil_div(g1 - g0, kEscapeTileRows) * ncb());
  }
  // A tile is as many pixels as kEscapeTileRows x kEscapeTileCols, but not a
  // stretch of a row: the package is cut into blocks of 64 pixels (16 x 4 where
  // its rows allow, escape_block_bits), one wave's, and tile t of nt takes every
  // nt-th block (the start rotated from one round of blocks to the next, so that
  // a tile's blocks do not all lie in one column). Blocks of 16 x 4 keep a
  // wave's orbits closer in length than rows of 64 (8192 x 8192, max_iter
  // 4096: the wave's longest is 117 steps on average against 155), and tiles
  // spread over the whole package cost nearly the same.
  __device__ void run(uint64_t g0, uint64_t g1, uint32_t t) const {
    const uint32_t all = blocks(g0, g1), nt = ntiles(g0, g1);
    for (uint32_t i = __builtin_amdgcn_readfirstlane(thread_index() >> 6); i * nt < all; i += kBlockThreads / 64)
      run_part(g0, g1, t, i);
  }
  __device__ __forceinline__ uint32_t blocks(uint64_t g0, uint64_t g1) const {
    const uint32_t bits = escape_block_bits(g1 - g0, least_bits);
    return escape_blocks_across(p.w, bits) * (uint32_t)escape_blocks_down(g1 - g0, bits);
  }
  // Blocks of a tile, at most, and block i of tile t: a wave's.
  __device__ __forceinline__ uint32_t tile_parts(uint64_t g0, uint64_t g1) const {
    const uint32_t all = blocks(g0, g1), nt = ntiles(g0, g1);
    return all / nt + (all % nt != 0);
  }
  __device__ __forceinline__ void run_part(uint64_t g0, uint64_t g1, uint32_t t, uint32_t i) const {
    const uint32_t bits = escape_block_bits(g1 - g0, least_bits), per_row = escape_blocks_across(p.w, bits), nt = ntiles(g0, g1);
    const uint32_t turn = per_row * 5 / 8 < nt / 8 ? (per_row * 5 / 8) | 1u : nt / 8;
    uint32_t place = t + i * turn;
    while (place >= nt) place -= nt;
    const uint32_t b = i * nt + place;
    if (b >= blocks(g0, g1)) return;
    uint32_t bx, by;
    if (bits == 4) {
      by = across.split(b, &bx);
    } else {
      by = b / per_row;
      bx = b - by * per_row;
    }
    pixel(g0, g1, __builtin_amdgcn_readfirstlane(by), __builtin_amdgcn_readfirstlane(bx), bits, thread_index() & 63u);
  }
  // This lane's pixel of the block that is the by-th down and the bx-th across
  // of a package of rows g0 .. g1.
  __device__ __forceinline__ void pixel(uint64_t g0, uint64_t g1, uint32_t by, uint32_t bx, uint32_t bits,
                                        uint32_t lane) const {
    const uint64_t r = g0 + ((uint64_t)by << (6u - bits)) + (lane >> bits);
    const uint32_t c = (bx << bits) + (lane & ((1u << bits) - 1u));
    if (r < g1 && c < p.w) {
      const float cr = p.x0 + (float)c * p.dx;
      const float ci = p.y0 + (float)r * p.dy;
      out[r * p.w + c] = escape_count(cr, ci, p.max_iter);
    }
  }
};

// 5x5 blur (Gaussian program, section 7.2): out(y,x) = sum over dy, dx of
// w(dy,dx) in(clamp(y+dy), clamp(x+dx)), accumulated by fma with dy outer,
// dx inner, ascending. Each thread owns 4 adjacent columns and walks down the
// tile's rows with a 5-row window of 8 columns (x-2 .. x+5) in registers.
// DPP controls (GFX9 data-parallel primitives): whole-wave shift by one lane.
constexpr int kDppWaveShl1 = 0x130;  // lane i reads lane i+1
constexpr int kDppWaveShr1 = 0x138;  // lane i reads lane i-1
__device__ __forceinline__ float dpp_from_left(float edge, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), kDppWaveShr1, 0xF, 0xF,
                                                    false));
}
__device__ __forceinline__ float dpp_from_right(float edge, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), kDppWaveShl1, 0xF, 0xF,
                                                    false));
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // at any float's address

// kFresh: the input may have been written after the launch began (the
// serving kernel reuses memory while it runs), so wave-uniform reads, which
// the compiler would serve from the scalar cache, use coherent vector loads.
template <bool kFresh>
struct Blur5TileT {
  // Five resident workgroups per CU keep enough loads in flight for HBM; in
  // the plain launch of a large image seven are slower than six (16384^2:
  // 450 against 424 us).
  static constexpr int kMinBlocksPerCu = 5;
  static constexpr int kMaxBlocksPerCu = 6;
  static constexpr bool kWavesAlone = false;
  ce_blur5_params p;
  const float* in;
  const float* wt;
  float* out;
  uint32_t row_bits;  // of a tile's rows (blur_tile_row_bits)
  float w[25];
  __device__ __forceinline__ float uniform_load(const float* a) const {
    if constexpr (kFresh) {
      const uint32_t v = __hip_atomic_load(const_cast<uint32_t*>(reinterpret_cast<const uint32_t*>(a)),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return __uint_as_float(__builtin_amdgcn_readfirstlane(v));
    } else {
      return *a;
    }
  }
  // Weights are read once per workgroup in uniform control flow, so they
  // live in scalar registers and feed the FMAs as scalar operands.
  __device__ void load_constants() {
#pragma unroll
    for (int k = 0; k < 25; ++k) w[k] = uniform_load(wt + k);
  }
  __host__ __device__ uint32_t ncb() const { return (uint32_t)ceil_div(p.w, kBlurTileCols); }
  __host__ __device__ uint64_t granules() const { return p.h; }
  __host__ __device__ uint32_t ntiles(uint64_t g0, uint64_t g1) const {
    return (uint32_t)((g1 - g0 + ((1u << row_bits) - 1u)) >> row_bits) * ncb();
  }
  __device__ __forceinline__ const float* row_ptr(int64_t yy) const {
    yy = yy < 0 ? 0 : (yy >= (int64_t)p.h ? (int64_t)p.h - 1 : yy);
    return in + (size_t)yy * p.w;
  }
  // One output row for this lane's 4 columns from a 5-row window of the 8
  // input columns x-2 .. x+5, in the fixed tap order.
  __device__ __forceinline__ void out4(const float* r0, const float* r1, const float* r2, const float* r3,
                                       const float* r4, float o[4]) const {
    const float* r[5] = {r0, r1, r2, r3, r4};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float acc = 0.0f;
#pragma unroll
      for (int dy = 0; dy < 5; ++dy)
#pragma unroll
        for (int dx = 0; dx < 5; ++dx) acc = __builtin_fmaf(w[dy * 5 + dx], r[dy][q + dx], acc);
      o[q] = acc;
    }
  }

  // Fast path: the wave's 256 columns lie inside the image (at any alignment:
  // a 16-byte load needs four-byte alignment only). Each lane loads its
  // float4; the two columns on either
  // side come from the neighbouring lanes by DPP, and the wave's outer halo
  // from four uniform (scalar) loads clamped to the image.
  struct Raw {
    f32x4 c;
    float l0, l1, r0, r1;
  };
  __device__ __forceinline__ void load_raw(int64_t yy, uint32_t x, uint32_t xw, Raw& a) const {
    const float* row = row_ptr(yy);
    a.c = *reinterpret_cast<const f32x4u*>(row + x);
    a.l0 = uniform_load(row + (xw >= 2 ? xw - 2 : 0));
    a.l1 = uniform_load(row + (xw >= 1 ? xw - 1 : 0));
    a.r0 = uniform_load(row + (xw + 256 < p.w ? xw + 256 : p.w - 1));
    a.r1 = uniform_load(row + (xw + 257 < p.w ? xw + 257 : p.w - 1));
  }
  __device__ __forceinline__ void expand(const Raw& a, float v[8]) const {
    v[0] = dpp_from_left(a.l0, a.c.z);
    v[1] = dpp_from_left(a.l1, a.c.w);
    v[2] = a.c.x;
    v[3] = a.c.y;
    v[4] = a.c.z;
    v[5] = a.c.w;
    v[6] = dpp_from_right(a.r0, a.c.x);
    v[7] = dpp_from_right(a.r1, a.c.y);
  }
  __device__ void run_fast(uint64_t r0, uint64_t r1, uint32_t x, uint32_t xw) const {
    // Rotating window of 6 rows: row y lives in slot (y - r0 + 2) mod 6; the
    // row two below the current one is requested one step ahead.
    float v[6][8];
    Raw pend;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      Raw a;
      load_raw((int64_t)r0 - 2 + j, x, xw, a);
      expand(a, v[j]);
    }
    load_raw((int64_t)r0 + 2, x, xw, pend);
    for (uint64_t yb = r0; yb < r1; yb += 6) {
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const uint64_t y = yb + k;
        if (y >= r1) break;
        expand(pend, v[(k + 4) % 6]);  // row y + 2
        if (y + 1 < r1) load_raw((int64_t)y + 3, x, xw, pend);
        float o[4];
        out4(v[k % 6], v[(k + 1) % 6], v[(k + 2) % 6], v[(k + 3) % 6], v[(k + 4) % 6], o);
        // Streaming store: the output is not read again by this kernel, so
        // it should not push the input rows (reused as halo) out of L2.
        const f32x4 ov = {o[0], o[1], o[2], o[3]};
        __builtin_nontemporal_store(ov, reinterpret_cast<f32x4u*>(out + (size_t)y * p.w + x));
      }
    }
  }

  // General path (images narrower than a wave's 256 columns): per-element
  // clamped loads.
  __device__ void load8(int64_t yy, uint32_t x, float v[8]) const {
    const float* row = row_ptr(yy);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      int64_t xx = (int64_t)x - 2 + k;
      xx = xx < 0 ? 0 : (xx >= (int64_t)p.w ? (int64_t)p.w - 1 : xx);
      v[k] = row[xx];
    }
  }
  __device__ void run_general(uint64_t r0, uint64_t r1, uint32_t x) const {
    if (x >= p.w) return;
    float win[5][8];
#pragma unroll
    for (int j = 0; j < 4; ++j) load8((int64_t)r0 - 2 + j, x, win[j + 1]);
    for (uint64_t y = r0; y < r1; ++y) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int k = 0; k < 8; ++k) win[j][k] = win[j + 1][k];
      load8((int64_t)y + 2, x, win[4]);
      float o[4];
      out4(win[0], win[1], win[2], win[3], win[4], o);
      float* orow = out + (size_t)y * p.w;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (x + q < p.w) __builtin_nontemporal_store(o[q], orow + x + q);
    }
  }

  __device__ void run(uint64_t g0, uint64_t g1, uint32_t t) const {
    const uint32_t nc = ncb();
    const uint64_t r0 = g0 + ((uint64_t)(t / nc) << row_bits), end = r0 + (1u << row_bits);
    const uint64_t r1 = end < g1 ? end : g1;
    // first column of this wave (uniform) and of this lane
    const uint32_t tid = thread_index();
    const uint32_t xw = (t % nc) * kBlurTileCols + (__builtin_amdgcn_readfirstlane(tid) & ~63u) * 4u;
    if (xw >= p.w) return;
    if (p.w >= 256) {
      // The wave at the right edge takes the last 256 columns: the ones it
      // shares with its neighbour get the same values from both. With its own
      // columns and per-element loads, and those for every wave where the
      // width is no multiple of four, 4099 x 3001 took 96 us, now 33, and
      // 8190 x 8192 444 us, now 101.
      const uint32_t xs = xw + 256 <= p.w ? xw : p.w - 256;
      run_fast(r0, r1, xs + (tid & 63u) * 4u, xs);
    } else {
      run_general(r0, r1, xw + (tid & 63u) * 4u);
    }
  }
};

using Blur5Tile = Blur5TileT<false>;
using Blur5TileFresh = Blur5TileT<true>;

// All-pairs acceleration of body i (NBody program, force part): the sum of
// m_j d_ij / (|d_ij|^2 + eps2)^(3/2) over j ascending, one FP32 sum per
// component.
//
// The order of a body's sum is fixed, but only three of an interaction's 24
// instructions are the sum. So a group of 64 bodies, one per lane, is worked
// on by all the waves of a workgroup: wave w takes the chunks w, w + kWaves,
// ... of kChunk consecutive j, works out a chunk's terms (f, dx, dy, dz) in
// registers, waits until the chunk before has been added, adds its own in
// index order and hands the sums on through LDS (`turn` counts the chunks
// added). With one thread per body the GPU held 1024 waves at 65,536 bodies,
// one per SIMD, and a SIMD issues the FP32 instructions of one wave only
// every 5.1 cycles where two or four waves reach 2.6; and below 65,536 bodies
// most SIMDs were idle.
//
// A wave stages its own chunks in LDS (two slots; a chunk is loaded a turn
// before it is needed) and reads them in batches of eight bodies, each batch
// a phase ahead of its arithmetic. LDS operations of one wave take effect in
// order, so a reader that sees `turn` sees the sums stored before it.
constexpr uint32_t kNbodyGroup = 64;  // bodies per tile: one per lane
constexpr uint32_t kNbodyBatch = 8;
constexpr uint32_t kNbodyChunk = 24;  // of a 256-thread workgroup: 128 registers, four waves per SIMD

template <uint32_t kWaves, uint32_t kChunk>
struct NbodyShared {
  f32x4 stage[kWaves][2][kChunk];
  f32x4 sum[kNbodyGroup];
  uint32_t turn;
};

// The forms of one kernel share their LDS: the four or five workgroups of a
// compute unit have 160 KB between them.
template <uint32_t kBytes>
__device__ __forceinline__ unsigned char* nbody_lds() {
  __shared__ __align__(16) unsigned char lds[kBytes];
  return lds;
}

// A zero that the compiler does not keep in registers over the tile loop.
__device__ __forceinline__ float fresh_zero() {
  float x = 0.0f;
  asm volatile("" : "+v"(x));
  return x;
}

template <bool STRICT>
struct NbodyTerms {
  float eps2;
  // Lomont, "Fast Inverse Square Root" (2003): integer estimate then three
  // Newton-Raphson steps y <- y (1.5 - (x/2) y^2) written as t = y*y,
  // u = fma(-(x/2), t, 1.5), y = y*u. Same operation sequence as the host.
  __device__ __forceinline__ float rsqrt_lomont(float x) const {
    float y = __uint_as_float(0x5f375a86u - (__float_as_uint(x) >> 1));
    const float hx = 0.5f * x;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const float t = y * y;
      const float u = __builtin_fmaf(-hx, t, 1.5f);
      y = y * u;
    }
    return y;
  }
  // (dx, dy, dz, f) of body pj = (x, y, z, m) as seen from pi
  __device__ __forceinline__ f32x4 operator()(const f32x4 pj, const f32x4 pi) const {
    const float dx = pj.x - pi.x;
    const float dy = pj.y - pi.y;
    const float dz = pj.z - pi.z;
    const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
    const float rinv = STRICT ? rsqrt_lomont(r2) : __builtin_amdgcn_rsqf(r2);
    const float s = (rinv * rinv) * rinv;
    return f32x4{dx, dy, dz, pj.w * s};
  }
};

__device__ __forceinline__ void nbody_add(f32x4& a, const f32x4 t) {
  a.x = __builtin_fmaf(t.w, t.x, a.x);
  a.y = __builtin_fmaf(t.w, t.y, a.y);
  a.z = __builtin_fmaf(t.w, t.z, a.z);
}

// The acceleration of this lane's body pi. Every wave of the workgroup takes
// part; true in the one wave that returns the sums.
template <bool STRICT, uint32_t kWaves, uint32_t kChunk>
__device__ __forceinline__ bool nbody_accumulate(const f32x4* pos, uint32_t n, float eps2, uint32_t lane,
                                                 const f32x4 pi, NbodyShared<kWaves, kChunk>& sh, f32x4& acc) {
  static_assert(kChunk % kNbodyBatch == 0 && kChunk <= 64, "whole batches, one body per lane to stage");
  const NbodyTerms<STRICT> terms{eps2};
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t chunks = n / kChunk;  // whole ones
  f32x4(*const slot)[kChunk] = sh.stage[w];
  // Every wait ends: chunk c is added by a wave of this workgroup, which
  // waits only for the chunks before it.
  const auto sums_at = [&](uint32_t c) {
    while ((uint32_t)__builtin_amdgcn_readfirstlane(
               __hip_atomic_load(&sh.turn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != c) {
    }
    asm volatile("" ::: "memory");
    return sh.sum[lane];
  };
  __syncthreads();  // the tile before is done with `sh`
  if (w == 0) {
    const float zero = fresh_zero();
    sh.sum[lane] = f32x4{zero, zero, zero, zero};
    if (lane == 0) sh.turn = 0;
  }
  if (lane < kChunk && w < chunks) slot[0][lane] = pos[w * kChunk + lane];
  __syncthreads();
  f32x4 t[kChunk], next = pi;  // any value: a lane or turn that does not load does not use it
  uint32_t s = 0;
  for (uint32_t c = w; c < chunks; c += kWaves) {
    // two batches, then one more ahead of each batch's arithmetic
#pragma unroll
    for (uint32_t k = 0; k < 2 * kNbodyBatch && k < kChunk; ++k) t[k] = slot[s][k];
    if (lane < kChunk && c + kWaves < chunks) next = pos[(c + kWaves) * kChunk + lane];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (uint32_t q = 0; q < kChunk; q += kNbodyBatch) {
      if (q > 0 && q + kNbodyBatch < kChunk) {
#pragma unroll
        for (uint32_t k = q + kNbodyBatch; k < q + 2 * kNbodyBatch; ++k) t[k] = slot[s][k];
        __builtin_amdgcn_sched_barrier(0);
      }
      // A few bodies interleaved at a time (all eight would spill), and
      // worked out here: without the fences the compiler moves the arithmetic
      // past the wait below. Two bodies hide the latency of an instruction
      // with four waves per SIMD, four with two.
      constexpr uint32_t kTogether = kWaves > 4 ? 4 : 2;
#pragma unroll
      for (uint32_t k0 = q; k0 < q + kNbodyBatch; k0 += kTogether) {
#pragma unroll
        for (uint32_t k = k0; k < k0 + kTogether; ++k) t[k] = terms(t[k], pi);
#pragma unroll
        for (uint32_t k = k0; k < k0 + kTogether; ++k) asm volatile("" : "+v"(t[k]));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    acc = sums_at(c);
    __builtin_amdgcn_s_setprio(3);  // the other waves wait for this chain
#pragma unroll
    for (uint32_t k = 0; k < kChunk; ++k) nbody_add(acc, t[k]);
    sh.sum[lane] = acc;
    asm volatile("" ::: "memory");
    __hip_atomic_store(&sh.turn, c + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_s_setprio(0);
    s ^= 1u;
    if (lane < kChunk) slot[s][lane] = next;
  }
  if (w != chunks % kWaves) return false;
  // the bodies past the last whole chunk, and the result
  const uint32_t j0 = chunks * kChunk, m = n - j0;
  if (lane < m) slot[0][lane] = pos[j0 + lane];
  acc = sums_at(chunks);
#pragma unroll 1
  for (uint32_t k = 0; k < m; ++k) nbody_add(acc, terms(slot[0][k], pi));
  return true;
}

// The same acceleration with one thread per body: a tile of 256 bodies, each
// j read from LDS by all four waves, staged 256 at a time; every thread of the
// workgroup takes part in the staging, and loads its part of the next stage
// while the current one is computed. Two batches of eight bodies in
// registers: the next batch is read from LDS while the current one is
// computed (scheduling fences keep each batch's reads a phase ahead of its
// arithmetic). Nothing is handed on, so it is the faster form where it
// alone gives every SIMD two or four waves.
constexpr uint32_t kNbodyWhole = 256;

template <bool STRICT>
__device__ __forceinline__ f32x4 nbody_accumulate_whole(const f32x4* pos, uint32_t n, float eps2, uint32_t tid,
                                                        const f32x4 pi, f32x4 (&stages)[2 * kNbodyWhole]) {
  const NbodyTerms<STRICT> terms{eps2};
  __syncthreads();  // the tile before may still be read
  f32x4 acc = {0.f, 0.f, 0.f, 0.f}, stage = pi;
  if (tid < n) stage = pos[tid];
  for (uint32_t j0 = 0; j0 < n; j0 += kNbodyWhole) {
    // two stages in turn: the barrier before a stage's arithmetic also says
    // that every wave is done with the stage before
    f32x4* const sh = stages + (j0 & kNbodyWhole);
    sh[tid] = stage;
    __syncthreads();
    if (j0 + kNbodyWhole + tid < n) stage = pos[j0 + kNbodyWhole + tid];
    const uint32_t m = (n - j0 < kNbodyWhole) ? n - j0 : kNbodyWhole;
    uint32_t jj = 0;
    if (m >= kNbodyBatch) {
      f32x4 a[kNbodyBatch], b[kNbodyBatch];
#pragma unroll
      for (uint32_t k = 0; k < kNbodyBatch; ++k) a[k] = sh[k];
      for (; jj + 2 * kNbodyBatch <= m; jj += 2 * kNbodyBatch) {
#pragma unroll
        for (uint32_t k = 0; k < kNbodyBatch; ++k) b[k] = sh[jj + kNbodyBatch + k];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (uint32_t k = 0; k < kNbodyBatch; ++k) nbody_add(acc, terms(a[k], pi));
        __builtin_amdgcn_sched_barrier(0);
        // the batch after (read within the stage; unused past its end)
#pragma unroll
        for (uint32_t k = 0; k < kNbodyBatch; ++k) a[k] = sh[(jj + 2 * kNbodyBatch + k) & (kNbodyWhole - 1)];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (uint32_t k = 0; k < kNbodyBatch; ++k) nbody_add(acc, terms(b[k], pi));
        __builtin_amdgcn_sched_barrier(0);
      }
      if (jj + kNbodyBatch <= m) {
#pragma unroll
        for (uint32_t k = 0; k < kNbodyBatch; ++k) nbody_add(acc, terms(a[k], pi));
        jj += kNbodyBatch;
      }
    }
    for (; jj < m; ++jj) nbody_add(acc, terms(sh[jj], pi));
  }
  return acc;
}

// The same acceleration for few bodies, where the chain of the sums bounds the
// run: a tile of 16 bodies, one wave that only adds and kWaves - 1 that work out
// the terms. Those write (dx, dy, dz, f) of kChunk bodies j each and phase into
// LDS; in the adding wave a lane is one component of one body, reads one float
// per j and takes f from its neighbour (lane 3 of four) by DPP, so a sum costs
// one instruction per j instead of three, and nothing is handed on. Three phases
// of the ring: one being written, one complete, whose first half is read before
// the barrier, one being added. The bodies past n are padded with d = -0, f = 0,
// which leave a sum as it is, its sign and a NaN included.
//
// An addition takes 11 to 12 cycles (8 to 9 of them the latency of the fma), the
// relay above 22. 4,096 bodies, strict, a whole call of the GPU alone: 38 us, with
// the wide groups 49; in packages of 256 bodies 67 against 82.
constexpr uint32_t kNbodyFeedGroup = 16;
constexpr uint32_t kNbodyFeedChunk = 16;  // of a 256-thread workgroup
// Two tiles per compute unit, where it is no slower than groups of 64 for the GPU
// alone (8,192 bodies, strict: 83.8 us against 84.6) and faster in packages (117
// against 139); beyond, the terms bound the run and groups work them out with
// fewer instructions (12,000: kernel alone 125 us against about 108).
constexpr uint32_t kNbodyFeedMax = 8192;

template <uint32_t kWaves, uint32_t kChunk>
struct NbodyRing {
  static constexpr uint32_t kPhase = (kWaves - 1) * kChunk;
  f32x4 term[3][kPhase][kNbodyFeedGroup];
};
constexpr uint32_t kNbodyLds = sizeof(NbodyRing<kBlockThreads / 64, kNbodyFeedChunk>);  // the largest

// sum += f d, twelve or four j after one another. One block, as the compiler
// puts a wait or an s_nop between any two. The s_nop is the distance that a DPP
// operand needs from a vector instruction that writes it.
#define CE_NBODY_FMAC(k) "v_fmac_f32_dpp %0, %" #k ", %" #k " quad_perm:[3,3,3,3] row_mask:0xf bank_mask:0xf\n\t"
template <int kCount>
__device__ __forceinline__ void nbody_sum(float& a, const float* v) {
  if constexpr (kCount >= 12) {
    asm("s_nop 1\n\t" CE_NBODY_FMAC(1) CE_NBODY_FMAC(2) CE_NBODY_FMAC(3) CE_NBODY_FMAC(4) CE_NBODY_FMAC(5)
            CE_NBODY_FMAC(6) CE_NBODY_FMAC(7) CE_NBODY_FMAC(8) CE_NBODY_FMAC(9) CE_NBODY_FMAC(10) CE_NBODY_FMAC(11)
                CE_NBODY_FMAC(12)
        : "+v"(a)
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]), "v"(v[8]), "v"(v[9]),
          "v"(v[10]), "v"(v[11]));
    nbody_sum<kCount - 12>(a, v + 12);
  } else if constexpr (kCount > 0) {
    static_assert(kCount >= 4, "batches of twelve and four");
    asm("s_nop 1\n\t" CE_NBODY_FMAC(1) CE_NBODY_FMAC(2) CE_NBODY_FMAC(3) CE_NBODY_FMAC(4)
        : "+v"(a)
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]));
    nbody_sum<kCount - 4>(a, v + 4);
  }
}
#undef CE_NBODY_FMAC

// The sums of the 16 bodies from b0 on: true in the adding wave, whose lane l
// returns component l & 3 of body b0 + (l >> 2) (l & 3 == 3: any value).
template <bool STRICT, uint32_t kWaves, uint32_t kChunk>
__device__ __forceinline__ bool nbody_feed(const f32x4* pos, uint32_t n, float eps2, uint32_t b0, uint32_t lane,
                                           NbodyRing<kWaves, kChunk>& ring, float& sum) {
  constexpr uint32_t kPhase = NbodyRing<kWaves, kChunk>::kPhase, kHalf = kPhase / 2, kSteps = kChunk / 4;
  constexpr uint32_t kSlotFloats = kPhase * kNbodyFeedGroup * 4;
  static_assert(kChunk % 8 == 0, "whole steps of four j, halves of whole batches");
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t phases = n / kPhase + (n % kPhase != 0);
  // Every wave passes phases + 3 barriers.
  __syncthreads();  // the tile before is done with `ring`
  if (w == 0) {
    __builtin_amdgcn_s_setprio(3);  // the other waves wait for this chain
    const float* const base = reinterpret_cast<const float*>(&ring) + lane;
    const float* cur = base;
    float a[kHalf], b[kHalf];
    sum = fresh_zero();
    __syncthreads();
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kHalf; ++k) a[k] = cur[k * 64];
    uint32_t slot = 0;
#pragma unroll 1
    for (uint32_t p = 0; p < phases; ++p) {
#pragma unroll
      for (uint32_t k = 0; k < kHalf; ++k) b[k] = cur[(kHalf + k) * 64];
      __builtin_amdgcn_sched_barrier(0);
      nbody_sum<kHalf>(sum, a);
      __builtin_amdgcn_sched_barrier(0);
      slot = slot == 2 ? 0 : slot + 1;
      cur = base + slot * kSlotFloats;
#pragma unroll
      for (uint32_t k = 0; k < kHalf; ++k) a[k] = cur[k * 64];  // unused past the last phase
      __builtin_amdgcn_sched_barrier(0);
      nbody_sum<kHalf>(sum, b);
      __builtin_amdgcn_sched_barrier(0);
      __syncthreads();
    }
    __builtin_amdgcn_s_setprio(0);
    return true;
  }
  const NbodyTerms<STRICT> terms{eps2};
  const uint32_t body = lane & 15u, i = b0 + body, j0 = (w - 1) * kChunk + (lane >> 4);
  const f32x4 pi = pos[i < n ? i : n - 1];
  const auto load = [&](uint32_t p, f32x4(&x)[kSteps]) {
#pragma unroll
    for (uint32_t k = 0; k < kSteps; ++k) {
      const uint32_t j = p * kPhase + j0 + k * 4;
      x[k] = pos[j < n ? j : n - 1];
    }
  };
  uint32_t slot = 0, p = 0;
  // a phase's terms, and the bodies of the phase after the next
  const auto feed = [&](f32x4(&x)[kSteps]) {
#pragma unroll
    for (uint32_t k = 0; k < kSteps; ++k) {
      f32x4 t = terms(x[k], pi);
      if ((p + 1) * kPhase > n && p * kPhase + j0 + k * 4 >= n) t = f32x4{-0.0f, -0.0f, -0.0f, 0.0f};
      ring.term[slot][j0 + k * 4][body] = t;
    }
    load(p + 2, x);
    slot = slot == 2 ? 0 : slot + 1;
    ++p;
    __syncthreads();
  };
  f32x4 x0[kSteps], x1[kSteps];
  load(0, x0);
  load(1, x1);
#pragma unroll 1
  while (p + 2 <= phases + 2) {
    feed(x0);
    feed(x1);
  }
  if (p < phases + 2) feed(x0);
  return false;
}

// Whether the engine's tiles are whole granules: where those give most of the
// 256 compute units two, so two waves per SIMD, and groups of 64, more than
// six (hardware 1/sqrt: seven) per compute unit, a second round as full as the
// first. Whole against groups, in ms, GPU alone and in packages of 256 bodies.
// Strict 1/sqrt: 131,072 bodies 6.90 and 6.99 against 7.00 and 7.70; 118,000
// 5.92 and 5.97 against 6.49 and 7.10; 110,000 5.39 and 5.44 against 5.27 and
// 5.33 (on a slower card 5.6 and 5.6 against 5.54 and 5.71); 100,000 4.88 and
// 4.93 against 4.86 and 4.92; 98,304 4.76 against 4.16 (alone). Hardware
// 1/sqrt: 131,072 5.43 and 5.43 against 5.30 and 5.63; 118,000 4.89 and 4.88
// against 4.82 and 5.14; 114,688 4.86 and 4.95 against 4.11 and 4.13. With
// three or four granules per compute unit groups are faster or equal (strict,
// 196,608: 16.3 against 19.1; 262,144: 28.3 against 28.5).
template <bool STRICT>
__host__ __device__ inline bool nbody_whole(uint32_t n) {
  const uint32_t granules = n / kNbodyGranule + (n % kNbodyGranule != 0);
  return granules > (STRICT ? 384u : 448u) && granules <= 512u;
}

// Tiles of a range of 256-body granules in groups of `group` bodies.
__host__ __device__ inline uint32_t nbody_tiles(uint32_t n, uint64_t g0, uint64_t g1, uint32_t group = kNbodyGroup) {
  const uint64_t end = g1 * kNbodyGranule < n ? g1 * kNbodyGranule : n;
  return g0 * kNbodyGranule < end ? (uint32_t)ceil_div(end - g0 * kNbodyGranule, group) : 0;
}
// The form of the engine's tiles, from the bodies alone (a share or package of
// the space has its tiles in the form of the whole): what counts tiles, runs
// them or picks a kernel for them asks here.
enum class NbodyForm { kFed, kGroups, kWhole };
template <bool STRICT>
__host__ __device__ inline NbodyForm nbody_form(uint32_t n) {
  return n <= kNbodyFeedMax ? NbodyForm::kFed : nbody_whole<STRICT>(n) ? NbodyForm::kWhole : NbodyForm::kGroups;
}
template <bool STRICT>
__host__ __device__ inline uint32_t nbody_engine_tiles(uint32_t n, uint64_t g0, uint64_t g1) {
  switch (nbody_form<STRICT>(n)) {
    case NbodyForm::kFed: return nbody_tiles(n, g0, g1, kNbodyFeedGroup);
    case NbodyForm::kWhole: return (uint32_t)(g1 - g0);
    default: return nbody_tiles(n, g0, g1);
  }
}

// Accelerations: a granule is 256 bodies, a tile 64 of them or all.
template <bool STRICT>
struct NbodyTile {
  // four workgroups per CU: four waves per SIMD, 128 registers each
  static constexpr int kMinBlocksPerCu = 4;
  static constexpr int kMaxBlocksPerCu = 8;
  static constexpr bool kWavesAlone = false;
  ce_nbody_params p;
  const float4* pos;
  float4* out;
  __device__ void load_constants() {}
  __host__ __device__ uint64_t granules() const { return ceil_div(p.n, kNbodyGranule); }
  __host__ __device__ uint32_t ntiles(uint64_t g0, uint64_t g1) const {
    return nbody_engine_tiles<STRICT>(p.n, g0, g1);
  }
  __host__ __device__ NbodyForm form() const { return nbody_form<STRICT>(p.n); }
  __device__ void run(uint64_t g0, uint64_t, uint32_t t) const {
    const NbodyForm f = form();
    if (f == NbodyForm::kFed)
      run_feed<kBlockThreads / 64, kNbodyFeedChunk, kNbodyLds>(g0, t);
    else if (f == NbodyForm::kWhole)
      run_whole<kNbodyLds>(g0, t);
    else
      run_group<kBlockThreads / 64, kNbodyChunk, kNbodyLds>(g0, t);
  }
  template <uint32_t kWaves, uint32_t kChunk, uint32_t kLds = sizeof(NbodyShared<kWaves, kChunk>)>
  __device__ __forceinline__ void run_group(uint64_t g0, uint32_t t) const {
    static_assert(sizeof(NbodyShared<kWaves, kChunk>) <= kLds, "");
    auto& sh = *reinterpret_cast<NbodyShared<kWaves, kChunk>*>(nbody_lds<kLds>());
    const uint32_t lane = thread_index() & 63u;
    const uint64_t i = g0 * kNbodyGranule + (uint64_t)t * kNbodyGroup + lane;
    const bool active = i < p.n;
    const f32x4* const p4 = reinterpret_cast<const f32x4*>(pos);
    const f32x4 pi = active ? p4[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 a;
    if (nbody_accumulate<STRICT, kWaves, kChunk>(p4, p.n, p.eps2, lane, pi, sh, a) && active) store(i, a);
  }
  template <uint32_t kWaves, uint32_t kChunk, uint32_t kLds = sizeof(NbodyRing<kWaves, kChunk>)>
  __device__ __forceinline__ void run_feed(uint64_t g0, uint32_t t) const {
    auto& ring = *reinterpret_cast<NbodyRing<kWaves, kChunk>*>(nbody_lds<kLds>());
    const uint32_t b0 = (uint32_t)(g0 * kNbodyGranule) + t * kNbodyFeedGroup;
    const uint32_t lane = thread_index() & 63u;
    float a;
    if (nbody_feed<STRICT, kWaves, kChunk>(reinterpret_cast<const f32x4*>(pos), p.n, p.eps2, b0, lane, ring, a)) {
      const uint32_t k = b0 * 4 + (thread_index() & 63u);
      if (k < p.n * 4) store_component(k, a);
    }
  }
  template <uint32_t kLds>
  __device__ __forceinline__ void run_whole(uint64_t g0, uint32_t t) const {
    static_assert(sizeof(f32x4[2 * kNbodyWhole]) <= kLds, "");
    auto& sh = *reinterpret_cast<f32x4(*)[2 * kNbodyWhole]>(nbody_lds<kLds>());
    const uint32_t tid = thread_index();
    const uint64_t i = (g0 + t) * kNbodyGranule + tid;
    const f32x4* const p4 = reinterpret_cast<const f32x4*>(pos);
    const f32x4 pi = i < p.n ? p4[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    const f32x4 a = nbody_accumulate_whole<STRICT>(p4, p.n, p.eps2, tid, pi, sh);
    if (i < p.n) store((g0 + t) * kNbodyGranule + thread_index(), a);
  }
  // float k of the output
  __device__ __forceinline__ void store_component(uint32_t k, float a) const {
    reinterpret_cast<float*>(out)[k] = (k & 3u) == 3u ? 0.0f : a;
  }
  __device__ __forceinline__ void store(uint64_t i, const f32x4 a) const {
    out[i] = make_float4(a.x, a.y, a.z, 0.0f);
  }
};

// Integration step (NBody program: positions and velocities in and out):
// with the acceleration above, v' = v + a dt and x' = x + v dt + a dt^2/2,
// per component as h = (dt dt) 0.5, x' = (x + v dt) + a h, v' = v + a dt;
// the mass and the velocity's w are copied.
template <bool STRICT>
struct NbodyStepTile {
  static constexpr int kMinBlocksPerCu = 4;
  static constexpr int kMaxBlocksPerCu = 8;
  static constexpr bool kWavesAlone = false;
  ce_nbody_step_params p;
  const float4* pos;
  const float4* vel;
  float4* pos_out;
  float4* vel_out;
  __device__ void load_constants() {}
  __host__ __device__ uint64_t granules() const { return ceil_div(p.n, kNbodyGranule); }
  __host__ __device__ uint32_t ntiles(uint64_t g0, uint64_t g1) const {
    return nbody_engine_tiles<STRICT>(p.n, g0, g1);
  }
  __host__ __device__ NbodyForm form() const { return nbody_form<STRICT>(p.n); }
  __device__ void run(uint64_t g0, uint64_t, uint32_t t) const {
    const NbodyForm f = form();
    if (f == NbodyForm::kFed)
      run_feed<kBlockThreads / 64, kNbodyFeedChunk, kNbodyLds>(g0, t);
    else if (f == NbodyForm::kWhole)
      run_whole<kNbodyLds>(g0, t);
    else
      run_group<kBlockThreads / 64, kNbodyChunk, kNbodyLds>(g0, t);
  }
  template <uint32_t kWaves, uint32_t kChunk, uint32_t kLds = sizeof(NbodyShared<kWaves, kChunk>)>
  __device__ __forceinline__ void run_group(uint64_t g0, uint32_t t) const {
    static_assert(sizeof(NbodyShared<kWaves, kChunk>) <= kLds, "");
    auto& sh = *reinterpret_cast<NbodyShared<kWaves, kChunk>*>(nbody_lds<kLds>());
    const uint32_t lane = thread_index() & 63u;
    const uint64_t i = g0 * kNbodyGranule + (uint64_t)t * kNbodyGroup + lane;
    const bool active = i < p.n;
    const f32x4* const p4 = reinterpret_cast<const f32x4*>(pos);
    const f32x4 pi = active ? p4[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 a;
    if (nbody_accumulate<STRICT, kWaves, kChunk>(p4, p.n, p.eps2, lane, pi, sh, a) && active) store(i, pi, a);
  }
  template <uint32_t kWaves, uint32_t kChunk, uint32_t kLds = sizeof(NbodyRing<kWaves, kChunk>)>
  __device__ __forceinline__ void run_feed(uint64_t g0, uint32_t t) const {
    auto& ring = *reinterpret_cast<NbodyRing<kWaves, kChunk>*>(nbody_lds<kLds>());
    const uint32_t b0 = (uint32_t)(g0 * kNbodyGranule) + t * kNbodyFeedGroup;
    const uint32_t lane = thread_index() & 63u;
    float a;
    if (nbody_feed<STRICT, kWaves, kChunk>(reinterpret_cast<const f32x4*>(pos), p.n, p.eps2, b0, lane, ring, a)) {
      const uint32_t k = b0 * 4 + (thread_index() & 63u);
      if (k < p.n * 4) store_component(k, a);
    }
  }
  template <uint32_t kLds>
  __device__ __forceinline__ void run_whole(uint64_t g0, uint32_t t) const {
    static_assert(sizeof(f32x4[2 * kNbodyWhole]) <= kLds, "");
    auto& sh = *reinterpret_cast<f32x4(*)[2 * kNbodyWhole]>(nbody_lds<kLds>());
    const uint32_t tid = thread_index();
    const uint64_t i = (g0 + t) * kNbodyGranule + tid;
    const f32x4* const p4 = reinterpret_cast<const f32x4*>(pos);
    const f32x4 pi = i < p.n ? p4[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    const f32x4 a = nbody_accumulate_whole<STRICT>(p4, p.n, p.eps2, tid, pi, sh);
    if (i < p.n) store((g0 + t) * kNbodyGranule + thread_index(), pi, a);
  }
  __device__ __forceinline__ void store_component(uint32_t k, float a) const {
    const float x = reinterpret_cast<const float*>(pos)[k], v = reinterpret_cast<const float*>(vel)[k];
    const float dt = p.dt;
    const float h = (dt * dt) * 0.5f;
    const bool copy = (k & 3u) == 3u;
    reinterpret_cast<float*>(pos_out)[k] = copy ? x : (x + v * dt) + a * h;
    reinterpret_cast<float*>(vel_out)[k] = copy ? v : v + a * dt;
  }
  __device__ __forceinline__ void store(uint64_t i, const f32x4 pi, const f32x4 a) const {
    const float4 vi = vel[i];
    const float dt = p.dt;
    const float h = (dt * dt) * 0.5f;
    float4 xo, vo;
    xo.x = (pi.x + vi.x * dt) + a.x * h;
    xo.y = (pi.y + vi.y * dt) + a.y * h;
    xo.z = (pi.z + vi.z * dt) + a.z * h;
    xo.w = pi.w;
    vo.x = vi.x + a.x * dt;
    vo.y = vi.y + a.y * dt;
    vo.z = vi.z + a.z * dt;
    vo.w = vi.w;
    pos_out[i] = xo;
    vel_out[i] = vo;
  }
};

// Binomial option pricing: a granule is one work-group pricing four calls
// (one float4 of spots). At each level of the backward induction a node is
// pu V[j+1] + pd V[j] (two products, then their sum), so a tree of N levels
// takes 3 N (N + 1) / 2 instructions per call at the least. Two forms keep a
// tree inside a wave, with no barrier, and differ in how many lanes share it.
//
// pu and pd are held in vector registers: a product with a scalar operand
// issues at half the rate.
__device__ __forceinline__ float binomial_constant(float x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ float binomial_leaf(float S, float f, float X) {
  const float a = S * f - X;
  return a > 0.0f ? a : 0.0f;
}

// Group form: a wave prices one group. Lane i holds leaves 4i .. 4i+3 of each
// call, so only the last of four nodes needs another lane's value (a product
// with a DPP wave shift, no instruction of its own), and lanes above the level
// produce values that no later level reads. When the nodes left fit half the
// lanes, two calls' registers are merged into one (the upper half of one
// swapped with the lower half of the other), and again at a quarter, so that
// at most half of the lanes idle; trees of fewer levels start merged. Bound by
// VALU issue: 254 steps, 256 groups 56.6 -> 23.8 us, 4096 groups 137 -> 66 us,
// against a workgroup per pair of groups with a barrier at every level.
struct BinomialTile {
  static constexpr int kMinBlocksPerCu = 8;
  static constexpr int kMaxBlocksPerCu = 8;
  static constexpr bool kWavesAlone = false;
  static constexpr uint32_t kGroupsPerTile = kBlockThreads / 64;
  ce_binomial_params p;
  const float4* spots;
  const float* factors;
  float4* out;
  __device__ void load_constants() {}
  __host__ __device__ uint64_t granules() const { return p.n_groups; }
  __host__ __device__ uint32_t ntiles(uint64_t g0, uint64_t g1) const {
    return (uint32_t)((g1 - g0 + kGroupsPerTile - 1) / kGroupsPerTile);
  }
  // Lane i receives lane i + 1's value (DPP wave_shl:1), the last lane zero.
  static __device__ __forceinline__ float from_next_lane(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kDppWaveShl1, 0xf, 0xf, true));
  }
  // One level of kSets calls (or sets of merged calls), four nodes per lane.
  template <int kSets>
  static __device__ __forceinline__ void level(float (&v)[kSets][4], float pu, float pd) {
#pragma unroll
    for (int s = 0; s < kSets; ++s) {
      const float up = pu * from_next_lane(v[s][0]);
      v[s][0] = pu * v[s][1] + pd * v[s][0];
      v[s][1] = pu * v[s][2] + pd * v[s][1];
      v[s][2] = pu * v[s][3] + pd * v[s][2];
      v[s][3] = up + pd * v[s][3];
    }
  }
  // a takes b's lower half into its upper half
  static __device__ __forceinline__ float merge_halves(float a, float b) {
    return __uint_as_float(__builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false)[0]);
  }
  // rows 1 and 3 of a take rows 0 and 2 of b
  static __device__ __forceinline__ float merge_rows(float a, float b) {
    return __uint_as_float(__builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false)[0]);
  }
  __device__ void run(uint64_t g0, uint64_t g1, uint32_t t) const {
    const uint32_t tid = thread_index();
    const uint64_t grp = g0 + (uint64_t)t * kGroupsPerTile + __builtin_amdgcn_readfirstlane(tid >> 6);
    if (grp >= g1) return;
    const uint32_t lane = tid & 63u, n = p.steps;
    const float X = p.strike, pu = binomial_constant(p.pu), pd = binomial_constant(p.pd);
    const float4 S = spots[grp];
    const auto leaf = [&](float s, uint32_t j) { return j <= n ? binomial_leaf(s, factors[j], X) : 0.0f; };
    uint32_t l = n;    // the level held: nodes 0 .. l
    float half[2][4];  // calls x|y and z|w, 32 lanes each
    if (n > 127) {
      float v[4][4];
#pragma unroll
      for (uint32_t r = 0; r < 4; ++r) {
        v[0][r] = leaf(S.x, lane * 4 + r);
        v[1][r] = leaf(S.y, lane * 4 + r);
        v[2][r] = leaf(S.z, lane * 4 + r);
        v[3][r] = leaf(S.w, lane * 4 + r);
      }
#pragma unroll 1
      for (; l > 127; --l) level<4>(v, pu, pd);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        half[0][r] = merge_halves(v[0][r], v[1][r]);
        half[1][r] = merge_halves(v[2][r], v[3][r]);
      }
    } else {
      const float s0 = lane < 32 ? S.x : S.y, s1 = lane < 32 ? S.z : S.w;
#pragma unroll
      for (uint32_t r = 0; r < 4; ++r) {
        half[0][r] = leaf(s0, (lane & 31u) * 4 + r);
        half[1][r] = leaf(s1, (lane & 31u) * 4 + r);
      }
    }
#pragma unroll 1
    for (; l > 63; --l) level<2>(half, pu, pd);
    float row[1][4];  // calls x, z, y, w, 16 lanes each
#pragma unroll
    for (int r = 0; r < 4; ++r) row[0][r] = merge_rows(half[0][r], half[1][r]);
#pragma unroll 1
    for (; l > 0; --l) level<1>(row, pu, pd);
    if ((lane & 15u) == 0) {
      const uint32_t q = lane >> 4;
      reinterpret_cast<float*>(out + grp)[(q & 1u) * 2 + (q >> 1)] = row[0][0];
    }
  }
};

// Call form, where the groups fill the GPU: a lane prices one call, its nodes
// in registers, so nothing moves between lanes and no lane idles. A level is
// unrolled over the nodes still alive, to the next multiple of 16. 256
// registers hold nodes 0 .. 191; a deeper tree first runs its nodes from 192
// up through all their levels and leaves node 192's value of each level in
// LDS (64 KiB per workgroup), where the lower nodes take it up. Two workgroups
// per compute unit: two waves per SIMD, which issue at 2.1 cycles per
// instruction of a possible 2. 254 steps: 1,048,576 groups 27.3 -> 5.95 ms
// (12.0 in the group form), 32,768 groups 887 -> 206 us (410), 16,384 groups
// about 190 (205), 8,192 188 (120): a wave takes 185 us however few there are.
struct BinomialCallTile {
  static constexpr int kMinBlocksPerCu = 2;
  static constexpr int kMaxBlocksPerCu = 8;
  static constexpr bool kWavesAlone = false;
  static constexpr uint32_t kGroupsPerTile = kBlockThreads / 4;
  static constexpr int kLow = 192, kHigh = 64, kStep = 16;
  ce_binomial_params p;
  const float4* spots;
  const float* factors;
  float4* out;
  __device__ void load_constants() {}
  __host__ __device__ uint64_t granules() const { return p.n_groups; }
  __host__ __device__ uint32_t ntiles(uint64_t g0, uint64_t g1) const {
    return (uint32_t)((g1 - g0 + kGroupsPerTile - 1) / kGroupsPerTile);
  }
  // One level of nodes 0 .. kCount - 2 (the node above each is in v).
  template <int kCount, int kSize>
  static __device__ __forceinline__ void level(float (&v)[kSize], float pu, float pd) {
#pragma unroll
    for (int k = 0; k + 1 < kCount; ++k) v[k] = pu * v[k + 1] + pd * v[k];
  }
  // From level l down to 0 of the nodes 0 .. kCount - 1, fewer at each level.
  template <int kCount>
  static __device__ __forceinline__ void low_levels(float (&v)[kLow], uint32_t& l, float pu, float pd) {
    if constexpr (kCount > 0) {
#pragma unroll 1
      for (; l + kStep >= kCount && l > 0; --l) level<kCount>(v, pu, pd);
      low_levels<kCount - kStep>(v, l, pu, pd);
    }
  }
  // From level l down to kLow of the nodes kLow .. kLow + kCount - 1, node
  // kLow's value of each level into `edge`.
  template <int kCount>
  static __device__ __forceinline__ void high_levels(float (&u)[kHigh], uint32_t& l, float (*edge)[64], uint32_t lane,
                                                     float pu, float pd) {
    if constexpr (kCount > 0) {
#pragma unroll 1
      for (; l - kLow + kStep >= kCount && l > kLow; --l) {
        level<kCount>(u, pu, pd);
        edge[l - 1 - kLow][lane] = u[0];
      }
      high_levels<kCount - kStep>(u, l, edge, lane, pu, pd);
    }
  }
  __device__ void run(uint64_t g0, uint64_t g1, uint32_t t) const {
    __shared__ float fac[kLow + kHigh];
    __shared__ float edges[kBlockThreads / 64][kHigh][64];  // a wave's own: [level - kLow][lane]
    const uint32_t tid = thread_index(), lane = tid & 63u, n = p.steps;
    const uint64_t call = (g0 + (uint64_t)t * kGroupsPerTile) * 4 + tid, end = g1 * 4;
    __syncthreads();  // the tile before is done with `fac`
    fac[tid] = factors[tid <= n ? tid : n];
    __syncthreads();
    const float S = reinterpret_cast<const float*>(spots)[call < end ? call : end - 1];
    const float X = p.strike, pu = binomial_constant(p.pu), pd = binomial_constant(p.pd);
    float(*const edge)[64] = edges[tid >> 6];
    if (n >= kLow) {
      float u[kHigh];
#pragma unroll
      for (int k = 0; k < kHigh; ++k) u[k] = binomial_leaf(S, fac[kLow + k], X);
      uint32_t l = n;
      edge[l - kLow][lane] = u[0];
      high_levels<kHigh>(u, l, edge, lane, pu, pd);
    }
    float v[kLow];
#pragma unroll
    for (int k = 0; k < kLow; ++k) v[k] = binomial_leaf(S, fac[k], X);
    uint32_t l = n;
#pragma unroll 1
    for (; l >= kLow; --l) {
      const float top = edge[l - kLow][lane];
      level<kLow>(v, pu, pd);
      v[kLow - 1] = pu * top + pd * v[kLow - 1];
    }
    low_levels<kLow>(v, l, pu, pd);
    if (call < end) reinterpret_cast<float*>(out)[call] = v[0];
  }
};

}  // namespace ce
