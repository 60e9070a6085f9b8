// Per-work-item payload arithmetic on the GPU, shared by the persistent,
// plain and batched kernels. Each function fixes one FP32 operation sequence
// (compiled with -ffp-contract=off) that the host workers repeat exactly.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ce {

// Escape-time count (Mandelbrot program, section 7.2): z <- z^2 + c from 0,
// first n >= 1 with |z_n|^2 > 4, capped at max_iter; one step is x2 = zr zr,
// y2 = zi zi, zi <- fma(zr + zr, zi, ci), zr <- (x2 - y2) + cr.
//
// The main loop takes kBlock steps per test and keeps a = 2 zr, b = 2 zi,
// whose step b <- fma(a, b, 2 ci), a <- fma(a a - b b, 1/2, 2 cr) is five
// instructions with the same roundings (every operation is the plain step's,
// scaled by a power of two). Three facts make its counts those of the plain
// loop, for the c it takes:
//  - |c|^2 <= 3.9999: once |z|^2 > 4 in FP32, |z'| >= |z|^2 - |c| keeps it
//    above 4 by 5e-5 or more, far beyond the rounding, at every later step
//    (to infinity and NaN, which fail the test too). So one test per block
//    sees every escape, and the steps of that block are taken again one by
//    one to find where.
//  - a component of c of at least 2^-20, and ci zero or at least 2^-60: a
//    product that underflows (rounded differently when scaled) is then added
//    to something it is far too small to change, or is the whole of a zr
//    that is itself too small to change the next z.
//  - the step maps (zr, zi) to (zr, zi) and nothing else enters it: when a
//    state comes back bit for bit, the orbit is a cycle without an escape and
//    the count is max_iter. The state is compared with one kept at the last
//    power of two of the step count (Brent's method), so a cycle is found
//    soon after the orbit has entered it. Points inside the set settle into
//    a cycle within some tens to hundreds of steps, where the plain loop runs
//    to max_iter: they are nearly all the work of an image with a high cap.
// Every other c takes the plain loop from the start (|c| > 2 escapes at
// once, c = -2 is a cycle), except that a c below 2^-20 in both components stays below 2^-19.
//
// Bound by FP32 issue, and by the longest orbit of a wave where the image is
// small. A run of the whole set, against four plain steps per test: 8192 x
// 8192 with max_iter 4096 9.75 -> 1.64 ms; 256 x 256 with 256 24.4 -> 19.7 us
// (kernel 13.9 -> 9.1); the batch of 256 jobs 20.2 -> 4.1 ms.
// max_iter must be the same in every lane of the wave; which lanes are still
// in the main loop is kept as one wave-uniform mask, and a lane that has left
// computes on without effect, so that the loop holds no per-lane branch.
__device__ __forceinline__ void escape_step(float& a, float& b, float cr2, float ci2) {
  const float d = a * a - b * b;
  b = __builtin_fmaf(a, b, ci2);
  a = __builtin_fmaf(d, 0.5f, cr2);
}

__device__ __forceinline__ uint32_t escape_count(float cr, float ci, uint32_t max_iter) {
  constexpr uint32_t kBlock = 8;
  const float big = 0x1p-20f, least = 0x1p-60f;
  const float mr = __builtin_fabsf(cr), mi = __builtin_fabsf(ci);
  const uint32_t cap = __builtin_amdgcn_readfirstlane(max_iter);
  const uint32_t lane = __lane_id();
  const float cr2 = cr + cr, ci2 = ci + ci;
  float a = 0.0f, b = 0.0f;    // the state after m steps
  float ea = 0.0f, eb = 0.0f;  // the state after n steps of a lane that has left
  uint32_t m = 0, n = 0;
  const bool tiny = mr < big && mi < big;
  if (tiny) n = cap;
  uint64_t live = __builtin_amdgcn_ballot_w64(!tiny && cr * cr + ci * ci <= 3.9999f && (ci == 0.0f || mi >= least));
  uint64_t escaped = 0, cycled = 0;
  for (uint32_t run = kBlock; live != 0 && m + kBlock <= cap; run *= 2) {
    const uint32_t ka = __float_as_uint(a), kb = __float_as_uint(b);  // the state kept
    const uint32_t stop = cap - m > run ? m + run : cap;
    do {
      float u = a, v = b;
#pragma unroll
      for (uint32_t k = 0; k < kBlock; ++k) escape_step(u, v, cr2, ci2);
      const uint64_t out = live & ~__builtin_amdgcn_ballot_w64(u * u + v * v <= 16.0f);
      if (out != 0) {
        if ((out >> lane) & 1u) {
          ea = a;
          eb = b;
          n = m;
        }
        escaped |= out;
        live &= ~out;
      }
      a = u;
      b = v;
      m += kBlock;
      const uint64_t back = live & __builtin_amdgcn_ballot_w64(__float_as_uint(u) == ka) &
                            __builtin_amdgcn_ballot_w64(__float_as_uint(v) == kb);
      cycled |= back;
      live &= ~back;
    } while (live != 0 && m + kBlock <= stop);
  }
  if (escaped != 0) {
    // where in its block a lane escaped: |z|^2 stays above 4 from there on
    float u = ea, v = eb;
    uint32_t q = n + 1;
#pragma unroll
    for (uint32_t k = 1; k < kBlock; ++k) {
      escape_step(u, v, cr2, ci2);
      q += u * u + v * v <= 16.0f ? 1u : 0u;
    }
    if ((escaped >> lane) & 1u) return q;
  }
  if ((cycled >> lane) & 1u) n = cap;
  if ((live >> lane) & 1u) {
    ea = a;
    eb = b;
    n = m;
  }
  // The plain loop: the last steps before the cap, and every step of the c
  // that the main loop does not take. It looks for cycles too: c = -2, a
  // corner of many images, stays on z = 2.
  float zr = 0.5f * ea, zi = 0.5f * eb, kr = zr, ki = zi;
  while (n < cap) {
    const float x2 = zr * zr;
    const float y2 = zi * zi;
    if (x2 + y2 > 4.0f) break;
    const float t = zr + zr;
    zi = __builtin_fmaf(t, zi, ci);
    zr = (x2 - y2) + cr;
    ++n;
    if (__float_as_uint(zr) == __float_as_uint(kr) && __float_as_uint(zi) == __float_as_uint(ki)) return cap;
    if ((n & (n - 1)) == 0) {
      kr = zr;
      ki = zi;
    }
  }
  return n;
}

}  // namespace ce
