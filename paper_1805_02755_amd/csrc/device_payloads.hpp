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
// The main loop takes 8 or 16 steps per test and keeps a = 2 zr, b = 2 zi,
// whose step b <- fma(a, b, 2 ci), a <- fma(a a - b b, 1/2, 2 cr) is five
// instructions with the same roundings (every operation is the plain step's,
// scaled by a power of two). Four facts make its counts those of the plain
// loop, for the c it takes:
//  - |c|^2 <= 3.9999: once |z|^2 > 4 in FP32, |z'| >= |z|^2 - |c| keeps it
//    above 4 by 5e-5 or more, far beyond the rounding, at every later step
//    (to infinity and NaN, which fail the test too). So one test per block
//    sees every escape, and counting the steps of that block that are still
//    inside finds where.
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
//  - most of these have an attracting fixed point alpha = alpha^2 + c, and are
//    done sooner: where |2 alpha| + s <= 0.99, no orbit leaves the disc of
//    radius s around alpha, since there |z' - alpha| = |z - alpha| |z - alpha +
//    2 alpha| <= 0.99 s. What FP32 adds, the rounding of a step (below 1e-6)
//    and the residual of the alpha found (below 1e-5: s >= 2^-8 keeps its
//    square root away from the cut), is less than the 0.01 s left. Left of
//    -3/4 the same holds for two steps and a cycle of two, beta near 0 and
//    -1 - beta, whose multiplier is 4 (c + 1): |z'' - beta| <= r (|4 (c + 1)| +
//    r (|2 (1 + beta)| + (|2 beta| + r)^2)) for |z - beta| <= r, at even steps.
//    The disc is looked at where a state is kept. 8192 x 8192, max_iter 256:
//    391 us without, 303 with the fixed point's, 287 with both; 4096: 904, 757,
//    727.
// Every other c takes the plain loop from the start (|c| > 2 escapes at
// once, c = -2 is a cycle), except that a c below 2^-20 in both components
// stays below 2^-19.
//
// The first block counts as it goes (most points outside escape in it); later
// blocks only test, and the block an orbit escaped in is taken again. Blocks
// of 16 from step 64 on halve what a block costs besides its steps.
//
// Bound by FP32 issue, and by the longest orbit where the image is small. A
// run on the GPU alone, against four plain steps per test (and rows of 512
// pixels dealt by tickets): the whole set at 8192 x 8192 with max_iter 4096
// 9.0 -> 0.73 ms, 1920 x 1080 with 1000 368 -> 47 us, 1024 x 1024 with 256
// 40 -> 26 us, 256 x 256 24 -> 18 us (of which 15 are the launch and the
// wait for it). max_iter must be the same in every lane of the wave; which
// lanes are still in the main loop is kept as one wave-uniform mask, and a lane
// that has left computes on without effect, so that the loop holds no per-lane
// branch.
struct EscapeOrbit {
  float cr2, ci2;              // 2 c
  float a = 0.0f, b = 0.0f;    // 2 z after m steps
  float ea = 0.0f, eb = 0.0f;  // 2 z after n steps, of a lane that has left
  float lr, li, near2;         // 2 alpha or 2 beta, and the square of the disc's 2 s; negative: no disc
  uint32_t lane, m = 0, n = 0;
  uint64_t live = 0;           // lanes in the main loop
  uint64_t escaped = 0;        // lanes that left it in the block from step n on
  uint64_t cycled = 0;         // lanes that left it in a cycle
  __device__ __forceinline__ void step(float& x, float& y) const {
    const float d = x * x - y * y;
    y = __builtin_fmaf(x, y, ci2);
    x = __builtin_fmaf(d, 0.5f, cr2);
  }
  static __device__ __forceinline__ bool inside(float x, float y) { return x * x + y * y <= 16.0f; }
  __device__ __forceinline__ bool has(uint64_t mask) const { return ((mask >> lane) & 1u) != 0; }
  // The disc, from q = sqrt(1 - 4 c), 2 alpha = 1 - q, or with a c left of
  // -3/4 q = sqrt(-3 - 4 c), 2 beta = q - 1. A q of zero gives a NaN, which no
  // distance is below.
  __device__ __forceinline__ void find_disc() {
    const bool two = cr2 < -1.5f;
    const float dr = __builtin_fmaf(cr2, -2.0f, two ? -3.0f : 1.0f), di = -2.0f * ci2;
    const float d = __builtin_amdgcn_sqrtf(__builtin_fmaf(dr, dr, di * di));  // |q|^2
    const float re = __builtin_amdgcn_sqrtf(0.5f * (d + dr)), im = 0.5f * di * __builtin_amdgcn_rcpf(re);
    const float g = 1.0f - re, f = 1.0f - dr, t = __builtin_amdgcn_sqrtf(__builtin_fmaf(g, g, im * im));
    const float l = __builtin_amdgcn_sqrtf(__builtin_fmaf(f, f, di * di));  // |4 (c + 1)| of a c left of -3/4
    const float k = t + 0.4f;
    const float s = two ? __builtin_fminf((0.99f - l) * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_sqrtf(d) + k * k), 0.4f)
                        : 0.99f - t;
    lr = two ? -g : g;
    li = two ? im : -im;
    near2 = s >= 0x1p-8f ? 4.0f * s * s : -1.0f;
  }
  // Lanes whose orbit has entered the disc that it cannot leave.
  __device__ __forceinline__ void test_disc() {
    const float x = a - lr, y = b - li;
    const uint64_t in = live & __builtin_amdgcn_ballot_w64(__builtin_fmaf(x, x, y * y) <= near2);
    cycled |= in;
    live &= ~in;
  }
  // Blocks of kBlock steps while a lane is left and the next block ends by `stop`.
  template <uint32_t kBlock>
  __device__ __forceinline__ void blocks(uint32_t stop) {
    if (live == 0 || m + kBlock > stop) return;
    test_disc();
    if (live == 0) return;
    const uint32_t ka = __float_as_uint(a), kb = __float_as_uint(b);  // the state kept
    do {
      float u = a, v = b;
#pragma unroll
      for (uint32_t k = 0; k < kBlock; ++k) step(u, v);
      const uint64_t out = live & ~__builtin_amdgcn_ballot_w64(inside(u, v));
      if (out != 0) {
        if (has(out)) {
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
};

__device__ __forceinline__ uint32_t escape_count(float cr, float ci, uint32_t max_iter) {
  constexpr uint32_t kFirst = 8, kLong = 64;
  const float big = 0x1p-20f, least = 0x1p-60f;
  const float mr = __builtin_fabsf(cr), mi = __builtin_fabsf(ci);
  const uint32_t cap = __builtin_amdgcn_readfirstlane(max_iter);
  EscapeOrbit o;
  o.lane = __lane_id();
  o.cr2 = cr + cr;
  o.ci2 = ci + ci;
  const bool tiny = mr < big && mi < big;
  uint32_t q = tiny ? cap : 0u;  // the count, of a lane that has one
  bool counted = tiny;
  const bool fast = !tiny && cr * cr + ci * ci <= 3.9999f && (ci == 0.0f || mi >= least);
  if (kFirst <= cap) {
    float u = 0.0f, v = 0.0f;
    uint32_t in = 1;
    bool last = false;
#pragma unroll
    for (uint32_t k = 1; k <= kFirst; ++k) {
      o.step(u, v);
      last = EscapeOrbit::inside(u, v);
      if (k < kFirst) in += last ? 1u : 0u;
    }
    if (fast && !last) {
      q = in;
      counted = true;
    }
    o.live = __builtin_amdgcn_ballot_w64(fast && last);
    o.a = u;
    o.b = v;
    o.m = kFirst;
    // to steps 16, 32, 64 in blocks of 8, then to each power of two in blocks
    // of 16, the state at each start kept for the cycle test
    if (o.live != 0) o.find_disc();
    uint32_t next = 2 * kFirst;
    for (; o.live != 0 && o.m + kFirst <= cap && next <= kLong; next *= 2) o.blocks<8>(next < cap ? next : cap);
    for (; o.live != 0 && o.m + 16 <= cap; next *= 2) o.blocks<16>(next < cap ? next : cap);
    o.blocks<8>(cap);
    if (o.escaped != 0) {
      float x = o.ea, y = o.eb;
      uint32_t e = o.n + 1;
#pragma unroll
      for (uint32_t k = 1; k < 8; ++k) {
        o.step(x, y);
        e += EscapeOrbit::inside(x, y) ? 1u : 0u;
      }
      if (o.m > kLong) {  // some block may have been one of 16
#pragma unroll
        for (uint32_t k = 8; k < 16; ++k) {
          o.step(x, y);
          e += EscapeOrbit::inside(x, y) ? 1u : 0u;
        }
      }
      if (o.has(o.escaped)) {
        q = e;
        counted = true;
      }
    }
    if (o.has(o.cycled)) {
      q = cap;
      counted = true;
    }
  }
  if (counted) return q;
  // The plain loop: the last steps before the cap, and every step of the c
  // that the main loop does not take. It looks for cycles too: c = -2, a
  // corner of many images, stays on z = 2.
  uint32_t n = o.has(o.live) ? o.m : 0u;
  float zr = n != 0 ? 0.5f * o.a : 0.0f, zi = n != 0 ? 0.5f * o.b : 0.0f, kr = zr, ki = zi;
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
