// kk_tri_dev.hpp -- device helpers of the triangular kernels on bit planes
// (kk_hex.hip, kk_ring.hip): bitwise functions, random draws, the decision of
// a word of centres.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kk_common.hpp"
#include "kk_kernels.hpp"
#include "kk_tri.hpp"

namespace kk {
namespace {

constexpr uint32_t kTagTri = 6u, kTagTriOrder = 7u, kTagMpkkK = 8u, kTagMpkk = 9u;

__device__ __forceinline__ uint32_t tri_nb(uint32_t i, uint32_t d, uint32_t L, uint32_t N) {
  // +1, -1, +L, -L, +(L-1), -(L-1) on the ring of N sites
  const uint32_t mag = d < 2 ? 1u : (d < 4 ? L : L - 1u);
  if ((d & 1u) == 0u) {
    const uint32_t j = i + mag;
    return j >= N ? j - N : j;
  }
  return i >= mag ? i - mag : i + N - mag;
}

// Three-input bitwise functions by truth table, a = 0xF0, b = 0xCC, c = 0xAA.
constexpr unsigned kA = 0xF0u, kB = 0xCCu, kC = 0xAAu;
template <unsigned TT>
__device__ __forceinline__ uint32_t lut3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, TT & 0xFFu);
}
__device__ __forceinline__ uint32_t mux(uint32_t s, uint32_t one, uint32_t zero) {
  return lut3<(kA & kB) | (~kA & kC)>(s, one, zero);
}
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return lut3<kA ^ kB ^ kC>(a, b, c); }
__device__ __forceinline__ uint32_t rotr(uint32_t x, uint32_t n) { return __builtin_amdgcn_alignbit(x, x, n); }

// plane = 2 * plane + (u < thr), plane = 2 * plane + (u >= thr): the compare's
// carry goes straight into an add-with-carry.
__device__ __forceinline__ void push_lt(uint32_t& plane, uint32_t u, uint32_t thr) {
  asm("v_cmp_gt_u32_e32 vcc, %2, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc" : "+v"(plane) : "v"(u), "s"(thr) : "vcc");
}
__device__ __forceinline__ void push_ge(uint32_t& plane, uint32_t u, uint32_t thr) {
  asm("v_cmp_le_u32_e32 vcc, %2, %1\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc" : "+v"(plane) : "v"(u), "s"(thr) : "vcc");
}

// The random state of one word of centres, bit by bit: sign and axis (0: +-1,
// 1: +-L, 2: +-(L-1); ax1 = axis >= 1, ax2 = axis == 2) of the direction, and
// U < T for the three thresholds.
struct Draw {
  uint32_t sgn, ax1, ax2, a0, a1, a2;
};

// Philox4x32-10 of counter (b, j, t_lo, t_hi) where only b differs between the
// lanes: the products of t_lo and of the first round's uniform word, and all
// that follows from them, stay in scalar registers, which leaves 18 multiplies
// per block.
struct Head {
  uint32_t u0c, u2x, u3;  // round 1: hi(t_lo M1) ^ j ^ k0 multiplied out, lo(t_lo M1)
  uint32_t th1, k0, k1;
};
__device__ __forceinline__ Head philox_head(uint32_t j, uint32_t tl, uint32_t th, uint32_t k0, uint32_t k1) {
  const uint64_t p1 = (uint64_t)tl * 0xCD9E8D57u;
  const uint64_t p0 = (uint64_t)((uint32_t)(p1 >> 32) ^ j ^ k0) * 0xD2511F53u;
  Head h;
  h.u0c = (uint32_t)p1 ^ (k0 + 0x9E3779B9u);              // round 2's c1 ^ k0
  h.u2x = (uint32_t)(p0 >> 32) ^ (k1 + 0xBB67AE85u);      // round 2's hi(p0) ^ k1
  h.u3 = (uint32_t)p0;                                    // round 2's new c3
  h.th1 = th ^ k1;                                        // round 1's c3 ^ k1
  h.k0 = k0;
  h.k1 = k1;
  return h;
}
__device__ __forceinline__ Philox4 philox_tail(const Head& h, uint32_t b) {
  const uint64_t q0 = (uint64_t)b * 0xD2511F53u;
  uint32_t c2 = (uint32_t)(q0 >> 32) ^ h.th1, c3 = (uint32_t)q0;
  const uint64_t q1 = (uint64_t)c2 * 0xCD9E8D57u;
  uint32_t c0 = (uint32_t)(q1 >> 32) ^ h.u0c, c1 = (uint32_t)q1;
  c2 = h.u2x ^ c3;
  c3 = h.u3;
  uint32_t k0 = h.k0 + 2u * 0x9E3779B9u, k1 = h.k1 + 2u * 0xBB67AE85u;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint64_t p0 = (uint64_t)c0 * 0xD2511F53u;
    const uint64_t p1 = (uint64_t)c2 * 0xCD9E8D57u;
    const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0), n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return Philox4{c0, c1, c2, c3};
}

// One attempt's outcomes shifted into its draw: direction word w, uniform u.
// d = (w * 6) >> 32: d >= 2 and d >= 4 are comparisons of w with 2^33/6 and
// 2^34/6 (rounded up), and d mod 2 is the top bit of 3w mod 2^32.
__device__ __forceinline__ void push_attempt(Draw& q, uint32_t w, uint32_t u, const HexAccept& acc) {
  q.sgn = __builtin_amdgcn_alignbit(q.sgn, (w << 1) + w, 31);
  push_ge(q.ax1, w, 0x55555556u);
  push_ge(q.ax2, w, 0xAAAAAAABu);
  push_lt(q.a0, u, acc.thr[0]);
  push_lt(q.a1, u, acc.thr[1]);
  push_lt(q.a2, u, acc.thr[2]);
}

// The window words a decision reads, aligned to the centre's bits; the centre
// is a, its neighbours e (+1), w (-1), s (+L), n (-L), sw (+(L-1)), ne
// (-(L-1)), and the twelve cells two steps away.
struct Around {
  uint32_t a, e, w, s, n, sw, ne;
  uint32_t e2, w2, s2, n2, sw2, ne2;  // two steps straight on
  uint32_t se, nw;                    // (+1, +1), (-1, -1)
  uint32_t nee, sww;                  // (-1, +2), (+1, -2)
  uint32_t ssw, nne;                  // (+2, -1), (-2, +1)
};

// The accepted centres of a word.  For direction k of the six in cyclic order
// (e, s, sw, w, n, ne) the centre's own neighbours are the three opposite the
// partner and the partner's own are the three beyond it; the two common ones
// add 2 to n whatever they hold.  First the sign picks between each cell and
// its mirror image through the centre, then the axis picks among three.  m = n
// - 1 = 1 (the partner) + unlike own neighbours, in 1..7, is summed relative
// to the centre by a bit-sliced 7 -> 3 counter; slot (m & 3) - 1 holds U < T.
__device__ __forceinline__ uint32_t decide(const Around& v, const Draw& q, uint32_t negmask, uint32_t cmask) {
  const uint32_t s = q.sgn;
  const uint32_t pe = mux(s, v.w, v.e), ps = mux(s, v.n, v.s), psw = mux(s, v.ne, v.sw);
  const uint32_t me = mux(s, v.e, v.w), ms = mux(s, v.s, v.n), msw = mux(s, v.sw, v.ne);
  const uint32_t q1 = mux(s, v.w2, v.e2), q2 = mux(s, v.n2, v.s2), q3 = mux(s, v.ne2, v.sw2);
  const uint32_t q4 = mux(s, v.nw, v.se), q5 = mux(s, v.sww, v.nee), q5m = mux(s, v.nee, v.sww);
  const uint32_t q6 = mux(s, v.nne, v.ssw);
  const uint32_t b = mux(q.ax2, psw, mux(q.ax1, ps, pe));
  const uint32_t x2 = mux(q.ax2, msw, me), x3 = mux(q.ax2, pe, mux(q.ax1, msw, psw));
  const uint32_t y1 = mux(q.ax2, q3, mux(q.ax1, q2, q1));
  const uint32_t y2 = mux(q.ax2, q6, q4), y3 = mux(q.ax2, q5m, mux(q.ax1, q6, q5));
  constexpr unsigned kMaj = (kA & kB) | (kA & kC) | (kB & kC);
  const uint32_t s1 = xor3(ms, x2, x3), c1 = lut3<kMaj>(ms, x2, x3);
  const uint32_t s2 = lut3<~(kA ^ kB ^ kC)>(y1, y2, y3), c2 = lut3<~kMaj>(y1, y2, y3);
  const uint32_t c3 = lut3<kMaj>(s1, s2, b);
  const uint32_t m0 = xor3(s1, s2, b) ^ v.a;
  const uint32_t m1 = xor3(c1, c2, c3) ^ v.a;
  const uint32_t m2 = lut3<kMaj>(c1, c2, c3) ^ v.a;
  const uint32_t live = lut3<kA & (kB ^ kC)>(cmask, v.a, b);
  const uint32_t rm = lut3<~kA & (kB | kC)>(m2 ^ negmask, m0, m1);
  const uint32_t acc = mux(m1, mux(m0, q.a2, q.a1), q.a0);
  return lut3<kA & (~kB | kC)>(live, rm, acc);
}

// The class order of a sweep from Philox blocks 0 .. 3 of the order's counters.
template <class Block>
__host__ __device__ __forceinline__ uint64_t order_of(Block block) {
  uint32_t w[16];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const Philox4 b = block(j);
    w[4 * j] = b.x;
    w[4 * j + 1] = b.y;
    w[4 * j + 2] = b.z;
    w[4 * j + 3] = b.w;
  }
  return shuffle_nibbles(w, 16);
}
// Of sweep t, for a wavefront: a block per lane, and the shuffle in scalar registers.
__device__ __forceinline__ uint64_t hex_order(uint32_t k0, uint32_t k1, uint64_t t) {
  const Philox4 b = philox10(threadIdx.x & 3u, 0u, (uint32_t)t, ctr_hi(t, kTagTriOrder), k0, k1);
  return order_of([&](int j) {
    return Philox4{(uint32_t)__builtin_amdgcn_readlane((int)b.x, j), (uint32_t)__builtin_amdgcn_readlane((int)b.y, j),
                   (uint32_t)__builtin_amdgcn_readlane((int)b.z, j), (uint32_t)__builtin_amdgcn_readlane((int)b.w, j)};
  });
}

// Sum of every thread's count, added to *dst by thread 0.
__device__ __forceinline__ void add_count(uint32_t cnt, uint32_t* total, unsigned long long* dst) {
  for (int off = 32; off > 0; off >>= 1) cnt += __shfl_down(cnt, off, 64);
  if ((threadIdx.x & 63u) == 0u && cnt) atomicAdd(total, cnt);
  __syncthreads();
  if (threadIdx.x == 0 && *total) atomicAdd(dst, (unsigned long long)*total);
}

}  // namespace
}  // namespace kk
