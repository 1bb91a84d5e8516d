// kk_sweep.hip -- the Kawasaki sweep kernel (the hot loop).
//
// One launch performs complete sweeps (8 class phases each) on LDS-resident
// tiles of the lattice, stored one bit per site.  Each 32-bit LDS word holds
// 32 consecutive sites of a row; a phase touches every 4th bit of every
// other row, and the 8 centres of a word are decided together with bitwise
// (SWAR) logic against the word's 12 bit-sliced random planes.
//
// Two tile modes:
//  * halo tiles (one word and 16 rows per sweep on each side): two sweeps per
//    launch with 32 rows, or one with 16.  A phase's dependency radius is 2
//    sites, so a sweep's 8 phases leave the interior exact while the outermost
//    16 rows / 16 bits of the halo may be stale (32 of both after two sweeps:
//    the one word is enough for them); the counter-based random numbers make
//    the redundant halo work reproduce exactly what the neighbouring tile
//    computes.
//  * cyclic tile (whole lattice, L % 32 == 0): rows and words wrap inside
//    LDS, so no halo exists and any number of sweeps runs in one launch.
//
// Within a phase all chosen pairs are at L1 distance >= 2 from one another
// (classes 2*((x - y) mod 4) + (y mod 2)), so no pair writes a site that
// another pair reads: the LDS updates are xor-flips of disjoint bits issued
// with ds_xor, and a workgroup barrier separates phases.
#include <algorithm>
#include <type_traits>

#include "kk_common.hpp"
#include "kk_kernels.hpp"

namespace kk {

namespace {

__device__ __forceinline__ uint32_t sel4(uint32_t d1, uint32_t d0, uint32_t v0, uint32_t v1, uint32_t v2,
                                         uint32_t v3) {
  // direction (d1 d0): 0 -> v0 (+x), 1 -> v1 (-x), 2 -> v2 (+y), 3 -> v3 (-y), per bit
  const uint32_t lo = (d0 & v1) | (~d0 & v0);
  const uint32_t hi = (d0 & v3) | (~d0 & v2);
  return (d1 & hi) | (~d1 & lo);
}

__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
  return (a & b) | (a & c) | (b & c);
}

// Pack 32 bytes (each 0 or 1) into one word, byte b -> bit b.
__device__ __forceinline__ uint32_t pack4(uint32_t d) {
  return (d | (d >> 7) | (d >> 14) | (d >> 21)) & 0xFu;
}

// Spread 4 bits into 4 bytes (bit b -> byte b, value 0/1).
__device__ __forceinline__ uint32_t spread4(uint32_t n) {
  return (n * 0x00204081u) & 0x01010101u;
}

template <int LAYOUT>
__device__ uint32_t load_word(const SweepParams& p, int yv, int Xw) {
  const int L = p.L;
  const int y = imod(yv, L);
  if (LAYOUT == kLayoutBits) {
    const int xw = imod(Xw, L);  // a multiple of 32: the bit-packed layout needs L % 32 == 0
    return static_cast<const uint32_t*>(p.src)[(size_t)y * p.wpr + (xw >> 5)];
  } else {
    const uint8_t* row = static_cast<const uint8_t*>(p.src) + (size_t)y * L;
    if (Xw >= 0 && Xw + 32 <= L) {
      uint32_t v = 0;
      if ((L & 15) == 0) {
        const uint4* d = reinterpret_cast<const uint4*>(row + Xw);
        const uint4 a = d[0], b = d[1];
        v = pack4(a.x) | (pack4(a.y) << 4) | (pack4(a.z) << 8) | (pack4(a.w) << 12) | (pack4(b.x) << 16) |
            (pack4(b.y) << 20) | (pack4(b.z) << 24) | (pack4(b.w) << 28);
      } else {
        const uint32_t* d = reinterpret_cast<const uint32_t*>(row + Xw);
#pragma unroll
        for (int k = 0; k < 8; ++k) v |= pack4(d[k]) << (4 * k);
      }
      return v;
    }
    uint32_t v = 0;
    for (int b = 0; b < 32; ++b) v |= (uint32_t)(row[imod(Xw + b, L)] & 1u) << b;
    return v;
  }
}

// Store the low `nbits` sites of word v at true coordinates (x0, y).
template <int LAYOUT>
__device__ void store_word(const SweepParams& p, int y, int x0, uint32_t v, int nbits) {
  if (LAYOUT == kLayoutBits) {
    static_cast<uint32_t*>(p.dst)[(size_t)y * p.wpr + (x0 >> 5)] = v;
  } else {
    uint8_t* row = static_cast<uint8_t*>(p.dst) + (size_t)y * p.L;
    if (nbits == 32) {
      if ((p.L & 15) == 0) {
        uint4* d = reinterpret_cast<uint4*>(row + x0);
        d[0] = make_uint4(spread4(v & 0xFu), spread4((v >> 4) & 0xFu), spread4((v >> 8) & 0xFu),
                          spread4((v >> 12) & 0xFu));
        d[1] = make_uint4(spread4((v >> 16) & 0xFu), spread4((v >> 20) & 0xFu), spread4((v >> 24) & 0xFu),
                          spread4(v >> 28));
      } else {
        uint32_t* d = reinterpret_cast<uint32_t*>(row + x0);
#pragma unroll
        for (int k = 0; k < 8; ++k) d[k] = spread4((v >> (4 * k)) & 0xFu);
      }
    } else {
      // a ragged last word: nbits is a multiple of 4 (x0 and L are)
      uint32_t* d = reinterpret_cast<uint32_t*>(row + x0);
      for (int k = 0; k < nbits / 4; ++k) d[k] = spread4((v >> (4 * k)) & 0xFu);
    }
  }
}

// The 12 random planes of the 32 virtual sites starting at virtual x = Xw in
// virtual row yv for sweep t.  Segment-aligned windows take the three Philox
// blocks of their segment directly; windows that straddle the periodic wrap
// of an L % 32 != 0 lattice (or L < 32) gather from the segments they cover.
__device__ void gen_planes(const SweepParams& p, int yv, int Xw, uint64_t t, uint32_t* pl) {
  const int L = p.L;
  const uint32_t y = (uint32_t)imod(yv, L);
  const uint32_t tl = (uint32_t)t, thi = ctr_hi(t, kTagSweep);
  const int x0 = imod(Xw, L);
  if ((x0 & 31) == 0 && x0 + 32 <= L) {
    const uint32_t g4 = (uint32_t)(x0 >> 5) * 4u;
    const Philox4 a = philox10(y, g4 + 0u, tl, thi, p.k0, p.k1);
    const Philox4 b = philox10(y, g4 + 1u, tl, thi, p.k0, p.k1);
    const Philox4 c = philox10(y, g4 + 2u, tl, thi, p.k0, p.k1);
    pl[0] = a.x; pl[1] = a.y; pl[2] = a.z; pl[3] = a.w;
    pl[4] = b.x; pl[5] = b.y; pl[6] = b.z; pl[7] = b.w;
    pl[8] = c.x; pl[9] = c.y; pl[10] = c.z; pl[11] = c.w;
    return;
  }
#pragma unroll
  for (int k = 0; k < kPlanes; ++k) pl[k] = 0u;
  int b = 0;
  while (b < 32) {
    const int x = imod(Xw + b, L);
    const int off = x & 31;
    int len = 32 - off;
    if (L - x < len) len = L - x;
    if (32 - b < len) len = 32 - b;
    const uint32_t g4 = (uint32_t)(x >> 5) * 4u;
    const Philox4 q0 = philox10(y, g4 + 0u, tl, thi, p.k0, p.k1);
    const Philox4 q1 = philox10(y, g4 + 1u, tl, thi, p.k0, p.k1);
    const Philox4 q2 = philox10(y, g4 + 2u, tl, thi, p.k0, p.k1);
    const uint32_t P[12] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w, q2.x, q2.y, q2.z, q2.w};
    const uint32_t m = (len == 32) ? 0xFFFFFFFFu : ((1u << len) - 1u);
#pragma unroll
    for (int k = 0; k < kPlanes; ++k) pl[k] |= ((P[k] >> off) & m) << b;
    b += len;
  }
}


// Bit-packed or int8 word at true row y, 32 sites from true x0 (which may
// straddle the periodic wrap only when L % 32 != 0 or L < 32).
template <int LAYOUT>
__device__ __forceinline__ uint32_t load_word_at(const SweepParams& p, int y, int x0) {
  if (LAYOUT == kLayoutBits) return static_cast<const uint32_t*>(p.src)[(size_t)y * p.wpr + (x0 >> 5)];
  const int L = p.L;
  const uint8_t* row = static_cast<const uint8_t*>(p.src) + (size_t)y * L;
  if (x0 + 32 <= L) {
    uint32_t v = 0;
    if ((L & 15) == 0) {
      const uint4* d = reinterpret_cast<const uint4*>(row + x0);
      const uint4 a = d[0], b = d[1];
      v = pack4(a.x) | (pack4(a.y) << 4) | (pack4(a.z) << 8) | (pack4(a.w) << 12) | (pack4(b.x) << 16) |
          (pack4(b.y) << 20) | (pack4(b.z) << 24) | (pack4(b.w) << 28);
    } else {
      const uint32_t* d = reinterpret_cast<const uint32_t*>(row + x0);
#pragma unroll
      for (int k = 0; k < 8; ++k) v |= pack4(d[k]) << (4 * k);
    }
    return v;
  }
  // the word passes the end of the row: eight 4-byte pieces, each inside the
  // row (x0 and L are multiples of 4), the start of each wrapped; the loads
  // are independent, so they are all in flight at once
  uint32_t v = 0;
  int x = x0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    v |= pack4(*reinterpret_cast<const uint32_t*>(row + x)) << (4 * k);
    x += 4;
    if (x >= L) x -= L;
  }
  return v;
}

// A word of 32 sites as loaded, packed later, so that the loads of several
// words are in flight together.  GRID: L % 32 == 0, no word passes the wrap;
// else an int8 word is eight 4-byte pieces, the start of each wrapped.
template <int LAYOUT>
struct RawWord {
  uint32_t d[LAYOUT == kLayoutBits ? 1 : 8];
  template <bool GRID>
  __device__ __forceinline__ void load(const SweepParams& p, int y, int x0) {
    if constexpr (LAYOUT == kLayoutBits) {
      d[0] = static_cast<const uint32_t*>(p.src)[(size_t)y * p.wpr + (x0 >> 5)];
    } else {
      const uint8_t* row = static_cast<const uint8_t*>(p.src) + (size_t)y * p.L;
      if constexpr (GRID) {
        const uint4* q = reinterpret_cast<const uint4*>(row + x0);
        const uint4 a = q[0], b = q[1];
        d[0] = a.x, d[1] = a.y, d[2] = a.z, d[3] = a.w, d[4] = b.x, d[5] = b.y, d[6] = b.z, d[7] = b.w;
      } else {
        int x = x0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          d[k] = *reinterpret_cast<const uint32_t*>(row + x);
          x += 4;
          x = x >= p.L ? x - p.L : x;
        }
      }
    }
  }
  __device__ __forceinline__ uint32_t word() const {
    if constexpr (LAYOUT == kLayoutBits) {
      return d[0];
    } else {
      uint32_t v = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) v |= pack4(d[k]) << (4 * k);
      return v;
    }
  }
};

// Layout chosen at run time (LAYOUT == 0) or at compile time.
template <int LAYOUT>
__device__ __forceinline__ uint32_t load_word_any(const SweepParams& p, int y, int x0) {
  if constexpr (LAYOUT == 0)
    return p.layout == kLayoutBits ? load_word_at<kLayoutBits>(p, y, x0) : load_word_at<kLayoutInt8>(p, y, x0);
  else
    return load_word_at<LAYOUT>(p, y, x0);
}

template <int LAYOUT>
__device__ __forceinline__ void store_word_any(const SweepParams& p, int y, int x0, uint32_t v, int nbits) {
  if constexpr (LAYOUT == 0) {
    if (p.layout == kLayoutBits) store_word<kLayoutBits>(p, y, x0, v, nbits);
    else store_word<kLayoutInt8>(p, y, x0, v, nbits);
  } else {
    store_word<LAYOUT>(p, y, x0, v, nbits);
  }
}

// Three-input bitwise function with a truth table built from the operand
// patterns a = 0xF0, b = 0xCC, c = 0xAA (one v_bitop3_b32).
#define KK_TA 0xF0u
#define KK_TB 0xCCu
#define KK_TC 0xAAu
#define KK_TT(expr) ((unsigned)((expr) & 0xFFu))
template <unsigned TT>
__device__ __forceinline__ uint32_t bop3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, TT);
}
// a ? b : c, per bit
__device__ __forceinline__ uint32_t bsel(uint32_t a, uint32_t b, uint32_t c) {
  return bop3<KK_TT((KK_TA & KK_TB) | (~KK_TA & KK_TC))>(a, b, c);
}
constexpr unsigned kXor3 = KK_TT(KK_TA ^ KK_TB ^ KK_TC);
constexpr unsigned kMaj3 = KK_TT((KK_TA & KK_TB) | (KK_TA & KK_TC) | (KK_TB & KK_TC));

// 10-bit (u < K) and (u == K) over bit-sliced u, planes[2] = MSB .. planes[11] = LSB,
// for a K that is the same on every lane.  Less-than is the borrow chain of
// u - K from the least significant bit, lt' = maj(~u_k, K_k, lt), one
// three-input op per bit; equality is the AND of u_k XNOR K_k, one XNOR per bit
// and a tree of three-input ANDs.
__device__ __forceinline__ void cmp10(const uint32_t* pl, uint32_t K, uint32_t& lt, uint32_t& eq,
                                      uint32_t bin = 0u, uint32_t em = 0xFFFFFFFFu) {
  constexpr unsigned kBorrow = KK_TT((~KK_TA & KK_TB) | (~KK_TA & KK_TC) | (KK_TB & KK_TC));
  constexpr unsigned kAnd3 = KK_TT(KK_TA & KK_TB & KK_TC);
  uint32_t l = bin, x[10];
#pragma unroll
  for (int k = 0; k < 10; ++k) {
    const uint32_t u = pl[11 - k];
    const uint32_t kb = 0u - ((K >> k) & 1u);
    l = bop3<kBorrow>(u, kb, l);
    x[k] = ~(u ^ kb);
  }
  lt = l;
  eq = bop3<kAnd3>(bop3<kAnd3>(bop3<kAnd3>(x[0], x[1], x[2]), bop3<kAnd3>(x[3], x[4], x[5]),
                                bop3<kAnd3>(x[6], x[7], x[8])),
                   x[9], em);
}

template <bool CYC>
__device__ __forceinline__ unsigned sweep_item(uint32_t* S, const SweepParams& p, int stride, int r, int w,
                                               const uint32_t* pl, uint32_t cmask, uint32_t intmask, int yv,
                                               int Xw, uint64_t t) {
  int rn, rs, rnn, rss, wl, wr;
  if (CYC) {
    const int R = p.R, C = p.C;
    rn = (r == 0) ? R - 1 : r - 1;
    rs = (r + 1 == R) ? 0 : r + 1;
    rnn = (rn == 0) ? R - 1 : rn - 1;
    rss = (rs + 1 == R) ? 0 : rs + 1;
    wl = (w == 0) ? C - 1 : w - 1;
    wr = (w + 1 == C) ? 0 : w + 1;
  } else {
    rn = r - 1;
    rs = r + 1;
    rnn = r - 2;
    rss = r + 2;
    wl = w - 1;  // the pad words at -1 and C are never part of a result
    wr = w + 1;
  }
#define KK_AT(rr, ww) S[(rr) * stride + (ww) + 1]
  const uint32_t c0 = KK_AT(r, w), cL = KK_AT(r, wl), cR = KK_AT(r, wr);
  const uint32_t n0 = KK_AT(rn, w), nL = KK_AT(rn, wl), nR = KK_AT(rn, wr);
  const uint32_t s0 = KK_AT(rs, w), sL = KK_AT(rs, wl), sR = KK_AT(rs, wr);
  const uint32_t nn = KK_AT(rnn, w), ss = KK_AT(rss, w);

  // value of the site at x+1 / x-1 / x+2 / x-2, aligned to bit x
  const uint32_t cE = __builtin_amdgcn_alignbit(cR, c0, 1);
  const uint32_t cW = __builtin_amdgcn_alignbit(c0, cL, 31);
  const uint32_t cE2 = __builtin_amdgcn_alignbit(cR, c0, 2);
  const uint32_t cW2 = __builtin_amdgcn_alignbit(c0, cL, 30);
  const uint32_t nE = __builtin_amdgcn_alignbit(nR, n0, 1);
  const uint32_t nW = __builtin_amdgcn_alignbit(n0, nL, 31);
  const uint32_t sE = __builtin_amdgcn_alignbit(sR, s0, 1);
  const uint32_t sW = __builtin_amdgcn_alignbit(s0, sL, 31);

  const uint32_t d0 = pl[0], d1 = pl[1];
  // partner b: +x east, -x west, +y the row below (y+1), -y the row above
  const uint32_t B = sel4(d1, d0, cE, cW, s0, n0);
  const uint32_t A = (c0 ^ B) & cmask;  // centres of this class whose partner is unlike

  // m = n + 1 = (unlike neighbours of c, partner included) + (neighbours of b
  // other than c that equal c, i.e. are unlike b)
  const uint32_t o1 = sel4(d1, d0, cE2, cW2, ss, nn);
  const uint32_t o2 = sel4(d1, d0, nE, nW, sW, nW);
  const uint32_t o3 = sel4(d1, d0, sE, sW, sE, nE);
  const uint32_t uE = c0 ^ cE, uW = c0 ^ cW, uN = c0 ^ n0, uS = c0 ^ s0;
  const uint32_t e1 = ~(c0 ^ o1), e2 = ~(c0 ^ o2), e3 = ~(c0 ^ o3);
  const uint32_t s1 = uE ^ uW ^ uN, c1 = maj3(uE, uW, uN);
  const uint32_t s2 = uS ^ e1 ^ e2, c2 = maj3(uS, e1, e2);
  const uint32_t m0 = s1 ^ s2 ^ e3, c3 = maj3(s1, s2, e3);
  const uint32_t m1 = c1 ^ c2 ^ c3, m2 = maj3(c1, c2, c3);

  uint32_t F = A;  // accepted exchanges
  if (p.acc.restricted) {
    uint32_t lt0, eq0, lt1, eq1, lt2, eq2;
    if (p.acc.hi[0] < 1024u) cmp10(pl, p.acc.hi[0], lt0, eq0); else { lt0 = 0xFFFFFFFFu; eq0 = 0u; }
    if (p.acc.hi[1] < 1024u) cmp10(pl, p.acc.hi[1], lt1, eq1); else { lt1 = 0xFFFFFFFFu; eq1 = 0u; }
    if (p.acc.hi[2] < 1024u) cmp10(pl, p.acc.hi[2], lt2, eq2); else { lt2 = 0xFFFFFFFFu; eq2 = 0u; }
    const uint32_t rm = ~(m2 ^ p.acc.negmask) & (m0 | m1);  // m in the rejectable range
    const uint32_t ltsel = (m1 & ((m0 & lt2) | (~m0 & lt1))) | (~m1 & lt0);
    const uint32_t eqsel = (m1 & ((m0 & eq2) | (~m0 & eq1))) | (~m1 & eq0);
    F = A & (~rm | ltsel);
    uint32_t tie = A & rm & eqsel;
    while (tie) {  // u10 equals the threshold prefix: draw the low 32 bits
      const int bp = __builtin_ctz(tie);
      tie &= tie - 1u;
      const uint32_t x = (uint32_t)imod(Xw + bp, p.L), y = (uint32_t)imod(yv, p.L);
      const Philox4 e = philox10(y, x >> 2, (uint32_t)t, ctr_hi(t, kTagExt), p.k0, p.k1);
      const uint32_t xs = x & 3u;
      const uint32_t ext = xs == 0 ? e.x : xs == 1 ? e.y : xs == 2 ? e.z : e.w;
      const uint32_t j = ((((m1 >> bp) & 1u) << 1) | ((m0 >> bp) & 1u)) - 1u;
      const uint32_t lo = j == 0 ? p.acc.lo[0] : j == 1 ? p.acc.lo[1] : p.acc.lo[2];
      if (ext < lo) F |= 1u << bp;
    }
  }

  const uint32_t Fpx = F & ~d1 & ~d0, Fmx = F & ~d1 & d0;
  const uint32_t Fpy = F & d1 & ~d0, Fmy = F & d1 & d0;
  const uint32_t flip = F ^ (Fpx << 1) ^ (Fmx >> 1);
  if (flip) atomicXor(&KK_AT(r, w), flip);
  if (Fpx >> 31) atomicXor(&KK_AT(r, wr), 1u);
  if (Fmx & 1u) atomicXor(&KK_AT(r, wl), 0x80000000u);
  if (Fpy) atomicXor(&KK_AT(rs, w), Fpy);
  if (Fmy) atomicXor(&KK_AT(rn, w), Fmy);
#undef KK_AT
  return (unsigned)__builtin_popcount(F & intmask);
}

template <int LAYOUT, bool CYC, int KU>
__global__ __launch_bounds__(KU == 1 ? 1024 : 768) void sweep_kernel(SweepParams p) {
  extern __shared__ uint32_t S[];
  const int stride = p.C + 2;
  const int tile = blockIdx.x;
  const int tx = tile % p.tiles_x, ty = tile / p.tiles_x;
  const int X0 = tx * p.tww * 32, Y0 = ty * p.th;
  const int XL = X0 - 32 * p.hx;  // virtual x of LDS word 0
  const int YT = Y0 - p.hy;       // virtual y of LDS row 0
  const int xend = min(X0 + p.tww * 32, p.L);  // interior is [X0, xend) x [Y0, yend)
  const int yend = min(Y0 + p.th, p.L);

  // stage the tile (with halo) into LDS, one bit per site
  for (int i = threadIdx.x; i < p.R * stride; i += blockDim.x) {
    const int r = i / stride, w = i - r * stride - 1;
    S[i] = (w >= 0 && w < p.C) ? load_word<LAYOUT>(p, YT + r, XL + 32 * w) : 0u;
  }

  // units owned by this thread: (row pair q, word w); rows r0 = row0 + 2q and r0 + 1
  int ur0[KU], uw[KU];
  bool uok[KU];
#pragma unroll
  for (int k = 0; k < KU; ++k) {
    const int u = threadIdx.x + k * blockDim.x;
    uok[k] = u < p.nunits;
    const int q = uok[k] ? u / p.C : 0;
    uw[k] = uok[k] ? u - q * p.C : 0;
    ur0[k] = p.row0 + 2 * q;
  }
  // interior bit masks of each owned word (for counting accepted moves)
  uint32_t imask[KU][2];
#pragma unroll
  for (int k = 0; k < KU; ++k) {
    const int Xw = XL + 32 * uw[k];
    uint32_t wm = 0u;
    if (Xw + 32 <= X0 || Xw >= xend) wm = 0u;
    else {
      const int lo = max(Xw, X0), hi = min(Xw + 32, xend);
      const int n = hi - lo, sh = lo - Xw;
      wm = (n == 32 ? 0xFFFFFFFFu : ((1u << n) - 1u)) << sh;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int yv = YT + ur0[k] + h;
      imask[k][h] = (uok[k] && yv >= Y0 && yv < yend) ? wm : 0u;
    }
  }

  unsigned count = 0;
  for (int s = 0; s < p.nsweeps; ++s) {
    const uint64_t t = p.t0 + (uint64_t)s;
    uint32_t pl[KU][2][kPlanes];
#pragma unroll
    for (int k = 0; k < KU; ++k) {
      if (!uok[k]) continue;
#pragma unroll
      for (int h = 0; h < 2; ++h) gen_planes(p, YT + ur0[k] + h, XL + 32 * uw[k], t, pl[k][h]);
    }
    const uint32_t perm = class_order(p.k0, p.k1, t);
    __syncthreads();  // staging (or the previous sweep) complete
    for (int ph = 0; ph < 8; ++ph) {
      const uint32_t cls = (perm >> (4 * ph)) & 0xFu;
      const int a = (int)(cls >> 1);
      // Every unit starts on an even virtual row (tiles start on even rows and
      // the halo is even), so the active row of the pair is row r0 + (class
      // parity): uniform over the workgroup, which keeps the plane arrays in
      // registers.
      if ((cls & 1u) == 0u) {
#pragma unroll
        for (int k = 0; k < KU; ++k) {
          if (!uok[k]) continue;
          const int yv = YT + ur0[k];
          count += sweep_item<CYC>(S, p, stride, ur0[k], uw[k], pl[k][0], 0x11111111u << ((a + yv) & 3),
                                   imask[k][0], yv, XL + 32 * uw[k], t);
        }
      } else {
#pragma unroll
        for (int k = 0; k < KU; ++k) {
          if (!uok[k]) continue;
          const int yv = YT + ur0[k] + 1;
          count += sweep_item<CYC>(S, p, stride, ur0[k] + 1, uw[k], pl[k][1], 0x11111111u << ((a + yv) & 3),
                                   imask[k][1], yv, XL + 32 * uw[k], t);
        }
      }
      __syncthreads();
    }
  }

  // write the interior back
  const int iw = (xend - X0 + 31) / 32, ih = yend - Y0;
  for (int i = threadIdx.x; i < iw * ih; i += blockDim.x) {
    const int rr = i / iw, ww = i - rr * iw;
    const int x0 = X0 + 32 * ww;
    const int nb = min(32, xend - x0);
    const uint32_t v = S[(p.hy + rr) * stride + p.hx + ww + 1];
    store_word<LAYOUT>(p, Y0 + rr, x0, nb == 32 ? v : (v & ((1u << nb) - 1u)), nb);
  }

  // Accepted-move count: reduce over the workgroup, then one plain
  // read-modify-write of this tile's own partial sum.  (One device-scope
  // atomic per wave on a single address serialises across the XCDs and
  // cost more than the sweep itself.)
  unsigned c = count;
  for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
  unsigned* red = reinterpret_cast<unsigned*>(S + p.R * stride);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long tot = 0;
    for (int wv = 0; wv < (int)(blockDim.x >> 6); ++wv) tot += red[wv];
    p.accepted[tile] += tot;
  }
}


// Per-row random state for one sweep: the two direction planes and, for each
// of the three rejectable classes of moves (slot j), the plane of sites whose
// 42-bit uniform U = u10 * 2^32 + ext32 lies below the slot's threshold T_j.
// The 10-bit prefix decides every site whose u10 differs from T_j's top bits;
// for the others (about 3 sites in 1024 per slot) the low word ext32 is drawn
// here, once per sweep, so the phases decide with bitwise logic alone and
// never branch on a tie.
struct RowRand {
  uint32_t d0, d1, acc0, acc1, acc2;
};

// The threshold prefixes pass through an empty asm so that their per-bit masks
// are rebuilt (a few scalar ops) at every use instead of being hoisted and
// kept live across the kernel, which overflows the scalar registers.
__device__ __forceinline__ uint32_t opaque_sgpr(uint32_t v) {
  asm volatile("" : "+s"(v));
  return v;
}

// Ties: u10 equals a threshold prefix, and the low 32 bits of U decide.  About
// one row word in eleven has one, so that resolving them where they arise runs
// a Philox block or two per row word for a few lanes of the wave.  Instead a
// wave lists the ties of all its row words in LDS and resolves the list once,
// a tie per lane (six ties per wave and row word on average); a row word's ties
// share three words of results (one per slot), which its lane then joins to its
// planes.  No other wave is involved, so no barrier is needed.
constexpr uint32_t kTieCap = 64;                      // listed ties per wave; further ones are resolved in place
constexpr uint32_t kTieWaveWords = kTieCap * (2 + 3);  // an entry and three result words each
struct TieList {
  uint2* entry;   // site (y << 16 | x); result index << 8 | bit << 3 | slots
  uint32_t* out;  // three words per result index
  uint32_t n;     // listed so far (uniform)
};
__device__ __forceinline__ TieList tie_list(uint32_t* lds) {  // lds: 8-byte aligned, kTieWaveWords per wave
  uint32_t* w = lds + kTieWaveWords * (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  return TieList{reinterpret_cast<uint2*>(w), w + 2 * kTieCap, 0u};
}

__device__ __forceinline__ uint32_t tie_word(const SweepParams& p, uint32_t y, uint32_t x, uint64_t t) {
  const Philox4 e = philox10(y, x >> 2, (uint32_t)t, ctr_hi(t, kTagExt), p.k0, p.k1);
  const uint32_t s1 = 0u - (x & 1u), s2 = 0u - ((x >> 1) & 1u);
  return bsel(s2, bsel(s1, e.w, e.z), bsel(s1, e.y, e.x));
}

// eq[j] holds the tied sites of slot j among the 32 sites from true column
// xtrue of true row ytrue (xtrue + b may pass the wrap only for L % 32 != 0 or
// L < 32).  Returns the result index of the row word, -1 without ties.
__device__ __forceinline__ int list_ties(const SweepParams& p, TieList& tl, int ytrue, int xtrue, uint64_t t,
                                         const uint32_t* eq, uint32_t* lt) {
  uint32_t tie = eq[0] | eq[1] | eq[2];
  int idx = -1;
  for (;;) {
    const uint64_t m = __ballot(tie != 0u);
    if (!m) break;
    if (tie) {
      const int bp = __builtin_ctz(tie);
      tie &= tie - 1u;
      int x = xtrue + bp;
      if (x >= p.L) x = imod(x, p.L);
      const uint32_t slots = ((eq[0] >> bp) & 1u) | (((eq[1] >> bp) & 1u) << 1) | (((eq[2] >> bp) & 1u) << 2);
      const uint32_t pos =
          tl.n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      if (pos < kTieCap) {
        if (idx < 0) {
          idx = (int)pos;
          tl.out[3 * pos] = tl.out[3 * pos + 1] = tl.out[3 * pos + 2] = 0u;
        }
        tl.entry[pos] =
            make_uint2(((uint32_t)ytrue << 16) | (uint32_t)x, ((uint32_t)idx << 8) | ((uint32_t)bp << 3) | slots);
      } else {
        const uint32_t ext = tie_word(p, (uint32_t)ytrue, (uint32_t)x, t);
#pragma unroll
        for (int j = 0; j < 3; ++j)
          if (((slots >> j) & 1u) && ext < p.acc.lo[j]) lt[j] |= 1u << bp;
      }
    }
    tl.n += (uint32_t)__popcll(m);
  }
  return idx;
}

// The wave's list, once; after it join_ties may be called.
__device__ __forceinline__ void resolve_list(const SweepParams& p, const TieList& tl, uint64_t t) {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const uint32_t i = threadIdx.x & 63u;
  if (i < min(tl.n, kTieCap)) {
    const uint2 e = tl.entry[i];
    const uint32_t ext = tie_word(p, e.x >> 16, e.x & 0xFFFFu, t);
    uint32_t* out = tl.out + 3 * (e.y >> 8);
#pragma unroll
    for (int j = 0; j < 3; ++j)
      if (((e.y >> j) & 1u) && ext < p.acc.lo[j]) atomicOr(&out[j], 1u << ((e.y >> 3) & 31u));
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

__device__ __forceinline__ void join_ties(const TieList& tl, int idx, RowRand& q) {
  if (idx >= 0) {
    q.acc0 |= tl.out[3 * idx];
    q.acc1 |= tl.out[3 * idx + 1];
    q.acc2 |= tl.out[3 * idx + 2];
  }
}

// Rounds R0 .. R1 - 1 of N Philox4x32-10 blocks at once, round by round across
// the blocks: the multiplies of different blocks are independent and issue back
// to back instead of waiting on one block's chain.  c0..c3: counters in,
// outputs out.
template <int N, int R0 = 0, int R1 = 10>
__device__ __forceinline__ void philox10_n(uint32_t* c0, uint32_t* c1, uint32_t* c2, uint32_t* c3, uint32_t k0,
                                           uint32_t k1) {
  k0 += (uint32_t)R0 * 0x9E3779B9u;
  k1 += (uint32_t)R0 * 0xBB67AE85u;
#pragma unroll
  for (int r = R0; r < R1; ++r) {
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const uint64_t p0 = (uint64_t)c0[n] * 0xD2511F53u;
      const uint64_t p1 = (uint64_t)c2[n] * 0xCD9E8D57u;
      const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1[n], k0, 0x96);
      const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3[n], k1, 0x96);
      c1[n] = (uint32_t)p1;
      c3[n] = (uint32_t)p0;
      c0[n] = n0;
      c2[n] = n2;
    }
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

// u10 < K and u10 == K over the planes (2 .. 11: bits 9 .. 0 of u10) for a
// slot's threshold prefix K = hi.  Each bit of K becomes one all-zeros /
// all-ones scalar mask (a signed one-bit field extract) for the borrow chain
// and the equality chain, one three-input op per bit and chain.  A prefix of
// 1024 or more accepts every site: its compare runs with a borrow-in (u < 1023
// + 1) and an empty equality mask instead of a branch.
__device__ __forceinline__ void compare_slot(const uint32_t* pl, uint32_t hi, bool live, uint32_t& lt, uint32_t& eq) {
  constexpr unsigned kBorrow = KK_TT((~KK_TA & KK_TB) | (~KK_TA & KK_TC) | (KK_TB & KK_TC));
  constexpr unsigned kEqStep = KK_TT(KK_TA & ~(KK_TB ^ KK_TC));
  const bool all = hi >= 1024u;
  const uint32_t K = opaque_sgpr(all ? 1023u : hi);
  lt = all ? 0xFFFFFFFFu : 0u;
  eq = all || !live ? 0u : 0xFFFFFFFFu;
#pragma unroll
  for (int k = 0; k < 10; ++k) {
    const uint32_t kb = (uint32_t)((int32_t)(K << (31 - k)) >> 31);
    lt = bop3<kBorrow>(pl[11 - k], kb, lt);
    eq = bop3<kEqStep>(eq, pl[11 - k], kb);
  }
}

// The 12 planes of segment g (32 sites from 32 g) of true row y.
__device__ __forceinline__ void segment_planes(const SweepParams& p, uint64_t t, int y, int g, uint32_t* pl) {
  const uint32_t tl = (uint32_t)t, thi = ctr_hi(t, kTagSweep);
  uint32_t c0[3], c1[3], c2[3], c3[3];
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    c0[b] = (uint32_t)y;
    c1[b] = (uint32_t)g * 4u + (uint32_t)b;
    c2[b] = tl;
    c3[b] = thi;
  }
  philox10_n<3>(c0, c1, c2, c3, p.k0, p.k1);
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    pl[4 * b] = c0[b];
    pl[4 * b + 1] = c1[b];
    pl[4 * b + 2] = c2[b];
    pl[4 * b + 3] = c3[b];
  }
}

// Random state of the row word of 32 sites from true column x of true row y:
// its three Philox blocks are drawn together, then its compares.  Off-grid
// lattices (GRID false: L % 32 != 0) have a few words that do not sit on the
// 32-site segment grid, next to the wrap; those gather their planes from the
// segments they cover, where a wave holds any: one or two more draws for the
// wave (drawing all of a word's segments anew, block by block: 1036^2 8.5 us per
// sweep, now 7.7; 400^2 6.3, now 5.8; twelve 400^2 lattices 11.4, now 10.0).
// Returns the index of the row word's tie results, -1 without ties or for a
// lane that owns no unit (live false).
template <bool GRID>
__device__ __forceinline__ int rand_row(const SweepParams& p, TieList& ties, uint64_t t, int y, int x, bool live,
                                        RowRand& q) {
  uint32_t pl[kPlanes];
  segment_planes(p, t, y, x >> 5, pl);
  if constexpr (!GRID) {
    const bool gather = live && ((x & 31) != 0 || x + 32 > p.L);
    if (__any(gather)) {
      if (gather) {  // the planes above are the first segment's; the rest of the word from those that follow
        int n = min(32 - (x & 31), p.L - x);  // sites of the first segment
        const uint32_t m = n == 32 ? 0xFFFFFFFFu : (1u << n) - 1u;
#pragma unroll
        for (int k = 0; k < kPlanes; ++k) pl[k] = (pl[k] >> (x & 31)) & m;
        int xs = x + n;  // a whole segment's start, or the wrap
#pragma unroll 1
        while (n < 32) {
          xs = xs >= p.L ? 0 : xs;
          uint32_t seg[kPlanes];
          segment_planes(p, t, y, xs >> 5, seg);
          const int len = min(32, p.L - xs);  // what lies past bit 31 is shifted out
          const uint32_t ms = len == 32 ? 0xFFFFFFFFu : (1u << len) - 1u;
#pragma unroll
          for (int k = 0; k < kPlanes; ++k) pl[k] |= (seg[k] & ms) << n;
          n += len;
          xs += len;
        }
      }
    }
  }
  uint32_t lt[3], eq[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) compare_slot(pl, p.acc.hi[j], live, lt[j], eq[j]);
  const int idx = list_ties(p, ties, y, x, t, eq, lt);
  q = RowRand{pl[0], pl[1], lt[0], lt[1], lt[2]};
  return idx;
}


// Decide the exchanges of the centres in `cmask` of one 32-site word.
// v: the word (0), its west/east neighbours (1, 2), the same three in the
// row above (3..5) and below (6..8), and the words two rows above / below
// (9, 10).  Returns the accepted centres.
__device__ __forceinline__ uint32_t decide_word(const uint32_t* v, const RowRand& q, const SweepParams& p,
                                                uint32_t cmask) {
  const uint32_t c0 = v[0], n0 = v[3], s0 = v[6];
  const uint32_t cE = __builtin_amdgcn_alignbit(v[2], c0, 1);
  const uint32_t cW = __builtin_amdgcn_alignbit(c0, v[1], 31);
  const uint32_t cE2 = __builtin_amdgcn_alignbit(v[2], c0, 2);
  const uint32_t cW2 = __builtin_amdgcn_alignbit(c0, v[1], 30);
  const uint32_t nE = __builtin_amdgcn_alignbit(v[5], n0, 1);
  const uint32_t nW = __builtin_amdgcn_alignbit(n0, v[4], 31);
  const uint32_t sE = __builtin_amdgcn_alignbit(v[8], s0, 1);
  const uint32_t sW = __builtin_amdgcn_alignbit(s0, v[7], 31);
  const uint32_t d0 = q.d0, d1 = q.d1;
  // direction (d1 d0): 0 +x east, 1 -x west, 2 +y the row below, 3 -y the row above.
  // B: the partner; o1..o3: the partner's neighbours other than the centre.
  const uint32_t B = bsel(d1, bsel(d0, n0, s0), bsel(d0, cW, cE));
  const uint32_t o1 = bsel(d1, bsel(d0, v[9], v[10]), bsel(d0, cW2, cE2));
  const uint32_t o2 = bsel(bop3<KK_TT(KK_TA & ~KK_TB)>(d1, d0, d0), sW, bsel(d0, nW, nE));
  const uint32_t o3 = bsel(d0, bsel(d1, nE, sW), sE);
  const uint32_t A = bop3<KK_TT(KK_TA & (KK_TB ^ KK_TC))>(cmask, c0, B);  // active: unlike partner
  // m = n + 1 = #(neighbours of c unlike c, partner included) + #(o_i equal to c),
  // summed by a bit-sliced 7 -> 3 counter written relative to c so the xors with c cancel
  const uint32_t X1 = bop3<kXor3>(cE, cW, n0);
  const uint32_t M1 = bop3<kMaj3>(cE, cW, n0);
  const uint32_t X2 = bop3<kXor3>(s0, o1, o2);
  const uint32_t M2 = bop3<KK_TT((KK_TA & ~KK_TB) | (KK_TA & ~KK_TC) | (~KK_TB & ~KK_TC))>(s0, o1, o2);
  const uint32_t M3 = bop3<KK_TT((KK_TA & KK_TB) | (KK_TA & ~KK_TC) | (KK_TB & ~KK_TC))>(X1, X2, o3);
  const uint32_t m0 = ~(bop3<kXor3>(X1, X2, o3) ^ c0);
  const uint32_t m1 = bop3<kXor3>(M1, M2, M3) ^ c0;
  const uint32_t m2 = bop3<kMaj3>(M1, M2, M3) ^ c0;
  // rejectable: m in {1,2,3} for omega > 0 (dU = 6,4,2), {5,6,7} for omega < 0;
  // slot j = (m & 3) - 1 holds the acceptance plane of that move class.  No
  // branch on omega == 0: there every slot's plane is all ones.  (A branch
  // here split the neighbourhood reads into two LDS round trips per unit.)
  const uint32_t rm = bop3<KK_TT(~KK_TA & (KK_TB | KK_TC))>(m2 ^ p.acc.negmask, m0, m1);
  const uint32_t accsel = bsel(m1, bsel(m0, q.acc2, q.acc1), q.acc0);
  return bop3<KK_TT(KK_TA & (~KK_TB | KK_TC))>(A, rm, accsel);
}

// LDS row stride of a row of C words: at least C + 2 (one pad word each side),
// and congruent to C/2 modulo 32 so that the words a phase touches (every other
// row, consecutive words) fall in consecutive LDS banks.
__host__ __device__ constexpr int halo_stride(int C) { return C % 2 == 0 ? C / 2 + 32 : 34; }
template <int TWW>
struct HaloGeom {
  static constexpr int C = TWW + 2;  // LDS words per row: the tile plus one halo word each side
  static constexpr int ST = halo_stride(C);
};

// LDS words of a halo tile of R rows of C words before the tie lists (an even
// number): the rows, 16 spare words and the row and column tables.
__host__ __device__ constexpr int halo_tie_offset(int R, int C) { return (R * halo_stride(C) + 16 + R + C + 1) & ~1; }

// One phase of the halo kernel for the thread's units, active row = r0 + H.
// Branch-free over the units: a unit beyond the tile reads a valid word and
// has an empty centre mask, so it decides nothing and writes nothing.
template <int ST, int KU, int H>
__device__ __forceinline__ unsigned halo_phase(uint32_t* S, const SweepParams& p, const int* base0,
                                               const uint32_t* okm, const RowRand (*rr)[2],
                                               const uint32_t (*imask)[2], int a) {
  uint32_t v[KU][11];
#pragma unroll
  for (int k = 0; k < KU; ++k) {
    const int b = base0[k] + H * ST;
    v[k][0] = S[b];
    v[k][1] = S[b - 1];
    v[k][2] = S[b + 1];
    v[k][3] = S[b - ST];
    v[k][4] = S[b - ST - 1];
    v[k][5] = S[b - ST + 1];
    v[k][6] = S[b + ST];
    v[k][7] = S[b + ST - 1];
    v[k][8] = S[b + ST + 1];
    v[k][9] = S[b - 2 * ST];
    v[k][10] = S[b + 2 * ST];
  }
  uint32_t F[KU];
#pragma unroll
  for (int k = 0; k < KU; ++k) {
    // class mask: the unit's base pattern rotated left by a (its period is 4)
    const uint32_t cmask = __builtin_amdgcn_alignbit(okm[k * 2 + H], okm[k * 2 + H], (32 - a) & 31);
    F[k] = decide_word(v[k], rr[k][H], p, cmask);
  }
  unsigned count = 0;
#pragma unroll
  for (int k = 0; k < KU; ++k) {
    const uint32_t d0 = rr[k][H].d0, d1 = rr[k][H].d1;
    const uint32_t f = F[k];
    const uint32_t Fpx = bop3<KK_TT(KK_TA & ~KK_TB & ~KK_TC)>(f, d1, d0);
    const uint32_t Fmx = bop3<KK_TT(KK_TA & ~KK_TB & KK_TC)>(f, d1, d0);
    const uint32_t Fpy = bop3<KK_TT(KK_TA & KK_TB & ~KK_TC)>(f, d1, d0);
    const uint32_t Fmy = bop3<KK_TT(KK_TA & KK_TB & KK_TC)>(f, d1, d0);
    const int b = base0[k] + H * ST;
    // centres of one class sit 4 sites apart, so f, Fpx << 1 and Fmx >> 1
    // never share a bit and their xor is their or.  Zero masks are harmless:
    // every update goes out unconditionally (the two carries into the
    // neighbouring words are mostly zero, but a masked store costs more issue
    // slots than an xor with zero, and skipping a wave's carries when none is
    // set measured slower: 16.45 against 16.1 us per 4096^2 sweep at one sweep
    // per launch of 16 x 128 tiles)
    atomicXor(&S[b], (Fpx << 1) | f | (Fmx >> 1));
    atomicXor(&S[b + ST], Fpy);
    atomicXor(&S[b - ST], Fmy);
    atomicXor(&S[b + 1], Fpx >> 31);
    atomicXor(&S[b - 1], Fmx << 31);
    count += (unsigned)__builtin_popcount(f & imask[k][H]);
  }
  return count;
}

// Sum over a wavefront of a per-lane count below 256, from eight ballots
// (scalar popcounts; no LDS round trip).
__device__ __forceinline__ unsigned wave_sum8(unsigned c) {
  unsigned s = 0;
#pragma unroll
  for (int b = 0; b < 8; ++b) s += (unsigned)__popcll(__ballot((c >> b) & 1u)) << b;
  return s;
}

// Halo-tile sweep with a compile-time tile width: the LDS row stride is a
// constant, so every neighbour of a unit is an immediate offset from one
// base address.  Each thread owns KU (row pair, word) units; their random
// state lives in registers for the whole sweep.  In a phase the thread reads
// the neighbourhoods of all its units before issuing any exchange (the
// conflict-free schedule makes that reordering exact), so the LDS latency of
// the second unit hides behind the first.
// One sweep of tile `tile` of the lattice described by p (halo mode), `order`
// the sweep's class order.  What bounds it: at 4096^2 (256 tiles of 8 x 256, in
// turn, 28.3 us per launch) VALU issue: of a workgroup's 63000 cycles 3000 are
// staging, 29000 the two sweeps' draws, 30000 their phases, 1000 the stores.  On
// small lattices, whose tiles have one or two waves per sweep, the chain of them:
// 400^2 (tiles of 1 x 24, side by side, 11.7 us per launch), 24400 cycles: 3500
// tables and loads, 8500 draws, ties and packing, 12300 the 16 phases (with one
// sweep per launch 12.9 -> 10.2 us, 1036^2 14.7 -> 12.6 us: loads without a branch
// between them, ties in one list, spare lanes on words of their own).
// Two sweeps in one launch: the window has 16 more rows on each side (its halo
// columns, 32, are enough for two sweeps as they are), and the launch, the
// staging and the stores are paid once.
// kSideBySide: the first half_threads threads hold the first sweep's units,
// which reach 16 rows beyond the tile's own halo, the rest the second's, so that
// both sweeps' draws run at once (400^2 10.2 -> 6.6 us per sweep, 1036^2 12.6 ->
// 9.2, 1024^2 9.3 -> 6.4, tiles unchanged).  kInTurn: all threads do one sweep,
// then the other, for tiles whose two sweeps need more threads than a workgroup
// has (4096^2 15.6 -> 14.3 us per sweep).
enum HaloMode { kOneSweep, kSideBySide, kInTurn };
// With `sweeps` 1 the second is left out (a batch's replica whose run ends).
// Returns the workgroup's accepted count for the tile interior (the same in
// every thread).
__host__ __device__ constexpr int halo_rows(int th, int ns) { return th + 32 * ns; }
__host__ __device__ constexpr int halo_pairs(int th, int ns, int sweep) { return (halo_rows(th, ns - sweep) - 4) / 2; }
// Threads for the units of one of the two sweeps.
__host__ __device__ constexpr int half_threads(int th, int C, int KU, int sweep) {
  return ((halo_pairs(th, 2, sweep) * C + KU - 1) / KU + 63) & ~63;
}

template <int LAYOUT, int TWW, int KU, HaloMode MODE>
__device__ __forceinline__ unsigned halo_tile_sweep(uint32_t* S, const SweepParams& p, int tile, uint32_t order0,
                                                    uint32_t order1, int sweeps = 2) {
  constexpr int NS = MODE == kOneSweep ? 1 : 2;
  constexpr int C = HaloGeom<TWW>::C;
  constexpr int ST = HaloGeom<TWW>::ST;
  const int CP = C + 2;       // staged words per row (the pads included)
  constexpr int NSTG = 4;     // staged global words per thread
  const int tx = tile % p.tiles_x, ty = tile / p.tiles_x;
  constexpr int TW = TWW;
  const int X0 = tx * TW * 32, Y0 = ty * p.th;
  const int XL = X0 - 32, YT = Y0 - 16 * NS;
  const int xend = min(X0 + TW * 32, p.L), yend = min(Y0 + p.th, p.L);
  const int R = halo_rows(p.th, NS);
  const int total = R * CP;
  // side by side: the sweep this thread's units belong to, and its place among their threads
  int mine = 0, tid = (int)threadIdx.x, nthreads = (int)blockDim.x;
  if constexpr (MODE == kSideBySide) {
    const int ta = half_threads(p.th, C, KU, 0);
    mine = __builtin_amdgcn_readfirstlane(tid >= ta ? 1 : 0);
    tid -= mine ? ta : 0;
    nthreads = mine ? nthreads - ta : ta;
  }
  // LDS words that can reach the interior: the left halo word, the interior
  // words and one halo word past them.  In a ragged last tile the words after
  // that behave like the zero pad of a full tile: they are neither loaded nor
  // computed (for L % 32 != 0 they would also sit off the 32-site segment grid).
  const int wneed = min(C, (xend - X0 + 31) / 32 + 2);
  // true (wrapped) row of every LDS row and true column of every LDS word
  int* ytab = reinterpret_cast<int*>(S + R * ST + 16);
  int* xtab = ytab + R;
  for (int i = threadIdx.x; i < R + C; i += blockDim.x) {
    if (i < R) ytab[i] = imod(YT + i, p.L);
    else xtab[i - R] = imod(XL + 32 * (i - R), p.L);
  }
  // the workgroup's accepted count, in the gap between the rows and the
  // tables; the tie lists after the tables
  uint32_t* acc_total = S + R * ST;
  TieList ties = tie_list(S + halo_tie_offset(R, C));
  if (threadIdx.x == 0) *acc_total = 0u;
  __syncthreads();

  // Global loads first; they complete while the random state is computed.  No
  // branch stands between them (a lane without a word loads a valid one and
  // drops it), so that all are in flight together.
  RawWord<LAYOUT> stg[NSTG];
  auto load_words = [&](auto on_grid) {
#pragma unroll
    for (int j = 0; j < NSTG; ++j) {
      const int i = min((int)(threadIdx.x + j * blockDim.x), total - 1);
      const int r = i / CP, w = max(i - r * CP - 1, 0);
      if (j * (int)blockDim.x < total) stg[j].template load<decltype(on_grid)::value>(p, ytab[r], xtab[min(w, wneed - 1)]);
    }
  };
  if ((p.L & 31) == 0) load_words(std::true_type{});
  else load_words(std::false_type{});
  for (int i = threadIdx.x + NSTG * blockDim.x; i < total; i += blockDim.x) {
    const int r = i / CP, w = i - r * CP - 1;
    S[r * ST + w + 1] = (w >= 0 && w < wneed) ? load_word_at<LAYOUT>(p, ytab[r], xtab[w]) : 0u;
  }

  // one sweep of the window: the thread's units, their draws, the phases
  auto sweep = [&](int sw, auto first) {
    const int npairs = halo_pairs(p.th, NS, sw), nunits = npairs * C;
    const uint64_t t = p.t0 + (uint64_t)sw;
    ties.n = 0u;
    int base0[KU];         // LDS base
    uint32_t okm[KU * 2];  // class-0 centre pattern of each row (0 for a unit beyond the tile)
    uint32_t imask[KU][2];
    RowRand rr[KU][2];
    int tie[KU][2];              // index of each row word's tie results
    int ry[KU * 2], rx[KU * 2];  // true row and column of each of the thread's rows
    bool okk[KU];
#pragma unroll
    for (int k = 0; k < KU; ++k) {
      const int u = tid + k * nthreads;
      const bool in = u < nunits;
      // A lane beyond the tile's units shares the place of an earlier unit, one
      // each: its exchanges are empty, but xors of one wave to one LDS word run
      // one after another, and 40 lanes on one word cost more than the phase.
      const int v = in ? u : (u - nunits < nunits ? u - nunits : 0);
      int q, wu;
      if ((p.L & 31) == 0) {
        q = v / C;
        wu = v - q * C;
      } else {
        // off-grid lattices: the two edge words of every row gather their random
        // planes from two or three segments; numbering them after all inner
        // words confines that slower path to the last waves
        const int nin = npairs * (C - 2);
        if (v < nin) {
          q = v / (C - 2);
          wu = 1 + (v - q * (C - 2));
        } else {
          const int e = v - nin;
          q = e >> 1;
          wu = (e & 1) ? C - 1 : 0;
        }
      }
      const bool ok = in && wu < wneed && (MODE != kSideBySide || sw < sweeps);
      const int w = ok ? wu : 0;
      const int r0 = 2 + 16 * sw + 2 * q;
      base0[k] = r0 * ST + wu + 1;  // also for a word past wneed, which holds the zero pad
      // class a = 0 centres of a row with virtual y sit at x = y (mod 4); the
      // virtual x of bit 0 is a multiple of 32
      okm[2 * k] = ok ? (0x11111111u << ((YT + r0) & 3)) : 0u;
      okm[2 * k + 1] = ok ? (0x11111111u << ((YT + r0 + 1) & 3)) : 0u;
      const int Xw = XL + 32 * w;
      uint32_t wm = 0u;
      if (Xw + 32 > X0 && Xw < xend) {
        const int lo = max(Xw, X0), hi = min(Xw + 32, xend);
        const int n = hi - lo;
        wm = (n == 32 ? 0xFFFFFFFFu : ((1u << n) - 1u)) << (lo - Xw);
      }
      okk[k] = ok;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int yv = YT + r0 + h;
        imask[k][h] = (ok && yv >= Y0 && yv < yend) ? wm : 0u;
        ry[2 * k + h] = ytab[r0 + h];
        rx[2 * k + h] = xtab[w];
      }
    }
    // row by row (a lane beyond the tile's units draws for a valid row and
    // decides nothing: its centre masks are empty); a wave whose units of one
    // index all lie beyond the tile skips them.  Drawing more rows at once, to
    // overlap more Philox chains, measured slower: 16.3 us per 4096^2 sweep for a
    // unit's two rows, 18.7 us for all four rows of a thread, against 16.2 us row
    // by row (at one sweep per launch of 16 x 128 tiles).
    auto draw_rows = [&](auto on_grid) {
#pragma unroll
      for (int k = 0; k < KU; ++k) {
        if (__any(okk[k])) {
#pragma unroll
          for (int h = 0; h < 2; ++h)
            tie[k][h] = rand_row<decltype(on_grid)::value>(p, ties, t, ry[2 * k + h], rx[2 * k + h], okk[k], rr[k][h]);
        } else {
          rr[k][0] = rr[k][1] = RowRand{0u, 0u, 0u, 0u, 0u};
          tie[k][0] = tie[k][1] = -1;
        }
      }
  };
  if ((p.L & 31) == 0) draw_rows(std::true_type{});
  else draw_rows(std::false_type{});
  resolve_list(p, ties, t);
#pragma unroll
  for (int k = 0; k < KU; ++k)
#pragma unroll
    for (int h = 0; h < 2; ++h) join_ties(ties, tie[k][h], rr[k][h]);
  if constexpr (decltype(first)::value) {
#pragma unroll
    for (int j = 0; j < NSTG; ++j) {
      const int i = threadIdx.x + j * blockDim.x;
      const int r = i / CP, w = i - r * CP;
      if (i < total) S[r * ST + w] = w >= 1 && w <= wneed ? stg[j].word() : 0u;
    }
    __syncthreads();
  }
  const uint32_t perm = sw ? order1 : order0;

  unsigned count = 0;
  const bool last = KU == 1 || __any(okk[KU - 1]);  // uniform: this wave has all its units
#pragma unroll 1
  for (int ph = 0; ph < (MODE == kSideBySide ? 8 * sweeps : 8); ++ph) {
    if (MODE == kSideBySide && (ph >> 3) != sw) {  // the other sweep's phase
      __syncthreads();
      continue;
    }
    const uint32_t cls = (perm >> (4 * (ph & 7))) & 0xFu;
    const int a = (int)(cls >> 1);
    // pairs start on even rows, so the active row of every pair is the class
    // parity: a uniform branch keeps each row's random state in registers
    if (last) {
      if (cls & 1u) count += halo_phase<ST, KU, 1>(S, p, base0, okm, rr, imask, a);
      else count += halo_phase<ST, KU, 0>(S, p, base0, okm, rr, imask, a);
    } else {
      if (cls & 1u) count += halo_phase<ST, 1, 1>(S, p, base0, okm, rr, imask, a);
      else count += halo_phase<ST, 1, 0>(S, p, base0, okm, rr, imask, a);
    }
    if ((ph & 7) == 7) {  // each wave adds its count before the last barrier
      const unsigned ws = wave_sum8(count);
      if ((threadIdx.x & 63) == 0) atomicAdd(acc_total, ws);
    }
    __syncthreads();
  }
  };
  sweep(mine, std::true_type{});
  if (MODE == kInTurn && sweeps == 2) sweep(1, std::false_type{});

  // write the interior back (a full-width tile divides by a constant)
  const int iw = (xend - X0 + 31) / 32, ih = yend - Y0;
  if (xend - X0 == TW * 32) {
    for (int i = threadIdx.x; i < TW * ih; i += blockDim.x) {
      const int rr2 = i / TW, ww = i - rr2 * TW;
      store_word<LAYOUT>(p, Y0 + rr2, X0 + 32 * ww, S[(16 * NS + rr2) * ST + 1 + ww + 1], 32);
    }
  } else {
    for (int i = threadIdx.x; i < iw * ih; i += blockDim.x) {
      const int rr2 = i / iw, ww = i - rr2 * iw;
      const int x0 = X0 + 32 * ww;
      const int nb = min(32, xend - x0);
      const uint32_t val = S[(16 * NS + rr2) * ST + 1 + ww + 1];
      store_word<LAYOUT>(p, Y0 + rr2, x0, nb == 32 ? val : (val & ((1u << nb) - 1u)), nb);
    }
  }

  return *acc_total;
}

// Block-wide sum of the per-thread accepted counts, added to *dst by thread 0.
__device__ __forceinline__ void add_block_count(uint32_t* red_lds, unsigned count, unsigned long long* dst) {
  unsigned c = count;
  for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red_lds[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long tot = 0;
    for (int wv = 0; wv < (int)(blockDim.x >> 6); ++wv) tot += red_lds[wv];
    // one workgroup per address: an add without a returned value does not wait
    // for a read of the old sum at the end of the kernel
    atomicAdd(dst, tot);
  }
}

template <int LAYOUT, int TWW, int KU, HaloMode MODE>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4))) void halo_kernel(SweepParams p,
                                                                                               uint32_t order0,
                                                                                               uint32_t order1) {
  extern __shared__ __attribute__((aligned(16))) uint32_t S[];
  const unsigned total =
      halo_tile_sweep<LAYOUT, TWW, KU, MODE>(S, p, xcd_tile((int)blockIdx.x, (int)gridDim.x), order0, order1);
  // one workgroup per address: an add without a returned value does not wait
  // for a read of the old sum at the end of the kernel
  if (threadIdx.x == 0) atomicAdd(p.accepted + blockIdx.x, (unsigned long long)total);
}

// ---------------------------------------------------------------------------
// Cyclic lattices (2 .. kResidentMaxC words per row): a sweep is a chain of draws
// and eight phases, so the draws run ahead of it.  The first PW wavefronts hold
// KU units per lane and do nothing but phases; RW others draw the next sweep's
// random state (NT row words per lane) into LDS between the phases' barriers:
// in eight slices, each shorter than a phase, where a lane draws up to three
// row words (SLICED), else a whole row word in each of the intervals 1 .. NT.
// The phase waves take a sweep's draws into registers in the first interval,
// before any of the next sweep's are written.  The class orders of the launch's
// sweeps are computed before the first, a sweep per lane.  Rows and words wrap
// through addresses held per lane, so no cell has a second copy to keep (at two
// words per row every exchange had up to three).
//
// Up to six words per row a phase is one wave's latency (about 600 cycles), with
// more of them the SIMDs' issue rate bounds it.  Per sweep, one wave set doing
// draws and phases in turn -> this: 64^2 4.9 -> 2.0 us, 128^2 6.0 -> 2.8, 160^2
// 7.9 -> 4.4, 192^2 8.2 -> 6.0, 224^2 10.6 -> 7.8, 256^2 9.9 -> 8.9, 288^2 19.7
// -> 11.5.
// ---------------------------------------------------------------------------
constexpr int kPipeMaxSweeps = 256;  // per launch (class orders held in LDS)
template <int C>
struct Pipe {
  static constexpr int RC = 32 * C * C;                       // row words (R = 32 C)
  static constexpr int KU = C <= 6 ? 1 : (C <= 8 ? 2 : 3);    // units per lane of a phase wave
  static constexpr int PW = (RC / 2 + 64 * KU - 1) / (64 * KU);
  static constexpr int T = (RC + 63) / 64;                    // waves of row words
  static constexpr int NT = C <= 4 ? 1 : (C == 5 ? 2 : (C <= 7 ? 3 : (C == 8 ? 4 : 5)));
  static constexpr bool SLICED = C <= 6;
  static constexpr int RW = (T + NT - 1) / NT;
  static constexpr int kThreads = 64 * (PW + RW);
  static constexpr int kWords = RC + 5 * RC + kPipeMaxSweeps + RW * (int)kTieWaveWords + 16;
  static_assert(kThreads <= 1024 && NT <= 7 && kWords % 2 == 0, "wave roles");
};

// A unit's words: row base addresses of rows r0 - 2 .. r0 + 3, word w and its
// two neighbours.
struct PipeUnit {
  int row[6], w, we, ww;
};

template <int KU, int H>
__device__ __forceinline__ unsigned pipe_phase(uint32_t* S, const SweepParams& p, const PipeUnit* u,
                                               const RowRand (*rr)[2], const uint32_t (*ok)[2], const bool* live,
                                               uint32_t turn) {
  uint32_t v[KU][11];
#pragma unroll
  for (int k = 0; k < KU; ++k) {
    const int* r = u[k].row + H;  // rows -2 .. +2 around the active one
    const int w = u[k].w, we = u[k].we, ww = u[k].ww;
    v[k][0] = S[r[2] + w];
    v[k][1] = S[r[2] + ww];
    v[k][2] = S[r[2] + we];
    v[k][3] = S[r[1] + w];
    v[k][4] = S[r[1] + ww];
    v[k][5] = S[r[1] + we];
    v[k][6] = S[r[3] + w];
    v[k][7] = S[r[3] + ww];
    v[k][8] = S[r[3] + we];
    v[k][9] = S[r[0] + w];
    v[k][10] = S[r[4] + w];
  }
  unsigned count = 0;
#pragma unroll
  for (int k = 0; k < KU; ++k) {
    const int* r = u[k].row + H;
    const RowRand& q = rr[k][H];
    const uint32_t f = decide_word(v[k], q, p, __builtin_amdgcn_alignbit(ok[k][H], ok[k][H], turn));
    if (live[k]) {
      const uint32_t px = bop3<KK_TT(KK_TA & ~KK_TB & ~KK_TC)>(f, q.d1, q.d0);
      const uint32_t mx = bop3<KK_TT(KK_TA & ~KK_TB & KK_TC)>(f, q.d1, q.d0);
      atomicXor(&S[r[2] + u[k].w], (px << 1) | f | (mx >> 1));
      atomicXor(&S[r[3] + u[k].w], bop3<KK_TT(KK_TA & KK_TB & ~KK_TC)>(f, q.d1, q.d0));
      atomicXor(&S[r[1] + u[k].w], bop3<KK_TT(KK_TA & KK_TB & KK_TC)>(f, q.d1, q.d0));
      atomicXor(&S[r[2] + u[k].we], px >> 31);
      atomicXor(&S[r[2] + u[k].ww], mx << 31);
    }
    count += (unsigned)__builtin_popcount(f);
  }
  return count;
}

// Whole lattice in one workgroup, p.nsweeps (at most kPipeMaxSweeps) sweeps
// from p.t0.  Threads beyond Pipe<C>::kThreads only take part in the staging
// and the barriers.  Returns the thread's accepted count.
template <int LAYOUT, int C>
__device__ __forceinline__ unsigned pipe_sweeps(uint32_t* S, const SweepParams& p) {
  using P = Pipe<C>;
  constexpr int R = 32 * C, RC = P::RC, KU = P::KU, NT = P::NT;
  uint32_t* D = S + RC;  // five planes of RC words
  uint32_t* orders = D + 5 * RC;
  const int lane = (int)(threadIdx.x & 63u);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (int i = threadIdx.x; i < RC; i += blockDim.x) S[i] = load_word_any<LAYOUT>(p, i / C, 32 * (i % C));
  for (int i = threadIdx.x; i < p.nsweeps; i += blockDim.x) orders[i] = class_order(p.k0, p.k1, p.t0 + (uint64_t)i);
  unsigned count = 0;
  if (wave < P::PW) {
    PipeUnit u[KU];
    uint32_t ok[KU][2];
    bool live[KU];
    int d0[KU];
#pragma unroll
    for (int k = 0; k < KU; ++k) {
      const int un = 64 * (wave + k * P::PW) + lane;
      live[k] = un < RC / 2;
      const int v = live[k] ? un : un - RC / 2;  // spare lanes: another unit's words, no centres
      const int q = v / C, w = v - q * C, r0 = 2 * q;
#pragma unroll
      for (int j = 0; j < 6; ++j) {
        int y = r0 - 2 + j;
        y = y < 0 ? y + R : (y >= R ? y - R : y);
        u[k].row[j] = y * C;
      }
      u[k].w = w;
      u[k].we = w + 1 == C ? 0 : w + 1;
      u[k].ww = w == 0 ? C - 1 : w - 1;
      ok[k][0] = live[k] ? 0x11111111u << (r0 & 3) : 0u;
      ok[k][1] = live[k] ? 0x11111111u << ((r0 + 1) & 3) : 0u;
      d0[k] = r0 * C + w;
    }
#pragma unroll 1
    for (int i = 0; i < 8; ++i) __syncthreads();  // the first sweep's draws
#pragma unroll 1
    for (int s = 0; s < p.nsweeps; ++s) {
      RowRand rr[KU][2];
#pragma unroll
      for (int k = 0; k < KU; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t* d = D + d0[k] + h * C;
          rr[k][h] = RowRand{d[0], d[RC], d[2 * RC], d[3 * RC], d[4 * RC]};
        }
      const uint32_t perm = (uint32_t)__builtin_amdgcn_readfirstlane((int)orders[s]);
#pragma unroll 1
      for (int ph = 0; ph < 8; ++ph) {
        const uint32_t cls = (perm >> (4 * ph)) & 0xFu, turn = (32u - (cls >> 1)) & 31u;
        if (cls & 1u) count += pipe_phase<KU, 1>(S, p, u, rr, ok, live, turn);
        else count += pipe_phase<KU, 0>(S, p, u, rr, ok, live, turn);
        __syncthreads();
      }
    }
  } else if (wave < P::PW + P::RW) {
    uint32_t* tw = orders + kPipeMaxSweeps + (wave - P::PW) * (int)kTieWaveWords;
    TieList ties{reinterpret_cast<uint2*>(tw), tw + 2 * kTieCap, 0u};
    int rid[NT], y[NT], x[NT];
    bool live[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      rid[i] = 64 * ((wave - P::PW) * NT + i) + lane;
      live[i] = rid[i] < RC;
      rid[i] = live[i] ? rid[i] : RC - 1;
      y[i] = rid[i] / C;
      x[i] = 32 * (rid[i] - y[i] * C);
    }
    auto store = [&](int i, RowRand q, int tie) {
      join_ties(ties, tie, q);
      uint32_t* d = D + rid[i];
      if (live[i]) {
        d[0] = q.d0;
        d[RC] = q.d1;
        d[2 * RC] = q.acc0;
        d[3 * RC] = q.acc1;
        d[4 * RC] = q.acc2;
      }
    };
#pragma unroll 1
    for (int s = 0; s < p.nsweeps; ++s) {
      const uint64_t t = p.t0 + (uint64_t)s;
      if constexpr (P::SLICED) {
        uint32_t c0[3 * NT], c1[3 * NT], c2[3 * NT], c3[3 * NT];
        const uint32_t thi = ctr_hi(t, kTagSweep);
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            c0[3 * i + b] = (uint32_t)y[i];
            c1[3 * i + b] = (uint32_t)(x[i] >> 5) * 4u + (uint32_t)b;
            c2[3 * i + b] = (uint32_t)t;
            c3[3 * i + b] = thi;
          }
        philox10_n<3 * NT, 0, 4>(c0, c1, c2, c3, p.k0, p.k1);
        __syncthreads();
        philox10_n<3 * NT, 4, 7>(c0, c1, c2, c3, p.k0, p.k1);
        __syncthreads();
        philox10_n<3 * NT, 7, 10>(c0, c1, c2, c3, p.k0, p.k1);
        __syncthreads();
        uint32_t pl[NT][kPlanes], lt[NT][3], eq[NT][3];
        int tie[NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) {
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            pl[i][4 * b] = c0[3 * i + b];
            pl[i][4 * b + 1] = c1[3 * i + b];
            pl[i][4 * b + 2] = c2[3 * i + b];
            pl[i][4 * b + 3] = c3[3 * i + b];
          }
          compare_slot(pl[i], p.acc.hi[0], live[i], lt[i][0], eq[i][0]);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NT; ++i) {
          compare_slot(pl[i], p.acc.hi[1], live[i], lt[i][1], eq[i][1]);
          compare_slot(pl[i], p.acc.hi[2], live[i], lt[i][2], eq[i][2]);
        }
        __syncthreads();
        ties.n = 0u;
#pragma unroll
        for (int i = 0; i < NT; ++i) tie[i] = list_ties(p, ties, y[i], x[i], t, eq[i], lt[i]);
        __syncthreads();
        resolve_list(p, ties, t);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NT; ++i)
          store(i, RowRand{pl[i][0], pl[i][1], lt[i][0], lt[i][1], lt[i][2]}, tie[i]);
        __syncthreads();
      } else {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 7; ++i) {
          if (i < NT) {
            RowRand q;
            ties.n = 0u;
            const int tie = rand_row<true>(p, ties, t, y[i < NT ? i : 0], x[i < NT ? i : 0], live[i < NT ? i : 0], q);
            resolve_list(p, ties, t);
            store(i < NT ? i : 0, q, tie);
          }
          __syncthreads();
        }
      }
    }
#pragma unroll 1
    for (int i = 0; i < 8; ++i) __syncthreads();  // the last sweep's phases
  } else {
#pragma unroll 1
    for (int i = 0; i < 8 * (p.nsweeps + 1); ++i) __syncthreads();
  }
  for (int i = threadIdx.x; i < RC; i += blockDim.x) store_word_any<LAYOUT>(p, i / C, 32 * (i % C), S[i], 32);
  return count;
}

template <int LAYOUT, int C>
__global__ __launch_bounds__(Pipe<C>::kThreads) void pipe_kernel(SweepParams p) {
  extern __shared__ __attribute__((aligned(16))) uint32_t S[];
  const unsigned count = pipe_sweeps<LAYOUT, C>(S, p);
  add_block_count(S + Pipe<C>::kWords - 16, count, p.accepted);
}

// ---------------------------------------------------------------------------
// Batch kernels
// ---------------------------------------------------------------------------
// The class orders of sweeps s .. s + kBatchChunk - 1 of every replica, one per
// thread (replica = blockIdx.x): computed by every tile's workgroup they were
// 150 instructions of each wave.
__global__ __launch_bounds__(kBatchChunk) void batch_orders_kernel(const SweepParams* reps, unsigned s,
                                                                   uint32_t* orders) {
  const SweepParams& p = reps[blockIdx.x];
  orders[(size_t)blockIdx.x * kBatchChunk + threadIdx.x] = class_order(p.k0, p.k1, p.t0 + s + threadIdx.x);
}

// A launch does sweep s of the run, or s and s + 1 (MODE); the buffers change
// places with every launch.  512 threads, two workgroups per CU (four waves per
// SIMD, at most 128 VGPRs each), or up to 1024 side by side.
template <int KU, HaloMode MODE>
__global__ __launch_bounds__(MODE == kSideBySide ? 1024 : kBatchTileThreads) __attribute__((amdgpu_waves_per_eu(4)))
void batch_tile_kernel(const SweepParams* reps, const BatchTileJob* jobs, const uint32_t* orders, unsigned s) {
  extern __shared__ __attribute__((aligned(16))) uint32_t S[];
  constexpr unsigned NS = MODE == kOneSweep ? 1 : 2;
  const BatchTileJob job = jobs[blockIdx.x];
  SweepParams p = reps[job.rep];
  if (s < (unsigned)p.nsweeps) {
    if ((s / NS) & 1u) {  // p.src holds the lattice at the start of the run, p.dst the other buffer
      const void* t = p.src;
      p.src = p.dst;
      p.dst = const_cast<void*>(t);
    }
    p.t0 += s;
    // compile-time tile width (8 or 16 words: immediate, bank-conflict-free
    // LDS offsets) chosen per replica by a uniform switch; a replica's last
    // tile column may be ragged
    const uint32_t* o = orders + (size_t)job.rep * kBatchChunk + s % kBatchChunk;
    const uint32_t o0 = o[0], o1 = NS == 2 ? o[1] : 0u;  // s is even with two
    const int sweeps = min((int)NS, p.nsweeps - (int)s);
    unsigned count;
    if (p.layout == kLayoutBits) {
      if (p.tww == 8) count = halo_tile_sweep<kLayoutBits, 8, KU, MODE>(S, p, job.tile, o0, o1, sweeps);
      else count = halo_tile_sweep<kLayoutBits, 16, KU, MODE>(S, p, job.tile, o0, o1, sweeps);
    } else {
      if (p.tww == 8) count = halo_tile_sweep<kLayoutInt8, 8, KU, MODE>(S, p, job.tile, o0, o1, sweeps);
      else count = halo_tile_sweep<kLayoutInt8, 16, KU, MODE>(S, p, job.tile, o0, o1, sweeps);
    }
    if (threadIdx.x == 0) atomicAdd(p.accepted + job.tile, (unsigned long long)count);
  }
}

// Resident replicas, one workgroup each: the width is a uniform run-time switch
// over per-width instantiations (disjoint code regions share one register
// allocation) and the layout is a run-time branch of the staging and the final
// store.  Two launches, so that a small replica does not hold the waves and
// the LDS of a large one.
template <int C>
__device__ __forceinline__ void resident_sweeps(uint32_t* S, const SweepParams& p) {
  const unsigned count = pipe_sweeps<0, C>(S, p);
  add_block_count(S + Pipe<C>::kWords - 16, count, p.accepted);
}
__device__ __forceinline__ bool resident_chunk(SweepParams& p, unsigned s) {
  if (s >= (unsigned)p.nsweeps) return false;
  p.t0 += s;  // this launch: up to kBatchChunk sweeps from run sweep s
  p.nsweeps = min(kBatchChunk, p.nsweeps - (int)s);
  return true;
}
__global__ __launch_bounds__(kResidentThreads) void batch_resident_all_kernel(const SweepParams* reps, const int* ids,
                                                                              unsigned s) {
  extern __shared__ __attribute__((aligned(16))) uint32_t S[];
  SweepParams p = reps[ids[blockIdx.x]];
  if (!resident_chunk(p, s)) return;
  switch (p.C) {
    case 5: resident_sweeps<5>(S, p); break;
    case 6: resident_sweeps<6>(S, p); break;
    case 7: resident_sweeps<7>(S, p); break;
    case 8: resident_sweeps<8>(S, p); break;
    default: resident_sweeps<9>(S, p); break;
  }
}
__global__ __launch_bounds__(kResidentSmallThreads) void batch_resident_small_kernel(const SweepParams* reps,
                                                                                     const int* ids, unsigned s) {
  extern __shared__ __attribute__((aligned(16))) uint32_t S[];
  SweepParams p = reps[ids[blockIdx.x]];
  if (!resident_chunk(p, s)) return;
  switch (p.C) {
    case 2: resident_sweeps<2>(S, p); break;
    case 3: resident_sweeps<3>(S, p); break;
    default: resident_sweeps<4>(S, p); break;
  }
}
static_assert(Pipe<4>::kThreads <= kResidentSmallThreads && Pipe<5>::kThreads <= kResidentThreads &&
              Pipe<7>::kThreads <= kResidentThreads && Pipe<9>::kThreads <= kResidentThreads, "resident threads");

}  // namespace

namespace {
// class_order on the host.
uint32_t class_order_host(uint32_t k0, uint32_t k1, uint64_t t) {
  uint32_t w[8];
  for (uint32_t j = 0; j < 2; ++j) {
    const Philox4 b = philox10_host(0u, j, (uint32_t)t, ctr_hi(t, kTagOrder), k0, k1);
    w[4 * j] = b.x;
    w[4 * j + 1] = b.y;
    w[4 * j + 2] = b.z;
    w[4 * j + 3] = b.w;
  }
  return (uint32_t)shuffle_nibbles(w, 8);
}
}  // namespace

namespace {
// How a halo tile is launched: the mode, units per thread, threads.
struct HaloPlan {
  HaloMode mode;
  int ku, threads;
};
size_t halo_lds_bytes(const SweepParams& p, const HaloPlan& pl) {
  return ((size_t)halo_tie_offset(halo_rows(p.th, pl.mode == kOneSweep ? 1 : 2), p.C) +
          (size_t)(pl.threads / 64) * kTieWaveWords) * sizeof(uint32_t);
}
HaloPlan one_sweep_plan(const SweepParams& p, int ku) {
  const int threads = ((p.nunits + ku - 1) / ku + 63) & ~63;
  // two units per thread: four waves per SIMD issue a multiply or a shift
  // every 4.5 cycles, three (one wave each for 768 threads' units) only every
  // 5.8, so the first threads take two units and the rest one -- but for tiles
  // whose rows leave no room for the tie lists of 16 waves (one word wide, 992
  // rows or more: 992 take 143440 B, a wave's list 1280)
  const HaloPlan full{kOneSweep, ku, ku == 2 && p.nunits > 1024 ? 1024 : threads};
  return halo_lds_bytes(p, full) <= 160 * 1024 ? full : HaloPlan{kOneSweep, ku, threads};
}
// Rounds of workgroups that a launch takes: 16 wavefronts (halo_kernel's
// registers) and 160 KiB of LDS per CU.
int halo_rounds(const SweepParams& p, const HaloPlan& pl) {
  const int tiles = p.tiles_x * ((p.L + p.th - 1) / p.th);
  const int per_cu = std::min(1024 / pl.threads, (int)(160 * 1024 / halo_lds_bytes(p, pl)));
  return (tiles + 256 * per_cu - 1) / (256 * per_cu);
}
// How pairs of sweeps are launched: two per launch if that takes no more rounds
// of workgroups than one, and with several rounds only from 56 rows on, where
// the window of two sweeps has at most a fifth more units than two of one.  us
// per sweep, one and two per launch: bits 4096^2 in tiles of 16 x 128 (one round
// either way) 15.9 and 14.4, of 8 x 64 (one round becomes four) 21.5 and 34.5, of
// 16 x 40 (four rounds either way) 36.0 and 40.5; 2048^2 in tiles of 2 x 32 (one
// becomes three) 11.3 and 24.9.  Over 2349 tiles on sides of 64 .. 8192 the choice
// is within 1.14 of the better but for a few int8 tiles, 0.7 % from it on average;
// tiles of the default rule always take two.
HaloPlan pair_plan(const SweepParams& p, int ku) {
  const HaloPlan one = one_sweep_plan(p, ku);
  const bool rows_fit = (size_t)halo_rows(p.th, 2) * HaloGeom<16>::ST * 4 + 32768 <= 160 * 1024;  // the widest stride
  if (!rows_fit) return one;
  HaloPlan two = one;
  for (int k = 2; k >= 1; --k) {
    const int n = half_threads(p.th, p.C, k, 0) + half_threads(p.th, p.C, k, 1);
    if (n <= 1024) two = HaloPlan{kSideBySide, k, n};
  }
  if (two.mode == kOneSweep && half_threads(p.th, p.C, 2, 0) <= 1024) two = HaloPlan{kInTurn, 2, 1024};
  const int rounds = halo_rounds(p, one);
  return halo_rounds(p, two) <= rounds && (rounds == 1 || p.th >= 56) ? two : one;
}
bool halo_width(const SweepParams& p) { return p.tww == 1 || p.tww == 2 || p.tww == 4 || p.tww == 8 || p.tww == 16; }
}  // namespace

int sweeps_per_launch(const SweepParams& p, bool cyclic, int ku) {
  if (cyclic) return 256;
  return halo_width(p) && pair_plan(p, ku).mode != kOneSweep ? 2 : 1;
}

hipError_t launch_sweep(const SweepParams& p, int layout, bool cyclic, int ku, int threads, hipStream_t stream) {
  const int tiles_y = (p.L + p.th - 1) / p.th;
  const dim3 grid(p.tiles_x * tiles_y), block(threads);
  const size_t lds = (size_t)p.R * (p.C + 2) * sizeof(uint32_t) + 16 * sizeof(unsigned);
  if (cyclic && p.C >= 2 && p.C <= kResidentMaxC && p.nsweeps <= kPipeMaxSweeps) {
#define KK_PIPE(CC)                                                                                                  \
  case CC:                                                                                                           \
    if (layout == kLayoutBits)                                                                                       \
      hipLaunchKernelGGL((pipe_kernel<kLayoutBits, CC>), grid, dim3(Pipe<CC>::kThreads), Pipe<CC>::kWords * 4, stream, p); \
    else                                                                                                             \
      hipLaunchKernelGGL((pipe_kernel<kLayoutInt8, CC>), grid, dim3(Pipe<CC>::kThreads), Pipe<CC>::kWords * 4, stream, p); \
    break
    switch (p.C) {
      KK_PIPE(2); KK_PIPE(3); KK_PIPE(4); KK_PIPE(5); KK_PIPE(6); KK_PIPE(7); KK_PIPE(8); KK_PIPE(9);
    }
#undef KK_PIPE
    return hipGetLastError();
  }
  if (!cyclic && halo_width(p)) {
    const HaloPlan pl = p.nsweeps == 2 ? pair_plan(p, ku) : one_sweep_plan(p, ku);
    const uint32_t o0 = class_order_host(p.k0, p.k1, p.t0);
    const uint32_t o1 = pl.mode == kOneSweep ? 0u : class_order_host(p.k0, p.k1, p.t0 + 1);
#define KK_HALO(LY, TW)                                                                                              \
  do {                                                                                                               \
    const size_t hl = halo_lds_bytes(p, pl);                                                                          \
    const dim3 nt(pl.threads);                                                                                       \
    if (pl.mode == kInTurn) hipLaunchKernelGGL((halo_kernel<LY, TW, 2, kInTurn>), grid, nt, hl, stream, p, o0, o1);  \
    else if (pl.mode == kSideBySide && pl.ku == 1)                                                                   \
      hipLaunchKernelGGL((halo_kernel<LY, TW, 1, kSideBySide>), grid, nt, hl, stream, p, o0, o1);                    \
    else if (pl.mode == kSideBySide)                                                                                 \
      hipLaunchKernelGGL((halo_kernel<LY, TW, 2, kSideBySide>), grid, nt, hl, stream, p, o0, o1);                    \
    else if (pl.ku == 1) hipLaunchKernelGGL((halo_kernel<LY, TW, 1, kOneSweep>), grid, nt, hl, stream, p, o0, o1);   \
    else hipLaunchKernelGGL((halo_kernel<LY, TW, 2, kOneSweep>), grid, nt, hl, stream, p, o0, o1);                   \
  } while (0)
#define KK_HALO_W(LY)                          \
  do {                                         \
    switch (p.tww) {                           \
      case 1: KK_HALO(LY, 1); break;           \
      case 2: KK_HALO(LY, 2); break;           \
      case 4: KK_HALO(LY, 4); break;           \
      case 8: KK_HALO(LY, 8); break;           \
      default: KK_HALO(LY, 16); break;         \
    }                                          \
  } while (0)
    if (layout == kLayoutBits) KK_HALO_W(kLayoutBits);
    else KK_HALO_W(kLayoutInt8);
#undef KK_HALO_W
#undef KK_HALO
    return hipGetLastError();
  }
#define KK_LAUNCH(LY, CY, KUV) hipLaunchKernelGGL((sweep_kernel<LY, CY, KUV>), grid, block, lds, stream, p)
  if (layout == kLayoutBits) {
    if (cyclic) { if (ku == 1) KK_LAUNCH(kLayoutBits, true, 1); else KK_LAUNCH(kLayoutBits, true, 2); }
    else { if (ku == 1) KK_LAUNCH(kLayoutBits, false, 1); else KK_LAUNCH(kLayoutBits, false, 2); }
  } else {
    if (cyclic) { if (ku == 1) KK_LAUNCH(kLayoutInt8, true, 1); else KK_LAUNCH(kLayoutInt8, true, 2); }
    else { if (ku == 1) KK_LAUNCH(kLayoutInt8, false, 1); else KK_LAUNCH(kLayoutInt8, false, 2); }
  }
#undef KK_LAUNCH
  return hipGetLastError();
}

}  // namespace kk

namespace kk {

size_t batch_resident_lds_bytes(int L) {
  static constexpr int words[] = {Pipe<2>::kWords, Pipe<3>::kWords, Pipe<4>::kWords, Pipe<5>::kWords,
                                  Pipe<6>::kWords, Pipe<7>::kWords, Pipe<8>::kWords, Pipe<9>::kWords};
  static_assert(sizeof words / sizeof words[0] == kResidentMaxC - 1, "one per width");
  return (size_t)words[L / 32 - 2] * sizeof(uint32_t);
}

int batch_tile_threads(int tww, int th) { return half_threads(th, tww + 2, 1, 0) + half_threads(th, tww + 2, 1, 1); }
bool batch_tile_in_turn(int tww, int th) { return half_threads(th, tww + 2, 2, 0) <= kBatchTileThreads; }

hipError_t launch_batch_tiles(const SweepParams* reps, const BatchTileJob* jobs, int njobs, const uint32_t* orders,
                              unsigned s, const BatchTilePlan& pl, hipStream_t stream) {
  const int rows = halo_tie_offset(halo_rows(pl.max_th, pl.sweeps), kBatchMaxTww + 2);  // the widest tile's stride
  const size_t lds = ((size_t)rows + (size_t)(pl.threads / 64) * kTieWaveWords) * sizeof(uint32_t);
  const dim3 grid(njobs), block(pl.threads);
#define KK_BATCH(KU, MODE) \
  hipLaunchKernelGGL((batch_tile_kernel<KU, MODE>), grid, block, lds, stream, reps, jobs, orders, s)
  if (pl.sweeps == 2 && pl.side_by_side) KK_BATCH(1, kSideBySide);
  else if (pl.sweeps == 2) KK_BATCH(2, kInTurn);
  else if (pl.ku == 1) KK_BATCH(1, kOneSweep);
  else KK_BATCH(2, kOneSweep);
#undef KK_BATCH
  return hipGetLastError();
}

hipError_t launch_batch_orders(const SweepParams* reps, int nreps, unsigned s, uint32_t* orders, hipStream_t stream) {
  hipLaunchKernelGGL(batch_orders_kernel, dim3(nreps), dim3(kBatchChunk), 0, stream, reps, s, orders);
  return hipGetLastError();
}

hipError_t launch_batch_resident(const SweepParams* reps, const int* ids, int n, size_t lds_bytes, bool small,
                                 unsigned s, hipStream_t stream) {
  if (small)
    hipLaunchKernelGGL(batch_resident_small_kernel, dim3(n), dim3(kResidentSmallThreads), lds_bytes, stream, reps,
                       ids, s);
  else
    hipLaunchKernelGGL(batch_resident_all_kernel, dim3(n), dim3(kResidentThreads), lds_bytes, stream, reps, ids, s);
  return hipGetLastError();
}

}  // namespace kk
