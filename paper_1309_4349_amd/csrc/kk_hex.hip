// kk_hex.hip -- whole-sweep kernels of the triangular lattice on bit planes
// (Materials and Methods, "Monte Carlo model with Kawasaki based kinetics",
// Fig. 2; "Massive Parallel Kawasaki Kinetics", Fig. 4).  Gfx950 (CDNA4, wave64).
//
// A workgroup holds a window of the ring in LDS (rows of consecutive ring
// sites, cell (r, c) = site base + r*L + c), one bit per site, the columns of
// a row dealt into G classes c mod G: word (r, q) holds the cells c = G*j + q,
// bit j.  All centres of one class of a row are then one word, decided
// together with bitwise logic, and the neighbours of the whole word are words
// of the rows r-2 .. r+2 and classes q-2 .. q+2 mod G, turned by one bit where
// the class wraps.  G = 16 for the class schedule (class = ring index mod 16:
// one column class per row and phase), G = 14 for the literal MPKK (centres
// every 7 sites: two column classes per row and iteration, the even and the
// odd domains, which share their Philox blocks).
//
// Random numbers: each attempt needs its direction d in 0..5 and the
// comparisons of its uniform U with three thresholds.  The two sites a and b
// of an exchange have two common neighbours, each unlike exactly one of the
// two, so the count n of unlike neighbours lies in 2..8 and only n = 2, 3, 4
// (omega > 0) or 6, 7, 8 (omega < 0) can be rejected.  So an attempt's random
// state is six bits -- sign and axis of d, U < T for three thresholds -- drawn
// for the whole sweep before the first phase: each lane draws one Philox block
// for two sites of its row and shifts the twelve outcomes into twelve words
// (compare and add-with-carry), and the blocks are computed once instead of
// once per site.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kk_common.hpp"
#include "kk_kernels.hpp"
#include "kk_tri.hpp"
#include "kk_tri_dev.hpp"

namespace kk {
namespace {

// Where a lane finds the words around its own: A[d + 2] the word of class
// q + d mod G two rows above (so that every row offset is a positive
// immediate), rot[d + 2] the turn that aligns that class's words to the
// centres (1 where the class passed G - 1, -1 where it passed 0).
struct Place {
  int A[5];
  uint32_t rot[5];
};
template <int G, int ROW>
__device__ __forceinline__ Place class_place(int r, int q) {
  Place p;
#pragma unroll
  for (int d = -2; d <= 2; ++d) {
    // arithmetic instead of selects: a compare, its scalar mask and the select
    // that reads it are a longer chain
    const int k = q + d;
    if constexpr (G == 16) {
      p.A[d + 2] = (r - 2) * ROW + (k & 15);
      p.rot[d + 2] = (uint32_t)(k >> 4);  // -1 turns by 31
    } else {
      const int lo = k >> 31, hi = (G - 1 - k) >> 31;
      p.A[d + 2] = (r - 2) * ROW + k + (lo & G) - (hi & G);
      p.rot[d + 2] = (uint32_t)(lo - hi);
    }
  }
  return p;
}

template <int ROW>
__device__ __forceinline__ Around read_around(const uint32_t* S, const Place& p) {
  const int* A = p.A;
  Around v;
  v.n2 = S[A[2]];
  v.n = S[A[2] + ROW];
  v.a = S[A[2] + 2 * ROW];
  v.s = S[A[2] + 3 * ROW];
  v.s2 = S[A[2] + 4 * ROW];
  v.nne = rotr(S[A[3]], p.rot[3]);
  v.ne = rotr(S[A[3] + ROW], p.rot[3]);
  v.e = rotr(S[A[3] + 2 * ROW], p.rot[3]);
  v.se = rotr(S[A[3] + 3 * ROW], p.rot[3]);
  v.nw = rotr(S[A[1] + ROW], p.rot[1]);
  v.w = rotr(S[A[1] + 2 * ROW], p.rot[1]);
  v.sw = rotr(S[A[1] + 3 * ROW], p.rot[1]);
  v.ssw = rotr(S[A[1] + 4 * ROW], p.rot[1]);
  v.ne2 = rotr(S[A[4]], p.rot[4]);
  v.nee = rotr(S[A[4] + ROW], p.rot[4]);
  v.e2 = rotr(S[A[4] + 2 * ROW], p.rot[4]);
  v.w2 = rotr(S[A[0] + 2 * ROW], p.rot[0]);
  v.sww = rotr(S[A[0] + 3 * ROW], p.rot[0]);
  v.sw2 = rotr(S[A[0] + 4 * ROW], p.rot[0]);
  return v;
}

// Flip the accepted centres F and their partners.  Lanes without a row stay
// out: their zero flips would all go to one word, and xors of one wave to one
// word run one after another (62 such lanes cost 1650 cycles per iteration).
template <int ROW>
__device__ __forceinline__ void exchange(uint32_t* S, const Place& p, const Draw& q, uint32_t F) {
  const int* A = p.A;
  const uint32_t f0 = lut3<kA & ~kB>(F, q.ax1, q.ax1), f1 = lut3<kA & kB & ~kC>(F, q.ax1, q.ax2);
  const uint32_t f2 = F & q.ax2;
  // the turn that aligned the cell to the centre, undone
  const uint32_t re = 0u - p.rot[3], rw = 0u - p.rot[1];
  atomicXor(&S[A[2] + 2 * ROW], F);
  atomicXor(&S[A[3] + 2 * ROW], rotr(f0 & ~q.sgn, re));
  atomicXor(&S[A[1] + 2 * ROW], rotr(f0 & q.sgn, rw));
  atomicXor(&S[A[2] + 3 * ROW], f1 & ~q.sgn);
  atomicXor(&S[A[2] + ROW], f1 & q.sgn);
  atomicXor(&S[A[1] + 3 * ROW], rotr(f2 & ~q.sgn, rw));
  atomicXor(&S[A[3] + ROW], rotr(f2 & q.sgn, re));
}

// Bits j of class q whose columns G*j + q lie in [c0, c1), c0 >= G > q, at most 31 of them.
template <int G>
__device__ __forceinline__ uint32_t column_mask(int q, int c0, int c1) {
  const uint32_t lo = (uint32_t)(c0 + G - 1 - q) / G, hi = (uint32_t)(c1 + G - 1 - q) / G;
  return ((1u << (hi - lo)) - 1u) << lo;
}

// One row's draws of two classes in halves: lanes 0..31 hold the first h bits
// of both classes, lanes 32..63 the bits from h on of the same rows.  After
// it lanes 0..31 hold the whole words of the first class and lanes 32..63
// those of the second.
__device__ __forceinline__ uint32_t join_halves(uint32_t first, uint32_t second, uint32_t h) {
  const auto p = __builtin_amdgcn_permlane32_swap(first, second, false, false);
  return p[0] | (p[1] << h);
}
__device__ __forceinline__ Draw join_draws(const Draw& a, const Draw& b, uint32_t h) {
  return Draw{join_halves(a.sgn, b.sgn, h), join_halves(a.ax1, b.ax1, h), join_halves(a.ax2, b.ax2, h),
              join_halves(a.a0, b.a0, h),   join_halves(a.a1, b.a1, h),   join_halves(a.a2, b.a2, h)};
}

// A draw whose first bit is group j0's.
__device__ __forceinline__ void store_draw(uint32_t* D, const Draw& q, uint32_t j0, const HexAccept& acc) {
  uint2* p = reinterpret_cast<uint2*>(D);
  p[0] = make_uint2(q.sgn << j0, q.ax1 << j0);
  p[1] = make_uint2(q.ax2 << j0, (q.a0 << j0) | acc.all[0]);
  p[2] = make_uint2((q.a1 << j0) | acc.all[1], (q.a2 << j0) | acc.all[2]);
}
__device__ __forceinline__ Draw load_draw(const uint32_t* D) {
  const uint2* p = reinterpret_cast<const uint2*>(D);
  const uint2 x = p[0], y = p[1], z = p[2];
  return Draw{x.x, x.y, y.x, y.y, z.x, z.y};
}

struct Bytes16 {
  uint32_t x[4];
};
// Ring sites s .. s + 15 (mod N).  Only lanes that reach the ring's end take
// them one by one.
__device__ __forceinline__ Bytes16 ring_bytes(const uint8_t* __restrict__ in, uint32_t s, uint32_t N) {
  Bytes16 v;
  s = s >= N ? s - N : s;
  if (s + 16u <= N) {
    __builtin_memcpy(&v, in + s, 16);
  } else {
    v = Bytes16{};
#pragma unroll 1
    for (int b = 0; b < 16; ++b) {
      uint32_t i = s + (uint32_t)b;
      i = i >= N ? i - N : i;
      const uint32_t x = (uint32_t)in[i] << (8 * (b & 3));
#pragma unroll
      for (int k = 0; k < 4; ++k) v.x[k] |= (b >> 2) == k ? x : 0u;
    }
  }
  return v;
}

// OR over the eight lanes of a group, in every lane.
__device__ __forceinline__ uint32_t or8(uint32_t x) {
  x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, false);   // lane ^ 1
  x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, false);   // lane ^ 2
  x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xF, 0xF, false);  // 7 - lane
  return x;
}

// Stage and unstage: eight neighbouring lanes take eight neighbouring groups
// of G sites of a row (lane l the group l), 16 bytes each, so that a
// wavefront's loads and stores are contiguous.  Bit l of byte q of the eight
// lanes' bytes shifted by their lane and ORed together is site q of group l:
// one byte of each of the row's G class words, of which lane l stores (or
// reads) the classes 2l and 2l + 1.
template <int G>
__device__ __forceinline__ void stage_bytes(uint8_t* B, const Bytes16& v, int l) {
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = or8(v.x[k] << l);
  const uint32_t x = l < 4 ? (l < 2 ? w[0] : w[1]) : (l < 6 ? w[2] : w[3]);
  const uint32_t y = (l & 1) ? x >> 16 : x;
  if (2 * l < G) {
    B[8 * l] = (uint8_t)y;
    B[8 * l + 4] = (uint8_t)(y >> 8);
  }
}
template <int G>
__device__ __forceinline__ Bytes16 unstage_bytes(const uint8_t* B, int l) {
  uint32_t y = 0u;
  if (2 * l < G) y = (uint32_t)B[8 * l] | ((uint32_t)B[8 * l + 4] << 8);
  y = (l & 1) ? y << 16 : y;
  Bytes16 v;
#pragma unroll
  for (int k = 0; k < 4; ++k) v.x[k] = (or8((l >> 1) == k ? y : 0u) >> l) & 0x01010101u;
  return v;
}

// i / n for 0 <= i < 4096 and n = 1 .. 4, inv = 65536 / n + 1.
__device__ __forceinline__ int div_small(int i, int inv) { return (int)(((uint32_t)i * (uint32_t)inv) >> 16); }

// ---------------------------------------------------------------------------
// One sweep of the 16 classes on the tile (tx, ty) of TW x TR sites, from `in`
// to `out`.  The window holds kHexLeft columns and kTriHalo rows before the
// tile and at least kTriHalo after it; a cell's value after a phase depends on
// cells within two steps, so the cells at least 33 from the window's edge --
// the tile -- are exact after 16 phases.  Every phase works on all the rows
// that have two rows around them; what the outer cells and the unused bits
// hold never reaches the tile.
//
// What bounds it: the draws, by VALU issue (66 instructions per two sites: 18
// multiplies and ten compare/add pairs among them, about 300 of a SIMD's
// cycles at four waves), then the 16 phases, by one wave's latency (about 105
// dependent instructions, 19 LDS reads, 7 LDS xors and a barrier; the rows of a
// window fill 2 to 6 waves, so a phase cannot be shortened by more of them).
// 4092^2 (256 x 256 tiles, one per CU): of a workgroup's 99000 cycles 5000 go by
// until the loads are issued, the draws and the packing end at 70500, 16 phases
// of 1240 follow, and the stores take the rest: 46.4 us per sweep against 104 us
// with one byte per site and a Philox block per attempt.  404 x 412 (29 x 23
// tiles), 27000 cycles: 2200, 9100, 16 x 970, 1000: 14.9 against 23.9 us;
// 1028^2 18.6 against 31.1 us.
__device__ __forceinline__ void hex_sweep_body(const uint8_t* __restrict__ in, uint8_t* __restrict__ out, uint32_t L,
                                               uint32_t H, uint32_t TW, uint32_t TR, uint32_t tx, uint32_t ty,
                                               uint32_t k0, uint32_t k1, uint64_t t, uint64_t order,
                                               const HexAccept& acc, unsigned long long* partials, uint32_t* lds) {
  constexpr int G = 16, ROW = kHexRow16;
  __shared__ uint32_t phase_s[16], total_s, next_s;  // phase_s: the phase of each class
  const uint32_t N = L * H;
  const int WR = (int)TR + 2 * (int)kTriHalo, NJ = hex_groups(TW);
  const int N8 = (NJ + 7) >> 3;  // eight-group blocks per row
  const uint32_t x0 = tx * TW, y0 = ty * TR;
  const int TWe = (int)min(TW, L - x0), TRe = (int)min(TR, H - y0);
  // ring index of window cell (0, 0), a multiple of 4
  uint32_t base = (y0 >= kTriHalo ? y0 - kTriHalo : y0 + H - kTriHalo) * L + x0;
  base = base >= kHexLeft ? base - kHexLeft : base + N - kHexLeft;
  const int lane = (int)(threadIdx.x & 63u), nthreads = (int)blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), nwaves = nthreads >> 6;
  uint32_t* S = lds;                            // WR rows of ROW words
  uint32_t* D = lds + hex_spin_words(WR, ROW);  // draws: [class][row][6]
  auto row_base = [&](int r) {
    const uint32_t s = base + (uint32_t)r * L;
    return s >= N ? s - N : s;
  };
  if (threadIdx.x < 16) phase_s[(uint32_t)(order >> (4u * threadIdx.x)) & 15u] = threadIdx.x;
  if (threadIdx.x == 0) {
    total_s = 0u;
    next_s = (uint32_t)nwaves;
  }
  // the window: eight lanes per (row, eight groups); the loads of the first
  // kPre rounds are issued here and packed after the draws
  constexpr int kPre = 8;
  const int l8 = lane & 7, nblk = WR * N8, step = nthreads >> 3;
  const int blk0 = (int)(threadIdx.x >> 3), inv8 = 65536 / N8 + 1;
  auto load_blk = [&](int i) {
    const int r = div_small(i, inv8);
    return ring_bytes(in, row_base(r) + (uint32_t)(G * (8 * (i - r * N8) + l8)), N);
  };
  auto store_blk = [&](int i, const Bytes16& v) {
    const int r = div_small(i, inv8);
    stage_bytes<G>(reinterpret_cast<uint8_t*>(S + r * ROW) + (i - r * N8), v, l8);
  };
  Bytes16 v[kPre];
#pragma unroll
  for (int k = 0; k < kPre; ++k)
    if (k * step < nblk) v[k] = load_blk(min(blk0 + k * step, nblk - 1));  // a uniform test; spare lanes load twice
  __syncthreads();
  // The draws: task = (pair of classes, 32 rows), each row in two halves.  A
  // class of phase p is needed within 31 - 2p cells of the tile, a pair as far
  // as its earlier class.  The waves take the tasks as they finish (the
  // scheduler favours the oldest).
  {
    const Head hd = philox_head(0u, (uint32_t)t, ctr_hi(t, kTagTri), k0, k1);
    const int nb = (int)(N >> 1);
    auto margin = [&](int pair) { return 31 - 2 * (int)min(phase_s[2 * pair], phase_s[2 * pair + 1]); };
    int pair = 0, first = 0;  // the pair of the current task and the pair's first task
    int m = __builtin_amdgcn_readfirstlane(margin(0));
    for (int task = wave;;) {
      int blocks = (TRe + 2 * m + 31) >> 5;
      while (pair < 8 && task >= first + blocks) {
        first += blocks;
        if (++pair < 8) {
          m = __builtin_amdgcn_readfirstlane(margin(pair));
          blocks = (TRe + 2 * m + 31) >> 5;
        }
      }
      if (pair == 8) break;
      uint32_t nx = 0u;
      if (lane == 0) nx = atomicAdd(&next_s, 1u);
      const int j0 = ((int)kHexLeft - m) >> 4, nj = (((int)kHexLeft + TWe + m - 1) >> 4) + 1 - j0;
      const int h = (nj + 1) >> 1;
      const int r = min((int)kTriHalo - m + 32 * (task - first) + (lane & 31), (int)kTriHalo + TRe + m - 1);
      const uint32_t s = row_base(r);
      const int q = (2 * pair - (int)s) & 15;  // the column class of the pair's even class
      int blk = (int)((s + (uint32_t)q) >> 1) + 8 * (j0 + (lane < 32 ? h - 1 : 2 * h - 1));
      blk = blk >= nb ? blk - nb : blk;
      Draw e{}, o{};
      for (int j = 0; j < h; ++j) {
        const Philox4 w = philox_tail(hd, (uint32_t)blk);
        push_attempt(e, w.x, w.y, acc);
        push_attempt(o, w.z, w.w, acc);
        blk -= 8;
        blk = blk < 0 ? blk + nb : blk;
      }
      store_draw(D + 6 * ((q + (lane >> 5)) * WR + r), join_draws(e, o, (uint32_t)h), (uint32_t)j0, acc);
      task = __builtin_amdgcn_readfirstlane((int)nx);
    }
  }
#pragma unroll
  for (int k = 0; k < kPre; ++k)
    if (blk0 + k * step < nblk) store_blk(blk0 + k * step, v[k]);
  for (int i = blk0 + kPre * step; i < nblk; i += step) store_blk(i, load_blk(i));
  __syncthreads();
  // The phases are one wave's latency each: the rows need nb waves, and up to
  // three sets of nb waves take turns, so that a set finds its addresses and
  // draws for its next phase while the others work.
  const int nb = (WR - 4 + 63) >> 6, nsets = min(3, nwaves / nb);
  const int set = wave / nb;
  const int r = 2 + 64 * (wave - set * nb) + lane;
  const bool row_ok = r < WR - 2;
  const int rc = row_ok ? r : 2;
  const uint32_t cmask = row_ok ? 0xFFFFFFFFu : 0u;
  const int f = (int)(row_base(rc) & 15u);
  const uint32_t counted = row_ok && r >= (int)kTriHalo && r < (int)kTriHalo + TRe ? 0xFFFFFFFFu : 0u;
  uint32_t cnt = 0;
  Place pl{};
  Draw d{};
  int q = 0;
  auto prepare = [&](int p) {
    q = ((int)(order >> (4 * p)) - f) & 15;
    pl = class_place<G, ROW>(rc, q);
    d = load_draw(D + 6 * (q * WR + rc));
  };
  if (set < nsets) prepare(set);
  int turn = 0;
#pragma unroll 1
  for (int p = 0; p < 16; ++p) {
    uint32_t F = 0u;
    const bool mine = set == turn;
    if (mine) {
      F = decide(read_around<ROW>(S, pl), d, acc.negmask, cmask);
      if (row_ok) exchange<ROW>(S, pl, d, F);
    }
    __syncthreads();
    if (mine) {
      const uint32_t m = column_mask<G>(q, (int)kHexLeft, (int)kHexLeft + TWe);
      cnt += (uint32_t)__builtin_popcount(F & m & counted);
      if (p + nsets < 16) prepare(p + nsets);
    }
    turn = turn + 1 == nsets ? 0 : turn + 1;
  }
  // the tile, four sites at a time at its edges (its first column and width are multiples of 4)
  for (int i = blk0; i < TRe * N8; i += step) {
    const int rr = div_small(i, inv8), g8 = i - rr * N8;
    const Bytes16 y =
        unstage_bytes<G>(reinterpret_cast<const uint8_t*>(S + (rr + (int)kTriHalo) * ROW) + g8, l8);
    uint8_t* row = out + (size_t)(y0 + (uint32_t)rr) * L + x0;
    const int c = G * (8 * g8 + l8) - (int)kHexLeft;
    if (c >= 0 && c + 16 <= TWe) {
      __builtin_memcpy(row + c, &y, 16);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (c + 4 * k >= 0 && c + 4 * k < TWe) __builtin_memcpy(row + c + 4 * k, &y.x[k], 4);
    }
  }
  add_count(cnt, &total_s, partials + blockIdx.x % kTriPartials);
}

__global__ __launch_bounds__(1024) void hex_sweep(const uint8_t* __restrict__ in, uint8_t* __restrict__ out,
                                                  uint32_t L, uint32_t H, uint32_t TW, uint32_t TR, uint32_t ntx,
                                                  uint32_t k0, uint32_t k1, uint64_t t, uint64_t order,
                                                  HexAccept acc, unsigned long long* partials) {
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  const uint32_t tile = (uint32_t)xcd_tile((int)blockIdx.x, (int)gridDim.x);
  hex_sweep_body(in, out, L, H, TW, TR, tile % ntx, tile / ntx, k0, k1, t, order, acc, partials, lds);
}

// Many lattices in one launch: workgroup b does tile jobs[b].y of replica
// jobs[b].x, sweep k of the run (buffers and sweep counter from the table).
__global__ __launch_bounds__(1024) void hex_sweep_batch(const TriBatchRep* reps, const uint2* jobs, uint32_t k) {
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  const uint2 jb = jobs[blockIdx.x];
  const TriBatchRep& R = reps[jb.x];
  const uint32_t par = R.cur ^ (k & 1u);
  hex_sweep_body(R.lat[par], R.lat[par ^ 1u], R.L, R.H, R.TW, R.TR, jb.y % R.ntx, jb.y / R.ntx, R.k0, R.k1, R.t0 + k,
                 hex_order(R.k0, R.k1, R.t0 + k), R.acc, R.partials, lds);
}

// ---------------------------------------------------------------------------
// One whole literal-MPKK step (7 iterations) on a tile, from `in` to `out`.
// The window holds kMpkkHalo more cells on every side (a cell's value after an
// iteration depends on cells within three steps).  Every domain of an
// iteration decides from the lattice as it stood when the iteration began: the
// decisions of all words are taken, then a barrier, then the exchanges are
// written (domains are disjoint).  The centres of an iteration sit every 7
// sites of the ring; domain m = 2b and m = 2b + 1 take their numbers from
// Philox block b, so with 14 column classes the even domains of a row are one
// class, the odd ones the class 7 further on, and one block fills a bit of
// each.
//
// What bounds it: as for the class schedule, the draws by VALU issue and the
// seven iterations by one wave's latency (two barriers each).  4098 x 4095 (257 x
// 256 tiles), 100000 cycles: 8000 until the loads are issued, 55000 draws and
// packing, 7 x 2670, 18000 stores (of single bytes at a tile's edges): 50.6 us
// per step against 102.8 us with one byte per site.  404 x 420 (24 x 28 tiles),
// 22000 cycles: 2700, 6800, 7 x 1580, 1700: 13.1 against 17.1 us; 1027 x 1029
// 16.3 against 25.1 us.
__global__ __launch_bounds__(1024) void hex_mpkk_step(const uint8_t* __restrict__ in, uint8_t* __restrict__ out,
                                                      uint32_t L, uint32_t H, uint32_t TW, uint32_t TR, uint32_t ntx,
                                                      uint32_t k0, uint32_t k1, uint64_t t, uint32_t covers,
                                                      HexAccept acc, unsigned long long* partials) {
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  constexpr int G = 14, ROW = kHexRow14;
  __shared__ uint32_t total_s, next_s;
  const uint32_t N = L * H;
  const int WR = (int)TR + 2 * (int)kMpkkHalo, NJ = hex_mpkk_groups(TW);
  const int N8 = (NJ + 7) >> 3;
  const uint32_t tile = (uint32_t)xcd_tile((int)blockIdx.x, (int)gridDim.x);
  const uint32_t x0 = (tile % ntx) * TW, y0 = (tile / ntx) * TR;
  const int TWe = (int)min(TW, L - x0), TRe = (int)min(TR, H - y0);
  uint32_t base = (y0 >= kMpkkHalo ? y0 - kMpkkHalo : y0 + H - kMpkkHalo) * L + x0;
  base = base >= kMpkkHalo ? base - kMpkkHalo : base + N - kMpkkHalo;
  const int lane = (int)(threadIdx.x & 63u), nthreads = (int)blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), nwaves = nthreads >> 6;
  uint32_t* S = lds;
  uint32_t* D = lds + hex_spin_words(WR, ROW);  // draws: [iteration][even or odd domains][row][6]
  auto row_base = [&](int r) {
    const uint32_t s = base + (uint32_t)r * L;
    return s >= N ? s - N : s;
  };
  if (threadIdx.x == 0) {
    total_s = 0u;
    next_s = (uint32_t)nwaves;
  }
  constexpr int kPre = 8;
  const int l8 = lane & 7, nblk = WR * N8, step = nthreads >> 3;
  const int blk0 = (int)(threadIdx.x >> 3), inv8 = 65536 / N8 + 1;
  auto load_blk = [&](int i) {
    const int r = div_small(i, inv8);
    return ring_bytes(in, row_base(r) + (uint32_t)(G * (8 * (i - r * N8) + l8)), N);
  };
  auto store_blk = [&](int i, const Bytes16& v) {
    const int r = div_small(i, inv8);
    stage_bytes<G>(reinterpret_cast<uint8_t*>(S + r * ROW) + (i - r * N8), v, l8);
  };
  Bytes16 v[kPre];
#pragma unroll
  for (int k = 0; k < kPre; ++k)
    if (k * step < nblk) v[k] = load_blk(min(blk0 + k * step, nblk - 1));  // a uniform test; spare lanes load twice
  __syncthreads();
  // The draws: task = (iteration, 32 rows), the blocks of each row in two
  // halves.  Iteration i's centres are needed within 19 - 3i cells of the
  // tile: nj groups from group j0 on.  Bit i of the raw words is block
  // b0 + j0 - 1 + i, b0 the block of the row's first cell of the even class:
  // the odd domain of the block before the first group may be the first of its
  // class.
  {
    int m = 19, j0 = 0, h = 0;
    auto draw = [&](const Head& hd, int blk, Draw& e, Draw& o) {
      blk += j0 + (lane < 32 ? h - 2 : 2 * h - 2);
      for (int j = 0; j < h; ++j) {
        const Philox4 w = philox_tail(hd, (uint32_t)blk);
        push_attempt(e, w.x, w.y, acc);
        push_attempt(o, w.z, w.w, acc);
        --blk;
      }
    };
    auto shifted = [](const Draw& d, uint32_t n) {
      return Draw{d.sgn >> n, d.ax1 >> n, d.ax2 >> n, d.a0 >> n, d.a1 >> n, d.a2 >> n};
    };
    int it = 0, first = 0;  // the current task's iteration and the iteration's first task
    for (int task = wave;;) {
      int blocks = (TRe + 2 * m + 31) >> 5;
      while (it < 7 && task >= first + blocks) {
        first += blocks;
        ++it;
        m -= 3;
        blocks = (TRe + 2 * m + 31) >> 5;
      }
      if (it == 7) break;
      uint32_t nx = 0u;
      if (lane == 0) nx = atomicAdd(&next_s, 1u);
      j0 = ((int)kMpkkHalo - m) / G;
      h = (((int)kMpkkHalo + TWe + m - 1) / G + 1 - j0 + 2) >> 1;
      const int r = min((int)kMpkkHalo - m + 32 * (task - first) + (lane & 31), (int)kMpkkHalo + TRe + m - 1);
      const int k = (int)(covers >> (4 * it)) & 15;
      const uint32_t s = row_base(r);
      const Head hd = philox_head((uint32_t)it, (uint32_t)t, ctr_hi(t, kTagMpkk), k0, k1);
      int ke = k + 14 - (int)(s % 14u);
      ke = ke >= 14 ? ke - 14 : ke;
      Draw e{}, o{};
      draw(hd, (int)((s + (uint32_t)ke - (uint32_t)k) / 14u), e, o);
      Draw d = shifted(join_draws(e, o, (uint32_t)h), lane < 32 || ke < 7 ? 1u : 0u);
      // a row that reaches the ring's end goes on with site 0, where domain 0
      // begins: where N/7 is odd the classes of even and odd domains trade
      // places there, and the blocks start anew in any case
      if (__any(s + (uint32_t)(G * NJ) > N)) {
        const bool swap = N % 14u != 0u;
        int ke2 = swap ? ke + 7 : ke;
        ke2 = ke2 >= 14 ? ke2 - 14 : ke2;
        const int s2 = (int)(s - N);
        Draw e2{}, o2{};
        draw(hd, (s2 + ke2 - k) / 14, e2, o2);
        // lanes 0..31 hold the class of e (the row's first even domains), lanes 32..63 that of o
        const bool even2 = (lane < 32) != swap;
        const Draw d2 = shifted(swap ? join_draws(o2, e2, (uint32_t)h) : join_draws(e2, o2, (uint32_t)h),
                                even2 || ke2 < 7 ? 1u : 0u);
        int q = lane < 32 ? ke : ke + 7;
        q = q >= 14 ? q - 14 : q;
        const int seam = (int)(N - s);  // the first column after the ring's end
        const int js = max((seam > q ? (seam - q + G - 1) / G : 0) - j0, 0);
        const uint32_t after = js < 32 ? ~((1u << js) - 1u) : 0u;
        d = Draw{mux(after, d2.sgn, d.sgn), mux(after, d2.ax1, d.ax1), mux(after, d2.ax2, d.ax2),
                 mux(after, d2.a0, d.a0),   mux(after, d2.a1, d.a1),   mux(after, d2.a2, d.a2)};
      }
      store_draw(D + 6 * ((2 * it + (lane >> 5)) * WR + r), d, (uint32_t)j0, acc);
      task = __builtin_amdgcn_readfirstlane((int)nx);
    }
  }
#pragma unroll
  for (int k = 0; k < kPre; ++k)
    if (blk0 + k * step < nblk) store_blk(blk0 + k * step, v[k]);
  for (int i = blk0 + kPre * step; i < nblk; i += step) store_blk(i, load_blk(i));
  __syncthreads();
  // the even domains' words in the first nb waves, the odd domains' in the next nb
  const int nb = (WR - 4 + 63) >> 6;
  const int half = wave >= nb ? 1 : 0;
  const bool busy = wave < 2 * nb;
  const int r = 2 + 64 * (wave - half * nb) + lane;
  const bool row_ok = busy && r < WR - 2;
  const int rc = row_ok ? r : 2;
  const uint32_t cmask = row_ok ? 0xFFFFFFFFu : 0u;
  const int f = (int)(row_base(rc) % 14u);
  const uint32_t counted = row_ok && r >= (int)kMpkkHalo && r < (int)kMpkkHalo + TRe ? 0xFFFFFFFFu : 0u;
  uint32_t cnt = 0;
  Place pl{};
  Draw d{};
  int q = 0;
  auto prepare = [&](int it) {
    q = ((int)(covers >> (4 * it)) & 15) + 7 * half - f;  // -13 .. 13
    q += (q >> 31) & 14;
    pl = class_place<G, ROW>(rc, q);
    d = load_draw(D + 6 * ((2 * it + half) * WR + rc));
  };
  if (busy) prepare(0);
#pragma unroll 1
  for (int it = 0; it < 7; ++it) {
    uint32_t F = 0u;
    if (busy) F = decide(read_around<ROW>(S, pl), d, acc.negmask, cmask);
    __syncthreads();
    if (busy) {
      if (row_ok) exchange<ROW>(S, pl, d, F);
      const uint32_t m = column_mask<G>(q, (int)kMpkkHalo, (int)kMpkkHalo + TWe);
      cnt += (uint32_t)__builtin_popcount(F & m & counted);
      if (it + 1 < 7) prepare(it + 1);
    }
    __syncthreads();
  }
  for (int i = blk0; i < TRe * N8; i += step) {
    const int rr = div_small(i, inv8), g8 = i - rr * N8;
    const Bytes16 y =
        unstage_bytes<G>(reinterpret_cast<const uint8_t*>(S + (rr + (int)kMpkkHalo) * ROW) + g8, l8);
    uint8_t* row = out + (size_t)(y0 + (uint32_t)rr) * L + x0;
    const int c = G * (8 * g8 + l8) - (int)kMpkkHalo;
    if (c >= 0 && c + G <= TWe) {
      __builtin_memcpy(row + c, &y, G);
    } else {
#pragma unroll
      for (int k = 0; k < G; ++k)
        if (c + k >= 0 && c + k < TWe) row[c + k] = (uint8_t)(y.x[k >> 2] >> (8 * (k & 3)));
    }
  }
  add_count(cnt, &total_s, partials + blockIdx.x % kTriPartials);
}

// The class order of sweep t, for a launch that holds one sweep.
uint64_t class_order16(uint32_t k0, uint32_t k1, uint64_t t) {
  return order_of([&](int j) {
    return philox10_host((uint32_t)j, 0u, (uint32_t)t, ctr_hi(t, kTagTriOrder), k0, k1);
  });
}

// The domain covers k_j of the seven iterations of step t, nibble j each.
uint32_t mpkk_covers(uint32_t k0, uint32_t k1, uint64_t t) {
  uint32_t covers = 0u;
  for (uint32_t b = 0; b < 2; ++b) {
    const Philox4 p = philox10_host(b, 2u, (uint32_t)t, ctr_hi(t, kTagMpkkK), k0, k1);
    const uint32_t w[4] = {p.x, p.y, p.z, p.w};
    for (uint32_t i = 0; i < 4 && 4 * b + i < 7; ++i)
      covers |= (uint32_t)(((uint64_t)w[i] * 7u) >> 32) << (4 * (4 * b + i));
  }
  return covers;
}

}  // namespace

hipError_t launch_tri_tile_sweep(const uint8_t* in, uint8_t* out, int L, int H, int TW, int TR, uint32_t k0,
                                uint32_t k1, uint64_t t, const TriAccept& acc, unsigned long long* partials,
                                hipStream_t stream) {
  if (!tri_tile_fits(L, H, TW, TR)) return hipErrorInvalidValue;
  const HexTile ht = hex_tile(TW, TR);
  const uint32_t ntx = ((uint32_t)L + ht.tw - 1) / ht.tw, nty = ((uint32_t)H + ht.tr - 1) / ht.tr;
  hipLaunchKernelGGL(hex_sweep, dim3(ntx * nty), dim3(1024), hex_lds_bytes(ht.tr), stream, in, out, (uint32_t)L,
                     (uint32_t)H, ht.tw, ht.tr, ntx, k0, k1, t, class_order16(k0, k1, t), hex_accept(acc), partials);
  return hipGetLastError();
}

hipError_t launch_tri_tile_sweep_batch(const TriBatchRep* reps, const uint2* jobs, uint32_t njobs, uint32_t k,
                                       size_t lds_bytes, hipStream_t stream) {
  if (njobs == 0) return hipSuccess;
  hipLaunchKernelGGL(hex_sweep_batch, dim3(njobs), dim3(1024), lds_bytes, stream, reps, jobs, k);
  return hipGetLastError();
}

hipError_t launch_mpkk_tile_step(const uint8_t* in, uint8_t* out, int L, int H, int TW, int TR, uint32_t k0,
                                 uint32_t k1, uint64_t t, const TriAccept& acc, unsigned long long* partials,
                                 hipStream_t stream) {
  if (!mpkk_tile_fits(L, H, TW, TR)) return hipErrorInvalidValue;
  const HexTile ht = hex_mpkk_tile(TW, TR);
  const uint32_t ntx = ((uint32_t)L + ht.tw - 1) / ht.tw, nty = ((uint32_t)H + ht.tr - 1) / ht.tr;
  hipLaunchKernelGGL(hex_mpkk_step, dim3(ntx * nty), dim3(1024), hex_mpkk_lds_bytes(ht.tr), stream, in, out,
                     (uint32_t)L, (uint32_t)H, ht.tw, ht.tr, ntx, k0, k1, t, mpkk_covers(k0, k1, t), hex_accept(acc), partials);
  return hipGetLastError();
}

}  // namespace kk
