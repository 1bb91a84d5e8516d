// kk_ring.hip -- small rings of the triangular lattice: the whole ring of one
// replica in one workgroup's LDS (no halo), all of its sweeps in one launch,
// written back in place.  Workgroup b runs replica b of a table.  Gfx950
// (CDNA4, wave64).
//
// The ring is cut into B equal segments of K = N / B sites, K a multiple of 16,
// and dealt over the bits of K words: word k holds the sites k + K*j, bit
// 2 + j.  Every word then holds sites of one class (k mod 16) only, a class is
// W = K/16 words, the neighbours of a word at distance d are the one word k + d
// mod K, turned by one bit where k + d passes an end, and the ring has no
// edges.  Two more bits on either side repeat the segments across the ring's
// end, so that a turn by one bit needs no repair; an exchange flips them too.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kk_common.hpp"
#include "kk_kernels.hpp"
#include "kk_tri.hpp"
#include "kk_tri_dev.hpp"

namespace kk {
namespace {

__device__ __forceinline__ void count_ring(unsigned long long cnt, const TriResidentRep& R, unsigned long long* red) {
  for (int off = 32; off > 0; off >>= 1) cnt += __shfl_down(cnt, off, 64);
  if ((threadIdx.x & 63u) == 0u) red[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long tot = 0;
    for (uint32_t w = 0; w < blockDim.x >> 6; ++w) tot += red[w];
    if (tot) atomicAdd(&R.partials[0], tot);
  }
}

// ---------------------------------------------------------------------------
// Rings without equal segments (ring_segments == 0): one byte per site, one
// thread per centre, a barrier after each class; neighbours wrap modulo N.
__device__ __forceinline__ void byte_ring(const TriResidentRep& R, uint8_t* ring, unsigned long long* red) {
  __shared__ uint32_t perm_s[16], thr_s[11];
  __shared__ uint32_t all_s;
  const uint32_t L = R.L, N = R.L * R.H;
  uint8_t* lat = R.lat;
  if (threadIdx.x >= 64 && threadIdx.x < 64 + 11) {
    const uint32_t n = threadIdx.x - 64;
    const uint64_t T = R.acc.T[n];
    thr_s[n] = T >= 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)T;
    const uint32_t always = (uint32_t)__ballot(T >= 0x100000000ull);  // lanes 0..10 of wave 1
    if (n == 0) all_s = always;
  }
  for (uint32_t i = threadIdx.x; i < N; i += blockDim.x) ring[i] = lat[i];
  unsigned long long cnt = 0;
  const uint32_t M = N >> 4;
  for (uint32_t s = 0; s < R.sweeps; ++s) {
    const uint64_t t = R.t0 + s;
    __syncthreads();  // the previous sweep's last phase (and the load) are complete
    if (threadIdx.x < 64) {
      const uint64_t order = hex_order(R.k0, R.k1, t);
      if (threadIdx.x < 16) perm_s[threadIdx.x] = (uint32_t)(order >> (4u * threadIdx.x)) & 15u;
    }
    __syncthreads();
    const uint32_t always = all_s;
    const uint32_t tl = (uint32_t)t, th = ctr_hi(t, kTagTri);
    for (int p = 0; p < 16; ++p) {
      const uint32_t cls = perm_s[p];
      for (uint32_t j = threadIdx.x; j < M; j += blockDim.x) {
        const uint32_t i = cls + 16u * j;
        const Philox4 r = philox10(i >> 1, 0u, tl, th, R.k0, R.k1);
        const uint32_t wd = (i & 1u) ? r.z : r.x, u = (i & 1u) ? r.w : r.y;
        const uint32_t d = (uint32_t)(((uint64_t)wd * 6u) >> 32);
        const uint32_t b = tri_nb(i, d, L, N);
        const uint32_t vi = ring[i], vb = ring[b];
        if (vi == vb) continue;
        // the i-b bond is unlike and appears once in each neighbourhood
        uint32_t n = 0;
#pragma unroll
        for (uint32_t e = 0; e < 6; ++e) n += ring[tri_nb(i, e, L, N)] != vi;
#pragma unroll
        for (uint32_t e = 0; e < 6; ++e) n += ring[tri_nb(b, e, L, N)] != vb;
        n -= 2u;
        if (u < thr_s[n] || ((always >> n) & 1u)) {
          ring[i] = (uint8_t)vb;
          ring[b] = (uint8_t)vi;
          ++cnt;
        }
      }
      __syncthreads();
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < N; i += blockDim.x) lat[i] = ring[i];
  count_ring(cnt, R, red);
}

// ---------------------------------------------------------------------------
// Where a lane finds the words around its own.  Word w of class c at distance d
// is word w + ((c + d) >> 4), mod W, of class (c + d) mod 16.  With L = 16 a + M
// (M = 4 or 12) and c known when the code is compiled only the lane's part of
// the address is not: eleven places for all classes, each with the turn that
// aligns its bits to the centres' (right by one past the last word, left by one
// before the first).
struct RingLane {
  uint32_t* x[11];  // own; one word on, one back; a and a + 1 on; a + 1 and a back; 2L likewise on, back
  uint32_t rot[11];
};
// A lane without a word (w >= W) has the words w of all classes for its own
// (kRingWords): its flips are zero.
template <int M>
__device__ __forceinline__ RingLane ring_lane(uint32_t* S, int w, int W, int L) {
  const int a = L >> 4, b = 2 * a + (M == 12 ? 1 : 0);
  const int by[11] = {0, 1, -1, a, a + 1, -a - 1, -a, b, b + 1, -b - 1, -b};
  RingLane z;
#pragma unroll
  for (int i = 0; i < 11; ++i) {
    const int x = w < W ? w + by[i] : w;
    const int turn = w < W ? (x >= W ? 1 : (x < 0 ? -1 : 0)) : 0;
    z.x[i] = S + (x - turn * W);
    z.rot[i] = (uint32_t)turn;
  }
  return z;
}

// Indexes of RingLane for class C: T = C + d less the part of d that by[] holds.
constexpr int ring_near(int T) { return T < 0 ? 2 : (T > 15 ? 1 : 0); }
constexpr int ring_row(int T) { return (T & 15) * kRingStride; }
template <int I, int T>
__device__ __forceinline__ uint32_t ring_read(const RingLane& z) {
  return rotr(z.x[I][ring_row(T)], z.rot[I]);
}
template <int M, int C>
__device__ __forceinline__ Around ring_around(const RingLane& z) {
  Around v;
  v.a = z.x[0][ring_row(C)];
  v.e = ring_read<ring_near(C + 1), C + 1>(z);
  v.w = ring_read<ring_near(C - 1), C - 1>(z);
  v.s = ring_read<3 + ((C + M) >> 4), C + M>(z);
  v.n = ring_read<6 + ((C - M) >> 4), C - M>(z);
  v.sw = ring_read<3 + ((C + M - 1) >> 4), C + M - 1>(z);
  v.ne = ring_read<6 + ((C - M + 1) >> 4), C - M + 1>(z);
  v.se = ring_read<3 + ((C + M + 1) >> 4), C + M + 1>(z);
  v.nw = ring_read<6 + ((C - M - 1) >> 4), C - M - 1>(z);
  v.sww = ring_read<3 + ((C + M - 2) >> 4), C + M - 2>(z);
  v.nee = ring_read<6 + ((C - M + 2) >> 4), C - M + 2>(z);
  v.e2 = ring_read<ring_near(C + 2), C + 2>(z);
  v.w2 = ring_read<ring_near(C - 2), C - 2>(z);
  v.s2 = ring_read<7 + ((C + 8) >> 4), C + 8>(z);
  v.n2 = ring_read<10 + ((C - 8) >> 4), C - 8>(z);
  v.ssw = ring_read<7 + ((C + 7) >> 4), C + 7>(z);
  v.nne = ring_read<10 + ((C - 7) >> 4), C - 7>(z);
  v.sw2 = ring_read<7 + ((C + 6) >> 4), C + 6>(z);
  v.ne2 = ring_read<10 + ((C - 6) >> 4), C - 6>(z);
  return v;
}

// B bits from bit 2 on, repeated once around on both sides.
__device__ __forceinline__ uint32_t around_ends(uint32_t x, int B) { return x | (x >> B) | (x << B); }

// Flip bits X of class C's words where it lies T - C (less by[I]) away.
template <int I, int T>
__device__ __forceinline__ void ring_flip(const RingLane& z, uint32_t X) {
  atomicXor(&z.x[I][ring_row(T)], rotr(X, 0u - z.rot[I]));
}
// One phase: the accepted centres of a word, and their exchanges, the repeated
// bits with them (d's direction bits are repeated as well).
template <int M, int C>
__device__ __forceinline__ uint32_t ring_phase(const RingLane& z, const Draw& d, uint32_t negmask, uint32_t cmask,
                                               int B) {
  const uint32_t F = decide(ring_around<M, C>(z), d, negmask, cmask);
  const uint32_t X = around_ends(F, B);
  const uint32_t f0 = lut3<kA & ~kB>(X, d.ax1, d.ax1), f1 = lut3<kA & kB & ~kC>(X, d.ax1, d.ax2);
  const uint32_t f2 = X & d.ax2;
  atomicXor(&z.x[0][ring_row(C)], X);
  ring_flip<ring_near(C + 1), C + 1>(z, f0 & ~d.sgn);
  ring_flip<ring_near(C - 1), C - 1>(z, f0 & d.sgn);
  ring_flip<3 + ((C + M) >> 4), C + M>(z, f1 & ~d.sgn);
  ring_flip<6 + ((C - M) >> 4), C - M>(z, f1 & d.sgn);
  ring_flip<3 + ((C + M - 1) >> 4), C + M - 1>(z, f2 & ~d.sgn);
  ring_flip<6 + ((C - M + 1) >> 4), C - M + 1>(z, f2 & d.sgn);
  asm volatile("; class %0" ::"n"(C));  // keeps the compiler from joining the classes' ends
  return F;
}

// The class order of sweep s as a scalar.
__device__ __forceinline__ uint64_t ring_order(const uint64_t* orders, uint32_t s) {
  const uint64_t o = orders[s & 127u];
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)o);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(o >> 32));
  return (uint64_t)lo | ((uint64_t)hi << 32);
}

// The phase waves' part of all sweeps: returns the accepted count of the lane.
// One wave alone needs no barrier between its phases.
template <int M>
__device__ __forceinline__ unsigned long long ring_phases(uint32_t* S, const uint32_t* D, const uint64_t* orders,
                                                          int w, int W, int L, int B, uint32_t sweeps,
                                                          uint32_t negmask, bool alone) {
  const uint32_t cmask = w < W ? ((1u << B) - 1u) << 2 : 0u;
  const int wc = min(w, W - 1);
  const RingLane z = ring_lane<M>(S, w, W, L);
  unsigned long long cnt = 0;
#pragma unroll 1
  for (uint32_t s = 0; s < sweeps; ++s) {
    uint64_t order = ring_order(orders, s);
    const uint32_t* buf = D + 6 * ((int)(16u * (s & 1u)) * W + wc);
    auto load = [&](int c) {
      const uint2* q = reinterpret_cast<const uint2*>(buf + 6 * c * W);
      const uint2 x = q[0], y = q[1], v = q[2];
      return Draw{x.x, x.y, y.x, y.y, v.x, v.y};
    };
    int c = (int)order & 15;
    Draw next = load(c);
#pragma unroll 1
    for (int p = 0; p < 16; ++p) {
      const Draw d = next;
      order >>= 4;
      const int cn = (int)order & 15;
      next = load(cn);  // the last phase loads class 0 for nothing
      uint32_t F = 0u;
#define KK_RING_CLASS(C)                           \
  case C:                                          \
    F = ring_phase<M, C>(z, d, negmask, cmask, B); \
    break;
      switch (c) {
        KK_RING_CLASS(0)
        KK_RING_CLASS(1)
        KK_RING_CLASS(2)
        KK_RING_CLASS(3)
        KK_RING_CLASS(4)
        KK_RING_CLASS(5)
        KK_RING_CLASS(6)
        KK_RING_CLASS(7)
        KK_RING_CLASS(8)
        KK_RING_CLASS(9)
        KK_RING_CLASS(10)
        KK_RING_CLASS(11)
        KK_RING_CLASS(12)
        KK_RING_CLASS(13)
        KK_RING_CLASS(14)
        KK_RING_CLASS(15)
        default: break;  // a class is below 16
      }
#undef KK_RING_CLASS
      cnt += (unsigned)__builtin_popcount(F);
      c = cn;
      if (!alone && p < 15) __syncthreads();
    }
    __syncthreads();
  }
  return cnt;
}

// The waves share the work by role.  The W words of a class fill nb waves,
// which take the phases; the others draw the next sweep's random words into the
// other of two buffers, 64 (pair of classes, word) at a time, and every 64
// sweeps the last one computes the next 64 class orders, one per lane.  With one
// phase wave all meet once per sweep; with more they meet after every phase,
// and the draws are cut into 16 parts.
//
// What bounds it: one wave's latency in a phase (19 LDS reads, about 100
// dependent instructions, 7 LDS xors: 0.41 us, whatever the size); with more
// than one wave per class, the draws' VALU issue.  100^2 6.7 us per sweep
// against 16.8 with a byte per site and a Philox block per attempt, 12^2 6.8
// against 9.0, 132^2 9.5 against 23.9, 260 x 280 23.9 against 77.9; handing the
// phases around between three waves that compute general addresses 14.6 at
// 100^2.
__device__ __forceinline__ void hex_ring(const TriResidentRep& R, uint32_t* lds, unsigned long long* red) {
  const int L = (int)R.L, N = (int)(R.L * R.H), B = (int)R.seg;
  const int W = N / (16 * B), K = 16 * W;
  const int lane = (int)(threadIdx.x & 63u), nthreads = (int)blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), nwaves = nthreads >> 6;
  const int nb = (W + 63) >> 6, ndraw = nwaves - nb;
  uint32_t* S = lds;                      // [class][kRingStride]
  uint32_t* D = S + kRingWords;           // [buffer][class][W][6]
  uint64_t* orders = reinterpret_cast<uint64_t*>(D + 12 * K);  // of 128 sweeps
  const HexAccept acc = hex_accept(R.acc);
  for (int k = (int)threadIdx.x; k < K; k += nthreads) {
    uint32_t x = 0u;
#pragma unroll 4
    for (int j = 0; j < B; ++j) x |= (uint32_t)R.lat[k + K * j] << (2 + j);
    S[(k & 15) * kRingStride + (k >> 4)] = around_ends(x, B);
  }
  unsigned long long cnt = 0;
  if (wave < nb) {
    __builtin_amdgcn_s_setprio(3);
    __syncthreads();  // the ring, the first draws and orders
    const int w = 64 * wave + lane;
    cnt = (L & 15) == 4 ? ring_phases<4>(S, D, orders, w, W, L, B, R.sweeps, acc.negmask, nb == 1)
                        : ring_phases<12>(S, D, orders, w, W, L, B, R.sweeps, acc.negmask, nb == 1);
    __builtin_amdgcn_s_setprio(0);
  } else {
    auto draw_orders = [&](uint32_t first) {
      const uint64_t t = R.t0 + first + (uint32_t)lane;
      orders[(first + (uint32_t)lane) & 127u] = order_of(
          [&](int j) { return philox10((uint32_t)j, 0u, (uint32_t)t, ctr_hi(t, kTagTriOrder), R.k0, R.k1); });
    };
    const int inv = (1 << 20) / W + 1, ntask = (8 * W + 63) >> 6;
    // blocks of the longest wave's tasks per part of a sweep
    const int longest = (ntask + ndraw - 1) / ndraw * B, parts = nb == 1 ? 1 : 16, quota = (longest + parts - 1) / parts;
    Head hd{};
    Draw e{}, o{};
    int task = ntask, left = 0, blk = 0;
    uint32_t* dst = D;
    bool dst_ok = false;
    auto begin_task = [&](uint32_t buf) {
      const int f = 64 * task + lane, fc = min(f, 8 * W - 1);
      const int pair = (int)(((uint32_t)fc * (uint32_t)inv) >> 20), w = fc - pair * W;
      blk = pair + 8 * (w + W * (B - 1));
      dst = D + 6 * ((int)(16u * buf + 2u * (uint32_t)pair) * W + w);
      dst_ok = f < 8 * W;
      left = B;
      e = Draw{};
      o = Draw{};
    };
    auto begin_draws = [&](uint32_t s) {
      const uint64_t t = R.t0 + s;
      hd = philox_head(0u, (uint32_t)t, ctr_hi(t, kTagTri), R.k0, R.k1);
      task = wave - nb;
      if (task < ntask) begin_task(s & 1u);
    };
    auto store = [&](uint32_t* d, const Draw& q) {
      uint2* p = reinterpret_cast<uint2*>(d);
      p[0] = make_uint2(around_ends(q.sgn << 2, B), around_ends(q.ax1 << 2, B));
      p[1] = make_uint2(around_ends(q.ax2 << 2, B), (q.a0 << 2) | acc.all[0]);
      p[2] = make_uint2((q.a1 << 2) | acc.all[1], (q.a2 << 2) | acc.all[2]);
    };
    auto draw_blocks = [&](int n, uint32_t buf) {
#pragma unroll 1
      while (n > 0 && task < ntask) {
        const int m = min(n, left);
#pragma unroll 1
        for (int i = 0; i < m; ++i) {
          const Philox4 w = philox_tail(hd, (uint32_t)blk);
          push_attempt(e, w.x, w.y, acc);
          push_attempt(o, w.z, w.w, acc);
          blk -= 8 * W;
        }
        n -= m;
        left -= m;
        if (left == 0) {
          if (dst_ok) {
            store(dst, e);
            store(dst + 6 * W, o);
          }
          task += ndraw;
          if (task < ntask) begin_task(buf);
        }
      }
    };
    const bool last = wave == nwaves - 1;
    if (last) draw_orders(0u);
    begin_draws(0u);
    draw_blocks(longest, 0u);
    __syncthreads();
#pragma unroll 1
    for (uint32_t s = 0; s < R.sweeps; ++s) {
      const bool more = s + 1u < R.sweeps;
      if (more) begin_draws(s + 1u);
      if (last && (s & 63u) == 32u) draw_orders((s & ~63u) + 64u);
#pragma unroll 1
      for (int p = 0; p < parts; ++p) {
        if (more) draw_blocks(quota, (s + 1u) & 1u);
        __syncthreads();
      }
    }
  }
  for (int k = (int)threadIdx.x; k < K; k += nthreads) {
    const uint32_t x = S[(k & 15) * kRingStride + (k >> 4)];
#pragma unroll 4
    for (int j = 0; j < B; ++j) R.lat[k + K * j] = (uint8_t)((x >> (2 + j)) & 1u);
  }
  count_ring(cnt, R, red);
}

__device__ __forceinline__ void run_ring(const TriResidentRep& R, uint32_t* lds) {
  __shared__ unsigned long long red[16];
  if (R.sweeps == 0u) return;
  if (R.seg) hex_ring(R, lds, red);
  else byte_ring(R, reinterpret_cast<uint8_t*>(lds), red);
}

__global__ __launch_bounds__(1024) void ring_sweeps(const TriResidentRep* reps) {
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  run_ring(reps[blockIdx.x], lds);
}

__global__ __launch_bounds__(1024) void ring_sweeps_one(TriResidentRep R) {
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  run_ring(R, lds);
}

}  // namespace

hipError_t launch_tri_resident(const TriResidentRep* reps, uint32_t nreps, size_t lds_bytes, hipStream_t stream) {
  if (nreps == 0) return hipSuccess;
  hipLaunchKernelGGL(ring_sweeps, dim3(nreps), dim3(1024), lds_bytes, stream, reps);
  return hipGetLastError();
}

hipError_t launch_tri_resident_one(const TriResidentRep& rep, size_t lds_bytes, hipStream_t stream) {
  hipLaunchKernelGGL(ring_sweeps_one, dim3(1), dim3(1024), lds_bytes, stream, rep);
  return hipGetLastError();
}

}  // namespace kk
