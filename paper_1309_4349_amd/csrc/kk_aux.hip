// kk_aux.hip -- initial placement, energy, cluster labelling and layout
// conversion kernels of libkk.
#include <algorithm>

#include "kk_common.hpp"
#include "kk_kernels.hpp"
#include "kk_ccl.hpp"

namespace kk {

namespace {

constexpr uint32_t kNone = 0xFFFFFFFFu;

__device__ __forceinline__ int site_bit(const void* lat, int layout, int L, int x, int y) {
  if (layout == kLayoutBits)
    return (int)((static_cast<const uint32_t*>(lat)[(size_t)y * (L >> 5) + (x >> 5)] >> (x & 31)) & 1u);
  return (int)(static_cast<const uint8_t*>(lat)[(size_t)y * L + x] & 1u);
}

constexpr int kSumBlocks = 512;  // workgroups of a summing pass (each thread strides)

// ---------------------------------------------------------------------------
// Energy: N_AB = sum over sites of [s(x,y) != s(x+1,y)] + [s(x,y) != s(x,y+1)]
// (the Almeida one-parameter model, E/kT = omega * N_AB + const).  A thread's
// count stays below 2^32: at most 2 bonds of 2^30 sites over 2^17 threads.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void energy_bits(const uint32_t* lat, int L, unsigned long long* out,
                                                   bool spread) {
  const int wpr = L >> 5;
  const size_t nw = (size_t)L * wpr;
  unsigned acc = 0;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nw; i += (size_t)gridDim.x * blockDim.x) {
    const int y = (int)(i / wpr), g = (int)(i - (size_t)y * wpr);
    const uint32_t v = lat[i];
    const uint32_t nxt = lat[(size_t)y * wpr + (g + 1 == wpr ? 0 : g + 1)];
    const uint32_t east = __builtin_amdgcn_alignbit(nxt, v, 1);
    const uint32_t below = lat[(size_t)(y + 1 == L ? 0 : y + 1) * wpr + g];
    acc += (unsigned)__builtin_popcount(v ^ east) + (unsigned)__builtin_popcount(v ^ below);
  }
  add_block_sum(acc, out, spread);
}

// Four sites (one per byte) at a time: L is a multiple of 4.
__global__ __launch_bounds__(256) void energy_int8(const uint8_t* lat, int L, unsigned long long* out,
                                                   bool spread) {
  const uint32_t* w = reinterpret_cast<const uint32_t*>(lat);
  const int wpr = L >> 2;
  const size_t nw = (size_t)L * wpr;
  unsigned acc = 0;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nw; i += (size_t)gridDim.x * blockDim.x) {
    const int y = (int)(i / wpr), g = (int)(i - (size_t)y * wpr);
    const uint32_t v = w[i];
    const uint32_t nxt = w[(size_t)y * wpr + (g + 1 == wpr ? 0 : g + 1)];
    const uint32_t below = w[(size_t)(y + 1 == L ? 0 : y + 1) * wpr + g];
    acc += (unsigned)__builtin_popcount(v ^ __builtin_amdgcn_alignbit(nxt, v, 8)) +
           (unsigned)__builtin_popcount(v ^ below);
  }
  add_block_sum(acc, out, spread);
}

// Random-neighbour estimate of the similar first-neighbour fraction: every
// site draws one of its 4 neighbours (top two bits of its word of Philox block
// (y, x / 4, t, tag 5): +x, -x, +y, -y) and counts when both are of the same
// type.  One thread per 4-site group (one Philox block); L % 4 == 0.
__global__ __launch_bounds__(256) void similar_sampled(const void* lat, int layout, int L, uint32_t k0, uint32_t k1,
                                                       uint64_t t, unsigned long long* out, bool spread) {
  const int g4 = L >> 2;
  const size_t n = (size_t)L * g4;
  const uint32_t tl = (uint32_t)t, th = ctr_hi(t, kTagObserve);
  unsigned acc = 0;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int y = (int)(i / g4), q = (int)(i - (size_t)y * g4);
    const Philox4 r = philox10((uint32_t)y, (uint32_t)q, tl, th, k0, k1);
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int x = 4 * q + m;
      const uint32_t dir = w[m] >> 30;
      int nx = x, ny = y;
      if (dir == 0u) nx = (x + 1 == L) ? 0 : x + 1;
      else if (dir == 1u) nx = (x == 0) ? L - 1 : x - 1;
      else if (dir == 2u) ny = (y + 1 == L) ? 0 : y + 1;
      else ny = (y == 0) ? L - 1 : y - 1;
      acc += (site_bit(lat, layout, L, x, y) == site_bit(lat, layout, L, nx, ny));
    }
  }
  add_block_sum(acc, out, spread);
}

// ---------------------------------------------------------------------------
// Initial placement: each site's 64-bit key is Philox block (y, x, 0, tag 4)
// words 0 and 1; the n1 sites with the smallest (key, index) get type 1.
//  1. place_count_keys counts the keys by their top 10 bits.
//  2. place_mark finds the bin that holds the n1-th smallest key, gives the sites
//     below it type 1 and lists the sites in it (one in 1024).
//  3. place_select, one workgroup, takes the rest of them by a radix select over
//     the remaining key bits, then the index.
// The keys are computed again in the second pass instead of being kept: a block
// of Philox per site is cheaper than 8 bytes written and read.  Nothing returns
// to the host between the passes.  Eight passes over stored keys, each with its
// histogram on the host, made a 64^2 handle 0.46 ms and a 4096^2 one 1.3 ms to
// create; now 0.25 and 0.74, allocations for the most part.
// ---------------------------------------------------------------------------
constexpr int kPlaceBins = 1024;

struct PlaceList {
  uint64_t* key;
  uint32_t* idx;
  unsigned* count;
  uint32_t cap;
};

__device__ __forceinline__ uint64_t place_key(uint32_t i, uint32_t L, uint32_t k0, uint32_t k1) {
  const uint32_t y = i / L;
  const Philox4 r = philox10(y, i - y * L, 0u, kTagInit << 28, k0, k1);
  return ((uint64_t)r.x << 32) | (uint64_t)r.y;
}

__global__ __launch_bounds__(1024) void place_count_keys(uint32_t L, uint32_t n, uint32_t k0, uint32_t k1,
                                                         unsigned* hist) {
  __shared__ unsigned h[kPlaceBins];
  h[threadIdx.x] = 0u;
  __syncthreads();
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    atomicAdd(&h[place_key(i, L, k0, k1) >> 54], 1u);
  __syncthreads();
  if (h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
}

// Of NB counts (one per thread of the first NB), the bin that holds the
// need-th entry, and how many of its entries are needed.
struct PlaceBin {
  uint32_t bin, need, count;
};
template <int NB>
__device__ __forceinline__ PlaceBin place_bin(unsigned c, uint32_t need) {
  __shared__ uint32_t sum[NB / 64];
  __shared__ PlaceBin found;
  const int tid = (int)threadIdx.x, lane = tid & 63;
  uint32_t upto = c;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = __shfl_up(upto, off, 64);
    upto += lane >= off ? o : 0u;
  }
  if (tid < NB && lane == 63) sum[tid >> 6] = upto;
  __syncthreads();
  if (tid < NB) {
    for (int w = 0; w < (tid >> 6); ++w) upto += sum[w];
    if (upto >= need && upto - c < need) found = PlaceBin{(uint32_t)tid, need - (upto - c), c};
  }
  __syncthreads();
  const PlaceBin f = found;
  __syncthreads();
  return f;
}

// The list of sites in the bin: key and index.  A workgroup gathers its own
// first (one addition to the list's length instead of one per site).
__global__ __launch_bounds__(1024) void place_mark(uint32_t L, uint32_t n, int layout, uint32_t n1, uint32_t k0,
                                                   uint32_t k1, const unsigned* hist, void* lat, PlaceList list) {
  constexpr uint32_t kMine = 1024;
  __shared__ uint64_t key_s[kMine];
  __shared__ uint32_t idx_s[kMine];
  __shared__ uint32_t mine, base;
  if (threadIdx.x == 0) mine = 0u;
  const PlaceBin b = place_bin<kPlaceBins>(hist[threadIdx.x], n1);
  for (uint32_t i0 = blockIdx.x * blockDim.x; i0 < n; i0 += gridDim.x * blockDim.x) {
    const uint32_t i = i0 + threadIdx.x;
    const uint64_t k = i < n ? place_key(i, L, k0, k1) : ~0ull;
    const uint32_t top = (uint32_t)(k >> 54);
    const bool one = i < n && top < b.bin;
    if (layout == kLayoutBits) {  // L is a multiple of 32: half a wavefront per word, all of it in range or none
      const uint64_t m = __ballot(one);
      if ((threadIdx.x & 31u) == 0u && i < n) static_cast<uint32_t*>(lat)[i >> 5] = (uint32_t)(m >> (threadIdx.x & 32u));
    } else if (i < n) {
      static_cast<uint8_t*>(lat)[i] = (uint8_t)one;
    }
    if (i < n && top == b.bin) {
      const uint32_t s = atomicAdd(&mine, 1u);
      if (s < kMine) {
        key_s[s] = k;
        idx_s[s] = i;
      } else {
        const uint32_t g = atomicAdd(list.count, 1u);
        if (g < list.cap) {
          list.key[g] = k;
          list.idx[g] = i;
        }
      }
    }
  }
  __syncthreads();
  const uint32_t m = min(mine, kMine);
  if (threadIdx.x == 0) base = atomicAdd(list.count, m);
  __syncthreads();
  for (uint32_t s = threadIdx.x; s < m; s += blockDim.x)
    if (base + s < list.cap) {
      list.key[base + s] = key_s[s];
      list.idx[base + s] = idx_s[s];
    }
}

// One workgroup: digits of 8 bits, first the key's lower 56, then the index's
// 32, until a digit's bin is needed whole.  *length is the list's full length.
__global__ __launch_bounds__(1024) void place_select(int layout, uint32_t n1, const unsigned* hist, void* lat,
                                                     PlaceList list, uint32_t* length) {
  __shared__ unsigned h[256];
  uint32_t need = place_bin<kPlaceBins>(hist[threadIdx.x], n1).need;
  const uint32_t m = min(*list.count, list.cap);
  if (threadIdx.x == 0) *length = *list.count;
  uint64_t pk = m ? list.key[0] & 0xFF00000000000000ull : 0ull;  // the digits found so far (the bin has the first)
  uint32_t pi = 0u;
  // whether an entry agrees with the digits before this level, and its digit
  auto digit = [&](int level, uint64_t k, uint32_t i, bool& in) {
    if (level < 7) {
      in = ((k ^ pk) >> (56 - 8 * level)) == 0;
      return (uint32_t)(k >> (48 - 8 * level)) & 255u;
    }
    const int sh = 24 - 8 * (level - 7);
    in = k == pk && ((uint64_t)(i ^ pi) >> (sh + 8)) == 0;
    return (i >> sh) & 255u;
  };
  int level = 0;
  for (; level < 11; ++level) {
    if (threadIdx.x < 256) h[threadIdx.x] = 0u;
    __syncthreads();
    for (uint32_t s = threadIdx.x; s < m; s += blockDim.x) {
      bool in;
      const uint32_t d = digit(level, list.key[s], list.idx[s], in);
      if (in) atomicAdd(&h[d], 1u);
    }
    __syncthreads();
    const PlaceBin f = place_bin<256>(threadIdx.x < 256 ? h[threadIdx.x] : 0u, need);
    if (level < 7) pk |= (uint64_t)f.bin << (48 - 8 * level);
    else pi |= f.bin << (24 - 8 * (level - 7));
    need = f.need;
    if (f.need == f.count) break;
  }
  level = min(level, 10);
  for (uint32_t s = threadIdx.x; s < m; s += blockDim.x) {
    const uint64_t k = list.key[s];
    const uint32_t i = list.idx[s];
    bool take;
    if (level < 7) {
      take = (k >> (48 - 8 * level)) <= (pk >> (48 - 8 * level));
    } else {
      const int sh = 24 - 8 * (level - 7);
      take = k < pk || (k == pk && (i >> sh) <= (pi >> sh));
    }
    if (!take) continue;
    if (layout == kLayoutBits) atomicOr(&static_cast<uint32_t*>(lat)[i >> 5], 1u << (i & 31u));
    else static_cast<uint8_t*>(lat)[i] = 1;
  }
}

// Segregated start: the first n1 sites in index order i = y*L + x hold type 1
// (full rows 0 .. n1/L - 1 and the start of the next one).  Bit-packed words
// tile rows exactly, so word w holds sites 32w .. 32w + 31.
__global__ __launch_bounds__(256) void fill_segregated(void* lat, int layout, int L, int H, uint64_t n1) {
  const size_t n = (size_t)L * H;
  if (layout == kLayoutBits) {
    uint32_t* w = static_cast<uint32_t*>(lat);
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n / 32; i += (size_t)gridDim.x * blockDim.x) {
      const uint64_t lo = 32 * (uint64_t)i;
      w[i] = n1 >= lo + 32 ? 0xFFFFFFFFu : (n1 <= lo ? 0u : ((1u << (uint32_t)(n1 - lo)) - 1u));
    }
  } else {
    uint8_t* b = static_cast<uint8_t*>(lat);
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
      b[i] = (uint64_t)i < n1 ? 1 : 0;
  }
}

// ---------------------------------------------------------------------------
// Cluster sizes.  The lattice is cut into tiles of 64 x 64 sites.
//  1. ccl_tile labels each tile by itself in LDS (union-find over the runs of
//     each row, found as bits of the row's 64-site mask) and writes its
//     clusters compactly -- id = (sites of the tiles before) / 2 + k, as a tile
//     holds at most half as many clusters as sites -- with their sizes, and the
//     ids of the sites along its four edges.
//  2. ccl_border unites the clusters across the tiles' edges (lock-free
//     union-find over the ids: atomicMin links toward smaller ids, so no cycle
//     can form, and path halving).
//  3. ccl_sizes adds every cluster's size to its root's.
//  4. ccl_hist counts the roots by size: small sizes through a dense histogram
//     per workgroup in LDS, the few of kSmallSizes or more as a list.
// Only the lattice is read per site; all else is per cluster and per edge site.
// The per-site labelling before (parent and size words for every site, four
// passes over them, dependent reads of global memory) took 1.7 ms at 4096^2 and
// 4.1 ms on a 4092^2 triangular ring; now 0.16 and 0.28 ms, of which the first
// pass 0.10 and 0.14 (bound by the chains of dependent LDS reads of a tile's
// unions: 4 tiles per CU hold its 160 KB).  On lattices of a few tiles each pass
// is one workgroup's latency: 400^2 at omega -1.2, whose clusters are single
// sites for the most part, 12 + 4 + 6 + 7 us.  (27, 5, 6 and 30 us with four
// wavefronts per tile that load one row after another, a histogram workgroup for
// every 8 tiles, and an LDS addition for every cluster, nearly all on one word:
// slower than the labelling before up to 800^2.)
// ---------------------------------------------------------------------------
constexpr int kTile = 64;

__device__ __forceinline__ uint32_t ld_parent(const uint32_t* parent, uint32_t x) {
  return __hip_atomic_load(&parent[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of x with path halving: every visited node is re-linked to its
// grandparent.  Links only ever decrease (atomicMin) and always point to an
// ancestor in the same tree, so concurrent finds and unions stay consistent.
__device__ __forceinline__ uint32_t find_root_halving(uint32_t* parent, uint32_t x) {
  uint32_t p = ld_parent(parent, x);
  while (p != x) {
    const uint32_t g = ld_parent(parent, p);
    if (g != p) atomicMin(&parent[x], g);
    x = p;
    p = g;
  }
  return x;
}

__device__ void unite(uint32_t* parent, uint32_t a, uint32_t b) {
  for (;;) {
    a = find_root_halving(parent, a);
    b = find_root_halving(parent, b);
    if (a == b) return;
    if (a > b) {
      const uint32_t t = a;
      a = b;
      b = t;
    }
    const uint32_t old = atomicMin(&parent[b], a);
    if (old == b) return;
    b = old;
  }
}

// The same within a workgroup, on LDS.
__device__ __forceinline__ uint32_t lds_root(volatile uint32_t* par, uint32_t x) {
  uint32_t p = par[x];
  while (p != x) {
    x = p;
    p = par[x];
  }
  return x;
}
__device__ __forceinline__ void lds_unite(uint32_t* par, uint32_t a, uint32_t b) {
  for (;;) {
    a = lds_root(par, a);
    b = lds_root(par, b);
    if (a == b) return;
    const uint32_t hi = max(a, b), lo = min(a, b);
    const uint32_t old = atomicMin(&par[hi], lo);
    if (old == hi) return;
    a = lo;
    b = old;
  }
}

// First site of the run of mask m that holds bit x.
__device__ __forceinline__ uint32_t run_start(uint64_t m, uint32_t x) {
  const uint64_t gap = ~m & ((1ull << x) - 1ull);
  return gap ? 64u - (uint32_t)__clzll((long long)gap) : 0u;
}

struct CclShape {
  const void* lat;
  int layout, L, H;
};

struct CclTile {
  int tx, ty, x0, y0, w, h;
  uint32_t base;  // id of its first cluster
};
__device__ __forceinline__ CclTile ccl_place(const CclShape& g, int tile) {
  const int ntx = (g.L + kTile - 1) / kTile;
  CclTile t;
  t.ty = tile / ntx;
  t.tx = tile - t.ty * ntx;
  t.x0 = t.tx * kTile;
  t.y0 = t.ty * kTile;
  t.w = min(kTile, g.L - t.x0);
  t.h = min(kTile, g.H - t.y0);
  t.base = ((uint32_t)t.y0 * (uint32_t)g.L + (uint32_t)t.x0 * (uint32_t)t.h) / 2u;  // both products are even
  return t;
}

// One workgroup of NW wavefronts per tile (strided over the grid).
template <bool TRI, int NW>
__device__ __forceinline__ void ccl_tile_body(const CclShape& g, int species, const CclBuffers& b) {
  __shared__ uint64_t rows[kTile];
  __shared__ uint32_t par[kTile * kTile], cnt[kTile * kTile];
  __shared__ uint32_t nroot;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const size_t gt = blockIdx.x * (size_t)blockDim.x + threadIdx.x, nth = (size_t)gridDim.x * blockDim.x;
  for (size_t i = gt; i < (size_t)kSmallSizes; i += nth) b.hist[i] = 0u;
  if (gt == 0) *b.big_count = 0u;
  const int ntx = (g.L + kTile - 1) / kTile, nty = (g.H + kTile - 1) / kTile;
  for (int tile = (int)blockIdx.x; tile < ntx * nty; tile += (int)gridDim.x) {
    const CclTile t = ccl_place(g, tile);
    const int x0 = t.x0, y0 = t.y0, w = t.w, h = t.h;
    if (tid == 0) nroot = 0u;
    // a wave's rows, with all of its loads in flight at once
    if (g.layout == kLayoutBits) {  // a row per lane, one word (w == 32) or two
      if (lane < kTile / NW) {
        const int r = wave + NW * lane;
        const uint32_t* q =
            static_cast<const uint32_t*>(g.lat) + (size_t)(y0 + min(r, h - 1)) * (g.L >> 5) + (x0 >> 5);
        const uint64_t flip = species ? 0ull : ~0ull, in = w > 32 ? ~0ull : 0xFFFFFFFFull;
        const uint64_t m = (uint64_t)q[0] | ((uint64_t)q[w > 32 ? 1 : 0] << 32);
        rows[r] = r < h ? (m ^ flip) & in : 0ull;
      }
    } else {
      const uint8_t* q = static_cast<const uint8_t*>(g.lat) + (size_t)x0 + min(lane, w - 1);
      int site[kTile / NW];
#pragma unroll
      for (int k = 0; k < kTile / NW; ++k) site[k] = q[(size_t)(y0 + min(wave + NW * k, h - 1)) * g.L] & 1;
#pragma unroll
      for (int k = 0; k < kTile / NW; ++k) {
        const uint64_t m = __ballot(wave + NW * k < h && lane < w && site[k] == species);
        if (lane == 0) rows[wave + NW * k] = m;
      }
    }
    for (int r = wave; r < kTile; r += NW) {
      par[r * kTile + lane] = (uint32_t)(r * kTile + lane);
      cnt[r * kTile + lane] = 0u;
    }
    __syncthreads();
    // bonds to the row above, one union per stretch of them
    for (int r = wave == 0 ? NW : wave; r < h; r += NW) {
      const uint64_t m = rows[r], mp = rows[r - 1];
      const uint64_t o = m & mp, os = o & ~(o << 1);
      if ((os >> lane) & 1ull)
        lds_unite(par, (uint32_t)(r * kTile) + run_start(m, (uint32_t)lane),
                  (uint32_t)((r - 1) * kTile) + run_start(mp, (uint32_t)lane));
      if constexpr (TRI) {  // (r, x) and (r - 1, x + 1)
        const uint64_t d = m & (mp >> 1), ds = d & ~(d << 1);
        if ((ds >> lane) & 1ull)
          lds_unite(par, (uint32_t)(r * kTile) + run_start(m, (uint32_t)lane),
                    (uint32_t)((r - 1) * kTile) + run_start(mp, (uint32_t)lane + 1u));
      }
    }
    __syncthreads();
    // run starts: link to the root, add the run's length to it
    for (int r = wave; r < h; r += NW) {
      const uint64_t m = rows[r], st = m & ~(m << 1);
      if ((st >> lane) & 1ull) {
        const uint64_t run = ~(m >> lane);
        const uint32_t len = run ? (uint32_t)__ffsll((unsigned long long)run) - 1u : 64u;
        const uint32_t me = (uint32_t)(r * kTile + lane), root = lds_root(par, me);
        if (root != me) par[me] = root;
        atomicAdd(&cnt[root], len);
      }
    }
    __syncthreads();
    // the tile's clusters, numbered; cnt becomes the number of each root
    const uint32_t base = t.base;
    for (int r = wave; r < h; r += NW) {
      const uint64_t m = rows[r], st = m & ~(m << 1);
      const uint32_t me = (uint32_t)(r * kTile + lane);
      if (((st >> lane) & 1ull) && par[me] == me) {
        const uint32_t k = atomicAdd(&nroot, 1u);
        b.parent[base + k] = base + k;
        b.size[base + k] = cnt[me];
        cnt[me] = k;
      }
    }
    __syncthreads();
    {  // edges: top, bottom, left, right
      const int edge = wave;
      const int er = edge == 0 ? 0 : (edge == 1 ? h - 1 : lane), ec = edge == 2 ? 0 : (edge == 3 ? w - 1 : lane);
      uint32_t id = kNone;
      if (wave < 4 && er < h && ec < w) {
        const uint64_t m = rows[er];
        if ((m >> ec) & 1ull) id = base + cnt[par[(uint32_t)(er * kTile) + run_start(m, (uint32_t)ec)]];
      }
      if (wave < 4) b.border[(size_t)tile * 256 + tid] = id;
    }
    if (tid == 0) b.ncl[tile] = nroot;
    __syncthreads();
  }
}

// Unions across the tiles' edges, one thread per tile and edge site.  Square
// torus: the bonds to the right of the right column and below the bottom row,
// one per stretch.  Triangular ring (i + 1, i + L, i + L - 1): those of the
// right column, the bottom row and, for i + L - 1, the left column.
template <bool TRI>
__device__ __forceinline__ void ccl_border_body(const CclShape& g, const CclBuffers& b) {
  const int L = g.L, H = g.H, ntx = (L + kTile - 1) / kTile, nty = (H + kTile - 1) / kTile;
  const uint32_t* top = b.border;
  const uint32_t* bottom = b.border + 64;
  const uint32_t* left = b.border + 128;
  const uint32_t* right = b.border + 192;
  constexpr int E = TRI ? 3 : 2;
  const size_t n = (size_t)ntx * nty * (64 * E);
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int tile = (int)(i / (64 * E)), k = (int)(i - (size_t)tile * (64 * E));
    const int edge = k >> 6, pos = k & 63;
    const CclTile t = ccl_place(g, tile);
    const int tx = t.tx, ty = t.ty, y0 = t.y0, w = t.w, h = t.h;
    auto at = [&](const uint32_t* e, int ttx, int tty, int p) { return e[((size_t)tty * ntx + ttx) * 256 + p]; };
    auto link = [&](uint32_t a, uint32_t c) {
      if (a != kNone && c != kNone) unite(b.parent, a, c);
    };
    if (edge == 0) {  // right column, row pos: the site to the right
      if (pos >= h) continue;
      const uint32_t a = at(right, tx, ty, pos);
      if (TRI && tx == ntx - 1) {  // the ring goes on in the next row
        const int y = y0 + pos + 1 == H ? 0 : y0 + pos + 1;
        link(a, at(left, 0, y / kTile, y % kTile));
      } else {
        const int nx = tx + 1 == ntx ? 0 : tx + 1;
        const uint32_t c = at(left, nx, ty, pos);
        if (a == kNone || c == kNone) continue;
        if (pos > 0 && at(right, tx, ty, pos - 1) != kNone && at(left, nx, ty, pos - 1) != kNone) continue;
        unite(b.parent, a, c);
      }
    } else if (edge == 1) {  // bottom row, column pos: the sites below
      if (pos >= w) continue;
      const int ny = ty + 1 == nty ? 0 : ty + 1;
      const uint32_t a = at(bottom, tx, ty, pos), c = at(top, tx, ny, pos);
      if (a == kNone) continue;
      const bool stretch = pos > 0 && c != kNone && at(bottom, tx, ty, pos - 1) != kNone &&
                           at(top, tx, ny, pos - 1) != kNone;
      if (c != kNone && !stretch) unite(b.parent, a, c);
      if (TRI && pos > 0 && !(c != kNone && at(top, tx, ny, pos - 1) != kNone)) link(a, at(top, tx, ny, pos - 1));
    } else {  // left column, row pos: i + L - 1
      if (pos >= h) continue;
      const uint32_t a = at(left, tx, ty, pos);
      if (tx == 0) link(a, at(right, ntx - 1, ty, pos));
      else {
        const int y = y0 + pos + 1 == H ? 0 : y0 + pos + 1;
        link(a, at(right, tx - 1, y / kTile, y % kTile));
      }
    }
  }
}

// Every cluster's size onto its root's.  Most of a tile's additions go to one
// root (the largest cluster, whose id is among the smallest): those are summed
// in LDS first, one atomic per tile.
__device__ __forceinline__ void ccl_sizes_body(const CclShape& g, const CclBuffers& b) {
  __shared__ uint32_t main_root, main_sum;
  const int ntiles = ((g.L + kTile - 1) / kTile) * ((g.H + kTile - 1) / kTile);
  for (int tile = (int)blockIdx.x; tile < ntiles; tile += (int)gridDim.x) {
    const uint32_t n = b.ncl[tile], base = ccl_place(g, tile).base;
    if (threadIdx.x == 0) {
      main_root = kNone;
      main_sum = 0u;
    }
    __syncthreads();
    for (uint32_t k0 = 0; k0 < n; k0 += blockDim.x) {
      const uint32_t k = k0 + threadIdx.x;
      uint32_t r = kNone;
      if (k < n) {
        r = find_root_halving(b.parent, base + k);
        if (r == base + k) r = kNone;
      }
      if (r != kNone && k0 == 0) atomicMin(&main_root, r);
      __syncthreads();
      if (r != kNone) {
        const uint32_t s = b.size[base + k];  // a cluster that is no root keeps its own size
        if (r == main_root) atomicAdd(&main_sum, s);
        else atomicAdd(&b.size[r], s);
      }
    }
    __syncthreads();
    if (threadIdx.x == 0 && main_sum) atomicAdd(&b.size[main_root], main_sum);
    __syncthreads();
  }
}

__device__ __forceinline__ void ccl_hist_body(const CclShape& g, const CclBuffers& b, unsigned* h) {
  const int ntiles = ((g.L + kTile - 1) / kTile) * ((g.H + kTile - 1) / kTile);
  if ((int)blockIdx.x >= ntiles) return;
  for (int k = threadIdx.x; k < kSmallSizes; k += blockDim.x) h[k] = 0;
  __syncthreads();
  unsigned ones = 0;  // clusters of one site, the most frequent: additions to one word run one after another
  for (int tile = (int)blockIdx.x; tile < ntiles; tile += (int)gridDim.x) {
    const uint32_t n = b.ncl[tile], base = ccl_place(g, tile).base;
    for (uint32_t k = threadIdx.x; k < n; k += blockDim.x) {
      if (b.parent[base + k] != base + k) continue;
      const uint32_t s = b.size[base + k];
      if (s == 1u) ++ones;
      else if (s < (uint32_t)kSmallSizes) atomicAdd(&h[s], 1u);
      else {
        const unsigned slot = atomicAdd(b.big_count, 1u);
        if (slot < b.big_cap) b.big[slot] = s;
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) ones += __shfl_down(ones, off, 64);
  if ((threadIdx.x & 63) == 0) atomicAdd(&h[1], ones);
  __syncthreads();
  for (int k = threadIdx.x; k < kSmallSizes; k += blockDim.x)
    if (h[k]) atomicAdd(&b.hist[k], h[k]);
}

// The passes as kernels for one lattice, and for many square lattices at once:
// replica blockIdx.y of a table, each with its own buffers.
template <bool TRI, int NW>
__global__ __launch_bounds__(64 * NW) void ccl_tile(CclShape g, int species, CclBuffers b) {
  ccl_tile_body<TRI, NW>(g, species, b);
}
template <bool TRI>
__global__ __launch_bounds__(256) void ccl_border(CclShape g, CclBuffers b) {
  ccl_border_body<TRI>(g, b);
}
__global__ __launch_bounds__(256) void ccl_sizes(CclShape g, CclBuffers b) { ccl_sizes_body(g, b); }
__global__ __launch_bounds__(256) void ccl_hist(CclShape g, CclBuffers b) {
  __shared__ unsigned h[kSmallSizes];
  ccl_hist_body(g, b, h);
}
__device__ __forceinline__ CclShape ccl_shape(const CclRep& r) { return CclShape{r.lat, r.layout, r.L, r.L}; }
__global__ __launch_bounds__(256) void ccl_tile_many(const CclRep* reps, int species) {
  const CclRep r = reps[blockIdx.y];
  ccl_tile_body<false, 4>(ccl_shape(r), species, r.b);
}
__global__ __launch_bounds__(256) void ccl_border_many(const CclRep* reps) {
  const CclRep r = reps[blockIdx.y];
  ccl_border_body<false>(ccl_shape(r), r.b);
}
__global__ __launch_bounds__(256) void ccl_sizes_many(const CclRep* reps) {
  const CclRep r = reps[blockIdx.y];
  ccl_sizes_body(ccl_shape(r), r.b);
}
__global__ __launch_bounds__(256) void ccl_hist_many(const CclRep* reps) {
  __shared__ unsigned h[kSmallSizes];
  const CclRep r = reps[blockIdx.y];
  ccl_hist_body(ccl_shape(r), r.b, h);
}
// Every replica's result block (histogram, large-size count, first large
// sizes) into row blockIdx.y of one staging array of `words` per replica.
__global__ __launch_bounds__(256) void ccl_gather_many(const CclRep* reps, uint32_t* stage, uint32_t words) {
  const CclRep& r = reps[blockIdx.y];
  const uint32_t n = min(words, (uint32_t)kSmallSizes + 1u + r.b.big_cap);
  uint32_t* dst = stage + (size_t)blockIdx.y * words;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) dst[i] = r.b.hist[i];
}

// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_bits(const uint8_t* in, uint32_t* out, int L) {
  const size_t nw = (size_t)L * (L >> 5);
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nw; i += (size_t)gridDim.x * blockDim.x) {
    uint32_t v = 0;
    for (int b = 0; b < 32; ++b) v |= (uint32_t)(in[i * 32 + b] & 1u) << b;
    out[i] = v;
  }
}

// Sixteen sites (a half word of the lattice) per thread, one 16-byte store each:
// a wavefront's stores are one stretch, also where `out` is host memory.
__global__ __launch_bounds__(256) void unpack_bits(const uint32_t* in, uint8_t* out, int L) {
  const uint16_t* h = reinterpret_cast<const uint16_t*>(in);
  uint4* o = reinterpret_cast<uint4*>(out);
  const size_t n = (size_t)L * (L >> 4);
  auto spread = [](uint32_t nibble) { return (nibble * 0x00204081u) & 0x01010101u; };
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const uint32_t v = h[i];
    o[i] = make_uint4(spread(v & 15u), spread((v >> 4) & 15u), spread((v >> 8) & 15u), spread(v >> 12));
  }
}

// Read-back into host memory: a copy and a sum.  A copy command of the runtime
// takes about 8 us longer than a kernel that writes the bytes itself.
__global__ __launch_bounds__(256) void copy_bytes(const uint8_t* in, uint8_t* out, size_t n) {
  const uint4* v = reinterpret_cast<const uint4*>(in);
  uint4* o = reinterpret_cast<uint4*>(out);
  const size_t i0 = blockIdx.x * (size_t)blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
  for (size_t i = i0; i < n / 16; i += step) o[i] = v[i];
  for (size_t i = (n & ~(size_t)15) + i0; i < n; i += step) out[i] = in[i];
}
__global__ __launch_bounds__(256) void sum_words(const unsigned long long* in, size_t n, unsigned long long* out) {
  unsigned long long acc = 0;
  for (size_t i = threadIdx.x; i < n; i += 256) acc += in[i];
  add_block_sum(acc, out, true);
}

int grid_for(size_t n, int block) {
  size_t g = (n + block - 1) / block;
  if (g > 4096) g = 4096;
  if (g < 1) g = 1;
  return (int)g;
}

}  // namespace

hipError_t launch_energy(const void* lat, int layout, int L, unsigned long long* out, int* nsum, hipStream_t stream) {
  const bool bits = layout == kLayoutBits;
  const int n = std::min(grid_for((size_t)L * (L >> (bits ? 5 : 2)), 256), kSumBlocks);
  if (nsum) *nsum = n;
  if (bits)
    hipLaunchKernelGGL(energy_bits, dim3(n), dim3(256), 0, stream, static_cast<const uint32_t*>(lat), L, out,
                       nsum != nullptr);
  else
    hipLaunchKernelGGL(energy_int8, dim3(n), dim3(256), 0, stream, static_cast<const uint8_t*>(lat), L, out,
                       nsum != nullptr);
  return hipGetLastError();
}

hipError_t launch_similar_sampled(const void* lat, int layout, int L, uint32_t k0, uint32_t k1, uint64_t t,
                                  unsigned long long* out, int* nsum, hipStream_t stream) {
  const int n = std::min(grid_for((size_t)L * (L >> 2), 256), 4 * kSumBlocks);
  if (nsum) *nsum = n;
  hipLaunchKernelGGL(similar_sampled, dim3(n), dim3(256), 0, stream, lat, layout, L, k0, k1, t, out, nsum != nullptr);
  return hipGetLastError();
}

hipError_t launch_sum_words(const unsigned long long* in, size_t n, unsigned long long* out, hipStream_t stream) {
  hipLaunchKernelGGL(sum_words, dim3(1), dim3(256), 0, stream, in, n, out);
  return hipGetLastError();
}

hipError_t launch_copy_bytes(const void* in, void* out, size_t n, hipStream_t stream) {
  hipLaunchKernelGGL(copy_bytes, dim3(grid_for((n + 15) / 16, 256)), dim3(256), 0, stream,
                     static_cast<const uint8_t*>(in), static_cast<uint8_t*>(out), n);
  return hipGetLastError();
}

size_t place_cap(size_t n) { return n / (kPlaceBins / 2) + 1024; }
// key and index of every listed site, the list's length and the key counts
size_t place_bytes(size_t n) { return place_cap(n) * 12 + (kPlaceBins + 2) * sizeof(unsigned); }

hipError_t launch_place(int L, int H, int layout, size_t n1, uint32_t k0, uint32_t k1, void* lat, void* scratch,
                        uint32_t* length, hipStream_t stream) {
  const uint32_t n = (uint32_t)L * (uint32_t)H;
  PlaceList list;
  list.cap = (uint32_t)place_cap(n);
  list.key = static_cast<uint64_t*>(scratch);
  unsigned* hist = reinterpret_cast<unsigned*>(list.key + list.cap);
  list.count = hist + kPlaceBins;
  list.idx = list.count + 2;
  hipError_t e = hipMemsetAsync(hist, 0, (kPlaceBins + 1) * sizeof(unsigned), stream);
  if (e != hipSuccess) return e;
  const int grid = std::min(grid_for(n, 1024), 512);
  hipLaunchKernelGGL(place_count_keys, dim3(grid), dim3(1024), 0, stream, (uint32_t)L, n, k0, k1, hist);
  hipLaunchKernelGGL(place_mark, dim3(grid), dim3(1024), 0, stream, (uint32_t)L, n, layout, (uint32_t)n1, k0, k1, hist,
                     lat, list);
  hipLaunchKernelGGL(place_select, dim3(1), dim3(1024), 0, stream, layout, (uint32_t)n1, hist, lat, list, length);
  return hipGetLastError();
}

size_t ccl_tiles(int L, int H) {
  return (size_t)((L + kTile - 1) / kTile) * (size_t)((H + kTile - 1) / kTile);
}
size_t ccl_cluster_words(int L, int H) { return ((size_t)L * (size_t)H + 1) / 2; }
size_t ccl_border_words(int L, int H) { return ccl_tiles(L, H) * (256 + 1); }

namespace {
// Workgroups of each pass over n tiles: one per tile up to 4096; a thread per
// edge site; and up to 128 histograms, each of which clears and flushes 4096 bins.
struct CclGrid {
  unsigned tile, border, sizes, hist;
};
CclGrid ccl_grid(size_t n, bool triangular) {
  return CclGrid{(unsigned)std::min<size_t>(n, 4096), (unsigned)std::min<size_t>((n * (triangular ? 192 : 128) + 255) / 256, 4096),
                 (unsigned)std::min<size_t>(n, 4096), (unsigned)std::min<size_t>(n, 128)};
}
}  // namespace

hipError_t launch_ccl(const void* lat, int layout, int L, int H, int species, const CclBuffers& b, bool triangular,
                      hipStream_t stream) {
  const CclGrid n = ccl_grid(ccl_tiles(L, H), triangular);
  const CclShape g{lat, layout, L, H};
  // Up to a tile per CU, 16 wavefronts per tile: a wavefront's rows come one after
  // another (us of the first pass with 4 and with 16: 64^2 17.5 and 8.4, 400^2 22.2
  // and 11.9); with more tiles the four that share a CU fill it.
  const bool wide = n.tile <= 256;
  if (triangular) {
    if (wide) hipLaunchKernelGGL((ccl_tile<true, 16>), dim3(n.tile), dim3(1024), 0, stream, g, species, b);
    else hipLaunchKernelGGL((ccl_tile<true, 4>), dim3(n.tile), dim3(256), 0, stream, g, species, b);
    hipLaunchKernelGGL(ccl_border<true>, dim3(n.border), dim3(256), 0, stream, g, b);
  } else {
    if (wide) hipLaunchKernelGGL((ccl_tile<false, 16>), dim3(n.tile), dim3(1024), 0, stream, g, species, b);
    else hipLaunchKernelGGL((ccl_tile<false, 4>), dim3(n.tile), dim3(256), 0, stream, g, species, b);
    hipLaunchKernelGGL(ccl_border<false>, dim3(n.border), dim3(256), 0, stream, g, b);
  }
  hipLaunchKernelGGL(ccl_sizes, dim3(n.sizes), dim3(256), 0, stream, g, b);
  hipLaunchKernelGGL(ccl_hist, dim3(n.hist), dim3(256), 0, stream, g, b);
  return hipGetLastError();
}

hipError_t launch_ccl_many(const CclRep* d_reps, int nreps, int max_L, int species, uint32_t* stage, uint32_t words,
                           hipStream_t stream) {
  if (nreps <= 0) return hipSuccess;
  // every pass strides over its lattice's tiles; workgroups past a smaller
  // replica's tiles exit at once
  const CclGrid n = ccl_grid(ccl_tiles(max_L, max_L), false);
  const unsigned reps = (unsigned)nreps;
  hipLaunchKernelGGL(ccl_tile_many, dim3(n.tile, reps), dim3(256), 0, stream, d_reps, species);
  hipLaunchKernelGGL(ccl_border_many, dim3(n.border, reps), dim3(256), 0, stream, d_reps);
  hipLaunchKernelGGL(ccl_sizes_many, dim3(n.sizes, reps), dim3(256), 0, stream, d_reps);
  hipLaunchKernelGGL(ccl_hist_many, dim3(n.hist, reps), dim3(256), 0, stream, d_reps);
  hipLaunchKernelGGL(ccl_gather_many, dim3(8, reps), dim3(256), 0, stream, d_reps, stage, words);
  return hipGetLastError();
}

hipError_t launch_pack(const uint8_t* in, uint32_t* out, int L, hipStream_t stream) {
  hipLaunchKernelGGL(pack_bits, dim3(grid_for((size_t)L * (L >> 5), 256)), dim3(256), 0, stream, in, out, L);
  return hipGetLastError();
}

hipError_t launch_unpack(const uint32_t* in, uint8_t* out, int L, hipStream_t stream) {
  hipLaunchKernelGGL(unpack_bits, dim3(grid_for((size_t)L * (L >> 4), 256)), dim3(256), 0, stream, in, out, L);
  return hipGetLastError();
}

hipError_t launch_fill_segregated(void* lat, int layout, int L, int H, uint64_t n1, hipStream_t stream) {
  hipLaunchKernelGGL(fill_segregated, dim3(grid_for((size_t)L * H, 256)), dim3(256), 0, stream, lat, layout, L, H,
                     n1);
  return hipGetLastError();
}

}  // namespace kk
