// kk_kernels.hpp -- launch parameter blocks and host-side launchers of the
// libkk HIP kernels (internal to the library; the public API is kk.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kk_common.hpp"

namespace kk {

constexpr int kLayoutInt8 = 1;  // one byte (0/1) per site, row-major
constexpr int kLayoutBits = 2;  // one bit per site, L/32 words per row, bit b of word g = site 32g + b

struct SweepParams {
  const void* src;
  void* dst;
  unsigned long long* accepted;  // one running sum per tile (grid index)
  int L, wpr;                // side; words per row of the bit-packed layout
  int tww, th;               // interior words / rows per tile
  int hx, hy;                // halo words / rows on each side (1/16, or 0/0 for the cyclic tile)
  int tiles_x;
  int C, R;                  // LDS words per row, rows (tile + halo)
  int row0, npairs, nunits;  // first computed LDS row, computed row pairs, units = pairs * C
  int nsweeps;               // sweeps in this launch
  int layout;                // kLayoutInt8 or kLayoutBits (read by the batch kernels)
  uint32_t k0, k1;           // Philox key (seed)
  uint64_t t0;               // first sweep index
  Accept acc;
};

hipError_t launch_sweep(const SweepParams& p, int layout, bool cyclic, int ku, int threads, hipStream_t stream);
// Sweeps that one launch_sweep takes at most (p.nsweeps).
int sweeps_per_launch(const SweepParams& p, bool cyclic, int ku);

// Batch kernels.  Tiled replicas: one workgroup per (replica, tile) job and one
// launch per sweep, or per two, of the run.  A replica runs p.nsweeps sweeps from
// p.t0, ping-ponging between p.src (its lattice at the start) and p.dst.
// Resident replicas (L % 32 == 0, 2 <= L/32 <= kResidentMaxC): one workgroup per
// replica with the whole lattice in LDS, kBatchChunk sweeps per launch.
constexpr int kBatchMaxTww = 16, kBatchTh = 128;
// Tiled replicas run in 512-thread workgroups (more with two sweeps side by side), ku (1 or 2) units per thread,
// in tiles 8 or 16 words wide: a tile of tww words by th rows fits when its
// (th + 28) / 2 computed row pairs times tww + 2 words stay within ku * 512
// units.
constexpr int kBatchTileThreads = 512;
constexpr bool batch_tile_fits(int tww, int th, int ku = 2) {
  return (tww == 8 || tww == 16) && (ku == 1 || ku == 2) && th >= 2 && th <= kBatchTh &&
         ((th + 28) / 2) * (tww + 2) <= ku * kBatchTileThreads;
}
struct BatchTileJob {
  int rep, tile;
};
// How the tiles of a batch are launched.
struct BatchTilePlan {
  int sweeps;         // per launch, 1 or 2
  bool side_by_side;  // with two: both sweeps' units at once, else in turn
  int ku, threads;
  int max_th;         // rows of the tallest tile
};
int batch_tile_threads(int tww, int th);   // side by side, one unit per thread
bool batch_tile_in_turn(int tww, int th);  // fits 512 threads of two units
// Sweep s of the run, or s and s + 1; orders[rep * kBatchChunk + s % kBatchChunk] is replica
// rep's class order of that sweep (launch_batch_orders, once per kBatchChunk sweeps).
hipError_t launch_batch_tiles(const SweepParams* reps, const BatchTileJob* jobs, int njobs, const uint32_t* orders,
                              unsigned s, const BatchTilePlan& plan, hipStream_t stream);
hipError_t launch_batch_orders(const SweepParams* reps, int nreps, unsigned s, uint32_t* orders, hipStream_t stream);
// small: the 768-thread kernel for replicas of at most kResidentSmallMaxC words
// per row.  A launch runs up to kBatchChunk sweeps from sweep s of the run.
hipError_t launch_batch_resident(const SweepParams* reps, const int* ids, int n, size_t lds_bytes, bool small,
                                 unsigned s, hipStream_t stream);
constexpr int kBatchChunk = 256;
constexpr int kResidentMaxC = 9;
constexpr int kResidentSmallMaxC = 4, kResidentSmallThreads = 768, kResidentThreads = 1024;
size_t batch_resident_lds_bytes(int L);

// N_AB (unlike nearest-neighbour bonds) added into *out.
// nsum NULL: the sum is added to *out.  Else each of the *nsum workgroups (at most
// kMaxSums) writes its own word of out, host memory that the caller adds up.
constexpr int kMaxSums = 2048;
hipError_t launch_energy(const void* lat, int layout, int L, unsigned long long* out, int* nsum, hipStream_t stream);

// Count of sites whose randomly drawn neighbour has the same type, added into *out.
hipError_t launch_similar_sampled(const void* lat, int layout, int L, uint32_t k0, uint32_t k1, uint64_t t,
                                 unsigned long long* out, int* nsum, hipStream_t stream);

// Initial placement: n1 of the L x H sites (0 < n1 < L H).  scratch: place_bytes.
// *length (device or pinned memory) becomes the number of sites the selection
// had to order; beyond place_cap the placement is incomplete.
size_t place_cap(size_t n);
size_t place_bytes(size_t n);
hipError_t launch_place(int L, int H, int layout, size_t n1, uint32_t k0, uint32_t k1, void* lat, void* scratch,
                        uint32_t* length, hipStream_t stream);

// Connected components of one species (4-neighbour, periodic) and their size histogram.
struct CclBuffers {
  uint32_t* parent;     // ccl_cluster_words
  uint32_t* size;       // ccl_cluster_words
  uint32_t* border;     // ccl_border_words: 256 edge labels per tile,
  uint32_t* ncl;        // then the number of clusters per tile
  unsigned* hist;       // small-size histogram, kSmallSizes entries
  uint32_t* big;        // sizes >= kSmallSizes, appended
  unsigned* big_count;  // number of appended sizes
  unsigned big_cap;
};
constexpr int kSmallSizes = 4096;
size_t ccl_tiles(int L, int H);
size_t ccl_cluster_words(int L, int H);
size_t ccl_border_words(int L, int H);
// triangular: six neighbours under helical boundaries (the int8 ring of kk_tri.hip).
hipError_t launch_ccl(const void* lat, int layout, int L, int H, int species, const CclBuffers& b, bool triangular,
                      hipStream_t stream);

// Segregated start: sites 0 .. n1-1 (index y*L + x) set to 1, the rest 0.
hipError_t launch_fill_segregated(void* lat, int layout, int L, int H, uint64_t n1, hipStream_t stream);

// int8 <-> bit-packed conversion on the device (bit-packed needs L % 32 == 0).
hipError_t launch_pack(const uint8_t* in, uint32_t* out, int L, hipStream_t stream);
hipError_t launch_sum_words(const unsigned long long* in, size_t n, unsigned long long* out, hipStream_t stream);
hipError_t launch_copy_bytes(const void* in, void* out, size_t n, hipStream_t stream);  // both 16-byte aligned
hipError_t launch_unpack(const uint32_t* in, uint8_t* out, int L, hipStream_t stream);

}  // namespace kk
