// kk_tri.hpp -- launchers of the triangular-lattice kernels (kk_tri.hip, kk_hex.hip, kk_ring.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace kk {

// Triangular lattice, helical boundaries (kk_tri.hip): H rows of L sites on
// one ring of N = L*H.  Conflict-free classes: one launch per phase.  The
// literal MPKK variant: one launch per iteration, ping-pong buffers.
constexpr int kTriPartials = 64;  // accepted-move sums, indexed by workgroup % kTriPartials
struct TriAccept {
  uint64_t T[11];  // U < T[n] accepts, n = unlike neighbours of the pair (each excluding the other)
};
hipError_t launch_tri_phase(uint8_t* lat, int L, int H, uint32_t k0, uint32_t k1, uint64_t t, int p,
                            const TriAccept& acc, unsigned long long* partials, hipStream_t stream);
// What the bit-plane kernels (kk_hex.hip) need of the table: only n = 2, 3, 4
// (omega > 0) or 6, 7, 8 (omega < 0) can be rejected.
struct HexAccept {
  uint32_t thr[3];   // U < thr accepts
  uint32_t all[3];   // 0xFFFFFFFF: every U is accepted
  uint32_t negmask;  // 0xFFFFFFFF: the restricted counts are 6, 7, 8
};
__host__ __device__ inline HexAccept hex_accept(const TriAccept& acc) {
  HexAccept a{};
  const bool neg = acc.T[2] >= ((uint64_t)1 << 32);  // omega <= 0 (n = 2 is always accepted)
  a.negmask = neg ? 0xFFFFFFFFu : 0u;
  for (int j = 0; j < 3; ++j) {
    const uint64_t T = acc.T[neg ? 6 + j : 2 + j];
    a.all[j] = T >= ((uint64_t)1 << 32) ? 0xFFFFFFFFu : 0u;
    a.thr[j] = (uint32_t)(a.all[j] ? 0xFFFFFFFFu : T);
  }
  return a;
}
// Whole-sweep tiles (16 phases per launch on an LDS window, `in` -> `out`).
// Which tiles are taken: a byte per site of the window, rows of an odd number
// of words, next to 16 KiB, in one workgroup's LDS.
constexpr uint32_t kTriHalo = 33;  // 2 cells per phase, plus 1 for the first phase's reads
__host__ __device__ inline uint32_t tri_window_stride(uint32_t TW) {
  const uint32_t s = (TW + 2 * kTriHalo + 3u) & ~3u;  // whole words, an odd number of them
  return ((s >> 2) & 1u) ? s : s + 4u;
}
// The 16 KiB: they belong to the rule of which tiles are accepted.
constexpr uint32_t kTriQueue = 128, kTriQueueBytes = 16u * kTriQueue * 8u;
__host__ __device__ inline size_t tri_window_area(uint32_t TW, uint32_t TR) {
  return ((size_t)tri_window_stride(TW) * (TR + 2 * kTriHalo) + 7u) & ~(size_t)7u;
}
__host__ __device__ inline size_t tri_window_bytes(uint32_t TW, uint32_t TR) {
  return tri_window_area(TW, TR) + kTriQueueBytes;
}
// The bit-plane window of the class schedule: kHexLeft columns before the tile
// (a multiple of 4 not below kTriHalo, so that rows start on whole words of
// the ring), NJ groups of 16 columns in all, one bit per group in each of a
// row's 16 class words; after the rows, six random words per (class, row).
constexpr uint32_t kHexLeft = 36;
constexpr int kHexRow16 = 17;  // words per row: 16 classes and one of padding
constexpr uint32_t kHexMaxCols = 440, kHexMaxRows = 288;
__host__ __device__ inline int hex_groups(uint32_t TW) { return (int)((kHexLeft + TW + kTriHalo + 15u) / 16u); }
__host__ __device__ inline int hex_spin_words(int WR, int row) { return (WR * row + 3) & ~3; }
inline size_t hex_lds_bytes(uint32_t TR) {
  const int WR = (int)TR + 2 * (int)kTriHalo;
  return ((size_t)hex_spin_words(WR, kHexRow16) + (size_t)16 * WR * 6) * 4;
}
// The tile a launch works with: the columns a multiple of 4, and a tile beyond
// 32 groups or beyond the LDS in equal parts.
struct HexTile {
  uint32_t tw, tr;
};
inline HexTile hex_tile(int TW, int TR) {
  const uint32_t nx = ((uint32_t)TW + kHexMaxCols - 1) / kHexMaxCols, ny = ((uint32_t)TR + kHexMaxRows - 1) / kHexMaxRows;
  return HexTile{((((uint32_t)TW + nx - 1) / nx) + 3u) & ~3u, ((uint32_t)TR + ny - 1) / ny};
}
inline bool tri_tile_fits(int L, int H, int TW, int TR) {
  return TW >= 16 && TR >= 16 && TW + 2 * (int)kTriHalo <= L && TR + 2 * (int)kTriHalo <= H &&
         tri_window_bytes((uint32_t)TW, (uint32_t)TR) <= 160u * 1024u - 1024u;
}
// The whole ring in one workgroup's LDS (kk_ring.hip): up to a byte per site.
constexpr size_t kTriResidentMaxBytes = 160u * 1024u - 1024u;
inline bool tri_resident_fits(int L, int H) {
  return (size_t)L * (size_t)H <= kTriResidentMaxBytes;
}
// The segments of kk_ring.hip's bit planes (0: the ring has none and is held a
// byte per site): B equal parts of 16 W sites, B <= 28 bits of a word, at least
// 2L sites each, W such that two buffers of draws fit the LDS.  The fewest that
// leave one wave per class (more words, hence more lanes for the draws), else
// the most.
constexpr int kRingMaxBits = 28, kRingMaxWords = 194;
constexpr int kRingStride = 196;  // words per class, fixed so that a class's place is part of an instruction
// Lane w of the phase waves works at word w of a class, also past the class's
// last word: such a lane decides nothing and flips no bit, but it reads and xors
// too, at a word that no other lane of its wave has (xors of one wave to one word
// run one after another).  With 193 or 194 words there are four waves, whose last
// lanes reach into the next class, and past the last class into spare words.
constexpr int kRingLanes = (kRingMaxWords + 63) / 64 * 64;
constexpr int kRingWords = 16 * kRingStride + (kRingLanes - kRingStride);  // of LDS before the draws; an even number
inline uint32_t ring_segments(int L, int H) {
  const int M = L * H / 16;
  uint32_t best = 0;
  for (int B = 3; B <= kRingMaxBits && 2 * B <= H; ++B) {
    if (M % B != 0 || M / B > kRingMaxWords) continue;
    best = (uint32_t)B;
    if (M / B <= 64) break;
  }
  return best;
}
// LDS of a whole ring: words, two buffers of draws and 128 class orders; or bytes.
inline size_t ring_lds_bytes(int L, int H) {
  const uint32_t B = ring_segments(L, H);
  const size_t N = (size_t)L * (size_t)H;
  return B ? 4u * kRingWords + 12u * 4u * (N / B) + 1024u : N;
}
struct TriResidentRep {
  uint8_t* lat;  // the current buffer, updated in place
  uint32_t L, H, sweeps;
  uint32_t seg;  // ring_segments(L, H)
  uint32_t k0, k1;
  uint64_t t0;
  TriAccept acc;
  unsigned long long* partials;
};
// Workgroup b runs replica b (reps[b].sweeps sweeps); lds_bytes = the largest
// ring_lds_bytes.
hipError_t launch_tri_resident(const TriResidentRep* reps, uint32_t nreps, size_t lds_bytes, hipStream_t stream);
// One replica, its descriptor passed by value.
hipError_t launch_tri_resident_one(const TriResidentRep& rep, size_t lds_bytes, hipStream_t stream);
constexpr uint64_t kTriResidentChunk = 1024;  // sweeps per launch of a single handle

// One replica of a batched launch of whole-sweep tiles.  Sweep k of a run reads
// lat[cur ^ (k & 1)] and writes the other buffer with sweep counter t0 + k.
struct TriBatchRep {
  uint8_t* lat[2];
  uint32_t L, H, TW, TR, ntx, cur;  // TW x TR: a hex_tile
  uint32_t k0, k1;
  uint64_t t0;
  HexAccept acc;
  unsigned long long* partials;  // kTriPartials sums of the replica
};
// jobs[b] = (replica, tile) for workgroup b; lds_bytes = the largest window.
hipError_t launch_tri_tile_sweep_batch(const TriBatchRep* reps, const uint2* jobs, uint32_t njobs, uint32_t k,
                                       size_t lds_bytes, hipStream_t stream);
hipError_t launch_tri_tile_sweep(const uint8_t* in, uint8_t* out, int L, int H, int TW, int TR, uint32_t k0,
                                uint32_t k1, uint64_t t, const TriAccept& acc, unsigned long long* partials,
                                hipStream_t stream);
// Whole-step MPKK tiles (7 iterations per launch on an LDS window, `in` -> `out`).
constexpr uint32_t kMpkkHalo = 21;  // 3 cells per iteration
__host__ __device__ inline uint32_t mpkk_window_stride(uint32_t TW) {
  const uint32_t s = (TW + 2 * kMpkkHalo + 3u) & ~3u;  // whole words, an odd number of them
  return ((s >> 2) & 1u) ? s : s + 4u;
}
// Which tiles are taken, as for the class schedule.
__host__ __device__ inline size_t mpkk_window_area(uint32_t TW, uint32_t TR) {
  return ((size_t)mpkk_window_stride(TW) * (TR + 2 * kMpkkHalo) + 15u) & ~(size_t)15u;
}
__host__ __device__ inline size_t mpkk_window_bytes(uint32_t TW, uint32_t TR) {
  return mpkk_window_area(TW, TR) + kTriQueueBytes;
}
// The bit-plane window of a step: kMpkkHalo columns before the tile, groups of
// 14 columns (one group of draws before the first, so at most 31), six random
// words per (iteration, even or odd domains, row).
constexpr int kHexRow14 = 15;
constexpr uint32_t kHexMpkkMaxCols = 14 * 31 - 2 * kMpkkHalo, kHexMpkkMaxRows = 368;
__host__ __device__ inline int hex_mpkk_groups(uint32_t TW) { return (int)((TW + 2 * kMpkkHalo + 13u) / 14u); }
inline size_t hex_mpkk_lds_bytes(uint32_t TR) {
  const int WR = (int)TR + 2 * (int)kMpkkHalo;
  return ((size_t)hex_spin_words(WR, kHexRow14) + (size_t)14 * WR * 6) * 4;
}
inline HexTile hex_mpkk_tile(int TW, int TR) {
  const uint32_t nx = ((uint32_t)TW + kHexMpkkMaxCols - 1) / kHexMpkkMaxCols;
  const uint32_t ny = ((uint32_t)TR + kHexMpkkMaxRows - 1) / kHexMpkkMaxRows;
  return HexTile{((uint32_t)TW + nx - 1) / nx, ((uint32_t)TR + ny - 1) / ny};
}
inline bool mpkk_tile_fits(int L, int H, int TW, int TR) {
  return TW >= 16 && TR >= 16 && TW + 2 * (int)kMpkkHalo <= L && TR + 2 * (int)kMpkkHalo <= H &&
         mpkk_window_bytes((uint32_t)TW, (uint32_t)TR) <= 160u * 1024u - 1024u;
}
hipError_t launch_mpkk_tile_step(const uint8_t* in, uint8_t* out, int L, int H, int TW, int TR, uint32_t k0,
                                 uint32_t k1, uint64_t t, const TriAccept& acc, unsigned long long* partials,
                                 hipStream_t stream);
hipError_t launch_mpkk_iteration(const uint8_t* in, uint8_t* out, int L, int H, uint32_t k0, uint32_t k1, uint64_t t,
                                 int j, const TriAccept& acc, unsigned long long* partials, hipStream_t stream);
// Sums as launch_energy's (kk_kernels.hpp).
hipError_t launch_tri_energy(const uint8_t* lat, int L, int H, unsigned long long* out, int* nsum, hipStream_t stream);
hipError_t launch_tri_similar(const uint8_t* lat, int L, int H, uint32_t k0, uint32_t k1, uint64_t t,
                              unsigned long long* out, int* nsum, hipStream_t stream);

}  // namespace kk
