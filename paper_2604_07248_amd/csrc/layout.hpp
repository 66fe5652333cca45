// Launch geometry shared by the kernel files: elements per thread, rows per
// row-pass block, columns per column-pass strip, XCD-aware block order.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace turpy {

constexpr int kE = 16;  // elements per thread in every transform

template <int N>
constexpr int row_groups() {  // rows per block of the row kernels
  return (256 / (N / kE)) < N ? (256 / (N / kE)) : N;
}
template <int N>
constexpr int row_block() { return row_groups<N>() * (N / kE); }
// Columns per block of the column pass, of the screen synthesis and of the
// synthesis with the AR step fused into it, when no tuned choice is set.  The
// widest strip that pays on a full chip (times at R N^2 = 2^26 pixels, us for
// 4 / 8 / 16 columns, one launch bracketed by events):
//   column pass  n = 128 27.7 / 21.7 / 16.4 (R = 256); 512: 263 / 201 / 190;
//                1024: 268 / 220 / 277
//   synthesis    n = 512 86.4 / 85.9 / 87.2; 1024: 85.8 / 89.5 / 118
//   AR step      n = 512 226 / 180 / 151; 1024: 240 / 205 / 177 (a strip row of
//                16 columns is a whole line, written back past the cache)
// A launch over few planes takes narrower strips until it has a block for
// every CU (n = 512, 4 planes: 16 columns 15.4 us, 8 columns 13.7; n = 1024,
// one plane of the AR step: 23.0 us for 16 columns, 15.9 for 4), as long as
// a block keeps a whole wave.  A single realization's synthesis launches half
// the blocks and takes the same line: from n = 128 that is the best width of
// the three or one within 4 % (n = 512, four screens, us for 4 / 8 / 16 columns
// 12.9 / 11.3 / 14.1, where counting its own blocks would take 4).
constexpr int kFillBlocks = 256;
constexpr int fill_width(int n, int64_t planes, int widest) {
  int k = widest;
  while (k > 4 && (n / k) * planes < kFillBlocks && (k / 2) * (n / kE) >= 64) k /= 2;
  return k;
}
constexpr int widest_col(int n) { return n >= 1024 ? 8 : (n >= 128 ? 16 : 8); }
constexpr int widest_synth(int n) { return n >= 1024 ? 4 : (n >= 512 ? 8 : widest_col(n)); }
constexpr int widest_ar(int n) { return n >= 2048 ? 8 : (n >= 128 ? 16 : 8); }
// At N = 2048 one block of 8 columns takes a CU's whole LDS, and its waves wait
// at the same barriers; two lean blocks of 4 columns (col_lean) overlap.  They
// pay from three planes on (us for 8 / 4 columns: one plane 22.9 / 25.6, two
// 40.3 / 39.8, three 57.0 / 54.6, eight 145.5 / 140.2; a serving mix, one plane
// a launch beside other streams', 24.7 / 25.5 ms).
constexpr bool col_lean(int n, int k) { return n == 2048 && k == 4; }
constexpr int default_col_width(int n, int64_t planes) {
  return n == 2048 && planes >= 3 ? 4 : fill_width(n, planes, widest_col(n));
}
constexpr int default_synth_width(int n, int64_t planes) { return fill_width(n, planes, widest_synth(n)); }
constexpr int default_ar_width(int n, int64_t planes) { return fill_width(n, planes, widest_ar(n)); }
// Grouped launches and the receiver, whose members together fill the chip.
template <int N>
constexpr int col_width() { return widest_col(N); }
template <int N>
constexpr int col_block() { return col_width<N>() * (N / kE); }
template <int N>
constexpr int synth_width() { return widest_synth(N); }

// A strip of K columns is built for grid size N when its block (K N / 16
// threads) stays within 1024 threads and its LDS (K N complex words beside
// the N-entry twiddle and chirp tables) within the 160 KiB of a CU.  At
// N = 2048 this excludes 16 columns.
template <int N, int K>
constexpr bool strip_fits() {
  return K <= N && K * (N / kE) <= 1024 && (static_cast<long>(K) * N + 2L * N) * 8 <= 160L * 1024;
}
constexpr bool strip_fits_rt(int n, int k) {
  return (k == 4 || k == 8 || k == 16) && k <= n && k * (n / kE) <= 1024 &&
         (static_cast<long>(k) * n + 2L * n) * 8 <= 160L * 1024;
}

// Ensemble moments: the R realizations are summed in C contiguous chunks,
// chunk c holding realizations [c R / C, (c + 1) R / C), and the compensated
// sums of the non-empty chunks are joined into the stored ones in chunk order.
// C = 256 / (N / 16) clamped to [4, 64] depends on N alone: a block of the
// fused final row pass (one row, C chunks of N / 16 threads) then has 256
// threads for N = 64..1024.
constexpr int moment_chunks(int n) {
  return (256 / (n / kE)) < 4 ? 4 : ((256 / (n / kE)) > 64 ? 64 : 256 / (n / kE));
}

// Row-pair pass: each half of a block (whole waves for N >= 64) carries one
// realization of a pair over `pair_rows` rows.
template <int N>
constexpr int pair_rows() {
  return (128 / (N / kE)) < 1 ? 1 : ((128 / (N / kE)) < N ? (128 / (N / kE)) : N);
}
template <int N>
constexpr int pair_block() { return 2 * pair_rows<N>() * (N / kE); }

// Row pass with one worker per transform: a worker is one wave over
// `trio_rows` rows.
constexpr bool trio_fits(int n) { return n >= 64 && n <= 1024; }
// It runs up to 2^20 pixels of scratch planes in a launch (N/2 rows apiece for
// a single realization), where its shorter chain beats the busier blocks of the
// other schedules (us with it and without, forward, events around each launch:
// n = 256, 32 realizations 16.6 / 19.6, 64 22.6 / 21.8; n = 512, 8 realizations
// 18.4 / 21.7, 16 26.2 / 24.4; n = 1024, 2 realizations 20.7 / 22.1, 4 30.0 /
// 25.6; the adjoint's lines lie at the same sizes or one step above).
constexpr bool trio_takes(int n, int64_t planes, bool solo) {
  return trio_fits(n) && planes * (solo ? n / 2 : n) * n <= (int64_t(1) << 20);
}
template <int N>
constexpr int trio_rows() { return 64 / (N / kE); }
template <int N>
constexpr int trio_block() { return 3 * trio_rows<N>() * (N / kE); }

// Relay row pass: two workers of `relay_rows` rows each per block, over two
// row groups (2 relay_rows <= N).  Used where a worker is whole waves.
template <int N>
constexpr int relay_rows() { return pair_rows<N>() < N / 2 ? pair_rows<N>() : N / 2; }
template <int N>
constexpr int relay_block() { return 2 * relay_rows<N>() * (N / kE); }
template <int N>
constexpr bool relay_fits() { return (relay_rows<N>() * (N / kE)) % 64 == 0; }

// Place of subharmonic phasor i in its level's table: the phasors of a row
// pass's thread, n / 16 apart, lie in pairs, so that one load brings two.  The
// row passes wait on their loads' issue: 24 loads for three levels instead of
// 48 beside the 80 of a row pair took 256 realizations at N = 512 with 10
// screens from 6.18 to 6.13 ms, 3 at N = 2048 with 12 from 2.09 to 2.06 ms.
__host__ __device__ constexpr int sh_slot(int n, int i) {
  const int t = n / kE;
  return ((i / t / 2) * t + i % t) * 2 + i / t % 2;
}

// Grids on which a single realization's real screen is synthesised on its own
// (SynthArgs::solo): the row passes' halves must be whole waves on N/2 rows.
constexpr bool solo_fits(int n) { return n >= 64; }

// Blocks of `threads` for a pass over a plane of up to 2^32 pixels: one pixel a
// thread while a launch allows that many threads in x (fewer than 2^32).
constexpr uint32_t plane_blocks(int64_t pixels, int threads) {
  const int64_t b = (pixels + threads - 1) / threads, most = (int64_t(1) << 32) / threads - 1;
  return static_cast<uint32_t>(b < most ? b : most);
}
static_assert(plane_blocks(int64_t(1) << 32, 256) * int64_t(256) < int64_t(1) << 32, "one launch covers 2^32 pixels");

// Spread a 1-D block index so that consecutive logical tiles land on the same
// XCD (blocks are dealt round-robin over the 8 XCDs, each with its own L2).
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t nb) {
  if (nb % 8u != 0u) return b;
  return (b % 8u) * (nb / 8u) + b / 8u;
}

// Strip and plane of block b of a column pass over R planes of `strips`
// strips: plane-major, the planes from last to first, each XCD taking one
// contiguous eighth of every plane's strips (neighbouring strips, which share
// cache lines, stay on one XCD's L2).  The row passes run the planes from
// first to last, so a column pass starts on the planes the row pass before it
// wrote last, and the row pass after it on the planes it wrote last.  With a
// strip count that is not a multiple of 8: xcd_remap over (plane, strip).
__device__ __forceinline__ void col_tile(uint32_t b, uint32_t nb, int strips, int64_t R, int* strip, int64_t* r) {
  if (strips % 8 == 0) {
    const uint32_t x = b % 8u, i = b / 8u;
    const int per = strips / 8;
    *strip = static_cast<int>(x) * per + static_cast<int>(i % static_cast<uint32_t>(per));
    *r = R - 1 - static_cast<int64_t>(i / static_cast<uint32_t>(per));
  } else {
    const uint32_t t = xcd_remap(b, nb);
    *strip = static_cast<int>(t % static_cast<uint32_t>(strips));
    *r = t / static_cast<uint32_t>(strips);
  }
}

}  // namespace turpy
