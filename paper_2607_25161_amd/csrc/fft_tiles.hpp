// Tiles of the transform passes: the sides with two-step transforms, the rules of the run-time passes
// and the choice between them.
#pragma once
#include <cstddef>

namespace fsd {

// ---- sides with a two-step transform ----------------------------------------------------------
// A side has one when it is a product of two factors RA <= RB <= 16 (a thread's registers) that have a
// register transform: 2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16.  Of its products the most even one counts.
// (125, 162, 200, 216, 243 and 250 have none and keep the run-time passes.)
constexpr bool reg_factor(int f) {
  return f == 2 || f == 3 || f == 4 || f == 5 || f == 6 || f == 8 || f == 9 || f == 10 || f == 12 || f == 15 || f == 16;
}
constexpr int split_low(int N) {  // RA, or 0
  int best = 0;
  for (int f = 2; f * f <= N; ++f)
    if (N % f == 0 && reg_factor(f) && reg_factor(N / f)) best = f;
  return best;
}
// lines of a z or y pass per workgroup: the most that divide N^2 and that 256 threads (RB a line) transform in
// one go
constexpr int split_most_lines(int N) {
  int best = 1;
  for (int b = 1; b * (N / split_low(N)) <= 256; ++b)
    if (N * N % b == 0) best = b;
  return best;
}

// BL: lines of a z or y pass per workgroup in FP32; FP64 takes half where that leaves an even number (side
// 108, 18 lines: 35 us for the 3D transform, with 9 43).  GP: row pairs of an x+Green workgroup, 6 lines each.
template <int N>
struct Split {  // transforms of their own only
  static constexpr int RA = split_low(N), RB = N / RA, BL = split_most_lines(N), GP = 0;
};
#define FSD_SPLIT(N_, L_, G_)                                                             \
  template <>                                                                             \
  struct Split<N_> {                                                                      \
    static constexpr int RA = split_low(N_), RB = N_ / RA, BL = L_, GP = G_;               \
  };
// Sides of the wave-space passes: the multiples of 8, which the grid rule takes.  Their lines are powers of
// two (24 on side 72), so that a run of lines is whole cache lines.
FSD_SPLIT(8, 64, 10)
FSD_SPLIT(16, 64, 10)
FSD_SPLIT(24, 32, 7)
FSD_SPLIT(32, 32, 5)
FSD_SPLIT(40, 32, 5)
FSD_SPLIT(48, 32, 5)
FSD_SPLIT(64, 32, 4)
FSD_SPLIT(72, 24, 3)
FSD_SPLIT(80, 16, 3)
FSD_SPLIT(96, 16, 2)
FSD_SPLIT(120, 16, 2)
FSD_SPLIT(128, 16, 2)
FSD_SPLIT(144, 16, 1)
FSD_SPLIT(160, 16, 1)
FSD_SPLIT(192, 16, 1)
FSD_SPLIT(240, 16, 1)
FSD_SPLIT(256, 16, 1)
#undef FSD_SPLIT
#define FSD_WAVE_SIDES(X) \
  X(8) X(16) X(24) X(32) X(40) X(48) X(64) X(72) X(80) X(96) X(120) X(128) X(144) X(160) X(192) X(240) X(256)
#define FSD_OTHER_SIDES(X)                                                                                      \
  X(4) X(6) X(9) X(10) X(12) X(15) X(18) X(20) X(25) X(27) X(30) X(36) X(45) X(50) X(54) X(60) X(75) X(81) X(90) \
  X(100) X(108) X(135) X(150) X(180) X(225)
// the two lists hold every side that splits
constexpr bool is_listed(int N) {
  switch (N) {
#define X(N_) case N_:
    FSD_WAVE_SIDES(X)
    FSD_OTHER_SIDES(X)
#undef X
    return true;
  }
  return false;
}
constexpr bool all_listed() {
  for (int N = 1; N <= 512; ++N)
    if ((split_low(N) > 0) != is_listed(N)) return false;
  return true;
}
static_assert(all_listed(), "a side of the rule is missing, or one too many");

// lines of a z or y pass per workgroup, values of rbytes
template <int N>
constexpr int split_lines(size_t rbytes) {
  return rbytes == 8 && Split<N>::BL % 4 == 0 ? Split<N>::BL / 2 : Split<N>::BL;
}

// of a two-step wave-space pass: lines (0: the side has none), row pairs of x+Green
inline int two_step_lines(int N, int rbytes) {
  switch (N) {
#define X(N_) \
  case N_: return split_lines<N_>(rbytes);
    FSD_WAVE_SIDES(X)
#undef X
    default: return 0;
  }
}
inline int two_step_pairs(int N) {
  switch (N) {
#define X(N_) \
  case N_: return Split<N_>::GP;
    FSD_WAVE_SIDES(X)
#undef X
    default: return 0;
  }
}

// ---- run-time passes -----------------------------------------------------------------------------
// LDS distance, in elements of elem_bytes, between the B lines that one workgroup of a z
// or y pass transforms.  Loading B consecutive x of a grid row puts neighbouring lanes on
// different lines, so with a stride of N (a multiple of the 64 banks' width for every even
// N) they would all hit one bank.  A stride S with S / t odd, t = max(1, E / B) and E the
// elements per bank row, sends the lanes of one LDS cycle to distinct banks.
__host__ __device__ inline int fft_line_stride(int N, int B, int elem_bytes) {
  if (B <= 1) return N;
  const int E = 256 / elem_bytes, t = E / B > 1 ? E / B : 1;
  int S = N;
  while (S % (2 * t) != t) ++S;
  return S;
}

// LDS of the x+Green pass with G row slots and complex values of tb bytes: two buffers of
// 6 G lines (stride N | 1) and the twiddles, then (16-byte aligned) the 2 G row descriptors
__host__ __device__ inline size_t xgreen_rows_offset(int N, int G, int tb) {
  return (size_t(tb) * (12 * size_t(G) * (N | 1) + N) + 15) & ~size_t(15);
}
__host__ __device__ inline size_t xgreen_shm(int N, int G, int tb) {
  return xgreen_rows_offset(N, G, tb) + 2 * size_t(G) * 16;
}

// row slots per workgroup of the x+Green pass (measured: 2 is fastest at 64^3 and 128^3)
inline int fft_green_rows(int N) { return N >= 256 ? 1 : N >= 64 ? 2 : 256 / N; }

inline bool tile_b_fits(int N, int B, int rbytes) {
  return B >= 1 && (B & (B - 1)) == 0 && N % B == 0 &&
         size_t(2 * rbytes) * (2 * size_t(B) * fft_line_stride(N, B, 2 * rbytes) + N) <= (size_t(64) << 10);
}

inline bool tile_g_fits(int N, int G, int rbytes) {
  return G >= 1 && G <= 16 && xgreen_shm(N, G, 2 * rbytes) <= (size_t(64) << 10);
}

// lines per workgroup of the coalesced y/z passes: largest B in {16, 8, 4, 2, 1} dividing N
// whose two LDS buffers and twiddles fit in 64 KB
inline int fft_lines_b(int N, int rbytes) {
  for (int B = 16; B > 1; B /= 2)
    if (tile_b_fits(N, B, rbytes)) return B;
  return 1;
}

// The tile of a pass: of the two-step kernels, or of the run-time ones.  A measured tile counts where it
// fits at this precision (a mixed system's is measured in FP32, and its FP64 applies may not hold it);
// the run-time kernels never get a two-step size, which need not be a power of two or fit their buffers.
struct FftTile {
  bool two_step;
  int size;
};
inline FftTile line_tile(int N, int measured, int rbytes) {
  if (measured > 0 && tile_b_fits(N, measured, rbytes)) return {false, measured};
  const int two = two_step_lines(N, rbytes);
  return two ? FftTile{true, two} : FftTile{false, fft_lines_b(N, rbytes)};
}
inline FftTile green_tile(int N, int measured, int rbytes) {
  if (measured > 0 && tile_g_fits(N, measured, rbytes)) return {false, measured};
  const int two = two_step_pairs(N);
  return two ? FftTile{true, two} : FftTile{false, fft_green_rows(N)};
}

}  // namespace fsd
