// Tiles of the transform passes: the sides with two-step transforms, the rules of the run-time passes
// and the choice between them.
#pragma once
#include <cstddef>

namespace fsd {

// ---- sides with a two-step transform ----------------------------------------------------------
// RA <= RB, both at most 16 (a thread's registers).  BL: lines of a z or y pass per workgroup in
// FP32, dividing N^2, as many as 256 threads transform in one go (RB each); FP64 takes half.
// GP: row pairs of an x+Green workgroup, 6 lines each (even sides).
template <int N>
struct Split;
#define FSD_SPLIT(N_, A_, B_, L_, G_)                    \
  template <>                                            \
  struct Split<N_> {                                     \
    static constexpr int RA = A_, RB = B_, BL = L_, GP = G_; \
  };
// the sides that are multiples of 8, as the grid rule takes them
FSD_SPLIT(8, 2, 4, 64, 10)
FSD_SPLIT(16, 4, 4, 64, 10)
FSD_SPLIT(24, 4, 6, 32, 7)
FSD_SPLIT(32, 4, 8, 32, 5)
FSD_SPLIT(40, 5, 8, 32, 5)
FSD_SPLIT(48, 6, 8, 32, 5)
FSD_SPLIT(64, 8, 8, 32, 4)
FSD_SPLIT(72, 8, 9, 24, 3)
FSD_SPLIT(80, 8, 10, 16, 3)
FSD_SPLIT(96, 8, 12, 16, 2)
FSD_SPLIT(120, 10, 12, 16, 2)
FSD_SPLIT(128, 8, 16, 16, 2)
FSD_SPLIT(144, 12, 12, 16, 1)
FSD_SPLIT(160, 10, 16, 16, 1)
FSD_SPLIT(192, 12, 16, 16, 1)
FSD_SPLIT(240, 15, 16, 16, 1)
FSD_SPLIT(256, 16, 16, 16, 1)
// further sides of the 3D transform on its own
FSD_SPLIT(27, 3, 9, 27, 0)
FSD_SPLIT(36, 6, 6, 36, 0)
FSD_SPLIT(45, 5, 9, 25, 0)
FSD_SPLIT(50, 5, 10, 25, 0)
FSD_SPLIT(54, 6, 9, 27, 0)
FSD_SPLIT(60, 6, 10, 24, 0)
FSD_SPLIT(75, 5, 15, 15, 0)
FSD_SPLIT(81, 9, 9, 27, 0)
FSD_SPLIT(90, 9, 10, 20, 0)
FSD_SPLIT(100, 10, 10, 25, 0)
FSD_SPLIT(108, 9, 12, 16, 0)
FSD_SPLIT(135, 9, 15, 15, 0)
FSD_SPLIT(150, 10, 15, 15, 0)
FSD_SPLIT(180, 12, 15, 16, 0)
#undef FSD_SPLIT
#define FSD_WAVE_SIDES(X) \
  X(8) X(16) X(24) X(32) X(40) X(48) X(64) X(72) X(80) X(96) X(120) X(128) X(144) X(160) X(192) X(240) X(256)
#define FSD_OTHER_SIDES(X) \
  X(27) X(36) X(45) X(50) X(54) X(60) X(75) X(81) X(90) X(100) X(108) X(135) X(150) X(180)

// lines of a z or y pass per workgroup, values of rbytes
template <int N>
constexpr int split_lines(size_t rbytes) {
  return rbytes == 8 && Split<N>::BL % 2 == 0 ? Split<N>::BL / 2 : Split<N>::BL;
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
