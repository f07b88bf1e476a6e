// Transforms of lines held in registers: a line of N = RA RB points takes two steps, a DFT of RA
// points in the registers of each of RB threads, one exchange through LDS, and a DFT of RB points
// in each of RA threads.
#pragma once
#include "k_common.hpp"
#include "turn_consts.hpp"

namespace fsd {

template <int I, int N, typename Fn>
__device__ __forceinline__ void unroll_for(Fn&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unroll_for<I + 1, N>(f);
  }
}

// v exp(-2 pi i M / N)
template <int M, int N, typename T>
__device__ __forceinline__ T turn(T v) {
  using R = decltype(v.x);
  T r;
  if constexpr (M % N == 0) {
    r = v;
  } else if constexpr (4 * M == N) {
    r.x = v.y;
    r.y = -v.x;
  } else {
    constexpr R c = R(cos_turn(M, N)), s = R(sin_turn(M, N));
    r.x = c * v.x + s * v.y;
    r.y = c * v.y - s * v.x;
  }
  return r;
}

// ---- DFTs of N points in registers, in place, X_k = sum_n x_n exp(-2 pi i n k / N) ----------------
template <int N>
struct Dft;

template <>
struct Dft<2> {
  template <typename T>
  static __device__ __forceinline__ void run(T (&v)[2]) {
    const T a = v[0];
    v[0] = cadd(a, v[1]);
    v[1] = csub(a, v[1]);
  }
};
template <>
struct Dft<3> {
  template <typename T>
  static __device__ __forceinline__ void run(T (&v)[3]) {
    using R = decltype(v[0].x);
    const T s = cadd(v[1], v[2]), d = csub(v[1], v[2]);
    const R h = R(sin_turn(1, 3));
    T m, j;
    m.x = v[0].x - R(0.5) * s.x;
    m.y = v[0].y - R(0.5) * s.y;
    j.x = h * d.y;  // -i h d
    j.y = -h * d.x;
    v[0] = cadd(v[0], s);
    v[1] = cadd(m, j);
    v[2] = csub(m, j);
  }
};
template <>
struct Dft<4> {
  template <typename T>
  static __device__ __forceinline__ void run(T (&v)[4]) {
    const T s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]), s13 = cadd(v[1], v[3]),
            d13 = turn<1, 4>(csub(v[1], v[3]));
    v[0] = cadd(s02, s13);
    v[1] = cadd(d02, d13);
    v[2] = csub(s02, s13);
    v[3] = csub(d02, d13);
  }
};
template <>
struct Dft<5> {
  template <typename T>
  static __device__ __forceinline__ void run(T (&v)[5]) {
    using R = decltype(v[0].x);
    constexpr R c1 = R(cos_turn(1, 5)), c2 = R(cos_turn(2, 5)), s1 = R(sin_turn(1, 5)), s2 = R(sin_turn(2, 5));
    const T p = cadd(v[1], v[4]), q = cadd(v[2], v[3]), a = csub(v[1], v[4]), b = csub(v[2], v[3]);
    T m1, m2, j1, j2;
    m1.x = v[0].x + c1 * p.x + c2 * q.x;
    m1.y = v[0].y + c1 * p.y + c2 * q.y;
    m2.x = v[0].x + c2 * p.x + c1 * q.x;
    m2.y = v[0].y + c2 * p.y + c1 * q.y;
    j1.x = s1 * a.y + s2 * b.y;  // -i (s1 a + s2 b)
    j1.y = -(s1 * a.x + s2 * b.x);
    j2.x = s2 * a.y - s1 * b.y;
    j2.y = -(s2 * a.x - s1 * b.x);
    v[0] = cadd(v[0], cadd(p, q));
    v[1] = cadd(m1, j1);
    v[2] = cadd(m2, j2);
    v[3] = csub(m2, j2);
    v[4] = csub(m1, j1);
  }
};
// N = A B: B transforms of A points (stride B), the twiddles, A transforms of B points
template <int A, int B>
struct DftPair {
  template <typename T>
  static __device__ __forceinline__ void run(T (&v)[A * B]) {
    T w[B][A];
    unroll_for<0, B>([&](auto n2) {
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) w[n2][n1] = v[B * n1 + n2];
      Dft<A>::run(w[n2]);
      unroll_for<0, A>([&](auto k1) { w[n2][k1] = turn<(n2 * k1) % (A * B), A * B>(w[n2][k1]); });
    });
    unroll_for<0, A>([&](auto k1) {
      T u[B];
#pragma unroll
      for (int n2 = 0; n2 < B; ++n2) u[n2] = w[n2][k1];
      Dft<B>::run(u);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = u[k2];
    });
  }
};
// N = A B without a common factor: no twiddles between the two steps when the input is taken in the order
// B n1 + A n2 and the output, k mod A and k mod B, is put together by the remainders (Good's mapping).  With it
// and the nearest constants the rms error of a 3D transform is 2.4, 3.2, 2.9, 3.0 and 3.4e-16 on sides 24, 36, 48,
// 96 and 144, with twiddles between the steps and constants summed in FP64 2.8, 4.3, 3.7, 3.9 and 4.4e-16; times
// are the same but for x+Green on sides 192 (FP64 137 -> 145 us) and 240 (FP32 181 -> 185).
constexpr int inverse_mod(int a, int m) {
  for (int x = 1; x < m; ++x)
    if (a * x % m == 1) return x;
  return 0;
}
template <int A, int B>
struct DftCoprime {
  template <typename T>
  static __device__ __forceinline__ void run(T (&v)[A * B]) {
    constexpr int N = A * B, ea = B * inverse_mod(B % A, A), eb = A * inverse_mod(A % B, B);
    T w[B][A];
    unroll_for<0, B>([&](auto n2) {
#pragma unroll
      for (int n1 = 0; n1 < A; ++n1) w[n2][n1] = v[(B * n1 + A * n2) % N];
      Dft<A>::run(w[n2]);
    });
    unroll_for<0, A>([&](auto k1) {
      T u[B];
#pragma unroll
      for (int n2 = 0; n2 < B; ++n2) u[n2] = w[n2][k1];
      Dft<B>::run(u);
#pragma unroll
      for (int k2 = 0; k2 < B; ++k2) v[(ea * k1 + eb * k2) % N] = u[k2];
    });
  }
};
template <>
struct Dft<6> : DftCoprime<2, 3> {};
template <>
struct Dft<8> : DftPair<2, 4> {};
template <>
struct Dft<9> : DftPair<3, 3> {};
template <>
struct Dft<10> : DftCoprime<2, 5> {};
template <>
struct Dft<12> : DftCoprime<3, 4> {};
template <>
struct Dft<15> : DftCoprime<5, 3> {};
template <>
struct Dft<16> : DftPair<4, 4> {};

// Exchange in LDS: element e of a line at slot (e mod RA) PAD + e / RA, PAD >= RB odd.  The first
// step's thread b writes e = b RA + r (slots r PAD + b: neighbours side by side), the second
// step's reads e = b + r RA (slots b PAD + r: an odd stride) and, in place, may write its outputs
// k = b + r RA.
template <int N>
constexpr int kPad = Split<N>::RB | 1;
template <int N>
constexpr int kSlots = Split<N>::RA * kPad<N>;

template <typename R, int N>
struct LineTile {
  static constexpr int RA = Split<N>::RA, RB = Split<N>::RB;
  static constexpr int B = split_lines<N>(sizeof(R));
  static constexpr int kThreads = (B * RB + 63) / 64 * 64;
  static constexpr size_t kBytes = 2 * sizeof(R) * (size_t(B) * kSlots<N> + N);
  static_assert(RA <= RB && N * N % B == 0 && kThreads <= 256 && kBytes <= 65536, "one pass of 256 threads");
};

// One z (DIR 2) or y (DIR 1) pass over B consecutive lines of one component: line gl = o N + x.
// Neighbouring lanes hold neighbouring lines, so every access is a run of B complex values.
// sign +1 swaps real and imaginary parts on the way in and out (the inverse transform).
template <typename R, int N, int DIR, int SIGN>
__device__ __forceinline__ void lines_body(R* __restrict__ grid, const R* __restrict__ twiddle, unsigned char* smem,
                                           int blk) {
  using T = typename C2<R>::T;
  using Tile = LineTile<R, N>;
  constexpr int RA = Tile::RA, RB = Tile::RB, B = Tile::B, PAD = kPad<N>;
  T* buf = reinterpret_cast<T*>(smem);
  T* tw = buf + B * kSlots<N>;
  const int t = threadIdx.x, l = t % B, b = t / B;
  const unsigned gl = unsigned(blk) * B + l;
  constexpr unsigned es = DIR == 1 ? N : N * N;
  const unsigned base = DIR == 1 ? (gl / N) * unsigned(N * N) + gl % N : gl;
  if (b < RB) {
    T v[RA];
#pragma unroll
    for (int r = 0; r < RA; ++r) {
      const unsigned i = 2 * (base + (b + r * RB) * es);
      if (SIGN < 0)
        ldg2(grid, i, v[r].x, v[r].y);
      else
        ldg2(grid, i, v[r].y, v[r].x);
    }
    for (int k = t; k < N; k += B * RB) ldg2(twiddle, 2 * k, tw[k].x, tw[k].y);
    Dft<RA>::run(v);
#pragma unroll
    for (int r = 0; r < RA; ++r) buf[(r * PAD + b) * B + l] = v[r];
  }
  __syncthreads();
  if (b < RA) {
    T v[RB];
    v[0] = buf[b * PAD * B + l];
#pragma unroll
    for (int r = 1; r < RB; ++r) v[r] = cmul(buf[(b * PAD + r) * B + l], tw[r * b]);
    Dft<RB>::run(v);
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const unsigned i = 2 * (base + (b + r * RA) * es);
      if (SIGN < 0)
        stg2(grid, i, v[r].x, v[r].y);
      else
        stg2(grid, i, v[r].y, v[r].x);
    }
  }
}

// Lines along x (contiguous), one component of a 3D transform.
template <typename R, int N>
struct RowTile {
  static constexpr int RA = Split<N>::RA, RB = Split<N>::RB;
  static constexpr int kLines = 256 / RB;
  static constexpr size_t kBytes = 2 * sizeof(R) * (size_t(kLines) * kSlots<N> + N);
};

template <typename R, int N, int SIGN>
__device__ __forceinline__ void rows_body(R* __restrict__ grid, const R* __restrict__ twiddle, unsigned char* smem,
                                          int blk) {
  using T = typename C2<R>::T;
  using Tile = RowTile<R, N>;
  constexpr int RA = Tile::RA, RB = Tile::RB, PAD = kPad<N>;
  T* buf = reinterpret_cast<T*>(smem);
  T* tw = buf + Tile::kLines * kSlots<N>;
  const int t = threadIdx.x, l = t / RB, b = t % RB;
  const int line = blk * Tile::kLines + l;
  const bool live = l < Tile::kLines && line < N * N;
  const unsigned base = unsigned(line) * N;
  T* mine = buf + l * kSlots<N>;
  for (int k = t; k < N; k += 256) ldg2(twiddle, 2 * k, tw[k].x, tw[k].y);
  if (live) {
    T v[RA];
#pragma unroll
    for (int r = 0; r < RA; ++r) {
      if (SIGN < 0)
        ldg2(grid, 2 * (base + b + r * RB), v[r].x, v[r].y);
      else
        ldg2(grid, 2 * (base + b + r * RB), v[r].y, v[r].x);
    }
    Dft<RA>::run(v);
#pragma unroll
    for (int r = 0; r < RA; ++r) mine[r * PAD + b] = v[r];
  }
  __syncthreads();
  if (live && b < RA) {
    T v[RB];
    v[0] = mine[b * PAD];
#pragma unroll
    for (int r = 1; r < RB; ++r) v[r] = cmul(mine[b * PAD + r], tw[r * b]);
    Dft<RB>::run(v);
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      if (SIGN < 0)
        stg2(grid, 2 * (base + b + r * RA), v[r].x, v[r].y);
      else
        stg2(grid, 2 * (base + b + r * RA), v[r].y, v[r].x);
    }
  }
}

// The x+Green pass (see k_fft.hip) with two-step transforms: a workgroup takes G of the row pairs,
// six lines each, TPL threads a line.
template <typename R, int N>
struct GreenTile {
  static constexpr int RA = Split<N>::RA, RB = Split<N>::RB, TPL = RB;
  static constexpr int G = Split<N>::GP;
  static constexpr size_t kRows = (2 * sizeof(R) * (size_t(6 * G) * kSlots<N> + N) + 15) / 16 * 16;
  static constexpr size_t kBytes = kRows + sizeof(int4) * G;
  static_assert(G >= 1 && 6 * G * TPL <= 256 && kBytes <= 65536, "one pass of 256 threads");
};

template <int N>
__device__ __forceinline__ int slot_of(int e) {
  return (e % Split<N>::RA) * kPad<N> + e / Split<N>::RA;
}

template <typename R, int N, bool TABLE>
__device__ __forceinline__ void green_body(R* __restrict__ grid, const R* __restrict__ twiddle, const WaveParams& wp,
                                           unsigned char* smem, int blk) {
  using T = typename C2<R>::T;
  using Tile = GreenTile<R, N>;
  constexpr int RA = Tile::RA, RB = Tile::RB, PAD = kPad<N>, SL = kSlots<N>, G = Tile::G, H = N / 2;
  constexpr unsigned cs = 2u * N * N * N;
  T* buf = reinterpret_cast<T*>(smem);
  T* tw = buf + 6 * G * SL;
  int4* pairs = reinterpret_cast<int4*>(smem + Tile::kRows);
  const int t = threadIdx.x;
  // descriptor of slot g: x = kz, y = ky of its first row (x = -1: no row), z, w = the two rows
  if (t < G) {
    const int p = blk * G + t;
    int4 d = make_int4(-1, 0, 0, 0);
    if (p < N * N / 2 + 2) {
      const int r = green_row(p, N);
      const int kz = r / N, ky = r - kz * N;
      d = make_int4(kz, ky, r, (kz ? N - kz : 0) * N + (ky ? N - ky : 0));
    }
    pairs[t] = d;
  }
  for (int k = t; k < N; k += 256) ldg2(twiddle, 2 * k, tw[k].x, tw[k].y);
  __syncthreads();
  // line (g, c, q): component c of row q (0: r, 1: its partner) of slot g
  const int line = t / Tile::TPL, b = t % Tile::TPL, g = line / 6, c = (line - 6 * g) >> 1, q = line & 1;
  unsigned base = 0;
  bool live = line < 6 * G;
  if (live) {
    const int4 d = pairs[g];
    live = d.x >= 0 && (q == 0 || d.z != d.w);  // a self-paired row has no second line
    base = unsigned(c) * cs + 2u * unsigned(q ? d.w : d.z) * N;
  }
  T* mine = buf + line * SL;
  if (live) {
    T v[RA];
#pragma unroll
    for (int r = 0; r < RA; ++r) ldg2(grid, base + 2 * (b + r * RB), v[r].x, v[r].y);
    Dft<RA>::run(v);
#pragma unroll
    for (int r = 0; r < RA; ++r) mine[r * PAD + b] = v[r];
  }
  __syncthreads();
  if (live && b < RA) {
    T v[RB];
    v[0] = mine[b * PAD];
#pragma unroll
    for (int r = 1; r < RB; ++r) v[r] = cmul(mine[b * PAD + r], tw[r * b]);
    Dft<RB>::run(v);
#pragma unroll
    for (int r = 0; r < RB; ++r) mine[b * PAD + r] = v[r];
  }
  __syncthreads();
  // every mode k of the first row with its partner -k in the second (both are this thread's alone)
  const double gam = (!TABLE && wp.gam) ? *wp.gam : 0.0;
  for (int i = t; i < G * N; i += 256) {
    const int gi = i / N, kx = i - gi * N;
    const int4 d = pairs[gi];
    const bool self = d.z == d.w;
    if (d.x < 0 || (self && kx > H)) continue;
    T* z0 = buf + 6 * gi * SL + slot_of<N>(kx);
    T* z1 = buf + (6 * gi + (self ? 0 : 1)) * SL + slot_of<N>(kx ? N - kx : 0);
    const bool zero = kx == H || d.y == H || d.x == H || (kx == 0 && d.y == 0 && d.x == 0);
    T a[3], m[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      a[e] = z0[2 * e * SL];
      m[e] = z1[2 * e * SL];
    }
    if (zero) {
#pragma unroll
      for (int e = 0; e < 3; ++e) a[e].x = a[e].y = m[e].x = m[e].y = 0;
    } else {
      green_mode<R, TABLE>(wp, N, kx <= H ? kx : kx - N, d.y <= H ? d.y : d.y - N, d.x <= H ? d.x : d.x - N, gam, a, m);
    }
    // swapped, for the inverse transform
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      T s;
      s.x = m[e].y;
      s.y = m[e].x;
      z1[2 * e * SL] = s;
      s.x = a[e].y;
      s.y = a[e].x;
      z0[2 * e * SL] = s;
    }
  }
  __syncthreads();
  // the inverse takes the steps the other way round: RB points of k = b + r RA first
  if (live && b < RA) {
    T v[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) v[r] = mine[b * PAD + r];
    Dft<RB>::run(v);
#pragma unroll
    for (int r = 0; r < RB; ++r) mine[b * PAD + r] = v[r];
  }
  __syncthreads();
  if (live) {
    T v[RA];
    v[0] = mine[b];
#pragma unroll
    for (int r = 1; r < RA; ++r) v[r] = cmul(mine[r * PAD + b], tw[r * b]);
    Dft<RA>::run(v);
#pragma unroll
    for (int r = 0; r < RA; ++r) stg2(grid, base + 2 * (b + r * RB), v[r].y, v[r].x);
  }
}

}  // namespace fsd
