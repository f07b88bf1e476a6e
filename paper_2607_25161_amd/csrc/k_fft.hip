// Wave-space transforms: the z, y and x+Green passes of the mobility, their multi-system forms, and
// the 3D transform on its own.
#include <algorithm>
#include <mutex>

#include "k_common.hpp"
#include "k_rigid.hpp"

namespace fsd {

namespace {
constexpr int kThreads = 256;

__device__ inline void sinc_jv_d(double x, double& s, double& j) {
  if (x < 0.5) {
    const double x2 = x * x;
    s = 1.0 - x2 / 6.0 * (1.0 - x2 / 20.0 * (1.0 - x2 / 42.0 * (1.0 - x2 / 72.0 * (1.0 - x2 / 110.0))));
    j = 1.0 - x2 / 10.0 * (1.0 - x2 / 28.0 * (1.0 - x2 / 54.0 * (1.0 - x2 / 88.0 * (1.0 - x2 / 130.0))));
  } else {
    double sn, cn;
    sincos(x, &sn, &cn);
    s = sn / x;
    j = 3.0 * (sn - x * cn) / (x * x * x);
  }
}

// first row kz N + ky of pair number p of the N^2 / 2 + 2 pairs {row, row of (-kz, -ky)} (the four
// self-paired rows count as pairs of one)
__device__ __forceinline__ int green_row(int p, int N) {
  const int H = N / 2;
  if (p <= H) return p;                        // kz = 0, ky = 0 .. N/2
  p -= H + 1;
  if (p < (H - 1) * N) return N + p;           // kz = 1 .. N/2 - 1, all ky
  return H * N + (p - (H - 1) * N);            // kz = N/2, ky = 0 .. N/2
}

// Green's scaling of mode (mx, my, mz) and its partner -k: a and m hold the packed spectra
// Z(k) = F + i T of the three axes at k and at -k, and get Y = U + i W there.
template <typename R, bool TABLE, typename T>
__device__ __forceinline__ void green_mode(const WaveParams& wp, int N, int mx, int my, int mz, double gam, T (&a)[3],
                                           T (&m)[3]) {
  const double tp = 2.0 * M_PI / wp.L;
  // the per-mode arithmetic runs in the grid's precision R (the multipliers are tabulated
  // in FP64 and rounded once).  F, T below are twice the split spectra
  // F^ = (Z(k) + conj Z(-k)) / 2, T^ = (Z(k) - conj Z(-k)) / 2i; the halving moves into the
  // scalar factor Bk (exact: the products scale by powers of two)
  R Fr[3], Fi[3], Tr[3], Ti[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    Fr[c] = a[c].x + m[c].x;
    Fi[c] = a[c].y - m[c].y;
    Tr[c] = a[c].y + m[c].y;
    Ti[c] = m[c].x - a[c].x;
  }
  // Cartesian wave vector of the mode: (2 pi / L)(m_x, m_y - gam m_x, m_z) (the reciprocal
  // lattice of the sheared lattice; gam = 0 for the cube)
  const R k[3] = {R(tp * mx), R(tp * (my - gam * mx)), R(tp * mz)};
  R sk, jk, Bk, ikn;
  if (TABLE) {  // the multipliers depend on the integer |m|^2 alone
    const int m2 = mx * mx + my * my + mz * mz;
    if constexpr (sizeof(R) == 4) {  // the FP32 copy of the table (the same roundings)
      const float4 g4 = *reinterpret_cast<const float4*>(wp.gtab32 + 8 * m2);
      sk = g4.x;
      jk = g4.y;
      Bk = wp.brownian ? g4.w : g4.z;
      ikn = wp.gtab32[8 * m2 + 4];
    } else {
      const double* gt = wp.gtab + 5 * m2;
      sk = R(gt[0]);
      jk = R(gt[1]);
      Bk = R(wp.brownian ? gt[3] : gt[2]);
      ikn = R(gt[4]);
    }
  } else {
    const double kd[3] = {tp * mx, tp * (my - gam * mx), tp * mz};
    const double k2 = kd[0] * kd[0] + kd[1] * kd[1] + kd[2] * kd[2];
    const double kn = sqrt(k2);
    double skd, jkd;
    sinc_jv_d(kn * wp.a, skd, jkd);
    const double qq = k2 / (4.0 * wp.xi * wp.xi);
    const double damp = (1.0 + qq) * exp(-(1.0 - wp.eta_t) * qq) / wp.eta;
    sk = R(skd);
    jk = R(jkd);
    ikn = R(1.0 / kn);
    Bk = R(wp.brownian ? sqrt(wp.scale / (double(N) * N * N) * damp) / kn : wp.scale * damp / k2);
  }
  Bk *= R(0.5);
  const R hjk = R(0.5) * jk;
  const R kh[3] = {k[0] * ikn, k[1] * ikn, k[2] * ikn};
  R gr[3], gi[3];
  if (wp.brownian) {
    for (int a = 0; a < 3; ++a) {
      gr[a] = Fr[a];
      gi[a] = Fi[a];
    }
  } else {
    const R cxr[3] = {k[1] * Tr[2] - k[2] * Tr[1], k[2] * Tr[0] - k[0] * Tr[2], k[0] * Tr[1] - k[1] * Tr[0]};
    const R cxi[3] = {k[1] * Ti[2] - k[2] * Ti[1], k[2] * Ti[0] - k[0] * Ti[2], k[0] * Ti[1] - k[1] * Ti[0]};
    for (int a = 0; a < 3; ++a) {
      gr[a] = sk * Fr[a] - hjk * cxi[a];
      gi[a] = sk * Fi[a] + hjk * cxr[a];
    }
  }
  const R pr = kh[0] * gr[0] + kh[1] * gr[1] + kh[2] * gr[2];
  const R pim = kh[0] * gi[0] + kh[1] * gi[1] + kh[2] * gi[2];
  R ur[3], ui[3];
  for (int a = 0; a < 3; ++a) {
    ur[a] = Bk * (gr[a] - pr * kh[a]);
    ui[a] = Bk * (gi[a] - pim * kh[a]);
  }
  // U^ = sinc u^, W^ = (i/2) jv (k x u^); Y^ = U^ + i W^
  const R kur[3] = {k[1] * ur[2] - k[2] * ur[1], k[2] * ur[0] - k[0] * ur[2], k[0] * ur[1] - k[1] * ur[0]};
  const R kui[3] = {k[1] * ui[2] - k[2] * ui[1], k[2] * ui[0] - k[0] * ui[2], k[0] * ui[1] - k[1] * ui[0]};
  for (int c = 0; c < 3; ++c) {
    const R Ur = sk * ur[c], Ui = sk * ui[c];
    const R Wr = -hjk * kui[c], Wi = hjk * kur[c];
    a[c].x = Ur - Wi;
    a[c].y = Ui + Wr;
    // at -k, U and W take the conjugates (the components are real)
    m[c].x = Ur + Wi;
    m[c].y = Wr - Ui;
  }
}
}  // namespace
}  // namespace fsd

#include "fft_regs.hpp"

namespace fsd {

// ------------------------------------------------------------------------------------------
// Any side: lines staged in LDS and transformed by mixed-radix (8, 4, 2, 3, 5) Stockham stages
// with the radices known at run time.  The sides of fft_regs.hpp take its two-step transforms.
// ------------------------------------------------------------------------------------------

namespace {
// Quotient and remainder by a divisor known only at run time, for dividends below 2^21:
// the product with the FP32 reciprocal (v_rcp_f32, within 1 ulp) is within 1/4 of the true
// quotient, so truncating it and one correction step give the exact result (a hardware
// integer division sequence costs about 25 instructions per use in these index loops).
struct FastDiv {
  int d;
  float inv;
  __device__ explicit FastDiv(int d_) : d(d_), inv(__frcp_rn(float(d_))) {}
  __device__ __forceinline__ int div(int a) const {
    int q = int(float(a) * inv);
    const int r = a - q * d;
    q += (r >= d) - (r < 0);
    return q;
  }
  __device__ __forceinline__ void divmod(int a, int& q, int& r) const {
    q = div(a);
    r = a - q * d;
  }
};

// multiply by -i*sign... rot(v, s) = s * i * v
template <typename T>
__device__ inline T rot(T v, int s) {
  T r;
  r.x = -s * v.y;
  r.y = s * v.x;
  return r;
}
}  // namespace

namespace {
// One radix-Rd butterfly of a Stockham stage: reads Rd inputs nbf apart, twiddles them by
// w^(r k tstride) (w = exp(s 2 pi i / N), the table tw), transforms and writes them Ns apart.
template <typename T, typename R, int Rd>
__device__ __forceinline__ void butterfly(const T* li, T* lo, const T* tw, int b, int nbf, int k, int Ns, int tstride,
                                          int od, int s) {
  T v[Rd];
#pragma unroll
  for (int r = 0; r < Rd; ++r) v[r] = li[b + r * nbf];
  if (Ns > 1) {
#pragma unroll
    for (int r = 1; r < Rd; ++r) v[r] = cmul(v[r], tw[r * k * tstride]);
  }
  if constexpr (Rd == 8) {
    // even and odd halves by 4-point transforms, joined by w^k = exp(s 2 pi i k / 8)
    const T es02 = cadd(v[0], v[4]), ed02 = csub(v[0], v[4]), es13 = cadd(v[2], v[6]),
            ed13 = rot(csub(v[2], v[6]), s);
    const T os02 = cadd(v[1], v[5]), od02 = csub(v[1], v[5]), os13 = cadd(v[3], v[7]),
            od13 = rot(csub(v[3], v[7]), s);
    const T e0 = cadd(es02, es13), e1 = cadd(ed02, ed13), e2 = csub(es02, es13), e3 = csub(ed02, ed13);
    const T o0 = cadd(os02, os13), o1 = cadd(od02, od13), o2 = csub(os02, os13), o3 = csub(od02, od13);
    const R h8 = R(0.70710678118654752440), sr = R(s);
    T t1, t3;
    t1.x = h8 * (o1.x - sr * o1.y);  // w o1, w = (1 + s i) / sqrt 2
    t1.y = h8 * (o1.y + sr * o1.x);
    t3.x = -h8 * (o3.x + sr * o3.y);  // w^3 o3, w^3 = (-1 + s i) / sqrt 2
    t3.y = h8 * (sr * o3.x - o3.y);
    const T t2 = rot(o2, s);
    lo[od] = cadd(e0, o0);
    lo[od + 4 * Ns] = csub(e0, o0);
    lo[od + Ns] = cadd(e1, t1);
    lo[od + 5 * Ns] = csub(e1, t1);
    lo[od + 2 * Ns] = cadd(e2, t2);
    lo[od + 6 * Ns] = csub(e2, t2);
    lo[od + 3 * Ns] = cadd(e3, t3);
    lo[od + 7 * Ns] = csub(e3, t3);
  } else if constexpr (Rd == 4) {
    const T s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]), s13 = cadd(v[1], v[3]), d13 = rot(csub(v[1], v[3]), s);
    lo[od] = cadd(s02, s13);
    lo[od + Ns] = cadd(d02, d13);
    lo[od + 2 * Ns] = csub(s02, s13);
    lo[od + 3 * Ns] = csub(d02, d13);
  } else if constexpr (Rd == 2) {
    lo[od] = cadd(v[0], v[1]);
    lo[od + Ns] = csub(v[0], v[1]);
  } else if constexpr (Rd == 3) {
    const R c3 = R(-0.5), s3 = R(0.86602540378443864676);
    const T sm = cadd(v[1], v[2]), jd = rot(csub(v[1], v[2]), s);  // s i (v1 - v2)
    T m1, y1, y2;
    m1.x = v[0].x + c3 * sm.x;
    m1.y = v[0].y + c3 * sm.y;
    y1.x = m1.x + s3 * jd.x;
    y1.y = m1.y + s3 * jd.y;
    y2.x = m1.x - s3 * jd.x;
    y2.y = m1.y - s3 * jd.y;
    lo[od] = cadd(v[0], sm);
    lo[od + Ns] = y1;
    lo[od + 2 * Ns] = y2;
  } else {  // radix 5: cos and sin of 2 pi / 5 and 4 pi / 5
    const R c1 = R(0.30901699437494742410), c2 = R(-0.80901699437494742410);
    const R s1 = R(0.95105651629515357212), s2 = R(0.58778525229247312917);
    const T t1 = cadd(v[1], v[4]), t2 = cadd(v[2], v[3]);
    const T t3 = rot(csub(v[1], v[4]), s), t4 = rot(csub(v[2], v[3]), s);  // s i (v1 - v4), s i (v2 - v3)
    T m1, m2, p1, p2;
    m1.x = v[0].x + c1 * t1.x + c2 * t2.x;
    m1.y = v[0].y + c1 * t1.y + c2 * t2.y;
    m2.x = v[0].x + c2 * t1.x + c1 * t2.x;
    m2.y = v[0].y + c2 * t1.y + c1 * t2.y;
    p1.x = s1 * t3.x + s2 * t4.x;
    p1.y = s1 * t3.y + s2 * t4.y;
    p2.x = s2 * t3.x - s1 * t4.x;
    p2.y = s2 * t3.y - s1 * t4.y;
    lo[od] = cadd(v[0], cadd(t1, t2));
    lo[od + Ns] = cadd(m1, p1);
    lo[od + 2 * Ns] = cadd(m2, p2);
    lo[od + 3 * Ns] = csub(m2, p2);
    lo[od + 4 * Ns] = csub(m1, p1);
  }
}

// Stockham stages (radices 8, 4, 2, 3, 5) on `nl` lines of length N held in LDS `ls`
// elements apart (`in`, scratch `out`); returns the buffer holding the result.  The
// radices come from the plan's packed code (4 bits per stage), so the stage loop indexes
// no array.
template <typename T, typename R>
__device__ __forceinline__ T* stockham(T* in, T* out, const T* tw, int N, int ls, int nl, const FftPlan& plan,
                                       int s) {
  int Ns = 1;
  const unsigned long long code = plan.rcode;
  for (int stg = 0; stg < plan.nstage; ++stg) {
    const int Rd = int((code >> (4 * stg)) & 15ull);
    const int nbf = N / Rd;
    const int tstride = N / (Ns * Rd);
    const FastDiv dbf(nbf), dns(Ns);
    for (int t = threadIdx.x; t < nl * nbf; t += blockDim.x) {
      int l, b, j, k;
      dbf.divmod(t, l, b);
      dns.divmod(b, j, k);
      const T* li = in + l * ls;
      T* lo = out + l * ls;
      const int od = j * Ns * Rd + k;
      if (Rd == 8)
        butterfly<T, R, 8>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else if (Rd == 4)
        butterfly<T, R, 4>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else if (Rd == 2)
        butterfly<T, R, 2>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else if (Rd == 3)
        butterfly<T, R, 3>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else
        butterfly<T, R, 5>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
    }
    __syncthreads();
    T* tmp = in;
    in = out;
    out = tmp;
    Ns *= Rd;
  }
  return in;
}

// Stockham stages on B lines (B a power of two, 2^lb) held S elements apart, with the
// line as the fastest thread index: t -> (line t & (B - 1), butterfly t >> lb).  Lanes
// that differ in the line meet distinct banks (the stride of fft_line_stride), and the
// mapping needs one division per butterfly (by the stage's Ns) instead of two.
// As stockham_lines for any number of lines nl (held S apart, S odd so that consecutive
// lines start on distinct banks): t -> (line t mod nl, butterfly t / nl).
template <typename T, typename R>
__device__ __forceinline__ T* stockham_lm(T* in, T* out, const T* tw, int N, int S, int nl, const FftPlan& plan,
                                          int s) {
  int Ns = 1;
  const unsigned long long code = plan.rcode;
  const FastDiv dnl(nl);
  for (int stg = 0; stg < plan.nstage; ++stg) {
    const int Rd = int((code >> (4 * stg)) & 15ull);
    const int nbf = N / Rd;
    const int tstride = N / (Ns * Rd);
    const FastDiv dns(Ns);
    for (int t = threadIdx.x; t < nl * nbf; t += blockDim.x) {
      int b, l, j, k;
      dnl.divmod(t, b, l);
      dns.divmod(b, j, k);
      const T* li = in + l * S;
      T* lo = out + l * S;
      const int od = j * Ns * Rd + k;
      if (Rd == 8)
        butterfly<T, R, 8>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else if (Rd == 4)
        butterfly<T, R, 4>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else if (Rd == 2)
        butterfly<T, R, 2>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else if (Rd == 3)
        butterfly<T, R, 3>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else
        butterfly<T, R, 5>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
    }
    __syncthreads();
    T* tmp = in;
    in = out;
    out = tmp;
    Ns *= Rd;
  }
  return in;
}

template <typename T, typename R>
__device__ __forceinline__ T* stockham_lines(T* in, T* out, const T* tw, int N, int S, int B, int lb,
                                             const FftPlan& plan, int s) {
  int Ns = 1;
  const unsigned long long code = plan.rcode;
  for (int stg = 0; stg < plan.nstage; ++stg) {
    const int Rd = int((code >> (4 * stg)) & 15ull);
    const int nbf = N / Rd;
    const int tstride = N / (Ns * Rd);
    const FastDiv dns(Ns);
    for (int t = threadIdx.x; t < (nbf << lb); t += blockDim.x) {
      const int l = t & (B - 1), b = t >> lb;
      int j, k;
      dns.divmod(b, j, k);
      const T* li = in + l * S;
      T* lo = out + l * S;
      const int od = j * Ns * Rd + k;
      if (Rd == 8)
        butterfly<T, R, 8>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else if (Rd == 4)
        butterfly<T, R, 4>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else if (Rd == 2)
        butterfly<T, R, 2>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else if (Rd == 3)
        butterfly<T, R, 3>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
      else
        butterfly<T, R, 5>(li, lo, tw, b, nbf, k, Ns, tstride, od, s);
    }
    __syncthreads();
    T* tmp = in;
    in = out;
    out = tmp;
    Ns *= Rd;
  }
  return in;
}

}  // namespace

template <typename R, int DIR>
__global__ __launch_bounds__(256) void k_fft_pass(R* __restrict__ data, size_t cs, FftPlan plan,
                                                  const R* __restrict__ twiddle, int sign, int B, const int* __restrict__ skip) {
  if (skip && *skip) return;
  using T = typename C2<R>::T;
  extern __shared__ unsigned char smem_raw[];
  const int N = plan.n;
  const int S = fft_line_stride(N, B, int(sizeof(T)));
  T* buf0 = reinterpret_cast<T*>(smem_raw);
  T* buf1 = buf0 + B * S;
  T* tw = buf1 + B * S;
  T* base = reinterpret_cast<T*>(data + blockIdx.y * cs);
  const int line0 = blockIdx.x * B;
  const T* twg = reinterpret_cast<const T*>(twiddle);
  for (int t = threadIdx.x; t < N; t += blockDim.x) {
    T w = twg[t];
    if (sign > 0) w.y = -w.y;
    tw[t] = w;
  }
  for (int t = threadIdx.x; t < B * N; t += blockDim.x) {
    int l, e;
    if (DIR == 0) {
      l = t / N;
      e = t % N;
    } else {
      l = t % B;
      e = t / B;
    }
    const size_t gl = size_t(line0 + l);
    size_t off;
    if (DIR == 0)
      off = gl * N + e;
    else if (DIR == 1)
      off = ((gl / N) * N + e) * N + (gl % N);
    else
      off = (size_t(e) * N + (gl / N)) * N + (gl % N);
    buf0[l * S + e] = base[off];
  }
  __syncthreads();
  const T* in = stockham<T, R>(buf0, buf1, tw, N, S, B, plan, sign > 0 ? 1 : -1);
  for (int t = threadIdx.x; t < B * N; t += blockDim.x) {
    int l, e;
    if (DIR == 0) {
      l = t / N;
      e = t % N;
    } else {
      l = t % B;
      e = t / B;
    }
    const size_t gl = size_t(line0 + l);
    size_t off;
    if (DIR == 0)
      off = gl * N + e;
    else if (DIR == 1)
      off = ((gl / N) * N + e) * N + (gl % N);
    else
      off = (size_t(e) * N + (gl / N)) * N + (gl % N);
    base[off] = in[l * S + e];
  }
}

namespace {
int lines_per_block(int N) {
  int B = 1;
  while (B * 2 * N <= 1024 && (N % (B * 2)) == 0) B *= 2;
  return B;
}
}  // namespace

namespace {
// Block-wide copy of `count` elements, t -> store(t, load(t)), with U loads in flight per
// thread: each thread issues its next U loads before it writes any of them, so one wait
// covers U memory latencies (a plain strided loop waits once per element).
template <int U, typename T, typename Load, typename Store>
__device__ __forceinline__ void staged_copy(int count, Load&& load, Store&& store) {
  for (int t0 = threadIdx.x; t0 < count; t0 += U * int(blockDim.x)) {
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * int(blockDim.x);
      if (t < count) v[u] = load(t);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * int(blockDim.x);
      if (t < count) store(t, v[u]);
    }
  }
}

template <typename T>
__device__ inline void load_twiddles(T* tw, const T* twg, int N, int sign) {
  for (int t = threadIdx.x; t < N; t += blockDim.x) {
    T w = twg[t];
    if (sign > 0) w.y = -w.y;
    tw[t] = w;
  }
}
}  // namespace

// ------------------------------------------------------------------------------------------
// Coalesced wave-space pipeline for N <= 256 (5 passes, in place on the three packed
// complex grids Z_c = F_c + i T_c):
//   z, y  : transforms along z, then y; a workgroup takes B consecutive x of B lines,
//           so every load and store is a run of B contiguous complex values
//   x+G   : one workgroup per pair of rows (ky, kz) and (-ky, -kz) of all three grids:
//           forward x transform, split of the packed spectra by Hermitian symmetry
//           (F^(k) = (Z(k) + conj Z(-k)) / 2, T^(k) = (Z(k) - conj Z(-k)) / 2i, the -k
//           partner lies in the paired row), Green's-function scaling, repacking as
//           Y^ = U^ + i W^, inverse x transform
//   y, z  : inverse transforms
// The product is the same linear operator as the half-spectrum pipeline.
// ------------------------------------------------------------------------------------------

template <typename R, int DIR>
__device__ __forceinline__ void fft_lines_body(R* __restrict__ grid, size_t cs, FftPlan plan,
                                               const R* __restrict__ twiddle, int sign, int B,
                                               const int* __restrict__ skip, int bx_, int by_, int gx_) {
  if (skip && *skip) return;
  using T = typename C2<R>::T;
  extern __shared__ unsigned char smem_raw[];
  const int N = plan.n;
  const int S = fft_line_stride(N, B, int(sizeof(T)));
  T* buf0 = reinterpret_cast<T*>(smem_raw);
  T* buf1 = buf0 + B * S;
  T* tw = buf1 + B * S;
  T* base = reinterpret_cast<T*>(grid + by_ * cs);
  const int line0 = bx_ * B;  // line gl = o N + x: B consecutive x of one o (B divides N)
  const int o = line0 / N, x0 = line0 - o * N;
  const int lb = __ffs(B) - 1;  // B is a power of two
  // element e of line l sits at g[e * es + l]: a workgroup-uniform base and a 32-bit
  // offset (its byte offset stays below 2 N^3 sizeof(R) <= 2^28 for N <= 256)
  R* g = reinterpret_cast<R*>(base + (DIR == 1 ? size_t(o) * N * N : size_t(o) * N) + x0);
  const unsigned es = DIR == 1 ? N : N * N;
  load_twiddles(tw, reinterpret_cast<const T*>(twiddle), N, sign);
  staged_copy<8, T>(
      B * N,
      [&](int t) {
        T v;
        ldg2(g, 2 * (unsigned(t >> lb) * es + unsigned(t & (B - 1))), v.x, v.y);
        return v;
      },
      [&](int t, const T& v) { buf0[(t & (B - 1)) * S + (t >> lb)] = v; });
  __syncthreads();
  const T* Y = stockham_lines<T, R>(buf0, buf1, tw, N, S, B, lb, plan, sign);
  for (int t = threadIdx.x; t < B * N; t += blockDim.x) {
    const int l = t & (B - 1), e = t >> lb;
    const T y = Y[l * S + e];
    stg2(g, 2 * (unsigned(e) * es + unsigned(l)), y.x, y.y);
  }
}

template <typename R, int DIR>
__global__ __launch_bounds__(256) void k_fft_lines(R* __restrict__ grid, size_t cs, FftPlan plan,
                                                   const R* __restrict__ twiddle, int sign, int B,
                                                   const int* __restrict__ skip) {
  fft_lines_body<R, DIR>(grid, cs, plan, twiddle, sign, B, skip, blockIdx.x, blockIdx.y, gridDim.x);
}

// TABLE: the cube, multipliers read from the table by |m|^2; otherwise (the sheared lattice)
// computed per mode.  Two instantiations keep the per-mode FP64 arithmetic out of the
// cube's register budget.
template <typename R, bool TABLE>
__device__ __forceinline__ void fft_xgreen_body(R* __restrict__ grid, size_t cs, FftPlan plan,
                                                const R* __restrict__ twiddle, WaveParams wp, int G,
                                                const int* __restrict__ skip, int bx_, int by_, int gx_) {
  if (skip && *skip) return;
  using T = typename C2<R>::T;
  extern __shared__ unsigned char smem_raw[];
  const int N = plan.n, NN = N * N;
  // G row slots per workgroup; slot g takes the pair number p = bx G + g of the
  // N^2/2 + 2 pairs {r, rp} (r = kz N + ky, rp = its (-kz, -ky) partner, r <= rp; the
  // four self-paired rows have rp == r).  Line (g, c, q) = component c of row q (0: r,
  // 1: rp) sits at (6 g + 2 c + q) N; lines of idle slots are zero.
  const int NL = 6 * G, S = N | 1;  // lines S apart: an odd stride spreads them over the banks
  T* buf0 = reinterpret_cast<T*>(smem_raw);
  T* buf1 = buf0 + NL * S;
  T* tw = buf1 + NL * S;
  int4* rows = reinterpret_cast<int4*>(smem_raw + xgreen_rows_offset(N, G, int(sizeof(T))));
  const int npair = NN / 2 + 2;
  const FastDiv dn(N);
  // one descriptor per (slot g, row q), index 2 g + q: x = the row's (kz, ky) packed with
  // bit 31 set (0: no row), y, z = LDS offsets of its line and of its partner's line
  // (component 0), w = the row's index in the grid (-1: none)
  for (int i = threadIdx.x; i < 2 * G; i += blockDim.x) {
    const int g = i >> 1, q = i & 1, pn = bx_ * G + g;
    int4 v = make_int4(0, 0, 0, -1);
    if (pn < npair) {
      const int r = green_row(pn, N);
      int kz, ky;
      dn.divmod(r, kz, ky);
      const int rp = (kz ? N - kz : 0) * N + (ky ? N - ky : 0);  // the row of (-kz, -ky)
      if (q == 0 || rp != r) {
        if (q) dn.divmod(rp, kz, ky);
        const int qm = rp == r ? 0 : 1 - q;
        v.x = int(0x80000000u | (unsigned(kz) << 15) | unsigned(ky));
        v.y = (6 * g + q) * S;
        v.z = (6 * g + qm) * S;
        v.w = q ? rp : r;
      }
    }
    rows[i] = v;
  }
  load_twiddles(tw, reinterpret_cast<const T*>(twiddle), N, -1);
  __syncthreads();
  staged_copy<8, T>(
      NL * N,
      [&](int t) {
        int line, x;
        dn.divmod(t, line, x);
        const int g = line / 6, c = (line % 6) >> 1, q = line & 1;
        const int row = rows[2 * g + q].w;
        T v;
        v.x = 0;
        v.y = 0;
        if (row >= 0) ldg2(grid, unsigned(c * cs) + 2 * unsigned(row * N + x), v.x, v.y);
        return v;
      },
      [&](int t, const T& v) {
        int line, x;
        dn.divmod(t, line, x);
        buf0[line * S + x] = v;
      });
  __syncthreads();
  T* X = stockham_lm<T, R>(buf0, buf1, tw, N, S, NL, plan, -1);
  T* O = (X == buf0) ? buf1 : buf0;
  const double gam = (!TABLE && wp.gam) ? *wp.gam : 0.0;
  // items (row 2 g + q, x mode kx), kx fastest; each thread steps blockDim.x items at a time
  int gq, kx;
  dn.divmod(int(threadIdx.x), gq, kx);
  const int dq = int(blockDim.x) / N, dr = int(blockDim.x) - dq * N;
  for (; gq < 2 * G; gq += dq, kx += dr) {
    if (kx >= N) {
      kx -= N;
      if (++gq >= 2 * G) break;
    }
    const int4 ri = rows[gq];
    if (ri.x >= 0) continue;  // no row
    const int kz = (ri.x >> 15) & 0x7fff, ky = ri.x & 0x7fff;
    const int kxm = kx ? N - kx : 0;
    const int o = ri.y + kx, om = ri.z + kxm;  // this mode and its (-k) partner, component 0
    const bool nyq = (N % 2 == 0) && (kx == N / 2 || ky == N / 2 || kz == N / 2);
    if (nyq || (kx == 0 && ky == 0 && kz == 0)) {
      for (int c = 0; c < 3; ++c) {
        O[o + 2 * c * S].x = 0;
        O[o + 2 * c * S].y = 0;
      }
      continue;
    }
    T a[3], m[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      a[c] = X[o + 2 * c * S];
      m[c] = X[om + 2 * c * S];
    }
    green_mode<R, TABLE>(wp, N, kx <= N / 2 ? kx : kx - N, ky <= N / 2 ? ky : ky - N, kz <= N / 2 ? kz : kz - N, gam, a,
                         m);
#pragma unroll
    for (int c = 0; c < 3; ++c) O[o + 2 * c * S] = a[c];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < N; t += blockDim.x) tw[t].y = -tw[t].y;
  __syncthreads();
  const T* Y = stockham_lm<T, R>(O, X, tw, N, S, NL, plan, +1);
  for (int t = threadIdx.x; t < NL * N; t += blockDim.x) {
    int line, x;
    dn.divmod(t, line, x);
    const int g = line / 6, c = (line % 6) >> 1, q = line & 1;
    const int row = rows[2 * g + q].w;
    if (row < 0) continue;
    const T y = Y[line * S + x];
    stg2(grid, unsigned(c * cs) + 2 * unsigned(row * N + x), y.x, y.y);
  }
}

template <typename R, bool TABLE>
__global__ __launch_bounds__(256) void k_fft_xgreen(R* __restrict__ grid, size_t cs, FftPlan plan,
                                                    const R* __restrict__ twiddle, WaveParams wp, int G,
                                                    const int* __restrict__ skip) {
  fft_xgreen_body<R, TABLE>(grid, cs, plan, twiddle, wp, G, skip, blockIdx.x, blockIdx.y, gridDim.x);
}

// ------------------------------------------------------------------------------------------
// Two-step passes of the sides in fft_regs.hpp.  What bounds a pass: the grid is read and written
// once, and with every stage of a line in LDS (four or five exchanges, a barrier each, addresses
// and twiddles at run time) the passes over FP32 grids were slowed by that, not by memory: 66 us
// for a pass over 148 MB that stays in the last-level cache.  With both steps in registers a
// line crosses LDS once, with one barrier, and half the LDS lets twice the workgroups in; the
// x+Green pass crosses it four times instead of eight, and forms a mode and its partner -k at once.
// Measured, z or y pass and x+Green pass, before and after: 64 systems of 594 MB FP32 in groups
// 329 -> 205 us (5.8 TB/s) and 466 -> 277; 128^3 FP64 33.5 -> 30.5 us (6.6 TB/s) and 67 -> 41, FP32 22
// -> 16.5 and 39 -> 25; 64^3 FP64 7 -> 5.1 and 12.2 -> 7.8; 24^3 FP64 5.4 -> 2.9 and 10.2 -> 4.7 (launch and
// memory latency).  The 3D transform alone at 96^3: 47 -> 31 us.
// ------------------------------------------------------------------------------------------

template <typename R, int N, int DIR, int SIGN>
__global__ __launch_bounds__((LineTile<R, N>::kThreads)) void k_wave_lines(R* __restrict__ grid, size_t cs,
                                                                         const R* __restrict__ twiddle,
                                                                         const int* __restrict__ skip) {
  if (skip && *skip) return;
  extern __shared__ unsigned char smem_raw[];
  lines_body<R, N, DIR, SIGN>(grid + blockIdx.y * cs, twiddle, smem_raw, blockIdx.x);
}

template <int N, int SIGN>
__global__ __launch_bounds__(256) void k_fft_rows(double* __restrict__ grid, const double* __restrict__ twiddle) {
  extern __shared__ unsigned char smem_raw[];
  rows_body<double, N, SIGN>(grid, twiddle, smem_raw, blockIdx.x);
}

template <typename R, int N, bool TABLE>
__global__ __launch_bounds__(256) void k_wave_green(R* __restrict__ grid, const R* __restrict__ twiddle, WaveParams wp,
                                                    const int* __restrict__ skip) {
  if (skip && *skip) return;
  extern __shared__ unsigned char smem_raw[];
  green_body<R, N, TABLE>(grid, twiddle, wp, smem_raw, blockIdx.x);
}

namespace {
template <int N>
constexpr int green_pairs() {
  return N * N / 2 + 2;
}

// the stage's two-step launch, when the side has one
template <typename R, int N>
void launch_two_step(R* grid, const R* twiddle, const WaveParams& wp, int stage, hipStream_t st, const int* skip) {
  constexpr size_t cs = 2 * size_t(N) * N * N;
  if (stage == 2) {
    using G = GreenTile<R, N>;
    constexpr int nblk = (green_pairs<N>() + G::G - 1) / G::G;
    if (wp.gtab && !wp.gam)  // the cube: tabulated multipliers
      launch_k(k_wave_green<R, N, true>, nblk, 256, G::kBytes, st, grid, twiddle, wp, skip);
    else
      launch_k(k_wave_green<R, N, false>, nblk, 256, G::kBytes, st, grid, twiddle, wp, skip);
    return;
  }
  using L = LineTile<R, N>;
  const dim3 g(N * N / L::B, 3);
  switch (stage) {
    case 0: launch_k(k_wave_lines<R, N, 2, -1>, g, L::kThreads, L::kBytes, st, grid, cs, twiddle, skip); break;
    case 1: launch_k(k_wave_lines<R, N, 1, -1>, g, L::kThreads, L::kBytes, st, grid, cs, twiddle, skip); break;
    case 3: launch_k(k_wave_lines<R, N, 1, +1>, g, L::kThreads, L::kBytes, st, grid, cs, twiddle, skip); break;
    default: launch_k(k_wave_lines<R, N, 2, +1>, g, L::kThreads, L::kBytes, st, grid, cs, twiddle, skip); break;
  }
}

template <int N>
void launch_fft3d_two_step(double* grid, const double* twiddle, int sign, hipStream_t st) {
  using L = LineTile<double, N>;
  using Row = RowTile<double, N>;
  constexpr int rows = (N * N + Row::kLines - 1) / Row::kLines;
  const dim3 g(N * N / L::B, 1);
  if (sign < 0) {
    k_fft_rows<N, -1><<<rows, 256, Row::kBytes, st>>>(grid, twiddle);
    k_wave_lines<double, N, 1, -1><<<g, L::kThreads, L::kBytes, st>>>(grid, 0, twiddle, nullptr);
    k_wave_lines<double, N, 2, -1><<<g, L::kThreads, L::kBytes, st>>>(grid, 0, twiddle, nullptr);
  } else {
    k_fft_rows<N, +1><<<rows, 256, Row::kBytes, st>>>(grid, twiddle);
    k_wave_lines<double, N, 1, +1><<<g, L::kThreads, L::kBytes, st>>>(grid, 0, twiddle, nullptr);
    k_wave_lines<double, N, 2, +1><<<g, L::kThreads, L::kBytes, st>>>(grid, 0, twiddle, nullptr);
  }
}

}  // namespace

template <typename R>
void launch_fft3d(R* grid, int ncomp, size_t comp_stride, const FftPlan& plan, const R* twiddle, int sign,
                  hipStream_t st, int pass, const int* skip) {
  using T = typename C2<R>::T;
  const int N = plan.n;
  if (std::is_same<R, double>::value && ncomp == 1 && pass < 0 && !skip) {
    switch (N) {
#define X(N_) \
  case N_: launch_fft3d_two_step<N_>(reinterpret_cast<double*>(grid), reinterpret_cast<const double*>(twiddle), sign, st); return;
      FSD_WAVE_SIDES(X)
      FSD_OTHER_SIDES(X)
#undef X
    }
  }
  const int B = lines_per_block(N);
  const size_t shm = sizeof(T) * (2 * size_t(B) * fft_line_stride(N, B, int(sizeof(T))) + N);
  dim3 g(N * N / B, ncomp);
  if (pass < 0 || pass == 0) k_fft_pass<R, 0><<<g, kThreads, shm, st>>>(grid, comp_stride, plan, twiddle, sign, B, skip);
  if (pass < 0 || pass == 1) k_fft_pass<R, 1><<<g, kThreads, shm, st>>>(grid, comp_stride, plan, twiddle, sign, B, skip);
  if (pass < 0 || pass == 2) k_fft_pass<R, 2><<<g, kThreads, shm, st>>>(grid, comp_stride, plan, twiddle, sign, B, skip);
}

template <typename R>
void launch_wave_fft(R* grid, const FftPlan& plan, const R* twiddle, const WaveParams& wp, int stage,
                     hipStream_t st, const int* skip) {
  using T = typename C2<R>::T;
  const int N = plan.n;
  const size_t cs = 2 * size_t(N) * N * N;
  const FftTile tile = stage == 2 ? green_tile(N, wp.tile_g, sizeof(R)) : line_tile(N, wp.tile_b, sizeof(R));
  if (tile.two_step) {
    switch (N) {
#define X(N_) \
  case N_: launch_two_step<R, N_>(grid, twiddle, wp, stage, st, skip); return;
      FSD_WAVE_SIDES(X)
#undef X
    }
  }
  if (stage == 2) {
    const int G = tile.size;
    const size_t shm = xgreen_shm(N, G, int(sizeof(T)));
    const int nblk = (N * N / 2 + 2 + G - 1) / G;
    if (wp.gtab && !wp.gam)  // the cube: tabulated multipliers
      launch_k(k_fft_xgreen<R, true>, nblk, kThreads, shm, st, grid, cs, plan, twiddle, wp, G, skip);
    else
      launch_k(k_fft_xgreen<R, false>, nblk, kThreads, shm, st, grid, cs, plan, twiddle, wp, G, skip);
  } else {
    const int B = tile.size;
    const size_t shm = sizeof(T) * (2 * size_t(B) * fft_line_stride(N, B, int(sizeof(T))) + N);
    dim3 g(N * N / B, 3);
    const int sign = stage < 2 ? -1 : +1;
    if (stage == 0 || stage == 4)
      launch_k(k_fft_lines<R, 2>, g, kThreads, shm, st, grid, cs, plan, twiddle, sign, B, skip);
    else
      launch_k(k_fft_lines<R, 1>, g, kThreads, shm, st, grid, cs, plan, twiddle, sign, B, skip);
  }
}

// ------------------------------------------------------------------------------------------
// multi-system launches
// ------------------------------------------------------------------------------------------

template <typename R, int STAGE>
__global__ __launch_bounds__(256) void kb_fft(const BatchDesc* __restrict__ D, const int* __restrict__ off,
                                             int nsys) {
  const int s = batch_system(off, nsys, blockIdx.x);
  const BatchDesc& d = D[s];
  const int lb = blockIdx.x - off[s];
  const int N = d.plan.n;
  const size_t cs = 2 * size_t(N) * N * N;
  R* grid = static_cast<R*>(d.grid);
  const R* tw = pick<R>(d.tw64, d.tw32);
  const int* stop = &d.ctl->stop;
  extern __shared__ unsigned char smem_raw[];
  if (STAGE == 2 ? d.bg == 0 : d.bl == 0) {  // two-step passes (multi-system launches hold cubic systems only)
    if (*stop) return;
    switch (N) {
#define X(N_)                                                                                                      \
  case N_:                                                                                                         \
    if constexpr (STAGE == 2) {                                                                                    \
      green_body<R, N_, true>(grid, tw, d.wp, smem_raw, lb);                                                       \
    } else {                                                                                                       \
      constexpr int per = N_ * N_ / LineTile<R, N_>::B;                                                            \
      lines_body<R, N_, (STAGE == 0 || STAGE == 4) ? 2 : 1, STAGE < 2 ? -1 : +1>(grid + (lb / per) * cs, tw, smem_raw, \
                                                                                 lb % per);                        \
    }                                                                                                              \
    return;
      FSD_WAVE_SIDES(X)
#undef X
    }
    return;
  }
  if (STAGE == 2) {
    fft_xgreen_body<R, true>(grid, cs, d.plan, tw, d.wp, d.bg, stop, lb, 0, 0);
  } else {
    const int gx = N * N / d.bl;
    if (STAGE == 0 || STAGE == 4)
      fft_lines_body<R, 2>(grid, cs, d.plan, tw, STAGE == 0 ? -1 : +1, d.bl, stop, lb % gx, lb / gx, gx);
    else
      fft_lines_body<R, 1>(grid, cs, d.plan, tw, STAGE == 1 ? -1 : +1, d.bl, stop, lb % gx, lb / gx, gx);
  }
}

int batch_fft_blocks(const BatchDesc& d, int kind, int prec) {
  const int N = d.plan.n;
  if (kind == BK_FFT_GREEN) {
    const int G = d.bg ? d.bg : two_step_pairs(N);
    return (N * N / 2 + 2 + G - 1) / G;
  }
  return N * N / (d.bl ? d.bl : two_step_lines(N, prec ? 4 : 8)) * 3;
}

size_t batch_fft_shm(const BatchDesc& d, int kind, int prec) {
  const int N = d.plan.n, tb = prec ? 8 : 16;
  if (kind == BK_FFT_GREEN ? d.bg == 0 : d.bl == 0) {
    switch (N) {
#define X(N_)                                                                                        \
  case N_:                                                                                           \
    if (kind == BK_FFT_GREEN) return prec ? GreenTile<float, N_>::kBytes : GreenTile<double, N_>::kBytes; \
    return prec ? LineTile<float, N_>::kBytes : LineTile<double, N_>::kBytes;
      FSD_WAVE_SIDES(X)
#undef X
    }
  }
  if (kind == BK_FFT_GREEN) return xgreen_shm(N, d.bg, tb);
  return tb * (2 * size_t(d.bl) * fft_line_stride(N, d.bl, tb) + N);
}

namespace {
template <typename R>
void batch_fft(int stage, const BatchDesc* D, const int* off, int nsys, int total, size_t shm, hipStream_t st) {
  switch (stage) {
    case 0: kb_fft<R, 0><<<total, kThreads, shm, st>>>(D, off, nsys); break;
    case 1: kb_fft<R, 1><<<total, kThreads, shm, st>>>(D, off, nsys); break;
    case 2: kb_fft<R, 2><<<total, kThreads, shm, st>>>(D, off, nsys); break;
    case 3: kb_fft<R, 3><<<total, kThreads, shm, st>>>(D, off, nsys); break;
    default: kb_fft<R, 4><<<total, kThreads, shm, st>>>(D, off, nsys); break;
  }
}
}  // namespace

void launch_batch_fft(int prec, int stage, const BatchDesc* D, const int* off, int nsys, int total, size_t shm,
                      hipStream_t st) {
  if (prec)
    batch_fft<float>(stage, D, off, nsys, total, shm, st);
  else
    batch_fft<double>(stage, D, off, nsys, total, shm, st);
}

template void launch_wave_fft<double>(double*, const FftPlan&, const double*, const WaveParams&, int, hipStream_t,
                                      const int*);
template void launch_wave_fft<float>(float*, const FftPlan&, const float*, const WaveParams&, int, hipStream_t,
                                     const int*);

// ------------------------------------------------------------------------------------------
// the allocation-free transform (fsd_fft3d_noalloc): its twiddle table lives in file-scope
// device memory, one copy per GPU held until the process ends, sized for the largest n
// ------------------------------------------------------------------------------------------

static __device__ __align__(256) double scratch[2 * kNoAllocFftMax];

// exp(-2 pi i t / n) for t < n, interleaved (re, im)
__global__ void k_twiddles(int n, double* __restrict__ tw) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  double sv, cv;
  sincospi(2.0 * double(t) / double(n), &sv, &cv);
  tw[2 * t] = cv;
  tw[2 * t + 1] = -sv;
}

namespace {
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {nullptr};
}  // namespace

// the device address of this GPU's copy of `scratch`, looked up once per device
hipError_t noalloc_scratch(double** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_fft3d_noalloc(int n, int sign, double* data, const FftPlan& plan, hipStream_t st) {
  double* tw = nullptr;
  hipError_t e = noalloc_scratch(&tw);
  if (e != hipSuccess) return e;
  k_twiddles<<<(n + 255) / 256, 256, 0, st>>>(n, tw);
  launch_fft3d<double>(data, 1, 2 * size_t(n) * n * n, plan, tw, sign, st);
  return hipGetLastError();
}

template void launch_fft3d<double>(double*, int, size_t, const FftPlan&, const double*, int, hipStream_t, int, const int*);

}  // namespace fsd
