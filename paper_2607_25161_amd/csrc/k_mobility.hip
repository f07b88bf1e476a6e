// Far-field mobility M = M_real + M_wave of the positively split Ewald sum.
//
// Wave space (spectral Ewald, Gaussian spreading): bead (force, torque) are
// spread to three complex grids Z_c = F_c + i T_c (c = x, y, z), transformed,
// multiplied by the Hasimoto-damped FT-RPY Green's function, transformed back
// and interpolated to the beads, where the grid holds u_c + i w_c.
//
// Real space: per neighbour pair within the cutoff, the free-space RPY block
// minus the smooth inverse transform of the damped multiplier, held as
// piecewise polynomials of the distance.
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <type_traits>

#include "interp_choice.hpp"
#include "k_common.hpp"
#include "k_rigid.hpp"

namespace fsd {

namespace {
constexpr int kThreads = 256;
constexpr int kMaxP = 21;  // 3 * P weights computed by one 64-lane wavefront
inline int nblocks(long long n, int t = kThreads) { return int((n + t - 1) / t); }

// Workgroups are dealt to the 8 XCDs round robin; map workgroup b of nblk so that each
// XCD gets one contiguous range of logical blocks (neighbouring beads or grid blocks
// then share that XCD's L2).  A bijection on [0, nblk).
__device__ inline int xcd_remap(int b, int nblk) {
  const int q = nblk >> 3, r = nblk & 7, x = b & 7, k = b >> 3;
  return x * q + min(x, r) + k;
}

template <typename R>
__device__ inline R wave_sum(R v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
}  // namespace

// Gather-spreading plan: beads binned by the grid block holding the first point of
// their support, in sorted order with their support starts and weights.  On the cube a bead has
// P weights per axis; on a sheared lattice (8^3 blocks only) every grid row in y has its own
// window along x, so it has P x P weights of its (y, x) points, the row's x start, and P along z.
struct SpreadPlan {
  int nb = 0, BS = 0, nbin = 0, K = 0, P = 0;
  bool sheared = false;
  int wlen = 0;  // weights per bead: 3 P, or P P + P
  int *keys_in = nullptr, *keys_out = nullptr, *vals_in = nullptr, *perm = nullptr;
  int *bin_start = nullptr, *bin_end = nullptr;  // 4^3 blocks only
  // 8^3 blocks: for every block, a record of exactly the beads whose support reaches it
  // (cand[blk_start[b] .. blk_end[b]), in bead order): sorted index, bead, and the offsets of the
  // block's first point from the support's start, mod N, 8 bits an axis.  Each bead files kcx kc^2
  // slots (its blocks, then sentinels) that one stable sort groups by block
  int kc = 0, kcx = 0;
  int *blk_start = nullptr, *blk_end = nullptr, *pk_in = nullptr, *pk_out = nullptr, *pv_in = nullptr,
      *pv_out = nullptr;
  int4* cand = nullptr;
  int* where = nullptr;     // place in cand of every slot of sorted bead k (-1: unused), kcx kc^2 each
  // one allocation: the sort's keys, values and temporary storage while the plan is built, later
  // interpolation's six sums of every place in cand
  void* scratch = nullptr;
  void* ptemp = nullptr;
  size_t ptemp_bytes = 0;
  int4* starts = nullptr;   // (sx, sy, sz, bin) per bead, sorted order
  short* rows = nullptr;    // sheared: x start of each of the P grid rows, sorted order
  double* weights = nullptr;  // wlen weights per bead, sorted order
  float* weights32 = nullptr;  // the same in FP32
  void* temp = nullptr;
  size_t temp_bytes = 0;
};

// ------------------------------------------------------------------------------------------
// real-space pair sum: one group of LPR lanes per bead row
// ------------------------------------------------------------------------------------------

// Takes the smooth part of a pair, five scalars as piecewise polynomials of the distance (RealPoly), from
// its free-space functions v: interval q = int(r inv_w) (the last one at most), x = r inv_w - q - 1/2, Horner
// from the highest coefficient, the constant one straight from v (both are close there, so their difference has
// little rounding).  T points at the coefficients in LDS, read in 16-byte pieces; rows are an odd number of pieces
// apart, so that lanes at different distances meet different banks (an even number, 18, left FP64 half of
// the banks: 163 us instead of 154 at 81,920 beads).
template <typename R>
__device__ __forceinline__ void less_smooth_part(const R* T, R r, R inv_w, int last, R (&v)[5]) {
  using P = RealPoly<R>;
  const R u = r * inv_w;
  const int q = min(int(u), last);  // r < r_cut up to rounding
  const R x = u - R(q) - R(0.5);
  typedef R V __attribute__((ext_vector_type(16 / sizeof(R))));
  constexpr int L = 16 / sizeof(R);
  const V* row = reinterpret_cast<const V*>(T + q * P::kStride);
  V c[(5 * P::kCoef + L - 1) / L];
#pragma unroll
  for (int k = 0; k < int(sizeof(c) / sizeof(V)); ++k) c[k] = row[k];
  const auto at = [&](int i) { return c[i / L][i % L]; };
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    R p = at(k * P::kCoef);
#pragma unroll
    for (int m = 1; m < P::kCoef - 1; ++m) p = p * x + at(k * P::kCoef + m);
    v[k] = (v[k] - at(k * P::kCoef + P::kCoef - 1)) - p * x;
  }
}

// 1 / sqrt(r2) and sqrt(r2).  In FP32 to the last place: the hardware's estimate is off by up to one, and it enters
// the functions three times over.  The FP32 sum against the FP64 one, 300 to 30,000 beads: off by 2.5 to 2.9e-7 of its
// size with the plain estimate, c8 and the interval factor rounded and multiplied in, and the smooth part rounded
// before it is subtracted; by 1.4 to 1.5e-7 as it is (1.75 to 2.1e-7 with square roots, divisions and a table).
__device__ __forceinline__ void root(float r2, float& r, float& ir) {
  ir = rsqrtf(r2);
  r = r2 * ir;
  r = __builtin_fmaf(__builtin_fmaf(-r, r, r2), 0.5f * ir, r);
  ir = __builtin_fmaf(ir, __builtin_fmaf(-r, ir, 1.0f), ir);
}
__device__ __forceinline__ void root(double r2, double& r, double& ir) {
  ir = rsqrt(r2);
  r = r2 * ir;
}

// Out of the pair's separation vector d itself, with no unit vector and no division:
//   u += (tI + ..) f + B (d.f) d + C d x t,   w += rI t + rB (d.t) d + C d x f.
// What bounds it: per pair the position (32 B) and the force moments (48 B) are gathered, one
// cache line a lane.  The smooth part was gathered as well, four rows of a 262 KB table in L2,
// 12 of the 17 loads of a pair: at 15.5 million pairs (81,920 beads) 367 us in FP64 and 230 in
// FP32, the rate at which a CU looks up cache lines.  As 64 intervals of degree 6 (FP64) or 128
// of degree 3 (FP32) it is 18 or 10 KB that every workgroup copies to LDS, and is closer to the
// quadrature than the table was (2e-15 of the self mobility against 3e-14): with 32 lanes a row 140 us in FP64
// (with four wavefronts a SIMD; 154 with the three that its registers would leave) and 112 in FP32,
// with 16 132 and 108.  A workgroup takes a contiguous chunk of rows, in the plan's spatial order
// where there is one, so that the copy is paid once per many rows.
template <typename R, int LPR>
__device__ __forceinline__ void real_sum_body(int nb, const double4* __restrict__ pos,
                                              const double* __restrict__ lam, const int* __restrict__ rowptr,
                                              const uint32_t* __restrict__ col, const R* __restrict__ tab,
                                              const RealParams& rp, double* __restrict__ out, int accumulate,
                                              const int* __restrict__ order, const int* __restrict__ skip,
                                              unsigned char* smem, int bx, int nblk) {
  if (skip && *skip) return;
  using P = RealPoly<R>;
  R* T = reinterpret_cast<R*>(smem);
  {
    typedef R V __attribute__((ext_vector_type(16 / sizeof(R))));
    constexpr int NV = P::kIntervals * P::kStride * int(sizeof(R)) / 16;
    for (int h = 0; h < rp.fine; ++h)  // NV at a time: a constant count keeps all the loads in flight
      for (int k = threadIdx.x; k < NV; k += kThreads)
        reinterpret_cast<V*>(T)[h * NV + k] = reinterpret_cast<const V*>(tab)[h * NV + k];
  }
  __syncthreads();
  constexpr int kGroups = kThreads / LPR;
  int chunk = (nb + nblk - 1) / nblk;
  if (chunk > kGroups) chunk = (chunk + kGroups - 1) / kGroups * kGroups;  // whole passes
  const int lb = order ? xcd_remap(bx, nblk) : bx;  // with an order, each XCD takes one contiguous range
  const int r_end = min(nb, (lb + 1) * chunk), lane = threadIdx.x % LPR;
  // the functions are in units of c8 = 1 / (8 pi eta), which multiplies the sums in FP64
  const R a = R(rp.a), a2 = a * a, mt = R(rp.mt), mr = R(rp.mr);
  const double c8 = rp.c8;
  const int last = rp.fine * P::kIntervals - 1;
  const R inv_w = R(rp.inv_w) * R(rp.fine * P::kIntervals);
  const R touch = R(4) * a2;
  const double gam = rp.gam ? *rp.gam : 0.0;
  for (int rl = lb * chunk + int(threadIdx.x) / LPR; rl < r_end; rl += kGroups) {
    const int row = order ? order[rl] : rl;
    const double4 pi = pos[row];
    R u0 = 0, u1 = 0, u2 = 0, w0 = 0, w1 = 0, w2 = 0;
    const int e1 = rowptr[row + 1];
    for (int e = rowptr[row] + lane; e < e1; e += LPR) {
      const uint32_t c = col[e];
      const int j = int(c & 0x3FFFFFu);
      const double4 pj = pos[j];
      const double* lj = lam + 6 * size_t(j);
      const R fx = R(lj[0]), fy = R(lj[1]), fz = R(lj[2]);
      const R tx = R(lj[3]), ty = R(lj[4]), tz = R(lj[5]);
      const double dyd = pi.y - pj.y + (int((c >> 25) & 7u) - 3) * rp.L;  // Cartesian from sheared
      const R dx = R(pi.x - pj.x + (int((c >> 22) & 7u) - 3) * rp.L + gam * dyd);
      const R dy = R(dyd);
      const R dz = R(pi.z - pj.z + (int((c >> 28) & 7u) - 3) * rp.L);
      const R r2 = dx * dx + dy * dy + dz * dz;
      R r, ir;
      root(r2, r, ir);
      const R ir2 = ir * ir, ir3 = ir * ir2;
      // free-space force-torque RPY; C, tB and rB are the rt, tt and rr functions over r, r^2, r^2
      R f[5];
      if (r2 >= touch) {
        f[0] = ir * (R(1) + R(2.0 / 3.0) * a2 * ir2);
        f[1] = ir3 * (R(1) - R(2) * a2 * ir2);
        f[2] = R(-0.5) * ir3;
        f[3] = R(1.5) * ir3 * ir2;
        f[4] = -ir3;
      } else {  // overlapping spheres
        const R s = r / a;
        f[0] = mt * (R(1) - R(9.0 / 32.0) * s);
        f[1] = mt * R(3.0 / 32.0) * s * ir2;
        f[2] = mr * (R(1) - R(27.0 / 32.0) * s + R(5.0 / 64.0) * s * s * s);
        f[3] = mr * (R(9.0 / 32.0) * s - R(3.0 / 64.0) * s * s * s) * ir2;
        f[4] = -R(0.5) * mr * (R(1) - R(3.0 / 8.0) * s);
      }
      less_smooth_part<R>(T, r, inv_w, last, f);
      const R tI = f[0], tB = f[1], rI = f[2], rB = f[3], cc = f[4];
      const R fd = tB * (dx * fx + dy * fy + dz * fz), td = rB * (dx * tx + dy * ty + dz * tz);
      u0 += tI * fx + fd * dx + cc * (dy * tz - dz * ty);
      u1 += tI * fy + fd * dy + cc * (dz * tx - dx * tz);
      u2 += tI * fz + fd * dz + cc * (dx * ty - dy * tx);
      w0 += rI * tx + td * dx + cc * (dy * fz - dz * fy);
      w1 += rI * ty + td * dy + cc * (dz * fx - dx * fz);
      w2 += rI * tz + td * dz + cc * (dx * fy - dy * fx);
    }
    // the first exchange leaves the velocity with the lower half of the lanes and the angular
    // velocity with the upper one, so the others move three values instead of six
    bool up = false;
    if (LPR > 1) {
      up = lane & (LPR / 2);
      const R s0 = up ? u0 : w0, s1 = up ? u1 : w1, s2 = up ? u2 : w2;
      u0 = (up ? w0 : u0) + __shfl_xor(s0, LPR / 2, LPR);
      u1 = (up ? w1 : u1) + __shfl_xor(s1, LPR / 2, LPR);
      u2 = (up ? w2 : u2) + __shfl_xor(s2, LPR / 2, LPR);
#pragma unroll
      for (int o = LPR / 4; o >= 1; o >>= 1) {
        u0 += __shfl_xor(u0, o, LPR);
        u1 += __shfl_xor(u1, o, LPR);
        u2 += __shfl_xor(u2, o, LPR);
      }
    }
    if (LPR == 1 || (lane & (LPR / 2 - 1)) == 0) {
      const int h = up ? 3 : 0;
      const double* li = lam + 6 * size_t(row) + h;
      double* o = out + 6 * size_t(row) + h;
      const double self = up ? rp.self_r : rp.self_t;
      double v[6] = {c8 * u0 + self * li[0], c8 * u1 + self * li[1], c8 * u2 + self * li[2], 0, 0, 0};
      if (LPR == 1) {
        v[3] = c8 * w0 + rp.self_r * li[3];
        v[4] = c8 * w1 + rp.self_r * li[4];
        v[5] = c8 * w2 + rp.self_r * li[5];
      }
      for (int k = 0; k < (LPR == 1 ? 6 : 3); ++k) o[k] = accumulate ? o[k] + v[k] : v[k];
    }
  }
}

template <typename R, int LPR>
__global__ __launch_bounds__(256, 4) void k_real_sum(int nb, const double4* __restrict__ pos,
                                                  const double* __restrict__ lam, const int* __restrict__ rowptr,
                                                  const uint32_t* __restrict__ col, const R* __restrict__ tab,
                                                  RealParams rp, double* __restrict__ out, int accumulate,
                                                  const int* __restrict__ order, const int* __restrict__ skip) {
  extern __shared__ unsigned char smem_raw[];
  real_sum_body<R, LPR>(nb, pos, lam, rowptr, col, tab, rp, out, accumulate, order, skip, smem_raw, blockIdx.x,
                        gridDim.x);
}

namespace {
// Workgroups of a real-space sum over nb rows: one pass of 256 / LPR rows each up to
// kRealBlocks, so that small systems spread over the CUs; beyond it each takes more rows
// (twelve workgroups a CU hide the gathers, and the copy of the coefficients is paid 3,072 times)
constexpr int kRealBlocks = 3072;
inline int real_blocks(long long nb, int lpr) {
  return int(std::min<long long>((nb * lpr + kThreads - 1) / kThreads, kRealBlocks));
}
}  // namespace

template <typename R>
void launch_real_sum(int nb, const double* pos4, const double* lam, const int* rowptr, const uint32_t* col,
                     const R* table, const RealParams& rp, double* out, bool accumulate, int lpr, hipStream_t st,
                     const int* skip, const int* order) {
  const int acc = accumulate ? 1 : 0;
  const double4* p = (const double4*)pos4;
#define FSD_REAL(L_)                                                                                    \
  launch_k(k_real_sum<R, L_>, real_blocks(nb, L_), kThreads, RealPoly<R>::bytes(rp.fine), st, nb, p, lam, rowptr, col, table, rp, out, acc, order, skip)
  switch (lpr) {
    case 1: FSD_REAL(1); break;
    case 2: FSD_REAL(2); break;
    case 4: FSD_REAL(4); break;
    case 8: FSD_REAL(8); break;
    case 16: FSD_REAL(16); break;
    case 32: FSD_REAL(32); break;
    default: FSD_REAL(64); break;
  }
#undef FSD_REAL
}

// ------------------------------------------------------------------------------------------
// Gaussian spreading and interpolation: one wavefront per bead
// ------------------------------------------------------------------------------------------

namespace {
// 1D weights exp(-alpha (x_m - p)^2) for the P support points of each axis.
template <typename R>
__device__ inline void axis_weights(const double4& p, const WaveParams& wp, int lane, R* w, int* st) {
  const int P = wp.support;
  if (lane < 3 * P) {
    const int d = lane / P, k = lane % P;
    const double pd = d == 0 ? p.x : (d == 1 ? p.y : p.z);
    const double u = pd / wp.h;
    const int s = int(ceil(u - 0.5 * P));
    const double xm = (s + k) * wp.h - pd;
    w[d * kMaxP + k] = R(exp(-wp.alpha * xm * xm));
    if (k == 0) st[d] = s;
  }
}

__device__ inline int wrapi(int m, int n) {
  m %= n;
  return m < 0 ? m + n : m;
}
}  // namespace

template <typename R>
__global__ __launch_bounds__(256) void k_spread(int nb, const double4* __restrict__ pos,
                                                const double* __restrict__ lam, WaveParams wp, R* __restrict__ grid,
                                                size_t cs, const int* __restrict__ skip) {
  if (skip && *skip) return;
  __shared__ R wts[4][3 * kMaxP];
  __shared__ int sta[4][3];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + wv;
  const bool live = i < nb;
  const double4 p = live ? pos[i] : make_double4(0, 0, 0, 0);
  if (live) axis_weights<R>(p, wp, lane, wts[wv], sta[wv]);
  __syncthreads();
  if (!live) return;
  const int P = wp.support, N = wp.n;
  const double* li = lam + 6 * i;
  const R f0 = R(li[0]), f1 = R(li[1]), f2 = R(li[2]);
  const R t0 = R(li[3]), t1 = R(li[4]), t2 = R(li[5]);
  const int sx = sta[wv][0], sy = sta[wv][1], sz = sta[wv][2];
  const R* wx = wts[wv];
  const R* wy = wts[wv] + kMaxP;
  const R* wz = wts[wv] + 2 * kMaxP;
  const int P3 = P * P * P;
  for (int idx = lane; idx < P3; idx += 64) {
    const int kx = idx % P, ky = (idx / P) % P, kz = idx / (P * P);
    const R w = wx[kx] * wy[ky] * wz[kz];
    const size_t m = (size_t(wrapi(sz + kz, N)) * N + wrapi(sy + ky, N)) * N + wrapi(sx + kx, N);
    R* g = grid + 2 * m;
    atomicAdd(g, w * f0);
    atomicAdd(g + 1, w * t0);
    atomicAdd(g + cs, w * f1);
    atomicAdd(g + cs + 1, w * t1);
    atomicAdd(g + 2 * cs, w * f2);
    atomicAdd(g + 2 * cs + 1, w * t2);
  }
}

template <typename R>
void launch_spread(int nb, const double* pos4, const double* lam, const WaveParams& wp, R* grid, hipStream_t st,
                   const int* skip) {
  const size_t cs = 2 * size_t(wp.n) * wp.n * wp.n;
  launch_k(k_spread<R>, nblocks(nb, 4), kThreads, 0, st, nb, (const double4*)pos4, lam, wp, grid, cs, skip);
}

// ---- sheared lattice: one wavefront per bead, grid row j shifted along x -------------------
namespace {
// Weights of bead p in sheared coordinates: y and z as on the cube; for each of the P rows
// ky the start sxr[ky] and P x-weights, centred at p_x - gam (y_m - p_y), y_m = (sy + ky) h.
template <typename R>
__device__ inline void sheared_weights(const double4& p, const WaveParams& wp, int lane, R* wyz, int* st, R* wxr,
                                       int* sxr) {
  const int P = wp.support;
  const double h = wp.h, gam = wp.gam ? *wp.gam : 0.0;
  const int sy = int(ceil(p.y / h - 0.5 * P)), sz = int(ceil(p.z / h - 0.5 * P));
  if (lane < 2 * P) {
    const int d = lane / P, k = lane % P;
    const double xm = d == 0 ? (sy + k) * h - p.y : (sz + k) * h - p.z;
    wyz[d * kMaxP + k] = R(exp(-wp.alpha * xm * xm));
  }
  if (lane == 0) {
    st[0] = sy;
    st[1] = sz;
  }
  for (int t = lane; t < P * P; t += 64) {
    const int ky = t / P, kx = t - ky * P;
    const double cx = p.x - gam * ((sy + ky) * h - p.y);  // the row's centre along x
    const int sx = int(ceil(cx / h - 0.5 * P));
    const double xm = (sx + kx) * h - cx;
    wxr[ky * kMaxP + kx] = R(exp(-wp.alpha * xm * xm));
    if (kx == 0) sxr[ky] = sx;
  }
}
}  // namespace

template <typename R>
__global__ __launch_bounds__(256) void k_spread_sheared(int nb, const double4* __restrict__ pos,
                                                        const double* __restrict__ lam, WaveParams wp,
                                                        R* __restrict__ grid, size_t cs, const int* __restrict__ skip) {
  if (skip && *skip) return;
  __shared__ R wyz[4][2 * kMaxP];
  __shared__ R wxr[4][kMaxP * kMaxP];
  __shared__ int sxr[4][kMaxP];
  __shared__ int sta[4][2];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + wv;
  const bool live = i < nb;
  if (live) sheared_weights<R>(pos[i], wp, lane, wyz[wv], sta[wv], wxr[wv], sxr[wv]);
  __syncthreads();
  if (!live) return;
  const int P = wp.support, N = wp.n;
  const double* li = lam + 6 * i;
  const R f0 = R(li[0]), f1 = R(li[1]), f2 = R(li[2]);
  const R t0 = R(li[3]), t1 = R(li[4]), t2 = R(li[5]);
  const int sy = sta[wv][0], sz = sta[wv][1];
  const int P3 = P * P * P;
  for (int idx = lane; idx < P3; idx += 64) {
    const int kx = idx % P, ky = (idx / P) % P, kz = idx / (P * P);
    const R w = wxr[wv][ky * kMaxP + kx] * wyz[wv][ky] * wyz[wv][kMaxP + kz];
    const size_t m = (size_t(wrapi(sz + kz, N)) * N + wrapi(sy + ky, N)) * N + wrapi(sxr[wv][ky] + kx, N);
    R* g = grid + 2 * m;
    atomicAdd(g, w * f0);
    atomicAdd(g + 1, w * t0);
    atomicAdd(g + cs, w * f1);
    atomicAdd(g + cs + 1, w * t1);
    atomicAdd(g + 2 * cs, w * f2);
    atomicAdd(g + 2 * cs + 1, w * t2);
  }
}

template <typename R>
__global__ __launch_bounds__(256) void k_interp_sheared(int nb, const double4* __restrict__ pos,
                                                        const R* __restrict__ grid, size_t cs, WaveParams wp,
                                                        double* __restrict__ out, const int* __restrict__ skip,
                                                        const int* __restrict__ body, const double4* __restrict__ r4,
                                                        const double* __restrict__ V) {
  if (skip && *skip) return;
  __shared__ R wyz[4][2 * kMaxP];
  __shared__ R wxr[4][kMaxP * kMaxP];
  __shared__ int sxr[4][kMaxP];
  __shared__ int sta[4][2];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + wv;
  const bool live = i < nb;
  if (live) sheared_weights<R>(pos[i], wp, lane, wyz[wv], sta[wv], wxr[wv], sxr[wv]);
  __syncthreads();
  if (!live) return;
  const int P = wp.support, N = wp.n;
  const int sy = sta[wv][0], sz = sta[wv][1];
  R a0 = 0, a1 = 0, a2 = 0, a3 = 0, a4 = 0, a5 = 0;
  for (int pq = lane; pq < P * P; pq += 64) {  // lane -> (kx, ky) column, walking z
    const int ky = pq / P, kx = pq - ky * P;
    const int x = wrapi(sxr[wv][ky] + kx, N), y = wrapi(sy + ky, N);
    const R wxy = wxr[wv][ky * kMaxP + kx] * wyz[wv][ky];
    for (int kz = 0; kz < P; ++kz) {
      const R w = wxy * wyz[wv][kMaxP + kz];
      const R* g = grid + 2 * ((size_t(wrapi(sz + kz, N)) * N + y) * N + x);
      a0 += w * g[0];
      a3 += w * g[1];
      a1 += w * g[cs];
      a4 += w * g[cs + 1];
      a2 += w * g[2 * cs];
      a5 += w * g[2 * cs + 1];
    }
  }
  a0 = wave_sum(a0);
  a1 = wave_sum(a1);
  a2 = wave_sum(a2);
  a3 = wave_sum(a3);
  a4 = wave_sum(a4);
  a5 = wave_sum(a5);
  if (lane == 0) {
    double* o = out + 6 * size_t(i);
    double add[6] = {double(a0), double(a1), double(a2), double(a3), double(a4), double(a5)};
    if (V) {  // Sigma^T V: (U + W x r, W) of the bead's body
      const double* v = V + 6 * body[i];
      const double4 r = r4[i];
      add[0] += v[0] + (v[4] * r.z - v[5] * r.y);
      add[1] += v[1] + (v[5] * r.x - v[3] * r.z);
      add[2] += v[2] + (v[3] * r.y - v[4] * r.x);
      add[3] += v[3];
      add[4] += v[4];
      add[5] += v[5];
    }
    for (int k = 0; k < 6; ++k) o[k] += add[k];
  }
}

template <typename R>
void launch_spread_sheared(int nb, const double* pos4, const double* lam, const WaveParams& wp, R* grid,
                           hipStream_t st, const int* skip) {
  const size_t cs = 2 * size_t(wp.n) * wp.n * wp.n;
  launch_k(k_spread_sheared<R>, nblocks(nb, 4), kThreads, 0, st, nb, (const double4*)pos4, lam, wp, grid, cs, skip);
}

template <typename R>
void launch_interp_sheared(int nb, const double* pos4, const R* grid, const WaveParams& wp, double* out,
                           hipStream_t st, const int* skip, const int* body, const double* r4, const double* V) {
  const size_t cs = 2 * size_t(wp.n) * wp.n * wp.n;
  launch_k(k_interp_sheared<R>, nblocks(nb, 4), kThreads, 0, st, nb, (const double4*)pos4, grid, cs, wp, out, skip,
           body, (const double4*)r4, V);
}

// Interpolation on grids without a plan: one wavefront per bead, weights computed here.
template <typename R>
__global__ __launch_bounds__(256) void k_interp(int nb, const double4* __restrict__ pos,
                                                const R* __restrict__ grid, size_t cs, WaveParams wp,
                                                double* __restrict__ out, const int* __restrict__ skip,
                                                const int* __restrict__ body, const double4* __restrict__ r4,
                                                const double* __restrict__ V) {
  if (skip && *skip) return;
  __shared__ R wts[4][3 * kMaxP];
  __shared__ int sta[4][3];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + wv;
  const bool live = i < nb;
  if (live) axis_weights<R>(pos[i], wp, lane, wts[wv], sta[wv]);
  __syncthreads();
  if (!live) return;
  const int P = wp.support, N = wp.n;
  const int sx = sta[wv][0], sy = sta[wv][1], sz = sta[wv][2];
  const R* wx = wts[wv];
  const R* wy = wts[wv] + kMaxP;
  const R* wz = wts[wv] + 2 * kMaxP;
  R a0 = 0, a1 = 0, a2 = 0, a3 = 0, a4 = 0, a5 = 0;
  // lane -> (x pair, ky) of the support, each lane walking its two columns along z: the
  // pairs (2m, 2m + 1) that cover the support's P x values (P/2 + 1 of them at most, the
  // points outside the support weighted 0), so each load brings two grid points in one
  // aligned 16-byte (FP32) or 32-byte (FP64) read; for even N no pair straddles the
  // periodic wrap.  The grid is read through 32-bit offsets from the three component bases
  // (2 N^3 < 2^31 for N <= 256), in two runs split where the columns wrap in z.
  const int sxw = wrapi(sx, N), syw = wrapi(sy, N), szw = wrapi(sz, N);
  const unsigned plane = 2 * N * N;
  const int n1 = min(P, N - szw), half = N >> 1, m0 = sxw >> 1;
  const int npx = ((sxw + P - 1) >> 1) - m0 + 1;
  const R* g0 = grid;
  const R* g1 = grid + cs;
  const R* g2 = grid + 2 * cs;
  // an odd grid side (set by the caller) keeps one column per lane: its pairs would
  // straddle the wrap and lose the alignment.  So does FP64, where the pairs' registers
  // (128 VGPRs against 70) cost more occupancy than the wider loads gain (the 4096x20
  // system: 267 us against 233 per launch)
  const bool paired = sizeof(R) == 4 && !(N & 1);
  for (int pq = lane; !paired && pq < P * P; pq += 64) {
    const int ky = pq / P, kx = pq - ky * P;
    int x = sxw + kx, y = syw + ky;
    x -= x >= N ? N : 0;
    y -= y >= N ? N : 0;
    const R wxy = wx[kx] * wy[ky];
    const unsigned col = 2 * (y * N + x);
    unsigned off = col + szw * plane;
    for (int kz = 0; kz < P; ++kz) {
      if (kz == n1) off = col;
      const R w = wxy * wz[kz];
      R v0, v1, v2, v3, v4, v5;
      ldg2(g0, off, v0, v3);
      ldg2(g1, off, v1, v4);
      ldg2(g2, off, v2, v5);
      a0 += w * v0;
      a3 += w * v3;
      a1 += w * v1;
      a4 += w * v4;
      a2 += w * v2;
      a5 += w * v5;
      off += plane;
    }
  }
  for (int pq = lane; paired && pq < npx * P; pq += 64) {
    const int ky = pq / npx, mp = pq - ky * npx;
    int m = m0 + mp, y = syw + ky;
    m -= m >= half ? half : 0;
    y -= y >= N ? N : 0;
    const int kx0 = 2 * (m0 + mp) - sxw;  // support offset of the pair's first point (>= -1)
    const R wyk = wy[ky];
    const R wp0 = kx0 >= 0 ? wx[kx0] * wyk : R(0);
    const R wp1 = kx0 + 1 < P ? wx[kx0 + 1] * wyk : R(0);
    const unsigned col = 2 * (y * N + 2 * m);
    unsigned off = col + szw * plane;
    for (int kz = 0; kz < P; ++kz) {
      if (kz == n1) off = col;  // the columns wrap to z = 0
      const R w = wz[kz], u0 = wp0 * w, u1 = wp1 * w;
      R b0, b1, b2, b3;
      ldg4(g0, off, b0, b1, b2, b3);
      a0 += u0 * b0 + u1 * b2;
      a3 += u0 * b1 + u1 * b3;
      ldg4(g1, off, b0, b1, b2, b3);
      a1 += u0 * b0 + u1 * b2;
      a4 += u0 * b1 + u1 * b3;
      ldg4(g2, off, b0, b1, b2, b3);
      a2 += u0 * b0 + u1 * b2;
      a5 += u0 * b1 + u1 * b3;
      off += plane;
    }
  }
  a0 = wave_sum(a0);
  a1 = wave_sum(a1);
  a2 = wave_sum(a2);
  a3 = wave_sum(a3);
  a4 = wave_sum(a4);
  a5 = wave_sum(a5);
  if (lane == 0) {
    double* o = out + 6 * size_t(i);
    double add[6] = {double(a0), double(a1), double(a2), double(a3), double(a4), double(a5)};
    if (V) {  // Sigma^T V: (U + W x r, W) of the bead's body
      const double* v = V + 6 * body[i];
      const double4 r = r4[i];
      add[0] += v[0] + (v[4] * r.z - v[5] * r.y);
      add[1] += v[1] + (v[5] * r.x - v[3] * r.z);
      add[2] += v[2] + (v[3] * r.y - v[4] * r.x);
      add[3] += v[3];
      add[4] += v[4];
      add[5] += v[5];
    }
    for (int k = 0; k < 6; ++k) o[k] += add[k];
  }
}

const int* spread_plan_order(const SpreadPlan* sp) { return sp ? sp->perm : nullptr; }

// ------------------------------------------------------------------------------------------
// Gaussian spreading as a gather: beads are binned by the grid block that holds
// the first point of their support (sorted once per configuration); a workgroup
// owns one BS^3 block of grid points and sums the contributions of every bead
// whose support reaches it.  No atomics, deterministic, each grid value written
// once.
// ------------------------------------------------------------------------------------------



namespace {
int pick_block(int N) {
  if (N % 8 == 0) return 8;
  if (N % 4 == 0) return 4;
  return 0;
}

// Sizes of a plan (BS == 0: the grid has none), for its creation and for the memory estimate
struct PlanShape {
  int BS, nbin, K;
  int kc, kcx;         // 8^3 blocks: blocks a support can reach along y and z, and along x
  size_t wlen, slots;  // weights and block slots of a bead
};

PlanShape plan_shape(int N, int P, bool sheared) {
  PlanShape h{};
  h.BS = pick_block(N);
  if (sheared && h.BS != 8) h.BS = 0;
  if (h.BS == 0) return h;
  h.nbin = N / h.BS;
  h.wlen = sheared ? size_t(P) * P + P : size_t(3) * P;
  h.K = std::min(1 + (P - 1 + h.BS - 1) / h.BS, h.nbin);
  if (h.BS == 8) {
    h.kc = h.K;
    // the rows of a sheared support start up to ceil((P - 1) / 2) points apart (|strain| <= 1/2)
    h.kcx = sheared ? std::min(1 + (P + P / 2 - 1 + 7) / 8, h.nbin) : h.kc;
    h.slots = size_t(h.kcx) * h.kc * h.kc;
  }
  return h;
}
}  // namespace

size_t spread_plan_bytes(int nb, int N, int P, bool sheared) {
  const PlanShape h = plan_shape(N, P, sheared);
  if (h.BS == 0) return 0;
  // per bead: four sort arrays, the start, the weights in FP64 and FP32, the rows' starts; per slot: the
  // candidate record, the slot's place, and what spread_plan_create gives the scratch
  const size_t bead = 4 * sizeof(int) + sizeof(int4) + 12 * h.wlen + (sheared ? 2 * P : 0);
  const size_t slot = h.BS == 8 ? sizeof(int4) + sizeof(int) + 6 * sizeof(double) : 0;
  return nb * (bead + slot * h.slots) + sort_pairs_bytes(nb) + 2 * sizeof(int) * size_t(h.nbin) * h.nbin * h.nbin;
}

SpreadPlan* spread_plan_create(int nb, int N, int P, bool sheared) {
  const PlanShape h = plan_shape(N, P, sheared);
  const int BS = h.BS;
  // On a sheared lattice the eight blocks of side 16 (and the one of side 8) gather thousands of beads one
  // after the other; below 11 points a support the scatter is quicker then.  Sheared 16^3, us by gather / scatter,
  // P = 6: 4,096 beads 194 / 93 (FP32 175 / 79), 16,384 891 / 361; P = 10: 1,000 beads 88 / 106 (79 / 89), 4,096 356 /
  // 362 (313 / 268), 16,384 1,624 / 1,458 (1,483 / 1,052); P = 14: 4,096 409 / 893.  Side 24: gather, by 1.4 at least.
  const bool scatter = sheared && N <= 16 && ((P <= 9 && nb >= 512) || (P == 10 && nb >= 2048));
  if (BS == 0 || scatter) return nullptr;
  auto* sp = new SpreadPlan;
  sp->nb = nb;
  sp->BS = BS;
  sp->nbin = h.nbin;
  sp->P = P;
  sp->sheared = sheared;
  sp->wlen = int(h.wlen);
  sp->K = h.K;
  const int nbins = sp->nbin * sp->nbin * sp->nbin;
  const size_t nw = size_t(sp->wlen) * nb;
  bool ok = hipMalloc(&sp->keys_in, sizeof(int) * nb) == hipSuccess &&
            hipMalloc(&sp->keys_out, sizeof(int) * nb) == hipSuccess &&
            hipMalloc(&sp->vals_in, sizeof(int) * nb) == hipSuccess &&
            hipMalloc(&sp->perm, sizeof(int) * nb) == hipSuccess &&
            hipMalloc(&sp->starts, sizeof(int4) * nb) == hipSuccess &&
            hipMalloc(&sp->weights, sizeof(double) * nw) == hipSuccess &&
            hipMalloc(&sp->weights32, sizeof(float) * nw) == hipSuccess;
  if (sheared) ok = ok && hipMalloc(&sp->rows, sizeof(short) * size_t(P) * nb) == hipSuccess;
  size_t b = 0;
  hipcub::DeviceRadixSort::SortPairs(nullptr, b, sp->keys_in, sp->keys_out, sp->vals_in, sp->perm, nb);
  sp->temp_bytes = b;
  ok = ok && hipMalloc(&sp->temp, b) == hipSuccess;
  if (ok && BS == 4) {
    ok = hipMalloc(&sp->bin_start, sizeof(int) * nbins) == hipSuccess &&
         hipMalloc(&sp->bin_end, sizeof(int) * nbins) == hipSuccess;
  }
  if (ok && BS == 8) {
    sp->kc = h.kc;
    sp->kcx = h.kcx;
    const size_t slots = nb * h.slots;
    ok = hipMalloc(&sp->blk_start, sizeof(int) * nbins) == hipSuccess &&
         hipMalloc(&sp->blk_end, sizeof(int) * nbins) == hipSuccess &&
         hipMalloc(&sp->cand, sizeof(int4) * slots) == hipSuccess &&
         hipMalloc(&sp->where, sizeof(int) * slots) == hipSuccess;
    size_t pb = 0;
    hipcub::DeviceRadixSort::SortPairs(nullptr, pb, sp->pk_in, sp->pk_out, sp->pv_in, sp->pv_out, int(slots));
    sp->ptemp_bytes = pb;
    const size_t four = (4 * sizeof(int) * slots + 255) / 256 * 256;
    ok = ok && hipMalloc(&sp->scratch, std::max(four + pb, 6 * sizeof(double) * slots)) == hipSuccess;
    if (ok) {
      sp->pk_in = static_cast<int*>(sp->scratch);
      sp->pk_out = sp->pk_in + slots;
      sp->pv_in = sp->pk_out + slots;
      sp->pv_out = sp->pv_in + slots;
      sp->ptemp = static_cast<char*>(sp->scratch) + four;
    }
  }
  if (!ok) {
    spread_plan_destroy(sp);
    return nullptr;
  }
  return sp;
}

void spread_plan_destroy(SpreadPlan* sp) {
  if (!sp) return;
  (void)hipFree(sp->keys_in);
  (void)hipFree(sp->keys_out);
  (void)hipFree(sp->vals_in);
  (void)hipFree(sp->perm);
  (void)hipFree(sp->bin_start);
  (void)hipFree(sp->bin_end);
  (void)hipFree(sp->starts);
  (void)hipFree(sp->rows);
  (void)hipFree(sp->weights);
  (void)hipFree(sp->weights32);
  (void)hipFree(sp->temp);
  (void)hipFree(sp->blk_start);
  (void)hipFree(sp->blk_end);
  (void)hipFree(sp->cand);
  (void)hipFree(sp->where);
  (void)hipFree(sp->scratch);
  delete sp;
}

namespace {
// First of the P support points around coordinate u (in grid spacings), unwrapped.
__device__ inline int support_start(double u, int P) { return int(ceil(u - 0.5 * P)); }

// offset of point m from the start s of a support, mod N (both in [0, N))
__device__ __forceinline__ int point_offset(int m, int s, int N) {
  const int o = m - s;
  return o < 0 ? o + N : o;
}

// x centre of grid row sy + ky of a support on the lattice of strain gam
__device__ inline double row_centre(const double4& p, const WaveParams& wp, double gam, int sy, int ky) {
  return p.x - gam * ((sy + ky) * wp.h - p.y);
}
}  // namespace

// sort key of every bead: the block of its support's first point
__global__ void k_bead_keys(int nb, const double4* __restrict__ pos, WaveParams wp, int BS, int nbin,
                            int* __restrict__ keys, int* __restrict__ vals) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nb) return;
  const int P = wp.support, N = wp.n;
  const double4 p = pos[i];
  const int sx = wrapi(support_start(p.x / wp.h, P), N), sy = wrapi(support_start(p.y / wp.h, P), N),
            sz = wrapi(support_start(p.z / wp.h, P), N);
  keys[i] = ((sz / BS) * nbin + sy / BS) * nbin + sx / BS;
  vals[i] = i;
}

// weights and starts of the beads in sorted order, one thread per weight
template <bool SHEAR>
__global__ void k_bead_weights(int nb, int wlen, const double4* __restrict__ pos, WaveParams wp, int BS, int nbin,
                               const int* __restrict__ perm, double* __restrict__ w64, float* __restrict__ w32,
                               int4* __restrict__ starts, short* __restrict__ rows) {
  const size_t t = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= size_t(nb) * wlen) return;
  const int k = int(t / wlen), q = int(t - size_t(k) * wlen);
  const int P = wp.support, N = wp.n;
  const double4 p = pos[perm[k]];
  const int sy = support_start(p.y / wp.h, P), sz = support_start(p.z / wp.h, P);
  double xm, wy = 1.0;
  if (SHEAR && q < P * P) {
    const int ky = q / P, kx = q - ky * P;
    const double gam = wp.gam ? *wp.gam : 0.0, cx = row_centre(p, wp, gam, sy, ky);
    const int sx = support_start(cx / wp.h, P);
    xm = (sx + kx) * wp.h - cx;
    const double ym = (sy + ky) * wp.h - p.y;
    wy = exp(-wp.alpha * ym * ym);
    if (kx == 0) rows[size_t(k) * P + ky] = short(wrapi(sx, N));
  } else if (SHEAR) {
    xm = (sz + q - P * P) * wp.h - p.z;
  } else {
    const int d = q / P, m = q - d * P;
    const double pd = d == 0 ? p.x : (d == 1 ? p.y : p.z);
    xm = (support_start(pd / wp.h, P) + m) * wp.h - pd;
  }
  const double v = exp(-wp.alpha * xm * xm) * wy;
  w64[t] = v;
  w32[t] = float(v);
  if (q == 0) {
    const int x = wrapi(support_start(p.x / wp.h, P), N), y = wrapi(sy, N), z = wrapi(sz, N);
    starts[k] = make_int4(x, y, z, ((z / BS) * nbin + y / BS) * nbin + x / BS);
  }
}

__global__ void k_bin_bounds(int nb, const int* __restrict__ keys, int* start, int* end) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nb) return;
  const int c = keys[k];
  if (k == 0 || keys[k - 1] != c) start[c] = k;
  if (k == nb - 1 || keys[k + 1] != c) end[c] = k + 1;
}

// the slots of sorted bead k: the blocks its support reaches (their index as the key, the slot's
// number as the value), the remaining slots a sentinel key past the last block.  SHEAR: along x, the blocks from
// the first to the last point of the rows that lie in the block row
template <bool SHEAR>
__global__ void k_block_slots(int nb, const int4* __restrict__ starts, const double4* __restrict__ pos,
                              const int* __restrict__ perm, WaveParams wp, int nbin, int kc, int kcx,
                              int* __restrict__ keys, int* __restrict__ vals, int* __restrict__ where) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nb) return;
  const int P = wp.support;
  const int4 s = starts[k];
  const int cnt[3] = {min(((s.x & 7) + P - 1) / 8 + 1, nbin), min(((s.y & 7) + P - 1) / 8 + 1, nbin),
                      min(((s.z & 7) + P - 1) / 8 + 1, nbin)};
  const int b0[3] = {s.x >> 3, s.y >> 3, s.z >> 3};
  const int per = kcx * kc * kc, sentinel = nbin * nbin * nbin;
  int q = 0;
  for (int jy = 0; jy < cnt[1]; ++jy) {
    const int by = (b0[1] + jy) % nbin;
    int x0 = b0[0], nx = cnt[0];
    if (SHEAR) {
      const double4 p = pos[perm[k]];
      const double gam = wp.gam ? *wp.gam : 0.0;
      const int sy = support_start(p.y / wp.h, P);
      int lo = 1 << 30, hi = -(1 << 30);
      for (int iy = 0; iy < P; ++iy) {
        if (((s.y + iy) >> 3) % nbin != by) continue;
        const int sx = support_start(row_centre(p, wp, gam, sy, iy) / wp.h, P);
        lo = min(lo, sx);
        hi = max(hi, sx);
      }
      x0 = lo >> 3;  // arithmetic shift: lo may be negative
      nx = min(((hi + P - 1) >> 3) - x0 + 1, min(nbin, kcx));
    }
    for (int jz = 0; jz < cnt[2]; ++jz)
      for (int jx = 0; jx < nx; ++jx) {
        const int bz = (b0[2] + jz) % nbin, bx = wrapi(x0 + jx, nbin);
        keys[size_t(k) * per + q] = (bz * nbin + by) * nbin + bx;
        vals[size_t(k) * per + q] = k * per + q;
        ++q;
      }
  }
  for (; q < per; ++q) {
    keys[size_t(k) * per + q] = sentinel;
    vals[size_t(k) * per + q] = k * per + q;
    where[size_t(k) * per + q] = -1;
  }
}

// list bounds per block and the candidate records from the sorted slots (sentinels ignored)
__global__ void k_block_lists(int n, int nbin, int N, int per, const int* __restrict__ keys,
                              const int* __restrict__ vals, const int4* __restrict__ starts,
                              const int* __restrict__ perm, int* __restrict__ start, int* __restrict__ end,
                              int4* __restrict__ cand, int* __restrict__ where) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const int c = keys[p];
  if (c >= nbin * nbin * nbin) return;
  if (p == 0 || keys[p - 1] != c) start[c] = p;
  if (p == n - 1 || keys[p + 1] != c) end[c] = p + 1;
  const int k = vals[p] / per;
  where[vals[p]] = p;
  const int4 s = starts[k];
  const int ox = point_offset(8 * (c % nbin), s.x, N), oy = point_offset(8 * (c / nbin % nbin), s.y, N),
            oz = point_offset(8 * (c / (nbin * nbin)), s.z, N);
  cand[p] = make_int4(k, perm[k], ox | (oy << 8) | (oz << 16), 0);
}

hipError_t spread_plan_update(SpreadPlan* sp, const double* pos4, const WaveParams& wp, hipStream_t st) {
  const int nb = sp->nb;
  const double4* pos = (const double4*)pos4;
  k_bead_keys<<<nblocks(nb), kThreads, 0, st>>>(nb, pos, wp, sp->BS, sp->nbin, sp->keys_in, sp->vals_in);
  int bits = 1;
  const int nbins = sp->nbin * sp->nbin * sp->nbin;
  while ((1 << bits) < nbins) ++bits;
  size_t tb = sp->temp_bytes;
  hipError_t e = hipcub::DeviceRadixSort::SortPairs(sp->temp, tb, sp->keys_in, sp->keys_out, sp->vals_in, sp->perm,
                                                    nb, 0, bits, st);
  if (e != hipSuccess) return e;
  const int wblk = nblocks((long long)nb * sp->wlen);
  if (sp->sheared)
    k_bead_weights<true><<<wblk, kThreads, 0, st>>>(nb, sp->wlen, pos, wp, sp->BS, sp->nbin, sp->perm, sp->weights,
                                                    sp->weights32, sp->starts, sp->rows);
  else
    k_bead_weights<false><<<wblk, kThreads, 0, st>>>(nb, sp->wlen, pos, wp, sp->BS, sp->nbin, sp->perm, sp->weights,
                                                     sp->weights32, sp->starts, nullptr);
  if (sp->BS == 4) {
    if ((e = hipMemsetAsync(sp->bin_start, 0, sizeof(int) * nbins, st)) != hipSuccess) return e;
    if ((e = hipMemsetAsync(sp->bin_end, 0, sizeof(int) * nbins, st)) != hipSuccess) return e;
    k_bin_bounds<<<nblocks(nb), kThreads, 0, st>>>(nb, sp->keys_out, sp->bin_start, sp->bin_end);
  } else {  // the candidate list of every block
    const int kc = sp->kc, kcx = sp->kcx, slots = nb * kcx * kc * kc;
    if (sp->sheared)
      k_block_slots<true><<<nblocks(nb), kThreads, 0, st>>>(nb, sp->starts, pos, sp->perm, wp, sp->nbin, kc, kcx,
                                                            sp->pk_in, sp->pv_in, sp->where);
    else
      k_block_slots<false><<<nblocks(nb), kThreads, 0, st>>>(nb, sp->starts, pos, sp->perm, wp, sp->nbin, kc, kcx,
                                                             sp->pk_in, sp->pv_in, sp->where);
    int pbits = 1;
    while ((1 << pbits) <= nbins) ++pbits;  // the sentinel nbins included
    size_t pb = sp->ptemp_bytes;
    if ((e = hipcub::DeviceRadixSort::SortPairs(sp->ptemp, pb, sp->pk_in, sp->pk_out, sp->pv_in, sp->pv_out, slots, 0,
                                                pbits, st)) != hipSuccess)
      return e;
    if ((e = hipMemsetAsync(sp->blk_start, 0, sizeof(int) * nbins, st)) != hipSuccess) return e;
    if ((e = hipMemsetAsync(sp->blk_end, 0, sizeof(int) * nbins, st)) != hipSuccess) return e;
    k_block_lists<<<nblocks(slots), kThreads, 0, st>>>(slots, sp->nbin, wp.n, kcx * kc * kc, sp->pk_out, sp->pv_out,
                                                       sp->starts, sp->perm, sp->blk_start, sp->blk_end, sp->cand,
                                                       sp->where);
  }
  return hipGetLastError();
}

namespace {
constexpr int kChunk = 64;
}

template <typename R, int BS>
__global__ __launch_bounds__(BS* BS* BS) void k_spread_gather(const int* __restrict__ bin_start,
                                                               const int* __restrict__ bin_end,
                                                               const int* __restrict__ perm,
                                                               const int4* __restrict__ starts,
                                                               const R* __restrict__ weights,
                                                               const double* __restrict__ lam, WaveParams wp,
                                                               int nbin, int K, R* __restrict__ grid, size_t cs,
                                                               const int* __restrict__ skip) {
  if (skip && *skip) return;
  constexpr int NT = BS * BS * BS;
  __shared__ int4 sh_s[kChunk];
  __shared__ R sh_w[kChunk * 3 * kMaxP];
  __shared__ R sh_l[kChunk * 6];
  __shared__ int rb0[2 * 8 * 8], rlen[2 * 8 * 8], roff[2 * 8 * 8 + 1];
  const int P = wp.support, N = wp.n, P3 = 3 * P;
  const int bx = blockIdx.x % nbin, by = (blockIdx.x / nbin) % nbin, bz = blockIdx.x / (nbin * nbin);
  const int t = threadIdx.x;
  const int mx = bx * BS + t % BS, my = by * BS + (t / BS) % BS, mz = bz * BS + t / (BS * BS);
  // candidate beads: per (kz, ky) one or two contiguous runs of the sorted bead array
  // (bins bx-K+1 .. bx along x, split where they wrap); thread r computes run r
  const int x0 = bx - K + 1;
  const int nparts = x0 >= 0 ? 1 : 2;
  const int nruns = K * K * nparts;
  for (int rr = t; rr < nruns; rr += NT) {
    const int part = rr % nparts, ky = (rr / nparts) % K, kz = rr / (nparts * K);
    const int cz = (bz - kz + nbin) % nbin, cy = (by - ky + nbin) % nbin;
    int lo, hi;
    if (x0 >= 0) {
      lo = x0;
      hi = bx;
    } else if (part == 0) {
      lo = 0;
      hi = bx;
    } else {
      lo = x0 + nbin;
      hi = nbin - 1;
    }
    const int row = (cz * nbin + cy) * nbin;
    int b0 = 0, b1 = 0;
    bool any = false;
    for (int c = lo; c <= hi; ++c) {
      const int e0 = bin_start[row + c], e1 = bin_end[row + c];
      if (e1 > e0) {
        if (!any) b0 = e0;
        b1 = e1;
        any = true;
      }
    }
    rb0[rr] = b0;
    rlen[rr] = any ? b1 - b0 : 0;
  }
  __syncthreads();
  if (t == 0) {
    int acc = 0;
    for (int r = 0; r < nruns; ++r) {
      roff[r] = acc;
      acc += rlen[r];
    }
    roff[nruns] = acc;
  }
  __syncthreads();
  const int total = roff[nruns];
  R a0 = 0, a1 = 0, a2 = 0, a3 = 0, a4 = 0, a5 = 0;
  for (int c0 = 0; c0 < total; c0 += kChunk) {
    const int n = min(kChunk, total - c0);
    if (c0 > 0) __syncthreads();
    // stage candidates c0 .. c0+n-1 (run-major order) in LDS
    for (int q = t; q < n * (P3 + 7); q += NT) {
      const int cand = q / (P3 + 7), f = q % (P3 + 7);
      const int gidx = c0 + cand;
      int r = 0;
      while (roff[r + 1] <= gidx) ++r;
      const int k = rb0[r] + (gidx - roff[r]);
      if (f < P3) {
        sh_w[cand * P3 + f] = weights[size_t(k) * P3 + f];
      } else if (f == P3) {
        sh_s[cand] = starts[k];
      } else {
        sh_l[6 * cand + (f - P3 - 1)] = R(lam[6 * size_t(perm[k]) + (f - P3 - 1)]);
      }
    }
    __syncthreads();
    for (int q = 0; q < n; ++q) {
      const int4 s = sh_s[q];
      int ix = mx - s.x, iy = my - s.y, iz = mz - s.z;
      ix += ix < 0 ? N : 0;
      iy += iy < 0 ? N : 0;
      iz += iz < 0 ? N : 0;
      if (ix < P && iy < P && iz < P) {
        const R* wq = sh_w + q * P3;
        const R w = wq[ix] * wq[P + iy] * wq[2 * P + iz];
        const R* l = sh_l + 6 * q;
        a0 += w * l[0];
        a1 += w * l[1];
        a2 += w * l[2];
        a3 += w * l[3];
        a4 += w * l[4];
        a5 += w * l[5];
      }
    }
  }
  const size_t m = (size_t(mz) * N + my) * N + mx;
  R* g = grid + 2 * m;
  g[0] = a0;
  g[1] = a3;
  g[cs] = a1;
  g[cs + 1] = a4;
  g[2 * cs] = a2;
  g[2 * cs + 1] = a5;
}

// Gather spreading on 8^3 blocks as matrix products.  A grid point's value is
//   G_c(x, y, z) = sum_b A_b(x, y) B_b(z, c),  A = w_x w_y,  B = w_z l_c (c = 6 force moments),
// a product over the block's candidate beads b of a (points in the plane) x b and a
// b x (planes and components) matrix, so it runs on the matrix cores: a wavefront owns two of
// the block's rows in y, all eight points in x and all eight planes, and walks the candidates that
// reach its rows four at a time, three 16 x 16 x 4 products each (one per axis: 8 planes of force,
// 8 of torque).  Points inside the support fill 32% of the products at P = 10; with the whole
// plane they would fill 20%, with 4 x 4 quadrants 35%, but those store half lines.
// Weights are staged in LDS as windows over the block's 8 points per axis, zero outside the
// support, so the inner loop has no index tests; on a sheared lattice the window is the 8 x 8
// plane of A.  Lists are padded to four with a candidate of zero weights.  No atomics; every
// sum is in list order.  The products of 81,920 beads take 45 us in FP64 and 22 in FP32 at the
// matrix rate; what is left is the latency from the candidate's record to its weights and the
// store of the grid, which other blocks' wavefronts cover.  Measured in the first pass of the
// saddle operator (128^3, beside 132 and 108 us of pair sum): 224 us in FP64 and 159 in FP32; with
// one lane per (x, y) column on the vector units it took 415 and 278.  The scatter with atomics of
// the sheared lattice took 250 (FP64, 2,048 beads) to 410 us (FP32, 6,011), now 17 and 22.
template <typename R, bool SHEAR>
struct SpreadTile {
  static constexpr int kCand = SHEAR ? 32 : 64;       // candidates staged at a time
  static constexpr int kPlane = SHEAR ? 64 : 16;      // the window of A (SHEAR) or of w_x and w_y
  static constexpr int kUsed = kPlane + 8 + 6;        // then w_z and the moments
  static constexpr int kStride = SHEAR ? 80 : 40;     // spreads four candidates over the banks
  // windows, records, the four wavefronts' lists, and (SHEAR) the rows' offsets along x
  static constexpr size_t kBytes = sizeof(R) * (kCand + 1) * kStride + sizeof(int4) * kCand +
                                   sizeof(int) * 4 * (kCand + 4) + (SHEAR ? sizeof(int) * 8 * kCand : 0);
};

typedef double Acc64 __attribute__((ext_vector_type(4)));
typedef float Acc32 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ Acc64 mma4(double a, double b, Acc64 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ Acc32 mma4(float a, float b, Acc32 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// Up to here four wavefronts share a bead in interpolation by beads.  One wavefront / four, in us, FP64 and P = 10,
// 14, 21: 128 beads 5.9 / 4.1, 9.7 / 5.4, 18.8 / 8.3; 512 beads 5.9 / 5.1, 9.9 / 7.3, 20.2 / 14.2; 800 beads 6.2 / 6.3,
// 10.7 / 10.3, 21.1 / 22.8 (at P = 5 and 8 equal throughout; FP32 meets at 640 to 800 as well)
constexpr int kShareBeads = 512;
template <typename R>
struct AccOf {
  using T = Acc64;
};
template <>
struct AccOf<float> {
  using T = Acc32;
};

// What the block kernels read of a plan.
template <typename R>
struct BlockArgs {
  const int *blk_start, *blk_end;
  const int4* cand;
  const short* rows;
  const R* weights;
  int nbin;
};

// The weight windows of n staged candidates (records rec, on a sheared lattice the rows' offsets
// row_x) into win: the plane of A (or w_x and w_y), then w_z.  Eight lanes serve a candidate, so the
// addresses are shifts and a wrap (dividing a running index by the window's length took more
// instructions than the products).
template <typename R, bool SHEAR, int S>
__device__ __forceinline__ void stage_windows(R* win, const int4* rec, const int* row_x, const R* __restrict__ weights,
                                              int n, int P, int N, int wlen) {
  constexpr int A = SHEAR ? 9 : 3, C = SpreadTile<R, SHEAR>::kCand;
  const int i = threadIdx.x & 7;
#pragma unroll
  for (int c0 = 0; c0 < C; c0 += 32) {
    const int c = c0 + int(threadIdx.x >> 3);
    if (c >= n) break;
    const int4 rc = rec[c];
    R wv[A];
#pragma unroll
    for (int a = 0; a < A; ++a) {
      int o, at;
      if (a == A - 1) {
        o = ((rc.z >> 16) & 255) + i;
        at = wlen - P;
      } else if (SHEAR) {
        int oy = ((rc.z >> 8) & 255) + a;
        oy -= oy >= N ? N : 0;
        o = row_x[8 * c + a];
        o = o < N ? o + i : P;
        at = oy * P;
      } else {
        o = ((rc.z >> (8 * a)) & 255) + i;
        at = a * P;
      }
      o -= o >= N ? N : 0;
      wv[a] = 0;
      if (o < P) wv[a] = SHEAR ? weights[size_t(rc.x) * wlen + at + o] : ldg1(weights, rc.x * wlen + at + o);
    }
#pragma unroll
    for (int a = 0; a < A; ++a) win[c * S + 8 * a + i] = wv[a];
  }
}

// whether staged candidate c reaches rows y0 + qy and the next of the block (which it reaches):
// the offset of the first row below P, or of the second one after the wrap
template <bool SHEAR>
__device__ __forceinline__ bool reaches_rows(const int4* rec, const int* row_x, int c, int qy, int P, int N) {
  if (SHEAR) {
    bool hit = false;
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const int ox = row_x[8 * c + qy + y];
      hit = hit || ox < P || (ox > N - 8 && ox < N);
    }
    return hit;
  }
  int oy = ((rec[c].z >> 8) & 255) + qy;
  oy -= oy >= N ? N : 0;
  return oy < P || oy == N - 1;
}

// offset of x0 from the start of each candidate's rows y0 .. y0 + 7, or N: outside the support
template <typename R>
__device__ __forceinline__ void stage_rows(int* row_x, const int4* rec, const short* __restrict__ rows, int n, int x0,
                                           int P, int N) {
  for (int q = threadIdx.x; q < 8 * n; q += 256) {
    const int4 rc = rec[q >> 3];
    int oy = ((rc.z >> 8) & 255) + (q & 7);
    oy -= oy >= N ? N : 0;
    row_x[q] = oy < P ? point_offset(x0, rows[size_t(rc.x) * P + oy], N) : N;
  }
}

// the value of the lane 8 further in the row of 16
__device__ __forceinline__ float ror8(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xf, 0xf, true));
}
__device__ __forceinline__ double ror8(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), 0x128, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), 0x128, 0xf, 0xf, true));
}

template <typename R, bool SHEAR>
__device__ __forceinline__ void spread_tile_body(const BlockArgs<R>& ba, const double* __restrict__ lam,
                                                 const WaveParams& wp, R* __restrict__ grid, size_t cs,
                                                 const int* __restrict__ skip, unsigned char* smem, int bx_) {
  if (skip && *skip) return;
  using Tile = SpreadTile<R, SHEAR>;
  using Acc = typename AccOf<R>::T;
  constexpr int C = Tile::kCand, S = Tile::kStride;
  const int P = wp.support, N = wp.n, nbin = ba.nbin;
  const int wlen = SHEAR ? P * P + P : 3 * P;
  R* win = reinterpret_cast<R*>(smem);
  int4* rec = reinterpret_cast<int4*>(win + (C + 1) * S);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int* list = reinterpret_cast<int*>(rec + C) + wave * (C + 4);
  int* row_x = reinterpret_cast<int*>(rec + C) + 4 * (C + 4);
  const int bl = xcd_remap(bx_, nbin * nbin * nbin);  // each XCD takes a contiguous slab of blocks
  const int x0 = (bl % nbin) * 8, y0 = (bl / nbin % nbin) * 8, z0 = bl / (nbin * nbin) * 8;
  const int qy = 2 * wave;
  // operand lanes: row m = lane % 16 of A is point (xa, ya) of the wavefront's rows, column m of B
  // the component half (force, torque) and plane m % 8; both take candidate lane / 16 of the four.
  // The products leave point (x = lane / 16 + 4 (r % 2), y = r / 2) in register r: FP64 has row
  // 4 r + lane / 16 there, FP32 row 4 (lane / 16) + r, so the two number the points differently
  const int m = lane & 15, kq = lane >> 4;
  const int xa = sizeof(R) == 8 ? (m & 3) + 4 * ((m >> 2) & 1) : (m >> 2) + 4 * (m & 1);
  const int ya = qy + (sizeof(R) == 8 ? m >> 3 : (m >> 1) & 1);
  const int plane = m & 7, half = m >> 3;
  const int cb = ba.blk_start[bl], total = ba.blk_end[bl] - cb;
  Acc acc[3] = {};
  if (t < S) win[C * S + t] = 0;  // the candidate of zero weights
  constexpr int NW = Tile::kPlane + 8;               // window points of a candidate
  constexpr int UL = C / 32;                         // candidates per eight lanes
  for (int c0 = 0; c0 < total; c0 += C) {
    const int n = min(C, total - c0);
    if (c0 > 0) __syncthreads();
    if (t < n) rec[t] = ba.cand[cb + c0 + t];
    __syncthreads();
    if (SHEAR) {
      stage_rows<R>(row_x, rec, ba.rows, n, x0, P, N);
      __syncthreads();
    }
    // the moments' loads are issued before the first of the weights' is waited for
    double lv[UL];
#pragma unroll
    for (int u = 0; u < UL; ++u) {
      const int c = (t >> 3) + 32 * u;
      if (c < n && (t & 7) < 6) lv[u] = lam[6 * size_t(rec[c].y) + (t & 7)];
    }
    stage_windows<R, SHEAR, S>(win, rec, row_x, ba.weights, n, P, N, wlen);
#pragma unroll
    for (int u = 0; u < UL; ++u) {
      const int c = (t >> 3) + 32 * u;
      if (c < n && (t & 7) < 6) win[c * S + NW + (t & 7)] = R(lv[u]);
    }
    const bool hit = lane < n && reaches_rows<SHEAR>(rec, row_x, lane, qy, P, N);
    const unsigned long long hits = __ballot(hit);
    const int cnt = __popcll(hits);
    if (hit) list[__popcll(hits & ((1ull << lane) - 1ull))] = lane * S;
    if (lane < 4) list[cnt + lane] = C * S;
    __syncthreads();
    for (int e = 0; e < cnt; e += 4) {
      const R* w = win + list[e + kq];
      const R a = SHEAR ? w[8 * ya + xa] : w[xa] * w[8 + ya];
      const R wz = w[Tile::kPlane + plane];
      const R* l = w + NW + 3 * half;
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[c] = mma4(a, wz * l[c], acc[c]);
    }
  }
  // lanes of force and torque trade half of their points, so that each stores whole complex values
  // and an instruction covers the block's eight x of a row: 64 or 128 bytes in one piece
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const R keep = half ? acc[c][2 * y + 1] : acc[c][2 * y];
      const R got = ror8(half ? acc[c][2 * y] : acc[c][2 * y + 1]);
      const unsigned p = (unsigned(z0 + plane) * N + y0 + qy + y) * N + x0 + kq + 4 * half;
      stg2(grid + c * cs, 2 * p, half ? got : keep, half ? keep : got);
    }
}

template <typename R, bool SHEAR>
__global__ __launch_bounds__(256, 4) void k_spread_tile(BlockArgs<R> ba, const double* __restrict__ lam, WaveParams wp,
                                                     R* __restrict__ grid, size_t cs, const int* __restrict__ skip) {
  extern __shared__ unsigned char smem_raw[];
  spread_tile_body<R, SHEAR>(ba, lam, wp, grid, cs, skip, smem_raw, blockIdx.x);
}

namespace {
template <typename R>
const R* plan_weights(const SpreadPlan* sp);
template <>
const double* plan_weights<double>(const SpreadPlan* sp) {
  return sp->weights;
}
template <>
const float* plan_weights<float>(const SpreadPlan* sp) {
  return sp->weights32;
}
}  // namespace

namespace {
template <typename R>
BlockArgs<R> block_args(const SpreadPlan* sp) {
  return {sp->blk_start, sp->blk_end, sp->cand, sp->rows, plan_weights<R>(sp), sp->nbin};
}
}  // namespace

template <typename R>
void launch_spread_gather(const SpreadPlan* sp, const double* lam, const WaveParams& wp, R* grid, hipStream_t st,
                          const int* skip) {
  const size_t cs = 2 * size_t(wp.n) * wp.n * wp.n;
  const int nblk = sp->nbin * sp->nbin * sp->nbin;
  if (sp->BS == 4)
    launch_k(k_spread_gather<R, 4>, nblk, 64, 0, st, sp->bin_start, sp->bin_end, sp->perm, sp->starts,
                                                plan_weights<R>(sp), lam, wp, sp->nbin, sp->K, grid, cs, skip);
  else if (sp->sheared)
    launch_k(k_spread_tile<R, true>, nblk, 256, SpreadTile<R, true>::kBytes, st, block_args<R>(sp), lam, wp, grid, cs,
             skip);
  else
    launch_k(k_spread_tile<R, false>, nblk, 256, SpreadTile<R, false>::kBytes, st, block_args<R>(sp), lam, wp, grid, cs,
             skip);
}

// First pass of the saddle operator in one launch.  The Sigma/lubrication reduction, the
// real-space sum and the gather spreading all read only the input vector, so instead of
// three dependent launches (or a fork onto a second stream) they take three block ranges
// of one grid: the reduction first, then the real-space rows, then the 8^3 spreading
// blocks.  The two short ranges are padded to multiples of 8 blocks, so every spreading
// block keeps the XCD (block index mod 8) its slab mapping assumes, and they finish early,
// leaving their slots to the longer spreading blocks.
template <typename R, int LPR, bool SHEAR>
__global__ __launch_bounds__(256, 4) void k_spread_fused(BlockArgs<R> ba, const double* __restrict__ lam, WaveParams wp,
                                                      R* __restrict__ grid, size_t cs, const R* __restrict__ tab,
                                                      RealArgs ra, RigidArgs ga, int na_blk, int nr_blk,
                                                      const int* __restrict__ skip) {
  extern __shared__ unsigned char smem_raw[];
  int b = blockIdx.x;
  if (b < na_blk) {
    agg_lub_body(ga.na, ga.offsets, ga.body, ga.r4, lam, ga.V, ga.lrow, ga.lcol, ga.coef, ga.y2, skip, b, 0, na_blk);
    return;
  }
  b -= na_blk;
  if (b < nr_blk) {
    real_sum_body<R, LPR>(ra.nb, ra.pos, lam, ra.rowptr, ra.col, tab, ra.rp, ra.out, 0, ra.order, skip, smem_raw, b,
                          nr_blk);
    return;
  }
  spread_tile_body<R, SHEAR>(ba, lam, wp, grid, cs, skip, smem_raw, b - nr_blk);
}

bool spread_fuses(const SpreadPlan* sp) { return sp && sp->BS == 8; }

template <typename R>
void launch_spread_fused(const SpreadPlan* sp, const double* lam, const WaveParams& wp, R* grid, const R* table,
                         int lpr, const RealArgs& ra, const RigidArgs& ga, hipStream_t st, const int* skip) {
  const size_t cs = 2 * size_t(wp.n) * wp.n * wp.n;
  const int nblk = sp->nbin * sp->nbin * sp->nbin;
  const size_t shm = std::max(sp->sheared ? SpreadTile<R, true>::kBytes : SpreadTile<R, false>::kBytes,
                              RealPoly<R>::bytes(ra.rp.fine));
  auto pad8 = [](long long n) { return int((n + 7) / 8 * 8); };
  const int na_blk = pad8((ga.na + 3) / 4), nr_blk = pad8(real_blocks(ra.nb, lpr));
  const int total = na_blk + nr_blk + nblk;
#define FSD_FUSED(L_)                                                                                           \
  do {                                                                                                          \
    if (sp->sheared)                                                                                            \
      launch_k(k_spread_fused<R, L_, true>, total, 256, shm, st, block_args<R>(sp), lam, wp, grid, cs, table, ra, \
               ga, na_blk, nr_blk, skip);                                                                       \
    else                                                                                                        \
      launch_k(k_spread_fused<R, L_, false>, total, 256, shm, st, block_args<R>(sp), lam, wp, grid, cs, table, ra, \
               ga, na_blk, nr_blk, skip);                                                                       \
  } while (0)
  switch (lpr) {
    case 1: FSD_FUSED(1); break;
    case 2: FSD_FUSED(2); break;
    case 4: FSD_FUSED(4); break;
    case 8: FSD_FUSED(8); break;
    case 16: FSD_FUSED(16); break;
    case 32: FSD_FUSED(32); break;
    default: FSD_FUSED(64); break;
  }
#undef FSD_FUSED
}

// ------------------------------------------------------------------------------------------
// Interpolation with a plan: beads in the plan's spatial order, its weights and starts
// ------------------------------------------------------------------------------------------

// What interpolation reads of a plan.
template <typename R>
struct BeadArgs {
  const int* perm;
  const int4* starts;
  const short* rows;
  const R* weights;
};

// a wavefront-uniform load, through the scalar cache
template <typename T>
__device__ __forceinline__ T uload(const T* p, size_t i) {
  return ((__attribute__((address_space(4))) const T*)p)[i];
}

// a += b with the halves of the wavefront (the 16-lane rows of each half) merged: afterwards the
// lower half (the even rows) holds the sums of a, the upper half (the odd rows) those of b
__device__ __forceinline__ float merge32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float merge16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ double merge32(double a, double b) {
  const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}
__device__ __forceinline__ double merge16(double a, double b) {
  const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}
template <int CTRL>
__device__ __forceinline__ float row_move(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double row_move(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true));
}
template <typename R>
__device__ __forceinline__ R row_sum(R v) {  // over the 16 lanes of a row, in every lane
  v += row_move<0x128>(v);
  v += row_move<0x124>(v);
  v += row_move<0x122>(v);
  v += row_move<0x121>(v);
  return v;
}

// out_i += the grid's velocities at bead i (+ Sigma^T V): sum over the P^3 support points of
// w_x w_y w_z times six components.  Lanes take (x, y) columns of the support and walk z: in FP32
// pairs of x points (one aligned 16-byte load, points outside the support weighted 0), in FP64
// single columns (with pairs the wider support and the registers cost more than the loads save).
// What bounds it is the 48 P^3 (24 in FP32) bytes a bead that pass through the CU's first-level
// cache, so the rest is kept out of the way: the bead's order, start and w_z come through the
// scalar cache, its other weights by one load per lane, nothing goes through LDS, and the six sums are merged by lane swaps (6 -> 3 -> 2 values) before they are reduced.
// WPB wavefronts share a bead when there are too few beads to fill the chip: two halves of the
// columns times two halves of z, joined through LDS.
// Measured: 32 beads FP64 11.8 -> 5.3 us, 2,048 on 64^3 11.0 -> 9.7; on the sheared lattice, where weights
// and row starts were recomputed for every apply, 2,048 FP64 21 -> 12 us, 6,011 FP32 36 -> 16.
template <typename R, bool SHEAR, int WPB>
__device__ __forceinline__ void interp_plan_body(int nb, const BeadArgs<R>& ba, const R* __restrict__ grid,
                                                 size_t cs, const WaveParams& wp, double* __restrict__ out,
                                                 const int* __restrict__ skip, const int* __restrict__ body,
                                                 const double4* __restrict__ r4, const double* __restrict__ V, int bx,
                                                 int nblk) {
  if (skip && *skip) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k = xcd_remap(bx, nblk) * (4 / WPB) + (WPB == 1 ? wave : 0);
  if (k >= nb) return;  // whole wavefronts (WPB 1), whole workgroups (WPB 4)
  const int P = wp.support, N = wp.n, wlen = SHEAR ? P * P + P : 3 * P;
  const int i = uload(ba.perm, k);
  const int sx = uload(&ba.starts[k].x, 0), sy = uload(&ba.starts[k].y, 0), sz = uload(&ba.starts[k].z, 0);
  const R* w = ba.weights + size_t(k) * wlen;
  const unsigned plane = 2u * N * N;
  const int n1 = min(P, N - sz);  // planes before the columns wrap to z = 0
  const int zh = WPB == 1 ? 0 : (P + 1) / 2, z0 = WPB > 1 && wave >= 2 ? zh : 0, z1 = WPB > 1 && wave < 2 ? zh : P;
  const R *g0 = grid, *g1 = grid + cs, *g2 = grid + 2 * cs;
  R a[6] = {0, 0, 0, 0, 0, 0};
  constexpr bool kPaired = sizeof(R) == 4;
  const int ncol = kPaired ? P / 2 + 1 : P;  // columns, or pairs that can touch the support, per row
  for (int q = lane + (WPB == 1 ? 0 : 64 * (wave & 1)); q < ncol * P; q += WPB == 1 ? 64 : 128) {
    const int ky = q / ncol, cx = q - ky * ncol;
    int y = sy + ky;
    y -= y >= N ? N : 0;
    const int s = SHEAR ? int(ba.rows[size_t(k) * P + ky]) : sx;
    const R wy = SHEAR ? R(1) : w[P + ky];
    const R* wrow = SHEAR ? w + ky * P : w;
    R wa, wb = 0;
    int x;
    if (kPaired) {
      const int k0 = 2 * cx - (s & 1);  // support offset of the pair's first point, from -1
      x = (s & ~1) + 2 * cx;
      wa = k0 >= 0 && k0 < P ? wrow[k0] * wy : R(0);
      wb = k0 + 1 < P ? wrow[k0 + 1] * wy : R(0);
    } else {
      x = s + cx;
      wa = wrow[cx] * wy;
    }
    x -= x >= N ? N : 0;
    const unsigned col = 2u * (y * N + x);
    unsigned off = col + unsigned(z0 < n1 ? sz + z0 : z0 - n1) * plane;
#pragma unroll 4
    for (int kz = z0; kz < z1; ++kz) {
      if (kz == n1) off = col;
      const R wz = uload(w, wlen - P + kz);
      if (kPaired) {
        const R u0 = wa * wz, u1 = wb * wz;
        R b0, b1, b2, b3;
        ldg4(g0, off, b0, b1, b2, b3);
        a[0] += u0 * b0 + u1 * b2;
        a[3] += u0 * b1 + u1 * b3;
        ldg4(g1, off, b0, b1, b2, b3);
        a[1] += u0 * b0 + u1 * b2;
        a[4] += u0 * b1 + u1 * b3;
        ldg4(g2, off, b0, b1, b2, b3);
        a[2] += u0 * b0 + u1 * b2;
        a[5] += u0 * b1 + u1 * b3;
      } else {
        const R u = wa * wz;
        R f, t;
        ldg2(g0, off, f, t);
        a[0] += u * f;
        a[3] += u * t;
        ldg2(g1, off, f, t);
        a[1] += u * f;
        a[4] += u * t;
        ldg2(g2, off, f, t);
        a[2] += u * f;
        a[5] += u * t;
      }
      off += plane;
    }
  }
  // velocities to the lower half of the wavefront, angular velocities to the upper; then components
  // 0 and 1 to the even and odd rows, component 2 to both
  R s0 = merge32(a[0], a[3]), s1 = merge32(a[1], a[4]), s2 = merge32(a[2], a[5]);
  s0 = row_sum(merge16(s0, s1));
  s2 = row_sum(merge16(s2, s2));
  if (WPB > 1) {
    __shared__ R part[WPB][6];
    if ((lane & 15) == 0) {
      const int h = 3 * (lane >> 5), c = (lane >> 4) & 1;
      part[wave][h + c] = s0;
      if (c == 0) part[wave][h + 2] = s2;
    }
    __syncthreads();
    if (wave) return;
    const int h = 3 * (lane >> 5), c = (lane >> 4) & 1;
    s0 = part[0][h + c] + part[1][h + c] + (part[2][h + c] + part[3][h + c]);
    s2 = part[0][h + 2] + part[1][h + 2] + (part[2][h + 2] + part[3][h + 2]);
  }
  if (lane & 15) return;
  const int c = (lane >> 4) & 1;  // this lane's components: c, and 2 in an even row
  double add0 = double(s0), add2 = double(s2);
  if (V) {  // Sigma^T V: (U + W x r, W) of the bead's body
    const double* v = V + 6 * size_t(body[i]);
    const double4 r = r4[i];
    if (lane < 32) {
      add0 += c ? v[1] + (v[5] * r.x - v[3] * r.z) : v[0] + (v[4] * r.z - v[5] * r.y);
      add2 += v[2] + (v[3] * r.y - v[4] * r.x);
    } else {
      add0 += v[3 + c];
      add2 += v[5];
    }
  }
  double* o = out + 6 * size_t(i) + 3 * (lane >> 5);
  o[c] += add0;
  if (c == 0) o[2] += add2;
}

template <typename R, bool SHEAR, int WPB>
__global__ __launch_bounds__(256) void k_interp_plan(int nb, BeadArgs<R> ba, const R* __restrict__ grid, size_t cs,
                                                     WaveParams wp, double* __restrict__ out,
                                                     const int* __restrict__ skip, const int* __restrict__ body,
                                                     const double4* __restrict__ r4, const double* __restrict__ V) {
  interp_plan_body<R, SHEAR, WPB>(nb, ba, grid, cs, wp, out, skip, body, r4, V, blockIdx.x, gridDim.x);
}

// Interpolation by blocks (see interp_choice.hpp), the spreading product turned round: a wavefront holds its two rows
// of the block (16 points of a plane, 8 planes, 6 components) in registers as the A operand, each
// grid value read once, and takes the candidates that reach them 16 at a time,
//   T(z, c; b) = sum over (x, y) of G(z, c; x, y) A_b(x, y),
// 12 matrix products, then weights the planes by w_z and adds them, two in a lane (FP32: four), the
// others by swaps of lanes.  The four wavefronts' sums meet in LDS and go to the candidate's place in
// part; k_interp_join adds a bead's places.  The gather (interp_plan_body) moves every bead's support
// through the first-level cache, 84 KB of cache lines a bead in FP64 (57 in FP32): 229 and 149 us at
// 81,920 beads on 128^3.  Here the two kernels take 131 and 77, of which the joining 16 and 15; the
// products alone would take 60 and 30, the rest is staging (latency and address arithmetic) and
// groups of sixteen that are not full.  Candidates as rows and planes as columns, whose sums cross
// eight lanes each, took 178 and 109; windows 40 values apart (four candidates' groups of points on
// the same banks) 15 us more in FP64.
template <typename R, bool SHEAR>
struct InterpTile {
  using S = SpreadTile<R, SHEAR>;
  static constexpr int kStride = SHEAR ? 76 : 28;  // sixteen candidates' groups of four points on all banks
  static constexpr size_t kBytes = sizeof(R) * (S::kCand + 1) * kStride + sizeof(int4) * S::kCand +
                                   sizeof(int) * 4 * (S::kCand + 16) + (SHEAR ? sizeof(int) * 8 * S::kCand : 0) +
                                   sizeof(R) * 4 * 6 * (S::kCand + 1) + 4 * sizeof(unsigned long long);
};

template <typename R, bool SHEAR>
__device__ __forceinline__ void interp_tile_body(const BlockArgs<R>& ba, const WaveParams& wp,
                                                 const R* __restrict__ grid, size_t cs, R* __restrict__ part,
                                                 const int* __restrict__ skip, unsigned char* smem, int bx_) {
  if (skip && *skip) return;
  using Tile = SpreadTile<R, SHEAR>;
  using Acc = typename AccOf<R>::T;
  constexpr int C = Tile::kCand, S = InterpTile<R, SHEAR>::kStride, WZ = Tile::kPlane;
  const int P = wp.support, N = wp.n, nbin = ba.nbin, wlen = SHEAR ? P * P + P : 3 * P;
  R* win = reinterpret_cast<R*>(smem);
  int4* rec = reinterpret_cast<int4*>(win + (C + 1) * S);
  unsigned long long* masks = reinterpret_cast<unsigned long long*>(rec + C);
  R* sums = reinterpret_cast<R*>(masks + 4);  // [wavefront][candidate][6]
  int* lists = reinterpret_cast<int*>(sums + 4 * 6 * (C + 1));
  int* row_x = lists + 4 * (C + 16);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int* list = lists + wave * (C + 16);
  R* mine = sums + wave * 6 * (C + 1);
  const int bl = xcd_remap(bx_, nbin * nbin * nbin);
  const int cb = ba.blk_start[bl], total = ba.blk_end[bl] - cb;
  if (total <= 0) return;
  const int x0 = (bl % nbin) * 8, y0 = (bl / nbin % nbin) * 8, z0 = bl / (nbin * nbin) * 8, qy = 2 * wave;
  // A operand, step s: point (x = kq + 4 (s % 2), y = s / 2), row (half, plane); lanes of force and
  // torque trade what they load as in spreading
  const int m = lane & 15, kq = lane >> 4, plane = m & 7, half = m >> 3;
  R g[3][4];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const unsigned p = (unsigned(z0 + plane) * N + y0 + qy + y) * N + x0 + kq + 4 * half;
      R f, q;
      ldg2(grid + c * cs, 2 * p, f, q);
      const R got = ror8(half ? f : q);
      g[c][2 * y] = half ? got : f;
      g[c][2 * y + 1] = half ? q : got;
    }
  if (t < S) win[C * S + t] = 0;  // the candidate of zero weights
  int4 next;
  if (t < min(C, total)) next = ba.cand[cb + t];
  for (int c0 = 0; c0 < total; c0 += C) {
    const int n = min(C, total - c0);
    if (t < n) rec[t] = next;
    if (t < min(C, total - c0 - C)) next = ba.cand[cb + c0 + C + t];
    __syncthreads();
    if (SHEAR) {
      stage_rows<R>(row_x, rec, ba.rows, n, x0, P, N);
      __syncthreads();
    }
    stage_windows<R, SHEAR, S>(win, rec, row_x, ba.weights, n, P, N, wlen);
    const bool hit = lane < n && reaches_rows<SHEAR>(rec, row_x, lane, qy, P, N);
    const unsigned long long hits = __ballot(hit);
    const int cnt = __popcll(hits);
    if (hit) list[__popcll(hits & ((1ull << lane) - 1ull))] = lane;
    if (lane < 16) list[cnt + lane] = C;
    if (lane == 0) masks[wave] = hits;
    __syncthreads();
    for (int e = 0; e < cnt; e += 16) {
      const int ci = list[e + m];
      const R* w = win + ci * S;
      Acc acc[3] = {};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int x = kq + 4 * (s & 1), y = qy + (s >> 1);
        const R a = SHEAR ? w[8 * y + x] : w[x] * w[8 + y];
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[c] = mma4(g[c][s], a, acc[c]);
      }
      // rows of the products: FP64 has row 4 r + kq in register r, FP32 row 4 kq + r
      R u[3];
      if (sizeof(R) == 8) {
        const R za = w[WZ + kq], zb = w[WZ + 4 + kq];
#pragma unroll
        for (int c = 0; c < 3; ++c)
          u[c] = merge32(acc[c][0] * za + acc[c][1] * zb, acc[c][2] * za + acc[c][3] * zb);
      } else {
        const R* z = w + WZ + 4 * (kq & 1);
#pragma unroll
        for (int c = 0; c < 3; ++c) u[c] = acc[c][0] * z[0] + acc[c][1] * z[1] + acc[c][2] * z[2] + acc[c][3] * z[3];
      }
      R* out = mine + 6 * ci + 3 * (kq >> 1);
      out[kq & 1] = merge16(u[0], u[1]);
      const R last = merge16(u[2], u[2]);
      if (!(kq & 1)) out[2] = last;
    }
    __syncthreads();
    for (int q = t; q < 6 * n; q += 256) {
      const int c = q / 6;
      R u = 0;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (masks[v] >> c & 1) u += sums[v * 6 * (C + 1) + q];
      part[size_t(6) * (cb + c0) + q] = u;
    }
  }
}

template <typename R, bool SHEAR>
__global__ __launch_bounds__(256, 4) void k_interp_tile(BlockArgs<R> ba, WaveParams wp, const R* __restrict__ grid,
                                                        size_t cs, R* __restrict__ part,
                                                        const int* __restrict__ skip) {
  extern __shared__ unsigned char smem_raw[];
  interp_tile_body<R, SHEAR>(ba, wp, grid, cs, part, skip, smem_raw, blockIdx.x);
}

// out_i += the sums of bead i's places (+ Sigma^T V), one thread per bead and component
template <typename R>
__device__ __forceinline__ void interp_join_body(int nb, int per, const int* __restrict__ perm,
                                                 const int* __restrict__ where, const R* __restrict__ part,
                                                 double* __restrict__ out, const int* __restrict__ skip,
                                                 const int* __restrict__ body, const double4* __restrict__ r4,
                                                 const double* __restrict__ V, int t) {
  if (skip && *skip) return;
  const int k = t / 6, c = t - 6 * k;
  if (k >= nb) return;
  const int* w = where + size_t(k) * per;
  R u = 0;
  for (int q0 = 0; q0 < per; q0 += 4) {
    int p[4];
    R v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) p[j] = q0 + j < per ? w[q0 + j] : -1;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = p[j] >= 0 ? part[size_t(6) * p[j] + c] : R(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) u += v[j];
    if (p[3] < 0) break;  // the used slots come first
  }
  const int i = perm[k];
  double add = double(u);
  if (V) {
    const double* v = V + 6 * size_t(body[i]);
    const double4 r = r4[i];
    add += v[c];
    if (c == 0) add += v[4] * r.z - v[5] * r.y;
    if (c == 1) add += v[5] * r.x - v[3] * r.z;
    if (c == 2) add += v[3] * r.y - v[4] * r.x;
  }
  out[6 * size_t(i) + c] += add;
}

template <typename R>
__global__ __launch_bounds__(256) void k_interp_join(int nb, int per, const int* __restrict__ perm,
                                                     const int* __restrict__ where, const R* __restrict__ part,
                                                     double* __restrict__ out, const int* __restrict__ skip,
                                                     const int* __restrict__ body, const double4* __restrict__ r4,
                                                     const double* __restrict__ V) {
  interp_join_body<R>(nb, per, perm, where, part, out, skip, body, r4, V, blockIdx.x * 256 + threadIdx.x);
}

template <typename R>
void launch_interp(int nb, const double* pos4, const R* grid, const WaveParams& wp, double* out, hipStream_t st,
                   const int* skip, const int* body, const double* r4, const double* V, const SpreadPlan* sp) {
  const size_t cs = 2 * size_t(wp.n) * wp.n * wp.n;
  const double4* r = (const double4*)r4;
  if (!sp) {
    launch_k(k_interp<R>, nblocks(nb, 4), kThreads, 0, st, nb, (const double4*)pos4, grid, cs, wp, out, skip, body, r, V);
    return;
  }
  bool by_blocks = false;
  if (sp->BS == 8 && nb > kShareBeads) {
    InterpChoice choice(sp->sheared, sizeof(R));
    choice.add(nb, wp.n, wp.support);
    by_blocks = choice.by_blocks();
  }
  if (by_blocks) {
    const int nblk = sp->nbin * sp->nbin * sp->nbin;
    R* part = static_cast<R*>(sp->scratch);
    if (sp->sheared)
      launch_k(k_interp_tile<R, true>, nblk, 256, InterpTile<R, true>::kBytes, st, block_args<R>(sp), wp, grid, cs, part,
               skip);
    else
      launch_k(k_interp_tile<R, false>, nblk, 256, InterpTile<R, false>::kBytes, st, block_args<R>(sp), wp, grid, cs,
               part, skip);
    launch_k(k_interp_join<R>, nblocks(6LL * nb), 256, 0, st, nb, sp->kcx * sp->kc * sp->kc, sp->perm, sp->where, part,
             out, skip, body, r, V);
    return;
  }
  const BeadArgs<R> ba{sp->perm, sp->starts, sp->rows, plan_weights<R>(sp)};
  const bool share = nb <= kShareBeads;
#define FSD_INTERP(S_, W_) \
  launch_k(k_interp_plan<R, S_, W_>, nblocks(nb, 4 / W_), kThreads, 0, st, nb, ba, grid, cs, wp, out, skip, body, r, V)
  if (sp->sheared) {
    if (share) FSD_INTERP(true, 4); else FSD_INTERP(true, 1);
  } else {
    if (share) FSD_INTERP(false, 4); else FSD_INTERP(false, 1);
  }
#undef FSD_INTERP
}

// ------------------------------------------------------------------------------------------
// multi-system launches: block -> (system, local block) by the prefix table, then the
// single-system body with that system's pointers (the Arnoldi step maps z -> w)
// ------------------------------------------------------------------------------------------

namespace {

// Lanes per bead row of the batched real-space sum; a row pass a workgroup (two and four, to copy the
// coefficients less often: 64 systems in groups 83 and 106 us instead of 74, eight FP64 systems of
// 9,000 beads together 45 instead of 15).
constexpr int kBatchLpr = 16;
}  // namespace

template <typename R>
__global__ __launch_bounds__(256, 4) void kb_real(const BatchDesc* __restrict__ D, const int* __restrict__ off,
                                              int nsys) {
  const int s = batch_system(off, nsys, blockIdx.x);
  const BatchDesc& d = D[s];
  extern __shared__ unsigned char smem_raw[];
  real_sum_body<R, kBatchLpr>(d.nb, (const double4*)d.pos4, d.z, d.nrow, d.ncol, pick<R>(d.tab64, d.tab32), d.rp,
                              d.w, 0, d.perm, &d.ctl->stop, smem_raw, blockIdx.x - off[s], off[s + 1] - off[s]);
}

template <typename R>
__global__ __launch_bounds__(256, 4) void kb_spread(const BatchDesc* __restrict__ D, const int* __restrict__ off,
                                                int nsys) {
  const int s = batch_system(off, nsys, blockIdx.x);
  const BatchDesc& d = D[s];
  const size_t cs = 2 * size_t(d.wp.n) * d.wp.n * d.wp.n;
  extern __shared__ unsigned char smem_raw[];
  const BlockArgs<R> ba{d.blk_start, d.blk_end, d.cand, nullptr, pick<R>(d.w64, d.w32), d.nbin};
  spread_tile_body<R, false>(ba, d.z, d.wp, static_cast<R*>(d.grid), cs, &d.ctl->stop, smem_raw,
                             blockIdx.x - off[s]);
}

template <typename R>
__global__ __launch_bounds__(256) void kb_interp(const BatchDesc* __restrict__ D, const int* __restrict__ off,
                                                int nsys) {
  const int s = batch_system(off, nsys, blockIdx.x);
  const BatchDesc& d = D[s];
  const size_t cs = 2 * size_t(d.wp.n) * d.wp.n * d.wp.n;
  interp_plan_body<R, false, 1>(d.nb, {d.perm, d.starts, nullptr, pick<R>(d.w64, d.w32)},
                                static_cast<const R*>(d.grid), cs, d.wp, d.w, &d.ctl->stop, d.body,
                                (const double4*)d.r4, d.z + 6 * size_t(d.nb), blockIdx.x - off[s], off[s + 1] - off[s]);
}

template <typename R>
__global__ __launch_bounds__(256, 4) void kb_interp_tile(const BatchDesc* __restrict__ D, const int* __restrict__ off,
                                                         int nsys) {
  const int s = batch_system(off, nsys, blockIdx.x);
  const BatchDesc& d = D[s];
  const size_t cs = 2 * size_t(d.wp.n) * d.wp.n * d.wp.n;
  extern __shared__ unsigned char smem_raw[];
  const BlockArgs<R> ba{d.blk_start, d.blk_end, d.cand, nullptr, pick<R>(d.w64, d.w32), d.nbin};
  interp_tile_body<R, false>(ba, d.wp, static_cast<const R*>(d.grid), cs, static_cast<R*>(d.places), &d.ctl->stop,
                             smem_raw, blockIdx.x - off[s]);
}

template <typename R>
__global__ __launch_bounds__(256) void kb_interp_join(const BatchDesc* __restrict__ D, const int* __restrict__ off,
                                                      int nsys) {
  const int s = batch_system(off, nsys, blockIdx.x);
  const BatchDesc& d = D[s];
  interp_join_body<R>(d.nb, d.slots, d.perm, d.where, static_cast<const R*>(d.places), d.w, &d.ctl->stop, d.body,
                      (const double4*)d.r4, d.z + 6 * size_t(d.nb), (blockIdx.x - off[s]) * 256 + threadIdx.x);
}

// spreading fields of a batch descriptor (blk_start == nullptr: no plan of 8^3 blocks)
void spread_plan_desc(const SpreadPlan* sp, BatchDesc& d) {
  const bool ok = sp && sp->BS == 8;
  d.blk_start = ok ? sp->blk_start : nullptr;
  d.blk_end = ok ? sp->blk_end : nullptr;
  d.cand = ok ? sp->cand : nullptr;
  d.perm = ok ? sp->perm : nullptr;
  d.starts = ok ? sp->starts : nullptr;
  d.w64 = ok ? sp->weights : nullptr;
  d.w32 = ok ? sp->weights32 : nullptr;
  d.nbin = ok ? sp->nbin : 0;
  d.slots = ok ? sp->kcx * sp->kc * sp->kc : 0;
  d.where = ok ? sp->where : nullptr;
  d.places = ok ? sp->scratch : nullptr;
}

int batch_blocks(const BatchDesc& d, int kind, int prec) {
  switch (kind) {
    case BK_PRECOND:
    case BK_AGG:
      return (d.na + 3) / 4;
    case BK_REAL:
      return real_blocks(d.nb, kBatchLpr);
    case BK_SPREAD:
      return d.nbin * d.nbin * d.nbin;
    case BK_FFT_OUTER:
    case BK_FFT_MID:
    case BK_FFT_GREEN:
      return batch_fft_blocks(d, kind, prec);
    case BK_INTERP:
      return d.by_blocks ? d.nbin * d.nbin * d.nbin : (d.nb + 3) / 4;
    case BK_JOIN:
      return d.by_blocks ? (6 * d.nb + 255) / 256 : 0;
    case BK_CGS:
      return d.ncgs;
    default:
      return 0;
  }
}

size_t batch_shm(const BatchDesc& d, int kind, int prec) {
  switch (kind) {
    case BK_REAL:
      return prec ? RealPoly<float>::bytes(d.rp.fine) : RealPoly<double>::bytes(d.rp.fine);
    case BK_SPREAD:
      return prec ? SpreadTile<float, false>::kBytes : SpreadTile<double, false>::kBytes;
    case BK_INTERP:
      return !d.by_blocks ? 0 : prec ? InterpTile<float, false>::kBytes : InterpTile<double, false>::kBytes;
    case BK_FFT_OUTER:
    case BK_FFT_MID:
    case BK_FFT_GREEN:
      return batch_fft_shm(d, kind, prec);
    default:
      return 0;
  }
}

namespace {
template <typename R>
void batch_mobility(int kind, const BatchDesc* D, const int* off, int nsys, int total, size_t shm,
                    hipStream_t st) {
  switch (kind) {
    case BK_REAL:
      kb_real<R><<<total, kThreads, shm, st>>>(D, off, nsys);
      break;
    case BK_SPREAD:
      kb_spread<R><<<total, 256, shm, st>>>(D, off, nsys);
      break;
    case BK_INTERP:
      if (shm)
        kb_interp_tile<R><<<total, 256, shm, st>>>(D, off, nsys);
      else
        kb_interp<R><<<total, kThreads, 0, st>>>(D, off, nsys);
      break;
    case BK_JOIN:
      kb_interp_join<R><<<total, 256, 0, st>>>(D, off, nsys);
      break;
    default:
      break;
  }
}
}  // namespace

void launch_batch_mobility(int kind, int prec, int stage, const BatchDesc* D, const int* off, int nsys, int total,
                           size_t shm, hipStream_t st) {
  if (total <= 0) return;
  if (kind == BK_FFT_OUTER || kind == BK_FFT_MID || kind == BK_FFT_GREEN)
    launch_batch_fft(prec, stage, D, off, nsys, total, shm, st);
  else if (prec)
    batch_mobility<float>(kind, D, off, nsys, total, shm, st);
  else
    batch_mobility<double>(kind, D, off, nsys, total, shm, st);
}

template void launch_spread_gather<double>(const SpreadPlan*, const double*, const WaveParams&, double*, hipStream_t, const int*);
template void launch_spread_gather<float>(const SpreadPlan*, const double*, const WaveParams&, float*, hipStream_t, const int*);
template void launch_spread_fused<double>(const SpreadPlan*, const double*, const WaveParams&, double*, const double*,
                                          int, const RealArgs&, const RigidArgs&, hipStream_t, const int*);
template void launch_spread_fused<float>(const SpreadPlan*, const double*, const WaveParams&, float*, const float*, int,
                                         const RealArgs&, const RigidArgs&, hipStream_t, const int*);
template void launch_real_sum<double>(int, const double*, const double*, const int*, const uint32_t*, const double*,
                                      const RealParams&, double*, bool, int, hipStream_t, const int*, const int*);
template void launch_real_sum<float>(int, const double*, const double*, const int*, const uint32_t*, const float*,
                                     const RealParams&, double*, bool, int, hipStream_t, const int*, const int*);
template void launch_spread<double>(int, const double*, const double*, const WaveParams&, double*, hipStream_t, const int*);
template void launch_spread<float>(int, const double*, const double*, const WaveParams&, float*, hipStream_t, const int*);
template void launch_interp<double>(int, const double*, const double*, const WaveParams&, double*, hipStream_t, const int*,
                                    const int*, const double*, const double*, const SpreadPlan*);
template void launch_interp<float>(int, const double*, const float*, const WaveParams&, double*, hipStream_t, const int*,
                                   const int*, const double*, const double*, const SpreadPlan*);
template void launch_spread_sheared<double>(int, const double*, const double*, const WaveParams&, double*, hipStream_t,
                                            const int*);
template void launch_spread_sheared<float>(int, const double*, const double*, const WaveParams&, float*, hipStream_t,
                                           const int*);
template void launch_interp_sheared<double>(int, const double*, const double*, const WaveParams&, double*, hipStream_t,
                                            const int*, const int*, const double*, const double*);
template void launch_interp_sheared<float>(int, const double*, const float*, const WaveParams&, double*, hipStream_t,
                                           const int*, const int*, const double*, const double*);
}  // namespace fsd
