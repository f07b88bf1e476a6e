// Kernels of the saddle operator outside the mobility, the preconditioner and
// the FP64 Krylov vector operations.
#include <algorithm>

#include "fsd_impl.hpp"
#include "k_rigid.hpp"

namespace fsd {

namespace {
constexpr int kThreads = 256;
inline int nblocks(long long n, int t = kThreads) { return int((n + t - 1) / t); }
}  // namespace

// Magnitude of the conservative force between two beads of radius a at centre distance r,
// positive when repulsive (Section 4.2): van der Waals from the sphere-sphere Hamaker
// potential with the separation shifted by h_c (held at the contact value for r < 2a),
// the screened double layer a^2 Z exp(-kappa (r - 2a)) / r, and the Hertz contact
// k_n delta^1.5 for delta = 2a - r > 0.
__device__ inline double pair_force_mag(double r, const PairForceParams& p) {
  const double a = p.a, a2 = a * a;
  double f = 0.0;
  if (p.hamaker != 0.0) {
    // -dV/ds of V(s) = -(A/6) [2a^2/(s^2 - 4a^2) + 2a^2/s^2 + ln((s^2 - 4a^2)/s^2)], s = r + h_c
    const double sv = fmax(r, 2.0 * a) + p.hc, s2 = sv * sv, d = s2 - 4.0 * a2;
    f += (p.hamaker / 6.0) * (-4.0 * a2 * sv / (d * d) - 4.0 * a2 / (s2 * sv) + 2.0 * sv / d - 2.0 / sv);
  }
  if (p.Z != 0.0) f += p.Z * a2 * exp(-p.kappa * (r - 2.0 * a)) * (1.0 / (r * r) + p.kappa / r);
  if (r < 2.0 * a && p.kn > 0.0) {
    const double dl = 2.0 * a - r;
    f += p.kn * dl * sqrt(dl);
  }
  return f;
}

__global__ void k_pair_forces(int nb, const double4* __restrict__ pos, const int* __restrict__ body,
                              const int* __restrict__ rowptr, const uint32_t* __restrict__ col, PairForceParams p,
                              double* __restrict__ fe, int accumulate) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nb) return;
  const double4 pi = pos[i];
  const int bi = body[i];
  double fx = 0, fy = 0, fz = 0;
  for (int e = rowptr[i]; e < rowptr[i + 1]; ++e) {
    const uint32_t c = col[e];
    const int j = int(c & 0x3FFFFFu);
    if (body[j] == bi) continue;
    const double4 pj = pos[j];
    const double dy = pi.y - pj.y + (int((c >> 25) & 7u) - 3) * p.L;  // Cartesian from sheared
    const double dx = pi.x - pj.x + (int((c >> 22) & 7u) - 3) * p.L + p.gam * dy;
    const double dz = pi.z - pj.z + (int((c >> 28) & 7u) - 3) * p.L;
    const double r = sqrt(dx * dx + dy * dy + dz * dz);
    if (!(r < p.r_cut) || r == 0.0) continue;
    const double g = pair_force_mag(r, p) / r;  // along the unit vector from j to i
    fx += g * dx;
    fy += g * dy;
    fz += g * dz;
  }
  double* o = fe + 3 * size_t(i);
  const double b0 = accumulate ? o[0] : 0.0, b1 = accumulate ? o[1] : 0.0, b2 = accumulate ? o[2] : 0.0;
  o[0] = b0 - fx;
  o[1] = b1 - fy;
  o[2] = b2 - fz;
}

// flag = 1 when two beads of different bodies are closer than 1.5 a (the real-space list
// holds every pair within its cutoff; used when there is no lubrication list to check)
__global__ void k_overlap_check(int nb, const double4* __restrict__ pos, const int* __restrict__ body,
                                const int* __restrict__ rowptr, const uint32_t* __restrict__ col, double L,
                                double gam, double a, int* __restrict__ flag) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nb) return;
  const double4 pi = pos[i];
  const double lim2 = 2.25 * a * a;
  for (int e = rowptr[i]; e < rowptr[i + 1]; ++e) {
    const uint32_t c = col[e];
    const int j = int(c & 0x3FFFFFu);
    if (body[j] == body[i]) continue;
    const double4 pj = pos[j];
    const double dy = pi.y - pj.y + (int((c >> 25) & 7u) - 3) * L;
    const double dx = pi.x - pj.x + (int((c >> 22) & 7u) - 3) * L + gam * dy;
    const double dz = pi.z - pj.z + (int((c >> 28) & 7u) - 3) * L;
    if (dx * dx + dy * dy + dz * dz < lim2) {
      atomicOr(flag, 1);
      return;
    }
  }
}

void launch_overlap_check(int nb, const double* pos4, const int* body, const int* rowptr, const uint32_t* col,
                          double L, double gam, double a, int* flag, hipStream_t st) {
  k_overlap_check<<<nblocks(nb), kThreads, 0, st>>>(nb, (const double4*)pos4, body, rowptr, col, L, gam, a, flag);
}

void launch_pair_forces(int nb, const double* pos4, const int* body, const int* rowptr, const uint32_t* col,
                        const PairForceParams& pf, double* fe, int accumulate, hipStream_t st) {
  k_pair_forces<<<nblocks(nb), kThreads, 0, st>>>(nb, (const double4*)pos4, body, rowptr, col, pf, fe, accumulate);
}

// f_i = sgn sum_k R_pair,ik (w_i - w_k), R_pair = X nn + Y (I - nn)
__global__ void k_lub_apply(int nb, double sgn, const int* __restrict__ rowptr, const uint32_t* __restrict__ col,
                            const double* __restrict__ coef, const double* __restrict__ wt, double* __restrict__ f, const int* __restrict__ skip) {
  if (skip && *skip) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nb) return;
  const double wx = wt[3 * i], wy = wt[3 * i + 1], wz = wt[3 * i + 2];
  double ax = 0, ay = 0, az = 0;
  for (int e = rowptr[i]; e < rowptr[i + 1]; ++e) {
    const int k = int(col[e] & 0x3FFFFFu);
    const double* c = coef + 5 * e;
    const double dx = wx - wt[3 * k], dy = wy - wt[3 * k + 1], dz = wz - wt[3 * k + 2];
    const double nd = c[2] * dx + c[3] * dy + c[4] * dz;
    const double g = (c[0] - c[1]) * nd;
    ax += c[1] * dx + g * c[2];
    ay += c[1] * dy + g * c[3];
    az += c[1] * dz + g * c[4];
  }
  f[3 * i] = sgn * ax;
  f[3 * i + 1] = sgn * ay;
  f[3 * i + 2] = sgn * az;
}

void launch_lub_apply(int nb, double sgn, const int* rowptr, const uint32_t* col, const double* coef, const double* wt,
                      double* f, hipStream_t st, const int* skip) {
  k_lub_apply<<<nblocks(nb, 64), 64, 0, st>>>(nb, sgn, rowptr, col, coef, wt, f, skip);
}

// ------------------------------------------------------------------------------------------
// constraint stresslets (Eq. `stress_comp`)
// ------------------------------------------------------------------------------------------

// w_i = U_j + Omega_j x r_i: the translational rigid-body velocity of bead i from the
// aggregate part V of the solution (relative to the imposed flow)
__global__ void k_bead_rigid_vel(int nb, const int* __restrict__ body, const double4* __restrict__ r4,
                                 const double* __restrict__ V, double* __restrict__ w) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nb) return;
  const double* v = V + 6 * size_t(body[i]);
  const double4 r = r4[i];
  w[3 * i] = v[0] + v[4] * r.z - v[5] * r.y;
  w[3 * i + 1] = v[1] + v[5] * r.x - v[3] * r.z;
  w[3 * i + 2] = v[2] + v[3] * r.y - v[4] * r.x;
}

void launch_bead_rigid_vel(int nb, const int* body, const double* r4, const double* V, double* w, hipStream_t st) {
  k_bead_rigid_vel<<<nblocks(nb), kThreads, 0, st>>>(nb, body, (const double4*)r4, V, w);
}

// S_j = sum_{i in j} sym(r_i (F_i + f_i)): F the bead force moments (6 per bead, the
// translational three used), f further forces on the beads (3 per bead, may be null);
// one thread per aggregate, 9 values each (row-major)
__global__ void k_stresslets(int na, const int* __restrict__ offsets, const double4* __restrict__ r4,
                             const double* __restrict__ F, const double* __restrict__ f, double* __restrict__ S) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= na) return;
  double acc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int i = offsets[j]; i < offsets[j + 1]; ++i) {
    const double4 r = r4[i];
    const double rv[3] = {r.x, r.y, r.z};
    double fv[3];
    for (int a = 0; a < 3; ++a) fv[a] = F[6 * size_t(i) + a] + (f ? f[3 * size_t(i) + a] : 0.0);
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) acc[3 * a + b] += 0.5 * (rv[a] * fv[b] + rv[b] * fv[a]);
  }
  for (int k = 0; k < 9; ++k) S[9 * size_t(j) + k] = acc[k];
}

void launch_stresslets(int na, const int* offsets, const double* r4, const double* F, const double* f, double* S,
                       hipStream_t st) {
  k_stresslets<<<nblocks(na, 128), 128, 0, st>>>(na, offsets, (const double4*)r4, F, f, S);
}

// ------------------------------------------------------------------------------------------
// right-hand side of Eq. `spm_agg`
// ------------------------------------------------------------------------------------------

// b1_i = (E r_i, 0) [+ (u_B, w_B)_i]; e3_i = E r_i (ambient flow relative to the body)
__global__ void k_rhs_bead(int nb, const double4* __restrict__ r4, const double* __restrict__ E,
                           const double* __restrict__ ub, double* __restrict__ b1, double* __restrict__ e3) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nb) return;
  const double4 r = r4[i];
  double e[3];
  for (int a = 0; a < 3; ++a) e[a] = E[3 * a] * r.x + E[3 * a + 1] * r.y + E[3 * a + 2] * r.z;
  double* b = b1 + 6 * i;
  for (int a = 0; a < 3; ++a) {
    b[a] = e[a] + (ub ? ub[6 * i + a] : 0.0);
    b[3 + a] = ub ? ub[6 * i + 3 + a] : 0.0;
    e3[3 * i + a] = e[a];
  }
}

void launch_rhs(int nb, int na, const int* offsets, const int* body, const double* r4, const double* E,
                const double* force, const double* fnf, double* b1, double* e3, hipStream_t st) {
  (void)na;
  (void)offsets;
  (void)body;
  (void)force;
  k_rhs_bead<<<nblocks(nb), kThreads, 0, st>>>(nb, (const double4*)r4, E, fnf, b1, e3);
}

// b2_j = -F_j + Sigma (f_e, 0) with f_e = -R_nf e (so Sigma R_nf e = -Sigma f_e)
__global__ void k_rhs_agg(int na, const int* __restrict__ offsets, const double4* __restrict__ r4,
                          const double* __restrict__ force, const double* __restrict__ fe, double* __restrict__ b2) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= na) return;
  double F[3] = {0, 0, 0}, T[3] = {0, 0, 0};
  if (fe) {
    for (int i = offsets[j]; i < offsets[j + 1]; ++i) {
      const double fx = fe[3 * i], fy = fe[3 * i + 1], fz = fe[3 * i + 2];
      const double4 r = r4[i];
      F[0] += fx;
      F[1] += fy;
      F[2] += fz;
      T[0] += r.y * fz - r.z * fy;
      T[1] += r.z * fx - r.x * fz;
      T[2] += r.x * fy - r.y * fx;
    }
  }
  double* b = b2 + 6 * j;
  for (int a = 0; a < 3; ++a) {
    b[a] = -force[6 * j + a] + F[a];
    b[3 + a] = -force[6 * j + 3 + a] + T[a];
  }
}

void launch_rhs_agg(int na, const int* offsets, const double* r4, const double* force, const double* flub_e,
                    double* b2, hipStream_t st) {
  k_rhs_agg<<<nblocks(na, 128), 128, 0, st>>>(na, offsets, (const double4*)r4, force, flub_e, b2);
}

// U_j = V_j + (G X_j, W_inf)
__global__ void k_add_ambient(int na, const double* __restrict__ V, const double* __restrict__ com,
                              const double* __restrict__ G, const double* __restrict__ W, double* __restrict__ U) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= na) return;
  const double* X = com + 3 * j;
  for (int a = 0; a < 3; ++a) {
    U[6 * j + a] = V[6 * j + a] + G[3 * a] * X[0] + G[3 * a + 1] * X[1] + G[3 * a + 2] * X[2];
    U[6 * j + 3 + a] = V[6 * j + 3 + a] + W[a];
  }
}

void launch_add_ambient(int na, const double* V, const double* com, const double* G, const double* W, double* U,
                        hipStream_t st) {
  k_add_ambient<<<nblocks(na, 128), 128, 0, st>>>(na, V, com, G, W, U);
}

// ------------------------------------------------------------------------------------------
// Krylov vectors (FP64)
// ------------------------------------------------------------------------------------------

namespace {
constexpr int kDotThreads = 256;
constexpr int kDotChunk = 8;  // basis vectors reduced per pass

}  // namespace

int dot_blocks(size_t n) {
  long long b = (long long)((n + kDotThreads - 1) / kDotThreads);
  if (b > 1024) b = 1024;
  if (b < 1) b = 1;
  return int(b);
}

__global__ void k_axpby(size_t n, double a, const double* __restrict__ x, double b, double* __restrict__ y) {
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  y[i] = a * x[i] + b * y[i];
}

__global__ void k_set_value(double* p, double v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

void launch_set_value(double* p, double v, hipStream_t st) { k_set_value<<<1, 64, 0, st>>>(p, v); }

void launch_axpby(size_t n, double a, const double* x, double b, double* y, hipStream_t st) {
  k_axpby<<<nblocks((long long)n), kThreads, 0, st>>>(n, a, x, b, y);
}

// zero n 32-bit words (used instead of a memset so captured graphs hold kernels only)
__global__ void k_zero_words(size_t n, uint32_t* __restrict__ p) {
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

void launch_zero(void* p, size_t bytes, hipStream_t st) {
  const size_t n = bytes / 4;
  k_zero_words<<<nblocks((long long)n), kThreads, 0, st>>>(n, static_cast<uint32_t*>(p));
}

__global__ void k_copy(size_t n, const double* __restrict__ from, double* __restrict__ to) {
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) to[i] = from[i];
}

// either side may be pinned host memory
void launch_copy(size_t n, const double* from, double* to, hipStream_t st) {
  if (n) k_copy<<<nblocks((long long)n), kThreads, 0, st>>>(n, from, to);
}

// An empty kernel launched when per-kernel timing is switched on and again when it is
// switched off: in a profiler trace the launches between the two are the timed ones.
__global__ void k_timing_mark() {}

void launch_timing_mark(hipStream_t st) { k_timing_mark<<<1, 64, 0, st>>>(); }

thread_local LaunchEvents g_launch_events;

__global__ void k_sub(size_t n, const double* __restrict__ b, const double* __restrict__ ax, double* __restrict__ r) {
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  r[i] = b[i] - ax[i];
}

void launch_sub(size_t n, const double* b, const double* ax, double* r, hipStream_t st) {
  k_sub<<<nblocks((long long)n), kThreads, 0, st>>>(n, b, ax, r);
}

// ------------------------------------------------------------------------------------------
// GMRES cycle control on the device (right-preconditioned GMRES(m), Givens QR of H)
// ------------------------------------------------------------------------------------------

// start of a cycle: beta = sqrt(rr), g = (beta, 0, ...), scal = 1/beta; stop when the
// true residual already meets the tolerance or the iteration budget is spent
__global__ void k_gmres_begin(GmresCtl* ctl, const double* __restrict__ rr, double* __restrict__ g,
                              double* __restrict__ scal) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const double beta = sqrt(fmax(rr[0], 0.0));
  ctl->beta = beta;
  ctl->resid = ctl->bn > 0 ? beta / ctl->bn : 0.0;  // b = 0: x = 0 is exact
  ctl->k_used = 0;
  ctl->breakdown = 0;
  for (int i = 0; i <= ctl->m; ++i) g[i] = 0.0;
  g[0] = beta;
  scal[0] = beta > 0 ? 1.0 / beta : 0.0;
  ctl->stop = (ctl->resid <= ctl->tol || ctl->its >= ctl->maxit || beta == 0.0) ? 1 : 0;
}

void launch_gmres_begin(GmresCtl* ctl, const double* rr, double* g, double* scal, hipStream_t st) {
  k_gmres_begin<<<1, 64, 0, st>>>(ctl, rr, g, scal);
}

__global__ void k_gmres_init(GmresCtl* ctl, const double* __restrict__ bb, double tol, int maxit, int m) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  ctl->bn = sqrt(fmax(bb[0], 0.0));
  ctl->tol = tol;
  ctl->maxit = maxit;
  ctl->m = m;
  ctl->its = 0;
  ctl->stop = 0;
  ctl->k_used = 0;
  ctl->breakdown = 0;
  ctl->resid = 1.0;
}

void launch_gmres_init(GmresCtl* ctl, const double* bb, double tol, int maxit, int m, hipStream_t st) {
  k_gmres_init<<<1, 64, 0, st>>>(ctl, bb, tol, maxit, m);
}

// Arnoldi step j: H[:, j] = h1 + h2 (classical Gram-Schmidt, twice), H[j+1, j] = ||w||;
// previous Givens rotations applied, a new one formed, g updated; stop flag raised
// when |g_{j+1}| / ||b|| <= tol, the cycle is full, the budget is spent, or on breakdown.
__device__ void arnoldi_update(const ArnoldiArgs& a, double hn2) {
  GmresCtl* ctl = a.ctl;
  if (ctl->stop) return;
  const int j = a.j, m = ctl->m;
  const double hn = sqrt(fmax(hn2, 0.0));
  // column j of H, rotated by the previous Givens rotations as it streams in
  double ci = a.h1[0] + a.h2[0];
  for (int i = 0; i < j; ++i) {
    const double next = a.h1[i + 1] + a.h2[i + 1];
    a.H[size_t(i) * m + j] = a.cs[i] * ci + a.sn[i] * next;
    ci = -a.sn[i] * ci + a.cs[i] * next;
  }
  const double den = hypot(ci, hn);
  const double c = den > 0 ? ci / den : 1.0, s = den > 0 ? hn / den : 0.0;
  a.cs[j] = c;
  a.sn[j] = s;
  a.H[size_t(j) * m + j] = den;
  a.g[j + 1] = -s * a.g[j];
  a.g[j] = c * a.g[j];
  ctl->k_used = j + 1;
  ctl->its += 1;
  ctl->resid = fabs(a.g[j + 1]) / ctl->bn;
  if (hn == 0.0) ctl->breakdown = 1;
  if (ctl->resid <= ctl->tol || j + 1 == m || ctl->its >= ctl->maxit || hn == 0.0) ctl->stop = 1;
  a.scal[0] = hn > 0 ? 1.0 / hn : 0.0;
}

__global__ void k_arnoldi_step(ArnoldiArgs a, const double* __restrict__ hn2) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  arnoldi_update(a, hn2[0]);
}

void launch_arnoldi_step(const ArnoldiArgs& a, const double* hn2, hipStream_t st) {
  k_arnoldi_step<<<1, 64, 0, st>>>(a, hn2);
}

// y = R^-1 g over the k_used leading rows of the rotated Hessenberg matrix
// y = H^-1 g for the k_used x k_used upper-triangular Hessenberg part (row stride m).  Up to
// 64 columns one wavefront works column by column from LDS: lane q holds row q's running
// value, lane i divides, and y_i reaches the lanes above by a shuffle; larger k go row by row.
__global__ __launch_bounds__(64) void k_gmres_solve(const GmresCtl* ctl, const double* __restrict__ H,
                                                    const double* __restrict__ g, double* __restrict__ y) {
  if (blockIdx.x != 0) return;
  const int k = ctl->k_used, m = ctl->m, q = threadIdx.x;
  if (k <= 64) {
    __shared__ double sh[64 * 64];
    for (int e = q; e < k * k; e += 64) sh[e] = H[size_t(e / k) * m + e % k];
    __syncthreads();
    double t = q < k ? g[q] : 0.0;
    for (int i = k - 1; i >= 0; --i) {
      const double yi = __shfl(q == i ? t / sh[i * k + i] : 0.0, i, 64);
      if (q == i) y[i] = yi;
      if (q < i) t -= sh[q * k + i] * yi;
    }
    return;
  }
  if (q != 0) return;
  for (int i = k - 1; i >= 0; --i) {
    double t = g[i];
    for (int c = i + 1; c < k; ++c) t -= H[size_t(i) * m + c] * y[c];
    y[i] = t / H[size_t(i) * m + i];
  }
}

void launch_gmres_solve(const GmresCtl* ctl, const double* H, const double* g, double* y, hipStream_t st) {
  k_gmres_solve<<<1, 64, 0, st>>>(ctl, H, g, y);
}

// out = sum_{q < k_used} y_q V_q
__global__ void k_basis_combine(size_t n, const double* __restrict__ V, size_t ldv, const double* __restrict__ y,
                                const GmresCtl* __restrict__ ctl, double* __restrict__ out) {
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int k = ctl->k_used;
  double s = 0;
  for (int q = 0; q < k; ++q) s += y[q] * V[size_t(q) * ldv + i];
  out[i] = s;
}

void launch_basis_combine(size_t n, int m, const double* V, size_t ldv, const double* y, const GmresCtl* ctl,
                          double* out, hipStream_t st) {
  (void)m;
  k_basis_combine<<<nblocks((long long)n), kThreads, 0, st>>>(n, V, ldv, y, ctl, out);
}

// ------------------------------------------------------------------------------------------
// fused bead/aggregate kernels: one wavefront per aggregate
// ------------------------------------------------------------------------------------------


__global__ __launch_bounds__(256) void k_agg_lub(int na, const int* __restrict__ offsets, const int* __restrict__ body,
                                                 const double4* __restrict__ r4, const double* __restrict__ lam,
                                                 const double* __restrict__ V, const int* __restrict__ lrow,
                                                 const uint32_t* __restrict__ lcol, const double* __restrict__ coef,
                                                 double* __restrict__ y2, const int* __restrict__ skip) {
  agg_lub_body(na, offsets, body, r4, lam, V, lrow, lcol, coef, y2, skip, blockIdx.x, blockIdx.y, gridDim.x);
}

void launch_agg_lub(int na, const int* offsets, const int* body, const double* r4, const double* lam,
                    const double* V, const int* lrow, const uint32_t* lcol, const double* coef, double* y2,
                    hipStream_t st, const int* skip) {
  launch_k(k_agg_lub, (na + 3) / 4, 256, 0, st, na, offsets, body, (const double4*)r4, lam, V, lrow, lcol, coef, y2, skip);
}

// Preconditioner apply of Section 2.3.3 (block-triangular, block-diagonal Schur
// approximation) in one launch: the wavefront of aggregate j reduces y2 = r2 - Sigma M~^-1 r1
// over its beads, solves z2 = -A_j^-1 y2 in lane 0, and writes z1 = M~^-1 (r1 - Sigma^T z2).
// With scal != nullptr the input is r = scal[0] * src, and r is also stored to vout
// (the next Krylov basis vector is formed here instead of in a separate launch).
__device__ __forceinline__ void precond_fused_body(int nb, int na, const int* __restrict__ offsets,
                                                       const double4* __restrict__ r4, const double* __restrict__ lu,
                                                       const int* __restrict__ piv, double drag_t, double drag_r,
                                                       const double* __restrict__ src, const double* __restrict__ scal,
                                                       double* __restrict__ vout, double* __restrict__ z,
                                                       const int* __restrict__ skip, int bx_, int by_, int gx_) {
  if (skip && *skip) return;
  const int j = bx_ * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (j >= na) return;
  const double sc = scal ? scal[0] : 1.0;
  double p[6] = {0, 0, 0, 0, 0, 0};
  for (int i = offsets[j] + lane; i < offsets[j + 1]; i += 64) {
    const double* ls = src + 6 * size_t(i);
    double l[6];
    for (int c = 0; c < 6; ++c) l[c] = sc * ls[c];
    if (scal)
      for (int c = 0; c < 6; ++c) vout[6 * size_t(i) + c] = l[c];
    const double fx = drag_t * l[0], fy = drag_t * l[1], fz = drag_t * l[2];
    const double4 rv = r4[i];
    p[0] += fx;
    p[1] += fy;
    p[2] += fz;
    p[3] += drag_r * l[3] + (rv.y * fz - rv.z * fy);
    p[4] += drag_r * l[4] + (rv.z * fx - rv.x * fz);
    p[5] += drag_r * l[5] + (rv.x * fy - rv.y * fx);
  }
  double y[6];
  const double* r2 = src + 6 * size_t(nb) + 6 * j;
  for (int c = 0; c < 6; ++c) y[c] = sc * r2[c] - wsum(p[c]);
  if (scal && lane == 0)
    for (int c = 0; c < 6; ++c) vout[6 * size_t(nb) + 6 * j + c] = sc * r2[c];
  // every lane solves the same 6x6 system (uniform work, no broadcast needed)
  const double* A = lu + 36 * size_t(j);
  const int* pv = piv + 6 * size_t(j);
  for (int k = 0; k < 6; ++k) {
    const int q = pv[k];
    if (q != k) {
      const double t = y[k];
      y[k] = y[q];
      y[q] = t;
    }
  }
  for (int a = 1; a < 6; ++a)
    for (int b = 0; b < a; ++b) y[a] -= A[6 * a + b] * y[b];
  for (int a = 5; a >= 0; --a) {
    for (int b = a + 1; b < 6; ++b) y[a] -= A[6 * a + b] * y[b];
    y[a] /= A[6 * a + a];
  }
  for (int c = 0; c < 6; ++c) y[c] = -y[c];  // z2
  if (lane == 0) {
    double* z2 = z + 6 * size_t(nb) + 6 * j;
    for (int c = 0; c < 6; ++c) z2[c] = y[c];
  }
  for (int i = offsets[j] + lane; i < offsets[j + 1]; i += 64) {
    const double4 rv = r4[i];
    const double* ls = src + 6 * size_t(i);
    double l[6];
    for (int c = 0; c < 6; ++c) l[c] = sc * ls[c];
    double* o = z + 6 * size_t(i);
    o[0] = drag_t * (l[0] - (y[0] + (y[4] * rv.z - y[5] * rv.y)));
    o[1] = drag_t * (l[1] - (y[1] + (y[5] * rv.x - y[3] * rv.z)));
    o[2] = drag_t * (l[2] - (y[2] + (y[3] * rv.y - y[4] * rv.x)));
    o[3] = drag_r * (l[3] - y[3]);
    o[4] = drag_r * (l[4] - y[4]);
    o[5] = drag_r * (l[5] - y[5]);
  }
}

__global__ __launch_bounds__(256) void k_precond_fused(int nb, int na, const int* __restrict__ offsets,
                                                       const double4* __restrict__ r4, const double* __restrict__ lu,
                                                       const int* __restrict__ piv, double drag_t, double drag_r,
                                                       const double* __restrict__ src, const double* __restrict__ scal,
                                                       double* __restrict__ vout, double* __restrict__ z,
                                                       const int* __restrict__ skip) {
  precond_fused_body(nb, na, offsets, r4, lu, piv, drag_t, drag_r, src, scal, vout, z, skip, blockIdx.x, blockIdx.y, gridDim.x);
}

void launch_precond_fused(int nb, int na, const int* offsets, const double* r4, const double* lu, const int* piv,
                          double drag_t, double drag_r, const double* src, const double* scal, double* vout, double* z,
                          hipStream_t st, const int* skip) {
  launch_k(k_precond_fused, (na + 3) / 4, 256, 0, st, nb, na, offsets, (const double4*)r4, lu, piv, drag_t, drag_r, src,
                                                 scal, vout, z, skip);
}

// ------------------------------------------------------------------------------------------
// fused CGS2 kernels: one launch each, the last block to finish reduces the per-block
// partial sums in block order (deterministic) and resets its ticket counter
// ------------------------------------------------------------------------------------------

namespace {
// block-level sums of `cnt` (<= 8) per-thread values; result valid in thread 0
__device__ inline void block_sums8(double* acc, int cnt, double* sh /* [8][kDotThreads/64] */) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  for (int c = 0; c < cnt; ++c) {
    double v = acc[c];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    if (l == 0) sh[c * (kDotThreads / 64) + w] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    for (int c = 0; c < cnt; ++c) {
      double t = 0;
      for (int k = 0; k < kDotThreads / 64; ++k) t += sh[c * (kDotThreads / 64) + k];
      acc[c] = t;
    }
  __syncthreads();
}

// partial[q * G + block] are complete for q in [q0, q0 + cnt): the last block reduces them
__device__ inline void finish_dots(int q0, int cnt, const double* __restrict__ partial, double* __restrict__ out,
                                   unsigned* counter, double* sh) {
  __shared__ int last;
  __threadfence();
  if (threadIdx.x == 0) last = (atomicAdd(counter, 1u) == gridDim.x - 1) ? 1 : 0;
  __syncthreads();
  if (!last) return;
  __threadfence();
  double acc[kDotChunk];
  for (int c = 0; c < cnt; ++c) {
    double v = 0;
    for (int b = threadIdx.x; b < int(gridDim.x); b += blockDim.x) v += partial[size_t(q0 + c) * gridDim.x + b];
    acc[c] = v;
  }
  block_sums8(acc, cnt, sh);
  if (threadIdx.x == 0) {
    for (int c = 0; c < cnt; ++c) out[q0 + c] = acc[c];
    *counter = 0u;
  }
}
}  // namespace

// h[q] = V_q . w, q < nq (blockIdx.y selects a chunk of 8 basis vectors)
__global__ __launch_bounds__(kDotThreads) void k_dots(size_t n, int nq, const double* __restrict__ V, size_t ldv,
                                                      const double* __restrict__ w, double* __restrict__ partial,
                                                      double* __restrict__ out, unsigned* counters,
                                                      const int* __restrict__ skip) {
  if (skip && *skip) return;
  __shared__ double sh[kDotChunk * (kDotThreads / 64)];
  const int q0 = blockIdx.y * kDotChunk, cnt = min(kDotChunk, nq - q0);
  double acc[kDotChunk];
#pragma unroll
  for (int c = 0; c < kDotChunk; ++c) acc[c] = 0;
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x) {
    const double wi = w[i];
#pragma unroll
    for (int c = 0; c < kDotChunk; ++c)
      if (c < cnt) acc[c] += V[size_t(q0 + c) * ldv + i] * wi;
  }
  block_sums8(acc, cnt, sh);
  if (threadIdx.x == 0)
    for (int c = 0; c < cnt; ++c) partial[size_t(q0 + c) * gridDim.x + blockIdx.x] = acc[c];
  finish_dots(q0, cnt, partial, out, counters + blockIdx.y, sh);
}

// w -= sum_q h[q] V_q, then (mode 0) out[q] = V_q . w for q < nq, or (mode 1) out[0] = w . w
__global__ __launch_bounds__(kDotThreads) void k_axpy_dots(size_t n, int nq, const double* __restrict__ V, size_t ldv,
                                                           const double* __restrict__ h, double* __restrict__ w,
                                                           int mode, double* __restrict__ partial,
                                                           double* __restrict__ out, unsigned* counters,
                                                           const int* __restrict__ skip) {
  if (skip && *skip) return;
  __shared__ double sh[kDotChunk * (kDotThreads / 64)];
  // the update is element-local, so each thread updates the elements it later reduces
  for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x) {
    double s = 0;
    for (int q = 0; q < nq; ++q) s += h[q] * V[size_t(q) * ldv + i];
    w[i] -= s;
  }
  const int nout = mode == 0 ? nq : 1;
  for (int q0 = 0; q0 < nout; q0 += kDotChunk) {
    const int cnt = min(kDotChunk, nout - q0);
    double acc[kDotChunk];
#pragma unroll
    for (int c = 0; c < kDotChunk; ++c) acc[c] = 0;
    for (size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x) {
      const double wi = w[i];
      if (mode == 0) {
#pragma unroll
        for (int c = 0; c < kDotChunk; ++c)
          if (c < cnt) acc[c] += V[size_t(q0 + c) * ldv + i] * wi;
      } else {
        acc[0] += wi * wi;
      }
    }
    block_sums8(acc, cnt, sh);
    if (threadIdx.x == 0)
      for (int c = 0; c < cnt; ++c) partial[size_t(q0 + c) * gridDim.x + blockIdx.x] = acc[c];
    finish_dots(q0, cnt, partial, out, counters + q0 / kDotChunk, sh);
  }
}

// One inner product, the norms at a cycle's start.  A single workgroup up to kDotOne values, beyond
// it a pass that leaves a partial sum per workgroup and one that adds them: a launch between two
// passes costs less than the device-wide fence of finish_dots, which waits for whatever the chip
// still has to write back (516,000 values 66 -> 9.1 us, 12,500 8.7 -> 5.5).
constexpr size_t kDotOne = 32768;

template <int T>
__device__ __forceinline__ void block_sum_to(double v, double* out) {
  __shared__ double sh[T / 64];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0;
#pragma unroll
    for (int k = 0; k < T / 64; ++k) s += sh[k];
    *out = s;
  }
}

template <int T>
__global__ __launch_bounds__(T) void k_dot(size_t n, const double* __restrict__ a, const double* __restrict__ b,
                                           double* __restrict__ out, const int* __restrict__ skip) {
  if (skip && *skip) return;
  const size_t step = size_t(gridDim.x) * T;
  double v[4] = {0, 0, 0, 0};
  size_t i = size_t(blockIdx.x) * T + threadIdx.x;
  for (; i + 3 * step < n; i += 4 * step)
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] += a[i + k * step] * b[i + k * step];
  for (; i < n; i += step) v[0] += a[i] * b[i];
  block_sum_to<T>((v[0] + v[1]) + (v[2] + v[3]), out + blockIdx.x);
}

__global__ __launch_bounds__(256) void k_dot_sum(int n, const double* __restrict__ partial, double* __restrict__ out,
                                                 const int* __restrict__ skip) {
  if (skip && *skip) return;
  block_sum_to<256>(int(threadIdx.x) < n ? partial[threadIdx.x] : 0.0, out);
}

void launch_dots(size_t n, int nq, const double* V, size_t ldv, const double* w, double* partial, double* out,
                 unsigned* counters, hipStream_t st, const int* skip) {
  if (nq == 1) {
    if (n <= kDotOne) {
      launch_k(k_dot<1024>, 1, 1024, 0, st, n, V, w, out, skip);
    } else {
      launch_k(k_dot<256>, 256, 256, 0, st, n, V, w, partial, skip);
      launch_k(k_dot_sum, 1, 256, 0, st, 256, partial, out, skip);
    }
    return;
  }
  dim3 g(dot_blocks(n), (nq + kDotChunk - 1) / kDotChunk);
  launch_k(k_dots, g, kDotThreads, 0, st, n, nq, V, ldv, w, partial, out, counters, skip);
}

void launch_axpy_dots(size_t n, int nq, const double* V, size_t ldv, const double* h, double* w, int mode,
                      double* partial, double* out, unsigned* counters, hipStream_t st, const int* skip) {
  launch_k(k_axpy_dots, dot_blocks(n), kDotThreads, 0, st, n, nq, V, ldv, h, w, mode, partial, out, counters, skip);
}

// ------------------------------------------------------------------------------------------
// CGS2 passes with the basis in registers (restart length < kCgsMax).  Each lane holds
// its element of every basis vector, so the update and the new inner products read the
// basis once.  The nq per-lane sums are reduced across a wavefront by recursive halving
// (31 lane exchanges for 32 values instead of 6 per value), the four wavefronts of a
// workgroup through LDS.  The last workgroup to finish adds the per-workgroup partials
// in a fixed order (deterministic) and resets its ticket.
// ------------------------------------------------------------------------------------------

namespace {
constexpr int kCgsMax = 32;
constexpr int kCgsThreads = 256;
constexpr int kCgsWaves = kCgsThreads / 64;
constexpr int kCgsBlocks = 512;

// halving step: lanes with (lane & D) keep the upper half of a[0..2C), the others the
// lower half; the half given away is added by the partner lane (lane ^ D)
template <int C, int D>
__device__ inline void halve(double (&a)[kCgsMax], int lane) {
  const bool up = (lane & D) != 0;
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const double send = up ? a[j] : a[j + C];
    const double keep = up ? a[j + C] : a[j];
    a[j] = keep + __shfl_xor(send, D, 64);
  }
}

// total over the 64 lanes of a[q], returned in every lane whose cgs_q(lane) == q
__device__ inline double wave_transpose_sum(double (&a)[kCgsMax], int lane) {
  halve<16, 32>(a, lane);
  halve<8, 16>(a, lane);
  halve<4, 8>(a, lane);
  halve<2, 4>(a, lane);
  halve<1, 2>(a, lane);
  return a[0] + __shfl_xor(a[0], 1, 64);
}

__device__ inline int cgs_q(int lane) {
  return ((lane >> 5) & 1) * 16 + ((lane >> 4) & 1) * 8 + ((lane >> 3) & 1) * 4 + ((lane >> 2) & 1) * 2 +
         ((lane >> 1) & 1);
}

__device__ inline double wave_total(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// workgroup sums of acc[q], q < nout (nout == 1: acc[0] only); valid in sh[0][q] after the call
__device__ inline void block_sums(double (&acc)[kCgsMax], int nout, double (*sh)[kCgsMax]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (nout > 1) {
    const double tot = wave_transpose_sum(acc, lane);
    const int q = cgs_q(lane);
    if (!(lane & 1)) sh[wave][q] = tot;
  } else {
    const double tot = wave_total(acc[0]);
    if (lane == 0) sh[wave][0] = tot;
  }
  __syncthreads();
  if (threadIdx.x < nout) {
    double s = 0.0;
    for (int w = 0; w < kCgsWaves; ++w) s += sh[w][threadIdx.x];
    sh[0][threadIdx.x] = s;  // each thread rewrites only its own column, after reading it
  }
  __syncthreads();
}

// Arnoldi update with the column, rotations and sines staged in LDS (j < kCgsMax)
__device__ void arnoldi_update_staged(const ArnoldiArgs& a, double hn2, double* col, double* cs, double* sn) {
  GmresCtl* ctl = a.ctl;
  const int j = a.j;
  const bool stop = ctl->stop;
  if (!stop)
    for (int i = threadIdx.x; i <= j; i += blockDim.x) {
      col[i] = a.h1[i] + a.h2[i];
      cs[i] = a.cs[i];
      sn[i] = a.sn[i];
    }
  __syncthreads();
  if (stop || threadIdx.x != 0) return;
  const int m = ctl->m;
  const double hn = sqrt(fmax(hn2, 0.0));
  double ci = col[0];
  for (int i = 0; i < j; ++i) {
    const double next = col[i + 1];
    a.H[size_t(i) * m + j] = cs[i] * ci + sn[i] * next;
    ci = -sn[i] * ci + cs[i] * next;
  }
  const double den = hypot(ci, hn);
  const double c = den > 0 ? ci / den : 1.0, s = den > 0 ? hn / den : 0.0;
  a.cs[j] = c;
  a.sn[j] = s;
  a.H[size_t(j) * m + j] = den;
  const double gj = a.g[j];
  a.g[j + 1] = -s * gj;
  a.g[j] = c * gj;
  ctl->k_used = j + 1;
  ctl->its += 1;
  ctl->resid = fabs(s * gj) / ctl->bn;
  if (hn == 0.0) ctl->breakdown = 1;
  if (ctl->resid <= ctl->tol || j + 1 == m || ctl->its >= ctl->maxit || hn == 0.0) ctl->stop = 1;
  a.scal[0] = hn > 0 ? 1.0 / hn : 0.0;
}
}  // namespace

int cgs_blocks(size_t n) {
  long long b = (long long)((n + kCgsThreads - 1) / kCgsThreads);
  return int(b < 1 ? 1 : (b > kCgsBlocks ? kCgsBlocks : b));
}

// The CGS2 passes, MODE 0: out[q] = V_q . w (first Gram-Schmidt pass); MODE 1: w -= sum_q
// hin[q] V_q, out[q] = V_q . w (second pass, fused with the first update); MODE 2: w -= sum_q
// hin[q] V_q, out[0] = w . w.  Each workgroup writes its partial sums; the next launch of the
// chain adds them (reduce_partials).

// out[q] = sum over b of part[q * nblk + b] for q < nq (<= kCgsMax), in the same fixed order
// in every workgroup: thread t adds the terms b = t / 32 + 8 k of column q = t % 32, and the
// eight partial sums of a column are then added in order.  Valid in out[] after the call.
__device__ inline void reduce_partials(const double* __restrict__ part, int nblk, int nq, double* shq, double* out) {
  static_assert(kCgsThreads == 256 && kCgsMax == 32, "8 parts of 32 columns");
  const int q = threadIdx.x & 31, p = threadIdx.x >> 5;
  double v = 0.0;
  if (q < nq)
    for (int b = p; b < nblk; b += 8) v += part[size_t(q) * nblk + b];
  shq[p * 32 + q] = v;
  __syncthreads();
  if (threadIdx.x < nq) {
    double t = 0.0;
    for (int k = 0; k < 8; ++k) t += shq[k * 32 + threadIdx.x];
    out[threadIdx.x] = t;
  }
  __syncthreads();
}

// One CGS2 pass of the fence-free chain (see launch_cgs_chain): workgroup bx of nblk.
template <int MODE>
__device__ __forceinline__ void cgs_chain_body(size_t n, int nq, const double* __restrict__ V, size_t ldv,
                                               const double* __restrict__ pin, double* __restrict__ w,
                                               double* __restrict__ pout, double* __restrict__ hout, int bx,
                                               int nblk) {
  __shared__ double sh[kCgsWaves][kCgsMax];
  __shared__ double shq[8 * 32];
  __shared__ double hq[kCgsMax];
  if (MODE >= 1) {
    reduce_partials(pin, nblk, nq, shq, hq);
    if (bx == 0 && threadIdx.x < nq) hout[threadIdx.x] = hq[threadIdx.x];
  }
  double h[kCgsMax], acc[kCgsMax];
#pragma unroll
  for (int q = 0; q < kCgsMax; ++q) {
    h[q] = (MODE >= 1 && q < nq) ? hq[q] : 0.0;
    acc[q] = 0.0;
  }
  for (size_t i = size_t(bx) * kCgsThreads + threadIdx.x; i < n; i += size_t(nblk) * kCgsThreads) {
    double v[kCgsMax];
#pragma unroll
    for (int q = 0; q < kCgsMax; ++q) v[q] = q < nq ? V[size_t(q) * ldv + i] : 0.0;
    double wi = w[i];
    if (MODE >= 1) {
      double sv = 0.0;
#pragma unroll
      for (int q = 0; q < kCgsMax; ++q) sv += h[q] * v[q];
      wi -= sv;
      w[i] = wi;
    }
    if (MODE <= 1) {
#pragma unroll
      for (int q = 0; q < kCgsMax; ++q) acc[q] += v[q] * wi;
    } else {
      acc[0] += wi * wi;
    }
  }
  const int nout = MODE <= 1 ? nq : 1;
  block_sums(acc, nout, sh);
  if (threadIdx.x < nout) pout[size_t(threadIdx.x) * nblk + bx] = sh[0][threadIdx.x];
}

template <int MODE>
__global__ __launch_bounds__(kCgsThreads) void k_cgs_chain(size_t n, int nq, const double* __restrict__ V, size_t ldv,
                                                           const double* __restrict__ pin, double* __restrict__ w,
                                                           double* __restrict__ pout, double* __restrict__ hout,
                                                           const int* __restrict__ skip) {
  if (skip && *skip) return;
  cgs_chain_body<MODE>(n, nq, V, ldv, pin, w, pout, hout, blockIdx.x, gridDim.x);
}

// ------------------------------------------------------------------------------------------
// Lanczos steps of the Brownian square roots: the passes of the chain above for any number of
// basis vectors (the roots take up to lanczos_maxit).  Each workgroup owns a slice of the vectors
// and walks the basis 32 vectors at a time; partial sums go to part[b nq + q] and every workgroup of
// the next pass adds them in the same fixed order.  The earlier form (8 vectors at a time, the last
// workgroup adding the partials after a fence and a ticket) took 141 us for the three passes of a
// step at 50 of 100 vectors of 18,033 (6,011 beads), seven launches a step; these take 38, five launches.
// MODE 0: partials of V^T w.  MODE 1: h = the summed partials, w -= V h, partials of V^T w; *coef =
// the last of h.  MODE 2: the same update, partials of w.w; *coef += the last of h.  MODE 3: partials
// of w.w alone.
// ------------------------------------------------------------------------------------------
namespace {
constexpr int kLanBlocks = 256;  // partials a workgroup adds in one sweep of its threads
}

int lanczos_blocks(size_t n) { return int(std::min<size_t>((n + kCgsThreads - 1) / kCgsThreads, kLanBlocks)); }

template <int MODE>
__global__ __launch_bounds__(kCgsThreads) void k_lanczos_pass(size_t n, int nq, const double* __restrict__ V,
                                                              const double* __restrict__ pin, double* __restrict__ w,
                                                              double* __restrict__ pout, double* __restrict__ coef) {
  extern __shared__ double h[];  // nq
  __shared__ double sh[kCgsWaves][kCgsMax];
  __shared__ double other[128];
  const int t = threadIdx.x, G = gridDim.x;
  const size_t i0 = size_t(blockIdx.x) * kCgsThreads + t, step = size_t(G) * kCgsThreads;
  if (MODE == 1 || MODE == 2) {
    const int c = t & 127, mid = (G + 1) / 2, b0 = t < 128 ? 0 : mid, b1 = t < 128 ? mid : G;
    for (int q0 = 0; q0 < nq; q0 += 128) {
      double v = 0.0;
      if (q0 + c < nq) {
#pragma unroll 8
        for (int b = b0; b < b1; ++b) v += pin[size_t(b) * nq + q0 + c];
      }
      if (t >= 128) other[c] = v;
      __syncthreads();
      if (t < 128 && q0 + c < nq) h[q0 + c] = v + other[c];
      __syncthreads();
    }
    if (blockIdx.x == 0 && t == 0) coef[0] = MODE == 1 ? h[nq - 1] : coef[0] + h[nq - 1];
    for (size_t i = i0; i < n; i += step) {
      double s = 0.0;
#pragma unroll 16
      for (int q = 0; q < nq; ++q) s += h[q] * V[size_t(q) * n + i];
      w[i] -= s;
    }
  }
  double acc[kCgsMax];
  if (MODE <= 1) {
    for (int q0 = 0; q0 < nq; q0 += kCgsMax) {
      const int cnt = min(kCgsMax, nq - q0);
#pragma unroll
      for (int u = 0; u < kCgsMax; ++u) acc[u] = 0.0;
      for (size_t i = i0; i < n; i += step) {
        const double wi = w[i];
#pragma unroll
        for (int u = 0; u < kCgsMax; ++u)
          if (u < cnt) acc[u] += V[size_t(q0 + u) * n + i] * wi;
      }
      block_sums(acc, cnt, sh);
      if (t < cnt) pout[size_t(blockIdx.x) * nq + q0 + t] = sh[0][t];
      __syncthreads();
    }
  } else {
    acc[0] = 0.0;
    for (size_t i = i0; i < n; i += step) acc[0] += w[i] * w[i];
    block_sums(acc, 1, sh);
    if (t == 0) pout[blockIdx.x] = sh[0][0];
  }
}

// beta = ||w|| from the G <= 256 partials pin (stored to *beta), v = w / beta (0 at a breakdown);
// v == nullptr: the norm alone
__global__ __launch_bounds__(kCgsThreads) void k_lanczos_next(size_t n, int G, const double* __restrict__ pin,
                                                              const double* __restrict__ w, double* __restrict__ v,
                                                              double* __restrict__ beta) {
  __shared__ double sh[kCgsWaves];
  const double tot = wave_total(int(threadIdx.x) < G ? pin[threadIdx.x] : 0.0);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = tot;
  __syncthreads();
  const double b = sqrt(fmax(sh[0] + sh[1] + sh[2] + sh[3], 0.0)), sc = b > 0 ? 1.0 / b : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) *beta = b;
  const size_t i = size_t(blockIdx.x) * kCgsThreads + threadIdx.x;
  if (v && i < n) v[i] = sc * w[i];
}

void launch_lanczos_pass(int mode, size_t n, int nq, const double* V, const double* pin, double* w, double* pout,
                         double* coef, hipStream_t st) {
  const int g = lanczos_blocks(n);
  const uint32_t shm = uint32_t(sizeof(double)) * nq;
  if (mode == 0)
    launch_k(k_lanczos_pass<0>, g, kCgsThreads, shm, st, n, nq, V, pin, w, pout, coef);
  else if (mode == 1)
    launch_k(k_lanczos_pass<1>, g, kCgsThreads, shm, st, n, nq, V, pin, w, pout, coef);
  else if (mode == 2)
    launch_k(k_lanczos_pass<2>, g, kCgsThreads, shm, st, n, nq, V, pin, w, pout, coef);
  else
    launch_k(k_lanczos_pass<3>, g, kCgsThreads, shm, st, n, nq, V, pin, w, pout, coef);
}

void launch_lanczos_next(size_t n, const double* pin, const double* w, double* v, double* beta, hipStream_t st) {
  const int g = v ? nblocks((long long)n, kCgsThreads) : 1;
  launch_k(k_lanczos_next, g, kCgsThreads, 0, st, n, lanczos_blocks(n), pin, w, v, beta);
}

// w.w from the mode-2 partials, then the Arnoldi update (one workgroup)
__global__ __launch_bounds__(kCgsThreads) void k_arnoldi_reduce(ArnoldiArgs a, const double* __restrict__ pin, int nblk,
                                                                double* __restrict__ hn2) {
  if (a.ctl->stop) return;
  __shared__ double shq[8 * 32];
  __shared__ double tot[kCgsMax];
  __shared__ double st[3][kCgsMax];
  reduce_partials(pin, nblk, 1, shq, tot);
  if (threadIdx.x == 0) *hn2 = tot[0];
  arnoldi_update_staged(a, tot[0], st[0], st[1], st[2]);
}

bool cgs_fits(int nq) { return nq >= 1 && nq <= kCgsMax; }

void launch_cgs_chain(int mode, size_t n, int nq, const double* V, size_t ldv, const double* pin, double* w,
                      double* pout, double* hout, hipStream_t st, const int* skip) {
  const int g = cgs_blocks(n);
  if (mode == 0)
    launch_k(k_cgs_chain<0>, g, kCgsThreads, 0, st, n, nq, V, ldv, pin, w, pout, hout, skip);
  else if (mode == 1)
    launch_k(k_cgs_chain<1>, g, kCgsThreads, 0, st, n, nq, V, ldv, pin, w, pout, hout, skip);
  else
    launch_k(k_cgs_chain<2>, g, kCgsThreads, 0, st, n, nq, V, ldv, pin, w, pout, hout, skip);
}

void launch_arnoldi_reduce(const ArnoldiArgs& a, const double* pin, int nblk, double* hn2, hipStream_t st) {
  k_arnoldi_reduce<<<1, kCgsThreads, 0, st>>>(a, pin, nblk, hn2);
}

// The preconditioner of Arnoldi step j+1 with step j's Arnoldi update folded in: every
// workgroup reduces the ||w||^2 partials in the same fixed order (so all hold the same
// value), takes v_(j+1) = w / ||w|| and applies the preconditioner; workgroup 0 also makes
// the Hessenberg/Givens update and the stop decision of step j.  Once that update stops the
// cycle, the vectors this launch writes are not used.
__device__ __forceinline__ void precond_arnoldi_body(int nb, int na, const int* __restrict__ offsets,
                                                    const double4* __restrict__ r4, const double* __restrict__ lu,
                                                    const int* __restrict__ piv, double drag_t, double drag_r,
                                                    const double* __restrict__ src, double* __restrict__ vout,
                                                    double* __restrict__ z, const ArnoldiArgs& a,
                                                    const double* __restrict__ pin, int nblk,
                                                    double* __restrict__ hn2, const int* __restrict__ skip, int bx) {
  // workgroup 0 of this very launch may raise the stop flag while others start, so each
  // workgroup reads it once and all its wavefronts take the same branch (the barriers
  // below need every wavefront)
  __shared__ int quit;
  if (threadIdx.x == 0) quit = skip ? __atomic_load_n(skip, __ATOMIC_RELAXED) : 0;
  __syncthreads();
  if (quit) return;
  __shared__ double shq[8 * 32];
  __shared__ double tot[kCgsMax];
  __shared__ double st[3][kCgsMax];
  __shared__ double sc;
  reduce_partials(pin, nblk, 1, shq, tot);
  if (bx == 0) {
    if (threadIdx.x == 0) *hn2 = tot[0];
    arnoldi_update_staged(a, tot[0], st[0], st[1], st[2]);
  }
  if (threadIdx.x == 0) {
    const double hn = sqrt(fmax(tot[0], 0.0));  // as the update's scal
    sc = hn > 0 ? 1.0 / hn : 0.0;
  }
  __syncthreads();
  precond_fused_body(nb, na, offsets, r4, lu, piv, drag_t, drag_r, src, &sc, vout, z, nullptr, bx, 0, 0);
}

__global__ __launch_bounds__(256) void k_precond_arnoldi(int nb, int na, const int* __restrict__ offsets,
                                                         const double4* __restrict__ r4, const double* __restrict__ lu,
                                                         const int* __restrict__ piv, double drag_t, double drag_r,
                                                         const double* __restrict__ src, double* __restrict__ vout,
                                                         double* __restrict__ z, ArnoldiArgs a,
                                                         const double* __restrict__ pin, int nblk,
                                                         double* __restrict__ hn2, const int* __restrict__ skip) {
  precond_arnoldi_body(nb, na, offsets, r4, lu, piv, drag_t, drag_r, src, vout, z, a, pin, nblk, hn2, skip,
                       blockIdx.x);
}

void launch_precond_arnoldi(int nb, int na, const int* offsets, const double* r4, const double* lu, const int* piv,
                            double drag_t, double drag_r, const double* src, double* vout, double* z,
                            const ArnoldiArgs& a, const double* pin, int nblk, double* hn2, hipStream_t st,
                            const int* skip) {
  launch_k(k_precond_arnoldi, (na + 3) / 4, 256, 0, st, nb, na, offsets, (const double4*)r4, lu, piv, drag_t, drag_r,
           src, vout, z, a, pin, nblk, hn2, skip);
}

// ------------------------------------------------------------------------------------------
// multi-system launches of the preconditioner, the Sigma/lubrication reduction and the
// CGS2 passes (block -> system by the prefix table; see BatchDesc)
// ------------------------------------------------------------------------------------------

// Arnoldi step j: v_j = scal * (j == 0 ? r : w) formed in the preconditioner, z = P^-1 v_j
__global__ __launch_bounds__(256) void kb_precond(const BatchDesc* __restrict__ D, const int* __restrict__ off,
                                                 int nsys, int j) {
  const int s = batch_system(off, nsys, blockIdx.x);
  const BatchDesc& d = D[s];
  precond_fused_body(d.nb, d.na, d.offsets, (const double4*)d.r4, d.lu, d.piv, d.drag_t, d.drag_r, j == 0 ? d.r : d.w,
                     d.scal, d.basis + size_t(j) * d.n, d.z, &d.ctl->stop, blockIdx.x - off[s], 0, 0);
}

__global__ __launch_bounds__(256) void kb_agg(const BatchDesc* __restrict__ D, const int* __restrict__ off,
                                             int nsys) {
  const int s = batch_system(off, nsys, blockIdx.x);
  const BatchDesc& d = D[s];
  const size_t nb6 = 6 * size_t(d.nb);
  agg_lub_body(d.na, d.offsets, d.body, (const double4*)d.r4, d.z, d.z + nb6, d.lrow, d.lcol, d.lcoef, d.w + nb6,
               &d.ctl->stop, blockIdx.x - off[s], 0, 0);
}

// The fence-free CGS2 chain of every system (partials P0, P1, P2 of the system's part
// array, as the single-system chain): pass MODE of Arnoldi step j
template <int MODE>
__global__ __launch_bounds__(kCgsThreads) void kb_cgs(const BatchDesc* __restrict__ D, const int* __restrict__ off,
                                                     int nsys, int j) {
  const int s = batch_system(off, nsys, blockIdx.x);
  const BatchDesc& d = D[s];
  if (d.ctl->stop) return;
  const int G = d.ncgs;
  const double* pin = MODE == 0 ? nullptr : d.part + size_t(32) * G * (MODE - 1);
  double* pout = d.part + size_t(32) * G * MODE;
  double* hout = MODE == 1 ? d.h1 : d.h2;
  cgs_chain_body<MODE>(d.n, j + 1, d.basis, d.n, pin, d.w, pout, hout, blockIdx.x - off[s], G);
}

// Arnoldi step j > 0 inside a segment: step j-1's update (from its ||w||^2 partials) folded
// into the preconditioner that forms v_j, as k_precond_arnoldi
__global__ __launch_bounds__(256) void kb_precond_arnoldi(const BatchDesc* __restrict__ D,
                                                         const int* __restrict__ off, int nsys, int j) {
  const int s = batch_system(off, nsys, blockIdx.x);
  const BatchDesc& d = D[s];
  const ArnoldiArgs prev{j - 1, d.ctl, d.h1, d.h2, d.H, d.gcs, d.gsn, d.g, d.scal};
  precond_arnoldi_body(d.nb, d.na, d.offsets, (const double4*)d.r4, d.lu, d.piv, d.drag_t, d.drag_r, d.w,
                       d.basis + size_t(j) * d.n, d.z, prev, d.part + size_t(64) * d.ncgs, d.ncgs, d.hn2,
                       &d.ctl->stop, blockIdx.x - off[s]);
}

// the last step of a segment: its Arnoldi update alone, one workgroup per system
__global__ __launch_bounds__(kCgsThreads) void kb_arnoldi_reduce(const BatchDesc* __restrict__ D, int nsys, int j) {
  const BatchDesc& d = D[blockIdx.x];
  if (d.ctl->stop) return;
  __shared__ double shq[8 * 32];
  __shared__ double tot[kCgsMax];
  __shared__ double st[3][kCgsMax];
  const ArnoldiArgs a{j, d.ctl, d.h1, d.h2, d.H, d.gcs, d.gsn, d.g, d.scal};
  reduce_partials(d.part + size_t(64) * d.ncgs, d.ncgs, 1, shq, tot);
  if (threadIdx.x == 0) *d.hn2 = tot[0];
  arnoldi_update_staged(a, tot[0], st[0], st[1], st[2]);
}

// every system's stop flag into one array (one read-back per lock-step segment)
__global__ void kb_gather_stop(const BatchDesc* __restrict__ D, int nsys, int* __restrict__ out) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < nsys) out[k] = D[k].ctl->stop;
}

void launch_batch_gather_stop(const BatchDesc* D, int nsys, int* out, hipStream_t st) {
  if (nsys > 0) kb_gather_stop<<<(nsys + 255) / 256, 256, 0, st>>>(D, nsys, out);
}

void launch_batch_solver(int kind, int j, int cgs_mode, const BatchDesc* D, const int* off, int nsys, int total,
                         hipStream_t st) {
  if (total <= 0) return;
  if (kind == BK_PRECOND)
    kb_precond<<<total, 256, 0, st>>>(D, off, nsys, j);
  else if (kind == BK_PRECOND_ARNOLDI)
    kb_precond_arnoldi<<<total, 256, 0, st>>>(D, off, nsys, j);
  else if (kind == BK_ARNOLDI)
    kb_arnoldi_reduce<<<nsys, kCgsThreads, 0, st>>>(D, nsys, j);
  else if (kind == BK_AGG)
    kb_agg<<<total, 256, 0, st>>>(D, off, nsys);
  else if (kind == BK_CGS && cgs_mode == 0)
    kb_cgs<0><<<total, kCgsThreads, 0, st>>>(D, off, nsys, j);
  else if (kind == BK_CGS && cgs_mode == 1)
    kb_cgs<1><<<total, kCgsThreads, 0, st>>>(D, off, nsys, j);
  else if (kind == BK_CGS)
    kb_cgs<2><<<total, kCgsThreads, 0, st>>>(D, off, nsys, j);
}

}  // namespace fsd
