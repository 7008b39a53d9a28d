// Device set-up and operator application of libaim (gfx950).
//
//  * kernel sampling:  c[d] = g(eps |d|) for |d| <= m - 1, c[0] = 0 (Sec.
//    III-C), the other offsets of the length-n embedding (n >= 2m; for n = 2m
//    the ring |d| = m) zero; spectrum F(c) by the FFT kernels (eq. (8))
//  * numerical filter: quarter spectrum masked to |kappa| <= alpha (Sec. III-B)
//  * near field: exact Galerkin entries of eq. (4) / the Maue form of eq. (2)
//    minus their grid approximation, FP64, 16 lanes per nonzero; singular
//    segment pairs use the log/regular split g = -(1/2pi) J0(kR) ln R + F(R)
//  * anterpolation (transposed stencils, gather per active grid point) and
//    interpolation fused with the near-field product (16 lanes per row)
//  * Gram solve G^-1 (Sec. II): pulses diagonal, hats cyclic tridiagonal
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <mutex>
#include <type_traits>
#include <utility>

#include "aim_internal.h"
#include "wave.h"

namespace aim {

template <typename T>
aim_status launch_rows_fwd(int n, const cplx<T>* U, int n_act, const int32_t* row_ptr,
                           const int32_t* act_ix, int nr, int ldt, int kcut, int pairs, cplx<T>* Tb,
                           const cplx<T>* tw, hipStream_t s);
template <typename T>
aim_status launch_rows_fwd_at(int n, const AtMap& at, const double2* x, int64_t ldx, int nrhs, const int32_t* row_ptr,
                              const int32_t* act_ix, int nr, int ldt, int kcut, int pairs, cplx<T>* Tb,
                              const cplx<T>* tw, hipStream_t s);
bool rows_few_columns(int n, bool f32, int kcut, int n_act, int nr);
template <typename T>
aim_status launch_rows_inv(int n, const cplx<T>* Tb, int nr, int ldt, int kcut, const int32_t* row_ptr,
                           const int32_t* act_ix, int pairs, cplx<T>* V, int n_act,
                           const cplx<T>* tw, hipStream_t s);
template <typename T>
aim_status launch_cols(int n, int mode, cplx<T>* Tb, int nr, int ldt, int kcut, int pairs, const cplx<T>* Cq,
                       const cplx<T>* tw, hipStream_t s, hipEvent_t ev_start = nullptr,
                       hipEvent_t ev_stop = nullptr);
aim_status launch_rows_fft_inplace(int n, double2* A, const double2* tw, hipStream_t s);
template <typename T>
aim_status launch_cols_group(int n, int count, void* const* tiles, const int* nr, const int* ldt, int kcut,
                             const cplx<T>* Cq, const cplx<T>* tw, hipStream_t s);
int col_block(int n, bool f32);

static constexpr double kPi = 3.14159265358979323846264338327950288;
static constexpr double kInv2Pi = 0.15915494309189533576888376337251436;
static constexpr double kEuler = 0.57721566490153286060651209008240243;

// ---------------------------------------------------------------------------
// Green's function and its regular part
// ---------------------------------------------------------------------------
__device__ __forceinline__ double2 green(double R, double k) {
  const double x = k * R;
  return make_double2(-0.25 * y0(x), -0.25 * j0(x));
}

// F(R) = g(R) + (1/2pi) J0(kR) ln R (entire in R^2).  Ascending series for
// kR < 2:  Y0(x) = (2/pi)[(ln(x/2) + gamma) J0(x) + sum_{m>=1} (-1)^{m+1} H_m q^m/(m!)^2],
// q = x^2/4.
__device__ double2 green_regular(double R, double k) {
  const double x = k * R;
  if (x < 2.0) {
    const double q = 0.25 * x * x;
    double t = 1.0, jj = 1.0, S = 0.0, Hm = 0.0;
    for (int m = 1; m < 40; ++m) {
      t *= q / ((double)m * (double)m);
      Hm += 1.0 / m;
      if (m & 1) { jj -= t; S += Hm * t; }
      else { jj += t; S -= Hm * t; }
      if (t < 1e-19) break;
    }
    return make_double2(-kInv2Pi * (jj * (log(0.5 * k) + kEuler) + S), -0.25 * jj);
  }
  double2 g = green(R, k);
  g.x += kInv2Pi * j0(x) * log(R);
  return g;
}

__global__ void k_eval_green(int n, const double* R, double k, double2* out) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = green(R[i], k);
}

// ---------------------------------------------------------------------------
// grid kernel sampling (wrap-around layout of the n x n circulant)
// ---------------------------------------------------------------------------
// g at grid offsets depends on k eps only: g = -(j/4) H0^(2)(k eps |d|)
__device__ __forceinline__ double2 green_grid(double keps, int dx, int dy) {
  const double x = keps * sqrt((double)dx * dx + (double)dy * dy);
  return make_double2(-0.25 * y0(x), -0.25 * j0(x));
}

__global__ void k_sample_kernel(int m, int n, double keps, double2* c) {
  const int qx = blockIdx.x * blockDim.x + threadIdx.x;
  const int qy = blockIdx.y;
  if (qx >= n) return;
  // offsets |d| >= m (positions m .. n - m; for n = 2m the ring |d| = m) are
  // outside the grid's Toeplitz kernel and stay zero
  const int dx = qx < m ? qx : qx - n;
  const int dy = qy < m ? qy : qy - n;
  const bool in = (qx < m || qx > n - m) && (qy < m || qy > n - m);
  double2 v = make_double2(0.0, 0.0);
  if (in && (dx != 0 || dy != 0)) v = green_grid(keps, dx, dy);
  c[(size_t)qy * n + qx] = v;
}

// spectrum rows kxq <= n/2 in the folded column-FFT frequency order, scaled
// by 1/n^2
__global__ void k_extract_spectrum(int n, const double2* C, double2* Q, float2* Qf) {
  const int hs = spec_row_len(n);
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int kx = blockIdx.y;
  if (j >= hs) return;
  const int ky = ky_of_slot(n, j);
  const double s = 1.0 / ((double)n * (double)n);
  double2 v = C[(size_t)ky * n + kx];
  v.x *= s;
  v.y *= s;
  Q[(size_t)kx * hs + j] = v;
  if (Qf) Qf[(size_t)kx * hs + j] = make_float2((float)v.x, (float)v.y);
}

// ---------------------------------------------------------------------------
// analytically filtered grid kernel, eq. (6), in grid units (t = s eps,
// kap = k eps, a = alpha eps, rho = |d|):
//   g^alpha = (1/2pi) PV int_0^a J0(t rho) t / (t^2 - kap^2) dt - (j/4) J0(kap rho)
// The principal value is taken by subtracting the pole: with
// f(t) = t J0(t rho) / (t + kap),
//   PV int_0^a f(t)/(t - kap) dt = int_0^a (f(t) - f(kap))/(t - kap) dt
//                                  + f(kap) ln((a - kap)/kap),
// integrated with 16-point Gauss-Legendre panels on [0, kap] and [kap, a],
// at least four panels per half-period of J0(t rho).  One wave per sample
// (lanes over the nodes, fixed-order reduction); samples over the octant
// 0 <= dx <= dy <= m - 1, index dy (dy + 1) / 2 + dx.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_galpha_octant(int m, double kap, double a, const double* __restrict__ glx,
                                                       const double* __restrict__ glw, double2* __restrict__ table) {
  const int lane = threadIdx.x & 63;
  const int64_t s = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t nsamp = (int64_t)m * (m + 1) / 2;
  if (s >= nsamp) return;
  // invert s = dy (dy + 1) / 2 + dx
  int dy = (int)((sqrt(8.0 * (double)s + 1.0) - 1.0) * 0.5);
  while ((int64_t)dy * (dy + 1) / 2 > s) --dy;
  while ((int64_t)(dy + 1) * (dy + 2) / 2 <= s) ++dy;
  const int dx = (int)(s - (int64_t)dy * (dy + 1) / 2);
  const double rho = sqrt((double)dx * dx + (double)dy * dy);
  const double fk = 0.5 * j0(kap * rho);   // f(kap)
  const double osc = rho > 1.0 ? rho : 1.0;
  const int n1 = max(4, (int)ceil(kap * osc * 4.0 / kPi));
  const int n2 = max(4, (int)ceil((a - kap) * osc * 4.0 / kPi));
  const double h1 = kap / n1, h2 = (a - kap) / n2;
  double acc = 0.0;
  const int nodes = (n1 + n2) * 16;
  for (int q = lane; q < nodes; q += 64) {
    const int pnl = q >> 4, node = q & 15;
    const bool first = pnl < n1;
    const double h = first ? h1 : h2;
    const double t = (first ? pnl * h1 : kap + (pnl - n1) * h2) + h * glx[node];
    const double f = t * j0(t * rho) / (t + kap);
    acc += h * glw[node] * (f - fk) / (t - kap);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) {
    const double pv = acc + fk * log((a - kap) / kap);
    table[s] = make_double2(kInv2Pi * pv, -0.25 * j0(kap * rho));
  }
}

// circulant embedding (wrap-around layout) of the octant table, ring at |d| = m zero
__global__ void k_fill_from_octant(int m, int n, const double2* __restrict__ table, double2* __restrict__ c) {
  const int qx = blockIdx.x * blockDim.x + threadIdx.x;
  const int qy = blockIdx.y;
  if (qx >= n) return;
  double2 v = make_double2(0.0, 0.0);
  if ((qx < m || qx > n - m) && (qy < m || qy > n - m)) {   // |d| <= m - 1
    int ax = qx < m ? qx : n - qx, ay = qy < m ? qy : n - qy;
    if (ax > ay) {
      const int t = ax;
      ax = ay;
      ay = t;
    }
    v = table[(int64_t)ay * (ay + 1) / 2 + ax];
  }
  c[(size_t)qy * n + qx] = v;
}

// the same grid kernel at the small offsets the near-field correction needs
__global__ void k_small_table(int ks, double keps, double2* out) {
  const int dx = threadIdx.x, dy = blockIdx.x;
  if (dx >= ks || dy >= ks) return;
  out[dy * ks + dx] = (dx == 0 && dy == 0) ? make_double2(0.0, 0.0) : green_grid(keps, dx, dy);
}

// numerical filter: keep qx^2 + qy^2 <= thr (|qx|, |qy| the folded frequencies)
__global__ void k_filter(int n, double thr, bool all, const double2* Q, double2* Qa, float2* Qaf) {
  const int hs = spec_row_len(n);
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int kx = blockIdx.y;
  if (j >= hs) return;
  const int ky = ky_of_slot(n, j);
  const int kyq = ky <= n / 2 ? ky : n - ky;
  const double r2 = (double)kx * kx + (double)kyq * kyq;
  const size_t o = (size_t)kx * hs + j;
  double2 v = Q[o];
  if (!all && !(r2 <= thr)) v = make_double2(0.0, 0.0);
  Qa[o] = v;
  if (Qaf) Qaf[o] = make_float2((float)v.x, (float)v.y);
}

// ---------------------------------------------------------------------------
// singular-quadrature moments of segment pairs (FP64)
//   M_uv = int_a int_b g(|r - r'|) tau^u sigma^v ds ds'
// ---------------------------------------------------------------------------
struct NearGeo {
  const double *vx, *vy, *h, *tx, *ty;
  int N;
  double k;
  const double* gl;   // [x16 w16 x24 w24 x32 w32]
};

// The near field is built by groups of kNG = 16 lanes, one entry per group.
// The lanes evaluate the kernel at the quadrature nodes side by side and leave
// the terms in the group's LDS; every sum is then taken by one lane, term by
// term in node order, so an entry's value does not depend on the grouping.
struct NearGroup {
  int l;        // lane within the group
  double* t;    // kNearLds doubles of LDS
};
static constexpr int kNearTerms = 7 * 32;             // terms of one quadrature row or panel
static constexpr int kMaxPsiBreaks = 128;
static constexpr int kNearLds = kNearTerms + 8 + kMaxPsiBreaks;

// sums held by the lanes 0..7 -> every lane: v[k] = lane k's acc
__device__ __forceinline__ void group_share(const NearGroup& g, double acc, double* v) {
  wave_sync();
  if (g.l < 8) g.t[kNearTerms + g.l] = acc;
  wave_sync();
  for (int k = 0; k < 8; ++k) v[k] = g.t[kNearTerms + k];
}

__device__ void moments_self(const NearGroup& g, const NearGeo& G, double h, double2 M[2][2]) {
  const double* x24 = G.gl + 32;
  const double* w24 = G.gl + 56;
  // Q_uv(delta) coefficients (ascending powers)
  const double Q00[2] = {2.0, -2.0}, Q10[2] = {1.0, -1.0};
  const double Q11[4] = {2.0 / 3.0, -1.0, 0.0, 1.0 / 3.0};
  const double lnh = log(h);
  // log part: -(1/2pi) sum_m c_m h^{2m} sum_p Q_p (ln h / e - 1/e^2), e = 2m + p + 1
  double L00 = 0, L10 = 0, L11 = 0;
  double tm = 1.0;
  const double z = 0.25 * G.k * G.k * h * h;
  for (int m = 0; m < 60; ++m) {
    double s00 = 0, s10 = 0, s11 = 0;
    for (int p = 0; p < 4; ++p) {
      const double e = 2.0 * m + p + 1.0;
      const double f = lnh / e - 1.0 / (e * e);
      if (p < 2) { s00 += Q00[p] * f; s10 += Q10[p] * f; }
      s11 += Q11[p] * f;
    }
    L00 += tm * s00;
    L10 += tm * s10;
    L11 += tm * s11;
    tm *= -z / ((m + 1.0) * (m + 1.0));
    if (fabs(tm) < 1e-20) break;
  }
  // node i: q00, q10, q11, F.x, F.y
  for (int i = g.l; i < 24; i += kNG) {
    const double d = x24[i];
    const double2 F = green_regular(h * d, G.k);
    double* t = g.t + 5 * i;
    t[0] = w24[i] * (2.0 - 2.0 * d);
    t[1] = w24[i] * (1.0 - d);
    t[2] = w24[i] * (2.0 / 3.0 - d + d * d * d / 3.0);
    t[3] = F.x;
    t[4] = F.y;
  }
  wave_sync();
  double acc = 0.0, v[8];
  if (g.l < 6)   // F00.x, F00.y, F10.x, F10.y, F11.x, F11.y
    for (int i = 0; i < 24; ++i) acc += g.t[5 * i + (g.l >> 1)] * g.t[5 * i + 3 + (g.l & 1)];
  group_share(g, acc, v);
  const double hh = h * h;
  M[0][0] = make_double2(hh * (-kInv2Pi * L00 + v[0]), hh * v[1]);
  M[1][0] = make_double2(hh * (-kInv2Pi * L10 + v[2]), hh * v[3]);
  M[0][1] = M[1][0];
  M[1][1] = make_double2(hh * (-kInv2Pi * L11 + v[4]), hh * v[5]);
}

// Breakpoints (sorted, distinct) of the polar-angle panels about a shared
// vertex, psi in [0, pi/2]: the rectangle diagonal psid = atan(h_b / h_a);
// geometric grading away from it towards the poles of the radial limits
// (h_b / sin psi at 0, used beyond psid: psid 2^j; h_a / cos psi at pi/2,
// before psid: pi/2 - (pi/2 - psid) 2^j); and at an acute vertex (cab > 0)
// pi/4 and pi/4 +- delta 2^j, where ln r(psi), r^2 = 1 - sin(2 psi) cab, has
// complex poles at distance delta = sqrt((1 - cab) / (2 cab)).
__device__ int psi_breaks(double psid, double cab, double* bp) {
  const double hp = 0.5 * kPi, q = 0.25 * kPi;
  int n = 0;
  auto add = [&](double v) {
    if (!(v > 0.0 && v < hp) || n >= kMaxPsiBreaks - 2) return;
    int i = n;
    while (i > 0 && bp[i - 1] > v) {
      bp[i] = bp[i - 1];
      --i;
    }
    if (i > 0 && bp[i - 1] == v) {   // already present: undo the shift
      for (int k = i; k < n; ++k) bp[k] = bp[k + 1];
      return;
    }
    bp[i] = v;
    ++n;
  };
  add(psid);
  for (int j = 1; j < 48 && psid * exp2((double)j) < hp; ++j) add(psid * exp2((double)j));
  for (int j = 1; j < 48 && hp - (hp - psid) * exp2((double)j) > 0.0; ++j) add(hp - (hp - psid) * exp2((double)j));
  if (cab > 0.0) {
    const double delta = fmax(sqrt(fmax(1.0 - cab, 0.0) / (2.0 * cab)), 1e-12);
    add(q);
    for (int j = 0; j < 48 && delta * exp2((double)j) < q; ++j) {
      add(q - delta * exp2((double)j));
      add(q + delta * exp2((double)j));
    }
  }
  // ends
  for (int k = n; k > 0; --k) bp[k] = bp[k - 1];
  bp[0] = 0.0;
  bp[n + 1] = hp;
  return n + 2;
}

// segments a and b share a vertex; a_first: a ends where b starts
__device__ void moments_adjacent(const NearGroup& g, const NearGeo& G, int a, int b, bool a_first, double2 M[2][2]) {
  const int N = G.N;
  const int a1 = (a + 1) % N, b1 = (b + 1) % N;
  double Vx, Vy, Pax, Pay, Pbx, Pby, t0, t1, s0, s1;
  const double ha = G.h[a], hb = G.h[b];
  if (a_first) {   // V = end of a = start of b
    Vx = G.vx[a1]; Vy = G.vy[a1];
    Pax = G.vx[a]; Pay = G.vy[a];
    Pbx = G.vx[b1]; Pby = G.vy[b1];
    t0 = 1.0; t1 = -1.0 / ha;      // tau = 1 - s/ha
    s0 = 0.0; s1 = 1.0 / hb;       // sigma = s'/hb
  } else {         // V = start of a = end of b
    Vx = G.vx[a]; Vy = G.vy[a];
    Pax = G.vx[a1]; Pay = G.vy[a1];
    Pbx = G.vx[b]; Pby = G.vy[b];
    t0 = 0.0; t1 = 1.0 / ha;
    s0 = 1.0; s1 = -1.0 / hb;
  }
  const double eax = (Pax - Vx) / ha, eay = (Pay - Vy) / ha;
  const double ebx = (Pbx - Vx) / hb, eby = (Pby - Vy) / hb;
  const double cab = eax * ebx + eay * eby;
  const double k = G.k;
  // polar log part: B_ij = int int J0(kR) ln R s^i s'^j ds ds', psi over
  // the graded panels of psi_breaks
  const double* x32 = G.gl + 80;
  const double* w32 = G.gl + 112;
  const double psid = atan2(hb, ha);
  double* bp = g.t + kNearTerms + 8;
  int nbp = 0;
  if (g.l == 0) nbp = psi_breaks(psid, cab, bp);
  nbp = __shfl(nbp, 0, kNG);
  wave_sync();
  double accB = 0.0;   // lanes 0..3: B_00, B_10, B_01, B_11
  for (int pnl = 0; pnl + 1 < nbp; ++pnl) {
    const double lo = bp[pnl], hi = bp[pnl + 1];
    const bool upper = lo >= psid;   // radial limit h_b / sin(psi) beyond the diagonal
    const double len = hi - lo;
    for (int q = g.l; q < 32; q += kNG) {
      const double ps = lo + len * x32[q];
      const double wps = len * w32[q];
      double sp, cp;
      sincos(ps, &sp, &cp);
      const double r2 = 1.0 - 2.0 * cp * sp * cab;
      const double lnr = 0.5 * log(r2);
      const double P = upper ? hb / sp : ha / cp;
      const double lnP = log(P);
      const double zz = 0.25 * k * k * r2 * P * P;
      // sum over m for total degree d = i + j in {0,1,2}
      double Sd[3] = {0, 0, 0};
      for (int d = 0; d < 3; ++d) {
        double tm = 1.0;
        double Pe = pow(P, (double)(d + 2));   // P^{e} with e = d + 2 at m = 0
        double acc = 0.0;
        for (int m = 0; m < 60; ++m) {
          const double e = 2.0 * m + d + 2.0;
          acc += tm * Pe * ((lnP + lnr) / e - 1.0 / (e * e));
          tm *= -zz / ((m + 1.0) * (m + 1.0));
          if (fabs(tm) < 1e-20) break;
        }
        Sd[d] = acc;   // tm carries (k P r / 2)^{2m}/(m!)^2, Pe the rest
      }
      double* t = g.t + 7 * q;
      t[0] = wps;
      t[1] = wps * cp;
      t[2] = wps * sp;
      t[3] = wps * cp * sp;
      t[4] = Sd[0];
      t[5] = Sd[1];
      t[6] = Sd[2];
    }
    wave_sync();
    if (g.l < 4) {
      const int d = 4 + (g.l == 0 ? 0 : (g.l == 3 ? 2 : 1));
      for (int q = 0; q < 32; ++q) accB += g.t[7 * q + g.l] * g.t[7 * q + d];
    }
    wave_sync();
  }
  double v[8];
  group_share(g, accB, v);
  const double B[2][2] = {{v[0], v[2]}, {v[1], v[3]}};
  // smooth part by 16 x 16 Gauss-Legendre in (s, s')
  const double* x16 = G.gl;
  const double* w16 = G.gl + 16;
  double accF = 0.0;   // lanes 0..7: F_00, F_10, F_01, F_11, re and im
  for (int i = 0; i < 16; ++i) {
    const double S = x16[i] * ha;
    const double tau = t0 + t1 * S;
    wave_sync();
    {
      const int j = g.l;
      const double Sp = x16[j] * hb;
      const double sig = s0 + s1 * Sp;
      // S^2 + S'^2 - 2 S S' cos(angle), rounded in this order
      const double R = sqrt(fmax(fma(-(2.0 * S * Sp), cab, fma(Sp, Sp, S * S)), 0.0));
      const double2 f = green_regular(R, k);
      const double w = w16[i] * w16[j] * ha * hb;
      double* t = g.t + 6 * j;
      t[0] = w;
      t[1] = w * tau;
      t[2] = w * sig;
      t[3] = w * tau * sig;
      t[4] = f.x;
      t[5] = f.y;
    }
    wave_sync();
    if (g.l < 8)
      for (int j = 0; j < 16; ++j) accF += g.t[6 * j + (g.l >> 1)] * g.t[6 * j + 4 + (g.l & 1)];
  }
  group_share(g, accF, v);
  const double2 F[2][2] = {{make_double2(v[0], v[1]), make_double2(v[4], v[5])},
                           {make_double2(v[2], v[3]), make_double2(v[6], v[7])}};
  // tau^u sigma^v in powers of (s, s'): alpha^u_i, beta^v_j
  for (int u = 0; u < 2; ++u)
    for (int v = 0; v < 2; ++v) {
      const double al[2] = {u ? t0 : 1.0, u ? t1 : 0.0};
      const double be[2] = {v ? s0 : 1.0, v ? s1 : 0.0};
      double Lsum = 0.0;
      for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) Lsum += al[i] * be[j] * B[i][j];
      M[u][v] = make_double2(-kInv2Pi * Lsum + F[u][v].x, F[u][v].y);
    }
}

// distance between two segments that do not cross: the smallest of the
// four endpoint-to-segment distances
__device__ double pt_seg_dist(double px, double py, double ax, double ay, double bx, double by) {
  const double dx = bx - ax, dy = by - ay;
  const double L2 = dx * dx + dy * dy;
  const double t = L2 > 0.0 ? fmin(1.0, fmax(0.0, ((px - ax) * dx + (py - ay) * dy) / L2)) : 0.0;
  const double ex = px - (ax + t * dx), ey = py - (ay + t * dy);
  return sqrt(ex * ex + ey * ey);
}
__device__ double seg_seg_dist(double p0x, double p0y, double p1x, double p1y, double q0x, double q0y, double q1x,
                               double q1y) {
  return fmin(fmin(pt_seg_dist(p0x, p0y, q0x, q0y, q1x, q1y), pt_seg_dist(p1x, p1y, q0x, q0y, q1x, q1y)),
              fmin(pt_seg_dist(q0x, q0y, p0x, p0y, p1x, p1y), pt_seg_dist(q1x, q1y, p0x, p0y, p1x, p1y)));
}

// Disjoint segments: 16 x 16 Gauss-Legendre over parameter boxes
// [t0, t1] x [s0, s1] of the unit square.  A box whose two pieces lie closer
// than half the longer piece is split by halving the longer piece (depth at
// most 40), so next to a short segment the nearly singular kernel is still
// resolved; distant pairs are one box.
__device__ void moments_disjoint(const NearGroup& g, const NearGeo& G, int a, int b, double2 M[2][2]) {
  const int N = G.N;
  const int a1 = (a + 1) % N, b1 = (b + 1) % N;
  const double ax = G.vx[a], ay = G.vy[a], adx = G.vx[a1] - ax, ady = G.vy[a1] - ay;
  const double bx = G.vx[b], by = G.vy[b], bdx = G.vx[b1] - bx, bdy = G.vy[b1] - by;
  const double ha = G.h[a], hb = G.h[b];
  const double* x16 = G.gl;
  const double* w16 = G.gl + 16;
  double acc = 0.0;   // lanes 0..7: M_00, M_01, M_10, M_11, re and im
  constexpr int kStack = 48;
  double st[kStack][4];
  int dep[kStack];
  int top = 0;
  st[0][0] = 0.0; st[0][1] = 1.0; st[0][2] = 0.0; st[0][3] = 1.0;
  dep[0] = 0;
  top = 1;
  while (top > 0) {
    --top;
    const double t0 = st[top][0], t1 = st[top][1], s0 = st[top][2], s1 = st[top][3];
    const int d = dep[top];
    const double la = ha * (t1 - t0), lb = hb * (s1 - s0);
    const double dist = seg_seg_dist(ax + adx * t0, ay + ady * t0, ax + adx * t1, ay + ady * t1, bx + bdx * s0,
                                     by + bdy * s0, bx + bdx * s1, by + bdy * s1);
    if (!(dist >= 0.5 * fmax(la, lb) || d >= 40 || top + 2 > kStack)) {
      // split the longer piece; the first half is taken next
      const bool sa = la >= lb;
      const double m = sa ? 0.5 * (t0 + t1) : 0.5 * (s0 + s1);
      st[top][0] = sa ? m : t0; st[top][1] = t1; st[top][2] = sa ? s0 : m; st[top][3] = s1;
      dep[top] = d + 1;
      st[top + 1][0] = t0; st[top + 1][1] = sa ? m : t1; st[top + 1][2] = s0; st[top + 1][3] = sa ? s1 : m;
      dep[top + 1] = d + 1;
      top += 2;
      continue;
    }
    const double wt = t1 - t0, ws = s1 - s0;
    wave_sync();
    {
      const int i = g.l;
      const double ti = t0 + wt * x16[i];
      const double px = ax + adx * ti, py = ay + ady * ti;
      double2 r0 = make_double2(0, 0), r1 = make_double2(0, 0);
      for (int j = 0; j < 16; ++j) {
        const double sj = s0 + ws * x16[j];
        const double dx = px - (bx + bdx * sj), dy = py - (by + bdy * sj);
        const double2 gr = green(sqrt(dx * dx + dy * dy), G.k);
        const double w = ws * w16[j];
        r0.x += w * gr.x; r0.y += w * gr.y;
        r1.x += w * sj * gr.x; r1.y += w * sj * gr.y;
      }
      const double wi = wt * w16[i];
      double* t = g.t + 6 * i;
      t[0] = wi;
      t[1] = wi * ti;
      t[2] = r0.x;
      t[3] = r0.y;
      t[4] = r1.x;
      t[5] = r1.y;
    }
    wave_sync();
    if (g.l < 8)
      for (int i = 0; i < 16; ++i) acc += g.t[6 * i + (g.l >> 2)] * g.t[6 * i + 2 + (g.l & 3)];
  }
  double v[8];
  group_share(g, acc, v);
  const double s = ha * hb;
  for (int u = 0; u < 2; ++u)
    for (int w = 0; w < 2; ++w) M[u][w] = make_double2(s * v[4 * u + 2 * w], s * v[4 * u + 2 * w + 1]);
}

__device__ void segment_moments(const NearGroup& g, const NearGeo& G, int a, int b, double2 M[2][2]) {
  const int N = G.N;
  if (a == b) moments_self(g, G, G.h[a], M);
  else if ((a + 1) % N == b) moments_adjacent(g, G, a, b, true, M);
  else if ((b + 1) % N == a) moments_adjacent(g, G, a, b, false, M);
  else moments_disjoint(g, G, a, b, M);
}

// grid approximation (Lambda_i^T G_grid Lambda_j) of one channel pair
__device__ double2 grid_pair(const NearGroup& g, const double* Wi, const double* Wj, int dax, int day,
                             const double2* ks, int KS) {
  const int e = g.l, se = e & 3, te = e >> 2;
  double2 inner = make_double2(0, 0);
  for (int f = 0; f < 16; ++f) {
    const int sf = f & 3, tf = f >> 2;
    const int dx = abs(dax + se - sf), dy = abs(day + te - tf);
    const double2 kv = ks[dy * KS + dx];
    inner.x += Wj[f] * kv.x;
    inner.y += Wj[f] * kv.y;
  }
  wave_sync();
  g.t[2 * e] = inner.x;
  g.t[2 * e + 1] = inner.y;
  wave_sync();
  double acc = 0.0, v[8];
  if (g.l < 2)
    for (int q = 0; q < 16; ++q) acc += Wi[q] * g.t[2 * q + g.l];
  group_share(g, acc, v);
  return make_double2(v[0], v[1]);
}

// One entry per 16-lane group.  A thread per entry left the few entries of
// vertex-sharing segments (two per row, a serial chain of 256 + 64 series
// evaluations) as the kernel's length, with most of the chip idle: 5.4 ms for
// the entries of 3 328 pulses (1.0 ms here), 3.2 ms for 512 (0.42), 18.8 ms for
// 16 384 (5.6), 80 ms for 20 001 hats (28.8).  Bound by FP64 issue in the
// Bessel functions.  Held to two waves per SIMD, which spills 122 of its
// VGPRs (scratch 2.2 KB a lane, 1.7 of it the box stack of disjoint pairs);
// without spills one wave per SIMD fits: 1.6 ms; three or four waves spill
// more: 1.0 to 1.2 ms.
__global__ __launch_bounds__(kNearBlock, 2) void k_near_build(
    NearGeo G, int basis, int64_t nnz, const int32_t* __restrict__ rows, const int32_t* __restrict__ cols,
    const int32_t* __restrict__ anx, const int32_t* __restrict__ any, const double* W0, const double* W1,
    const double* W2, const double* W3, const double2* __restrict__ ks, int KS, double2* CS, double2* CN) {
  __shared__ double lds[kNearBlock / kNG][kNearLds];
  const int64_t q = (int64_t)blockIdx.x * (kNearBlock / kNG) + threadIdx.x / kNG;
  if (q >= nnz) return;   // whole groups exit together
  const NearGroup g{(int)(threadIdx.x % kNG), lds[threadIdx.x / kNG]};
  const int i = rows[q], j = cols[q];
  const int N = G.N;
  const int dax = anx[i] - anx[j], day = any[i] - any[j];
  double2 M[2][2];
  if (basis == AIM_PULSE) {
    segment_moments(g, G, i, j, M);
    const double2 gp = grid_pair(g, W0 + (size_t)i * 16, W0 + (size_t)j * 16, dax, day, ks, KS);
    if (g.l == 0) CS[q] = make_double2(M[0][0].x - gp.x, M[0][0].y - gp.y);
    return;
  }
  // hats: pieces (segment, c0, c1): rising on i-1, falling on i
  const int sa[2] = {(i - 1 + N) % N, i}, sb[2] = {(j - 1 + N) % N, j};
  const double c0[2] = {0.0, 1.0}, c1[2] = {1.0, -1.0};
  double2 S = make_double2(0, 0), Nn = make_double2(0, 0);
  const double k2 = G.k * G.k;
  for (int pa = 0; pa < 2; ++pa)
    for (int pb = 0; pb < 2; ++pb) {
      const int a = sa[pa], b = sb[pb];
      segment_moments(g, G, a, b, M);
      // phi_i phi_j moment: sum_uv p_u q_v M_uv with p = (c0, c1)
      const double pu[2] = {c0[pa], c1[pa]}, qv[2] = {c0[pb], c1[pb]};
      double2 pp = make_double2(0, 0);
      for (int u = 0; u < 2; ++u)
        for (int v = 0; v < 2; ++v) {
          pp.x += pu[u] * qv[v] * M[u][v].x;
          pp.y += pu[u] * qv[v] * M[u][v].y;
        }
      S.x += pp.x;
      S.y += pp.y;
      const double da = c1[pa] / G.h[a], db = c1[pb] / G.h[b];
      const double tt = G.tx[a] * G.tx[b] + G.ty[a] * G.ty[b];
      Nn.x += da * db * M[0][0].x - k2 * tt * pp.x;
      Nn.y += da * db * M[0][0].y - k2 * tt * pp.y;
    }
  const size_t oi = (size_t)i * 16, oj = (size_t)j * 16;
  const double2 gS = grid_pair(g, W0 + oi, W0 + oj, dax, day, ks, KS);
  const double2 gq = grid_pair(g, W1 + oi, W1 + oj, dax, day, ks, KS);
  const double2 gx = grid_pair(g, W2 + oi, W2 + oj, dax, day, ks, KS);
  const double2 gy = grid_pair(g, W3 + oi, W3 + oj, dax, day, ks, KS);
  if (g.l != 0) return;
  CS[q] = make_double2(S.x - gS.x, S.y - gS.y);
  CN[q] = make_double2(Nn.x - (gq.x - k2 * (gx.x + gy.x)), Nn.y - (gq.y - k2 * (gx.y + gy.y)));
}

// ---------------------------------------------------------------------------
// anterpolation: U[ch*nrhs + r][a] = sum_e w_ch[e] x[r*ldx + basis_e]
// ---------------------------------------------------------------------------
// right-hand sides per k_anterp block in batches of four or more
constexpr int kAnterpRhs = 4;

template <typename T, typename TW, int ARB>
__global__ __launch_bounds__(256) void k_anterp(int n_act, int nrhs, const int32_t* __restrict__ at_ptr,
                                                const int32_t* __restrict__ at_basis, const TW* __restrict__ w0,
                                                const TW* __restrict__ w1, const TW* __restrict__ w2,
                                                const double2* __restrict__ x, int64_t ldx,
                                                cplx<T>* __restrict__ U) {
  // 16 lanes per active grid point, shuffle reduction; blockIdx.y picks a
  // channel and a run of up to ARB right-hand sides, which share the entry
  // loads (basis index, weight) and keep their own sums
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int a = gid >> 4, l = gid & 15;
  const int nrb = (nrhs + ARB - 1) / ARB;
  const int ch = blockIdx.y / nrb, r0 = (blockIdx.y - ch * nrb) * ARB;
  if (a >= n_act) return;                   // whole 16-lane groups exit together
  const int nr = ARB == 1 ? 1 : min(ARB, nrhs - r0);
  const TW* w = ch == 0 ? w0 : (ch == 1 ? w1 : w2);
  const double2* xr = x + (size_t)r0 * ldx;
  T sx[ARB], sy[ARB];
#pragma unroll
  for (int k = 0; k < ARB; ++k) sx[k] = sy[k] = 0;
  const int e1 = at_ptr[a + 1];
  int e = at_ptr[a] + l;
  for (; e + 16 < e1; e += 32) {   // two entries per lane in flight
    const int b0 = at_basis[e], b1 = at_basis[e + 16];
    const T w0e = (T)w[e], w1e = (T)w[e + 16];
#pragma unroll
    for (int k = 0; k < ARB; ++k) {
      if (k < nr) {
        const double2 x0 = xr[(size_t)k * ldx + b0], x1 = xr[(size_t)k * ldx + b1];
        sx[k] += w0e * (T)x0.x;
        sy[k] += w0e * (T)x0.y;
        sx[k] += w1e * (T)x1.x;
        sy[k] += w1e * (T)x1.y;
      }
    }
  }
  if (e < e1) {
    const int b0 = at_basis[e];
    const T ww = (T)w[e];
#pragma unroll
    for (int k = 0; k < ARB; ++k) {
      if (k < nr) {
        const double2 xv = xr[(size_t)k * ldx + b0];
        sx[k] += ww * (T)xv.x;
        sy[k] += ww * (T)xv.y;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < ARB; ++k) {
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
      sx[k] += __shfl_xor(sx[k], off, 16);
      sy[k] += __shfl_xor(sy[k], off, 16);
    }
    if (l == 0 && k < nr) U[(size_t)(ch * nrhs + r0 + k) * n_act + a] = mk<T>(sx[k], sy[k]);
  }
}

// ---------------------------------------------------------------------------
// interpolation + near field: LANES lanes per basis row, S map points per row
// (16 for the 4 x 4 stencils: lanes 0..15 hold one point each for all rhs;
// wider per-node rows are strided over the lanes)
//   y = scale * ( sum_ch sgn_ch W_ch . V_ch + C_near x )
// ---------------------------------------------------------------------------
template <typename T, typename TW, int LANES>
__global__ __launch_bounds__(256) void k_interp_near(
    int N, int nrhs, int rpb, int nch, int S, const TW* __restrict__ W0, const TW* __restrict__ W1,
    const TW* __restrict__ W2, double sg, const int32_t* __restrict__ aidx,
    const cplx<T>* __restrict__ V, int n_act, const int32_t* __restrict__ nptr,
    const int32_t* __restrict__ ncol, const double2* __restrict__ C, const double2* __restrict__ x,
    int64_t ldx, double2* __restrict__ y, int64_t ldy, double2 scale) {
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int row = gid / LANES, l = gid % LANES;
  if (row >= N) return;          // whole lane groups exit together
  const bool st = l < S;         // lanes below S hold map points
  const size_t o = (size_t)row * S + (st ? l : 0);
  const int a = st ? aidx[o] : 0;
  const double w0 = st ? (double)W0[o] : 0.0;
  const double w1 = (st && nch > 1) ? (double)W1[o] : 0.0;
  const double w2 = (st && nch > 1) ? (double)W2[o] : 0.0;
  const int q0 = C ? nptr[row] : 0, q1 = C ? nptr[row + 1] : 0;
  const int r0 = blockIdx.y * rpb, r1 = min(nrhs, r0 + rpb);   // this block's right-hand sides
  for (int r = r0; r < r1; ++r) {
    double ax = 0.0, ay = 0.0;
    if (st) {
      const cplx<T> v0 = V[(size_t)r * n_act + a];
      ax = w0 * (double)v0.x;
      ay = w0 * (double)v0.y;
      if (nch > 1) {
        const cplx<T> v1 = V[(size_t)(nrhs + r) * n_act + a];
        const cplx<T> v2 = V[(size_t)(2 * nrhs + r) * n_act + a];
        ax += sg * (w1 * (double)v1.x + w2 * (double)v2.x);
        ay += sg * (w1 * (double)v1.y + w2 * (double)v2.y);
      }
    }
    for (int e = l + LANES; e < S; e += LANES) {   // map points beyond the first LANES
      const size_t oe = (size_t)row * S + e;
      const int ae = aidx[oe];
      const cplx<T> v0 = V[(size_t)r * n_act + ae];
      ax += (double)W0[oe] * (double)v0.x;
      ay += (double)W0[oe] * (double)v0.y;
      if (nch > 1) {
        const cplx<T> v1 = V[(size_t)(nrhs + r) * n_act + ae];
        const cplx<T> v2 = V[(size_t)(2 * nrhs + r) * n_act + ae];
        ax += sg * ((double)W1[oe] * (double)v1.x + (double)W2[oe] * (double)v2.x);
        ay += sg * ((double)W1[oe] * (double)v1.y + (double)W2[oe] * (double)v2.y);
      }
    }
    const double2* xr = x + (size_t)r * ldx;
    int q = q0 + l;
    for (; q + LANES < q1; q += 2 * LANES) {   // two entries per lane in flight
      const int k0 = ncol[q], k1 = ncol[q + LANES];
      const double2 c0 = C[q], c1 = C[q + LANES];
      const double2 x0 = xr[k0], x1 = xr[k1];
      ax += c0.x * x0.x - c0.y * x0.y;
      ay += c0.x * x0.y + c0.y * x0.x;
      ax += c1.x * x1.x - c1.y * x1.y;
      ay += c1.x * x1.y + c1.y * x1.x;
    }
    if (q < q1) {
      const double2 cv = C[q];
      const double2 xv = xr[ncol[q]];
      ax += cv.x * xv.x - cv.y * xv.y;
      ay += cv.x * xv.y + cv.y * xv.x;
    }
#pragma unroll
    for (int off = LANES / 2; off >= 1; off >>= 1) {
      ax += __shfl_xor(ax, off, LANES);
      ay += __shfl_xor(ay, off, LANES);
    }
    if (l == 0) y[(size_t)r * ldy + row] = make_double2(scale.x * ax - scale.y * ay, scale.x * ay + scale.y * ax);
  }
}

// ---------------------------------------------------------------------------
// banded symmetric near field: Cd[d][i] = C(i, (i + d) mod N) for d <= w
// ---------------------------------------------------------------------------
__global__ void k_near_to_band(int64_t nnz, int N, int w, const int32_t* __restrict__ rows,
                               const int32_t* __restrict__ cols, const double2* __restrict__ C,
                               double2* __restrict__ Cd) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= nnz) return;
  const int i = rows[q];
  int d = cols[q] - i;
  if (d < 0) d += N;
  if (d <= w) Cd[(size_t)d * N + i] = C[q];
}

// band widths below this take the several-rhs form of the band product
constexpr int kBandFastW = 64;
// A batch's right-hand sides are split over blocks while the launch has fewer
// than this many (six per CU): a block takes its share one after the other.
// Whole products, unsplit / split in us: 24 right-hand sides, N = 1024 (64
// blocks) 58.7 / 42.7, N = 3000 110 / 65, N = 6000 153 / 118; 8 right-hand
// sides, N = 1024 31.3 / 26.1.  From a thousand blocks on the shared band
// values are worth more (N = 16 000, two right-hand sides 85.0 / 86.9).
constexpr int kInterpBlocks = 1536;
struct RhsSplit {
  int per, blocks;   // right-hand sides per block, blocks along y
  RhsSplit(int nrhs, unsigned gx) {
    const int ny = std::max(1, std::min(nrhs, kInterpBlocks / (int)gx));
    per = (nrhs + ny - 1) / ny;
    blocks = (nrhs + per - 1) / per;
  }
};

// interpolation + banded near field, 16 lanes per basis row:
//   y_i = scale * ( sum_ch sgn_ch W_ch . V_ch + sum_{d<=w} Cd[d][i] x_{i+d}
//                   + sum_{1<=d<=w} Cd[d][i-d] x_{i-d} )   (indices mod N)
template <typename T, typename TW, bool FAST>
__global__ __launch_bounds__(256) void k_interp_band(
    int N, int nrhs, int rpb, int nch, const TW* __restrict__ W0, const TW* __restrict__ W1, const TW* __restrict__ W2,
    double sg, const int32_t* __restrict__ aidx, const cplx<T>* __restrict__ V, int n_act, int w,
    const double2* __restrict__ Cd, const double2* __restrict__ x, int64_t ldx, double2* __restrict__ y,
    int64_t ldy, double2 scale) {
  constexpr int L = 16;
  // XCD-aware block order: blocks are dealt round-robin over the 8 XCDs, so
  // logical block (bid mod 8) * per + bid / 8 gives each XCD a contiguous
  // range of rows.  Row i reads the band at columns i (upper half) and
  // i - d (lower half, d <= w): the lower reads then hit in the XCD's L2
  // the values its neighbouring blocks just fetched as upper reads, instead
  // of fetching each band value a second time.
  const int per = (int)((gridDim.x + 7) / 8);
  const int lblk = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  const int gid = lblk * blockDim.x + threadIdx.x;
  const int row = gid / L, l = gid % L;
  if (row >= N) return;          // whole lane groups exit together
  const size_t o = (size_t)row * 16 + l;
  const int a = aidx[o];
  const double w0 = (double)W0[o];
  const double w1 = nch > 1 ? (double)W1[o] : 0.0;
  const double w2 = nch > 1 ? (double)W2[o] : 0.0;
  // FAST (several rhs, a band up to KU * L - 1 wide): the lane's band values
  // (the same for every rhs) are loaded once, ahead of everything else, and
  // each rhs issues all its x loads before its first sum; the terms are
  // added in the order of the general loop below.  The held values take
  // registers (a third of the occupancy), which one rhs of a long contour
  // does not repay.
  constexpr int KU = kBandFastW / L;
  double2 cu[KU], cl[KU];
  int ju[KU], il[KU];
  if constexpr (FAST) {
#pragma unroll
    for (int k = 0; k < KU; ++k) {
      const int d = l + k * L, dl = d + 1;
      ju[k] = row + d >= N ? row + d - N : row + d;
      il[k] = row - dl < 0 ? row - dl + N : row - dl;
      cu[k] = d <= w ? Cd[(size_t)d * N + row] : make_double2(0.0, 0.0);
      cl[k] = dl <= w ? Cd[(size_t)dl * N + il[k]] : make_double2(0.0, 0.0);
    }
  }
  const int r0 = blockIdx.y * rpb, r1 = min(nrhs, r0 + rpb);   // this block's right-hand sides
  for (int r = r0; r < r1; ++r) {
    const double2* xr = x + (size_t)r * ldx;
    double2 xu[KU], xl[KU];
    if constexpr (FAST) {
#pragma unroll
      for (int k = 0; k < KU; ++k) {
        const int d = l + k * L;
        xu[k] = d <= w ? xr[ju[k]] : make_double2(0.0, 0.0);
        xl[k] = d + 1 <= w ? xr[il[k]] : make_double2(0.0, 0.0);
      }
    }
    const cplx<T> v0 = V[(size_t)r * n_act + a];
    double ax = w0 * (double)v0.x, ay = w0 * (double)v0.y;
    if (nch > 1) {
      const cplx<T> v1 = V[(size_t)(nrhs + r) * n_act + a];
      const cplx<T> v2 = V[(size_t)(2 * nrhs + r) * n_act + a];
      ax += sg * (w1 * (double)v1.x + w2 * (double)v2.x);
      ay += sg * (w1 * (double)v1.y + w2 * (double)v2.y);
    }
    if constexpr (FAST) {
#pragma unroll
      for (int k = 0; k < KU; ++k) {
        const int d = l + k * L;
        if (d > w) break;
        ax += cu[k].x * xu[k].x - cu[k].y * xu[k].y;
        ay += cu[k].x * xu[k].y + cu[k].y * xu[k].x;
        if (d + 1 <= w) {
          ax += cl[k].x * xl[k].x - cl[k].y * xl[k].y;
          ay += cl[k].x * xl[k].y + cl[k].y * xl[k].x;
        }
      }
    } else if (Cd) {
      for (int d = l; d <= w; d += L) {
        int ju = row + d;
        if (ju >= N) ju -= N;
        const double2 cu = Cd[(size_t)d * N + row], xu = xr[ju];
        ax += cu.x * xu.x - cu.y * xu.y;
        ay += cu.x * xu.y + cu.y * xu.x;
        const int dl = d + 1;                      // lower half: C(i - dl, i), dl = 1..w
        if (dl <= w) {
          int il = row - dl;
          if (il < 0) il += N;
          const double2 cl = Cd[(size_t)dl * N + il], xl = xr[il];
          ax += cl.x * xl.x - cl.y * xl.y;
          ay += cl.x * xl.y + cl.y * xl.x;
        }
      }
    }
#pragma unroll
    for (int off = L / 2; off >= 1; off >>= 1) {
      ax += __shfl_xor(ax, off, L);
      ay += __shfl_xor(ay, off, L);
    }
    if (l == 0) y[(size_t)r * ldy + row] = make_double2(scale.x * ax - scale.y * ay, scale.x * ay + scale.y * ax);
  }
}

// ---------------------------------------------------------------------------
// Gram solve
// ---------------------------------------------------------------------------
__global__ void k_gram_pulse(int N, int nrhs, const double* h, const double2* x, int64_t ldx, double2* y,
                             int64_t ldy) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  if (i >= N) return;
  const double2 v = x[(size_t)r * ldx + i];
  y[(size_t)r * ldy + i] = make_double2(v.x / h[i], v.y / h[i]);
}

// Hats, N >= GB + 2 GH: block of GB outputs from a truncated tridiagonal system
// extended by GH unknowns on each side.  The inverse of this Gram matrix
// decays at least like 0.268^|i-j| (condition number <= 3), so the
// truncation error is below 1e-18 relative.
constexpr int GB = 64, GH = 32, GM = GB + 2 * GH;

__global__ void k_gram_hat_blocks(int N, int nrhs, const double* h, const double2* x, int64_t ldx,
                                  double2* y, int64_t ldy) {
  const int blk = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  const int nblk = (N + GB - 1) / GB;
  if (blk >= nblk) return;
  const int i0 = blk * GB - GH;    // first unknown of the local system (cyclic)
  double cp[GM];
  double2 dp[GM];
  const double2* xr = x + (size_t)r * ldx;
  // Thomas: a_i y_{i-1} + d_i y_i + c_i y_{i+1} = b_i, local indices 0..GM-1
  double prev_c = 0.0;
  double2 prev_d = make_double2(0, 0);
  for (int l = 0; l < GM; ++l) {
    const int gi = ((i0 + l) % N + N) % N;
    const int gm = (gi - 1 + N) % N;
    const double d = (h[gm] + h[gi]) / 3.0;
    const double a = (l > 0) ? h[gm] / 6.0 : 0.0;
    const double c = (l < GM - 1) ? h[gi] / 6.0 : 0.0;
    const double den = d - a * prev_c;
    const double2 b = xr[gi];
    cp[l] = c / den;
    dp[l] = make_double2((b.x - a * prev_d.x) / den, (b.y - a * prev_d.y) / den);
    prev_c = cp[l];
    prev_d = dp[l];
  }
  double2 nxt = dp[GM - 1];
  double2* yr = y + (size_t)r * ldy;
  for (int l = GM - 1; l >= 0; --l) {
    double2 v = dp[l];
    if (l < GM - 1) { v.x -= cp[l] * nxt.x; v.y -= cp[l] * nxt.y; }
    nxt = v;
    if (l >= GH && l < GH + GB) {
      const int gi = i0 + l;
      if (gi < N) yr[gi] = v;
    }
  }
}

// Hats, N >= GP: parallel cyclic reduction of a truncated system in LDS.
// Block b solves the GP unknowns starting GH before its GP - 2 GH outputs
// (cyclic indices), with no coupling past the window's ends; by the same
// 0.268^d decay the outputs, GH or more unknowns from either end, carry a
// truncation error below 1e-18 relative.  Step s (s = 1, 2, .., GP/2)
// eliminates the couplings at distance s from every equation; after log2 GP
// steps each equation holds a single unknown.
constexpr int GP = 256, GPO = GP - 2 * GH;

__global__ __launch_bounds__(GP) void k_gram_hat_pcr(int N, const double* __restrict__ h,
                                                     const double2* __restrict__ x, int64_t ldx,
                                                     double2* __restrict__ y, int64_t ldy) {
  __shared__ double sa[GP], sb[GP], sc[GP], sdx[GP], sdy[GP];
  const int t = threadIdx.x, r = blockIdx.y;
  int gi = (int)((blockIdx.x * (int64_t)GPO - GH + t) % N);
  if (gi < 0) gi += N;
  const int gm = gi == 0 ? N - 1 : gi - 1;
  const double2 xv = x[(size_t)r * ldx + gi];
  // row gi of G: h_{i-1}/6, (h_{i-1} + h_i)/3, h_i/6; cut at the window's ends
  double a = t > 0 ? h[gm] / 6.0 : 0.0;
  double b = (h[gm] + h[gi]) / 3.0;
  double c = t < GP - 1 ? h[gi] / 6.0 : 0.0;
  double dx = xv.x, dy = xv.y;
#pragma unroll
  for (int st = 1; st < GP; st <<= 1) {
    sa[t] = a; sb[t] = b; sc[t] = c; sdx[t] = dx; sdy[t] = dy;
    __syncthreads();
    double na = 0.0, nc = 0.0, nb = b, ndx = dx, ndy = dy;
    if (t - st >= 0) {
      const double al = -a / sb[t - st];
      na = al * sa[t - st];
      nb += al * sc[t - st];
      ndx += al * sdx[t - st];
      ndy += al * sdy[t - st];
    }
    if (t + st < GP) {
      const double ga = -c / sb[t + st];
      nc = ga * sc[t + st];
      nb += ga * sa[t + st];
      ndx += ga * sdx[t + st];
      ndy += ga * sdy[t + st];
    }
    __syncthreads();
    a = na; b = nb; c = nc; dx = ndx; dy = ndy;
  }
  const int o = (int)(blockIdx.x * (int64_t)GPO) + t - GH;   // output index (not wrapped)
  if (t >= GH && t < GP - GH && o < N) y[(size_t)r * ldy + o] = make_double2(dx / b, dy / b);
}

// Hats, small N: cyclic Thomas with Sherman-Morrison, one thread per column.
// scratch: 3N doubles per column.
__global__ void k_gram_hat_small(int N, int nrhs, const double* h, const double2* x, int64_t ldx,
                                 double2* y, int64_t ldy, double* scratch) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nrhs) return;
  double* cp = scratch + (size_t)r * 5 * N;
  double* dy_re = cp + N;
  double* dy_im = dy_re + N;
  double* zz = dy_im + N;
  double* dd = zz + N;
  const double2* xr = x + (size_t)r * ldx;
  double2* yr = y + (size_t)r * ldy;
  // G = T + u v^T: gam = -d_0, corner e = h_{N-1}/6
  const double d0 = (h[N - 1] + h[0]) / 3.0;
  const double gam = -d0;
  const double ec = h[N - 1] / 6.0;
  for (int i = 0; i < N; ++i) {
    double d = (h[(i - 1 + N) % N] + h[i]) / 3.0;
    if (i == 0) d -= gam;
    if (i == N - 1) d -= ec * ec / gam;
    dd[i] = d;
  }
  // forward sweep for two right-hand sides (b and u)
  double pc = 0, pyr = 0, pyi = 0, pz = 0;
  for (int i = 0; i < N; ++i) {
    const double a = (i > 0) ? h[i - 1] / 6.0 : 0.0;
    const double c = (i < N - 1) ? h[i] / 6.0 : 0.0;
    const double den = dd[i] - a * pc;
    const double u = (i == 0) ? gam : (i == N - 1 ? ec : 0.0);
    cp[i] = c / den;
    dy_re[i] = (xr[i].x - a * pyr) / den;
    dy_im[i] = (xr[i].y - a * pyi) / den;
    zz[i] = (u - a * pz) / den;
    pc = cp[i]; pyr = dy_re[i]; pyi = dy_im[i]; pz = zz[i];
  }
  for (int i = N - 2; i >= 0; --i) {
    dy_re[i] -= cp[i] * dy_re[i + 1];
    dy_im[i] -= cp[i] * dy_im[i + 1];
    zz[i] -= cp[i] * zz[i + 1];
  }
  // v = (1, 0, .., 0, ec/gam)
  const double vz = zz[0] + ec / gam * zz[N - 1];
  const double vyr = dy_re[0] + ec / gam * dy_re[N - 1];
  const double vyi = dy_im[0] + ec / gam * dy_im[N - 1];
  const double fr = vyr / (1.0 + vz), fi = vyi / (1.0 + vz);
  for (int i = 0; i < N; ++i) yr[i] = make_double2(dy_re[i] - zz[i] * fr, dy_im[i] - zz[i] * fi);
}

// ---------------------------------------------------------------------------
// plane-wave right-hand sides; rcs reduction
// ---------------------------------------------------------------------------
__global__ void k_rhs(int N, int nrhs, int basis, int p, const double* gx, const double* gw, const double* vx,
                      const double* vy, const double* h, const double* tx, const double* ty,
                      const double* phi, double k, double eta, double amp, double2* b) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  if (i >= N) return;
  double cph, sph;
  sincos(phi[r], &sph, &cph);
  double accx = 0, accy = 0;
  const int npc = basis == AIM_PULSE ? 1 : 2;
  for (int pc = 0; pc < npc; ++pc) {
    int s;
    double c0, c1;
    if (basis == AIM_PULSE) { s = i; c0 = 1; c1 = 0; }
    else if (pc == 0) { s = (i - 1 + N) % N; c0 = 0; c1 = 1; }
    else { s = i; c0 = 1; c1 = -1; }
    const int s1 = (s + 1) % N;
    const double ax = vx[s], ay = vy[s], dx = vx[s1] - ax, dy = vy[s1] - ay;
    // TE: (jk/eta) * eta * amp * t.(z x khat) = jk amp (t.(-khat_y, khat_x))
    const double tdot = basis == AIM_PULSE ? 1.0 : (-tx[s] * sph + ty[s] * cph);
    for (int q = 0; q < p; ++q) {
      const double tau = gx[q];
      const double px = ax + dx * tau, py = ay + dy * tau;
      const double wk = h[s] * gw[q] * (c0 + c1 * tau) * tdot;
      double sn, cs;
      sincos(-k * (px * cph + py * sph), &sn, &cs);
      accx += wk * cs;
      accy += wk * sn;
    }
  }
  double2 out;
  if (basis == AIM_PULSE) out = make_double2(amp * accx, amp * accy);
  else out = make_double2(-k * amp * accy, k * amp * accx);   // multiply by j k amp
  b[(size_t)r * N + i] = out;
}

// partial dot products sum_i b_i J_i per column (no conjugate)
__global__ void k_dotu_cols(int N, const double2* a, const double2* b, double* out) {
  const int r = blockIdx.x;
  __shared__ double sx[256], sy[256];
  double ax = 0, ay = 0;
  for (int i = threadIdx.x; i < N; i += 256) {
    const double2 u = a[(size_t)r * N + i], v = b[(size_t)r * N + i];
    ax += u.x * v.x - u.y * v.y;
    ay += u.x * v.y + u.y * v.x;
  }
  sx[threadIdx.x] = ax;
  sy[threadIdx.x] = ay;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) { sx[threadIdx.x] += sx[threadIdx.x + s]; sy[threadIdx.x] += sy[threadIdx.x + s]; }
    __syncthreads();
  }
  if (threadIdx.x == 0) { out[2 * r] = sx[0]; out[2 * r + 1] = sy[0]; }
}

// row of each entry of a CSR pattern, a wave per row
__global__ __launch_bounds__(256) void k_entry_rows(int N, const int32_t* __restrict__ ptr, int32_t* __restrict__ rows) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= N) return;
  for (int q = ptr[i] + (threadIdx.x & 63); q < ptr[i + 1]; q += 64) rows[q] = i;
}

// ===========================================================================
// host side
// ===========================================================================
aim_status dev_alloc(Ctx* c, void** p, size_t bytes) {
  *p = nullptr;
  if (bytes == 0) return AIM_OK;
  if (hipMalloc(p, bytes) != hipSuccess) { *p = nullptr; return AIM_E_OOM; }
  c->allocs.push_back(*p);
  c->dev_bytes += bytes;
  return AIM_OK;
}

// Host tables on their way to the device: gathered in one host array, they
// take one allocation and one copy (each small copy or allocation costs some
// 20 us whatever its size, and set-up had 26 of each).  Tables start at
// multiples of 256 bytes.
struct Upload {
  std::vector<char> host;
  std::vector<std::pair<void**, size_t>> at;   // pointer to set, offset
  template <typename V> void add(V** dst, const void* src, size_t bytes) {
    *dst = nullptr;
    if (bytes == 0) return;
    at.push_back({(void**)dst, host.size()});
    host.insert(host.end(), (const char*)src, (const char*)src + bytes);
    host.resize((host.size() + 255) & ~(size_t)255);
  }
  template <typename V, typename F> void add(V** dst, const std::vector<F>& v) {
    if constexpr (std::is_same<V, F>::value) {
      add(dst, v.data(), v.size() * sizeof(V));
    } else {
      const std::vector<V> w(v.begin(), v.end());
      add(dst, w.data(), w.size() * sizeof(V));
    }
  }
  // copies the tables to `base` and sets their pointers
  aim_status send(void* base) {
    if (hipMemcpy(base, host.data(), host.size(), hipMemcpyHostToDevice) != hipSuccess) return AIM_E_HIP;
    for (auto& a : at) *a.first = (char*)base + a.second;
    return AIM_OK;
  }
  aim_status send(Ctx* c) {
    void* base = nullptr;
    const aim_status st = dev_alloc(c, &base, host.size());
    return st != AIM_OK || !base ? st : send(base);
  }
};

#define TRY(x)                         \
  do {                                 \
    aim_status s_ = (x);               \
    if (s_ != AIM_OK) return s_;       \
  } while (0)

// ---------------------------------------------------------------------------
// process-wide cache of grid-kernel spectra, keyed by (device, m, k eps, FP32
// copy).  The samples depend on k eps only, so a cached spectrum is the one
// a fresh context would compute.  Entries without users stay resident until
// aim_cache_clear or until the cache exceeds kSpecCacheBytes.
// ---------------------------------------------------------------------------
struct SpecEntry {
  int device = 0, m = 0;
  double keps = 0;
  bool f32 = false;
  double2* C = nullptr;
  float2* Cf = nullptr;
  int refs = 0;
  size_t bytes = 0;
  uint64_t last_use = 0;
};
static std::mutex g_spec_mu;
static std::vector<SpecEntry*> g_spec;
static uint64_t g_spec_clock = 0;
static constexpr size_t kSpecCacheBytes = (size_t)8 << 30;

static void spec_free(SpecEntry* e) {
  if (e->C) (void)hipFree(e->C);
  if (e->Cf) (void)hipFree(e->Cf);
  delete e;
}

static void spec_evict_locked(size_t budget) {
  size_t tot = 0;
  for (SpecEntry* e : g_spec) tot += e->bytes;
  while (tot > budget) {
    SpecEntry* victim = nullptr;
    for (SpecEntry* e : g_spec)
      if (e->refs == 0 && (!victim || e->last_use < victim->last_use)) victim = e;
    if (!victim) break;
    tot -= victim->bytes;
    g_spec.erase(std::find(g_spec.begin(), g_spec.end(), victim));
    spec_free(victim);
  }
}

aim_status acquire_spectrum(Ctx* c, double keps) {
  const int m = c->t.m, n = c->t.n, H = n / 2 + 1;
  const bool f32 = c->precision == AIM_MIXED;
  std::lock_guard<std::mutex> lk(g_spec_mu);
  for (SpecEntry* e : g_spec)
    if (e->device == c->device && e->m == m && e->keps == keps && (e->f32 || !f32)) {
      e->refs++;
      e->last_use = ++g_spec_clock;
      c->spec = e;
      c->d_C = e->C;
      c->d_Cf = e->Cf;
      return AIM_OK;
    }
  SpecEntry* e = new SpecEntry();
  e->device = c->device;
  e->m = m;
  e->keps = keps;
  e->f32 = f32;
  e->bytes = (size_t)H * spec_row_len(n) * (sizeof(double2) + (f32 ? sizeof(float2) : 0));
  spec_evict_locked(kSpecCacheBytes > e->bytes ? kSpecCacheBytes - e->bytes : 0);
  hipStream_t s = c->stream;
  double2* cfull = nullptr;
  bool ok = hipMalloc(&cfull, (size_t)n * n * sizeof(double2)) == hipSuccess;
  ok = ok && hipMalloc(&e->C, (size_t)H * spec_row_len(n) * sizeof(double2)) == hipSuccess;
  if (ok && f32) ok = hipMalloc(&e->Cf, (size_t)H * spec_row_len(n) * sizeof(float2)) == hipSuccess;
  if (!ok) {
    if (cfull) (void)hipFree(cfull);
    spec_free(e);
    return AIM_E_OOM;
  }
  hipLaunchKernelGGL(k_sample_kernel, dim3((n + 255) / 256, n), dim3(256), 0, s, m, n, keps, cfull);
  aim_status st = launch_rows_fft_inplace(n, cfull, c->d_tw, s);
  if (st == AIM_OK) st = launch_cols<double>(n, 1, cfull, n, n, n / 2, 1, nullptr, c->d_tw, s);
  if (st == AIM_OK) {
    hipLaunchKernelGGL(k_extract_spectrum, dim3((spec_row_len(n) + 255) / 256, H), dim3(256), 0, s, n, cfull, e->C, e->Cf);
    if (hipStreamSynchronize(s) != hipSuccess) st = AIM_E_HIP;
  }
  (void)hipFree(cfull);
  if (st != AIM_OK) {
    spec_free(e);
    return st;
  }
  e->refs = 1;
  e->last_use = ++g_spec_clock;
  g_spec.push_back(e);
  c->spec = e;
  c->d_C = e->C;
  c->d_Cf = e->Cf;
  return AIM_OK;
}

void release_spectrum(Ctx* c) {
  if (!c->spec) return;
  std::lock_guard<std::mutex> lk(g_spec_mu);
  ((SpecEntry*)c->spec)->refs--;
  c->spec = nullptr;
  c->d_C = nullptr;
  c->d_Cf = nullptr;
}

size_t cache_idle_bytes() {
  std::lock_guard<std::mutex> lk(g_spec_mu);
  size_t idle = 0;
  for (SpecEntry* e : g_spec)
    if (e->refs == 0) idle += e->bytes;
  return idle;
}

size_t cache_clear() {
  std::lock_guard<std::mutex> lk(g_spec_mu);
  size_t freed = 0;
  for (auto it = g_spec.begin(); it != g_spec.end();) {
    if ((*it)->refs == 0) {
      freed += (*it)->bytes;
      spec_free(*it);
      it = g_spec.erase(it);
    } else {
      ++it;
    }
  }
  return freed;
}

// ---------------------------------------------------------------------------
// Allocation-free RCS: the angles, plane-wave vectors, column sums and values
// of one call live in a fixed device array, one per GPU for the life of the
// process.  Host code never passes `scratch` itself to a kernel (it is only a
// host-side stand-in there): its device address is resolved once per device
// at set-up with that device current and kept in g_scratch_dev.
// ---------------------------------------------------------------------------
static __device__ __align__(256) double2 scratch[kNoAllocScratch];
static constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static double2* g_scratch_dev[kMaxDevices] = {};

// Called by setup_device with c->device current.
static aim_status resolve_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return AIM_E_HIP;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_dev[device]) return AIM_OK;
  void* p = nullptr;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return AIM_E_HIP;
  g_scratch_dev[device] = (double2*)p;
  return AIM_OK;
}

aim_status setup_device(Ctx* c) {
  HostTables& t = c->t;
  const int N = t.N, n = t.n;
  hipStream_t s = c->stream;
  TRY(resolve_scratch(c->device));
  // What the near-field build reads goes first; the rest of the tables are
  // gathered and the buffers allocated while it runs (set-up, right-hand sides
  // and one product of a 3 328-pulse star: 2.9 -> 2.4 ms).
  {
    Upload up;
    up.add(&c->d_vx, t.vx);
    up.add(&c->d_vy, t.vy);
    up.add(&c->d_h, t.h);
    up.add(&c->d_tx, t.tx);
    up.add(&c->d_ty, t.ty);
    up.add(&c->d_glx, t.gl_x);
    up.add(&c->d_glw, t.gl_w);
    for (int ch = 0; ch < t.nch; ++ch) up.add(&c->d_W[ch], t.W[ch]);
    up.add(&c->d_nr_ptr, t.nr_ptr);
    up.add(&c->d_nr_col, t.nr_col);
    TRY(up.send(c));
  }

  // grid kernel at small offsets (near-field correction)
  const double keps = t.k * t.eps;
  c->ks = t.R + 4;
  TRY(dev_alloc(c, (void**)&c->d_ksmall, (size_t)c->ks * c->ks * sizeof(double2)));
  hipLaunchKernelGGL(k_small_table, dim3(c->ks), dim3(64 * ((c->ks + 63) / 64)), 0, s, c->ks, keps, c->d_ksmall);

  // near field
  const int64_t nnz = (int64_t)t.nr_col.size();
  c->nnz = nnz;
  TRY(dev_alloc(c, (void**)&c->d_CS, nnz * sizeof(double2)));
  if (t.basis == AIM_HAT) TRY(dev_alloc(c, (void**)&c->d_CN, nnz * sizeof(double2)));
  // temporaries of the build (anchors, quadrature table, row of each entry);
  // the kernels read them: freed on every path after a wait
  struct Temp {
    hipStream_t s;
    void* p = nullptr;
    hipError_t release() {
      if (!p) return hipSuccess;
      const hipError_t e = hipStreamSynchronize(s);
      (void)hipFree(p);
      p = nullptr;
      return e;
    }
    ~Temp() { (void)release(); }
  } tmp{s};
  {
    int32_t *d_anx = nullptr, *d_any = nullptr;
    double* d_gl = nullptr;
    Upload up;
    up.add(&d_anx, t.anc_x);
    up.add(&d_any, t.anc_y);
    std::vector<double> gl;
    for (int pq : {16, 24, 32}) {
      std::vector<double> x, w;
      gauss_legendre01(pq, x, w);
      gl.insert(gl.end(), x.begin(), x.end());
      gl.insert(gl.end(), w.begin(), w.end());
    }
    up.add(&d_gl, gl);
    if (hipMalloc(&tmp.p, up.host.size() + nnz * 4) != hipSuccess) {
      tmp.p = nullptr;
      return AIM_E_OOM;
    }
    int32_t* d_rows = (int32_t*)((char*)tmp.p + up.host.size());
    TRY(up.send(tmp.p));
    if (nnz > 0) {
      NearGeo G{c->d_vx, c->d_vy, c->d_h, c->d_tx, c->d_ty, N, t.k, d_gl};
      hipLaunchKernelGGL(k_entry_rows, dim3((N + 3) / 4), dim3(256), 0, s, N, c->d_nr_ptr, d_rows);
      for (int64_t q0 = 0; q0 < nnz; q0 += kNearLaunch) {
        hipLaunchKernelGGL(k_near_build, dim3(near_blocks(q0, nnz)), dim3(kNearBlock), 0, s, G, t.basis,
                           std::min(nnz - q0, kNearLaunch), d_rows + q0, c->d_nr_col + q0, d_anx, d_any, c->d_W[0],
                           c->d_W[1], c->d_W[2], c->d_W[3], c->d_ksmall, c->ks, c->d_CS + q0,
                           c->d_CN ? c->d_CN + q0 : nullptr);
        AIM_HIP_CHECK(hipGetLastError());
      }
    }
    if (t.band_w >= 0 && nnz > 0) {
      const size_t bb = (size_t)(t.band_w + 1) * N * sizeof(double2);
      TRY(dev_alloc(c, (void**)&c->d_CSd, bb));
      if (t.basis == AIM_HAT) TRY(dev_alloc(c, (void**)&c->d_CNd, bb));
      AIM_HIP_CHECK(hipMemsetAsync(c->d_CSd, 0, bb, s));
      hipLaunchKernelGGL(k_near_to_band, dim3((unsigned)((nnz + 255) / 256)), dim3(256), 0, s, nnz, N, t.band_w,
                         d_rows, c->d_nr_col, c->d_CS, c->d_CSd);
      AIM_HIP_CHECK(hipGetLastError());
      if (t.basis == AIM_HAT) {
        AIM_HIP_CHECK(hipMemsetAsync(c->d_CNd, 0, bb, s));
        hipLaunchKernelGGL(k_near_to_band, dim3((unsigned)((nnz + 255) / 256)), dim3(256), 0, s, nnz, N, t.band_w,
                           d_rows, c->d_nr_col, c->d_CN, c->d_CNd);
        AIM_HIP_CHECK(hipGetLastError());
      }
    }
  }

  // matvec work buffers
  c->nch_max = (t.basis == AIM_HAT) ? 3 : 1;
  const size_t pairs = (size_t)c->nch_max * c->max_rhs;
  const size_t be = 16;   // FP64 complex (FP32 uses the first half)
  TRY(dev_alloc(c, &c->d_U, pairs * t.n_act * be));
  TRY(dev_alloc(c, &c->d_V, pairs * t.n_act * be));
  TRY(dev_alloc(c, &c->d_T, pairs * (size_t)tile_rows(t.nr) * n * be));
  TRY(dev_alloc(c, (void**)&c->d_tmp1, (size_t)N * c->max_rhs * 16));
  TRY(dev_alloc(c, (void**)&c->d_tmp2, (size_t)N * c->max_rhs * 16));
  TRY(dev_alloc(c, (void**)&c->d_rhs, (size_t)N * c->max_rhs * 16));
  TRY(dev_alloc(c, (void**)&c->d_phi, (size_t)AIM_MAX_RHS * 8));
  TRY(dev_alloc(c, (void**)&c->d_dot, (size_t)c->max_rhs * 24));   // sums, then the values
  // coherent pinned memory: the Givens kernel writes the estimates into it
  if (hipHostMalloc((void**)&c->h_resid, (size_t)c->max_rhs * kResidPitch * 8, hipHostMallocCoherent) != hipSuccess) {
    c->h_resid = nullptr;
    return AIM_E_OOM;
  }
  AIM_HIP_CHECK(hipHostGetDevicePointer((void**)&c->d_resid_map, c->h_resid, 0));
  AIM_HIP_CHECK(hipEventCreateWithFlags(&c->ev_resid, hipEventDisableTiming));
  TRY(dev_alloc(c, (void**)&c->d_red, (size_t)std::max(5 * N, 64) * std::max(c->max_rhs, 1) * 8));

  // the other tables
  {
    Upload up;
    for (int ch = 0; ch < t.nch; ++ch) {
      up.add(&c->d_at_w[ch], t.at_w[ch]);
      if (c->precision == AIM_MIXED) {
        up.add(&c->d_Wf[ch], t.W[ch]);
        up.add(&c->d_at_wf[ch], t.at_w[ch]);
      }
    }
    up.add(&c->d_aidx, t.aidx);
    up.add(&c->d_act_ix, t.act_ix);
    up.add(&c->d_row_ptr, t.row_ptr);
    up.add(&c->d_at_ptr, t.at_ptr);
    up.add(&c->d_at_basis, t.at_basis);
    std::vector<double> tw;
    twiddles(n, tw);
    up.add((double**)&c->d_tw, tw);
    if (c->precision == AIM_MIXED) up.add((float**)&c->d_twf, tw);
    TRY(up.send(c));
  }
  AIM_HIP_CHECK(tmp.release());
  // spectrum F(c_grid): shared through the process-wide cache
  TRY(acquire_spectrum(c, keps));
  TRY(apply_filter(c, INFINITY));
  AIM_HIP_CHECK(hipStreamSynchronize(s));
  return AIM_OK;
}

aim_status apply_filter(Ctx* c, double alpha) {
  const int n = c->t.n, H = n / 2 + 1;
  const bool all = !std::isfinite(alpha);
  int kcut = n / 2;
  if (all) {   // no truncation: the filtered operator uses the shared spectrum
    c->d_Ca = c->d_C;
    c->d_Caf = c->d_Cf;
  } else {
    if (!c->own_Ca) {
      TRY(dev_alloc(c, (void**)&c->own_Ca, (size_t)H * spec_row_len(n) * sizeof(double2)));
      if (c->precision == AIM_MIXED) TRY(dev_alloc(c, (void**)&c->own_Caf, (size_t)H * spec_row_len(n) * sizeof(float2)));
    }
    const double thr = ((alpha * n) * c->t.eps / (2.0 * kPi)) * ((alpha * n) * c->t.eps / (2.0 * kPi));
    // the largest |kx| the mask keeps (at ky = 0)
    while (kcut > 0 && !((double)kcut * kcut <= thr)) --kcut;
    hipLaunchKernelGGL(k_filter, dim3((spec_row_len(n) + 255) / 256, H), dim3(256), 0, c->stream, n, thr, false, c->d_C,
                       c->own_Ca, c->own_Caf);
    AIM_HIP_CHECK(hipGetLastError());
    c->d_Ca = c->own_Ca;
    c->d_Caf = c->own_Caf;
  }
  c->kcut = kcut;
  c->alpha = alpha;
  c->filtered = !all;
  return AIM_OK;
}

aim_status apply_filter_analytic(Ctx* c, double alpha) {
  const HostTables& t = c->t;
  const int m = t.m, n = t.n, H = n / 2 + 1;
  const double kap = t.k * t.eps, a = alpha * t.eps;
  if (!(alpha > t.k) || !std::isfinite(alpha)) return AIM_E_ARG;
  hipStream_t s = c->stream;
  if (!c->own_Ca) {
    TRY(dev_alloc(c, (void**)&c->own_Ca, (size_t)H * spec_row_len(n) * sizeof(double2)));
    if (c->precision == AIM_MIXED) TRY(dev_alloc(c, (void**)&c->own_Caf, (size_t)H * spec_row_len(n) * sizeof(float2)));
  }
  std::vector<double> gx, gw;
  gauss_legendre01(16, gx, gw);
  const int64_t nsamp = (int64_t)m * (m + 1) / 2;
  double2 *table = nullptr, *cfull = nullptr;
  double* gl = nullptr;
  bool ok = hipMalloc(&table, nsamp * sizeof(double2)) == hipSuccess;
  ok = ok && hipMalloc(&cfull, (size_t)n * n * sizeof(double2)) == hipSuccess;
  ok = ok && hipMalloc(&gl, 32 * sizeof(double)) == hipSuccess;
  aim_status st = ok ? AIM_OK : AIM_E_OOM;
  if (st == AIM_OK && (hipMemcpyAsync(gl, gx.data(), 16 * 8, hipMemcpyHostToDevice, s) != hipSuccess ||
                       hipMemcpyAsync(gl + 16, gw.data(), 16 * 8, hipMemcpyHostToDevice, s) != hipSuccess))
    st = AIM_E_HIP;
  if (st == AIM_OK) {
    hipLaunchKernelGGL(k_galpha_octant, dim3((unsigned)((nsamp + 3) / 4)), dim3(256), 0, s, m, kap, a, gl, gl + 16,
                       table);
    hipLaunchKernelGGL(k_fill_from_octant, dim3((n + 255) / 256, n), dim3(256), 0, s, m, n, table, cfull);
    st = hipGetLastError() == hipSuccess ? AIM_OK : AIM_E_HIP;
  }
  if (st == AIM_OK) st = launch_rows_fft_inplace(n, cfull, c->d_tw, s);
  if (st == AIM_OK) st = launch_cols<double>(n, 1, cfull, n, n, n / 2, 1, nullptr, c->d_tw, s);
  if (st == AIM_OK) {
    hipLaunchKernelGGL(k_extract_spectrum, dim3((spec_row_len(n) + 255) / 256, H), dim3(256), 0, s, n, cfull, c->own_Ca,
                       c->own_Caf);
    if (hipStreamSynchronize(s) != hipSuccess) st = AIM_E_HIP;
  }
  if (table) (void)hipFree(table);
  if (cfull) (void)hipFree(cfull);
  if (gl) (void)hipFree(gl);
  if (st != AIM_OK) return st;
  c->d_Ca = c->own_Ca;
  c->d_Caf = c->own_Caf;
  c->kcut = n / 2;
  c->alpha = alpha;
  c->filtered = true;
  return AIM_OK;
}

// grid part: V = [F^-1 (Chat . F(Lambda x))]_restr for nch channels, in
// three steps: anterpolation and forward row FFTs (grid_pre), the column
// pass (launch_cols, or one grouped launch for several contexts), inverse
// row FFTs (grid_post)
template <typename T>
static const cplx<T>* grid_spectrum(Ctx* c, bool filt) {
  const bool f32 = sizeof(T) == 4;
  return f32 ? (const cplx<T>*)(filt ? (void*)c->d_Caf : (void*)c->d_Cf)
             : (const cplx<T>*)(filt ? (void*)c->d_Ca : (void*)c->d_C);
}
template <typename T>
static const cplx<T>* grid_twiddles(Ctx* c) {
  return sizeof(T) == 4 ? (const cplx<T>*)c->d_twf : (const cplx<T>*)c->d_tw;
}

// the grid spectrum of a product is zero past this |kx|
static int grid_kcut(const Ctx* c, bool filt) { return filt ? c->kcut : c->t.n / 2; }

template <typename T>
static aim_status grid_pre(Ctx* c, const int* chans, int nch, bool filt, int nrhs, const double2* x, int64_t ldx) {
  HostTables& t = c->t;
  hipStream_t s = c->stream;
  const int pairs = nch * nrhs;
  cplx<T>* U = (cplx<T>*)c->d_U;
  cplx<T>* Tb = (cplx<T>*)c->d_T;
  const bool f32 = sizeof(T) == 4;
  const int kcut = grid_kcut(c, filt);
  const bool timed = ProfScope::due(c, AIM_K_ANTERP) || ProfScope::due(c, AIM_K_ROWS_FWD);
  if (anterp_in_rows(t.n, f32, t.nr, pairs, timed) && !rows_few_columns(t.n, f32, kcut, t.n_act, t.nr)) {
    AtMap at;
    at.ptr = c->d_at_ptr;
    at.basis = c->d_at_basis;
    for (int q = 0; q < nch; ++q) at.w[q] = f32 ? (const void*)c->d_at_wf[chans[q]] : (const void*)c->d_at_w[chans[q]];
    ProfScope pa(c, AIM_K_ANTERP), pr(c, AIM_K_ROWS_FWD);   // counted, not timed
    return launch_rows_fwd_at<T>(t.n, at, x, ldx, nrhs, c->d_row_ptr, c->d_act_ix, t.nr, tile_rows(t.nr), kcut,
                                    pairs, Tb, grid_twiddles<T>(c), s);
  }
  // a single rhs keeps one sum per lane; batches share the entry loads
  const int arb = nrhs >= kAnterpRhs ? kAnterpRhs : 1;
  dim3 ga((unsigned)(((size_t)t.n_act * 16 + 255) / 256), nch * ((nrhs + arb - 1) / arb));
  {
  ProfScope ps(c, AIM_K_ANTERP);
#define AIM_ANTERP(TW, WS)                                                                                          \
  if (arb == 1)                                                                                                     \
    hipLaunchKernelGGL((k_anterp<T, TW, 1>), ga, dim3(256), 0, s, t.n_act, nrhs, c->d_at_ptr, c->d_at_basis,       \
                       WS[chans[0]], WS[chans[nch > 1 ? 1 : 0]], WS[chans[nch > 2 ? 2 : 0]], x, ldx, U);             \
  else                                                                                                              \
    hipLaunchKernelGGL((k_anterp<T, TW, kAnterpRhs>), ga, dim3(256), 0, s, t.n_act, nrhs, c->d_at_ptr,             \
                       c->d_at_basis, WS[chans[0]], WS[chans[nch > 1 ? 1 : 0]], WS[chans[nch > 2 ? 2 : 0]], x, ldx, U);
  if (f32) {
    AIM_ANTERP(float, c->d_at_wf)
  } else {
    AIM_ANTERP(double, c->d_at_w)
  }
#undef AIM_ANTERP
  }
  AIM_HIP_CHECK(hipGetLastError());
  ProfScope ps(c, AIM_K_ROWS_FWD);
  return launch_rows_fwd<T>(t.n, U, t.n_act, c->d_row_ptr, c->d_act_ix, t.nr, tile_rows(t.nr), kcut,
                            pairs, Tb, grid_twiddles<T>(c), s);
}

template <typename T>
static aim_status grid_post(Ctx* c, int nch, bool filt, int nrhs) {
  HostTables& t = c->t;
  ProfScope ps(c, AIM_K_ROWS_INV);
  return launch_rows_inv<T>(t.n, (cplx<T>*)c->d_T, t.nr, tile_rows(t.nr), grid_kcut(c, filt), c->d_row_ptr, c->d_act_ix,
                            nch * nrhs, (cplx<T>*)c->d_V, t.n_act, grid_twiddles<T>(c), c->stream);
}

template <typename T>
static aim_status grid_apply(Ctx* c, const int* chans, int nch, bool filt, int nrhs, const double2* x,
                             int64_t ldx) {
  HostTables& t = c->t;
  TRY(grid_pre<T>(c, chans, nch, filt, nrhs, x, ldx));
  {
    // the dominant kernel's sampled launches carry their events in the
    // dispatch itself, so the interval is the kernel's own execution
    ProfScope ps(c, AIM_K_COLS, true);
    TRY(launch_cols<T>(t.n, 0, (cplx<T>*)c->d_T, t.nr, tile_rows(t.nr), grid_kcut(c, filt), nch * nrhs,
                       grid_spectrum<T>(c, filt), grid_twiddles<T>(c), c->stream, ps.start(), ps.stop()));
  }
  return grid_post<T>(c, nch, filt, nrhs);
}

template <typename T, int LANES>
static void launch_interp(Ctx* c, const int* chans, int nch, double sg, const double2* C, int nrhs,
                          const double2* x, int64_t ldx, double2* y, int64_t ldy, double2 scale) {
  HostTables& t = c->t;
  const int threads = 256;
  const unsigned gx = (unsigned)(((size_t)t.N * LANES + threads - 1) / threads);
  const RhsSplit rs(nrhs, gx);
  const dim3 g(gx, rs.blocks);
  const cplx<T>* V = (const cplx<T>*)c->d_V;
  if (sizeof(T) == 4) {
    hipLaunchKernelGGL((k_interp_near<T, float, LANES>), g, dim3(threads), 0, c->stream, t.N, nrhs, rs.per, nch, t.S,
                       c->d_Wf[chans[0]], c->d_Wf[chans[nch > 1 ? 1 : 0]], c->d_Wf[chans[nch > 2 ? 2 : 0]], sg,
                       c->d_aidx, V, t.n_act, c->d_nr_ptr, c->d_nr_col, C, x, ldx, y, ldy, scale);
  } else {
    hipLaunchKernelGGL((k_interp_near<T, double, LANES>), g, dim3(threads), 0, c->stream, t.N, nrhs, rs.per, nch, t.S,
                       c->d_W[chans[0]], c->d_W[chans[nch > 1 ? 1 : 0]], c->d_W[chans[nch > 2 ? 2 : 0]], sg,
                       c->d_aidx, V, t.n_act, c->d_nr_ptr, c->d_nr_col, C, x, ldx, y, ldy, scale);
  }
}

template <typename T>
static aim_status interp(Ctx* c, const int* chans, int nch, double sg, bool near, const double2* Cn, int nrhs,
                         const double2* x, int64_t ldx, double2* y, int64_t ldy, double2 scale) {
  const double2* C = near ? Cn : nullptr;
  ProfScope ps(c, AIM_K_INTERP);
  const HostTables& t = c->t;
  if (t.band_w >= 0) {
    // banded symmetric near field (or none)
    const double2* Cd = !near ? nullptr : (Cn == c->d_CS ? c->d_CSd : c->d_CNd);
    // a multiple of 8 blocks (the kernel's XCD-aware order); the extra ones exit
    const size_t nb = ((size_t)t.N * 16 + 255) / 256;
    const unsigned gx = (unsigned)(8 * ((nb + 7) / 8));
    const RhsSplit rs(nrhs, gx);
    const dim3 g(gx, rs.blocks);
    // one right-hand side repays the held band values while the launch is on
    // the chip at once (N = 512 20.5 -> 19.9 us, N = 16 384 55.5 -> 54.7 us)
    const bool fast = Cd && t.band_w < kBandFastW && (nrhs > 1 || gx <= 1024);
#define AIM_BAND(TW, WT, F)                                                                                   \
  hipLaunchKernelGGL((k_interp_band<T, TW, F>), g, dim3(256), 0, c->stream, t.N, nrhs, rs.per, nch, WT[chans[0]], \
                     WT[chans[nch > 1 ? 1 : 0]], WT[chans[nch > 2 ? 2 : 0]], sg, c->d_aidx, (const cplx<T>*)c->d_V, \
                     t.n_act, t.band_w, Cd, x, ldx, y, ldy, scale)
    if (sizeof(T) == 4) {
      if (fast) AIM_BAND(float, c->d_Wf, true);
      else AIM_BAND(float, c->d_Wf, false);
    } else {
      if (fast) AIM_BAND(double, c->d_W, true);
      else AIM_BAND(double, c->d_W, false);
    }
#undef AIM_BAND
    AIM_HIP_CHECK(hipGetLastError());
    return AIM_OK;
  }
  // wide lane groups when the near-field rows are long
  const bool wide = (near && c->nnz >= (int64_t)40 * c->t.N) || t.S > 16;
  if (wide) launch_interp<T, 64>(c, chans, nch, sg, C, nrhs, x, ldx, y, ldy, scale);
  else launch_interp<T, 16>(c, chans, nch, sg, C, nrhs, x, ldx, y, ldy, scale);
  AIM_HIP_CHECK(hipGetLastError());
  return AIM_OK;
}

template <typename T>
static aim_status op_grid(Ctx* c, int base_op, int nrhs, const double2* x, int64_t ldx, double2* y, int64_t ldy,
                          double2 scale) {
  static const int chS[1] = {0};
  static const int chN[3] = {1, 2, 3};
  const double k2 = c->t.k * c->t.k;
  switch (base_op) {
    case AIM_OP_S:
      TRY(grid_apply<T>(c, chS, 1, false, nrhs, x, ldx));
      return interp<T>(c, chS, 1, 0.0, true, c->d_CS, nrhs, x, ldx, y, ldy, scale);
    case AIM_OP_S_ALPHA:
      TRY(grid_apply<T>(c, chS, 1, true, nrhs, x, ldx));
      return interp<T>(c, chS, 1, 0.0, false, nullptr, nrhs, x, ldx, y, ldy, scale);
    case AIM_OP_N:
      TRY(grid_apply<T>(c, chN, 3, false, nrhs, x, ldx));
      return interp<T>(c, chN, 3, -k2, true, c->d_CN, nrhs, x, ldx, y, ldy, scale);
    case AIM_OP_N_ALPHA:
      TRY(grid_apply<T>(c, chN, 3, true, nrhs, x, ldx));
      return interp<T>(c, chN, 3, -k2, false, nullptr, nrhs, x, ldx, y, ldy, scale);
  }
  return AIM_E_ARG;
}

// ---------------------------------------------------------------------------
// dual pairing of the TM Calderon operators.  G_pd = diag(h) T with T the
// circulant (1/8, 3/4, 1/8); T^-1 is the circulant
//   tau_d = sqrt(2) (rho^d + rho^(N-d)) / (1 - rho^N),  rho = 2 sqrt(2) - 3,
// (the two geometric solutions of the three-term recurrence, matched at the
// wrap) whose terms fall below 1e-18 of tau_0 past |d| = 24, so it is
// applied as a (2D+1)-term cyclic convolution (all N terms when N <= 2D+1).
// Dual hats in refined hats: psi_j = h'_2j / 2 + h'_2j+1 + h'_2j+2 / 2.
// ---------------------------------------------------------------------------
static constexpr int kTauD = 24;

aim_status setup_dual(Ctx* c) {
  const int N = c->t.N;
  const bool full = N <= 2 * kTauD + 1;
  const int nt = full ? N : kTauD + 1;
  std::vector<double> tau(nt), ih(N);
  const long double rho = 2.0L * std::sqrt(2.0L) - 3.0L;
  const long double rN = std::pow(rho, (long double)N);
  for (int d = 0; d < nt; ++d)
    tau[d] = (double)(std::sqrt(2.0L) * (std::pow(rho, (long double)d) + std::pow(rho, (long double)(N - d))) /
                      (1.0L - rN));
  for (int i = 0; i < N; ++i) ih[i] = 1.0 / c->t.h[i];
  c->tau_D = full ? -1 : kTauD;   // -1: one-sided sum over all N offsets
  Upload up;
  up.add(&c->d_tau, tau.data(), nt * 8);
  up.add(&c->d_ih, ih);
  TRY(up.send(c));
  AIM_HIP_CHECK(hipStreamSynchronize(c->stream));
  return AIM_OK;
}

// (T^-1 diag(s) z)_i for column z (length N), s = 1 when sc is null:
// D >= 0 the two-sided band of kTauD terms each side, D < 0 all N offsets
__device__ __forceinline__ double2 tinv_at(int N, int D, const double* __restrict__ tau, int i,
                                           const double2* __restrict__ z, const double* __restrict__ sc) {
  double ax = 0.0, ay = 0.0;
  if (D < 0) {
    for (int d = 0; d < N; ++d) {
      int q = i + d;
      if (q >= N) q -= N;
      const double f = sc ? tau[d] * sc[q] : tau[d];
      ax += f * z[q].x;
      ay += f * z[q].y;
    }
  } else {
#pragma unroll
    for (int d = -kTauD; d <= kTauD; ++d) {
      int q = i + d;
      q = q < 0 ? q + N : (q >= N ? q - N : q);
      const double f = sc ? tau[d < 0 ? -d : d] * sc[q] : tau[d < 0 ? -d : d];
      ax += f * z[q].x;
      ay += f * z[q].y;
    }
  }
  return make_double2(ax, ay);
}

// u = R^T G_pd^-1 x (refined-hat coefficients, 2N per column): with
// z = T^-1 diag(1/h) x, u_2j+1 = z_j and u_2j = (z_j-1 + z_j) / 2.  Block b
// forms z_j for j = 255 b - 1 .. 255 b + 254 in LDS and writes u for the
// 255 indices j >= 255 b, so every z is computed once.
__global__ __launch_bounds__(256) void k_dual_in(int N, int nrhs, int D, const double* __restrict__ tau,
                                                 const double* __restrict__ ih, const double2* __restrict__ x,
                                                 int64_t ldx, double2* __restrict__ u, int64_t ldu) {
  __shared__ double2 zs[256];
  const int t = threadIdx.x, r = blockIdx.y;
  const int j = blockIdx.x * 255 + t - 1;       // this thread's z index (j = -1: the halo)
  const double2* xr = x + (size_t)r * ldx;
  if (j < N) zs[t] = tinv_at(N, D, tau, j < 0 ? N - 1 : j, xr, ih);
  __syncthreads();
  if (t >= 1 && j < N) {
    double2* ur = u + (size_t)r * ldu;
    const double2 zj = zs[t], zm = zs[t - 1];
    ur[2 * j + 1] = zj;
    ur[2 * j] = make_double2(0.5 * (zm.x + zj.x), 0.5 * (zm.y + zj.y));
  }
}

// k_dual_in for the banded T^-1 (D >= 0): the block's x and 1/h window
// (256 + 2 kTauD values, cyclic) is staged in LDS; each sum runs over the
// same terms in the same order as tinv_at.
__global__ __launch_bounds__(256) void k_dual_in_band(int N, const double* __restrict__ tau,
                                                      const double* __restrict__ ih, const double2* __restrict__ x,
                                                      int64_t ldx, double2* __restrict__ u, int64_t ldu) {
  constexpr int W = 256 + 2 * kTauD;
  __shared__ double2 xs[W];
  __shared__ double hs[W];
  __shared__ double2 zs[256];
  const int t = threadIdx.x, r = blockIdx.y;
  const double2* xr = x + (size_t)r * ldx;
  const int64_t base = (int64_t)blockIdx.x * 255 - 1 - kTauD;   // unknown of window slot 0
  for (int k = t; k < W; k += 256) {
    int q = (int)((base + k) % N);
    if (q < 0) q += N;
    xs[k] = xr[q];
    hs[k] = ih[q];
  }
  __syncthreads();
  const int j = blockIdx.x * 255 + t - 1;   // this thread's z index (j = -1: the halo)
  if (j < N) {
    double ax = 0.0, ay = 0.0;
#pragma unroll
    for (int d = -kTauD; d <= kTauD; ++d) {
      const int k = t + kTauD + d;
      const double f = tau[d < 0 ? -d : d] * hs[k];
      ax += f * xs[k].x;
      ay += f * xs[k].y;
    }
    zs[t] = make_double2(ax, ay);
  }
  __syncthreads();
  if (t >= 1 && j < N) {
    double2* ur = u + (size_t)r * ldu;
    const double2 zj = zs[t], zm = zs[t - 1];
    ur[2 * j + 1] = zj;
    ur[2 * j] = make_double2(0.5 * (zm.x + zj.x), 0.5 * (zm.y + zj.y));
  }
}

// k_dual_gather and k_dual_out in one pass for the banded T^-1: the block
// forms g_q = w_2q / 2 + w_2q+1 + w_2q+2 / 2 over its output window plus
// kTauD on each side (cyclic) in LDS, then y_i = (T^-1 g)_i / h_i with the
// terms in tinv_at's order.
__global__ __launch_bounds__(256) void k_dual_out_band(int N, const double* __restrict__ tau,
                                                       const double* __restrict__ ih, const double2* __restrict__ w,
                                                       int64_t ldw, double2* __restrict__ y, int64_t ldy) {
  constexpr int W = 256 + 2 * kTauD;
  __shared__ double2 gs[W];
  const int t = threadIdx.x, r = blockIdx.y;
  const double2* wr = w + (size_t)r * ldw;
  const int64_t base = (int64_t)blockIdx.x * 256 - kTauD;
  for (int k = t; k < W; k += 256) {
    int q = (int)((base + k) % N);
    if (q < 0) q += N;
    const double2 a = wr[2 * q], b = wr[2 * q + 1], e = wr[q == N - 1 ? 0 : 2 * q + 2];
    gs[k] = make_double2(0.5 * a.x + b.x + 0.5 * e.x, 0.5 * a.y + b.y + 0.5 * e.y);
  }
  __syncthreads();
  const int i = blockIdx.x * 256 + t;
  if (i >= N) return;
  double ax = 0.0, ay = 0.0;
#pragma unroll
  for (int d = -kTauD; d <= kTauD; ++d) {
    const int k = t + kTauD + d;
    const double f = tau[d < 0 ? -d : d];
    ax += f * gs[k].x;
    ay += f * gs[k].y;
  }
  y[(size_t)r * ldy + i] = make_double2(ax * ih[i], ay * ih[i]);
}

// g_j = w_2j / 2 + w_2j+1 + w_2j+2 / 2 (R w)
__global__ void k_dual_gather(int N, int nrhs, const double2* __restrict__ w, int64_t ldw, double2* __restrict__ g,
                              int64_t ldg) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  if (j >= N) return;
  const double2* wr = w + (size_t)r * ldw;
  const double2 a = wr[2 * j], b = wr[2 * j + 1], e = wr[j == N - 1 ? 0 : 2 * j + 2];
  g[(size_t)r * ldg + j] = make_double2(0.5 * a.x + b.x + 0.5 * e.x, 0.5 * a.y + b.y + 0.5 * e.y);
}

// y = G_pd^-T g = diag(1/h) T^-1 g
__global__ void k_dual_out(int N, int nrhs, int D, const double* __restrict__ tau, const double* __restrict__ ih,
                           const double2* __restrict__ g, int64_t ldg, double2* __restrict__ y, int64_t ldy) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  if (i >= N) return;
  const double2 t = tinv_at(N, D, tau, i, g + (size_t)r * ldg, nullptr);
  y[(size_t)r * ldy + i] = make_double2(t.x * ih[i], t.y * ih[i]);
}

// y = G_pd^-T N'(alpha) G_pd^-1 x through the dual hat context
static aim_status tm_precond(Ctx* c, bool filtered, bool f32, int nrhs, const double2* x, int64_t ldx, double2* y,
                             int64_t ldy) {
  Ctx* d = c->dual;
  const int N = c->t.N, N2 = d->t.N;
  const dim3 g((N + 255) / 256, nrhs);
  const bool band = c->tau_D >= 0;
  if (band)
    hipLaunchKernelGGL(k_dual_in_band, dim3((N + 254) / 255, nrhs), dim3(256), 0, c->stream, N, c->d_tau, c->d_ih, x,
                       ldx, d->d_tmp1, (int64_t)N2);
  else
    hipLaunchKernelGGL(k_dual_in, dim3((N + 254) / 255, nrhs), dim3(256), 0, c->stream, N, nrhs, c->tau_D,
                       c->d_tau, c->d_ih, x, ldx, d->d_tmp1, (int64_t)N2);
  AIM_HIP_CHECK(hipGetLastError());
  const int nop = (filtered ? AIM_OP_N_ALPHA : AIM_OP_N) | (f32 ? AIM_OP_GRID_FP32 : 0);
  TRY(matvec(d, nop, nrhs, d->d_tmp1, N2, d->d_tmp2, N2));
  if (band) {
    hipLaunchKernelGGL(k_dual_out_band, g, dim3(256), 0, c->stream, N, c->d_tau, c->d_ih, d->d_tmp2, (int64_t)N2, y,
                       ldy);
  } else {
    hipLaunchKernelGGL(k_dual_gather, g, dim3(256), 0, c->stream, N, nrhs, d->d_tmp2, (int64_t)N2, d->d_tmp1,
                       (int64_t)N);
    hipLaunchKernelGGL(k_dual_out, g, dim3(256), 0, c->stream, N, nrhs, c->tau_D, c->d_tau, c->d_ih, d->d_tmp1,
                       (int64_t)N, y, ldy);
  }
  AIM_HIP_CHECK(hipGetLastError());
  return AIM_OK;
}

static aim_status gram_inv(Ctx* c, int nrhs, const double2* x, int64_t ldx, double2* y, int64_t ldy) {
  HostTables& t = c->t;
  const int N = t.N;
  if (t.basis == AIM_PULSE) {
    hipLaunchKernelGGL(k_gram_pulse, dim3((N + 255) / 256, nrhs), dim3(256), 0, c->stream, N, nrhs, c->d_h, x, ldx,
                       y, ldy);
  } else if (N >= GP) {
    const int nblk = (N + GPO - 1) / GPO;
    hipLaunchKernelGGL(k_gram_hat_pcr, dim3(nblk, nrhs), dim3(GP), 0, c->stream, N, c->d_h, x, ldx, y, ldy);
  } else if (N >= GM) {
    const int nblk = (N + GB - 1) / GB;
    hipLaunchKernelGGL(k_gram_hat_blocks, dim3((nblk + 63) / 64, nrhs), dim3(64), 0, c->stream, N, nrhs, c->d_h, x,
                       ldx, y, ldy);
  } else {
    hipLaunchKernelGGL(k_gram_hat_small, dim3((nrhs + 63) / 64), dim3(64), 0, c->stream, N, nrhs, c->d_h, x, ldx,
                       y, ldy, c->d_red);
  }
  AIM_HIP_CHECK(hipGetLastError());
  return AIM_OK;
}

aim_status matvec(Ctx* c, int op, int nrhs, const double2* x, int64_t ldx, double2* y, int64_t ldy) {
  const bool f32 = (op & AIM_OP_GRID_FP32) != 0;
  const int base = op & 0xff;
  if (nrhs < 1 || nrhs > c->max_rhs) return AIM_E_ARG;
  if (f32 && c->precision != AIM_MIXED) return AIM_E_ARG;
  const bool hat = c->t.basis == AIM_HAT;
  if ((base == AIM_OP_N || base == AIM_OP_N_ALPHA || base == AIM_OP_TE_CP || base == AIM_OP_TE_CP_UNF) && !hat)
    return AIM_E_ARG;
  const bool tmc = base >= AIM_OP_TM_PC && base <= AIM_OP_TM_CP_UNF;
  if (tmc && hat) return AIM_E_ARG;
  if (tmc && !c->dual) return AIM_E_STATE;   // set up without the dual space
  // the per-node map has no near-field correction: only the filtered operators and G^-1
  if (c->t.node_order != 0 && base != AIM_OP_S_ALPHA && base != AIM_OP_N_ALPHA && base != AIM_OP_GRAM_INV)
    return AIM_E_STATE;
  const double2 one = make_double2(1.0, 0.0);
  auto grid = [&](int b, const double2* xx, int64_t lx, double2* yy, int64_t ly, double2 sc) {
    return f32 ? op_grid<float>(c, b, nrhs, xx, lx, yy, ly, sc) : op_grid<double>(c, b, nrhs, xx, lx, yy, ly, sc);
  };
  const int64_t N = c->t.N;
  switch (base) {
    case AIM_OP_S:
    case AIM_OP_S_ALPHA:
    case AIM_OP_N:
    case AIM_OP_N_ALPHA:
      return grid(base, x, ldx, y, ldy, one);
    case AIM_OP_TM_PC:
    case AIM_OP_TM_PC_UNF:
      return tm_precond(c, base == AIM_OP_TM_PC, f32, nrhs, x, ldx, y, ldy);
    case AIM_OP_TM_CP:
    case AIM_OP_TM_CP_UNF:
      TRY(grid(AIM_OP_S, x, ldx, c->d_tmp1, N, make_double2(0.0, c->t.k * c->t.eta)));
      return tm_precond(c, base == AIM_OP_TM_CP, f32, nrhs, c->d_tmp1, N, y, ldy);
    case AIM_OP_TM:
      return grid(AIM_OP_S, x, ldx, y, ldy, make_double2(0.0, c->t.k * c->t.eta));
    case AIM_OP_GRAM_INV:
      return gram_inv(c, nrhs, x, ldx, y, ldy);
    case AIM_OP_TE_CP:
    case AIM_OP_TE_CP_UNF:
      TRY(grid(AIM_OP_N, x, ldx, c->d_tmp1, N, one));
      TRY(gram_inv(c, nrhs, c->d_tmp1, N, c->d_tmp2, N));
      TRY(grid(base == AIM_OP_TE_CP ? AIM_OP_S_ALPHA : AIM_OP_S, c->d_tmp2, N, c->d_tmp1, N, one));
      return gram_inv(c, nrhs, c->d_tmp1, N, y, ldy);
  }
  return AIM_E_ARG;
}

// ---------------------------------------------------------------------------
// matvec split at its column pass (the grouped solver step): operators with
// one grid product run as matvec_pre -> column pass -> matvec_post, and the
// column passes of several contexts that share a spectrum go into one
// launch (launch_cols_jobs).  Each tile is computed as by matvec.
// ---------------------------------------------------------------------------
static bool split_parts(Ctx* c, int op, const int** chans, int* nch, bool* filt, bool* near, double* sg,
                        double2* scale) {
  static const int chS[1] = {0};
  static const int chN[3] = {1, 2, 3};
  const int base = op & 0xff;
  const bool hat = c->t.basis == AIM_HAT;
  *scale = make_double2(1.0, 0.0);
  switch (base) {
    case AIM_OP_S: case AIM_OP_S_ALPHA: case AIM_OP_TM:
      if (base == AIM_OP_TM && hat) return false;
      *chans = chS; *nch = 1; *sg = 0.0;
      *filt = base == AIM_OP_S_ALPHA;
      *near = !*filt;
      if (base == AIM_OP_TM) *scale = make_double2(0.0, c->t.k * c->t.eta);
      break;
    case AIM_OP_N: case AIM_OP_N_ALPHA:
      if (!hat) return false;
      *chans = chN; *nch = 3; *sg = -c->t.k * c->t.k;
      *filt = base == AIM_OP_N_ALPHA;
      *near = !*filt;
      break;
    default:
      return false;
  }
  if (c->t.node_order != 0 && *near) return false;
  if ((op & AIM_OP_GRID_FP32) && c->precision != AIM_MIXED) return false;
  return true;
}

bool matvec_splits(Ctx* c, int op) {
  const int* ch; int nch; bool filt, near; double sg; double2 sc;
  return split_parts(c, op, &ch, &nch, &filt, &near, &sg, &sc);
}

aim_status matvec_pre(Ctx* c, int op, int nrhs, const double2* x, int64_t ldx, ColsJob* job) {
  const int* ch; int nch; bool filt, near; double sg; double2 sc;
  if (nrhs < 1 || nrhs > c->max_rhs || !split_parts(c, op, &ch, &nch, &filt, &near, &sg, &sc)) return AIM_E_ARG;
  const bool f32 = (op & AIM_OP_GRID_FP32) != 0;
  job->n = c->t.n;
  job->nr = c->t.nr;
  job->ldt = tile_rows(c->t.nr);
  job->pairs = nch * nrhs;
  job->f32 = f32;
  job->tiles = c->d_T;
  job->kcut = grid_kcut(c, filt);
  if (f32) {
    job->Cq = grid_spectrum<float>(c, filt);
    job->tw = grid_twiddles<float>(c);
    return grid_pre<float>(c, ch, nch, filt, nrhs, x, ldx);
  }
  job->Cq = grid_spectrum<double>(c, filt);
  job->tw = grid_twiddles<double>(c);
  return grid_pre<double>(c, ch, nch, filt, nrhs, x, ldx);
}

aim_status matvec_post(Ctx* c, int op, int nrhs, const double2* x, int64_t ldx, double2* y, int64_t ldy) {
  const int* ch; int nch; bool filt, near; double sg; double2 sc;
  if (!split_parts(c, op, &ch, &nch, &filt, &near, &sg, &sc)) return AIM_E_ARG;
  const double2* Cn = near ? (nch == 1 ? c->d_CS : c->d_CN) : nullptr;
  if (op & AIM_OP_GRID_FP32) {
    TRY(grid_post<float>(c, nch, filt, nrhs));
    return interp<float>(c, ch, nch, sg, near, Cn, nrhs, x, ldx, y, ldy, sc);
  }
  TRY(grid_post<double>(c, nch, filt, nrhs));
  return interp<double>(c, ch, nch, sg, near, Cn, nrhs, x, ldx, y, ldy, sc);
}

// One column pass over the tile sets of `count` jobs with the same spectrum,
// twiddles, n and precision, in launches of up to ColBatch::kMax pairs.
aim_status launch_cols_jobs(const ColsJob* jobs, int count, hipStream_t s) {
  if (count < 1) return AIM_OK;
  const int n = jobs[0].n;
  const bool f32 = jobs[0].f32;
  const int cb = col_block(n, f32);
  if (cb <= 0) return AIM_E_ARG;
  std::vector<void*> tiles;
  std::vector<int> nr, ldt;
  for (int i = 0; i < count; ++i) {
    const ColsJob& j = jobs[i];
    if (j.n != n || j.f32 != f32 || j.Cq != jobs[0].Cq || j.kcut != jobs[0].kcut) return AIM_E_ARG;
    const size_t pair_bytes = (size_t)(n / cb) * j.ldt * cb * (f32 ? 8 : 16);
    for (int p = 0; p < j.pairs; ++p) {
      tiles.push_back((char*)j.tiles + p * pair_bytes);
      nr.push_back(j.nr);
      ldt.push_back(j.ldt);
    }
  }
  const int total = (int)tiles.size();
  for (int e0 = 0; e0 < total; e0 += kColBatchMax) {
    const int cnt = std::min(kColBatchMax, total - e0);
    if (f32)
      TRY(launch_cols_group<float>(n, cnt, tiles.data() + e0, nr.data() + e0, ldt.data() + e0, jobs[0].kcut,
                                   (const float2*)jobs[0].Cq, (const float2*)jobs[0].tw, s));
    else
      TRY(launch_cols_group<double>(n, cnt, tiles.data() + e0, nr.data() + e0, ldt.data() + e0, jobs[0].kcut,
                                    (const double2*)jobs[0].Cq, (const double2*)jobs[0].tw, s));
  }
  return AIM_OK;
}

// The angles go to the context's buffer; the call waits for the copy, so
// the caller's host array is free on return.
aim_status rhs_planewave(Ctx* c, int nrhs, const double* phi_host, double amp, double2* b) {
  HostTables& t = c->t;
  if (nrhs < 1 || nrhs > AIM_MAX_RHS) return AIM_E_ARG;
  AIM_HIP_CHECK(hipMemcpyAsync(c->d_phi, phi_host, (size_t)nrhs * 8, hipMemcpyHostToDevice, c->stream));
  hipLaunchKernelGGL(k_rhs, dim3((t.N + 127) / 128, nrhs), dim3(128), 0, c->stream, t.N, nrhs, t.basis, t.p,
                     c->d_glx, c->d_glw, c->d_vx, c->d_vy, c->d_h, c->d_tx, c->d_ty, c->d_phi, t.k, t.eta, amp, b);
  AIM_HIP_CHECK(hipGetLastError());
  AIM_HIP_CHECK(hipStreamSynchronize(c->stream));
  return AIM_OK;
}

// ---------------------------------------------------------------------------
// Fourier (Laplace-Beltrami) spectrum of an operator on a closed contour
// ---------------------------------------------------------------------------
// e[r][j] = exp(i 2 pi nu_r j / N), phase reduced exactly: (nu j) mod N
__global__ void k_fourier_modes(int N, int nrhs, const int32_t* __restrict__ nu, double2* __restrict__ e) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  if (j >= N || r >= nrhs) return;
  int64_t q = ((int64_t)nu[r] * j) % N;
  if (q < 0) q += N;
  double sn, cs;
  sincospi(2.0 * (double)q / (double)N, &sn, &cs);
  e[(size_t)r * N + j] = make_double2(cs, sn);
}

// out[r] = (1/N) sum_j conj(e[r][j]) y[r][j], fixed reduction order
__global__ __launch_bounds__(256) void k_mode_quotient(int N, const double2* __restrict__ e,
                                                       const double2* __restrict__ y, double2* __restrict__ out) {
  const int r = blockIdx.x;
  const double2* er = e + (size_t)r * N;
  const double2* yr = y + (size_t)r * N;
  double sx = 0.0, sy = 0.0;
  for (int j = threadIdx.x; j < N; j += 256) {
    const double2 a = er[j], b = yr[j];
    sx += a.x * b.x + a.y * b.y;
    sy += a.x * b.y - a.y * b.x;
  }
  __shared__ double rx[256], ry[256];
  rx[threadIdx.x] = sx;
  ry[threadIdx.x] = sy;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      rx[threadIdx.x] += rx[threadIdx.x + st];
      ry[threadIdx.x] += ry[threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) out[r] = make_double2(rx[0] / N, ry[0] / N);
}

aim_status fourier_spectrum(Ctx* c, int op, int n_modes, const int32_t* nu_host, double2* lambda_host) {
  const HostTables& t = c->t;
  const int base = op & 0xff;
  const bool galerkin = base == AIM_OP_S || base == AIM_OP_S_ALPHA || base == AIM_OP_N || base == AIM_OP_N_ALPHA ||
                        base == AIM_OP_TM;
  const bool precond = base == AIM_OP_TE_CP || base == AIM_OP_TE_CP_UNF || base == AIM_OP_TM_CP ||
                       base == AIM_OP_TM_CP_UNF;
  if (n_modes < 1 || !nu_host || !lambda_host || (!galerkin && !precond)) return AIM_E_ARG;
  const int N = t.N, R = c->max_rhs;
  if (!c->d_spec) TRY(dev_alloc(c, (void**)&c->d_spec, ((size_t)3 * N * R + 2 * (size_t)R) * sizeof(double2)));
  double2* E = c->d_spec;                      // modes
  double2* Y = E + (size_t)N * R;              // op e
  double2* Z = Y + (size_t)N * R;              // G^-1 op e
  double2* Q = Z + (size_t)N * R;              // quotients
  int32_t* nud = (int32_t*)(Q + R);
  for (int m0 = 0; m0 < n_modes; m0 += R) {
    const int nr = std::min(R, n_modes - m0);
    AIM_HIP_CHECK(hipMemcpyAsync(nud, nu_host + m0, nr * 4, hipMemcpyHostToDevice, c->stream));
    hipLaunchKernelGGL(k_fourier_modes, dim3((N + 255) / 256, nr), dim3(256), 0, c->stream, N, nr, nud, E);
    AIM_HIP_CHECK(hipGetLastError());
    TRY(matvec(c, op, nr, E, N, Y, N));
    const double2* out = Y;
    if (galerkin) {   // quotient of G^-1 op: the continuous operator's eigenvalue on the circle
      TRY(matvec(c, AIM_OP_GRAM_INV, nr, Y, N, Z, N));
      out = Z;
    }
    hipLaunchKernelGGL(k_mode_quotient, dim3(nr), dim3(256), 0, c->stream, N, E, out, Q);
    AIM_HIP_CHECK(hipGetLastError());
    AIM_HIP_CHECK(hipMemcpyAsync(lambda_host + m0, Q, nr * 16, hipMemcpyDeviceToHost, c->stream));
    AIM_HIP_CHECK(hipStreamSynchronize(c->stream));
  }
  return AIM_OK;
}

// sigma_r = scale |dot_r|^2
__global__ void k_sigma(int nrhs, double scale, const double2* __restrict__ dot, double* __restrict__ sigma) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < nrhs) sigma[r] = scale * (dot[r].x * dot[r].x + dot[r].y * dot[r].y);
}

// sigma_r = (k eta^2 / 4) |sum_j b_j(phi_r) J_jr|^2 with b the plane-wave
// right-hand side of unit amplitude, on device buffers phi_dev (nrhs
// angles), b_dev (N x nrhs), dot_dev (nrhs sums) and sig_dev (nrhs values);
// the values go to sigma_host, nothing else touches host memory
aim_status rcs_into(Ctx* c, int nrhs, const double2* J, const double* phi_host, double* sigma_host, double* phi_dev,
                    double2* b_dev, double2* dot_dev, double* sig_dev) {
  HostTables& t = c->t;
  AIM_HIP_CHECK(hipMemcpyAsync(phi_dev, phi_host, (size_t)nrhs * 8, hipMemcpyHostToDevice, c->stream));
  hipLaunchKernelGGL(k_rhs, dim3((t.N + 127) / 128, nrhs), dim3(128), 0, c->stream, t.N, nrhs, t.basis, t.p,
                     c->d_glx, c->d_glw, c->d_vx, c->d_vy, c->d_h, c->d_tx, c->d_ty, phi_dev, t.k, t.eta, 1.0, b_dev);
  hipLaunchKernelGGL(k_dotu_cols, dim3(nrhs), dim3(256), 0, c->stream, t.N, b_dev, J, (double*)dot_dev);
  hipLaunchKernelGGL(k_sigma, dim3((nrhs + 255) / 256), dim3(256), 0, c->stream, nrhs, t.k * t.eta * t.eta / 4.0,
                     dot_dev, sig_dev);
  AIM_HIP_CHECK(hipGetLastError());
  AIM_HIP_CHECK(hipMemcpyAsync(sigma_host, sig_dev, (size_t)nrhs * 8, hipMemcpyDeviceToHost, c->stream));
  AIM_HIP_CHECK(hipStreamSynchronize(c->stream));
  return AIM_OK;
}

aim_status rcs(Ctx* c, int nrhs, const double2* J, const double* phi_host, double* sigma) {
  if (c->t.basis != AIM_PULSE || nrhs < 1 || nrhs > c->max_rhs) return AIM_E_ARG;
  return rcs_into(c, nrhs, J, phi_host, sigma, c->d_phi, c->d_rhs, c->d_dot, (double*)(c->d_dot + c->max_rhs));
}

// Complex slots of scratch one call needs: angles and values (nrhs doubles
// each), sums (nrhs) and the plane-wave vectors (N x nrhs), each region
// rounded to 16 slots (256 bytes).
static size_t noalloc_slots(size_t N, size_t nrhs) {
  auto r16 = [](size_t v) { return (v + 15) / 16 * 16; };
  return 2 * r16((nrhs + 1) / 2) + r16(nrhs) + r16(N * nrhs);
}

aim_status rcs_noalloc(Ctx* c, int nrhs, const double2* J, const double* phi_host, double* sigma) {
  if (c->t.basis != AIM_PULSE || nrhs < 1 || nrhs > AIM_MAX_RHS) return AIM_E_ARG;
  if (noalloc_slots((size_t)c->t.N, (size_t)nrhs) > kNoAllocScratch) return AIM_E_ARG;
  if (c->device < 0 || c->device >= kMaxDevices) return AIM_E_HIP;
  double2* base;
  {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    base = g_scratch_dev[c->device];
  }
  if (!base) return AIM_E_STATE;
  auto r16 = [](size_t v) { return (v + 15) / 16 * 16; };
  const size_t nh = r16(((size_t)nrhs + 1) / 2);
  double* phi_dev = (double*)base;
  double* sig_dev = (double*)(base + nh);
  double2* dot_dev = base + 2 * nh;
  double2* b_dev = dot_dev + r16((size_t)nrhs);
  return rcs_into(c, nrhs, J, phi_host, sigma, phi_dev, b_dev, dot_dev, sig_dev);
}

aim_status eval_green(Ctx* c, int n, const double* R, double2* out) {
  if (n < 0) return AIM_E_ARG;
  if (n == 0) return AIM_OK;
  hipLaunchKernelGGL(k_eval_green, dim3((n + 255) / 256), dim3(256), 0, c->stream, n, R, c->t.k, out);
  AIM_HIP_CHECK(hipGetLastError());
  return AIM_OK;
}

}  // namespace aim
