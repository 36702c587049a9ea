// Reaction densities and Sommerfeld-type integrals on the GPU (plan time).
//
// * Densities sigma^{ab}_{l l'}(k) of App. A at complex k: the interface
//   conditions (u and eps du/dz continuous) are resolved by the stable
//   generalized-reflection recursion (downward and upward reflection
//   coefficients seen through every layer stack, then transmission from the
//   source layer to the target layer), valid for Re k >= 0.
// * Initial values S^n I_{n,0} (n <= nmax) and S^n I_{n,1} (1 <= n <= nmax) of
//   eq. scaledsommerfeldint: with two interfaces a series of images in closed
//   form; otherwise composite Gauss-Legendre quadrature with panels graded
//   geometrically towards 0, along the real axis when rho <= z + zinf,
//   otherwise along the imaginary axis in the K_m form of eq. contourchange
//   (Sec. 3.4), zinf being the density's decay length (eq. densityasymptotic).
// * The remaining orders by the forward recurrence of eq. recurrence.
// * Reaction near-field kernels (1/4pi) I_{00} for particle pairs.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "fmm_internal.h"

namespace fmmlm {
namespace {

constexpr int kGL = 16;
// The first panel [0, h0] is replaced by [0, h0 2^-Z] and [h0 2^-k, h0 2^-(k-1)],
// k = Z..1, which integrates the logarithmic singularity of K_0 at 0 to full accuracy.
constexpr int kZoom = 40;
__constant__ double c_glx[kGL];
__constant__ double c_glw[kGL];

// ---------------------------------------------------------------- densities
struct Scatter {
  double Rdn[kMaxL], Tdn[kMaxL], Rup[kMaxL], Tup[kMaxL];
};

__device__ void local_coeffs(const Medium& md, Scatter& sc) {
  for (int i = 0; i < md.L; ++i) {
    const double e0 = md.eps[i], e1 = md.eps[i + 1], s = e0 + e1;
    sc.Rdn[i] = (e0 - e1) / s;  // downgoing wave in layer i reflected at d_i
    sc.Tdn[i] = 2.0 * e0 / s;   // ... transmitted into layer i+1
    sc.Rup[i] = (e1 - e0) / s;  // upgoing wave in layer i+1 reflected at d_i
    sc.Tup[i] = 2.0 * e1 / s;   // ... transmitted into layer i
  }
}

// sigma^{ab}_{lt,ls}(k) of the classic conditions for md.eps; k complex with
// Re k >= 0.
__device__ cplx density_classic(const Medium& md, const Scatter& sc, int lt, int ls, int a, int b, cplx k) {
  const int L = md.L;
  // propagation factor across finite layer i (1 <= i <= L-1): e_i = exp(-k D_i)
  cplx e[kMaxL + 1], e2[kMaxL + 1];
  for (int i = 0; i <= L; ++i) {
    if (i >= 1 && i <= L - 1) {
      const double D = md.d[i - 1] - md.d[i];
      e[i] = cexp_dev(cmk(-k.re * D, -k.im * D));
    } else {
      e[i] = cmk(0.0, 0.0);
    }
    e2[i] = e[i] * e[i];
  }
  // generalized reflection looking down from layer i at d_i, and looking up
  // from layer i+1 at d_i
  cplx Gdn[kMaxL], Gup[kMaxL];
  Gdn[L - 1] = cmk(sc.Rdn[L - 1], 0.0);
  for (int i = L - 2; i >= 0; --i) {
    const cplx x = e2[i + 1] * Gdn[i + 1];
    const cplx num = (sc.Tdn[i] * sc.Tup[i]) * x;
    const cplx den = cmk(1.0, 0.0) - sc.Rup[i] * x;
    Gdn[i] = cmk(sc.Rdn[i], 0.0) + cdiv(num, den);
  }
  Gup[0] = cmk(sc.Rup[0], 0.0);
  for (int i = 1; i <= L - 1; ++i) {
    const cplx x = e2[i] * Gup[i - 1];
    const cplx num = (sc.Tup[i] * sc.Tdn[i]) * x;
    const cplx den = cmk(1.0, 0.0) - sc.Rdn[i] * x;
    Gup[i] = cmk(sc.Rup[i], 0.0) + cdiv(num, den);
  }
  // amplitudes in the source layer: u (upgoing at d_ls), w (downgoing at d_{ls-1})
  const cplx zero = cmk(0.0, 0.0), one = cmk(1.0, 0.0);
  const cplx Rd = (ls <= L - 1) ? Gdn[ls] : zero;
  const cplx Ru = (ls >= 1) ? Gup[ls - 1] : zero;
  const cplx es = e[ls];
  const cplx den = one - Rd * Ru * e2[ls];
  cplx u, w;
  if (b == 1) {
    u = cdiv(Rd, den);
    w = Ru * es * u;
  } else {
    w = cdiv(Ru, den);
    u = Rd * es * w;
  }
  if (lt == ls) return (a == 1) ? u : w;
  if (lt < ls) {
    // upgoing amplitude s1 at the bottom interface of each layer above the source
    cplx inc = (b == 2 ? one : zero) + es * u;  // upgoing at d_{ls-1} inside the source layer
    cplx s1 = zero;
    for (int i = ls - 1; i >= lt; --i) {
      const cplx g = (i >= 1) ? Gup[i - 1] : zero;
      const cplx dd = one - sc.Rdn[i] * (e2[i] * g);
      s1 = cdiv(sc.Tup[i] * inc, dd);
      inc = e[i] * s1;
    }
    if (a == 1) return s1;
    return (lt >= 1) ? Gup[lt - 1] * (e[lt] * s1) : zero;
  }
  // lt > ls: downgoing amplitude s2 at the top interface of each layer below
  cplx inc = (b == 1 ? one : zero) + es * w;  // downgoing at d_ls inside the source layer
  cplx s2 = zero;
  for (int i = ls + 1; i <= lt; ++i) {
    const cplx g = (i <= L - 1) ? Gdn[i] : zero;
    const cplx dd = one - sc.Rup[i - 1] * (e2[i] * g);
    s2 = cdiv(sc.Tdn[i - 1] * inc, dd);
    inc = e[i] * s2;
  }
  if (a == 2) return s2;
  return (lt <= L - 1) ? Gdn[lt] * (e[lt] * s2) : zero;
}

// sigma^{ab}_{lt,ls}(k) of the medium's interface conditions (factor a_ls / a_lt,
// exactly 1 for the classic conditions)
__device__ cplx density(const Medium& md, const Scatter& sc, int lt, int ls, int a, int b, cplx k) {
  if (md.L == 0) return cmk(1.0, 0.0);
  return (md.acoef[ls] / md.acoef[lt]) * density_classic(md, sc, lt, ls, a, b, k);
}

// ---------------------------------------------------------------- Bessel K_0, K_1
// K_m(x) = int_0^inf exp(-x cosh t) cosh(m t) dt (DLMF 10.32.9), trapezoidal
// rule with step 1/8: the integrand is analytic in |Im t| < pi/2 and decays
// double-exponentially, so the rule is accurate to roughly exp(-pi^2 / h).
__device__ void bessel_k01(double x, double* k0, double* k1) {
  const double h = 0.125;
  const double eh = exp(h);
  double E = 1.0;  // exp(t)
  double s0 = 0.5 * exp(-x), s1 = 0.5 * exp(-x);
  for (int i = 1; i < 4000; ++i) {
    E *= eh;
    const double ch = 0.5 * (E + 1.0 / E);
    const double f = exp(-x * ch);
    s0 += f;
    s1 += f * ch;
    if (x * ch > 745.0) break;
  }
  *k0 = h * s0;
  *k1 = h * s1;
}

// ---------------------------------------------------------------- quadrature
struct Panels {
  double h0, ratio, hmax, kmax;
};

// geometric grading from h0 (ratio 1.25) up to hmax, then uniform to kmax
__device__ inline double next_h(double h, const Panels& pn) {
  const double t = h * pn.ratio;
  return t < pn.hmax ? t : pn.hmax;
}

__device__ double min_thickness(const Medium& md) {
  double m = 0.0;
  for (int i = 1; i < md.L; ++i) {
    const double t = md.d[i - 1] - md.d[i];
    if (m == 0.0 || t < m) m = t;
  }
  return m;
}

__device__ double max_thickness(const Medium& md) {
  double m = 0.0;
  for (int i = 1; i < md.L; ++i) {
    const double t = md.d[i - 1] - md.d[i];
    if (t > m) m = t;
  }
  return m;
}

// ---------------------------------------------------------------- initial values
// A task's initial values are computed by a group of kTaskLanes lanes (four
// tasks a wave): lane g takes node g of every quadrature panel and images g,
// g + 16, ...; the orders' sums stay in registers (the order loops are unrolled
// to MAXN with a uniform exit) and meet across the group once, at the end.
// What bounds it: a task is a serial chain of 100 to 200 panels, each node a
// density, Bessel functions and 2 (nmax + 1) sums.  One thread a task ran that
// chain 16 times as long with its order sums in scratch memory and left most of
// the chip idle (10,007 points at nmax = 20 are 157 waves): 16.7 ms for two
// interfaces, now 0.034 ms by their image series (34 images) and 2.1 ms by the
// quadrature (three interfaces; five: 3.7 ms).
constexpr int kTaskLanes = kGL;
constexpr int kTaskBlock = 128;
constexpr int kBlockTasks = kTaskBlock / kTaskLanes;
constexpr int kMaxOrder = 2 * kPMax;

// f(std::integral_constant<int, n>()) for n = 0 .. N
template <class F, int... n>
__device__ inline void for_orders_impl(F f, std::integer_sequence<int, n...>) {
  (f(std::integral_constant<int, n>()), ...);
}
template <int N, class F>
__device__ inline void for_orders(F f) {
  for_orders_impl(f, std::make_integer_sequence<int, N + 1>());
}

__device__ inline double group_sum(double v) {
#pragma unroll
  for (int k = 1; k < kTaskLanes; k <<= 1) v += __shfl_xor(v, k, kTaskLanes);
  return v;
}

// amp S^n P~_n^m(Z/R) / R^{n+1}, R = sqrt(rho^2 + Z^2), added to a0[n] (m = 0,
// n <= nmax) and a1[n] (m = 1, 1 <= n <= nmax).  This is the normalised integral
// of the density amp e^{-k Zi} at z = Z - Zi (Sec. 3.4:
// int_0^inf J_m(k rho) k^n e^{-k Z} dk = (n-m)! P_n^m(Z/R) / R^{n+1}, P_n^m without the
// Condon-Shortley phase), with P~_n^m = sqrt((n-m)!/(n+m)!) P_n^m.
template <int MAXN>
__device__ inline void add_image(double amp, double S, double rho, double Z, int nmax, double* a0, double* a1) {
  const double R = sqrt(rho * rho + Z * Z);
  const double x = Z / R, sn = rho / R, t = S / R;
  double pw = amp / R;
  double q0 = 0.0, p0 = 1.0;  // P_{n-1}^0, P_n^0
  double q1 = 0.0, p1 = sn;   // P_{n-1}^1, P_n^1 (n >= 1)
  for_orders<MAXN>([&](auto order) {
    constexpr int n = decltype(order)::value;
    if (n > nmax) return;
    a0[n] += pw * p0;
    if constexpr (n >= 1) {
      a1[n] += pw * p1 * (1.0 / __builtin_sqrt((double)n * (n + 1)));
      const double r1 = ((2.0 * n + 1.0) / n) * x * p1 - ((n + 1.0) / n) * q1;
      q1 = p1;
      p1 = r1;
    }
    const double r0 = ((2.0 * n + 1.0) / (n + 1.0)) * x * p0 - (n / (n + 1.0)) * q0;
    q0 = p0;
    p0 = r0;
    pw *= t;
  });
}

// The lane's share of the quadrature of the remainder sigma(k) - sinf e^{-k zinf}
// (the leading term, eq. densityasymptotic, is integrated in closed form), which
// decays like e^{-k (zinf + 2 dmin)}: node `lane` of every panel, normalised by
// 1/sqrt((n+m)!(n-m)!), into a0[n], a1[n] (overwritten).
template <int MAXN>
__device__ void quadrature_share(const Medium& md, const CompInfo& c, double S, double rho, double z, int nmax,
                                 int lane, double* a0, double* a1) {
  Scatter sc;
  local_coeffs(md, sc);
#pragma unroll
  for (int n = 0; n <= MAXN; ++n) a0[n] = a1[n] = 0.0;
  const bool want1 = MAXN > 0 && rho > 0.0;
  const double dmin = min_thickness(md);
  const double zq = z + c.zinf + 2.0 * dmin;  // decay length of the remainder
  const bool contour = rho > zq;
  double small = 1.0;
  if (zq < small) small = zq;
  if (dmin < small) small = dmin;
  if (contour && rho < small) small = rho;
  Panels pn;
  pn.ratio = 1.25;
  pn.h0 = 1e-3 * small;
  if (!contour) {
    // real axis: J_m(k rho) (kS)^n e^{-kz} (sigma(k) - sinf e^{-k zinf})
    // panel widths are inverse lengths: the remainder decays on 1/zq (and
    // zq >= 2 dmin, so thin layers shrink it), J_m(k rho) oscillates on pi/rho
    pn.kmax = (2.0 * nmax + 50.0) / zq;
    double hmax = 2.0 / zq;
    if (rho > 0.0 && 3.14159265358979 / rho < hmax) hmax = 3.14159265358979 / rho;
    pn.hmax = hmax;
  } else {
    // imaginary axis: (2/pi) K_m(eta rho) (S eta)^n x {(-1)^{(n-m)/2} Re w, (-1)^{(n-m+1)/2} Im w},
    // w = e^{-i eta z} (sigma(i eta) - sinf e^{-i eta zinf})
    pn.kmax = (2.0 * nmax + 50.0) / rho;
    double hmax = 2.0 / rho;
    // sigma(i eta) does not decay along the imaginary axis: a wave reflected
    // through the whole stack oscillates like e^{-2 i eta (stack thickness)},
    // so the panels resolve two round trips through the stack (for three
    // layers the stack is the one finite layer)
    const double stack = md.L >= 2 ? md.d[0] - md.d[md.L - 1] : 0.0;
    const double osc = z + c.zinf + 4.0 * fmax(max_thickness(md), stack);
    if (3.14159265358979 / osc < hmax) hmax = 3.14159265358979 / osc;
    pn.hmax = hmax;
  }
  const double gx = 0.5 * (c_glx[lane] + 1.0), gw = 0.5 * c_glw[lane];
  double k0 = 0.0, h = pn.h0;
  int zoom = kZoom + 1;  // first panel [0, h0] split geometrically towards 0
  while (k0 < pn.kmax) {
    double lo = k0, hh = h;
    if (zoom > 0) {
      hh = (zoom > kZoom) ? ldexp(pn.h0, -kZoom) : ldexp(pn.h0, -zoom);
      lo = (zoom > kZoom) ? 0.0 : hh;
    }
    const double k = lo + hh * gx;
    // per order n: f0, f1 multiply (kS)^n for m = 0, 1; on the contour the two
    // parts of w alternate with signs, so four factors cover n mod 4
    double e0, o0, e1 = 0.0, o1 = 0.0;
    if (!contour) {
      const double sg = density(md, sc, c.lt, c.ls, c.a, c.b, cmk(k, 0.0)).re - c.sinf * exp(-k * c.zinf);
      const double base = hh * gw * exp(-k * z) * sg;
      e0 = o0 = base * ((rho > 0.0) ? j0(k * rho) : 1.0);
      if (want1) e1 = o1 = base * j1(k * rho);
    } else {
      const double wq = hh * gw * (2.0 / 3.14159265358979323846);
      cplx sg = density(md, sc, c.lt, c.ls, c.a, c.b, cmk(0.0, k));
      double sn, cs, si, ci;
      sincos(k * z, &sn, &cs);
      sincos(k * c.zinf, &si, &ci);
      sg.re -= c.sinf * ci;
      sg.im += c.sinf * si;
      const cplx wv = cmk(cs, -sn) * sg;
      double kk0, kk1;
      bessel_k01(k * rho, &kk0, &kk1);
      // m = 0: n even -> (-1)^{n/2} Re w ; n odd -> (-1)^{(n+1)/2} Im w
      // m = 1: n odd -> (-1)^{(n-1)/2} Re w ; n even -> (-1)^{n/2} Im w
      e0 = wq * kk0 * wv.re;
      o0 = -wq * kk0 * wv.im;
      if (want1) {
        e1 = wq * kk1 * wv.im;
        o1 = wq * kk1 * wv.re;
      }
    }
    double pw = 1.0;  // (kS)^n, with the sign (-1)^{floor(n/2)} on the contour
    const double ks = k * S, flip = contour ? -ks : ks;
    for_orders<MAXN>([&](auto order) {
      constexpr int n = decltype(order)::value;
      if (n > nmax) return;
      a0[n] += ((n & 1) ? o0 : e0) * pw;
      if constexpr (n >= 1) a1[n] += ((n & 1) ? o1 : e1) * pw;
      pw *= (n & 1) ? flip : ks;
    });
    if (zoom > 0) {
      --zoom;
      if (zoom > 0) continue;
    }
    k0 += h;
    h = next_h(h, pn);
  }
  double fn = 1.0;  // n!
  for_orders<MAXN>([&](auto order) {
    constexpr int n = decltype(order)::value;
    if (n > 0) fn *= n;
    a0[n] *= 1.0 / fn;
    // (n+1)! (n-1)! = n!^2 (n+1)/n
    if constexpr (n >= 1) a1[n] *= 1.0 / (fn * __builtin_sqrt((n + 1.0) / n));
  });
}

// The lane's share of S^n I_{n,0}, S^n I_{n,1} (a0, a1; overwritten): the
// remainder as a series of images where the component has one (c.nimg >= 0),
// else by the quadrature; with the leading term's image unless !with_image.
// QUAD = false leaves the quadrature out of kernels launched for components that
// all have a series (the quadrature's density holds 1.2 KB a lane in scratch
// and its registers leave one or two waves a SIMD).
template <int MAXN, bool QUAD = true>
__device__ void initial_share(const Medium& md, const CompInfo& c, double S, double rho, double z, int nmax,
                              int lane, double* a0, double* a1, bool with_image = true) {
  if (QUAD && c.nimg < 0) {
    quadrature_share<MAXN>(md, c, S, rho, z, nmax, lane, a0, a1);
  } else {
#pragma unroll
    for (int n = 0; n <= MAXN; ++n) a0[n] = a1[n] = 0.0;
    if (lane < c.nimg) {
      double amp = c.img1 * pow(c.imgq, (double)lane);
      const double step = pow(c.imgq, (double)kTaskLanes);
      for (int j = lane; j < c.nimg; j += kTaskLanes) {
        add_image<MAXN>(amp, S, rho, z + c.zinf + (j + 1) * c.imgd, nmax, a0, a1);
        amp *= step;
      }
    }
  }
  if (with_image && lane == kTaskLanes - 1) add_image<MAXN>(c.sinf, S, rho, z + c.zinf, nmax, a0, a1);
}

// Sums the shares over the group and calls put(n, v0, v1) on lane n mod 16.
template <int MAXN, class Put>
__device__ inline void group_put(int nmax, int lane, const double* a0, const double* a1, Put put) {
  for_orders<MAXN>([&](auto order) {
    constexpr int n = decltype(order)::value;
    if (n > nmax) return;
    const double v0 = group_sum(a0[n]);
    double v1 = 0.0;
    if constexpr (n >= 1) v1 = group_sum(a1[n]);
    if (lane == n % kTaskLanes) put(n, v0, v1);
  });
}

// Coefficients of eq. recurrence for the entries (n, m + 1), m >= 1:
// S^n I_{n,m+1} = ca (S / rho) S^{n-1} I_{n-1,m} - cb S^n I_{n,m-1}.
__device__ inline void recurrence_coefs(int nmax, double* ca, double* cb) {
  const int w = nmax + 1;
  for (int i = threadIdx.x; i < w * w; i += kTaskBlock) {
    const int n = i / w, m = i % w - 1;
    if (m < 1 || m >= n) continue;
    const double anpm = sqrt((double)(n + m) * (n + m + 1));
    ca[cidx(n, m + 1)] = 2.0 * m / anpm;
    cb[cidx(n, m + 1)] = sqrt((double)(n - m) * (n - m + 1)) / anpm;
  }
}

// Orders M >= 2 of every task's table o [cidx(n, m)] (one per group, in LDS) by
// eq. recurrence: an order's degrees are independent, one lane each.  Then the
// block's tables (tasks first .. first + kBlockTasks - 1) go out in whole rows.
template <class Src>
__device__ inline void recurrence_store(const Src& src, int ntask, int nmax, double s_rho, int lane, double* o,
                                        const double* ca, const double* cb, const double* tab,
                                        double* __restrict__ out) {
  __syncthreads();
  for (int m = 1; m + 1 <= nmax; ++m) {
    for (int n = m + 1 + lane; n <= nmax; n += kTaskLanes) {
      const int i = cidx(n, m + 1);
      o[i] = s_rho > 0.0 ? ca[i] * s_rho * o[cidx(n - 1, m)] - cb[i] * o[cidx(n, m - 1)] : 0.0;
    }
    __syncthreads();
  }
  const int nc = ncoef(nmax);
  const int t0 = blockIdx.x * kBlockTasks;
  for (int k = 0; k < kBlockTasks && t0 + k < ntask; ++k) {
    const bool ok = src.valid(t0 + k);
    for (int i = threadIdx.x; i < nc; i += kTaskBlock)
      out[(int64_t)(t0 + k) * nc + i] = ok ? tab[k * nc + i] : __builtin_nan("");
  }
}

// LDS of a table kernel: the block's tables and the recurrence's coefficients.
template <int MAXN>
struct TableLds {
  static constexpr int kNc = (MAXN + 1) * (MAXN + 2) / 2;
  double tab[kBlockTasks * kNc], ca[kNc], cb[kNc];
};

// Tasks from a list (a plan's), or one component at device points: a point with
// rho < 0, z <= 0 or a non-finite value is computed at a harmless place (rho = 0,
// z = 1, so the quadrature stays bounded) and NaN written over its outputs.
struct TaskList {
  const CompInfo* comps;
  const SommTask* tasks;
  __device__ SommTask task(int t) const { return tasks[t]; }
  __device__ CompInfo comp(const SommTask& tk) const { return comps[tk.comp]; }
  __device__ bool valid(int) const { return true; }
};
struct PointList {
  CompInfo c;
  double S;
  const double *rho, *z;
  __device__ bool valid(int t) const {
    return (rho[t] >= 0.0) && (z[t] > 0.0) && isfinite(rho[t]) && isfinite(z[t]);
  }
  __device__ SommTask task(int t) const {
    return valid(t) ? SommTask{0, S, rho[t], z[t]} : SommTask{0, S, 0.0, 1.0};
  }
  __device__ CompInfo comp(const SommTask&) const { return c; }
};

// One group per task: initial values, then eq. recurrence for M >= 2.
template <int MAXN, bool QUAD, class Src>
__global__ __launch_bounds__(kTaskBlock) void sommerfeld_table_kernel(Medium md, Src src, int ntask, int nmax,
                                                                      double* __restrict__ out) {
  __shared__ TableLds<MAXN> lds;
  const int lane = threadIdx.x % kTaskLanes, slot = threadIdx.x / kTaskLanes;
  const int t = blockIdx.x * kBlockTasks + slot;
  recurrence_coefs(nmax, lds.ca, lds.cb);
  double* o = lds.tab + slot * ncoef(nmax);
  double s_rho = 0.0;
  if (t < ntask) {
    const SommTask tk = src.task(t);
    const CompInfo c = src.comp(tk);
    double a0[MAXN + 1], a1[MAXN + 1];
    initial_share<MAXN, QUAD>(md, c, tk.S, tk.rho, tk.z, nmax, lane, a0, a1);
    group_put<MAXN>(nmax, lane, a0, a1, [&](int n, double v0, double v1) {
      o[cidx(n, 0)] = v0;
      if (n >= 1) o[cidx(n, 1)] = v1;
    });
    s_rho = tk.rho > 0.0 ? tk.S / tk.rho : 0.0;
  }
  recurrence_store(src, ntask, nmax, s_rho, lane, o, lds.ca, lds.cb, lds.tab, out);
}

// I_00 of a pair without the leading term and the 1/(4 pi), for the lanes with
// `need` set (every lane of the wave calls): each lane sums its component's
// images, or, where there is no series, the wave's groups take the lanes'
// quadratures in turn, four at a time.
template <bool QUAD = true>
__device__ double pair_remainder(const Medium& md, const CompInfo& c, double rho, double zeta, bool need) {
  double v = 0.0;
  if (need && c.nimg > 0) {
    double amp = c.img1, Z = zeta + c.zinf;
    const double r2 = rho * rho;
    for (int j = 0; j < c.nimg; ++j) {
      Z += c.imgd;
      v += amp * rsqrt(r2 + Z * Z);
      amp *= c.imgq;
    }
  }
  if (!QUAD) return v;
  unsigned long long todo = __ballot(need && c.nimg < 0);
  const int wl = threadIdx.x & 63, lane = wl % kTaskLanes, group = wl / kTaskLanes;
  while (todo) {
    int mine = -1;  // the wave lane whose pair this group takes
    for (int g = 0; g < 64 / kTaskLanes && todo; ++g) {
      const int b = __ffsll(todo) - 1;
      if (g == group) mine = b;
      todo &= todo - 1;
    }
    const int from = mine < 0 ? wl : mine;
    CompInfo cc;
    cc.lt = __shfl(c.lt, from);
    cc.ls = __shfl(c.ls, from);
    cc.a = __shfl(c.a, from);
    cc.b = __shfl(c.b, from);
    cc.zinf = __shfl(c.zinf, from);
    cc.sinf = __shfl(c.sinf, from);
    const double rr = __shfl(rho, from), zz = __shfl(zeta, from);
    double a0[1] = {0.0}, a1[1] = {0.0};
    if (mine >= 0) quadrature_share<0>(md, cc, 1.0, rr, zz, 0, lane, a0, a1);
    const double sum = group_sum(a0[0]);
    for (int g = 0; g < 64 / kTaskLanes; ++g) {
      const int to = __shfl(mine, g * kTaskLanes);
      const double sg = __shfl(sum, g * kTaskLanes);
      if (to == wl) v = sg;
    }
  }
  return v;
}

// the leading term's image in I_00
__device__ inline double pair_leading(const CompInfo& c, double rho, double zeta) {
  const double Z = zeta + c.zinf;
  return c.sinf / sqrt(rho * rho + Z * Z);
}

// Reaction near-field kernels, one lane a pair (whole waves: see pair_remainder).
// With a series of images a pair is one rsqrt and three multiply-adds an image,
// bound by the FP64 units: 12.1 M pairs of 34 images take 0.26 ms (by the
// quadrature, one thread a pair, 774 ms).
template <bool QUAD>
__global__ __launch_bounds__(256) void nearfield_kernel(Medium md, const CompInfo* __restrict__ comps,
                                                        const int32_t* __restrict__ tpt,
                                                        const int32_t* __restrict__ spt,
                                                        const int32_t* __restrict__ cmp, int64_t npairs,
                                                        const double* __restrict__ px, const double* __restrict__ py,
                                                        const double* __restrict__ ph, double* __restrict__ val) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool in = i < npairs;
  const int64_t k = in ? i : npairs - 1;
  const int32_t a = tpt[k], b = spt[k];
  const double dx = px[a] - px[b], dy = py[a] - py[b];
  const double rho = sqrt(dx * dx + dy * dy);
  const double zeta = ph[a] + ph[b];
  const CompInfo c = comps[cmp[k]];
  const double v = pair_leading(c, rho, zeta) + pair_remainder<QUAD>(md, c, rho, zeta, in);
  if (in) val[i] = v * (1.0 / (4.0 * 3.14159265358979323846));
}

// ---------------------------------------------------------------- learned form
// The density's remainder sigma(k) e^{k zinf} - sinf is approximated first by a
// ladder of exponentials sum_j c_j e^{-k j delta} (j = 1..kLadder, delta = 2 dmin,
// fitted once per component), each rung integrating in closed form like the
// leading term, as an image at zeta + zinf + j delta.  The network learns what
// the ladder leaves.
//
// Counter-based generator (splitmix64 finaliser of seed, stream and counter).
__device__ inline uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ inline double rng_unit(uint64_t seed, uint64_t stream, uint64_t i) {
  const uint64_t z = mix64(seed ^ mix64(stream + 0x9E3779B97F4A7C15ull * (i + 1)));
  return (double)(z >> 11) * 0x1.0p-53;
}

// The lane's share of sign * sum_j c_j S^n P~_n^m / R_j^{n+1} (rungs at Z + j delta), added to a0, a1.
template <int MAXN>
__device__ inline void ladder_share(const double* __restrict__ c, double delta, double sign, double S, double rho,
                                    double Z, int nmax, int lane, double* a0, double* a1) {
  static_assert(kLadder < kTaskLanes, "one rung a lane, the leading term on the last");
  if (lane < kLadder) add_image<MAXN>(sign * c[lane], S, rho, Z + (lane + 1) * delta, nmax, a0, a1);
}

// Network inputs for one (component, rho, zeta): with Z2 = zeta + zinf + 2 dmin
// and R2 = |(rho, Z2)|, f = (2 rho/rho_max - 1, 2 zeta/zeta_max - 1,
// 2 Z2/R2 - 1, 4 dmin/R2 - 1).  Returns R2.
__device__ inline double surrogate_features(const SurrogateDomain& dm, double zinf, double rho,
                                            double zeta, float4* f) {
  const double Z2 = zeta + zinf + 2.0 * dm.dmin;
  const double R2 = sqrt(rho * rho + Z2 * Z2);
  f->x = (float)(2.0 * rho / dm.rho_max - 1.0);
  f->y = (float)(2.0 * zeta / dm.zeta_max - 1.0);
  f->z = (float)(2.0 * Z2 / R2 - 1.0);
  f->w = (float)(4.0 * dm.dmin / R2 - 1.0);
  return R2;
}

__device__ inline bool surrogate_in_domain(const SurrogateDomain& dm, double rho, double zeta) {
  return rho >= 0.0 && rho <= dm.rho_max && zeta > 0.0 && zeta <= dm.zeta_max;
}

// Training samples: component uniform; (rho, zeta) half uniform over the
// domain, half concentrated towards 0 (cubes of uniforms), where the
// reaction near field and the finest M2L levels sit.  Target of output j
// (degree n_j, order m_j: j <= nmax -> (j, 0), else (j - nmax, 1)) is what the
// leading term and the ladder leave of the initial value (S = 1), times
// kSurDecay^{n_j} R2^{n_j + 1} / yscale: the weights follow how fast an error
// of degree n fades in the M2L result (the scaled multipole moments of a box
// fall off like (0.87 S / R)^n, S <= R / 2).
__global__ __launch_bounds__(kTaskBlock) void surrogate_sample_kernel(
    Medium md, const CompInfo* __restrict__ comps, int ncomp, const double* __restrict__ lad, SurrogateDomain dm,
    int nmax, uint64_t seed, int64_t n, int32_t* __restrict__ comp_out, float4* __restrict__ feat,
    float* __restrict__ y, double* __restrict__ rz) {
  const int lane = threadIdx.x % kTaskLanes;
  const int64_t i = (int64_t)blockIdx.x * kBlockTasks + threadIdx.x / kTaskLanes;
  if (i >= n) return;
  int c = (int)(rng_unit(seed, 1, i) * ncomp);
  if (c >= ncomp) c = ncomp - 1;
  double u = rng_unit(seed, 2, i), v = rng_unit(seed, 3, i);
  if (rng_unit(seed, 4, i) < 0.5) {
    u = u * u * u;
    v = v * v * v;
  }
  const double rho = u * dm.rho_max;
  const double zeta = fmax(v, 1e-6) * dm.zeta_max;
  const CompInfo ci = comps[c];
  float4 f;
  const double R2 = surrogate_features(dm, ci.zinf, rho, zeta, &f);
  double a0[kMaxOrder + 1], a1[kMaxOrder + 1];
  initial_share<kMaxOrder>(md, ci, 1.0, rho, zeta, nmax, lane, a0, a1, false);
  ladder_share<kMaxOrder>(lad + (int64_t)c * kLadder, dm.delta, -1.0, 1.0, rho, zeta + ci.zinf, nmax, lane, a0, a1);
  const int nout = 2 * nmax + 1;
  float* yo = y + i * nout;
  group_put<kMaxOrder>(nmax, lane, a0, a1, [&](int nn, double v0, double v1) {
    const double pw = R2 / dm.yscale * pow(R2 * kSurDecay, (double)nn);  // kSurDecay^n R2^{n+1} / yscale
    yo[nn] = (float)(v0 * pw);
    if (nn >= 1) yo[nmax + nn] = (float)(v1 * pw);
  });
  if (lane) return;
  comp_out[i] = c;
  feat[i] = f;
  if (rz) {
    rz[2 * i] = rho;
    rz[2 * i + 1] = zeta;
  }
}

// Features of the plan's Sommerfeld tasks (rho, z of a task are unscaled).
__global__ void surrogate_task_features_kernel(const CompInfo* __restrict__ comps,
                                               const int32_t* __restrict__ smap, SurrogateDomain dm,
                                               const SommTask* __restrict__ tasks, int ntask,
                                               int32_t* __restrict__ comp_out, float4* __restrict__ feat) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ntask) return;
  const SommTask tk = tasks[t];
  float4 f;
  surrogate_features(dm, comps[tk.comp].zinf, tk.rho, tk.z, &f);
  comp_out[t] = smap[tk.comp];
  feat[t] = f;
}

// A task's table from a group of lanes: inside the learned form's domain the
// leading term and the ladder (lad: this component's rungs) in closed form plus
// the remainder S^n yscale rem(j) / (kSurDecay^n R2^{n+1}) for m = 0, 1, where
// rem(j) is output j in output units (j = n for m = 0, ynmax + n for m = 1);
// outside it as sommerfeld_table_kernel.  Writes o [cidx(n, 0)], [cidx(n, 1)].
template <int MAXN, class Rem>
__device__ void learned_task_values(const Medium& md, const CompInfo& c, bool in, const double* __restrict__ lad,
                                    const SurrogateDomain& dm, const SommTask& tk, int nmax, int ynmax, int lane,
                                    Rem rem, double* o) {
  double a0[MAXN + 1], a1[MAXN + 1];
  if (in) {
#pragma unroll
    for (int n = 0; n <= MAXN; ++n) a0[n] = a1[n] = 0.0;
    ladder_share<MAXN>(lad, dm.delta, 1.0, tk.S, tk.rho, tk.z + c.zinf, nmax, lane, a0, a1);
    if (lane == kTaskLanes - 1) add_image<MAXN>(c.sinf, tk.S, tk.rho, tk.z + c.zinf, nmax, a0, a1);
  } else {
    initial_share<MAXN>(md, c, tk.S, tk.rho, tk.z, nmax, lane, a0, a1);
  }
  group_put<MAXN>(nmax, lane, a0, a1, [&](int n, double v0, double v1) {
    o[cidx(n, 0)] = v0;
    if (n >= 1) o[cidx(n, 1)] = v1;
  });
  if (!in) return;
  const double Z2 = tk.z + c.zinf + 2.0 * dm.dmin;
  const double R2 = sqrt(tk.rho * tk.rho + Z2 * Z2);
  for (int n = lane; n <= nmax; n += kTaskLanes) {  // the lane that put entry n
    const double pw = dm.yscale / R2 * pow(tk.S / (R2 * kSurDecay), (double)n);
    o[cidx(n, 0)] += pw * rem(n);
    if (n >= 1 && tk.rho > 0.0) o[cidx(n, 1)] += pw * rem(ynmax + n);
  }
}

// The learned form's near-field value I_00 (S = 1) without the 1/(4 pi): the
// closed-form parts plus yscale rem0 / R2.
__device__ inline double learned_pair_value(const CompInfo& c, const double* __restrict__ lad,
                                            const SurrogateDomain& dm, double rho, double zeta, double rem0) {
  double v0 = pair_leading(c, rho, zeta);
  for (int j = 0; j < kLadder; ++j) {
    const double Z = zeta + c.zinf + (j + 1) * dm.delta;
    v0 += lad[j] / sqrt(rho * rho + Z * Z);
  }
  const double Z2 = zeta + c.zinf + 2.0 * dm.dmin;
  return v0 + dm.yscale * rem0 / sqrt(rho * rho + Z2 * Z2);
}

// S^n I_{n,m} for a task: the leading term and the ladder in closed form plus
// the network's remainder S^n yscale y_j / (kSurDecay^n R2^{n+1}) (FP32
// network, FP64 here) for m = 0, 1; as without the network when (rho, z) lies
// outside the trained domain; then eq. recurrence.
template <int MAXN>
__global__ __launch_bounds__(kTaskBlock) void surrogate_table_kernel(
    Medium md, TaskList src, const int32_t* __restrict__ scomp, const double* __restrict__ lad, SurrogateDomain dm,
    int ntask, int nmax, const float* __restrict__ y, int ldy, int ynmax, double* __restrict__ out,
    int32_t* __restrict__ used) {
  __shared__ TableLds<MAXN> lds;
  const int lane = threadIdx.x % kTaskLanes, slot = threadIdx.x / kTaskLanes;
  const int t = blockIdx.x * kBlockTasks + slot;
  recurrence_coefs(nmax, lds.ca, lds.cb);
  double* o = lds.tab + slot * ncoef(nmax);
  double s_rho = 0.0;
  if (t < ntask) {
    const SommTask tk = src.task(t);
    const bool net = surrogate_in_domain(dm, tk.rho, tk.z);
    const float* yy = y + (int64_t)t * ldy;
    learned_task_values<MAXN>(md, src.comp(tk), net, lad + (int64_t)scomp[t] * kLadder, dm, tk, nmax, ynmax, lane,
                              [&](int j) { return (double)yy[j]; }, o);
    s_rho = tk.rho > 0.0 ? tk.S / tk.rho : 0.0;
    if (used && lane == 0) used[t] = net ? 1 : 0;
  }
  recurrence_store(src, ntask, nmax, s_rho, lane, o, lds.ca, lds.cb, lds.tab, out);
}

// Reaction near field through the network: per pair (component, rho, zeta)
// and in-domain flag; out-of-domain pairs take the quadrature.
__global__ void surrogate_pair_features_kernel(const CompInfo* __restrict__ comps,
                                               const int32_t* __restrict__ smap, SurrogateDomain dm,
                                               const int32_t* __restrict__ tpt, const int32_t* __restrict__ spt,
                                               const int32_t* __restrict__ cmp, int64_t npairs,
                                               const double* __restrict__ px, const double* __restrict__ py,
                                               const double* __restrict__ ph, int32_t* __restrict__ comp_out,
                                               float4* __restrict__ feat) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= npairs) return;
  const int32_t a = tpt[i], b = spt[i];
  const double dx = px[a] - px[b], dy = py[a] - py[b];
  const double rho = sqrt(dx * dx + dy * dy);
  const double zeta = ph[a] + ph[b];
  float4 f;
  surrogate_features(dm, comps[cmp[i]].zinf, rho, zeta, &f);
  comp_out[i] = smap[cmp[i]];
  feat[i] = f;
}

__global__ void surrogate_nearfield_kernel(Medium md, const CompInfo* __restrict__ comps,
                                           const int32_t* __restrict__ scomp, const double* __restrict__ lad,
                                           SurrogateDomain dm, const int32_t* __restrict__ tpt,
                                           const int32_t* __restrict__ spt, const int32_t* __restrict__ cmp,
                                           int64_t npairs, const double* __restrict__ px,
                                           const double* __restrict__ py, const double* __restrict__ ph,
                                           const float* __restrict__ y, int ldy, double* __restrict__ val,
                                           unsigned long long* __restrict__ nfallback) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool have = i < npairs;
  const int64_t k = have ? i : npairs - 1;
  const int32_t a = tpt[k], b = spt[k];
  const double dx = px[a] - px[b], dy = py[a] - py[b];
  const double rho = sqrt(dx * dx + dy * dy);
  const double zeta = ph[a] + ph[b];
  const CompInfo c = comps[cmp[k]];
  const bool in = surrogate_in_domain(dm, rho, zeta);
  const double rem = pair_remainder(md, c, rho, zeta, have && !in);
  if (!have) return;
  double v0;
  if (in) {
    v0 = learned_pair_value(c, lad + (int64_t)scomp[i] * kLadder, dm, rho, zeta, (double)y[i * ldy]);
  } else {
    v0 = pair_leading(c, rho, zeta) + rem;
    atomicAdd(nfallback, 1ull);
  }
  val[i] = v0 * (1.0 / (4.0 * 3.14159265358979323846));
}

// ---------------------------------------------------------------- table form
// Pre-computed 2-D tables for the initial values (the Remark after Table 3.1):
// per component, the remainder the network would learn (what the leading term
// and the ladder leave, times kSurDecay^n R2^{n+1}, a smooth O(1) function of
// (rho, zeta)) is tabulated on a grid of npr x npz panels over the domain, at
// kTabK Chebyshev points of the first kind per panel and direction, and
// interpolated by the barycentric formula (tensor product, degree kTabK - 1 in
// rho and in zeta: exact on polynomials of that degree).  Layout: component,
// panel (pr * npz + pz), output j, node (a * kTabK + b; a in rho, b in zeta).
__constant__ double c_chx[kTabK];  // cos((2k + 1) pi / (2 kTabK))
__constant__ double c_chw[kTabK];  // barycentric weights (-1)^k sin((2k + 1) pi / (2 kTabK))

// Lagrange basis values l[k] at x in [-1, 1] (barycentric formula; exact at nodes)
__device__ inline void cheb_lagrange(double x, double* l) {
  int hit = -1;
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < kTabK; ++k) {
    const double dx = x - c_chx[k];
    if (dx == 0.0) hit = k;
    const double t = c_chw[k] / (dx == 0.0 ? 1.0 : dx);
    l[k] = t;
    s += t;
  }
  if (hit >= 0) {
#pragma unroll
    for (int k = 0; k < kTabK; ++k) l[k] = (k == hit) ? 1.0 : 0.0;
    return;
  }
  const double is = 1.0 / s;
#pragma unroll
  for (int k = 0; k < kTabK; ++k) l[k] *= is;
}

// panel of (rho, zeta) (clamped to the grid) and the basis values in both directions
__device__ inline int table_cell(const TableGrid& g, double rho, double zeta, double* lr, double* lz) {
  int pr = (int)(rho / g.hr), pz = (int)(zeta / g.hz);
  pr = pr < 0 ? 0 : (pr >= g.npr ? g.npr - 1 : pr);
  pz = pz < 0 ? 0 : (pz >= g.npz ? g.npz - 1 : pz);
  cheb_lagrange(2.0 * (rho - pr * g.hr) / g.hr - 1.0, lr);
  cheb_lagrange(2.0 * (zeta - pz * g.hz) / g.hz - 1.0, lz);
  return pr * g.npz + pz;
}

// output j of a panel block [nout][kTabK * kTabK]
__device__ inline double table_value(const double* __restrict__ blk, int j, const double* lr, const double* lz) {
  const double* f = blk + (int64_t)j * kTabK * kTabK;
  double acc = 0.0;
#pragma unroll
  for (int a = 0; a < kTabK; ++a) {
    double r = 0.0;
#pragma unroll
    for (int b = 0; b < kTabK; ++b) r += lz[b] * f[a * kTabK + b];
    acc += lr[a] * r;
  }
  return acc;
}

// One group per (component, panel, node): the remainder's scaled initial values
// (the same targets as the network's training samples).
__global__ __launch_bounds__(kTaskBlock) void table_fill_kernel(Medium md, const CompInfo* __restrict__ comps,
                                                                int ncomp, const double* __restrict__ lad,
                                                                SurrogateDomain dm, TableGrid g, int nmax,
                                                                double* __restrict__ tab) {
  constexpr int KK = kTabK * kTabK;
  const int64_t per = (int64_t)g.npr * g.npz * KK;
  const int lane = threadIdx.x % kTaskLanes;
  const int64_t i = (int64_t)blockIdx.x * kBlockTasks + threadIdx.x / kTaskLanes;
  if (i >= per * ncomp) return;
  const int c = (int)(i / per);
  const int64_t r = i % per;
  const int cell = (int)(r / KK), ab = (int)(r % KK);
  const int pr = cell / g.npz, pz = cell % g.npz, a = ab / kTabK, b = ab % kTabK;
  const double rho = (pr + 0.5 + 0.5 * c_chx[a]) * g.hr;
  const double zeta = (pz + 0.5 + 0.5 * c_chx[b]) * g.hz;
  const CompInfo ci = comps[c];
  double a0[kMaxOrder + 1], a1[kMaxOrder + 1];
  initial_share<kMaxOrder>(md, ci, 1.0, rho, zeta, nmax, lane, a0, a1, false);
  ladder_share<kMaxOrder>(lad + (int64_t)c * kLadder, dm.delta, -1.0, 1.0, rho, zeta + ci.zinf, nmax, lane, a0, a1);
  const double Z2 = zeta + ci.zinf + 2.0 * dm.dmin;
  const double R2 = sqrt(rho * rho + Z2 * Z2);
  const int nout = 2 * nmax + 1;
  double* blk = tab + ((int64_t)c * g.npr * g.npz + cell) * nout * KK;
  group_put<kMaxOrder>(nmax, lane, a0, a1, [&](int n, double v0, double v1) {
    const double pw = R2 / dm.yscale * pow(R2 * kSurDecay, (double)n);  // kSurDecay^n R2^{n+1} / yscale
    blk[(int64_t)n * KK + ab] = v0 * pw;
    if (n >= 1) blk[(int64_t)(nmax + n) * KK + ab] = v1 * pw;
  });
}

// S^n I_{n,m} of tasks through the tables (outside the domain as sommerfeld_table_kernel), then
// eq. recurrence.  The lanes of a task's group share its 4p + 1 interpolations.
template <int MAXN>
__global__ __launch_bounds__(kTaskBlock) void table_task_kernel(
    Medium md, TaskList src, const int32_t* __restrict__ smap, const double* __restrict__ lad, SurrogateDomain dm,
    TableGrid g, const double* __restrict__ tab, int ynmax, int ntask, int nmax, double* __restrict__ out,
    int32_t* __restrict__ used) {
  __shared__ TableLds<MAXN> lds;
  const int lane = threadIdx.x % kTaskLanes, slot = threadIdx.x / kTaskLanes;
  const int t = blockIdx.x * kBlockTasks + slot;
  recurrence_coefs(nmax, lds.ca, lds.cb);
  double* o = lds.tab + slot * ncoef(nmax);
  double s_rho = 0.0;
  if (t < ntask) {
    const SommTask tk = src.task(t);
    const bool in = surrogate_in_domain(dm, tk.rho, tk.z);
    const int sc = smap[tk.comp];
    double lr[kTabK], lz[kTabK];
    const int cell = table_cell(g, tk.rho, tk.z, lr, lz);
    const double* blk = tab + ((int64_t)sc * g.npr * g.npz + cell) * (2 * ynmax + 1) * kTabK * kTabK;
    learned_task_values<MAXN>(md, src.comp(tk), in, lad + (int64_t)sc * kLadder, dm, tk, nmax, ynmax, lane,
                              [&](int j) { return table_value(blk, j, lr, lz); }, o);
    s_rho = tk.rho > 0.0 ? tk.S / tk.rho : 0.0;
    if (used && lane == 0) used[t] = in ? 1 : 0;
  }
  recurrence_store(src, ntask, nmax, s_rho, lane, o, lds.ca, lds.cb, lds.tab, out);
}

// Reaction near field through the tables (output 0, I_00); quadrature outside the domain.
__global__ void table_nearfield_kernel(Medium md, const CompInfo* __restrict__ comps,
                                       const int32_t* __restrict__ smap, const double* __restrict__ lad,
                                       SurrogateDomain dm, TableGrid g, const double* __restrict__ tab, int nout,
                                       const int32_t* __restrict__ tpt, const int32_t* __restrict__ spt,
                                       const int32_t* __restrict__ cmp, int64_t npairs,
                                       const double* __restrict__ px, const double* __restrict__ py,
                                       const double* __restrict__ ph, double* __restrict__ val,
                                       unsigned long long* __restrict__ nfallback) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool have = i < npairs;
  const int64_t k = have ? i : npairs - 1;
  const int32_t a = tpt[k], b = spt[k];
  const double dx = px[a] - px[b], dy = py[a] - py[b];
  const double rho = sqrt(dx * dx + dy * dy);
  const double zeta = ph[a] + ph[b];
  const CompInfo c = comps[cmp[k]];
  const bool in = surrogate_in_domain(dm, rho, zeta);
  const double rem = pair_remainder(md, c, rho, zeta, have && !in);
  if (!have) return;
  double v0;
  if (in) {
    const int sc = smap[cmp[i]];
    double lr[kTabK], lz[kTabK];
    const int cell = table_cell(g, rho, zeta, lr, lz);
    const double* blk = tab + ((int64_t)sc * g.npr * g.npz + cell) * nout * kTabK * kTabK;
    v0 = learned_pair_value(c, lad + (int64_t)sc * kLadder, dm, rho, zeta, table_value(blk, 0, lr, lz));
  } else {
    v0 = pair_leading(c, rho, zeta) + rem;
    atomicAdd(nfallback, 1ull);
  }
  val[i] = v0 * (1.0 / (4.0 * 3.14159265358979323846));
}

// The interpolation alone on given node values (tests): out[i][j] for nout outputs.
__global__ void interp2d_kernel(TableGrid g, int nout, const double* __restrict__ nodes, int64_t n,
                                const double* __restrict__ rho, const double* __restrict__ zeta,
                                double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double lr[kTabK], lz[kTabK];
  const int cell = table_cell(g, rho[i], zeta[i], lr, lz);
  const double* blk = nodes + (int64_t)cell * nout * kTabK * kTabK;
  for (int j = 0; j < nout; ++j) out[i * nout + j] = table_value(blk, j, lr, lz);
}

__global__ void density_kernel(Medium md, CompInfo c, int64_t nk, const double* __restrict__ kre,
                               const double* __restrict__ kim, double* __restrict__ ore,
                               double* __restrict__ oim) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nk) return;
  Scatter sc;
  local_coeffs(md, sc);
  const cplx v = density(md, sc, c.lt, c.ls, c.a, c.b, cmk(kre[i], kim[i]));
  ore[i] = v.re;
  oim[i] = v.im;
}

// Gauss-Legendre nodes on [-1, 1] (Newton on the three-term recurrence), host side.
void gl_nodes(int n, double* x, double* w) {
  for (int i = 0; i < n; ++i) {
    double t = std::cos(M_PI * (i + 0.75) / (n + 0.5));
    for (int it = 0; it < 100; ++it) {
      double p0 = 1.0, p1 = t;
      for (int j = 2; j <= n; ++j) {
        const double p2 = ((2.0 * j - 1.0) * t * p1 - (j - 1.0) * p0) / j;
        p0 = p1;
        p1 = p2;
      }
      const double dp = n * (t * p1 - p0) / (t * t - 1.0);
      const double dt = p1 / dp;
      t -= dt;
      if (std::fabs(dt) < 1e-16) break;
    }
    double p0 = 1.0, p1 = t;
    for (int j = 2; j <= n; ++j) {
      const double p2 = ((2.0 * j - 1.0) * t * p1 - (j - 1.0) * p0) / j;
      p0 = p1;
      p1 = p2;
    }
    const double dp = n * (t * p1 - p0) / (t * t - 1.0);
    x[i] = t;
    w[i] = 2.0 / ((1.0 - t * t) * dp * dp);
  }
}

// The node table lives in constant memory, one copy per device: it is
// written once on each device the library runs on.
constexpr int kMaxDevices = 64;
int upload_gl(hipStream_t st) {
  static std::mutex mu;
  static bool done[kMaxDevices] = {};
  (void)st;
  int dev = 0;
  FMM_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return FMMLM_EDEVICE;
  std::lock_guard<std::mutex> lk(mu);
  if (done[dev]) return FMMLM_OK;
  double x[kGL], w[kGL];
  gl_nodes(kGL, x, w);
  FMM_HIP_TRY(hipMemcpyToSymbol(HIP_SYMBOL(c_glx), x, sizeof(x)));
  FMM_HIP_TRY(hipMemcpyToSymbol(HIP_SYMBOL(c_glw), w, sizeof(w)));
  double cx[kTabK], cw[kTabK];
  for (int k = 0; k < kTabK; ++k) {
    const double th = M_PI * (2.0 * k + 1.0) / (2.0 * kTabK);
    cx[k] = std::cos(th);
    cw[k] = ((k & 1) ? -1.0 : 1.0) * std::sin(th);
  }
  FMM_HIP_TRY(hipMemcpyToSymbol(HIP_SYMBOL(c_chx), cx, sizeof(cx)));
  FMM_HIP_TRY(hipMemcpyToSymbol(HIP_SYMBOL(c_chw), cw, sizeof(cw)));
  done[dev] = true;
  return FMMLM_OK;
}

// Runs f(std::integral_constant<int, MAXN>) for the smallest compiled order bound >= nmax.
template <class F>
void with_order_bound(int nmax, F f) {
  if (nmax <= 20) {
    f(std::integral_constant<int, 20>());
  } else {
    f(std::integral_constant<int, kMaxOrder>());
  }
}
unsigned task_blocks(int64_t ntask) { return (unsigned)((ntask + kBlockTasks - 1) / kBlockTasks); }

// no component needs the quadrature
bool all_series(const CompInfo* comps, size_t n) {
  return std::all_of(comps, comps + n, [](const CompInfo& c) { return c.nimg >= 0; });
}

template <class Src>
void launch_tables(const Medium& md, bool series, const Src& src, int ntask, int nmax, double* out, hipStream_t st) {
  with_order_bound(nmax, [&](auto bound) {
    constexpr int MAXN = decltype(bound)::value;
    if (series) {
      sommerfeld_table_kernel<MAXN, false><<<task_blocks(ntask), kTaskBlock, 0, st>>>(md, src, ntask, nmax, out);
    } else {
      sommerfeld_table_kernel<MAXN, true><<<task_blocks(ntask), kTaskBlock, 0, st>>>(md, src, ntask, nmax, out);
    }
  });
}

}  // namespace

// Shortest ray path from the source's exit interface to the target's entry
// interface: the density decays like exp(-k zinf) (eq. densityasymptotic).
double zeta_inf(const Medium& md, int lt, int ls, int a, int b) {
  if (md.L == 0) return 0.0;
  auto D = [&](int l) { return (l >= 1 && l <= md.L - 1) ? md.d[l - 1] - md.d[l] : 0.0; };
  if (lt == ls) return (a == b) ? 0.0 : D(lt);
  if (lt < ls) return (b == 1 ? D(ls) : 0.0) + (md.d[lt] - md.d[ls - 1]) + (a == 2 ? D(lt) : 0.0);
  return (b == 2 ? D(ls) : 0.0) + (md.d[ls] - md.d[lt - 1]) + (a == 1 ? D(lt) : 0.0);
}

// Amplitude of the leading term of the density: the product of the local
// reflection and transmission coefficients met along the shortest ray path of
// zeta_inf (every other path crosses some finite layer twice more, so
// sigma(k) e^{k zinf} - sinf = O(e^{-2 k dmin})).
static double sigma_inf_classic(const Medium& md, int lt, int ls, int a, int b) {
  auto rdn = [&](int i) { return (md.eps[i] - md.eps[i + 1]) / (md.eps[i] + md.eps[i + 1]); };
  auto rup = [&](int i) { return (md.eps[i + 1] - md.eps[i]) / (md.eps[i] + md.eps[i + 1]); };
  auto tdn = [&](int i) { return 2.0 * md.eps[i] / (md.eps[i] + md.eps[i + 1]); };
  auto tup = [&](int i) { return 2.0 * md.eps[i + 1] / (md.eps[i] + md.eps[i + 1]); };
  if (lt == ls) {
    if (a == b) return (b == 1) ? rdn(ls) : rup(ls - 1);
    return rdn(ls) * rup(ls - 1);
  }
  if (lt < ls) {
    double s = (b == 2) ? 1.0 : rdn(ls);  // b = 1: down to d_ls and back up first
    for (int i = ls - 1; i >= lt; --i) s *= tup(i);
    return (a == 1) ? s : rup(lt - 1) * s;
  }
  double s = (b == 1) ? 1.0 : rup(ls - 1);
  for (int i = ls + 1; i <= lt; ++i) s *= tdn(i - 1);
  return (a == 2) ? s : rdn(lt) * s;
}

double sigma_inf(const Medium& md, int lt, int ls, int a, int b) {
  if (md.L == 0) return 1.0;
  return (md.acoef[ls] / md.acoef[lt]) * sigma_inf_classic(md, lt, ls, a, b);
}

// With two interfaces the one finite layer (thickness D) reflects with
// q = rup_0 rdn_1 a round trip, and every density is its leading term plus a
// geometric series: sigma(k) = sinf e^{-k zinf} + sum_j img1 q^j e^{-k (zinf + 2 D (j + 1))}.
// In the two outer layers' own components the leading term is the reflection at
// the near interface, and the series starts with the wave that crosses into the
// finite layer and back; everywhere else it goes on from the leading term
// (img1 = sinf q).  Each term integrates in closed form as an image.  The series
// ends where what is left, |q|^n / (1 - |q|) of its first term, falls under
// 2^-56.  Up to kImagesMost terms it is taken instead of the quadrature, which
// stays for |q| closer to 1 and for other stacks.  Measured on tables of 10,007
// points, nmax 10 / 20 / 32: 34 terms 0.023 / 0.034 / 0.082 ms, 2,029 terms
// 0.22 / 0.28 / 0.74 ms, the quadrature of three interfaces 1.9 / 2.1 / 2.4 ms; the
// costs would meet at 7,000 to 20,000 terms, the limit stays well under that since
// a series' rounding grows with its length.
constexpr int kImagesMost = 2048;

CompInfo make_comp(const Medium& md, int lt, int ls, int a, int b) {
  CompInfo c{lt, ls, a, b, zeta_inf(md, lt, ls, a, b), sigma_inf(md, lt, ls, a, b), 0.0, 0.0, 0.0, 0};
  if (md.L < 2) return c;  // the leading term is the density
  c.nimg = -1;
  if (md.L > 2) return c;
  const double e0 = md.eps[0], e1 = md.eps[1], e2 = md.eps[2];
  const double rup0 = (e1 - e0) / (e1 + e0), rdn1 = (e1 - e2) / (e1 + e2);
  c.imgq = rup0 * rdn1;
  c.imgd = 2.0 * (md.d[0] - md.d[1]);
  if (lt == ls && lt == 0) {  // (each factor at most 2: products of permittivities overflow from 1e154 on)
    c.img1 = (2.0 * e0 / (e0 + e1)) * (2.0 * e1 / (e0 + e1)) * rdn1;
  } else if (lt == ls && lt == 2) {
    c.img1 = (2.0 * e1 / (e1 + e2)) * (2.0 * e2 / (e1 + e2)) * rup0;
  } else {
    c.img1 = c.sinf * c.imgq;
  }
  const double aq = std::fabs(c.imgq);
  const double n = aq > 0.0 ? std::ceil(std::log(0x1.0p-56 * (1.0 - aq)) / std::log(aq)) : 0.0;
  if (!(aq < 1.0)) return c;  // the terms do not decay (|q| rounds to 1: contrasts from 1e16 on at both interfaces)
  if (c.img1 == 0.0) {
    c.nimg = 0;
  } else if (n + 1.0 <= kImagesMost) {
    c.nimg = (int)std::max(n, 0.0) + 1;
  }
  return c;
}

int gpu_sommerfeld_tables(const Medium& md, const std::vector<CompInfo>& comps,
                          const std::vector<SommTask>& tasks, int nmax, double* d_out,
                          hipStream_t st) {
  if (tasks.empty()) return FMMLM_OK;
  int rc = upload_gl(st);
  if (rc) return rc;
  CompInfo* dc = nullptr;
  SommTask* dt = nullptr;
  FMM_HIP_TRY(hipMalloc(&dc, comps.size() * sizeof(CompInfo)));
  FMM_HIP_TRY(hipMalloc(&dt, tasks.size() * sizeof(SommTask)));
  FMM_HIP_TRY(hipMemcpyAsync(dc, comps.data(), comps.size() * sizeof(CompInfo), hipMemcpyHostToDevice, st));
  FMM_HIP_TRY(hipMemcpyAsync(dt, tasks.data(), tasks.size() * sizeof(SommTask), hipMemcpyHostToDevice, st));
  const int nt = (int)tasks.size();
  launch_tables(md, all_series(comps.data(), comps.size()), TaskList{dc, dt}, nt, nmax, d_out, st);
  FMM_HIP_TRY(hipGetLastError());
  FMM_HIP_TRY(hipStreamSynchronize(st));
  hipFree(dc);
  hipFree(dt);
  return FMMLM_OK;
}

int gpu_reaction_nearfield(const Medium& md, const std::vector<CompInfo>& comps,
                           const int32_t* d_tpt, const int32_t* d_spt, const int32_t* d_comp,
                           int64_t npairs, const double* px, const double* py, const double* ph,
                           double* d_val, hipStream_t st) {
  if (npairs == 0) return FMMLM_OK;
  int rc = upload_gl(st);
  if (rc) return rc;
  CompInfo* dc = nullptr;
  FMM_HIP_TRY(hipMalloc(&dc, comps.size() * sizeof(CompInfo)));
  FMM_HIP_TRY(hipMemcpyAsync(dc, comps.data(), comps.size() * sizeof(CompInfo), hipMemcpyHostToDevice, st));
  const unsigned nb = (unsigned)((npairs + 255) / 256);
  if (all_series(comps.data(), comps.size())) {
    nearfield_kernel<false><<<nb, 256, 0, st>>>(md, dc, d_tpt, d_spt, d_comp, npairs, px, py, ph, d_val);
  } else {
    nearfield_kernel<true><<<nb, 256, 0, st>>>(md, dc, d_tpt, d_spt, d_comp, npairs, px, py, ph, d_val);
  }
  FMM_HIP_TRY(hipGetLastError());
  FMM_HIP_TRY(hipStreamSynchronize(st));
  hipFree(dc);
  return FMMLM_OK;
}

int gpu_density(const Medium& md, const CompInfo& c, int64_t nk, const double* kre,
                const double* kim, double* ore, double* oim, hipStream_t st) {
  double* buf = nullptr;
  FMM_HIP_TRY(hipMalloc(&buf, 4 * nk * sizeof(double)));
  FMM_HIP_TRY(hipMemcpyAsync(buf, kre, nk * 8, hipMemcpyHostToDevice, st));
  FMM_HIP_TRY(hipMemcpyAsync(buf + nk, kim, nk * 8, hipMemcpyHostToDevice, st));
  density_kernel<<<(unsigned)((nk + 63) / 64), 64, 0, st>>>(md, c, nk, buf, buf + nk, buf + 2 * nk,
                                                            buf + 3 * nk);
  FMM_HIP_TRY(hipGetLastError());
  FMM_HIP_TRY(hipMemcpyAsync(ore, buf + 2 * nk, nk * 8, hipMemcpyDeviceToHost, st));
  FMM_HIP_TRY(hipMemcpyAsync(oim, buf + 3 * nk, nk * 8, hipMemcpyDeviceToHost, st));
  FMM_HIP_TRY(hipStreamSynchronize(st));
  hipFree(buf);
  return FMMLM_OK;
}

int gpu_surrogate_samples(const Medium& md, const std::vector<CompInfo>& comps, const double* d_lad,
                          const SurrogateDomain& dm, int nmax, uint64_t seed, int64_t n, int32_t* d_comp,
                          float* d_feat, float* d_y, hipStream_t st, double* d_rz) {
  if (n == 0) return FMMLM_OK;
  int rc = upload_gl(st);
  if (rc) return rc;
  CompInfo* dc = nullptr;
  FMM_HIP_TRY(hipMalloc(&dc, comps.size() * sizeof(CompInfo)));
  FMM_HIP_TRY(hipMemcpyAsync(dc, comps.data(), comps.size() * sizeof(CompInfo), hipMemcpyHostToDevice, st));
  surrogate_sample_kernel<<<task_blocks(n), kTaskBlock, 0, st>>>(
      md, dc, (int)comps.size(), d_lad, dm, nmax, seed, n, d_comp, reinterpret_cast<float4*>(d_feat), d_y, d_rz);
  FMM_HIP_TRY(hipGetLastError());
  FMM_HIP_TRY(hipStreamSynchronize(st));
  hipFree(dc);
  return FMMLM_OK;
}

int gpu_surrogate_tables(const Medium& md, const std::vector<CompInfo>& comps,
                         const std::vector<int32_t>& smap, const double* d_lad, const SurrogateDomain& dm,
                         const std::vector<SommTask>& tasks, int nmax, const MlpNet& net, double* d_out,
                         int64_t* n_used, hipStream_t st, int32_t* h_used) {
  *n_used = 0;
  if (tasks.empty()) return FMMLM_OK;
  int rc = upload_gl(st);
  if (rc) return rc;
  const int nt = (int)tasks.size();
  const int ynmax = (net.nout - 1) / 2;
  CompInfo* dc = nullptr;
  SommTask* dt = nullptr;
  int32_t *dmap = nullptr, *dcomp = nullptr, *dused = nullptr;
  float *dfeat = nullptr, *dy = nullptr;
  FMM_HIP_TRY(hipMalloc(&dc, comps.size() * sizeof(CompInfo)));
  FMM_HIP_TRY(hipMalloc(&dt, tasks.size() * sizeof(SommTask)));
  FMM_HIP_TRY(hipMalloc(&dmap, smap.size() * sizeof(int32_t)));
  FMM_HIP_TRY(hipMalloc(&dcomp, nt * sizeof(int32_t)));
  FMM_HIP_TRY(hipMalloc(&dused, nt * sizeof(int32_t)));
  FMM_HIP_TRY(hipMalloc(&dfeat, (size_t)nt * 4 * sizeof(float)));
  FMM_HIP_TRY(hipMalloc(&dy, (size_t)nt * net.nout * sizeof(float)));
  FMM_HIP_TRY(hipMemcpyAsync(dc, comps.data(), comps.size() * sizeof(CompInfo), hipMemcpyHostToDevice, st));
  FMM_HIP_TRY(hipMemcpyAsync(dt, tasks.data(), tasks.size() * sizeof(SommTask), hipMemcpyHostToDevice, st));
  FMM_HIP_TRY(hipMemcpyAsync(dmap, smap.data(), smap.size() * sizeof(int32_t), hipMemcpyHostToDevice, st));
  surrogate_task_features_kernel<<<(nt + 63) / 64, 64, 0, st>>>(dc, dmap, dm, dt, nt, dcomp,
                                                                reinterpret_cast<float4*>(dfeat));
  FMM_HIP_TRY(hipGetLastError());
  rc = gpu_mlp_forward(net, dcomp, dfeat, nt, dy, net.nout, net.nout, nullptr, nullptr, nullptr, st);
  if (rc == FMMLM_OK) {
    with_order_bound(nmax, [&](auto bound) {
      surrogate_table_kernel<decltype(bound)::value><<<task_blocks(nt), kTaskBlock, 0, st>>>(
          md, TaskList{dc, dt}, dcomp, d_lad, dm, nt, nmax, dy, net.nout, ynmax, d_out, dused);
    });
    FMM_HIP_TRY(hipGetLastError());
    std::vector<int32_t> used(nt);
    FMM_HIP_TRY(hipMemcpyAsync(used.data(), dused, nt * sizeof(int32_t), hipMemcpyDeviceToHost, st));
    FMM_HIP_TRY(hipStreamSynchronize(st));
    for (int32_t u : used) *n_used += u;
    if (h_used) std::copy(used.begin(), used.end(), h_used);
  }
  hipFree(dc);
  hipFree(dt);
  hipFree(dmap);
  hipFree(dcomp);
  hipFree(dused);
  hipFree(dfeat);
  hipFree(dy);
  return rc;
}

int gpu_surrogate_nearfield(const Medium& md, const std::vector<CompInfo>& comps,
                            const std::vector<int32_t>& smap, const double* d_lad, const SurrogateDomain& dm,
                            const int32_t* d_tpt, const int32_t* d_spt, const int32_t* d_comp,
                            int64_t npairs, const double* px, const double* py, const double* ph,
                            const MlpNet& net, double* d_val, int64_t* n_fallback, hipStream_t st) {
  *n_fallback = 0;
  if (npairs == 0) return FMMLM_OK;
  int rc = upload_gl(st);
  if (rc) return rc;
  constexpr int64_t kChunk = (int64_t)1 << 22;
  const int64_t cap = std::min(npairs, kChunk);
  CompInfo* dc = nullptr;
  int32_t *dmap = nullptr, *dcomp = nullptr;
  float *dfeat = nullptr, *dy = nullptr;
  unsigned long long* dfb = nullptr;
  FMM_HIP_TRY(hipMalloc(&dc, comps.size() * sizeof(CompInfo)));
  FMM_HIP_TRY(hipMalloc(&dmap, smap.size() * sizeof(int32_t)));
  FMM_HIP_TRY(hipMalloc(&dcomp, cap * sizeof(int32_t)));
  FMM_HIP_TRY(hipMalloc(&dfeat, cap * 4 * sizeof(float)));
  FMM_HIP_TRY(hipMalloc(&dy, cap * sizeof(float)));
  FMM_HIP_TRY(hipMalloc(&dfb, sizeof(unsigned long long)));
  FMM_HIP_TRY(hipMemcpyAsync(dc, comps.data(), comps.size() * sizeof(CompInfo), hipMemcpyHostToDevice, st));
  FMM_HIP_TRY(hipMemcpyAsync(dmap, smap.data(), smap.size() * sizeof(int32_t), hipMemcpyHostToDevice, st));
  FMM_HIP_TRY(hipMemsetAsync(dfb, 0, sizeof(unsigned long long), st));
  for (int64_t o = 0; o < npairs && rc == FMMLM_OK; o += kChunk) {
    const int64_t m = std::min(kChunk, npairs - o);
    const unsigned nb = (unsigned)((m + 255) / 256);
    surrogate_pair_features_kernel<<<nb, 256, 0, st>>>(dc, dmap, dm, d_tpt + o, d_spt + o, d_comp + o, m,
                                                       px, py, ph, dcomp, reinterpret_cast<float4*>(dfeat));
    FMM_HIP_TRY(hipGetLastError());
    rc = gpu_mlp_forward(net, dcomp, dfeat, m, dy, 1, 1, nullptr, nullptr, nullptr, st);
    if (rc) break;
    surrogate_nearfield_kernel<<<nb, 256, 0, st>>>(md, dc, dcomp, d_lad, dm, d_tpt + o, d_spt + o, d_comp + o, m,
                                                   px, py, ph, dy, 1, d_val + o, dfb);
    FMM_HIP_TRY(hipGetLastError());
  }
  unsigned long long fb = 0;
  if (rc == FMMLM_OK) {
    FMM_HIP_TRY(hipMemcpyAsync(&fb, dfb, sizeof(fb), hipMemcpyDeviceToHost, st));
    FMM_HIP_TRY(hipStreamSynchronize(st));
  }
  *n_fallback = (int64_t)fb;
  hipFree(dc);
  hipFree(dmap);
  hipFree(dcomp);
  hipFree(dfeat);
  hipFree(dy);
  hipFree(dfb);
  return rc;
}

// ---- table form (host side)
int gpu_table_fill(const Medium& md, const std::vector<CompInfo>& comps, const double* d_lad,
                   const SurrogateDomain& dm, const TableGrid& g, int nmax, double* d_tab, hipStream_t st) {
  int rc = upload_gl(st);
  if (rc) return rc;
  CompInfo* dc = nullptr;
  FMM_HIP_TRY(hipMalloc(&dc, comps.size() * sizeof(CompInfo)));
  FMM_HIP_TRY(hipMemcpyAsync(dc, comps.data(), comps.size() * sizeof(CompInfo), hipMemcpyHostToDevice, st));
  const int64_t n = (int64_t)comps.size() * g.npr * g.npz * kTabK * kTabK;
  table_fill_kernel<<<task_blocks(n), kTaskBlock, 0, st>>>(md, dc, (int)comps.size(), d_lad, dm, g, nmax, d_tab);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  hipFree(dc);
  if (e != hipSuccess) {
    set_last_error(std::string("table fill: ") + hipGetErrorString(e));
    return FMMLM_EDEVICE;
  }
  return FMMLM_OK;
}

int gpu_table_tasks(const Medium& md, const std::vector<CompInfo>& comps, const std::vector<int32_t>& smap,
                    const double* d_lad, const SurrogateDomain& dm, const TableGrid& g, const double* d_tab,
                    int ynmax, const std::vector<SommTask>& tasks, int nmax, double* d_out, int64_t* n_used,
                    hipStream_t st, int32_t* h_used) {
  *n_used = 0;
  if (tasks.empty()) return FMMLM_OK;
  int rc = upload_gl(st);
  if (rc) return rc;
  const int nt = (int)tasks.size();
  CompInfo* dc = nullptr;
  SommTask* dt = nullptr;
  int32_t *dmap = nullptr, *dused = nullptr;
  hipError_t e = hipMalloc(&dc, comps.size() * sizeof(CompInfo));
  if (e == hipSuccess) e = hipMalloc(&dt, tasks.size() * sizeof(SommTask));
  if (e == hipSuccess) e = hipMalloc(&dmap, smap.size() * sizeof(int32_t));
  if (e == hipSuccess) e = hipMalloc(&dused, nt * sizeof(int32_t));
  if (e == hipSuccess)
    e = hipMemcpyAsync(dc, comps.data(), comps.size() * sizeof(CompInfo), hipMemcpyHostToDevice, st);
  if (e == hipSuccess)
    e = hipMemcpyAsync(dt, tasks.data(), tasks.size() * sizeof(SommTask), hipMemcpyHostToDevice, st);
  if (e == hipSuccess)
    e = hipMemcpyAsync(dmap, smap.data(), smap.size() * sizeof(int32_t), hipMemcpyHostToDevice, st);
  std::vector<int32_t> used(nt);
  if (e == hipSuccess) {
    with_order_bound(nmax, [&](auto bound) {
      table_task_kernel<decltype(bound)::value><<<task_blocks(nt), kTaskBlock, 0, st>>>(
          md, TaskList{dc, dt}, dmap, d_lad, dm, g, d_tab, ynmax, nt, nmax, d_out, dused);
    });
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(used.data(), dused, nt * sizeof(int32_t), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  hipFree(dc);
  hipFree(dt);
  hipFree(dmap);
  hipFree(dused);
  if (e != hipSuccess) {
    set_last_error(std::string("table tasks: ") + hipGetErrorString(e));
    return FMMLM_EDEVICE;
  }
  for (int32_t u : used) *n_used += u;
  if (h_used) std::copy(used.begin(), used.end(), h_used);
  return FMMLM_OK;
}

int gpu_table_nearfield(const Medium& md, const std::vector<CompInfo>& comps, const std::vector<int32_t>& smap,
                        const double* d_lad, const SurrogateDomain& dm, const TableGrid& g, const double* d_tab,
                        int nout, const int32_t* d_tpt, const int32_t* d_spt, const int32_t* d_comp, int64_t npairs,
                        const double* px, const double* py, const double* ph, double* d_val, int64_t* n_fallback,
                        hipStream_t st) {
  *n_fallback = 0;
  if (npairs == 0) return FMMLM_OK;
  int rc = upload_gl(st);
  if (rc) return rc;
  CompInfo* dc = nullptr;
  int32_t* dmap = nullptr;
  unsigned long long* dfb = nullptr;
  hipError_t e = hipMalloc(&dc, comps.size() * sizeof(CompInfo));
  if (e == hipSuccess) e = hipMalloc(&dmap, smap.size() * sizeof(int32_t));
  if (e == hipSuccess) e = hipMalloc(&dfb, sizeof(unsigned long long));
  if (e == hipSuccess)
    e = hipMemcpyAsync(dc, comps.data(), comps.size() * sizeof(CompInfo), hipMemcpyHostToDevice, st);
  if (e == hipSuccess)
    e = hipMemcpyAsync(dmap, smap.data(), smap.size() * sizeof(int32_t), hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipMemsetAsync(dfb, 0, sizeof(unsigned long long), st);
  unsigned long long fb = 0;
  if (e == hipSuccess) {
    table_nearfield_kernel<<<(unsigned)((npairs + 255) / 256), 256, 0, st>>>(
        md, dc, dmap, d_lad, dm, g, d_tab, nout, d_tpt, d_spt, d_comp, npairs, px, py, ph, d_val, dfb);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(&fb, dfb, sizeof(fb), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  hipFree(dc);
  hipFree(dmap);
  hipFree(dfb);
  if (e != hipSuccess) {
    set_last_error(std::string("table near field: ") + hipGetErrorString(e));
    return FMMLM_EDEVICE;
  }
  *n_fallback = (int64_t)fb;
  return FMMLM_OK;
}

int gpu_interp2d(const TableGrid& g, int nout, const double* d_nodes, int64_t n, const double* d_rho,
                 const double* d_zeta, double* d_out, hipStream_t st) {
  int rc = upload_gl(st);
  if (rc) return rc;
  interp2d_kernel<<<(unsigned)((n + 63) / 64), 64, 0, st>>>(g, nout, d_nodes, n, d_rho, d_zeta, d_out);
  FMM_HIP_TRY(hipGetLastError());
  return FMMLM_OK;
}

// S^N I_{N,M} for device arrays rho, z of npts points into out (device),
// asynchronous on st, with no allocation.  npts <= FMMLM_NOALLOC_MAX_POINTS
// (checked by the caller).
int gpu_sommerfeld_noalloc(const Medium& md, const CompInfo& c, double S, int64_t npts, const double* rho,
                           const double* z, int nmax, double* out, hipStream_t st) {
  if (npts < 1 || npts > FMMLM_NOALLOC_MAX_POINTS) return FMMLM_EINVAL;
  int rc = upload_gl(st);
  if (rc) return rc;
  launch_tables(md, all_series(&c, 1), PointList{c, S, rho, z}, (int)npts, nmax, out, st);
  FMM_HIP_TRY(hipGetLastError());
  return FMMLM_OK;
}

}  // namespace fmmlm
