// FP64 evaluation kernels of the layered-media FMM (Algorithm 1 / Algorithm 2
// of Sec. 3.3, with every reaction component folded into interface-anchored
// trees).
//
// Expansions are stored for m >= 0 only (real charges give X_{n,-m} =
// (-1)^m conj(X_{n,m})), scaled by the box size S as in Sec. 3.4:
//   M~_nm = M_nm / S^n,  L~_nm = L_nm S^n.
// Regular and irregular solid harmonics R_n^m = r^n Y_n^m, I_n^m = Y_n^m /
// r^{n+1} use the normalised Y of eq. sphericalharmonics (no Condon-Shortley
// phase in Y) and are generated by the standard three-term recurrences.
//
//   P2M  eq. freespaceexpcoef        M~_nm = sum_j q_j c_n^-2 conj(R_n^m((r_j - c)/S))
//   M2M  eq. metome                  child -> parent
//   M2L  eq. metole (c_n^2 reading) and eqs. metoleimage1/coefintable:
//        L~_nm += (1/S) (-1)^{n+m} A_n^m / c_n^2
//                 sum_{n',m'} G_{n+n'}^{m'-m} A_{n'}^{m'} s_{n'm'} M~_{n'm'}
//        with G = I_j^k(offset) / (4 pi A_j^k) for the free space and
//        G = S c_j e^{ik phi} S^j I_{jk} / (4 pi A_j^k) for a reaction component;
//        s = (-1)^{n'+m'} mirrors a polarization-source expansion across the
//        interface (Y_n^m(pi - theta, phi) = (-1)^{n+m} Y_n^m).
//   L2L  eq. letole                  parent -> child
//   L2P  eq. lefreespace             Phi += Re sum L~_nm R_n^m((r - c)/S)
//   P2P  eq. freereactioncomponents  near field, free space and reaction
#include <hip/hip_runtime.h>

#include <cmath>
#include <vector>

#include "fmm_internal.h"

namespace fmmlm {
namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr double kInv4Pi = 1.0 / (4.0 * kPi);

// Wave priority of the far-field chain (P2M, M2M, M2L, its reduction, L2L,
// L2P, combine).  An unprofiled evaluation runs the near field beside the
// chain on another stream; the chain is what the evaluation waits on, so its
// waves issue first on a shared SIMD and the near field fills the gaps.
__device__ __forceinline__ void far_chain_priority() { __builtin_amdgcn_s_setprio(2); }

__device__ inline double sgn1(int k) { return (k & 1) ? -1.0 : 1.0; }

// FP64 1/sqrt(r2): hardware estimate y (relative error about 2^-24) and one
// third-order step: with e = 1 - r2 y^2, y (1 - e)^{-1/2} = y (1 + e/2 + 3 e^2/8 + ..),
// what is left is 5/16 e^3, below 2^-68.  Five operations, where two Newton
// steps take eight.
__device__ inline double rsqrt_nr(double r2) {
  const double y = __builtin_amdgcn_rsq(r2);
  const double e = fma(-(r2 * y), y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// R_n^m(x, y, z) for one (n, m), m >= 0, by the diagonal then the n recurrence.
__device__ inline cplx regular_nm(int n, int m, double x, double y, double z) {
  cplx R = cmk(0.28209479177387814, 0.0);  // 1/sqrt(4 pi)
  const cplx w = cmk(x, y);
  for (int mm = 1; mm <= m; ++mm) R = sqrt((2.0 * mm + 1.0) / (2.0 * mm)) * (w * R);
  if (n == m) return R;
  const double r2 = x * x + y * y + z * z;
  cplx Rm2 = R;
  cplx Rm1 = (sqrt(2.0 * m + 3.0) * z) * R;
  for (int nn = m + 2; nn <= n; ++nn) {
    const double a = sqrt((4.0 * nn * nn - 1.0) / ((double)nn * nn - (double)m * m));
    const double b = sqrt(((double)(nn - 1) * (nn - 1) - (double)m * m) / (4.0 * (nn - 1) * (nn - 1) - 1.0));
    const cplx Rn = a * (z * Rm1 - (b * r2) * Rm2);
    Rm2 = Rm1;
    Rm1 = Rn;
  }
  return Rm1;
}

// I_n^m(x, y, z) = Y_n^m / r^{n+1} for one (n, m), m >= 0.
__device__ inline cplx irregular_nm(int n, int m, double x, double y, double z) {
  const double r2 = x * x + y * y + z * z;
  const double ir2 = 1.0 / r2;
  cplx I = cmk(0.28209479177387814 / sqrt(r2), 0.0);
  const cplx w = cmk(x * ir2, y * ir2);
  for (int mm = 1; mm <= m; ++mm) I = sqrt((2.0 * mm + 1.0) / (2.0 * mm)) * (w * I);
  if (n == m) return I;
  cplx Im2 = I;
  cplx Im1 = (sqrt(2.0 * m + 3.0) * z * ir2) * I;
  for (int nn = m + 2; nn <= n; ++nn) {
    const double a = sqrt((4.0 * nn * nn - 1.0) / ((double)nn * nn - (double)m * m));
    const double b = sqrt(((double)(nn - 1) * (nn - 1) - (double)m * m) / (4.0 * (nn - 1) * (nn - 1) - 1.0));
    const cplx In = a * ((z * ir2) * Im1 - (b * ir2) * Im2);
    Im2 = Im1;
    Im1 = In;
  }
  return Im1;
}

// value of a stored m >= 0 array at any m: X_{n,-m} = (-1)^m conj(X_{n,m})
__device__ inline cplx full_at(const cplx* X, int n, int m) {
  if (m >= 0) return X[cidx(n, m)];
  const cplx v = X[cidx(n, -m)];
  return ((-m) & 1) ? cmk(-v.re, v.im) : cmk(v.re, -v.im);
}

// Real layout of an expansion with real sources: (p+1)^2 doubles per box,
// row n holds Re X_n0, then (Re X_nm, Im X_nm) for m = 1..n.
__device__ inline cplx rload(const double* X, int n, int m) {
  return m ? cmk(X[n * n + 2 * m - 1], X[n * n + 2 * m]) : cmk(X[n * n], 0.0);
}
__device__ inline void rstore(double* X, int n, int m, cplx v) {
  if (m) {
    X[n * n + 2 * m - 1] = v.re;
    X[n * n + 2 * m] = v.im;
  } else {
    X[n * n] = v.re;
  }
}
// real-layout index -> (n, m, imaginary part?)
__device__ inline void rsplit(int idx, int* n, int* m, bool* im) {
  int nn = (int)sqrt((double)idx);
  while (nn * nn > idx) --nn;
  while ((nn + 1) * (nn + 1) <= idx) ++nn;
  const int r = idx - nn * nn;
  *n = nn;
  *m = (r + 1) / 2;
  *im = (r > 0) && ((r & 1) == 0);
}

__device__ inline int isqrt_row(int t) {
  // n with n(n+1)/2 <= t < (n+1)(n+2)/2
  int n = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
  while (cidx(n + 1, 0) <= t) ++n;
  while (cidx(n, 0) > t) --n;
  return n;
}

// ---------------------------------------------------------------- operators
// An operator's table in the frame turned so that its offset has azimuth 0: the
// real g(j, k) = G(j, k) e^{-i k phi} of eqs. metole, metoleimage1 for
// -j <= k <= j (g(j, -k) = (-1)^k g(j, k)) at [j j + j + k], j <= 2p.
__device__ inline void g_index(int i, int* j, int* k) {
  int r = (int)sqrt((double)i);
  while (r * r > i) --r;
  while ((r + 1) * (r + 1) <= i) ++r;
  *j = r;
  *k = i - r * r - r;
}

// free operators: r2dz [nops][2]
__global__ void build_free_ops_kernel(const int* __restrict__ r2dz, int64_t nops, int ngs,
                                      const double* __restrict__ coefA, double* __restrict__ G) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nops * ngs) return;
  const int64_t op = t / ngs;
  const int c = (int)(t % ngs);
  int j, k;
  g_index(c, &j, &k);
  const int ak = abs(k);
  const double g =
      (kInv4Pi / coefA[cidx(j, ak)]) * irregular_nm(j, ak, sqrt((double)r2dz[2 * op]), 0.0, r2dz[2 * op + 1]).re;
  G[t] = k < 0 ? g * sgn1(k) : g;
}

// reaction operators: one per Sommerfeld task
__global__ void build_reaction_ops_kernel(const double* __restrict__ Sl, int64_t nops, int ng, int ngs,
                                          const double* __restrict__ coefA, const double* __restrict__ tables,
                                          double* __restrict__ G) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nops * ngs) return;
  const int64_t op = t / ngs;
  const int c = (int)(t % ngs);
  int j, k;
  g_index(c, &j, &k);
  const int ak = abs(k);
  const double SI = tables[op * ng + cidx(j, ak)];
  const double cj = sqrt((2.0 * j + 1.0) / (4.0 * kPi));
  const double g = Sl[op] * cj * SI * kInv4Pi / coefA[cidx(j, ak)];
  G[t] = k < 0 ? g * sgn1(k) : g;
}

// e^{i k phi}, k <= p2, of the directions (dx, dy)
__global__ void build_phases_kernel(const int* __restrict__ dirs, int64_t n, int p2, cplx* __restrict__ E) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * (p2 + 1)) return;
  const int64_t f = t / (p2 + 1);
  const int k = (int)(t % (p2 + 1));
  double s, c;
  sincos(k * atan2((double)dirs[2 * f + 1], (double)dirs[2 * f]), &s, &c);
  E[t] = cmk(c, s);
}

// ---------------------------------------------------------------- eval kernels
__global__ void gather_kernel(const double* __restrict__ q, const int32_t* __restrict__ puser,
                              int64_t np, double* __restrict__ qt, float* __restrict__ qt32) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= np) return;
  const double v = q[puser[i]];
  qt[i] = v;
  if (qt32) qt32[i] = (float)v;
}

// phi (user order) = far field + near field at the (one or two) tree positions of each point.
__global__ void combine_kernel(const double* __restrict__ phit, const double* __restrict__ phin,
                               const int32_t* __restrict__ upos, int64_t n, double* __restrict__ phi) {
  far_chain_priority();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t a = upos[2 * i], b = upos[2 * i + 1];
  double v = 0.0;
  if (a >= 0) v += phit[a] + phin[a];
  if (b >= 0) v += phit[b] + phin[b];
  phi[i] = v;
}

// Batched P2M: one block per leaf.  Chunks of 32 points: the block computes
// each point's regular solid harmonics (eq. freespaceexpcoef: c_n^{-2} conj
// R_n^m, real layout, n <= p) into LDS, then lanes (one per charge vector)
// and waves (rows r = wave + 4 i) accumulate sum_j w[j][r] q[j][v] in FP64.
constexpr int kP2MBPts = 32;
constexpr int kP2MBRows = 32;  // rows per thread: (p+1)^2 <= 4 * 32
__global__ void __launch_bounds__(256)
p2m_batch_kernel(int p, int g, const int32_t* __restrict__ leaves, const int32_t* __restrict__ bstart,
                 const int32_t* __restrict__ bcount, const int32_t* __restrict__ blevel,
                 const double* __restrict__ bcx, const double* __restrict__ bcy, const double* __restrict__ bch,
                 const double* __restrict__ sc, const double* __restrict__ px, const double* __restrict__ py,
                 const double* __restrict__ ph, const double* __restrict__ qb, const double* __restrict__ coefR,
                 double* __restrict__ M, int64_t slab) {
  extern __shared__ double sm[];
  const int np1 = p + 1, nr = np1 * np1;
  double* w = sm;                          // [kP2MBPts][nr]
  double* qs = sm + kP2MBPts * nr;         // [kP2MBPts][64]
  const int b = leaves[blockIdx.x];
  const double inv = sc[blevel[b]];
  const double cx = bcx[b], cy = bcy[b], ch = bch[b];
  const int s0 = bstart[b], cnt = bcount[b];
  const int tid = threadIdx.x, v = tid & 63, wave = tid >> 6;
  const int ncp = ncoef(p);
  double acc[kP2MBRows];
#pragma unroll
  for (int i = 0; i < kP2MBRows; ++i) acc[i] = 0.0;
  for (int c0 = 0; c0 < cnt; c0 += kP2MBPts) {
    const int nc_ = min(kP2MBPts, cnt - c0);
    __syncthreads();  // the previous chunk is consumed
    for (int i = tid; i < kP2MBPts * 64; i += blockDim.x) {
      const int j = i >> 6, r = i & 63;
      qs[i] = (j < nc_ && r < g) ? qb[(int64_t)(s0 + c0 + j) * 64 + r] : 0.0;
    }
    for (int i = tid; i < kP2MBPts * np1; i += blockDim.x) {
      const int j = i / np1, m = i % np1;
      double* wj = w + j * nr;
      if (j >= nc_) {
        for (int n = m; n <= p; ++n) {
          if (m == 0) {
            wj[n * n] = 0.0;
          } else {
            wj[n * n + 2 * m - 1] = 0.0;
            wj[n * n + 2 * m] = 0.0;
          }
        }
        continue;
      }
      const int gp = s0 + c0 + j;
      const double x = (px[gp] - cx) * inv, y = (py[gp] - cy) * inv, z = (ph[gp] - ch) * inv;
      const double r2 = x * x + y * y + z * z;
      double dg = 0.28209479177387814;
      double wr = 1.0, wi = 0.0;  // (x + iy)^m
      for (int mm = 1; mm <= m; ++mm) {
        dg *= coefR[2 * ncp + mm];
        const double tr = wr * x - wi * y;
        wi = wr * y + wi * x;
        wr = tr;
      }
      cplx Rm2 = cmk(dg * wr, dg * wi), Rm1 = cmk(0.0, 0.0);
      for (int n = m; n <= p; ++n) {
        cplx Rn;
        if (n == m) {
          Rn = Rm2;
        } else if (n == m + 1) {
          Rn = (coefR[2 * ncp + np1 + m] * z) * Rm2;
        } else {
          Rn = coefR[cidx(n, m)] * (z * Rm1 - (coefR[ncp + cidx(n, m)] * r2) * Rm2);
        }
        if (n >= m + 2) {
          Rm2 = Rm1;
        }
        if (n >= m + 1) Rm1 = Rn;
        const double c2inv = 4.0 * kPi / (2.0 * n + 1.0);
        if (m == 0) {
          wj[n * n] = c2inv * Rn.re;
        } else {
          wj[n * n + 2 * m - 1] = c2inv * Rn.re;
          wj[n * n + 2 * m] = -c2inv * Rn.im;
        }
      }
    }
    __syncthreads();
    for (int j = 0; j < nc_; ++j) {
      const double qv = qs[j * 64 + v];
      const double* wj = w + j * nr;
#pragma unroll
      for (int i = 0; i < kP2MBRows; ++i) {
        const int r = wave + 4 * i;
        if (r < nr) acc[i] = fma(wj[r], qv, acc[i]);
      }
    }
  }
  if (v < g) {
#pragma unroll
    for (int i = 0; i < kP2MBRows; ++i) {
      const int r = wave + 4 * i;
      if (r < nr) M[(int64_t)v * slab + (int64_t)b * nr + r] = acc[i];
    }
  }
}

// P2M: thread (leaf, m) streams the recurrence for R_n^m, n = m..p, over the
// leaf's particles; its accumulators live in the thread's own LDS slice.
constexpr int kP2MThreads = 128;
__global__ void __launch_bounds__(kP2MThreads)
p2m_kernel(int p, int64_t nleaves, const int32_t* __restrict__ leaves,
           const int32_t* __restrict__ bstart, const int32_t* __restrict__ bcount,
           const int32_t* __restrict__ blevel, const double* __restrict__ bcx,
           const double* __restrict__ bcy, const double* __restrict__ bch,
           const double* __restrict__ sc, const double* __restrict__ px,
           const double* __restrict__ py, const double* __restrict__ ph,
           const double* __restrict__ qt, const double* __restrict__ coefR, double* __restrict__ M,
           int64_t qstride = 0, int64_t mstride = 0) {
  far_chain_priority();
  extern __shared__ double sacc[];  // [kP2MThreads][2 (p+1)]
  qt += blockIdx.y * qstride;       // vector blockIdx.y of a batched pass
  M += blockIdx.y * mstride;
  const int np1 = p + 1;
  const int lpb = kP2MThreads / np1;
  const int t = threadIdx.x;
  const int64_t lf = (int64_t)blockIdx.x * lpb + t / np1;
  const int m = t % np1;
  if (t >= lpb * np1 || lf >= nleaves) return;
  double* acc = sacc + (size_t)t * 2 * np1;
  for (int n = 0; n < 2 * np1; ++n) acc[n] = 0.0;
  const int b = leaves[lf];
  const double inv = sc[blevel[b]];
  const double cx = bcx[b], cy = bcy[b], ch = bch[b];
  const int s0 = bstart[b], cnt = bcount[b];
  const int ncp = ncoef(p);
  const double* ra = coefR;        // [cidx(n, m)]
  const double* rb = coefR + ncp;  // [cidx(n, m)]
  double dg = 1.0;  // prod_{mm <= m} sqrt((2mm+1)/(2mm))
  for (int mm = 1; mm <= m; ++mm) dg *= coefR[2 * ncp + mm];
  dg *= 0.28209479177387814;
  const double s23 = coefR[2 * ncp + np1 + m];  // sqrt(2m+3)
  for (int j = 0; j < cnt; ++j) {
    const int g = s0 + j;
    const double x = (px[g] - cx) * inv, y = (py[g] - cy) * inv, z = (ph[g] - ch) * inv;
    const double r2 = x * x + y * y + z * z;
    // (x + iy)^m
    double wr = 1.0, wi = 0.0;
    for (int mm = 0; mm < m; ++mm) {
      const double tr = wr * x - wi * y;
      wi = wr * y + wi * x;
      wr = tr;
    }
    const double q = qt[g];
    cplx Rm2 = cmk(dg * wr, dg * wi);
    acc[2 * m] += q * Rm2.re;
    acc[2 * m + 1] -= q * Rm2.im;
    if (m + 1 > p) continue;
    cplx Rm1 = (s23 * z) * Rm2;
    acc[2 * (m + 1)] += q * Rm1.re;
    acc[2 * (m + 1) + 1] -= q * Rm1.im;
    for (int n = m + 2; n <= p; ++n) {
      const double a = ra[cidx(n, m)], bb = rb[cidx(n, m)];
      const cplx Rn = a * (z * Rm1 - (bb * r2) * Rm2);
      acc[2 * n] += q * Rn.re;
      acc[2 * n + 1] -= q * Rn.im;
      Rm2 = Rm1;
      Rm1 = Rn;
    }
  }
  double* Mb = M + (int64_t)b * np1 * np1;
  for (int n = m; n <= p; ++n) {
    const double c2inv = 4.0 * kPi / (2.0 * n + 1.0);
    rstore(Mb, n, m, cmk(acc[2 * n] * c2inv, acc[2 * n + 1] * c2inv));
  }
}

// P2M, one wave per leaf, order P fixed at compile time.  The lanes take the
// leaf's particles in turn and accumulate, in registers, the charge times
// c_n^{-2} conj R_n^m (eq. freespaceexpcoef, scaled form) for one group of
// orders m at a time, a group holding at most 64 real-layout terms.  A
// recursive-halving reduce-scatter over the wave then leaves term k of the
// group, summed over the leaf, in lane k, which stores it.
constexpr int kP2MWWaves = 4;  // leaves (waves) per block
constexpr int kP2MGroup = 48;   // terms per group (<= 64): about 160 VGPRs, 3 waves per SIMD
constexpr int p2m_terms(int P, int m) { return (P + 1 - m) * (m ? 2 : 1); }
// first order of group G (consecutive orders, at most 64 terms a group); P + 1
// past the last group
constexpr int p2m_group_m0(int P, int G) {
  int g = 0, cnt = 0;
  for (int m = 0; m <= P; ++m) {
    if (cnt + p2m_terms(P, m) > kP2MGroup) {
      ++g;
      cnt = 0;
    }
    if (g == G && cnt == 0) return m;
    cnt += p2m_terms(P, m);
  }
  return P + 1;
}
// position of term (n = m, m) within the group that starts at order M0
constexpr int p2m_koff(int P, int M0, int m) {
  int k = 0;
  for (int mm = M0; mm < m; ++mm) k += p2m_terms(P, mm);
  return k;
}

template <int P, int M0, int M1>
__device__ __forceinline__ void p2m_wave_group(int lane, int s0, int cnt, double inv, double cx, double cy,
                                               double ch, const double* __restrict__ px,
                                               const double* __restrict__ py, const double* __restrict__ ph,
                                               const double* __restrict__ qt, const double* __restrict__ coefR,
                                               double* __restrict__ Mb) {
  constexpr int ncp = (P + 1) * (P + 2) / 2;
  const double* ra = coefR;        // [cidx(n, m)]
  const double* rb = coefR + ncp;  // [cidx(n, m)]
  // R_m^m = dg_m (x + iy)^m with dg_m = Y_0^0 prod_{mm <= m} sqrt((2mm+1)/(2mm))
  double dg[M1 - M0];
  {
    double d = 0.28209479177387814;
#pragma unroll
    for (int mm = 1; mm <= M0; ++mm) d *= coefR[2 * ncp + mm];
    dg[0] = d;
#pragma unroll
    for (int m = M0 + 1; m < M1; ++m) {
      d *= coefR[2 * ncp + m];
      dg[m - M0] = d;
    }
  }
  double acc[kP2MGroup];
#pragma unroll
  for (int k = 0; k < kP2MGroup; ++k) acc[k] = 0.0;
  for (int j = lane; j < cnt; j += 64) {
    const int g = s0 + j;
    const double x = (px[g] - cx) * inv, y = (py[g] - cy) * inv, z = (ph[g] - ch) * inv;
    const double r2 = x * x + y * y + z * z;
    const double q = qt[g];
    double wr = 1.0, wi = 0.0;  // (x + iy)^m
#pragma unroll
    for (int mm = 0; mm < M0; ++mm) {
      const double tr = wr * x - wi * y;
      wi = wr * y + wi * x;
      wr = tr;
    }
#pragma unroll
    for (int m = M0; m < M1; ++m) {
      const int st = m ? 2 : 1;
      int k = p2m_koff(P, M0, m);
      cplx Rm2 = cmk(dg[m - M0] * wr, dg[m - M0] * wi);
      acc[k] += q * Rm2.re;
      if (m) acc[k + 1] -= q * Rm2.im;
      k += st;
      if (m + 1 <= P) {
        cplx Rm1 = (coefR[2 * ncp + (P + 1) + m] * z) * Rm2;  // sqrt(2m+3) z R_m^m
        acc[k] += q * Rm1.re;
        if (m) acc[k + 1] -= q * Rm1.im;
        k += st;
#pragma unroll
        for (int n = m + 2; n <= P; ++n) {
          const double a = ra[cidx(n, m)], bb = rb[cidx(n, m)];
          const cplx Rn = a * (z * Rm1 - (bb * r2) * Rm2);
          acc[k] += q * Rn.re;
          if (m) acc[k + 1] -= q * Rn.im;
          k += st;
          Rm2 = Rm1;
          Rm1 = Rn;
        }
      }
      if (m + 1 < M1) {
        const double tr = wr * x - wi * y;
        wi = wr * y + wi * x;
        wr = tr;
      }
    }
  }
  // reduce-scatter: after the step over lane bit h a lane keeps the half of its
  // terms selected by that bit (terms past the group are zero), summed with its
  // partner's copy of that half; lane k ends with term k
#pragma unroll
  for (int h = 32; h >= 1; h >>= 1) {
    const bool up = (lane & h) != 0;
#pragma unroll
    for (int i = 0; i < h && i < kP2MGroup; ++i) {
      const double lo = acc[i];
      const double hi = (i + h < kP2MGroup) ? acc[i + h] : 0.0;
      const double keep = up ? hi : lo;
      const double send = up ? lo : hi;
      acc[i] = keep + __shfl_xor(send, h);
    }
  }
  constexpr int K = p2m_koff(P, M0, M1);
  if (lane < K) {
    int k = lane, m = M0;
    while (k >= p2m_terms(P, m)) k -= p2m_terms(P, m++);
    const int n = m + (m ? k / 2 : k);
    const int row = n * n + (m ? 2 * m - 1 + (k & 1) : 0);
    Mb[row] = acc[0] * (4.0 * kPi / (2.0 * n + 1.0));
  }
}

template <int P, int G>
__device__ __forceinline__ void p2m_wave_groups(int lane, int s0, int cnt, double inv, double cx, double cy,
                                                double ch, const double* __restrict__ px,
                                                const double* __restrict__ py, const double* __restrict__ ph,
                                                const double* __restrict__ qt, const double* __restrict__ coefR,
                                                double* __restrict__ Mb) {
  constexpr int m0 = p2m_group_m0(P, G), m1 = p2m_group_m0(P, G + 1);
  if constexpr (m0 <= P) {
    p2m_wave_group<P, m0, m1>(lane, s0, cnt, inv, cx, cy, ch, px, py, ph, qt, coefR, Mb);
    p2m_wave_groups<P, G + 1>(lane, s0, cnt, inv, cx, cy, ch, px, py, ph, qt, coefR, Mb);
  }
}

template <int P>
__global__ void __launch_bounds__(64 * kP2MWWaves)
p2m_wave_kernel(int64_t nleaves, const int32_t* __restrict__ leaves, const int32_t* __restrict__ bstart,
                const int32_t* __restrict__ bcount, const int32_t* __restrict__ blevel,
                const double* __restrict__ bcx, const double* __restrict__ bcy, const double* __restrict__ bch,
                const double* __restrict__ sc, const double* __restrict__ px, const double* __restrict__ py,
                const double* __restrict__ ph, const double* __restrict__ qt, const double* __restrict__ coefR,
                double* __restrict__ M) {
  far_chain_priority();
  const int lane = threadIdx.x & 63;
  const int64_t lf = (int64_t)blockIdx.x * kP2MWWaves + (threadIdx.x >> 6);
  if (lf >= nleaves) return;  // whole waves
  const int b = leaves[lf];
  p2m_wave_groups<P, 0>(lane, bstart[b], bcount[b], sc[blevel[b]], bcx[b], bcy[b], bch[b], px, py, ph, qt,
                        coefR, M + (int64_t)b * (P + 1) * (P + 1));
}

// Coefficient (n, m) of the parent's multipole expansion from one child
// (eq. metome, scaled form): Rv = R_n^m of the child centre relative to the
// parent centre in parent box units, Mc = the child's expansion (m >= 0).
// M_nm = sum_{n'<=n} sum_{m'} (-1)^{|m|-|m-m'|} A_{n'}^{m'} A_{n-n'}^{m-m'}
//        R_{n'}^{-m'} / (c_{n'}^2 A_n^m) 2^{-(n-n')} M^c_{n-n', m-m'}
__device__ inline cplx m2m_coef(int n, int m, const cplx* Rv, const cplx* Mc, const double* __restrict__ coefA) {
  double re = 0.0, im = 0.0;
  for (int n2 = 0; n2 <= n; ++n2) {
    const double c2inv = 4.0 * kPi / (2.0 * n2 + 1.0);
    const double sc2 = ldexp(1.0, -(n - n2));
    for (int m2 = -n2; m2 <= n2; ++m2) {
      const int mr = m - m2;
      if (mr > n - n2 || mr < -(n - n2)) continue;
      const double f = sgn1(abs(m) - abs(mr)) * coefA[cidx(n2, abs(m2))] * coefA[cidx(n - n2, abs(mr))] *
                       c2inv * sc2 / coefA[cidx(n, m)];
      const cplx v = full_at(Rv, n2, -m2) * full_at(Mc, n - n2, mr);
      re += f * v.re;
      im += f * v.im;
    }
  }
  return cmk(re, im);
}

// Coefficient (n, m) of a child's local expansion from its parent's
// (eq. letole, scaled form): Rv = R_n^m of the parent centre relative to the
// child centre in parent box units, Lp = the parent's local expansion.
__device__ inline cplx l2l_coef(int p, int n, int m, const cplx* Rv, const cplx* Lp,
                                const double* __restrict__ coefA) {
  double re = 0.0, im = 0.0;
  const double cn2inv = 4.0 * kPi / (2.0 * n + 1.0);
  const double s2 = ldexp(1.0, -n);
  for (int n2 = n; n2 <= p; ++n2) {
    const double cn2p = (2.0 * n2 + 1.0) / (4.0 * kPi);
    const double cdinv = 4.0 * kPi / (2.0 * (n2 - n) + 1.0);
    for (int m2 = -n2; m2 <= n2; ++m2) {
      const int md = m2 - m;
      if (md > n2 - n || md < -(n2 - n)) continue;
      const double f = sgn1(n2 - n - abs(md) + abs(m2) - abs(m)) * cn2p * coefA[cidx(n2 - n, abs(md))] *
                       coefA[cidx(n, m)] * cdinv * cn2inv * s2 / coefA[cidx(n2, abs(m2))];
      const cplx v = full_at(Rv, n2 - n, md) * full_at(Lp, n2, m2);
      re += f * v.re;
      im += f * v.im;
    }
  }
  return cmk(re, im);
}

// Real-form translation operators in parent box units, one per child octant o
// (bit 0: x, bit 1: y, bit 2: h; a set bit puts the child on the + side, at
// +1/4): ops 0..7 move a child's multipole expansion to its parent
// (eq. metome), ops 8..15 a parent's local expansion to its child
// (eq. letole).  Column k of an operator is its image of the k-th real-layout
// unit vector; T[op][k][row], rows padded to mr, k to nrk (zeros).
__global__ void build_xlate_ops_kernel(int p, int nrk, int mr, const double* __restrict__ coefA,
                                       double* __restrict__ T) {
  extern __shared__ char smem[];
  const int nc = ncoef(p), nr = (p + 1) * (p + 1);
  cplx* Rv = reinterpret_cast<cplx*>(smem);  // [nc]
  cplx* X = Rv + nc;                          // [nc] the unit input
  const int op = blockIdx.y, k = blockIdx.x;
  const int o = op & 7;
  const bool up = op < 8;
  const double sgn = up ? 1.0 : -1.0;  // child - parent for M2M, parent - child for L2L
  const double dx = sgn * ((o & 1) ? 0.25 : -0.25), dy = sgn * ((o & 2) ? 0.25 : -0.25),
               dz = sgn * ((o & 4) ? 0.25 : -0.25);
  int n2, m2;
  bool im2;
  rsplit(k, &n2, &m2, &im2);
  for (int t = threadIdx.x; t < nc; t += blockDim.x) {
    const int nn = isqrt_row(t), mm = t - cidx(nn, 0);
    Rv[t] = regular_nm(nn, mm, dx, dy, dz);
    X[t] = (nn == n2 && mm == m2) ? (im2 ? cmk(0.0, 1.0) : cmk(1.0, 0.0)) : cmk(0.0, 0.0);
  }
  __syncthreads();
  double* Tk = T + ((int64_t)op * nrk + k) * mr;
  for (int t = threadIdx.x; t < nc; t += blockDim.x) {
    const int n = isqrt_row(t), m = t - cidx(n, 0);
    const cplx v = up ? m2m_coef(n, m, Rv, X, coefA) : l2l_coef(p, n, m, Rv, X, coefA);
    if (m == 0) {
      Tk[n * n] = v.re;
    } else {
      Tk[n * n + 2 * m - 1] = v.re;
      Tk[n * n + 2 * m] = v.im;
    }
  }
  (void)nr;
}


// M2L in operator frames, on the matrix cores, in FP64 or FP32.  In the frame
// turned to an operator's azimuth its table g is real, so with
//   a + i b = e^{i m' phi} M_{n'm'}   and   L_nm = e^{-i m phi} (c + i s)
// the real parts c come from the a by one matrix and the imaginary parts s from
// the b by another (m' >= 1):
//   c:  f [g(n+n', m'-m) + (-1)^m g(n+n', m'+m)]   (m' = 0: the first term only),
//   s:  f [g(n+n', m'-m) - (-1)^m g(n+n', m'+m)],
// half the multiply-adds of the real form of G, and one operator serves every
// azimuth: 24,840 pairs of the top levels have 2,812 operators, 330 frames.
// Pairs (n, m) are taken orders m >= 1 first (pair_dec), so the s matrix is over
// the first ns of the nc pairs.  build_frame_ops_kernel folds in every constant of
// eqs. metole, metoleimage1 and the mirror sign, into the matrices.
// Layout: column (pair of the source) by column, its RC 16-row blocks of c, then
// its RS of s; whole k-steps of four columns, zeros past nc.
__host__ __device__ constexpr int frame_ksteps(int n) { return (n + 3) / 4; }

template <class T>
__global__ void build_frame_ops_kernel(int p, int nc, int ns, int rc, int rt, int ksteps, int64_t nops, int64_t nfree,
                                       const int32_t* __restrict__ frame_op, const int32_t* __restrict__ dec,
                                       const double* __restrict__ G, int ngs, const double* __restrict__ coefA,
                                       T* __restrict__ A) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int per = 4 * ksteps * rt;
  if (t >= nops * per) return;
  const int64_t fo = frame_op[t / per];
  const int col = (int)(t % per) / rt, row = (int)(t % per) % rt;
  const bool c = row < 16 * rc;
  const int r = c ? row : row - 16 * rc;
  double v = 0.0;
  if (c ? (r < nc && col < nc) : (r < ns && col < ns)) {
    const int m = dec[r] >> 16, m2 = dec[col] >> 16;
    const int n = (int)sqrt((double)(dec[r] & 0xffff) + 0.5), n2 = (int)sqrt((double)(dec[col] & 0xffff) + 0.5);
    const double* Gj = G + fo * ngs + (n + n2) * (n + n2) + n + n2;
    v = Gj[m2 - m];
    if (m2 > 0) v += (c ? sgn1(m) : -sgn1(m)) * Gj[m2 + m];
    double f = sgn1(n + m) * coefA[cidx(n, m)] * (4.0 * kPi / (2.0 * n + 1.0)) * coefA[cidx(n2, m2)];
    if (fo >= nfree && ((n2 + m2) & 1)) f = -f;
    v *= f;
  }
  A[t] = (T)v;
}

typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
__device__ inline doublex4 mfma4(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline floatx4 mfma4(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
template <class T>
struct FrameTypes;
template <>
struct FrameTypes<double> {
  using Acc = doublex4;
  static __device__ int row(int lk, int v) { return lk + 4 * v; }  // result row of register v
};
template <>
struct FrameTypes<float> {
  using Acc = floatx4;
  static __device__ int row(int lk, int v) { return 4 * lk + v; }
};

// A block takes one unit (64 columns, up to kM2LGroupOps steps), each of its four
// waves 16 columns.  A k-step's operand fragment wants pair 4 k + l / 16 of column
// l % 16 on lane l, which that lane gathers (two values of its column's source,
// always FP64) and turns itself, so the operands need no LDS; the operator, which
// all waves read, goes through LDS in double-buffered batches of KB k-steps, one
// barrier each, loads of both a batch ahead.  Waves whose columns are empty only
// load.
// A kernel of dense real-form operators took, launch alone, at 2^20 charges,
// p = 10: FP64 1.30 ms, this one 0.77; 262,144 clustered charges, p = 12: 4.9
// and 2.44 ms; the top levels' own kernel (24,840 pairs) 0.106 and 0.054 ms.  Now
// bound by the matrix cores (busy 0.50 of the FP64 launch's time, 0.45 of the FP32
// one's, 0.43 ms) and the gathers' cache accesses (54 and 41 M requests to the L2,
// 0.72 of them hits); the top levels, 431 units, by latency (matrix cores 0.10
// busy).  Measured on the way: one unit of 16 columns a wave without LDS,
// operators through the vector cache: 1.67 ms (p = 10); phases read from memory
// instead of LDS: half again as many cache accesses; results stored straight
// from the fragments: 32-byte pieces.
typedef int intx4 __attribute__((ext_vector_type(4)));
constexpr int kFrCols = 64;
template <class T, int RC, int RS, int KB>
__global__ void __launch_bounds__(256, 2)
m2l_frame_kernel(int nr, int nc, int ns, int ne, int wr, const int32_t* __restrict__ step0,
                 const int32_t* __restrict__ kind, const int32_t* __restrict__ uphi,
                 const int32_t* __restrict__ step_op, const int32_t* __restrict__ step_src,
                 const int32_t* __restrict__ dec, unsigned parts, const T* __restrict__ A,
                 const double* __restrict__ M, const cplx* __restrict__ E, T* __restrict__ W) {
  far_chain_priority();
  constexpr int RT = 16 * (RC + RS);
  constexpr int KV = 4 * RT * (int)sizeof(T) / 16;     // 16-byte vectors of a k-step of the operator
  constexpr int PER = (KB * KV + 255) / 256;
  using Acc = typename FrameTypes<T>::Acc;
  extern __shared__ cplx Es[];  // [p + 1][64] phases of the columns
  __shared__ intx4 As[2][KB * KV];
  __shared__ int32_t ds[(kPMax + 1) * (kPMax + 2) / 2];
  const int64_t u = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), col = 16 * wave + li;
  const int s0 = step0[u], s1 = (parts & (unsigned)kind[u]) ? step0[u + 1] : s0;  // (off: zeros are stored)
  const int kc = frame_ksteps(nc), ks = frame_ksteps(ns);
  for (int i = tid; i < nc; i += 256) ds[i] = dec[i];
  for (int i = tid; i < (nc - ns) * kFrCols; i += 256)
    Es[i] = E[(int64_t)uphi[u * kFrCols + i % kFrCols] * ne + i / kFrCols];
  // (a unit's columns in use come first)
  const bool work = step_src[(int64_t)step0[u] * kFrCols + 16 * wave] >= 0;
  Acc ac[RC], as[RS];
#pragma unroll
  for (int i = 0; i < RC; ++i) ac[i] = Acc{0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < RS; ++i) as[i] = Acc{0, 0, 0, 0};
  intx4 va[PER];
  auto load_a = [&](int s, int k0) {
    const intx4* Ap = reinterpret_cast<const intx4*>(A) + ((int64_t)step_op[s] * kc + k0) * KV;
    const int n = min(KB, kc - k0) * KV;
#pragma unroll
    for (int r = 0; r < PER; ++r)
      if (tid + 256 * r < n) va[r] = Ap[tid + 256 * r];
  };
  auto stash_a = [&](int buf) {
#pragma unroll
    for (int r = 0; r < PER; ++r)
      if (tid + 256 * r < KB * KV) As[buf][tid + 256 * r] = va[r];
  };
  struct __attribute__((packed, aligned(8))) Pair {
    double re, im;
  };
  Pair x[KB];
  int m[KB];
  auto load_b = [&](const double* Mj, int k0) {
#pragma unroll
    for (int t = 0; t < KB; ++t) {
      const int d = ds[min(4 * (k0 + t) + lk, nc - 1)];  // (columns from nc on are zero in A)
      x[t] = *reinterpret_cast<const Pair*>(Mj + (d & 0xffff));  // (order 0: im not used, the s columns are zero there)
      m[t] = d >> 16;
    }
  };
  auto source = [&](int s) { return step_src[(int64_t)s * kFrCols + col]; };
  __syncthreads();  // ds
  int src = -1, snext = -1;
  if (s0 < s1) {
    load_a(s0, 0);
    src = source(s0);
    if (work) load_b(M + (int64_t)max(src, 0) * nr, 0);
    stash_a(0);
  }
  __syncthreads();
  int buf = 0;
  for (int s = s0; s < s1; ++s) {
    if (s + 1 < s1) snext = source(s + 1);
    for (int k0 = 0; k0 < kc; k0 += KB) {
      const bool last = k0 + KB >= kc;
      const bool more = !last || s + 1 < s1;
      if (more) load_a(last ? s + 1 : s, last ? 0 : k0 + KB);
      if (work) {
        T a[KB], b[KB];
#pragma unroll
        for (int t = 0; t < KB; ++t) {
          const cplx v = Es[m[t] * kFrCols + col] * cmk(x[t].re, x[t].im);
          a[t] = src >= 0 ? (T)v.re : (T)0;
          b[t] = src >= 0 ? (T)v.im : (T)0;
        }
        if (more) load_b(M + (int64_t)max(last ? snext : src, 0) * nr, last ? 0 : k0 + KB);
        const T* Ab = reinterpret_cast<const T*>(As[buf]) + lk * RT + li;
#pragma unroll
        for (int t = 0; t < KB; ++t) {
          if (k0 + t >= kc) break;
#pragma unroll
          for (int i = 0; i < RC; ++i) ac[i] = mfma4(Ab[4 * t * RT + 16 * i], a[t], ac[i]);
          if (k0 + t < ks) {
#pragma unroll
            for (int i = 0; i < RS; ++i) as[i] = mfma4(Ab[4 * t * RT + 16 * (RC + i)], b[t], as[i]);
          }
        }
      }
      if (more) {
        stash_a(buf ^ 1);  // last read before the previous barrier
        __syncthreads();
        buf ^= 1;
      }
    }
    src = snext;
  }
  // out through LDS, PB row blocks at a time, so that each column's rows leave
  // contiguous (8-byte stores of four rows a column wrote 4.4 times the bytes)
  constexpr int PB0 = 2 * KB * KV * 16 / (1024 * (int)sizeof(T)), PB = PB0 < RC + RS ? PB0 : RC + RS;
  static_assert(PB >= 1, "a row block of every wave must fit the operator's buffers");
  T* o = reinterpret_cast<T*>(As) + wave * (256 * PB);  // [column][16 PB] of this wave
#pragma unroll
  for (int i0 = 0; i0 < RC + RS; i0 += PB) {
    __syncthreads();  // (the previous batch's, then the previous piece's readers are done)
#pragma unroll
    for (int i = i0; i < i0 + PB && i < RC + RS; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        o[li * 16 * PB + 16 * (i - i0) + FrameTypes<T>::row(lk, v)] = i < RC ? ac[i < RC ? i : 0][v] : as[i < RC ? 0 : i - RC][v];
    __syncthreads();
    if (!work) continue;
    T* w = W + (u * kFrCols + 16 * wave) * wr;
    for (int i = lane; i < 256 * PB; i += 64) {
      const int c = i / (16 * PB), r = 16 * i0 + i % (16 * PB);
      if (r < nc) {
        w[(int64_t)c * wr + r] = o[i];
      } else if (r >= 16 * RC && r < 16 * RC + ns) {
        w[(int64_t)c * wr + nc + r - 16 * RC] = o[i];
      }
    }
  }
}

// Each target box turns its slots' products back (e^{-i m phi}) and sums them in
// FP64 in a fixed order, scaled by 1/S of its level, into its local expansion.
// One block per target box: NT / nc groups of nc threads (one a pair)
// take every so many-th slot, four in flight, and the groups' sums are added in
// LDS in group order.  Bound by the latency of the slots' indirect rows and phases
// (waves wait 0.84 to 0.93 of their life): at 2^20 charges, p = 10, 0.295 GB in
// 0.12 ms (FP32) and 0.58 GB in 0.165 ms (FP64), 2.5 and 3.5 TB/s where a copy
// reaches 5.4.
template <class T, int NT>
__global__ void __launch_bounds__(NT)
m2l_frame_reduce_kernel(int nr, int nc, int ns, int ne, int wr, const int32_t* __restrict__ boxes,
                        const int32_t* __restrict__ sptr, const int32_t* __restrict__ slots,
                        const int32_t* __restrict__ sphi, const int32_t* __restrict__ dec,
                        const int32_t* __restrict__ blevel, const double* __restrict__ sc,
                        const T* __restrict__ W, const cplx* __restrict__ E, double* __restrict__ Lx) {
  far_chain_priority();
  __shared__ cplx sum[NT];
  const int b = boxes[blockIdx.x];
  const int k0 = sptr[blockIdx.x], k1 = sptr[blockIdx.x + 1];
  const int groups = NT / nc;
  const int g = threadIdx.x / nc, j = threadIdx.x - g * nc;
  const int d = dec[j], m = d >> 16;
  if (g < groups) {
    const int js = j < ns ? nc + j : j;  // (order 0 has no imaginary part)
    double re = 0.0, im = 0.0;
    constexpr int U = 4;
    for (int k = k0 + g; k < k1; k += U * groups) {
      T c[U], s[U];
      cplx e[U];
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int kk = min(k + q * groups, k1 - 1);
        const T* w = W + (int64_t)slots[kk] * wr;
        c[q] = w[j];
        s[q] = w[js];
        e[q] = E[(int64_t)sphi[kk] * ne + m];
      }
#pragma unroll
      for (int q = 0; q < U; ++q) {
        if (k + q * groups >= k1) break;
        re += (double)c[q] * e[q].re + (double)s[q] * e[q].im;
        im += (double)s[q] * e[q].re - (double)c[q] * e[q].im;
      }
    }
    sum[threadIdx.x] = cmk(re, im);
  }
  __syncthreads();
  if (g > 0) return;
  cplx v = sum[j];
  for (int q = 1; q < groups; ++q) v = v + sum[q * nc + j];
  const double inv = sc[blevel[b]];
  double* l = Lx + (int64_t)b * nr + (d & 0xffff);
  l[0] += v.re * inv;
  if (m) l[1] += v.im * inv;
}

// M2M / L2L of a level (eqs. metome, letole as the real-form octant operators
// of build_xlate_ops_kernel) with the operands taken straight from global
// memory into the FP64 matrix-core fragments: no LDS staging, no partials in
// memory.  A wave owns one 16 x 16 block of one unit's product (rows 16 rb..,
// columns 16 cb.. of a 32-column tile) and keeps two batches of kXlDirectKB
// k-steps in flight, so a level costs a few memory latencies and one launch
// (a GEMM staged through LDS paid one latency per K slice, plus a reduction
// launch for M2M).  Lane layout (v_mfma_f64_16x16x4f64): A[row = l % 16][k =
// l / 16], B[k = l / 16][col = l % 16], D[row = l / 16 + 4 v][col = l % 16];
// k runs in order, so the products do not depend on the batch size.
// UP (M2M): block (tile, rb, cb), wave w = the tile's unit w (one per child
// octant present, at most 8); the units' blocks meet in LDS and are added in
// unit order into the parents' expansions.
// L2L: block (unit, group of 8 row blocks, cb), wave w = row block 8 y + w; a
// level's tiles hold each child once, so each wave adds its block directly.
constexpr int kXlDirectKB = 4;  // k-steps (of 4) a load batch
template <bool UP>
__global__ void __launch_bounds__(512)
xlate_direct_kernel(int nr, int nrk, int mr, int64_t tile0, int64_t unit0, const int32_t* __restrict__ tile_unit_ptr,
                    const int32_t* __restrict__ unit_s, const int32_t* __restrict__ step_op,
                    const int32_t* __restrict__ step_src, const int32_t* __restrict__ unit_mask,
                    const int32_t* __restrict__ tile_tgt, const double* __restrict__ T,
                    const double* __restrict__ X, double* dst) {
  far_chain_priority();
  constexpr int TB = 32, KB = kXlDirectKB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int cb = blockIdx.z;
  const int nrb = (nr + 15) >> 4;
  int64_t unit, tile;
  int rb;
  bool act;
  if constexpr (UP) {
    tile = tile0 + blockIdx.x;
    const int u0 = tile_unit_ptr[tile], u1 = tile_unit_ptr[tile + 1];
    unit = u0 + wave;
    rb = blockIdx.y;
    act = unit < u1;
  } else {
    unit = unit0 + blockIdx.x;
    tile = tile0 + blockIdx.x;  // an L2L tile is one unit
    rb = 8 * blockIdx.y + wave;
    act = rb < nrb;
  }
  doublex4 acc = doublex4{0.0, 0.0, 0.0, 0.0};
  // a 16-column block whose two 8-column groups hold no source is zero (exact)
  if (act && ((unit_mask[unit] >> (2 * cb)) & 3)) {
    const int s = unit_s[2 * unit];
    const int sb = step_src[(int64_t)s * TB + 16 * cb + li];
    const double* To = T + (int64_t)step_op[s] * nrk * mr + 16 * rb + li;
    const double* Xs = X + (int64_t)(sb < 0 ? 0 : sb) * nr;
    const int nks = nrk >> 2;
    double a0[KB], b0[KB], a1[KB], b1[KB];
    auto ld = [&](double(&a)[KB], double(&b)[KB], int kb) {
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        const int k = 4 * (kb + j) + lk;
        const bool in = kb + j < nks;
        a[j] = in ? To[(int64_t)k * mr] : 0.0;
        b[j] = (in && sb >= 0 && k < nr) ? Xs[k] : 0.0;
      }
    };
    auto mm = [&](const double(&a)[KB], const double(&b)[KB], int kb) {
#pragma unroll
      for (int j = 0; j < KB; ++j)
        if (kb + j < nks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[j], b[j], acc, 0, 0, 0);
    };
    ld(a0, b0, 0);
    if (KB < nks) ld(a1, b1, KB);
    for (int kb = 0; kb < nks; kb += 2 * KB) {
      mm(a0, b0, kb);
      if (kb + 2 * KB < nks) ld(a0, b0, kb + 2 * KB);
      if (kb + KB < nks) {
        mm(a1, b1, kb + KB);
        if (kb + 3 * KB < nks) ld(a1, b1, kb + 3 * KB);
      }
    }
  }
  if constexpr (UP) {
    __shared__ double red[8][4][64];
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][v][lane] = acc[v];
    __syncthreads();
    if (threadIdx.x >= 256) return;
    const int l = threadIdx.x & 63, v = threadIdx.x >> 6;
    const int nu = tile_unit_ptr[tile + 1] - tile_unit_ptr[tile];
    double sum = 0.0;
    for (int w = 0; w < nu; ++w) sum += red[w][v][l];
    const int row = 16 * rb + (l >> 4) + 4 * v;
    const int tg = tile_tgt[tile * TB + 16 * cb + (l & 15)];
    if (tg >= 0 && row < nr) dst[(int64_t)tg * nr + row] += sum;
  } else {
    if (!act) return;
    const int tg = tile_tgt[tile * TB + 16 * cb + li];
    if (tg < 0) return;
    double* Dt = dst + (int64_t)tg * nr;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = 16 * rb + lk + 4 * v;
      if (row < nr) Dt[row] += acc[v];
    }
  }
}

// ---------------------------------------------------------------- batched form
// Many charge vectors in one evaluation: expansions are stored RHS-major
// ([rhs][box][(p+1)^2]).  The translations (M2M, L2L) run one block per target
// box whose columns are the charge vectors: each entry is one octant operator
// applied to the source box's expansions of all G <= 64 vectors, in FP64 on the
// matrix cores (v_mfma_f64_16x16x4f64; lane l: A[row
// l % 16][k l / 16], B[k l / 16][column l % 16], result D[row l / 16 + 4 v]
// [column l % 16], verified on the GPU by an in-bounds probe).  Four waves, 2 x 2
// over the tile of 32 MRT operator rows x 64 vectors, each owning MRT x 2 blocks
// of 16 x 16; operator and operand slices of KC columns double-buffered in LDS.
template <int MRT>
__global__ void __launch_bounds__(256)
xlate_batch_kernel(int nr, int nrk, int g, int64_t nb, const int32_t* __restrict__ boxes, int64_t box0,
                   const int32_t* __restrict__ ptr, const int32_t* __restrict__ src,
                   const int32_t* __restrict__ op, const double* __restrict__ T, const double* __restrict__ X,
                   double* __restrict__ dst) {
  far_chain_priority();
  constexpr int KC = (MRT <= 4) ? 16 : 8;
  constexpr int MR = 32 * MRT;
  constexpr int TB = 64;
  constexpr int TS = MR + 4;     // LDS row strides (doubles), padded against bank conflicts
  constexpr int BSR = TB + 1;    // (the operand slice is stored transposed)
  constexpr int NTR = KC * MR / 256;
  constexpr int NBR = KC * TB / 256;
  static_assert(NTR * 256 == KC * MR && NBR * 256 == KC * TB, "slice must split evenly over the threads");
  __shared__ double Ts[2][KC * TS];
  __shared__ double Bs[2][KC * BSR];
  const int b = boxes[box0 + blockIdx.x];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int row0 = (wave & 1) * (MR / 2), col0 = (wave >> 1) * 32;
  const int li = lane & 15, lk = lane >> 4;
  doublex4 acc[MRT][2];
#pragma unroll
  for (int i = 0; i < MRT; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
  const int s0 = ptr[b], s1 = ptr[b + 1];
  const int nch = nrk / KC;
  const int total = (s1 - s0) * nch;
  const int64_t slab = nb * (int64_t)nr;  // one vector's expansions
  double rt[NTR], rb[NBR];
  auto load = [&](int q) {
    const int s = s0 + q / nch, k0 = (q % nch) * KC;
    const double* Tc = T + ((int64_t)op[s] * nrk + k0) * MR;
    const int sb = src[s];
#pragma unroll
    for (int r = 0; r < NTR; ++r) rt[r] = Tc[tid + 256 * r];
#pragma unroll
    for (int r = 0; r < NBR; ++r) {
      const int i = tid + 256 * r, col = i / KC, k = k0 + i % KC;
      rb[r] = (col < g && k < nr) ? X[col * slab + (int64_t)sb * nr + k] : 0.0;
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int r = 0; r < NTR; ++r) {
      const int i = tid + 256 * r;
      Ts[buf][(i / MR) * TS + (i % MR)] = rt[r];
    }
#pragma unroll
    for (int r = 0; r < NBR; ++r) {
      const int i = tid + 256 * r;
      Bs[buf][(i % KC) * BSR + i / KC] = rb[r];
    }
  };
  if (total > 0) {
    load(0);
    stash(0);
    if (total > 1) load(1);
  }
  __syncthreads();
  for (int q = 0; q < total; ++q) {
    const double* Tb = Ts[q & 1];
    const double* Bb = Bs[q & 1];
#pragma unroll
    for (int ks = 0; ks < KC; ks += 4) {
      double a[MRT], bv[2];
#pragma unroll
      for (int i = 0; i < MRT; ++i) a[i] = Tb[(ks + lk) * TS + row0 + 16 * i + li];
#pragma unroll
      for (int j = 0; j < 2; ++j) bv[j] = Bb[(ks + lk) * BSR + col0 + 16 * j + li];
#pragma unroll
      for (int i = 0; i < MRT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], bv[j], acc[i][j], 0, 0, 0);
    }
    if (q + 1 < total) {
      // the other buffer was last read before the previous barrier
      stash((q & 1) ^ 1);
      if (q + 2 < total) load(q + 2);
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = col0 + 16 * j + li;
    if (col >= g) continue;
#pragma unroll
    for (int i = 0; i < MRT; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = row0 + 16 * i + lk + 4 * v;
        if (row >= nr) continue;
        dst[col * slab + (int64_t)b * nr + row] += acc[i][j][v];
      }
  }
}

// The batched FP64 top levels' work items of one box, in item order, scaled by
// 1/S of its level, added to its local expansions (all vectors).
__global__ void __launch_bounds__(256)
m2l_btop_reduce_kernel(int nr, int g, const int32_t* __restrict__ boxes, const int32_t* __restrict__ iptr,
                       const double* __restrict__ part, const int32_t* __restrict__ blevel,
                       const double* __restrict__ sc, int64_t slab, double* __restrict__ Lx) {
  far_chain_priority();
  const int b = boxes[blockIdx.x];
  const int i0 = iptr[blockIdx.x], i1 = iptr[blockIdx.x + 1];
  const double inv = sc[blevel[b]];
  for (int t = threadIdx.x; t < g * nr; t += blockDim.x) {
    const int col = t / nr, row = t - col * nr;
    double v = 0.0;
    for (int it = i0; it < i1; ++it) v += part[((int64_t)it * 64 + col) * nr + row];
    Lx[col * slab + (int64_t)b * nr + row] += v * inv;
  }
}

// Expansions of all vectors, vector-minor, for the batched M2L: X [box][pair][gw]
// (re, im) of M [vector][box][(p+1)^2], zeros from vector g on.  One block per box;
// tiles of 64 coefficients x the vectors are read row by row and turned in LDS
// (read column by column they took 0.82 ms at 7,571 boxes, p = 10, 64 vectors).
template <class T>
__global__ void __launch_bounds__(256)
vector_minor_kernel(int nr, int nc, int ns, int g, int gw, int64_t slab, const double* __restrict__ M,
                    T* __restrict__ X) {
  __shared__ double tile[64][65];
  const int64_t b = blockIdx.x;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int c0 = 0; c0 < nr; c0 += 64) {
    __syncthreads();  // the previous tile's readers are done
    for (int v = wave; v < gw; v += 4)
      tile[v][lane] = v < g && c0 + lane < nr ? M[v * slab + b * nr + c0 + lane] : 0.0;
    __syncthreads();
    if (lane >= gw) continue;
    for (int c = c0 + wave; c < min(nr, c0 + 64); c += 4) {
      int n, m;
      bool im;
      rsplit(c, &n, &m, &im);
      T* x = X + ((b * nc + (m ? cidx(n - 1, m - 1) : ns + n)) * gw + lane) * 2;
      x[im ? 1 : 0] = (T)tile[lane][c - c0];
      if (m == 0) x[1] = (T)0;
    }
  }
}

// Batched M2L in operator frames (FP32; FP64 form and top levels in FP64): a block
// takes one target box, or a run of its entries (items), and up to 64 vectors,
// 16 a wave.  Entry by entry the wave turns the source's pairs (one azimuth for
// all its vectors, rows of 16 vectors contiguous) into the operand fragments; the
// operator goes through LDS as in m2l_frame_kernel, with the entry's phases.  Each
// entry's product is turned back and added to FP64 totals by itself (products of
// one azimuth added up in FP32 first: 11.1 against 11.9 ms, but half again the
// error).  swizzle: each XCD takes a contiguous range of the boxes, whose sources
// its L2 shares.
// Bound by the operators' and sources' bytes out of the caches and, at two to three
// waves a SIMD, their latency (1.69 M pairs x 64 vectors, batches of 2: 30.8 ms,
// matrix cores 0.40 busy, 0.44 of 1.16 G requests to the L2 hit): 604,000 pairs x 64
// vectors at p = 10, 14.2 ms by the dense operators (box by box, FP32), 11.9 ms;
// the FP64 top levels (42,708 pairs) 2.18 and 1.47 ms.  At three waves a SIMD
// (batches of 2) 11.9 ms against 13.9 at two (batches of 4), in XCD ranges 14.2 (they
// end unevenly); 1.69 M pairs in box order / XCD ranges: batches of 2 30.8 / 38.4, of 4
// 35.2 / 36.6, of 8 32.1 / 31.5 ms, so both orders are among the tuner's choices.
template <class T, int RC, int RS, int KB>
__global__ void __launch_bounds__(256, sizeof(T) == 4 && KB == 2 && RC + RS <= 9 ? 3 : 2)
m2l_frame_batch_kernel(int nr, int nc, int ns, int ne, int g, int gw, int64_t slab, int64_t nblk, int swizzle, XcdSplit xcd,
                       const int32_t* __restrict__ boxes, const int32_t* __restrict__ items,
                       const int32_t* __restrict__ bptr, int64_t box0, const int32_t* __restrict__ eop,
                       const int32_t* __restrict__ ephi, const int32_t* __restrict__ esrc,
                       const int32_t* __restrict__ ekind, const int32_t* __restrict__ dec, unsigned parts,
                       const T* __restrict__ A, const T* __restrict__ X, const cplx* __restrict__ E,
                       const int32_t* __restrict__ blevel, const double* __restrict__ sc, double* __restrict__ Lx,
                       double* __restrict__ part) {
  far_chain_priority();
  constexpr int RT = 16 * (RC + RS);
  constexpr int KV = 4 * RT * (int)sizeof(T) / 16;  // 16-byte vectors of a k-step of the operator
  constexpr int PER = (KB * KV + 255) / 256;
  using Acc = typename FrameTypes<T>::Acc;
  typedef T Pair __attribute__((ext_vector_type(2)));
  __shared__ intx4 As[2][KB * KV];
  // phases of an entry's azimuth, entry e in row e mod 3: a wave may still turn entry
  // e - 1 back while another stores those of e + 1
  __shared__ cplx Es[3][kPMax + 1];
  __shared__ int32_t ds[(kPMax + 1) * (kPMax + 2) / 2];
  int64_t i = blockIdx.x;
  if (swizzle) {
    const int x = (int)(i & 7);
    i = xcd.off[x] + (i >> 3);
    if (i >= xcd.off[x + 1]) return;
  } else if (i >= nblk) {
    return;
  }
  const int b = boxes[items ? items[3 * i] : i];
  const int e0 = items ? items[3 * i + 1] : bptr[b - box0], e1 = items ? items[3 * i + 2] : bptr[b - box0 + 1];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), vec = 16 * wave + li;
  const bool work = 16 * wave < g;
  const int kc = frame_ksteps(nc), ks = frame_ksteps(ns);
  for (int j = tid; j < nc; j += 256) ds[j] = dec[j];
  Acc ac[RC], as[RS];
  double tc[RC][4], ts[RS][4];
#pragma unroll
  for (int r = 0; r < RC; ++r) {
    ac[r] = Acc{0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < 4; ++v) tc[r][v] = 0.0;
  }
#pragma unroll
  for (int r = 0; r < RS; ++r) {
    as[r] = Acc{0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < 4; ++v) ts[r][v] = 0.0;
  }
  intx4 va[PER];
  cplx ev = cmk(0.0, 0.0);
  auto load_a = [&](int e, int k0) {
    const intx4* Ap = reinterpret_cast<const intx4*>(A) + ((int64_t)eop[e] * kc + k0) * KV;
    const int n = min(KB, kc - k0) * KV;
    if (k0 == 0 && tid < nc - ns) ev = E[(int64_t)ephi[e] * ne + tid];
#pragma unroll
    for (int r = 0; r < PER; ++r)
      if (tid + 256 * r < n) va[r] = Ap[tid + 256 * r];
  };
  auto stash_a = [&](int buf, int e, int k0) {
    if (k0 == 0 && tid < nc - ns) Es[e % 3][tid] = ev;
#pragma unroll
    for (int r = 0; r < PER; ++r)
      if (tid + 256 * r < KB * KV) As[buf][tid + 256 * r] = va[r];
  };
  Pair x[KB];
  auto load_b = [&](int e, int k0) {
    const Pair* Xb = reinterpret_cast<const Pair*>(X) + (int64_t)esrc[e] * nc * gw + vec;
#pragma unroll
    for (int t = 0; t < KB; ++t) {
      const int j = min(4 * (k0 + t) + lk, nc - 1);  // (columns from nc on are zero in A)
      x[t] = Xb[j * gw];
    }
  };
  // an entry's products turned back (e^{-i m phi}) into the totals
  auto turn_back = [&](const cplx* Ee) {
#pragma unroll
    for (int r = 0; r < RC; ++r)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int j = min(16 * r + FrameTypes<T>::row(lk, v), nc - 1);  // (rows from nc on are dropped)
        const cplx w = Ee[ds[j] >> 16];
        const double c = (double)ac[r][v], s = r < RS ? (double)as[r < RS ? r : 0][v] : 0.0;
        tc[r][v] += c * w.re + s * w.im;
        if (r < RS) ts[r < RS ? r : 0][v] += s * w.re - c * w.im;
        if (v & 1) __builtin_amdgcn_sched_barrier(0);  // (two phases in flight: registers)
      }
#pragma unroll
    for (int r = 0; r < RC; ++r) ac[r] = Acc{0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < RS; ++r) as[r] = Acc{0, 0, 0, 0};
  };
  __syncthreads();  // ds
  if (e0 < e1) {
    load_a(e0, 0);
    if (work) load_b(e0, 0);
    stash_a(0, e0, 0);
  }
  __syncthreads();
  int buf = 0;
  for (int e = e0; e < e1; ++e) {
    const bool on = (parts & (unsigned)ekind[e]) != 0;
    for (int k0 = 0; k0 < kc; k0 += KB) {
      const bool last = k0 + KB >= kc;
      const bool more = !last || e + 1 < e1;
      if (more) load_a(last ? e + 1 : e, last ? 0 : k0 + KB);
      if (work) {
        T a[KB], c[KB];
#pragma unroll
        for (int t = 0; t < KB; ++t) {
          const int j = min(4 * (k0 + t) + lk, nc - 1);
          const cplx v = Es[e % 3][ds[j] >> 16] * cmk((double)x[t].x, (double)x[t].y);
          a[t] = on ? (T)v.re : (T)0;
          c[t] = on ? (T)v.im : (T)0;
        }
        if (more) load_b(last ? e + 1 : e, last ? 0 : k0 + KB);
        const T* Ab = reinterpret_cast<const T*>(As[buf]) + lk * RT + li;
#pragma unroll
        for (int t = 0; t < KB; ++t) {
          if (k0 + t >= kc) break;
#pragma unroll
          for (int r = 0; r < RC; ++r) ac[r] = mfma4(Ab[4 * t * RT + 16 * r], a[t], ac[r]);
          if (k0 + t < ks) {
#pragma unroll
            for (int r = 0; r < RS; ++r) as[r] = mfma4(Ab[4 * t * RT + 16 * (RC + r)], c[t], as[r]);
          }
        }
      }
      if (more) {
        stash_a(buf ^ 1, last ? e + 1 : e, last ? 0 : k0 + KB);  // last read before the previous barrier
        __syncthreads();
        buf ^= 1;
      }
    }
    if (work) turn_back(Es[e % 3]);
  }
  if (vec >= g) return;
  const double inv = items ? 1.0 : sc[blevel[b]];
  double* o = items ? part + (i * 64 + vec) * nr : Lx + vec * slab + (int64_t)b * nr;
#pragma unroll
  for (int r = 0; r < RC; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int j = 16 * r + FrameTypes<T>::row(lk, v);
      if (j >= nc) continue;
      const int d = ds[j], off = d & 0xffff;
      if (items) {
        o[off] = tc[r][v];
        if (d >> 16) o[off + 1] = r < RS ? ts[r < RS ? r : 0][v] : 0.0;
      } else {
        o[off] += tc[r][v] * inv;
        if (d >> 16) o[off + 1] += (r < RS ? ts[r < RS ? r : 0][v] : 0.0) * inv;
      }
    }
}


// Batched gather and combine through point-major copies, so that every global
// access is coalesced: tiles of 64 points x 64 vectors go through LDS.
// q [r][user] -> qu [user][64] (vectors past g are zero).
__global__ void __launch_bounds__(256)
transpose_users_kernel(const double* __restrict__ q, int64_t ldq, int g, int64_t n, double* __restrict__ qu) {
  __shared__ double tile[64][65];
  const int64_t u0 = (int64_t)blockIdx.x * 64;
  const int t = threadIdx.x, lo = t & 63, hi = t >> 6;
  for (int r = hi; r < 64; r += 4) tile[r][lo] = (r < g && u0 + lo < n) ? q[r * ldq + u0 + lo] : 0.0;
  __syncthreads();
  for (int ul = hi; ul < 64; ul += 4)
    if (u0 + ul < n) qu[(u0 + ul) * 64 + lo] = tile[lo][ul];
}

// tree point i: qt[r][i], qb64 / qb32 [i][r] from the point-major qu
__global__ void __launch_bounds__(256)
gather_rows_kernel(const double* __restrict__ qu, const int32_t* __restrict__ puser, int64_t np, int g,
                   double* __restrict__ qt, double* __restrict__ qb64, float* __restrict__ qb32) {
  __shared__ double tile[64][65];
  const int64_t i0 = (int64_t)blockIdx.x * 64;
  const int t = threadIdx.x, lo = t & 63, hi = t >> 6;
  for (int il = hi; il < 64; il += 4) {
    const int64_t i = i0 + il;
    double v = 0.0;
    if (i < np) {
      v = qu[(int64_t)puser[i] * 64 + lo];
      if (qb64) qb64[i * 64 + lo] = v;
      if (qb32) qb32[i * 64 + lo] = (float)v;
    }
    tile[lo][il] = v;
  }
  __syncthreads();
  for (int r = hi; r < g; r += 4)
    if (i0 + lo < np) qt[r * np + i0 + lo] = tile[r][lo];
}

// phit [r][i] -> pt [i][64]
__global__ void __launch_bounds__(256)
transpose_points_kernel(const double* __restrict__ phit, int64_t np, int g, double* __restrict__ pt) {
  __shared__ double tile[64][65];
  const int64_t i0 = (int64_t)blockIdx.x * 64;
  const int t = threadIdx.x, lo = t & 63, hi = t >> 6;
  for (int r = hi; r < 64; r += 4) tile[r][lo] = (r < g && i0 + lo < np) ? phit[r * np + i0 + lo] : 0.0;
  __syncthreads();
  for (int il = hi; il < 64; il += 4)
    if (i0 + il < np) pt[(i0 + il) * 64 + lo] = tile[lo][il];
}

// phi [r][user] = far + near field at the (one or two) tree positions, from pt
__global__ void __launch_bounds__(256)
combine_rows_kernel(const double* __restrict__ pt, int g, const int32_t* __restrict__ upos, int64_t n,
                    double* __restrict__ phi, int64_t ldphi) {
  __shared__ double tile[64][65];
  const int64_t u0 = (int64_t)blockIdx.x * 64;
  const int t = threadIdx.x, lo = t & 63, hi = t >> 6;
  for (int ul = hi; ul < 64; ul += 4) {
    const int64_t u = u0 + ul;
    double v = 0.0;
    if (u < n) {
      const int32_t a = upos[2 * u], b = upos[2 * u + 1];
      if (a >= 0) v += pt[(int64_t)a * 64 + lo];
      if (b >= 0) v += pt[(int64_t)b * 64 + lo];
    }
    tile[lo][ul] = v;
  }
  __syncthreads();
  for (int r = hi; r < g; r += 4)
    if (u0 + lo < n) phi[r * ldphi + u0 + lo] = tile[r][lo];
}


// Batched free-space P2P: 1/r computed once per pair and applied to every
// vector (charges vector-minor, qb[source][64]).  FP64 variant.
__global__ void __launch_bounds__(64)
p2p_free_batch64_kernel(int64_t g0, int64_t n, int g, const int32_t* __restrict__ pleaf,
                        const int32_t* __restrict__ ptr, const int32_t* __restrict__ rng,
                        const double* __restrict__ px, const double* __restrict__ py,
                        const double* __restrict__ ph, const double* __restrict__ qb, int64_t np,
                        double* __restrict__ phit) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int gi = (int)(g0 + i);
  const int lf = pleaf[gi];
  const double xi = px[gi], yi = py[gi], hi = ph[gi];
  double acc[64];
#pragma unroll
  for (int r = 0; r < 64; ++r) acc[r] = 0.0;
  const int e1 = ptr[lf + 1];
  for (int e = ptr[lf]; e < e1; ++e) {
    const int s0 = rng[2 * e], scn = rng[2 * e + 1];
    for (int j = 0; j < scn; ++j) {
      const int s = s0 + j;
      const double dx = xi - px[s], dy = yi - py[s], dz = hi - ph[s];
      const double r2 = dx * dx + dy * dy + dz * dz;
      const double y = (s != gi) ? rsqrt_nr(r2) : 0.0;
      const double* qs = qb + (int64_t)s * 64;
#pragma unroll
      for (int r = 0; r < 64; ++r) acc[r] = fma(qs[r], y, acc[r]);
    }
  }
  for (int r = 0; r < g; ++r) phit[r * np + gi] += acc[r] * kInv4Pi;
}


// Batched reaction near field on the matrix cores (FP32 form), spread over the
// GPU: a wave takes one entry (a target leaf, a source range) and 16 of its
// target rows, and forms the 16 x 64 product of the stored kernel values K
// (row-major targets x sources, FP64, rounded to FP32 here) with the sources'
// 64 charge vectors, 4 sources a step (lane l: A = K[row l % 16][source l / 16],
// B = q[source l / 16][vector block + l % 16]).  The product, one FP32 sum on
// the matrix cores, goes to the entry's partial rows; a second kernel adds a
// leaf's partials in FP64, in entry order.
__global__ void __launch_bounds__(256)
p2p_reaction_batch_rows_kernel(int64_t nunits, const int32_t* __restrict__ units, const int32_t* __restrict__ rng,
                               const int64_t* __restrict__ voff, const int32_t* __restrict__ rowoff,
                               const double* __restrict__ val, const float* __restrict__ qb,
                               float* __restrict__ part) {
  const int64_t u = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (u >= nunits) return;  // whole waves
  const int lane = threadIdx.x & 63;
  const int l16 = lane & 15, lk = lane >> 4;
  const int e = units[3 * u], r0 = units[3 * u + 1], tc = units[3 * u + 2];
  const int s0 = rng[2 * e], sc = rng[2 * e + 1];
  const int ta = r0 + l16;  // this lane's target row for the A fragment
  const double* kv = val + voff[e] + (int64_t)min(ta, tc - 1) * sc;
  floatx4 acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int ks = 0; ks < sc; ks += 4) {
    const int sk = ks + lk;
    const bool ok = sk < sc;
    const float a = (ok && ta < tc) ? (float)kv[sk] : 0.f;
    const float* qs = qb + (int64_t)(s0 + (ok ? sk : 0)) * 64 + l16;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float bq = ok ? qs[16 * j] : 0.f;
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bq, acc[j], 0, 0, 0);
    }
  }
  float* pe = part + (int64_t)rowoff[e] * 64;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int t = r0 + 4 * lk + v;
      if (t < tc) pe[(int64_t)t * 64 + 16 * j + l16] = acc[j][v];
    }
}

__global__ void __launch_bounds__(256)
p2p_reaction_batch_sum_kernel(int g, const int32_t* __restrict__ leaves, const int32_t* __restrict__ bstart,
                              const int32_t* __restrict__ bcount, const int32_t* __restrict__ ptr,
                              const int32_t* __restrict__ rowoff, const float* __restrict__ part, int64_t np,
                              double* __restrict__ phit) {
  const int lf = blockIdx.x;
  const int e0 = ptr[lf], e1 = ptr[lf + 1];
  if (e0 == e1) return;
  const int b = leaves[lf];
  const int t0 = bstart[b], tc = bcount[b];
  for (int i = threadIdx.x; i < tc * 64; i += blockDim.x) {
    const int t = i >> 6, v = i & 63;
    if (v >= g) continue;
    double acc = 0.0;
    for (int e = e0; e < e1; ++e) acc += (double)part[((int64_t)rowoff[e] + t) * 64 + v];
    phit[(int64_t)v * np + t0 + t] += acc;
  }
}

// Batched reaction P2P: one block per target leaf, one wavefront per target
// row, one lane per vector; kernel values are wavefront broadcasts.
__global__ void __launch_bounds__(256)
p2p_reaction_batch_kernel(int g, const int32_t* __restrict__ leaves, const int32_t* __restrict__ bstart,
                          const int32_t* __restrict__ bcount, const int32_t* __restrict__ ptr,
                          const int32_t* __restrict__ rng, const int64_t* __restrict__ voff,
                          const double* __restrict__ val, const double* __restrict__ qb, int64_t np,
                          double* __restrict__ phit) {
  const int lf = blockIdx.x;
  const int e0 = ptr[lf], e1 = ptr[lf + 1];
  if (e0 == e1) return;
  const int b = leaves[lf];
  const int t0 = bstart[b], tc = bcount[b];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int ti = wave; ti < tc; ti += 4) {
    double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int e = e0; e < e1; ++e) {
      const int s0 = rng[2 * e], scn = rng[2 * e + 1];
      const double* row = val + voff[e] + (int64_t)ti * scn;
      const double* qs = qb + (int64_t)s0 * 64 + lane;
      int j = 0;
      for (; j + 8 <= scn; j += 8) {
        double v[8], w[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          v[u] = row[j + u];
          w[u] = qs[(int64_t)(j + u) * 64];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = fma(v[u], w[u], a[u]);
      }
      for (; j < scn; ++j) a[0] = fma(row[j], qs[(int64_t)j * 64], a[0]);
    }
    const double tot = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    if (lane < g) phit[lane * np + t0 + ti] += tot;
  }
}

__global__ void zero_kernel(double* __restrict__ a, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0.0;
}

// x = hi + lo with hi = (float)x and lo = (float)(x - hi)
__global__ void split_f32_kernel(const double* __restrict__ a, int64_t n, float* __restrict__ hi,
                                 float* __restrict__ lo) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float h = (float)a[i];
  hi[i] = h;
  lo[i] = (float)(a[i] - (double)h);
}


// Batched L2P: one block per leaf, 16 vectors a wave.  A chunk of points' harmonics
// (with the weight 2 of orders m > 0, signs of the real layout) go to LDS once for
// all vectors, and the FP64 matrix cores multiply them with the leaf's local
// expansions, which each wave holds in its fragments: D [vector][point], so that
// 16 consecutive points of a vector leave together.  A block per leaf and vector
// computed the harmonics 64 times over: 1.06 ms at 131,072 charges, p = 10, 64
// vectors; now 0.22 ms.  KN: k-steps the fragments hold.
template <int KN>
__global__ void __launch_bounds__(256)
l2p_batch_kernel(int p, int g, const int32_t* __restrict__ leaves, const int32_t* __restrict__ bstart,
                 const int32_t* __restrict__ bcount, const int32_t* __restrict__ blevel,
                 const double* __restrict__ bcx, const double* __restrict__ bcy, const double* __restrict__ bch,
                 const double* __restrict__ sc, const double* __restrict__ px, const double* __restrict__ py,
                 const double* __restrict__ ph, const double* __restrict__ Lx, const double* __restrict__ coefR,
                 double* __restrict__ phit, int64_t lstride, int64_t pstride) {
  far_chain_priority();
  extern __shared__ double w[];  // [PT][ld]
  constexpr int PT = KN <= 31 ? 32 : 16;
  const int np1 = p + 1, nr = np1 * np1, nks = (nr + 3) / 4, ld = 4 * nks + 1;
  const int b = leaves[blockIdx.x];
  const double inv = sc[blevel[b]];
  const double cx = bcx[b], cy = bcy[b], ch = bch[b];
  const int s0 = bstart[b], cnt = bcount[b];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int ncp = ncoef(p);
  double a[KN];
#pragma unroll
  for (int ks = 0; ks < KN; ++ks) {
    const int vec = 16 * wave + li, k = 4 * ks + lk;
    a[ks] = vec < g && k < nr ? Lx[vec * lstride + (int64_t)b * nr + k] : 0.0;
  }
  for (int i = tid; i < PT * (ld - nr); i += 256) w[i / (ld - nr) * ld + nr + i % (ld - nr)] = 0.0;
  for (int c0 = 0; c0 < cnt; c0 += PT) {
    const int np = min(PT, cnt - c0);
    __syncthreads();  // the previous chunk is consumed
    for (int i = tid; i < PT * np1; i += 256) {
      const int j = i / np1, m = i % np1;
      double* wj = w + j * ld;
      const int gp = s0 + c0 + min(j, np - 1);  // (rows past the last point are not stored)
      const double x = (px[gp] - cx) * inv, y = (py[gp] - cy) * inv, z = (ph[gp] - ch) * inv;
      const double r2 = x * x + y * y + z * z;
      cplx Rmm = cmk(0.28209479177387814, 0.0);
      for (int mm = 1; mm <= m; ++mm) Rmm = coefR[2 * ncp + mm] * (cmk(x, y) * Rmm);
      cplx Rm2 = cmk(0.0, 0.0), Rm1 = Rmm;
      for (int n = m; n <= p; ++n) {
        if (n > m) {
          const cplx Rn = n == m + 1 ? (coefR[2 * ncp + np1 + m] * z) * Rmm
                                     : coefR[cidx(n, m)] * (z * Rm1 - (coefR[ncp + cidx(n, m)] * r2) * Rm2);
          Rm2 = Rm1;
          Rm1 = Rn;
        }
        if (m == 0) {
          wj[n * n] = Rm1.re;
        } else {
          wj[n * n + 2 * m - 1] = 2.0 * Rm1.re;
          wj[n * n + 2 * m] = -2.0 * Rm1.im;
        }
      }
    }
    __syncthreads();
    if (16 * wave >= g) continue;
    for (int p0 = 0; p0 < np; p0 += 16) {
      doublex4 acc = {0.0, 0.0, 0.0, 0.0};
      const double* wp = w + (p0 + li) * ld + lk;
#pragma unroll
      for (int ks = 0; ks < KN; ++ks)
        if (ks < nks) acc = mfma4(a[ks], wp[4 * ks], acc);
      if (p0 + li < np)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int vec = 16 * wave + lk + 4 * v;
          if (vec < g) phit[vec * pstride + s0 + c0 + p0 + li] = acc[v];
        }
    }
  }
}

// L2P of the single-vector evaluation with the order P fixed at compile time,
// so the recurrence over (n, m) unrolls and its coefficients become scalar
// loads at fixed offsets: the same harmonics and sum as the batched form's, with the
// weight 2 of the m > 0 terms folded into the local expansion in LDS.
template <int P>
__global__ void __launch_bounds__(64)
l2p_fixed_kernel(const int32_t* __restrict__ leaves, const int32_t* __restrict__ bstart,
                 const int32_t* __restrict__ bcount, const int32_t* __restrict__ blevel,
                 const double* __restrict__ bcx, const double* __restrict__ bcy, const double* __restrict__ bch,
                 const double* __restrict__ sc, const double* __restrict__ px, const double* __restrict__ py,
                 const double* __restrict__ ph, const double* __restrict__ Lx, const double* __restrict__ coefR,
                 double* __restrict__ phit) {
  far_chain_priority();
  constexpr int nc = (P + 1) * (P + 2) / 2;
  __shared__ cplx Ls[nc];
  const int b = leaves[blockIdx.x];
  for (int i = threadIdx.x; i < nc; i += 64) {
    const int nn = isqrt_row(i), mm = i - cidx(nn, 0);
    const cplx v = rload(Lx + (int64_t)b * (P + 1) * (P + 1), nn, mm);
    Ls[i] = mm ? cmk(2.0 * v.re, 2.0 * v.im) : v;
  }
  __syncthreads();
  const double inv = sc[blevel[b]];
  const double cx = bcx[b], cy = bcy[b], ch = bch[b];
  const int s0 = bstart[b], cnt = bcount[b];
  for (int j = threadIdx.x; j < cnt; j += 64) {
    const int g = s0 + j;
    const double x = (px[g] - cx) * inv, y = (py[g] - cy) * inv, z = (ph[g] - ch) * inv;
    const double r2 = x * x + y * y + z * z;
    const cplx w = cmk(x, y);
    cplx Rmm = cmk(0.28209479177387814, 0.0);
    double acc = 0.0;
#pragma unroll 1
    for (int m = 0; m <= P; ++m) {
      if (m > 0) Rmm = coefR[2 * nc + m] * (w * Rmm);
      cplx L = Ls[cidx(m, m)];
      acc += L.re * Rmm.re - L.im * Rmm.im;
      if (m + 1 <= P) {
        cplx Rm2 = Rmm;
        cplx Rm1 = (coefR[2 * nc + P + 1 + m] * z) * Rmm;
        L = Ls[cidx(m + 1, m)];
        acc += L.re * Rm1.re - L.im * Rm1.im;
#pragma unroll 2
        for (int n = m + 2; n <= P; ++n) {
          const double a = coefR[cidx(n, m)], bb = coefR[nc + cidx(n, m)];
          const cplx Rn = a * (z * Rm1 - (bb * r2) * Rm2);
          L = Ls[cidx(n, m)];
          acc += L.re * Rn.re - L.im * Rn.im;
          Rm2 = Rm1;
          Rm1 = Rn;
        }
      }
    }
    phit[g] = acc;
  }
}

// ---- free-space P2P: one workgroup (4 waves) per work unit ---------------
// A unit's source ranges are concatenated and staged through LDS in chunks of
// kPLChunk sources as (x, y, h, q) relative to the target leaf's centre
// (formed in FP64, then rounded to the kernel's type, so that the target's
// own entry is bitwise equal to itself and pairs at zero distance, the self
// pair, are skipped).  Lanes own targets in groups (below), the 4 waves split
// each chunk's sources, and their partial sums meet in LDS.
// The FP32 kernel sums each chunk in FP32 and combines the chunks with
// compensated (Neumaier) summation; the waves' results are added in FP64.
constexpr int kPLThreads = 256;
// LDS the FP32 free P2P launch may reserve beyond its own use when it runs
// beside the far field (unprofiled evaluations), so that its blocks leave LDS
// and wave slots to the far-field chain: 28 KiB holds a CU to 3 P2P blocks,
// 40 KiB to 2, with room for one block of the main M2L beside them.  The
// evaluation-level tuner keeps the fastest of these and no reserve.
constexpr size_t kPLPads[3] = {28672, 40960, 0};
constexpr int kPLChunk = 512;
constexpr int kPLRanges = 256;

// Ranges [eg, eg + nr) of a leaf's list into LDS: starts rs[], exclusive
// prefix sums of the counts rpre[0..nr].  Returns the total count.
__device__ inline int pl_stage_ranges(const int32_t* __restrict__ rng, int eg, int nr, int* rs, int* rpre) {
  const int tid = threadIdx.x;
  if (tid < nr) {
    rs[tid] = rng[2 * (eg + tid)];
    rpre[tid + 1] = rng[2 * (eg + tid) + 1];
  }
  __syncthreads();
  if (tid < 64) {  // wave 0: inclusive scan of rpre[1..nr] in segments of 64
    int carry = 0;
    for (int base = 0; base < nr; base += 64) {
      const int i = base + tid;
      int v = (i < nr) ? rpre[i + 1] : 0;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int u = __shfl_up(v, d, 64);
        if (tid >= d) v += u;
      }
      if (i < nr) rpre[i + 1] = v + carry;
      carry += __shfl(v, 63, 64);
    }
    if (tid == 0) rpre[0] = 0;
  }
  __syncthreads();
  return rpre[nr];
}

// Source index of position pos of the concatenated ranges.
__device__ inline int pl_source(const int* rs, const int* rpre, int nr, int pos) {
  int lo = 0, hi = nr;  // rpre[lo] <= pos < rpre[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (rpre[mid] <= pos) lo = mid; else hi = mid;
  }
  return rs[lo] + (pos - rpre[lo]);
}

template <class T>
struct PLVec;
template <>
struct PLVec<float> { using type = float4; };
template <>
struct PLVec<double> { using type = double4; };

template <class T>
__device__ inline T pl_rsqrt(T r2);
template <>
__device__ inline float pl_rsqrt<float>(float r2) { return __builtin_amdgcn_rsqf(r2); }
template <>
__device__ inline double pl_rsqrt<double>(double r2) { return rsqrt_nr(r2); }

// Lanes of a wave form 4 groups of 16.  In a unit of up to 16 TPL targets
// of the leaf, lane slot s = lane % 16 owns targets s, s + 16, ..., s + 16 (TPL - 1),
// and group g = lane / 16 takes the sources j0 + g, j0 + g + 4, ... of the
// wave's share of each staged chunk.  A leaf of tc targets then wastes fewer
// than 16 lane slots per source (instead of up to 63 with one target a lane),
// and every source read from LDS serves TPL targets.
// MT: most targets a lane, kNS: sources of a group in flight, kWaves a SIMD.  FP64 at
// 8 targets keeps 124 bytes a lane in scratch memory and at 4 none, but reads each
// source and adds its row for half the targets: the plan chooses (pl_targets).
template <class T, int MT>
struct PLCfg {
  static constexpr int kNS = sizeof(T) == 4 || MT <= 4 ? 4 : 2, kWaves = sizeof(T) == 4 ? 4 : 3;
};

// One pair: MASK skips pairs at zero distance (the self pair, or two points at
// one position, which share a leaf): only sources of the target leaf itself
// can be at zero distance from its points.  OK false adds nothing (tail lanes).
template <class T, bool MASK, bool TAIL>
__device__ inline void pl_one(const typename PLVec<T>::type& sv, bool ok, T x, T y, T z, T& p) {
  const T dx = x - sv.x, dy = y - sv.y, dz = z - sv.z;
  const T r2 = dx * dx + dy * dy + dz * dz;
  const T r = pl_rsqrt<T>(r2);
  const T v = MASK ? (r2 > T(0) ? r : T(0)) : r;
  if (TAIL)
    p += ok ? sv.w * v : T(0);
  else
    p += sv.w * v;
}

// Sources [j0, j1) (wave-uniform) of the staged chunk for the lane's TPL
// targets; group g takes j0 + g + 4 i, four of them read ahead of their
// arithmetic, so that each target's sum runs in source order.
template <class T, int TPL, bool MASK>
__device__ inline void pl_range(const typename PLVec<T>::type* __restrict__ src, int j0, int j1, int g,
                                const T* x, const T* y, const T* z, T* p) {
  using V = typename PLVec<T>::type;
  j0 = __builtin_amdgcn_readfirstlane(j0);
  j1 = __builtin_amdgcn_readfirstlane(j1);
  int j = j0;
  for (; j + 16 <= j1; j += 16) {
    const V s0 = src[j + g], s1 = src[j + 4 + g], s2 = src[j + 8 + g], s3 = src[j + 12 + g];
#pragma unroll
    for (int t = 0; t < TPL; ++t) {
      pl_one<T, MASK, false>(s0, true, x[t], y[t], z[t], p[t]);
      pl_one<T, MASK, false>(s1, true, x[t], y[t], z[t], p[t]);
      pl_one<T, MASK, false>(s2, true, x[t], y[t], z[t], p[t]);
      pl_one<T, MASK, false>(s3, true, x[t], y[t], z[t], p[t]);
    }
  }
  for (; j < j1; j += 4) {
    const int jj = j + g;
    const bool ok = jj < j1;
    const V sv = src[ok ? jj : j0];
#pragma unroll
    for (int t = 0; t < TPL; ++t) pl_one<T, MASK, true>(sv, ok, x[t], y[t], z[t], p[t]);
  }
}

// Neumaier step: (acc, cmp) += x.
__device__ inline void pl_neumaier(float& acc, float& cmp, float x) {
  const float t = acc + x;
  cmp += (fabsf(acc) >= fabsf(x)) ? (acc - t) + x : (x - t) + acc;
  acc = t;
}

// ---- mutual free P2P (single vector)
// A unit is up to 16 TPL targets of leaf A against A itself (one way, zero
// distance skipped) and the ranges after A in tree order (both ways).  The
// block's 4 waves split each staged chunk of sources; within a wave, lane slot
// sl = lane % 16 owns targets sl, sl + 16, ..., and lane group g = lane / 16
// takes every fourth source, so each source read from LDS serves TPL targets.
// For a pair (t, s) of the later ranges, one 1/r adds q_s / r to t's sum and
// q_t / r to s's: each lane forms its TPL targets' share of s's sum, the 16
// lanes of the group (a DPP row) add their shares, and the sum is stored in
// s's row for this unit.  Target-side sums: FP32 chunk sums combined by
// compensated summation in the FP32 form; groups and waves added in FP64.

// v from lane CTRL's partner in the lane's DPP row (row_mask, bank_mask all)
template <int CTRL>
__device__ inline float pl_dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ inline double pl_dpp(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b & 0xffffffffull), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
// Sum over the 16 lanes of a row; every lane ends with the same value (each
// step adds two partial sums, which commute).
template <class T>
__device__ inline T pl_row_sum(T v) {
  v += pl_dpp<0xB1>(v);   // quad_perm [1, 0, 3, 2]: lane pairs
  v += pl_dpp<0x4E>(v);   // quad_perm [2, 3, 0, 1]: quads
  v += pl_dpp<0x141>(v);  // row_half_mirror: halves of 8
  v += pl_dpp<0x140>(v);  // row_mirror: the row of 16
  return v;
}

// One pair both ways: p += q_s / r, b += q_t / r.
template <class T, bool TAIL>
__device__ inline void pl_two(const typename PLVec<T>::type& sv, bool ok, T x, T y, T z, T qt, T& p, T& b) {
  const T dx = x - sv.x, dy = y - sv.y, dz = z - sv.z;
  const T r2 = dx * dx + dy * dy + dz * dz;
  const T r = pl_rsqrt<T>(r2);
  if (TAIL)
    p += ok ? sv.w * r : T(0);
  else
    p += sv.w * r;
  b += qt * r;
}

// Sources [j0, j1) (wave-uniform) of the staged chunk, both ways: group g
// takes j0 + g + 4 i; the source-side sum of chunk source j goes to
// out[oidx[j]].
template <class T, int TPL, int NS>
__device__ inline void pl_mrange(const typename PLVec<T>::type* __restrict__ src, int j0, int j1, int g, int sl,
                                 const T* x, const T* y, const T* z, const T* q, T* p, const int* oidx,
                                 T* __restrict__ out) {
  using V = typename PLVec<T>::type;
  j0 = __builtin_amdgcn_readfirstlane(j0);
  j1 = __builtin_amdgcn_readfirstlane(j1);
  int j = j0;
  for (; j + 4 * NS <= j1; j += 4 * NS) {
    V s[NS];
    T b[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      s[k] = src[j + 4 * k + g];
      b[k] = T(0);
    }
#pragma unroll
    for (int t = 0; t < TPL; ++t)
#pragma unroll
      for (int k = 0; k < NS; ++k) pl_two<T, false>(s[k], true, x[t], y[t], z[t], q[t], p[t], b[k]);
#pragma unroll
    for (int k = 0; k < NS; ++k) b[k] = pl_row_sum(b[k]);
    // lane slot k < NS of group g stores source j + 4 k + g: 4 NS consecutive values
    T bv = b[NS - 1];
#pragma unroll
    for (int k = NS - 2; k >= 0; --k) bv = sl == k ? b[k] : bv;
    if (sl < NS) out[oidx[j + 4 * sl + g]] = bv;
  }
  for (; j < j1; j += 4) {
    const int jj = j + g;
    const bool ok = jj < j1;
    const V sv = src[ok ? jj : j0];
    T b = T(0);
#pragma unroll
    for (int t = 0; t < TPL; ++t) pl_two<T, true>(sv, ok, x[t], y[t], z[t], q[t], p[t], b);
    b = pl_row_sum(b);
    if (sl == 0 && ok) out[oidx[jj]] = b;
  }
}

// One unit: targets [tb, tb + tcp) of the leaf at t0 (tc points); ranges
// [e0, e1) of mu_rng, the first the leaf itself.
template <class T, int TPL, int MT>
__device__ void pl_mpass(int tb, int tcp, int t0, int tc, double cx, double cy, double ch, int e0, int e1,
                         const int32_t* __restrict__ rng, const double* __restrict__ px,
                         const double* __restrict__ py, const double* __restrict__ ph,
                         const double* __restrict__ qt, int64_t boff, const int32_t* __restrict__ bidx,
                         double* __restrict__ abuf, T* __restrict__ bbuf, typename PLVec<T>::type* src, int* oidx,
                         int* rs, int* rpre, double* red) {
  using V = typename PLVec<T>::type;
  constexpr int RW = 16 * MT;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int sl = lane & 15, g = lane >> 4;
  // idle target slots sit far away with zero charge: they add nothing to a
  // source's sum (and their own sums are dropped)
  T x[TPL], y[TPL], z[TPL], q[TPL], acc[TPL], cmp[TPL];
#pragma unroll
  for (int t = 0; t < TPL; ++t) {
    const int i = sl + 16 * t;
    x[t] = y[t] = z[t] = T(1e18);
    q[t] = T(0);
    if (i < tcp) {
      x[t] = (T)(px[t0 + tb + i] - cx);
      y[t] = (T)(py[t0 + tb + i] - cy);
      z[t] = (T)(ph[t0 + tb + i] - ch);
      q[t] = (T)qt[t0 + tb + i];
    }
    acc[t] = cmp[t] = T(0);
  }
  int64_t gbase = 0;  // position of the range group's first source in the unit's list
  for (int eg = e0; eg < e1; eg += kPLRanges) {
    const int nr = min(kPLRanges, e1 - eg);
    __syncthreads();  // previous users of rs/rpre are done
    const int total = pl_stage_ranges(rng, eg, nr, rs, rpre);
    constexpr int SPT = kPLChunk / kPLThreads;
    double gx[SPT], gy[SPT], gz[SPT], gq[SPT];
    int gi[SPT];
    auto fetch = [&](int c0) {
      const int n = min(kPLChunk, total - c0);
#pragma unroll
      for (int k = 0; k < SPT; ++k) {
        const int j = tid + k * kPLThreads;
        if (j < n) {
          const int sidx = pl_source(rs, rpre, nr, c0 + j);
          gx[k] = px[sidx];
          gy[k] = py[sidx];
          gz[k] = ph[sidx];
          gq[k] = qt[sidx];
          // where the source-side sum goes (positions after the leaf's own points)
          const int64_t pos = gbase + c0 + j - tc;
          gi[k] = pos >= 0 ? bidx[boff + pos] : 0;
        }
      }
    };
    if (total > 0) fetch(0);
    for (int c0 = 0; c0 < total; c0 += kPLChunk) {
      const int n = min(kPLChunk, total - c0);
      __syncthreads();
#pragma unroll
      for (int k = 0; k < SPT; ++k) {
        const int j = tid + k * kPLThreads;
        if (j < n) {
          V v;
          v.x = (T)(gx[k] - cx);
          v.y = (T)(gy[k] - cy);
          v.z = (T)(gz[k] - ch);
          v.w = (T)gq[k];
          src[j] = v;
          oidx[j] = gi[k];
        }
      }
      __syncthreads();
      if (c0 + kPLChunk < total) fetch(c0 + kPLChunk);
      // chunk sources [0, ns) are the leaf's own points (one way)
      const int64_t cg = gbase + c0;
      const int ns = (int)max<int64_t>(0, min<int64_t>(n, (int64_t)tc - cg));
      const int qn = (n + 3) >> 2;
      const int j0 = min(n, wave * qn), j1 = min(n, j0 + qn);
      T pp[TPL];
#pragma unroll
      for (int t = 0; t < TPL; ++t) pp[t] = T(0);
      const int ja = min(j1, ns), jb = max(j0, ns);
      if (j0 < ja) pl_range<T, TPL, true>(src, j0, ja, g, x, y, z, pp);
      if (jb < j1) pl_mrange<T, TPL, PLCfg<T, MT>::kNS>(src, jb, j1, g, sl, x, y, z, q, pp, oidx, bbuf);
#pragma unroll
      for (int t = 0; t < TPL; ++t) {
        if constexpr (sizeof(T) == 4)
          pl_neumaier(acc[t], cmp[t], pp[t]);
        else
          acc[t] += pp[t];
      }
    }
    gbase += total;
  }
#pragma unroll
  for (int t = 0; t < TPL; ++t) {
    double v = (double)acc[t] + (double)cmp[t];
    v = v + __shfl_xor(v, 16, 64);
    v = v + __shfl_xor(v, 32, 64);
    if (g == 0) red[wave * RW + sl + 16 * t] = v;
  }
  __syncthreads();
  if (tid < tcp) abuf[t0 + tb + tid] = (red[tid] + red[RW + tid]) + (red[2 * RW + tid] + red[3 * RW + tid]);
}

template <class T, int MT>
__global__ void __launch_bounds__(kPLThreads, (PLCfg<T, MT>::kWaves))
p2p_mutual_kernel(int64_t u0, const int32_t* __restrict__ mu_order, const int32_t* __restrict__ mu_leaf,
                  const int32_t* __restrict__ mu_tb,
                  const int32_t* __restrict__ mu_rptr, const int32_t* __restrict__ mu_rng,
                  const int64_t* __restrict__ mu_boff, const int32_t* __restrict__ mu_bidx,
                  const int32_t* __restrict__ leaves, const int32_t* __restrict__ bstart,
                  const int32_t* __restrict__ bcount, const double* __restrict__ bcx,
                  const double* __restrict__ bcy, const double* __restrict__ bch, const double* __restrict__ px,
                  const double* __restrict__ py, const double* __restrict__ ph, const double* __restrict__ qt,
                  double* __restrict__ abuf, T* __restrict__ bbuf) {
  using V = typename PLVec<T>::type;
  __shared__ V src[kPLChunk];
  __shared__ int oidx[kPLChunk];
  __shared__ int rs[kPLRanges], rpre[kPLRanges + 1];
  __shared__ double red[4 * 16 * MT];
  const int64_t u = mu_order[u0 + blockIdx.x];
  const int b = leaves[mu_leaf[u]];
  const int t0 = bstart[b], tc = bcount[b];
  const int tb = mu_tb[u], tcp = min(16 * MT, tc - tb);
  const int tpl = (tcp + 15) >> 4;
#define PM_CASE(k)                                                                                        \
  case k:                                                                                                 \
    if constexpr (k <= MT)                                                                                \
      pl_mpass<T, k, MT>(tb, tcp, t0, tc, bcx[b], bcy[b], bch[b], mu_rptr[u], mu_rptr[u + 1], mu_rng, px, py, \
                     ph, qt, mu_boff[u], mu_bidx, abuf, bbuf, src, oidx, rs, rpre, red);                  \
    break;
  switch (tpl) {
    PM_CASE(1) PM_CASE(2) PM_CASE(3) PM_CASE(4) PM_CASE(5) PM_CASE(6) PM_CASE(7) PM_CASE(8)
    default: break;
  }
#undef PM_CASE
}

// Per leaf: each point's target-side sum and its source-side rows, in row
// (unit) order, times 1/(4 pi), added to phin; rows 8 at a time (coalesced
// loads in flight).
constexpr int kCBThreads = 128;
template <class T>
__global__ void __launch_bounds__(kCBThreads)
p2p_combine_kernel(const int32_t* __restrict__ leaves, const int32_t* __restrict__ bstart,
                   const int32_t* __restrict__ bcount, const int64_t* __restrict__ cb_base,
                   const int32_t* __restrict__ cb_n, const double* __restrict__ abuf,
                   const T* __restrict__ bbuf, double* __restrict__ phin) {
  const int li = blockIdx.x;
  const int nrow = cb_n[li];
  if (nrow < 0) return;
  const int b = leaves[li];
  const int t0 = bstart[b], tc = bcount[b];
  const T* rows = bbuf + cb_base[li];
  for (int i = threadIdx.x; i < tc; i += kCBThreads) {
    double v = abuf[t0 + i];
    int k = 0;
    for (; k + 8 <= nrow; k += 8) {
      T w[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) w[r] = rows[(int64_t)(k + r) * tc + i];
#pragma unroll
      for (int r = 0; r < 8; ++r) v += (double)w[r];
    }
    for (; k < nrow; ++k) v += (double)rows[(int64_t)k * tc + i];
    phin[t0 + i] += v * kInv4Pi;
  }
}

// Batched free-space P2P on the matrix cores (FP32 form): per target leaf,
// Phi[t][v] += sum_s q[s][v] / |x_t - x_s| is a product of the kernel matrix
// K[t][s] (computed on the fly) and the charges q[s][v] of the 64 vectors.
// One workgroup (4 waves) per leaf; the leaf's sources are staged through LDS
// in chunks of kPBChunk as leaf-relative (x, y, h) and their 64 charges.  For
// v_mfma_f32_16x16x4f32, lane l computes the A entry K[target l % 16][source
// l / 16] (1/r in FP32, zero at zero distance: the self pair), and reads the B
// entry q[source l / 16][vector block + l % 16] from LDS.  Each wave owns
// two blocks of 16 targets (pass of 128 targets) x 4 blocks of 16 vectors;
// chunk sums from the matrix cores are combined by compensated summation.
constexpr int kPBChunk = 128;
__global__ void __launch_bounds__(256)
p2p_batch32_kernel(int g, const int32_t* __restrict__ pl_leaves, const int32_t* __restrict__ leaves,
                   const int32_t* __restrict__ bstart, const int32_t* __restrict__ bcount,
                   const double* __restrict__ bcx, const double* __restrict__ bcy, const double* __restrict__ bch,
                   const int32_t* __restrict__ ptr, const int32_t* __restrict__ rng, const double* __restrict__ px,
                   const double* __restrict__ py, const double* __restrict__ ph, const float* __restrict__ qb,
                   int64_t np, double* __restrict__ phit) {
  __shared__ float4 sx[kPBChunk];
  __shared__ float sq[kPBChunk * 64];
  __shared__ int rs[kPLRanges], rpre[kPLRanges + 1];
  const int li = pl_leaves[blockIdx.x];
  const int b = leaves[li];
  const int t0 = bstart[b], tc = bcount[b];
  const double cx = bcx[b], cy = bcy[b], ch = bch[b];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int l16 = lane & 15, lk = lane >> 4;
  const int e0 = ptr[li], e1 = ptr[li + 1];
  for (int tp = 0; tp < tc; tp += 128) {
    // this wave's two target blocks: tp + 16 (2 wave + u), u = 0, 1
    float tx[2], ty[2], tz[2];
    bool tok[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int t = tp + 16 * (2 * wave + u) + l16;
      tok[u] = t < tc;
      tx[u] = tok[u] ? (float)(px[t0 + t] - cx) : 0.f;
      ty[u] = tok[u] ? (float)(py[t0 + t] - cy) : 0.f;
      tz[u] = tok[u] ? (float)(ph[t0 + t] - ch) : 0.f;
    }
    const bool active = tp + 32 * wave < tc;  // uniform per wave
    floatx4 part[2][4], acc[2][4], cmp[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        part[u][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        acc[u][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        cmp[u][j] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
    for (int eg = e0; eg < e1; eg += kPLRanges) {
      const int nr_ = min(kPLRanges, e1 - eg);
      __syncthreads();
      const int total = pl_stage_ranges(rng, eg, nr_, rs, rpre);
      for (int c0 = 0; c0 < total; c0 += kPBChunk) {
        const int n = min(kPBChunk, total - c0);
        __syncthreads();
        for (int j = tid; j < kPBChunk; j += 256) {
          float4 v = make_float4(0.f, 0.f, 0.f, -1.f);  // w < 0: padding (no source)
          if (j < n) {
            const int sidx = pl_source(rs, rpre, nr_, c0 + j);
            v = make_float4((float)(px[sidx] - cx), (float)(py[sidx] - cy), (float)(ph[sidx] - ch), 1.f);
          }
          sx[j] = v;
        }
        for (int i = tid; i < kPBChunk * 16; i += 256) {
          const int j = i >> 4, c4 = (i & 15) * 4;
          float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
          if (j < n) {
            const int sidx = pl_source(rs, rpre, nr_, c0 + j);
            v = *reinterpret_cast<const float4*>(qb + (int64_t)sidx * 64 + c4);
          }
          *reinterpret_cast<float4*>(sq + j * 64 + c4) = v;
        }
        __syncthreads();
        if (active) {
          for (int ks = 0; ks < n; ks += 4) {
            const float4 sv = sx[ks + lk];
            float a[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const float dx = tx[u] - sv.x, dy = ty[u] - sv.y, dz = tz[u] - sv.z;
              const float r2 = dx * dx + dy * dy + dz * dz;
              a[u] = (sv.w > 0.f && r2 > 0.f) ? __builtin_amdgcn_rsqf(r2) : 0.f;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const float bq = sq[(ks + lk) * 64 + 16 * j + l16];
#pragma unroll
              for (int u = 0; u < 2; ++u)
                part[u][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], bq, part[u][j], 0, 0, 0);
            }
          }
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const float x = part[u][j][v], a0 = acc[u][j][v], t = a0 + x;
                cmp[u][j][v] += (fabsf(a0) >= fabsf(x)) ? (a0 - t) + x : (x - t) + a0;
                acc[u][j][v] = t;
              }
              part[u][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
        }
      }
    }
    if (active) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int col = 16 * j + l16;  // vector
          if (col >= g) continue;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int t = tp + 16 * (2 * wave + u) + 4 * lk + v;
            if (t < tc)
              phit[(int64_t)col * np + t0 + t] += ((double)acc[u][j][v] + (double)cmp[u][j][v]) * kInv4Pi;
          }
        }
    }
  }
}


// Reaction near field (polarization-source P2P), phi_i += sum_j K_ij q_j with
// the stored kernel values of each entry (a target leaf, a source range).  The
// dot products are spread over the GPU: a wave takes kRPUnitRows rows of one
// entry, 8 lanes a row, and stores each row's sum in the entry's partial-sum
// slot; a second kernel adds a leaf's partials to its targets, in entry order.
constexpr int kRPThreads = 256;
static_assert(kRPUnitRows == 8, "a wave holds 8 rows of 8 lanes");
// TV: the stored values' type (FP64, or FP32 in the FP32 form); products and
// sums in FP64
template <class TV>
__global__ void __launch_bounds__(kRPThreads)
p2p_reaction_rows_kernel(int64_t nunits, const int32_t* __restrict__ units, const int32_t* __restrict__ rng,
                         const int64_t* __restrict__ voff, const int32_t* __restrict__ rowoff,
                         const TV* __restrict__ val, const double* __restrict__ qt,
                         double* __restrict__ part) {
  const int64_t u = (int64_t)blockIdx.x * (kRPThreads / 64) + (threadIdx.x >> 6);
  if (u >= nunits) return;  // whole waves
  const int e = units[3 * u], ti = units[3 * u + 1] + ((threadIdx.x & 63) >> 3), tc = units[3 * u + 2];
  const int l8 = threadIdx.x & 7;
  const int s0 = rng[2 * e], sc = rng[2 * e + 1];
  const TV* row = val + voff[e] + (int64_t)min(ti, tc - 1) * sc;
  const double* qs = qt + s0;
  double a0 = 0.0, a1 = 0.0;
  int j = l8;
  for (; j + 8 < sc; j += 16) {
    a0 = fma((double)row[j], qs[j], a0);
    a1 = fma((double)row[j + 8], qs[j + 8], a1);
  }
  if (j < sc) a0 = fma((double)row[j], qs[j], a0);
  double a = a0 + a1;
  a += __shfl_xor(a, 4, 8);
  a += __shfl_xor(a, 2, 8);
  a += __shfl_xor(a, 1, 8);
  if (l8 == 0 && ti < tc) part[rowoff[e] + ti] = a;
}

__global__ void __launch_bounds__(kRPThreads)
p2p_reaction_sum_kernel(const int32_t* __restrict__ leaves, const int32_t* __restrict__ bstart,
                        const int32_t* __restrict__ bcount, const int32_t* __restrict__ ptr,
                        const int32_t* __restrict__ rowoff, const double* __restrict__ part,
                        double* __restrict__ phit) {
  const int lf = blockIdx.x;
  const int e0 = ptr[lf], e1 = ptr[lf + 1];
  if (e0 == e1) return;
  const int b = leaves[lf];
  const int t0 = bstart[b], tc = bcount[b];
  for (int i = threadIdx.x; i < tc; i += kRPThreads) {
    double acc = 0.0;
    for (int e = e0; e < e1; ++e) acc += part[rowoff[e] + i];
    phit[t0 + i] += acc;
  }
}

}  // namespace

int gpu_build_ops(fmmlm_plan_s* P, const std::vector<int>& free_r2dz, const std::vector<SommTask>& tasks,
                  const std::vector<int>& dirs, const double* d_tables, hipStream_t st) {
  const int64_t nfree = P->ng_free, nreac = P->ng_ops - nfree;
  const int p2 = 2 * P->p;
  const size_t ni = free_r2dz.size() + dirs.size();
  int* di = nullptr;
  double* dS = nullptr;
  if (ni > 0) {
    std::vector<int> hi(free_r2dz);
    hi.insert(hi.end(), dirs.begin(), dirs.end());
    FMM_HIP_TRY(hipMalloc(&di, ni * sizeof(int)));
    hipError_t e = hipMemcpyAsync(di, hi.data(), ni * sizeof(int), hipMemcpyHostToDevice, st);
    if (e == hipSuccess && nfree > 0) {
      const int64_t tot = nfree * P->ngs;
      build_free_ops_kernel<<<(unsigned)((tot + 255) / 256), 256, 0, st>>>(di, nfree, P->ngs, P->coefA, P->G);
      e = hipGetLastError();
    }
    if (e == hipSuccess && P->n_phi > 0) {
      const int64_t tot = P->n_phi * (p2 + 1);
      build_phases_kernel<<<(unsigned)((tot + 255) / 256), 256, 0, st>>>(di + free_r2dz.size(), P->n_phi, p2,
                                                                        reinterpret_cast<cplx*>(P->E));
      e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(di);
    FMM_HIP_TRY(e);
  }
  if (nreac > 0) {
    std::vector<double> S;
    for (const SommTask& t : tasks) S.push_back(t.S);
    FMM_HIP_TRY(hipMalloc(&dS, nreac * sizeof(double)));
    hipError_t e = hipMemcpyAsync(dS, S.data(), nreac * sizeof(double), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) {
      const int64_t tot = nreac * P->ngs;
      build_reaction_ops_kernel<<<(unsigned)((tot + 255) / 256), 256, 0, st>>>(
          dS, nreac, P->ng, P->ngs, P->coefA, d_tables, P->G + nfree * P->ngs);
      e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(dS);
    FMM_HIP_TRY(e);
  }
  return FMMLM_OK;
}

namespace {
// 16-row blocks of the two frame matrices
struct FrameRows {
  int nc, ns, rc, rs;
};
FrameRows frame_rows(int p) {
  const int nc = ncoef(p), ns = nc - p - 1;
  return FrameRows{nc, ns, (nc + 15) / 16, (ns + 15) / 16};
}
}  // namespace

int64_t frame_op_len(int p, int64_t* row_len) {
  const FrameRows r = frame_rows(p);
  const int64_t rt = 16 * (r.rc + r.rs);
  if (row_len) *row_len = rt;
  return 4 * frame_ksteps(r.nc) * rt;
}

int gpu_build_frame_ops(fmmlm_plan_s* P, M2LUnits& U, bool f32, hipStream_t st) {
  const FrameRows r = frame_rows(P->p);
  int64_t rt = 0;
  const int64_t tot = U.nops * frame_op_len(P->p, &rt);
  if (tot == 0) return FMMLM_OK;
  const unsigned nb = (unsigned)((tot + 255) / 256);
  if (f32)
    build_frame_ops_kernel<<<nb, 256, 0, st>>>(P->p, r.nc, r.ns, r.rc, (int)rt, frame_ksteps(r.nc), U.nops,
                                               P->ng_free, U.frame_op, P->pair_dec, P->G, P->ngs, P->coefA,
                                               static_cast<float*>(U.A));
  else
    build_frame_ops_kernel<<<nb, 256, 0, st>>>(P->p, r.nc, r.ns, r.rc, (int)rt, frame_ksteps(r.nc), U.nops,
                                               P->ng_free, U.frame_op, P->pair_dec, P->G, P->ngs, P->coefA,
                                               static_cast<double*>(U.A));
  FMM_HIP_TRY(hipGetLastError());
  return FMMLM_OK;
}

int gpu_build_xlate_ops(fmmlm_plan_s* P, hipStream_t st) {
  const int mr = 32 * P->mrt, nr = (P->p + 1) * (P->p + 1);
  FMM_HIP_TRY(hipMemsetAsync(P->Txl, 0, (size_t)16 * P->nrk * mr * sizeof(double), st));
  build_xlate_ops_kernel<<<dim3((unsigned)nr, 16), 64, 2 * P->nc * sizeof(cplx), st>>>(P->p, P->nrk, mr, P->coefA,
                                                                                        P->Txl);
  FMM_HIP_TRY(hipGetLastError());
  return FMMLM_OK;
}

__global__ void round_f32_kernel(const double* __restrict__ a, int64_t n, float* __restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = (float)a[i];
}

int gpu_round_f32(const double* a, int64_t n, float* b, hipStream_t st) {
  if (n <= 0) return FMMLM_OK;
  round_f32_kernel<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(a, n, b);
  FMM_HIP_TRY(hipGetLastError());
  return FMMLM_OK;
}

// One wave per work unit of the reaction near field (rows of one entry): the
// pairs' indices in rp_val's order.  Bound by its 12 bytes a pair of writes;
// listing 12.1 M pairs on the host and copying the lists (145 MB) took
// about 65 ms of a plan; the launch takes 0.025 ms.
__global__ void __launch_bounds__(256)
expand_pairs_kernel(int64_t nunits, const int32_t* __restrict__ units, const int32_t* __restrict__ rng,
                    const int64_t* __restrict__ voff, const int32_t* __restrict__ tgt0,
                    const int32_t* __restrict__ comp, int32_t* __restrict__ tpt, int32_t* __restrict__ spt,
                    int32_t* __restrict__ cmp) {
  const int64_t u = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (u >= nunits) return;
  const int lane = threadIdx.x & 63;
  const int e = units[3 * u], r0 = units[3 * u + 1], r1 = min(r0 + kRPUnitRows, units[3 * u + 2]);
  const int s0 = rng[2 * e], sc = rng[2 * e + 1], t0 = tgt0[e], c = comp[e];
  for (int i = r0; i < r1; ++i) {
    const int64_t v = voff[e] + (int64_t)i * sc;
    for (int j = lane; j < sc; j += 64) {
      tpt[v + j] = t0 + i;
      spt[v + j] = s0 + j;
      cmp[v + j] = c;
    }
  }
}

int gpu_expand_pairs(fmmlm_plan_s* P, const std::vector<int32_t>& tgt0, const std::vector<int32_t>& comp,
                     int32_t* tpt, int32_t* spt, int32_t* cmp, hipStream_t st) {
  if (P->n_rp_units == 0) return FMMLM_OK;
  const size_t n = tgt0.size();
  int32_t* d = nullptr;
  FMM_HIP_TRY(hipMalloc(&d, 2 * n * sizeof(int32_t)));
  hipError_t e = hipMemcpyAsync(d, tgt0.data(), n * sizeof(int32_t), hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipMemcpyAsync(d + n, comp.data(), n * sizeof(int32_t), hipMemcpyHostToDevice, st);
  if (e == hipSuccess) {
    expand_pairs_kernel<<<(unsigned)((P->n_rp_units + 3) / 4), 256, 0, st>>>(P->n_rp_units, P->rp_units, P->rp_src,
                                                                           P->rp_voff, d, d + n, tpt, spt, cmp);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  (void)hipFree(d);
  if (e != hipSuccess) {
    set_last_error(std::string("reaction near-field pairs: ") + hipGetErrorString(e));
    return FMMLM_EDEVICE;
  }
  return FMMLM_OK;
}

int gpu_build_fp32(fmmlm_plan_s* P, hipStream_t st) {
  const unsigned nb = (unsigned)((P->NP + 255) / 256);
  split_f32_kernel<<<nb, 256, 0, st>>>(P->px, P->NP, P->pxh, P->pxl);
  split_f32_kernel<<<nb, 256, 0, st>>>(P->py, P->NP, P->pyh, P->pyl);
  split_f32_kernel<<<nb, 256, 0, st>>>(P->ph, P->NP, P->phh, P->phl);
  FMM_HIP_TRY(hipGetLastError());
  FMM_HIP_TRY(hipStreamSynchronize(st));
  return FMMLM_OK;
}

// The M2L units of one precision.  Variant v: operator batches of 4, 2 or 8
// k-steps (v % 3), from v = 3 on with LDS reserved so that two blocks fit a CU
// (room for the near field's blocks); every variant gives the same sums.
template <class T, int KB>
int launch_frame_kb(const fmmlm_plan_s* P, const M2LUnits& U, size_t reserve, unsigned parts, const double* M,
                    hipStream_t st) {
  const FrameRows r = frame_rows(P->p);
#define FR(RC, RS)                                                                                             \
  if (r.rc == RC && r.rs == RS) {                                                                              \
    const size_t used = (size_t)(2 * KB * 4 * 16 * (RC + RS)) * sizeof(T) + 1024;                              \
    const size_t es = (size_t)(P->p + 1) * kFrCols * sizeof(cplx);                                             \
    m2l_frame_kernel<T, RC, RS, KB><<<(unsigned)U.n, 256, std::max(es, reserve > used ? reserve - used : 0), st>>>( \
        (P->p + 1) * (P->p + 1), r.nc, r.ns, 2 * P->p + 1, P->nrk, U.step0, U.kind, U.phi, U.op, U.src,        \
        P->pair_dec, parts, static_cast<const T*>(U.A), M, reinterpret_cast<const cplx*>(P->E),                \
        static_cast<T*>(U.W));                                                                                 \
    FMM_HIP_TRY(hipGetLastError());                                                                            \
    return FMMLM_OK;                                                                                           \
  }
  if constexpr (KB == 4) {  // p = 1..16
    FR(1, 1) FR(2, 1) FR(2, 2) FR(3, 2)
  }
  if constexpr (KB == 2 || sizeof(T) == 4) {  // the tuner's orders (m2l_variants)
    FR(3, 3) FR(4, 3) FR(5, 4)
  }
  if constexpr (KB == (sizeof(T) == 8 ? 2 : 4)) {
    FR(5, 5) FR(6, 5) FR(7, 6)
  }
  if constexpr (KB == 2) {
    FR(8, 7) FR(9, 8) FR(10, 9)
  }
#undef FR
  return FMMLM_EUNSUPPORTED;
}

template <class T>
int launch_frame(const fmmlm_plan_s* P, const M2LUnits& U, int variant, unsigned parts, const double* M,
                 hipStream_t st) {
  if (U.n <= 0) return FMMLM_OK;
  const size_t reserve = variant >= 3 ? 61440 : 0;
  // k-steps of a batch, at 262,144 charges, leaf cap 64, launch in ms with 2 / 4.
  // FP64 from p = 8 on 2, which leaves registers for a third wave a SIMD: p = 8
  // 0.378 / 0.409, 10 0.727 / 0.818, 12 1.086 / 1.220, 13 1.569 / 1.516; below p = 8
  // 4 (p = 6 0.198 / 0.204, 7 0.279 / 0.298; up to p = 5 a batch of 2 has no room for
  // the epilogue's rows).  FP32 from p = 14 on 2 (14 0.885 / 0.935, 16 1.414 / 1.591),
  // at the orders with variants the tuner's choice (8 0.188 / 0.203, 9 0.242 / 0.277,
  // 10 0.375 / 0.379), elsewhere 4 (6 0.107 / 0.115, 7 0.143 / 0.188, 11 0.450 /
  // 0.432, 12 0.554 / 0.545, 13 0.704 / 0.774)
  if (P->p > 13 || (sizeof(T) == 8 && P->p >= 8)) return launch_frame_kb<T, 2>(P, U, 0, parts, M, st);
  switch (variant % 3) {  // (0 where there are no variants)
    case 1: return launch_frame_kb<T, 2>(P, U, reserve, parts, M, st);
    case 2: return launch_frame_kb<T, 8>(P, U, reserve, parts, M, st);
    default: return launch_frame_kb<T, 4>(P, U, reserve, parts, M, st);
  }
}

template <class T>
int launch_frame_reduce(const fmmlm_plan_s* P, const M2LUnits& U, double* Lx, hipStream_t st) {
  if (U.nboxes <= 0) return FMMLM_OK;
  const FrameRows r = frame_rows(P->p);
#define FRR(NT)                                                                                               \
  m2l_frame_reduce_kernel<T, NT><<<(unsigned)U.nboxes, NT, 0, st>>>(                                          \
      (P->p + 1) * (P->p + 1), r.nc, r.ns, 2 * P->p + 1, P->nrk, U.boxes, U.ptr, U.slots, U.slot_phi,         \
      P->pair_dec, P->blevel, P->sc_levels, static_cast<const T*>(U.W), reinterpret_cast<const cplx*>(P->E), Lx)
  // few boxes (long slot lists, top levels): more groups a box, 512 threads, from p = 10
  // on (7 groups and fewer at 512) 1,024.  This launch, FP64, us, with 256 / 512 / 1,024
  // threads, 227 boxes in the tree: p = 5 11.1 / 8.8 / 8.0, 8 18.6 / 12.7 / 10.0, 10 26.3 /
  // 15.9 / 11.8, 16 69.5 / 32.4 / 21.5; 1,897 boxes: p = 2 - / 10.4 / 15.3, 5 13.8 / 13.2 / 16.8,
  // 8 22.8 / 19.0 / 20.0, 10 32.4 / 24.0 / 23.9, 16 116 / 66 / 58.  More boxes, with 256 / 512:
  // 4,526 p = 5 14.4 / 16.2, 8 24.5 / 22.5, 10 35.4 / 28.5; 11,810 p = 5 36.0 / 43.7, 8 86.4 /
  // 89.9, 10 131 / 125: the line is where p = 5 starts to lose.  Top levels beside an FP32
  // launch keep 512: blocks of 16 waves wait for room there (six layers, 524,288 charges,
  // 1,598 against 1,610 us an evaluation)
  const bool beside = P->fp32 && P->u32.n > 0;
  if (U.nboxes < 2048 && r.nc > 64 && !beside) {
    FRR(1024);
  } else if (U.nboxes < 2048) {
    FRR(512);
  } else {
    FRR(256);
  }
#undef FRR
  FMM_HIP_TRY(hipGetLastError());
  return FMMLM_OK;
}

int m2l_variants(const fmmlm_plan_s* P) { return P->mrt == 4 ? kM2LVariants : 1; }

// Autotuner of the FP32 M2L launch: every variant runs the plan's own
// units (sources cleared) once to warm up and three times timed with HIP
// events; the fastest is kept.  Times go to the plan's stats.
int gpu_tune_m2l(fmmlm_plan_s* P, hipStream_t st) {
  P->m2l_variant = 0;
  const int nv = m2l_variants(P);
  if (!P->fp32 || P->u32.n <= 0 || nv < 2) return FMMLM_OK;
  const int64_t nr = (int64_t)(P->p + 1) * (P->p + 1);
  FMM_HIP_TRY(hipMemsetAsync(P->M, 0, (size_t)(P->NB * nr) * sizeof(double), st));
  hipEvent_t e0, e1;
  FMM_HIP_TRY(hipEventCreate(&e0));
  FMM_HIP_TRY(hipEventCreate(&e1));
  int rc = FMMLM_OK;
  double best = 1e300;
  for (int v = 0; v < nv && rc == FMMLM_OK; ++v) {
    double tmin = 1e300;
    for (int rep = 0; rep < 4 && rc == FMMLM_OK; ++rep) {
      (void)hipEventRecord(e0, st);
      rc = launch_frame<float>(P, P->u32, v, FMMLM_FREE | FMMLM_REACTION, P->M, st);
      (void)hipEventRecord(e1, st);
      if (rc) break;
      if (hipEventSynchronize(e1) != hipSuccess) {
        rc = FMMLM_EDEVICE;
        break;
      }
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, e0, e1);
      if (rep > 0) tmin = std::min(tmin, (double)ms);
    }
    if (v < kM2LVariants) P->stats.m2l_variant_ms[v] = tmin;
    if (tmin < best) {
      best = tmin;
      P->m2l_variant = v;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  P->stats.m2l_variant = P->m2l_variant;
  return rc;
}

// Second stage of the FP32 M2L choice: the main M2L shares the GPU with the
// near field and the FP64 top levels in an unprofiled evaluation, so the
// variant that is fastest alone need not be fastest there.  Every variant times
// whole evaluations (zero charges: the arithmetic does not depend on them),
// one to warm up and three timed; the fastest evaluation decides.  Then the
// same timing picks how much of the free P2P starts at the fork, the rest
// following the main M2L launch.
int gpu_tune_eval(fmmlm_plan_s* P, hipStream_t st) {
  const int nv = m2l_variants(P);
  if (!P->fp32 || P->u32.n <= 0) return FMMLM_OK;
  double *q = nullptr, *phi = nullptr;
  FMM_HIP_TRY(hipMalloc(&q, (size_t)P->N * sizeof(double)));
  if (hipMalloc(&phi, (size_t)P->N * sizeof(double)) != hipSuccess) {
    (void)hipFree(q);
    return FMMLM_ENOMEM;
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  int rc = FMMLM_OK;
  if (hipMemsetAsync(q, 0, (size_t)P->N * sizeof(double), st) != hipSuccess || hipEventCreate(&e0) != hipSuccess ||
      hipEventCreate(&e1) != hipSuccess)
    rc = FMMLM_EDEVICE;
  // best of three whole evaluations after one to warm up
  auto time_evals = [&]() -> double {
    double tmin = 1e300;
    for (int rep = 0; rep < 4 && rc == FMMLM_OK; ++rep) {
      (void)hipEventRecord(e0, st);
      rc = gpu_eval_one(P, q, phi, FMMLM_FREE | FMMLM_REACTION, st, nullptr);
      (void)hipEventRecord(e1, st);
      if (rc) break;
      if (hipEventSynchronize(e1) != hipSuccess) {
        rc = FMMLM_EDEVICE;
        break;
      }
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, e0, e1);
      if (rep > 0) tmin = std::min(tmin, (double)ms);
    }
    return tmin;
  };
  // the main M2L's variant, with the whole free P2P at the fork
  P->pl_split = P->n_mu_units;
  double best = 1e300;
  int pick = P->m2l_variant;
  for (int v = 0; v < nv && nv > 1 && rc == FMMLM_OK; ++v) {
    P->m2l_variant = v;
    const double t = time_evals();
    if (v < kM2LVariants) P->stats.m2l_eval_ms[v] = t;
    if (t < best) {
      best = t;
      pick = v;
    }
  }
  P->m2l_variant = pick;
  P->stats.m2l_variant = pick;
  // then the share of the free P2P launched at the fork (the rest follows the
  // main M2L)
  static constexpr int kSplitPct[5] = {100, 75, 50, 25, 0};
  best = 1e300;
  int pct = 100;
  for (int i = 0; i < 5 && rc == FMMLM_OK; ++i) {
    P->pl_split = P->n_mu_units * kSplitPct[i] / 100;
    const double t = time_evals();
    P->stats.p2p_split_ms[i] = t;
    if (t < best) {
      best = t;
      pct = kSplitPct[i];
    }
  }
  P->pl_split = P->n_mu_units * pct / 100;
  P->stats.p2p_split_pct = pct;
  // then the LDS the P2P blocks reserve
  best = 1e300;
  size_t pad = P->pl_pad;
  for (int i = 0; i < 3 && rc == FMMLM_OK; ++i) {
    P->pl_pad = kPLPads[i];
    const double t = time_evals();
    P->stats.p2p_reserve_ms[i] = t;
    if (t < best) {
      best = t;
      pad = kPLPads[i];
    }
  }
  P->pl_pad = pad;
  P->stats.p2p_lds_reserve = (int32_t)pad;
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(q);
  (void)hipFree(phi);
  return rc;
}

// Batched M2L in operator frames over n boxes (or items) of one precision.
// Variant v: operator batches of 4, 2 or 8 k-steps, or of 4 or 2 with LDS reserved
// so that two blocks fit a CU (v % kBatchShapes), boxes in XCD-contiguous order
// (v < kBatchShapes) or as they come.
int batch_variants(const fmmlm_plan_s* P) { return P->mrt == 4 ? 2 * kBatchShapes : 2; }

template <class T, int KB>
int launch_frame_batch_kb(const fmmlm_plan_s* P, const M2LUnits& U, int g, int64_t n, const int32_t* boxes,
                          const int32_t* items, bool swizzle, size_t reserve, unsigned parts, const T* X,
                          double* part, hipStream_t st) {
  const FrameRows r = frame_rows(P->p);
  const int64_t slab = P->NB * (int64_t)(P->p + 1) * (P->p + 1);
  const unsigned nb = (unsigned)(swizzle ? 8 * (int64_t)P->bbox_xcd_len : n);
#define FB(RC, RS)                                                                                              \
  if (r.rc == RC && r.rs == RS) {                                                                               \
    const size_t used = (size_t)(2 * KB * 4 * 16 * (RC + RS)) * sizeof(T) + 1024;                               \
    m2l_frame_batch_kernel<T, RC, RS, KB><<<nb, 256, reserve > used ? reserve - used : 0, st>>>(                \
        (P->p + 1) * (P->p + 1), r.nc, r.ns, 2 * P->p + 1, g, P->gw, slab, n, swizzle ? 1 : 0, P->bbox_xcd, boxes, items, \
        U.bptr, U.box0, U.be_op, U.be_phi, U.be_src, U.be_kind, P->pair_dec, parts,                             \
        static_cast<const T*>(U.A), X, reinterpret_cast<const cplx*>(P->E), P->blevel, P->sc_levels, P->Lx,     \
        part);                                                                                                  \
    FMM_HIP_TRY(hipGetLastError());                                                                             \
    return FMMLM_OK;                                                                                            \
  }
  if constexpr (sizeof(T) == 4) {
    if constexpr (KB == 4) {  // p = 1..16
      FB(1, 1) FB(2, 1) FB(2, 2) FB(3, 2) FB(5, 5) FB(6, 5) FB(7, 6)
    }
    FB(3, 3) FB(4, 3) FB(5, 4)  // the tuner's orders (batch_variants)
    if constexpr (KB == 2) {
      FB(8, 7) FB(9, 8) FB(10, 9)
    }
  } else if constexpr (KB == 2) {  // (launch_batch64)
    FB(1, 1) FB(4, 3) FB(5, 4) FB(5, 5) FB(6, 5) FB(7, 6) FB(8, 7) FB(9, 8) FB(10, 9)
  } else if constexpr (KB == 3) {
    FB(1, 1) FB(2, 1) FB(3, 2)
  } else {
    FB(1, 1) FB(2, 2) FB(3, 3)
  }
#undef FB
  return FMMLM_EUNSUPPORTED;
}

int launch_batch32(const fmmlm_plan_s* P, int variant, int g, int64_t n, unsigned parts, hipStream_t st) {
  if (n <= 0) return FMMLM_OK;
  const int nv = P->mrt == 4 ? kBatchShapes : 1;
  const bool sw = variant < nv;
  const int32_t* bx = P->bbox + P->bbox_split;
  const int shape = variant % nv;
  const size_t reserve = shape >= 3 ? 61440 : 0;
  // k-steps of a batch at the orders without variants, launch in ms with 2 / 4 at
  // 131,072 charges, 64 vectors, leaf cap 64: 4 up to p = 13 (p = 4 2.94 / 2.67, 5
  // 5.07 / 5.00, 6 7.34 / 6.22, 7 10.0 / 10.5, 11 44.1 / 36.9, 12 54.6 / 46.2, 13
  // 67.8 / 62.2); from p = 14 on, where they are equal (60,000 charges: 14 26.0 / 26.0,
  // 16 51.1 / 50.9), 2 for its smaller LDS
  if (P->p > 13) return launch_frame_batch_kb<float, 2>(P, P->u32, g, n, bx, nullptr, sw, 0, parts, P->M32, nullptr, st);
  if (shape == 1 || shape == 4)
    return launch_frame_batch_kb<float, 2>(P, P->u32, g, n, bx, nullptr, sw, reserve, parts, P->M32, nullptr, st);
  if (shape == 2)
    return launch_frame_batch_kb<float, 8>(P, P->u32, g, n, bx, nullptr, sw, 0, parts, P->M32, nullptr, st);
  return launch_frame_batch_kb<float, 4>(P, P->u32, g, n, bx, nullptr, sw, reserve, parts, P->M32, nullptr, st);
}

// The batched M2L in FP64: n boxes, or n work items.  Up to p = 8 an entry's k-steps go
// in as few batches as batches of at most 4 allow, evenly (p = 3, 5, 7: 3; 4, 6, 8: 4):
// with batches of 2 the barriers and the turn back kept it behind the dense operators,
// which fit their tiles at p = 3 and 7.  M2L of 6,000 charges' 64 vectors, us, dense / 2 /
// these: p = 3 216 / 292 / 211, 5 628 / 516 / 460, 7 851 / 961 / 797, 8 2051 / 1224 / 977;
// p = 9 2394 / 1586 / 1595 (4), so from there on 2 and its registers.
int launch_batch64(const fmmlm_plan_s* P, int g, int64_t n, const int32_t* items, unsigned parts, double* part,
                   hipStream_t st) {
  const int kc = frame_ksteps(P->nc), batches = (kc + 3) / 4, kb = (kc + batches - 1) / batches;
  if (P->p > 8 || kb <= 2)
    return launch_frame_batch_kb<double, 2>(P, P->u64, g, n, P->bbox, items, false, 0, parts, P->M64, part, st);
  if (kb == 3)
    return launch_frame_batch_kb<double, 3>(P, P->u64, g, n, P->bbox, items, false, 0, parts, P->M64, part, st);
  return launch_frame_batch_kb<double, 4>(P, P->u64, g, n, P->bbox, items, false, 0, parts, P->M64, part, st);
}

// Autotuner of the batched FP32 M2L: each variant runs the plan's boxes for
// the plan's G vectors (operands cleared) once to warm up and twice timed; the
// fastest is kept.  Times go to the plan's stats.
int gpu_tune_batch(fmmlm_plan_s* P, hipStream_t st) {
  P->batch_variant = 0;
  const int64_t n32 = P->nbbox - P->bbox_split;
  const int nv = batch_variants(P);
  if (!P->fp32 || P->gmax < 2 || n32 <= 0) return FMMLM_OK;
  FMM_HIP_TRY(hipMemsetAsync(P->M32, 0, (size_t)P->NB * P->nc * P->gw * 2 * sizeof(float), st));
  hipEvent_t e0, e1;
  FMM_HIP_TRY(hipEventCreate(&e0));
  FMM_HIP_TRY(hipEventCreate(&e1));
  int rc = FMMLM_OK;
  double best = 1e300;
  for (int v = 0; v < nv && rc == FMMLM_OK; ++v) {
    double tmin = 1e300;
    for (int rep = 0; rep < 3 && rc == FMMLM_OK; ++rep) {
      (void)hipEventRecord(e0, st);
      rc = launch_batch32(P, v, P->gmax, n32, FMMLM_FREE | FMMLM_REACTION, st);
      (void)hipEventRecord(e1, st);
      if (rc) break;
      if (hipEventSynchronize(e1) != hipSuccess) {
        rc = FMMLM_EDEVICE;
        break;
      }
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, e0, e1);
      if (rep > 0) tmin = std::min(tmin, (double)ms);
    }
    if (v < 2 * kBatchShapes) P->stats.batch_variant_ms[v] = tmin;
    if (tmin < best) {
      best = tmin;
      P->batch_variant = v;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  P->stats.batch_variant = P->batch_variant;
  return rc;
}

// M2M (up = true, into M) or L2L (into Lx) of one level through the
// translation tiles of 32 target boxes (M2M: parents, one unit per child
// octant present; L2L: children of one octant, one unit), one launch of
// xlate_direct_kernel a level.
int launch_xlate_level(const fmmlm_plan_s* P, const std::array<int64_t, 4>& r, bool up, double* M, double* Lx,
                       hipStream_t st) {
  const int64_t nt = r[2] - r[0], nu = r[3] - r[1];
  if (nt <= 0 || nu <= 0) return FMMLM_OK;
  const int mr = 32 * P->mrt, nr = (P->p + 1) * (P->p + 1);
  // an L2L level's i-th unit is its i-th tile (the plan adds them together)
  if ((!up && nt != nu) || P->xl_tile_cols != 32) {
    set_last_error("internal: translation tiles do not match the kernel");
    return FMMLM_EUNSUPPORTED;
  }
  const unsigned nrb = (unsigned)((nr + 15) / 16);
  if (up)
    xlate_direct_kernel<true><<<dim3((unsigned)nt, nrb, 2), 512, 0, st>>>(
        nr, P->nrk, mr, r[0], r[1], P->xl_tile_unit_ptr, P->xl_unit_s, P->xl_step_op, P->xl_step_src,
        P->xl_unit_mask, P->xl_tile_tgt, P->Txl, M, M);
  else
    xlate_direct_kernel<false><<<dim3((unsigned)nu, (nrb + 7) / 8, 2), 512, 0, st>>>(
        nr, P->nrk, mr, r[0], r[1], P->xl_tile_unit_ptr, P->xl_unit_s, P->xl_step_op, P->xl_step_src,
        P->xl_unit_mask, P->xl_tile_tgt, P->Txl, Lx, Lx);
  return FMMLM_OK;
}

// The batched translations over an entry list: targets boxes[b0, b0 + nb), per
// target the entries [ptr[b], ptr[b + 1]) of (source box, operator of T);
// dst[vector][box] += sum of T[op] X[vector][source].
int launch_xlate_batch(const fmmlm_plan_s* P, int g, const int32_t* boxes, int64_t b0, int64_t nb,
                        const int32_t* ptr, const int32_t* src, const int32_t* op, const double* T,
                        const double* X, double* dst, hipStream_t st) {
  if (nb <= 0) return FMMLM_OK;
  const int nr = (P->p + 1) * (P->p + 1);
  switch (P->mrt) {
#define BL(R)                                                                                                \
  case R:                                                                                                    \
    xlate_batch_kernel<R><<<(unsigned)nb, 256, 0, st>>>(nr, P->nrk, g, P->NB, boxes, b0, ptr, src, op, T, X, dst); \
    break;
    BL(2) BL(4) BL(6) BL(8) BL(10)
#undef BL
    default:
      return FMMLM_EUNSUPPORTED;
  }
  FMM_HIP_TRY(hipGetLastError());
  return FMMLM_OK;
}

int gpu_eval_batch(fmmlm_plan_s* P, int g, const double* q, int64_t ldq, double* phi, int64_t ldphi,
                   uint32_t parts, hipStream_t st, hipEvent_t* ev) {
  int stage = 0;
  auto mark = [&]() {
    if (ev) (void)hipEventRecord(ev[stage], st);
    ++stage;
  };
  const int p = P->p, nc = P->nc;
  const int nr = (p + 1) * (p + 1);
  const int64_t slab = P->NB * (int64_t)nr;
  const bool f32 = P->fp32;
  mark();
  transpose_users_kernel<<<(unsigned)((P->N + 63) / 64), 256, 0, st>>>(q, ldq, g, P->N, P->qu);
  gather_rows_kernel<<<(unsigned)((P->NP + 63) / 64), 256, 0, st>>>(P->qu, P->puser, P->NP, g, P->qt, P->qb64,
                                                                    f32 ? P->qb32 : nullptr);
  mark();
  // parents' expansions accumulate from their children (M2M below)
  zero_kernel<<<(unsigned)((slab * g + 255) / 256), 256, 0, st>>>(P->M, slab * g);
  if (nr <= 4 * kP2MBRows) {
    // the harmonics of a point once for all vectors
    p2m_batch_kernel<<<(unsigned)P->nleaves, 256, (size_t)kP2MBPts * (nr + 64) * sizeof(double), st>>>(
        p, g, P->leaves, P->bstart, P->bcount, P->blevel, P->bcx, P->bcy, P->bch, P->sc_levels, P->px, P->py,
        P->ph, P->qb64, P->coefR, P->M, slab);
  } else {
    const int lpb = kP2MThreads / (p + 1);
    p2m_kernel<<<dim3((unsigned)((P->nleaves + lpb - 1) / lpb), (unsigned)g), kP2MThreads,
                 (size_t)kP2MThreads * 2 * (p + 1) * sizeof(double), st>>>(
        p, P->nleaves, P->leaves, P->bstart, P->bcount, P->blevel, P->bcx, P->bcy, P->bch, P->sc_levels, P->px,
        P->py, P->ph, P->qt, P->coefR, P->M, P->NP, slab);
  }
  mark();
  // M2M per level: parents of level l from their children, all vectors at once
  // (the 8 octant operators through the batched FP64 GEMM)
  for (int l = P->maxlev - 1; l >= 0; --l)
    if (P->xl_need_m2m[l])
      if (int rc = launch_xlate_batch(P, g, P->bu_boxes, P->bu_lev[l], P->bu_lev[l + 1] - P->bu_lev[l], P->bu_ptr,
                                       P->bu_src, P->bu_op, P->Txl, P->M, P->M, st))
        return rc;
  mark();
  {
    const int64_t nl = slab * g;
    zero_kernel<<<(unsigned)((nl + 255) / 256), 256, 0, st>>>(P->Lx, nl);
    const int64_t n64 = f32 ? P->bbox_split : P->nbbox;
    const int64_t n32 = f32 ? P->nbbox - P->bbox_split : 0;
    if (!f32) mark();  // the FP64 form has one M2L launch over every level
    if (n64 > 0) {
      // the FP32 form's FP64 top levels as work items (few boxes, long entry
      // lists), then a reduction per box; the FP64 form one block per box
      vector_minor_kernel<<<(unsigned)P->ntop, 256, 0, st>>>(nr, nc, nc - p - 1, g, P->gw, slab, P->M, P->M64);
      if (int rc = launch_batch64(P, g, f32 ? P->n_btop_items : n64, f32 ? P->btop_items : nullptr, parts, P->Pbtop, st))
        return rc;
      if (f32)
        m2l_btop_reduce_kernel<<<(unsigned)n64, 256, 0, st>>>(nr, g, P->bbox, P->btop_iptr, P->Pbtop, P->blevel,
                                                              P->sc_levels, slab, P->Lx);
    }
    if (n32 > 0)
      vector_minor_kernel<<<(unsigned)P->NB, 256, 0, st>>>(nr, nc, nc - p - 1, g, P->gw, slab, P->M, P->M32);
    if (f32) mark();
    if (n32 > 0) {
      if (int rc = launch_batch32(P, P->batch_variant, g, n32, parts, st)) return rc;
    }
  }
  mark();
  mark();  // no separate reduction in the batched form
  for (int l = 1; l <= P->maxlev; ++l)
    if (P->xl_need_l2l[l])
      if (int rc = launch_xlate_batch(P, g, P->bd_boxes, P->bd_lev[l], P->bd_lev[l + 1] - P->bd_lev[l], P->bd_ptr,
                                       P->bd_src, P->bd_op, P->Txl, P->Lx, P->Lx, st))
        return rc;
  mark();
  {
    const int nks = (nr + 3) / 4;
#define L2PB(KN)                                                                                             \
  if (nks <= KN) {                                                                                           \
    l2p_batch_kernel<KN><<<(unsigned)P->nleaves, 256, (size_t)(KN <= 31 ? 32 : 16) * (4 * nks + 1) * 8, st>>>( \
        p, g, P->leaves, P->bstart, P->bcount, P->blevel, P->bcx, P->bcy, P->bch, P->sc_levels, P->px, P->py, \
        P->ph, P->Lx, P->coefR, P->phit, slab, P->NP);                                                       \
  } else
    L2PB(9) L2PB(21) L2PB(31) L2PB(43) L2PB(73) return FMMLM_EUNSUPPORTED;
#undef L2PB
  }
  mark();
  if ((parts & FMMLM_FREE) && f32 && P->n_pl_leaves > 0) {
    p2p_batch32_kernel<<<(unsigned)P->n_pl_leaves, 256, 0, st>>>(
        g, P->pl_leaves, P->leaves, P->bstart, P->bcount, P->bcx, P->bcy, P->bch, P->p2p_ptr, P->p2p_src, P->px,
        P->py, P->ph, P->qb32, P->NP, P->phit);
  } else if (parts & FMMLM_FREE) {
    for (const auto& fr : P->free_ranges) {
      if (fr.second <= 0) continue;
      const unsigned nb = (unsigned)((fr.second + 63) / 64);
      p2p_free_batch64_kernel<<<nb, 64, 0, st>>>(fr.first, fr.second, g, P->pleaf, P->p2p_ptr, P->p2p_src,
                                                 P->px, P->py, P->ph, P->qb64, P->NP, P->phit);
    }
  }
  mark();
  if ((parts & FMMLM_REACTION) && P->stats.p2p_reaction_pairs > 0) {
    if (f32) {
      if (P->n_rp_units16 > 0) {
        p2p_reaction_batch_rows_kernel<<<(unsigned)((P->n_rp_units16 + 3) / 4), 256, 0, st>>>(
            P->n_rp_units16, P->rp_units16, P->rp_src, P->rp_voff, P->rp_row, P->rp_val, P->qb32, P->Prb);
        p2p_reaction_batch_sum_kernel<<<(unsigned)P->nleaves, 256, 0, st>>>(
            g, P->leaves, P->bstart, P->bcount, P->rp_ptr, P->rp_row, P->Prb, P->NP, P->phit);
      }
    } else {
      p2p_reaction_batch_kernel<<<(unsigned)P->nleaves, 256, 0, st>>>(g, P->leaves, P->bstart, P->bcount,
                                                                      P->rp_ptr, P->rp_src, P->rp_voff,
                                                                      P->rp_val, P->qb64, P->NP, P->phit);
    }
  }
  mark();
  // the near field is done: qb64 holds the point-major far + near field
  transpose_points_kernel<<<(unsigned)((P->NP + 63) / 64), 256, 0, st>>>(P->phit, P->NP, g, P->qb64);
  combine_rows_kernel<<<(unsigned)((P->N + 63) / 64), 256, 0, st>>>(P->qb64, g, P->user_pos, P->N, phi, ldphi);
  mark();
  FMM_HIP_TRY(hipGetLastError());
  return FMMLM_OK;
}

int gpu_eval_one(fmmlm_plan_s* P, const double* q, double* phi, uint32_t parts, hipStream_t st,
                 hipEvent_t* ev) {
  int stage = 0;
  auto mark = [&]() {
    if (ev) (void)hipEventRecord(ev[stage], st);
    ++stage;
  };
  const int p = P->p;
  double* M = P->M;
  double* Lx = P->Lx;
  mark();
  gather_kernel<<<(unsigned)((P->NP + 255) / 256), 256, 0, st>>>(q, P->puser, P->NP, P->qt, P->qt32);
  mark();
  // Near field (P2P free, P2P reaction) into phin.  Unprofiled evaluations run
  // it on its own stream alongside the far field: the free P2P units
  // [0, pl_split) from the fork, the rest of the near field behind them, in the
  // FP32 form once its main M2L is done (the far field's latency-bound stages
  // before and after the M2L leave the GPU to it).  Without that launch, and in
  // the FP64 form, waiting for the M2L only puts the rest at the end: 600
  // charges, p = 16, FP32 138 us waiting, 124 not; 20,011 charges, p = 10, FP64 180
  // and 173.  Profiled evaluations run it in stage order.
  const bool overlap = (ev == nullptr);
  // units [u0, u1) of the mutual free P2P; the last part adds the combine pass
  auto p2p_free = [&](hipStream_t sn, int64_t u0, int64_t u1, size_t pad, bool last) {
    if (!(parts & FMMLM_FREE)) return;
    if (u1 > u0) {
      const unsigned nb = (unsigned)(u1 - u0);
#define PL_LAUNCH(T, MT, PAD)                                                                                       \
  p2p_mutual_kernel<T, MT><<<nb, kPLThreads, PAD, sn>>>(                                                            \
      u0, P->mu_order, P->mu_leaf, P->mu_tb, P->mu_rptr, P->mu_rng, P->mu_boff, P->mu_bidx, P->leaves, P->bstart,   \
      P->bcount, P->bcx, P->bcy, P->bch, P->px, P->py, P->ph, P->qt, P->mu_a, static_cast<T*>(P->mu_b))
      if (P->fp32)
        PL_LAUNCH(float, kPLUnitTargets / 16, pad);
      else if (P->pl_targets == kPLUnitTargetsFew)
        PL_LAUNCH(double, kPLUnitTargetsFew / 16, 0);
      else
        PL_LAUNCH(double, kPLUnitTargets / 16, 0);
#undef PL_LAUNCH
    }
    if (last && P->n_mu_units > 0) {
      if (P->fp32)
        p2p_combine_kernel<float><<<(unsigned)P->nleaves, kCBThreads, 0, sn>>>(
            P->leaves, P->bstart, P->bcount, P->cb_base, P->cb_n, P->mu_a, static_cast<const float*>(P->mu_b),
            P->phin);
      else
        p2p_combine_kernel<double><<<(unsigned)P->nleaves, kCBThreads, 0, sn>>>(
            P->leaves, P->bstart, P->bcount, P->cb_base, P->cb_n, P->mu_a, static_cast<const double*>(P->mu_b),
            P->phin);
    }
  };
  auto p2p_reaction = [&](hipStream_t sn) {
    if ((parts & FMMLM_REACTION) && P->stats.p2p_reaction_pairs > 0 && P->n_rp_units > 0) {
      const int64_t upb = kRPThreads / 64;
      if (P->rp_val32)
        p2p_reaction_rows_kernel<float><<<(unsigned)((P->n_rp_units + upb - 1) / upb), kRPThreads, 0, sn>>>(
            P->n_rp_units, P->rp_units, P->rp_src, P->rp_voff, P->rp_row, P->rp_val32, P->qt, P->Prp);
      else
        p2p_reaction_rows_kernel<double><<<(unsigned)((P->n_rp_units + upb - 1) / upb), kRPThreads, 0, sn>>>(
            P->n_rp_units, P->rp_units, P->rp_src, P->rp_voff, P->rp_row, P->rp_val, P->qt, P->Prp);
      p2p_reaction_sum_kernel<<<(unsigned)P->nleaves, kRPThreads, 0, sn>>>(P->leaves, P->bstart, P->bcount,
                                                                           P->rp_ptr, P->rp_row, P->Prp, P->phin);
    }
  };
  const int64_t split = std::min(std::max<int64_t>(P->pl_split, 0), P->n_mu_units);
  if (overlap) {
    FMM_HIP_TRY(hipEventRecord(P->ev_q, st));
    FMM_HIP_TRY(hipStreamWaitEvent(P->s_near, P->ev_q, 0));
    zero_kernel<<<(unsigned)((P->NP + 255) / 256), 256, 0, P->s_near>>>(P->phin, P->NP);
    p2p_free(P->s_near, 0, split, P->pl_pad, false);
  }
  {
    // parents' expansions accumulate from their children (M2M below)
    const int64_t nm = P->NB * (int64_t)(p + 1) * (p + 1);
    zero_kernel<<<(unsigned)((nm + 255) / 256), 256, 0, st>>>(M, nm);
    const unsigned nb = (unsigned)((P->nleaves + kP2MWWaves - 1) / kP2MWWaves);
    switch (p) {
#define FMMLM_P2M_WAVE(PO)                                                                                     \
  case PO:                                                                                                     \
    p2m_wave_kernel<PO><<<nb, 64 * kP2MWWaves, 0, st>>>(P->nleaves, P->leaves, P->bstart, P->bcount, P->blevel, \
                                                        P->bcx, P->bcy, P->bch, P->sc_levels, P->px, P->py,   \
                                                        P->ph, P->qt, P->coefR, M);                           \
    break;
      FMMLM_P2M_WAVE(1) FMMLM_P2M_WAVE(2) FMMLM_P2M_WAVE(3) FMMLM_P2M_WAVE(4) FMMLM_P2M_WAVE(5)
      FMMLM_P2M_WAVE(6) FMMLM_P2M_WAVE(7) FMMLM_P2M_WAVE(8) FMMLM_P2M_WAVE(9) FMMLM_P2M_WAVE(10)
      FMMLM_P2M_WAVE(11) FMMLM_P2M_WAVE(12) FMMLM_P2M_WAVE(13) FMMLM_P2M_WAVE(14) FMMLM_P2M_WAVE(15)
      FMMLM_P2M_WAVE(16)
#undef FMMLM_P2M_WAVE
      default:
        return FMMLM_EINVAL;
    }
  }
  mark();
  for (int l = P->maxlev - 1; l >= 0; --l)
    if (P->xl_need_m2m[l])
      if (int rc = launch_xlate_level(P, P->xl_m2m[l], true, M, Lx, st)) return rc;
  mark();
  {
    const int64_t nl = P->NB * (int64_t)(p + 1) * (p + 1);
    zero_kernel<<<(unsigned)((nl + 255) / 256), 256, 0, st>>>(Lx, nl);
  }
  // the FP32 form's top levels stay FP64 and write other boxes than the rest: on
  // their own stream (unprofiled), joined before L2L
  const bool top = P->fp32 && P->u64.n > 0;
  const bool top_side = overlap && top && P->u32.n > 0;
  if (top_side) {
    FMM_HIP_TRY(hipEventRecord(P->ev_m, st));
    FMM_HIP_TRY(hipStreamWaitEvent(P->s_top, P->ev_m, 0));
  }
  if (top) {
    hipStream_t ss = top_side ? P->s_top : st;
    if (int rc = launch_frame<double>(P, P->u64, 0, parts, M, ss)) return rc;
    if (int rc = launch_frame_reduce<double>(P, P->u64, Lx, ss)) return rc;
  }
  if (top_side) FMM_HIP_TRY(hipEventRecord(P->ev_top, P->s_top));
  mark();
  if (P->fp32) {
    if (int rc = launch_frame<float>(P, P->u32, P->m2l_variant, parts, M, st)) return rc;
  } else if (int rc = launch_frame<double>(P, P->u64, 0, parts, M, st)) {
    return rc;
  }
  if (overlap) {
    if (P->fp32 && P->u32.n > 0) {
      FMM_HIP_TRY(hipEventRecord(P->ev_l, st));
      FMM_HIP_TRY(hipStreamWaitEvent(P->s_near, P->ev_l, 0));
    }
    p2p_free(P->s_near, split, P->n_mu_units, P->pl_pad, true);
    p2p_reaction(P->s_near);
    FMM_HIP_TRY(hipEventRecord(P->ev_near, P->s_near));
  }
  mark();
  // each target's products, in slot order
  if (P->fp32) {
    if (int rc = launch_frame_reduce<float>(P, P->u32, Lx, st)) return rc;
  } else if (int rc = launch_frame_reduce<double>(P, P->u64, Lx, st)) {
    return rc;
  }
  mark();
  if (top_side) FMM_HIP_TRY(hipStreamWaitEvent(st, P->ev_top, 0));
  for (int l = 1; l <= P->maxlev; ++l)
    if (P->xl_need_l2l[l])
      if (int rc = launch_xlate_level(P, P->xl_l2l[l], false, M, Lx, st)) return rc;
  mark();
  switch (p) {
#define FMMLM_L2P_FIXED(PO)                                                                                    \
  case PO:                                                                                                     \
    l2p_fixed_kernel<PO><<<(unsigned)P->nleaves, 64, 0, st>>>(P->leaves, P->bstart, P->bcount, P->blevel,      \
                                                             P->bcx, P->bcy, P->bch, P->sc_levels, P->px, P->py, \
                                                             P->ph, Lx, P->coefR, P->phit);                   \
    break;
    FMMLM_L2P_FIXED(1) FMMLM_L2P_FIXED(2) FMMLM_L2P_FIXED(3) FMMLM_L2P_FIXED(4) FMMLM_L2P_FIXED(5)
    FMMLM_L2P_FIXED(6) FMMLM_L2P_FIXED(7) FMMLM_L2P_FIXED(8) FMMLM_L2P_FIXED(9) FMMLM_L2P_FIXED(10)
    FMMLM_L2P_FIXED(11) FMMLM_L2P_FIXED(12) FMMLM_L2P_FIXED(13) FMMLM_L2P_FIXED(14) FMMLM_L2P_FIXED(15)
    FMMLM_L2P_FIXED(16)
#undef FMMLM_L2P_FIXED
    default:
      return FMMLM_EINVAL;
  }
  mark();
  if (overlap) {
    mark();
    mark();
    FMM_HIP_TRY(hipStreamWaitEvent(st, P->ev_near, 0));
  } else {
    zero_kernel<<<(unsigned)((P->NP + 255) / 256), 256, 0, st>>>(P->phin, P->NP);
    p2p_free(st, 0, P->n_mu_units, 0, true);
    mark();
    p2p_reaction(st);
    mark();
  }
  combine_kernel<<<(unsigned)((P->N + 255) / 256), 256, 0, st>>>(P->phit, P->phin, P->user_pos, P->N, phi);
  mark();
  FMM_HIP_TRY(hipGetLastError());
  return FMMLM_OK;
}

}  // namespace fmmlm
