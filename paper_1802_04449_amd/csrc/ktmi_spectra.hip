// ktmi_spectra.hip -- smooth Cooper-Frye spectra on the GPU (arXiv:1802.04449,
// Sec. IV, eq. cooper_frye with f_eq and delta f of eqn. feq; App. A.2: the sum
// over surface elements runs on the GPU, elements shared inside a workgroup).
//
// dN/(dY pT dpT dphi) = g / (2 pi hbarc)^3 sum_elements p^mu dSigma_mu f (1 + df)
// for every (species, Y, pT, phi) bin, with (tilde components, element centre
// (tau, eta_s)) p~ = (m_T cosh(Y - eta_s), pT cos phi, pT sin phi, m_T sinh(Y - eta_s)),
// p^mu dSigma_mu = p~^tau dS_tau + p~^x dS_x + p~^y dS_y + (p~^eta / tau) dS_eta,
// p.u = p~^tau u~^tau - p~^x u~^x - p~^y u~^y - p~^eta u~^eta,
// f = 1 / (exp((p.u - mu)/T) + sigma), df = (1 - sigma f) p~_a p~_b pi~^{ab} / (2 T^2 (e + P)).
//
// The exponential factorises: with x_L = (p~^tau u~^tau - p~^eta u~^eta - mu)/T, which
// depends on (species, Y, pT), and x_T = -(p~^x u~^x + p~^y u~^y)/T, which depends on
// (pT, phi), exp((p.u - mu)/T) = e^{x_L} e^{x_T}; p.dSigma and p~p~pi~ split the same
// way into a longitudinal part, a transverse part and (pi~ only) p~^tau and p~^eta
// times two transverse sums.  A workgroup therefore computes, per element, one record
// for each of its (species, Y, pT) and one for each of its (pT, phi), stages both in
// LDS, and every thread evaluates a small outer product of them: per bin one product
// for the exponential, one reciprocal and a few multiply-adds, instead of an
// exponential, a division and the whole quadratic form.
//
// Layout of the work: a thread owns TS (species, Y) pairs x TP phi bins of one pT; 16
// lanes run over the pairs and 16 slots over groups of TP phi bins (of any pT), so a
// workgroup of 256 covers 16 TS pairs x 16 TP transverse bins and one slice of the
// elements.  Slices give the chip enough workgroups; their partial sums are added in
// slice order by a second kernel, so the result does not depend on scheduling.
//
// Bound by FP64 VALU issue: about 21 instruction slots per (element, bin), the
// reciprocal four of them, plus a sixth for the records (FP64 instructions issue at
// 0.7-0.85 of the nominal one per CU and clock under this load).  41660 elements x 8
// species x 41 x 15 x 48 bins with delta f: 23.0 ms -> 9.06 ms a call (4.3e11 -> 1.09e12
// element-bin evaluations/s); an exponential and a division per bin took about 80
// slots.
#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>
#include <vector>

#include "../../include/ktmi.h"
#include "ktmi_spectra.hpp"

namespace ktmi {

namespace {

constexpr int kSpecBlock = 256;
constexpr int kLanes = 16;   // lanes over (species, Y) pairs, and slots over phi groups
// LDS for the records of one stage (as many elements as fit, at least one): three
// workgroups of 256 per CU also leave 160 KB / 3 each
constexpr int kStageBytes = 40 * 1024;

// Launch shape of one (TS, TP) variant.
struct SpecShape {
  int nsy;    // (species, Y) pairs
  int gpp;    // groups of TP phi bins per pT
  int ntg;    // such groups in all
  int npb;    // largest number of different pT in a workgroup's 16 slots
  int nel;    // elements per stage
  int nby;    // workgroups over the transverse groups
};

// e^x = m 2^k with |m - 1| < 0.42 (cut at |x| = 7e8, where the value over- or underflows all
// the same and the sum of two such k fits 32 bits; NaN stays NaN): k = round(x log2 e), then the
// Taylor series of e^r, |r| <= ln2 / 2, to r^13 / 13! (remainder < 1e-17).
__device__ __forceinline__ double split_exp(double x, int& k) {
  x = x > 7e8 ? 7e8 : x;
  x = x < -7e8 ? -7e8 : x;
  const double kd = rint(x * 1.4426950408889634);
  double r = fma(kd, -0.6931471805599453, x);
  r = fma(kd, -2.3190468138462996e-17, r);
  double p = 1.0 / 6227020800.0;
  p = fma(p, r, 1.0 / 479001600.0);
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  k = (int)kd;
  return p;
}

// 1 / x: the hardware estimate y, one third-order step y (1 + e + e^2) with e = 1 - x y,
// and the fix-up instruction for x = 0, infinite or NaN (about one ulp; no division
// sequence).
__device__ __forceinline__ double recip(double x) {
  double y = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, y, 1.0);
  y = fma(y, fma(e, e, e), y);
  return __builtin_amdgcn_div_fixup(y, x, 1.0);
}

// Three waves per SIMD (a TS = 3, TP = 6 thread fits without spills; without the
// bound the compiler takes 200 registers and two waves: 10.1 -> 9.4 ms for TP = 8 on
// the 41660-element surface below).
template <int TS, int TP, bool DF>
__global__ __launch_bounds__(kSpecBlock) __attribute__((amdgpu_waves_per_eu(3))) void k_spectra(SpectraArgs a, SpecShape sh) {
  constexpr int NS = kLanes * TS, NT = kLanes * TP;  // pairs and transverse bins covered
  constexpr int NR = DF ? 3 : 2;                     // double2 values per record
  extern __shared__ double2 smem[];
  double2* const recA = smem;                             // [nel][NR][npb][NS]
  double2* const recB = recA + sh.nel * NR * sh.npb * NS;  // [nel][NR][NT]
  double* const shmT = (double*)(recB + sh.nel * NR * NT);  // [npb][NS]
  double* const shY = shmT + sh.npb * NS;                  // [NS]
  double* const shmu = shY + NS;                           // [NS]
  double* const shpx = shmu + NS;                          // [NT]
  double* const shpy = shpx + NT;                          // [NT]
  const gdouble* el = (const gdouble*)a.elements;
  const gdouble* tab = (const gdouble*)a.tables;
  const int tid = threadIdx.x;
  const int sy0 = (int)(blockIdx.x / sh.nby) * NS, tg0 = (int)(blockIdx.x % sh.nby) * kLanes;
  const int ip0 = tg0 / sh.gpp;
  // tables: mass, dof, stat, mu (ns each), Y (nY), pT (npt), cos phi, sin phi (nphi each)
  const gdouble* tpt = tab + 4 * a.ns + a.nY;
  const gdouble* cphi = tpt + a.npt;
  const gdouble* sphi = cphi + a.nphi;
  for (int k = tid; k < sh.npb * NS; k += kSpecBlock) {
    const int sy = min(sy0 + k % NS, sh.nsy - 1), ip = min(ip0 + k / NS, a.npt - 1);
    const double m = tab[sy / a.nY], pt = tpt[ip];
    shmT[k] = sqrt(m * m + pt * pt);
  }
  for (int k = tid; k < NS; k += kSpecBlock) {
    const int sy = min(sy0 + k, sh.nsy - 1);
    shY[k] = tab[4 * a.ns + sy % a.nY];
    shmu[k] = tab[3 * a.ns + sy / a.nY];
  }
  for (int k = tid; k < NT; k += kSpecBlock) {
    const int tg = min(tg0 + k / TP, sh.ntg - 1), iq = (tg % sh.gpp) * TP + k % TP;
    const bool ok = iq < a.nphi;
    const double pt = tpt[tg / sh.gpp];
    shpx[k] = ok ? pt * cphi[iq] : 0.0;
    shpy[k] = ok ? pt * sphi[iq] : 0.0;
  }
  const int lane = tid % kLanes, slot = tid / kLanes;
  const int tg = min(tg0 + slot, sh.ntg - 1);
  const int pb = tg / sh.gpp - ip0;  // this thread's pT among the workgroup's
  double sig[TS], acc[TS][TP];
#pragma unroll
  for (int t = 0; t < TS; ++t) {
    sig[t] = tab[2 * a.ns + min(sy0 + lane + kLanes * t, sh.nsy - 1) / a.nY];
#pragma unroll
    for (int q = 0; q < TP; ++q) acc[t][q] = 0.0;
  }
  const double invT = 1.0 / a.T;
  const double dfc = DF ? 1.0 / (2.0 * a.T * a.T * a.eps_plus_P) : 0.0;
  // this workgroup's slice of the elements
  const long per = (a.n + gridDim.y - 1) / gridDim.y;
  const long e0 = (long)blockIdx.y * per;
  const long e1 = e0 + per < a.n ? e0 + per : a.n;
  for (long c0 = e0; c0 < e1; c0 += sh.nel) {
    const int cn = (int)(e1 - c0 < sh.nel ? e1 - c0 : sh.nel);
    __syncthreads();
    // longitudinal records: (e^{x_L}, p.dSigma), (p~^tau, p~^eta), (p~p~pi~, k_L)
    for (int k = tid; k < cn * sh.npb * NS; k += kSpecBlock) {
      const int e = k / (sh.npb * NS), r = k - e * (sh.npb * NS);
      const gdouble* g = el + (c0 + e) * kSurfRec;
      const double yrel = shY[r % NS] - g[4], ux = g[9], uy = g[10], ue = g[11];
      const double ut2 = 1.0 + ux * ux + uy * uy + ue * ue;
      const double ut = sqrt(ut2 < a.far2 ? ut2 : NAN);  // NaN: left to the fold
      int ke, kl;
      const double ey = ldexp(split_exp(yrel, ke), ke), iey = recip(ey);
      // sinh by its series where the exponentials cancel (|yrel| < 0.3: y^15 / 15! < 2e-20)
      const double y2 = yrel * yrel;
      double ss = fma(y2, 1.0 / 6227020800.0, 1.0 / 39916800.0);
      ss = fma(y2, ss, 1.0 / 362880.0);
      ss = fma(y2, ss, 1.0 / 5040.0);
      ss = fma(y2, ss, 1.0 / 120.0);
      ss = fma(y2, ss, 1.0 / 6.0);
      const double sy = fabs(yrel) < 0.3 ? fma(yrel * y2, ss, yrel) : 0.5 * (ey - iey);
      const double mT = shmT[r], p0 = mT * (0.5 * (ey + iey)), p3 = mT * sy;
      const double eL = split_exp((p0 * ut - p3 * ue - shmu[r % NS]) * invT, kl);
      double2* out = recA + (e * NR * sh.npb) * NS + r;
      out[0] = double2{eL, p0 * g[5] + p3 / g[1] * g[8]};
      if constexpr (DF) {
        const double ppi = p0 * p0 * g[12] + p3 * p3 * g[21] - 2.0 * p0 * p3 * g[15];
        out[sh.npb * NS] = double2{p0, p3};
        out[2 * sh.npb * NS] = double2{ppi * dfc, __hiloint2double(0, kl)};
      } else {
        out[sh.npb * NS] = double2{__hiloint2double(0, kl), 0.0};
      }
    }
    // transverse records: (e^{x_T}, p.dSigma), (the factors of p~^tau and p~^eta), (p~p~pi~, k_T)
    for (int k = tid; k < cn * NT; k += kSpecBlock) {
      const int e = k / NT, r = k - e * NT;
      const gdouble* g = el + (c0 + e) * kSurfRec;
      const double x = shpx[r], y = shpy[r];
      int kt;
      const double eT = split_exp(-(x * g[9] + y * g[10]) * invT, kt);
      double2* out = recB + (e * NR) * NT + r;
      out[0] = double2{eT, x * g[6] + y * g[7]};
      if constexpr (DF) {
        const double ppi = x * x * g[16] + y * y * g[19] + 2.0 * (x * y * g[17]);
        out[NT] = double2{-2.0 * (x * g[13] + y * g[14]) * dfc, 2.0 * (x * g[18] + y * g[20]) * dfc};
        out[2 * NT] = double2{ppi * dfc, __hiloint2double(0, kt)};
      } else {
        out[NT] = double2{__hiloint2double(0, kt), 0.0};
      }
    }
    __syncthreads();
    for (int e = 0; e < cn; ++e) {
      const double2* A = recA + (e * NR * sh.npb + pb) * NS + lane;
      const double2* B = recB + e * NR * NT + slot * TP;
      double2 a0[TS], a1[TS], a2[TS];
#pragma unroll
      for (int t = 0; t < TS; ++t) {
        a0[t] = A[kLanes * t];
        a1[t] = A[sh.npb * NS + kLanes * t];
        if constexpr (DF) a2[t] = A[2 * sh.npb * NS + kLanes * t];
      }
#pragma unroll
      for (int q = 0; q < TP; ++q) {
        const double2 b0 = B[q], b1 = B[NT + q];
        double2 b2 = {0.0, 0.0};
        if constexpr (DF) b2 = B[2 * NT + q];
        const int kb = __double2loint(DF ? b2.y : b1.x);
#pragma unroll
        for (int t = 0; t < TS; ++t) {
          const int ka = __double2loint(DF ? a2[t].y : a1[t].x);
          const double f = recip(ldexp(a0[t].x * b0.x, ka + kb) + sig[t]);
          const double pdS = a0[t].y + b0.y;
          if constexpr (DF) {
            const double ppi = fma(a1[t].x, b1.x, fma(a1[t].y, b1.y, a2[t].x + b2.x));
            const double w = fma(fma(-sig[t], f, 1.0), ppi, 1.0);
            acc[t][q] = fma(pdS, f * w, acc[t][q]);
          } else {
            acc[t][q] = fma(pdS, f, acc[t][q]);
          }
        }
      }
    }
  }
  if (tg0 + slot >= sh.ntg) return;
  gdouble* part = (gdouble*)a.partial + (long)blockIdx.y * a.nbins;
#pragma unroll
  for (int t = 0; t < TS; ++t) {
    const int sy = sy0 + lane + kLanes * t;
    if (sy >= sh.nsy) continue;
#pragma unroll
    for (int q = 0; q < TP; ++q) {
      const int iq = (tg % sh.gpp) * TP + q;
      if (iq < a.nphi) part[((long)sy * a.npt + tg / sh.gpp) * a.nphi + iq] = acc[t][q];
    }
  }
}

// Sum of elements e0 .. e1 - 1 for one bin, with one exponential for the whole exponent.
__device__ double bin_sum(const SpectraArgs& a, long bin, long e0, long e1) {
  const gdouble* tab = (const gdouble*)a.tables;
  const gdouble* tpt = tab + 4 * a.ns + a.nY;
  const int iq = (int)(bin % a.nphi), ip = (int)(bin / a.nphi % a.npt);
  const int sy = (int)(bin / ((long)a.nphi * a.npt)), s = sy / a.nY;
  const double m = tab[s], sig = tab[2 * a.ns + s], mu = tab[3 * a.ns + s];
  const double Y = tab[4 * a.ns + sy % a.nY], pt = tpt[ip], mT = sqrt(m * m + pt * pt);
  const double x = pt * tpt[a.npt + iq], y = pt * tpt[a.npt + a.nphi + iq], invT = 1.0 / a.T;
  double sum = 0.0;
  for (long e = e0; e < e1; ++e) {
    const gdouble* g = (const gdouble*)a.elements + e * kSurfRec;
    const double ux = g[9], uy = g[10], ue = g[11];
    const double p0 = mT * cosh(Y - g[4]), p3 = mT * sinh(Y - g[4]);
    const double pu = p0 * sqrt(1.0 + ux * ux + uy * uy + ue * ue) - p3 * ue - x * ux - y * uy;
    const double f = 1.0 / (exp((pu - mu) * invT) + sig);
    double w = 1.0;
    if (a.eps_plus_P > 0.0) {
      const double ppi = p0 * p0 * g[12] + x * x * g[16] + y * y * g[19] + p3 * p3 * g[21] +
                         2.0 * (-p0 * x * g[13] - p0 * y * g[14] - p0 * p3 * g[15] + x * y * g[17] +
                                x * p3 * g[18] + y * p3 * g[20]);
      w = 1.0 + (1.0 - sig * f) * ppi / (2.0 * a.T * a.T * a.eps_plus_P);
    }
    sum += (p0 * g[5] + p3 / g[1] * g[8] + x * g[6] + y * g[7]) * f * w;
  }
  return sum;
}

// out[bin] = dof[s] / (2 pi hbarc)^3 * sum over slices (in slice order).  A slice's sum is NaN
// where an element is (its sum here is too), or for a far element: flow so fast, or infinite,
// that the exponents of both factors might reach the cut while they cancel in the bin (p_T
// u~^tau / T > 1e6 for the largest p_T: SpectraArgs::far2).
__global__ __launch_bounds__(kSpecBlock) void k_spectra_fold(SpectraArgs a, int nslice) {
  const long bin = (long)blockIdx.x * kSpecBlock + threadIdx.x;
  if (bin >= a.nbins) return;
  const gdouble* part = (const gdouble*)a.partial;
  const gdouble* tab = (const gdouble*)a.tables;
  double sum = 0.0;
#pragma unroll 8
  for (int k = 0; k < nslice; ++k) sum += part[(long)k * a.nbins + bin];
  if (sum != sum) {
    const long per = (a.n + nslice - 1) / nslice;
    sum = 0.0;
    for (int k = 0; k < nslice; ++k) {
      const double v = part[(long)k * a.nbins + bin];
      const long e0 = k * per;
      sum += v != v ? bin_sum(a, bin, e0, e0 + per < a.n ? e0 + per : a.n) : v;
    }
  }
  const int s = (int)(bin / ((long)a.nY * a.npt * a.nphi));
  const double pref = 1.0 / ((2.0 * M_PI * kHbarc) * (2.0 * M_PI * kHbarc) * (2.0 * M_PI * kHbarc));
  ((gdouble*)a.out)[bin] = tab[a.ns + s] * pref * sum;
}

}  // namespace

int spectra_min_slices(long n) {
  const long s = (n + 255) / 256;  // at least 256 elements per slice
  return (int)(s < 1 ? 1 : (s > kMinSlicesCap ? kMinSlicesCap : s));
}

// Few bins or few elements leave most of the chip without a workgroup: there, slices
// down to 16 elements, until about 2048 workgroups of the largest tile (48 pairs x 96
// transverse bins) are out.  568 elements on 88 x 18 x 1 bins: 3 slices 448 us a call,
// 36 slices 58 us; 7596 elements on 5 x 16 x 20: 166 -> 91 us.
int spectra_slices(long n, long nbins) {
  const long wg = (nbins + 4607) / 4608;
  const long more = std::min({(n + 15) / 16, 2048 / wg, (long)kMaxSlices});
  return (int)std::max<long>(spectra_min_slices(n), more);
}

namespace {

SpecShape spec_shape(const SpectraArgs& a, int TS, int TP, bool df, size_t* lds) {
  const int NS = kLanes * TS, NT = kLanes * TP, NR = df ? 3 : 2;
  SpecShape sh;
  sh.nsy = a.ns * a.nY;
  sh.gpp = (a.nphi + TP - 1) / TP;
  sh.ntg = a.npt * sh.gpp;
  sh.npb = std::min((kLanes - 2 + sh.gpp) / sh.gpp + 1, a.npt);
  const size_t one = (size_t)NR * (sh.npb * NS + NT) * sizeof(double2);
  sh.nel = (int)std::max<size_t>(1, std::min<size_t>(8, kStageBytes / one));
  sh.nby = (sh.ntg + kLanes - 1) / kLanes;
  *lds = sh.nel * one + (size_t)(sh.npb * NS + 2 * NS + 2 * NT) * sizeof(double);
  return sh;
}

// Estimated instruction slots per element of a variant: bins of whole workgroups at 22
// slots, or the LDS reads of the two record sets (8 clocks per 16 bytes a lane) where
// those take longer, plus the records themselves (75 and 50 slots).
double spec_cost(const SpectraArgs& a, int TS, int TP, bool df) {
  size_t lds;
  const SpecShape sh = spec_shape(a, TS, TP, df, &lds);
  const double wg = (double)((sh.nsy + kLanes * TS - 1) / (kLanes * TS)) * sh.nby;
  const double eval = std::max(22.0 * TS * TP, 8.0 * (df ? 3 : 2) * (TS + TP));
  return wg * (kSpecBlock * eval + 75.0 * sh.npb * kLanes * TS + 50.0 * kLanes * TP);
}

template <int TS, int TP>
void launch_variant(const SpectraArgs& a, int nslice, hipStream_t s) {
  const bool df = a.eps_plus_P > 0.0;
  size_t lds;
  const SpecShape sh = spec_shape(a, TS, TP, df, &lds);
  const dim3 grid((unsigned)((sh.nsy + kLanes * TS - 1) / (kLanes * TS)) * sh.nby, (unsigned)nslice);
  if (df)
    hipLaunchKernelGGL((k_spectra<TS, TP, true>), grid, dim3(kSpecBlock), lds, s, a, sh);
  else
    hipLaunchKernelGGL((k_spectra<TS, TP, false>), grid, dim3(kSpecBlock), lds, s, a, sh);
}

}  // namespace

int launch_spectra(const SpectraArgs& a, int nslice, hipStream_t s) {
  // the variant with the fewest estimated slots: the larger tiles share more, the
  // smaller ones pad less where there are few pairs or phi bins
  static const struct {
    int ts, tp;
    void (*fn)(const SpectraArgs&, int, hipStream_t);
  } kVar[] = {{3, 6, launch_variant<3, 6>}, {3, 4, launch_variant<3, 4>}, {3, 1, launch_variant<3, 1>},
              {1, 6, launch_variant<1, 6>}, {1, 4, launch_variant<1, 4>}, {1, 1, launch_variant<1, 1>}};
  int best = 0;
  double cost = 1e300;
  for (int v = 0; v < (int)(sizeof(kVar) / sizeof(kVar[0])); ++v) {
    const double c = spec_cost(a, kVar[v].ts, kVar[v].tp, a.eps_plus_P > 0.0);
    if (c < cost) {
      cost = c;
      best = v;
    }
  }
  kVar[best].fn(a, nslice, s);
  const long fx = (a.nbins + kSpecBlock - 1) / kSpecBlock;
  hipLaunchKernelGGL(k_spectra_fold, dim3((unsigned)fx), dim3(kSpecBlock), 0, s, a, nslice);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ktmi

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
using namespace ktmi;

static size_t spectra_table_doubles(int ns, int nY, int npt, int nphi) {
  return ((size_t)4 * ns + nY + npt + 2 * (size_t)nphi + 31) / 32 * 32;
}

extern "C" {

size_t ktmi_spectra_workspace_bytes(long n, int ns, int nY, int npt, int nphi) {
  if (n < 0 || ns < 1 || nY < 1 || npt < 1 || nphi < 1) return 0;
  const size_t nbins = (size_t)ns * nY * npt * nphi;
  return (spectra_table_doubles(ns, nY, npt, nphi) + (size_t)spectra_slices(n, (long)nbins) * nbins) *
         sizeof(double);
}

int ktmi_spectra(const double* elements, long n, double T, double eps_plus_P, int ns,
                 const double* mass, const double* dof, const int* stat, const double* mu, int nY,
                 const double* Y, int npt, const double* pt, int nphi, const double* phi,
                 double* out, void* ws, size_t ws_bytes, void* stream) {
  if (n < 0 || (n > 0 && !elements) || !(T > 0) || !(eps_plus_P >= 0) || ns < 1 || nY < 1 ||
      npt < 1 || nphi < 1 || !mass || !dof || !stat || !mu || !Y || !pt || !phi || !out || !ws)
    return KTMI_EINVAL;
  // as many slices as the workspace holds, up to what ktmi_spectra_workspace_bytes asks
  // for; the fewest the call takes are those of spectra_min_slices
  const size_t ntab = spectra_table_doubles(ns, nY, npt, nphi);
  const size_t nbins = (size_t)ns * nY * npt * nphi, room = ws_bytes / sizeof(double);
  const size_t fit = room < ntab ? 0 : (room - ntab) / nbins;
  if (fit < (size_t)spectra_min_slices(n)) return KTMI_EINVAL;
  const int nslice = (int)std::min<size_t>(fit, (size_t)spectra_slices(n, (long)nbins));
  for (int s = 0; s < ns; ++s)
    if (!(mass[s] >= 0) || stat[s] < -1 || stat[s] > 1) return KTMI_EINVAL;
  std::vector<double> tab(ntab, 0.0);
  for (int s = 0; s < ns; ++s) {
    tab[s] = mass[s];
    tab[ns + s] = dof[s];
    tab[2 * ns + s] = (double)stat[s];
    tab[3 * ns + s] = mu[s];
  }
  for (int i = 0; i < nY; ++i) tab[4 * ns + i] = Y[i];
  for (int i = 0; i < npt; ++i) tab[4 * ns + nY + i] = pt[i];
  for (int i = 0; i < nphi; ++i) {
    tab[4 * ns + nY + npt + i] = cos(phi[i]);
    tab[4 * ns + nY + npt + nphi + i] = sin(phi[i]);
  }
  hipStream_t st = (hipStream_t)stream;
  double* dtab = (double*)ws;
  if (hipMemcpyAsync(dtab, tab.data(), tab.size() * sizeof(double), hipMemcpyHostToDevice, st) !=
      hipSuccess)
    return KTMI_EHIP;
  // the host table must outlive the copy
  if (hipStreamSynchronize(st) != hipSuccess) return KTMI_EHIP;
  SpectraArgs a;
  a.elements = elements;
  a.n = n;
  a.T = T;
  a.eps_plus_P = eps_plus_P;
  a.ns = ns;
  a.nY = nY;
  a.npt = npt;
  a.nphi = nphi;
  a.nbins = (long)nbins;
  double ptm = 0.0;
  for (int k = 0; k < npt; ++k) ptm = std::max(ptm, fabs(pt[k]));
  a.far2 = (1e6 * T / ptm) * (1e6 * T / ptm);  // (infinite for p_T = 0)
  a.tables = dtab;
  a.partial = dtab + tab.size();
  a.out = out;
  return launch_spectra(a, nslice, st) == 0 ? KTMI_OK : KTMI_EHIP;
}

}  // extern "C"
