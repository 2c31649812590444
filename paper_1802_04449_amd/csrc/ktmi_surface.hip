// ktmi_surface.hip -- freeze-out hypersurface finder on the GPU (arXiv:1802.04449,
// Sec. IV: surface elements dSigma_mu of constant freeze-out energy density e_f;
// App. A.2: the surface is found on the device between stored time slices, so
// the fields never travel to the host).
//
// One thread per hypercube of 2 x 2 x 2 x 2 grid points (two slices, two
// neighbouring cells per axis; an axis with one cell spans that cell's width).
// With phi = e - e_f at its 16 corners, the surface inside the hypercube is the
// zero set of the piecewise-linear interpolant of phi on the Kuhn triangulation.
// By the divergence theorem over the hot part (phi > 0) of the hypercube, the
// surface covector pointing out of the hot region is
//   S_mu = V_mu (f_lo(mu) - f_hi(mu)),
// V_mu the coordinate volume of the 3-faces normal to axis mu and f the hot
// volume fraction of a face: the mean over its six Kuhn tetrahedra of the exact
// fraction of a linear function.  Neighbouring hypercubes share faces, so sums
// of S telescope exactly.  dSigma_mu = tau_c S_mu (1 in Cartesian mode), tau_c
// the time of the element's centre: the mean of the sign changes along the 32
// edges; e, u~ and pi~ there are multilinear interpolants of the corners.
//
// Passes: a light count (one thread per hypercube, e only) of the hypercubes
// that straddle e_f per workgroup, an exclusive prefix sum of those counts, a
// compaction that writes each straddling hypercube's index to its slot, and the
// element pass over the slots, densely packed, so the heavy arithmetic runs only
// where there is surface.  No atomics: records come out in hypercube order, and
// the arithmetic is written in a fixed order with contraction off, so the output
// is reproducible bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ktmi_surface.hpp"

#pragma clang fp contract(off)

namespace ktmi {

namespace {

constexpr int kSurfBlock = 256;

// Hot fraction of a tetrahedron on which phi is linear (vertex values v0..v3).
// The hot and cold vertices are taken in vertex order; every term is a sum or
// product of positive ones.  Without branches, since the lanes of a wave hold every
// case: with one vertex apart from the three others (value s0; r0, r1, r2) its corner
// is s0^3 / prod (s0 + r), hot or cold; with two hot (a, b) and two cold (c, d) the
// volume is [a^2 b^2 + a b (a + b)(c + d) + c d (a^2 + a b + b^2)] / [(a+c)(a+d)(b+c)(b+d)],
// whose quotient takes the place of the first one: 3 divisions instead of 7.
__device__ __forceinline__ double tet_hot(double v0, double v1, double v2, double v3) {
  const bool h0 = v0 > 0.0, h1 = v1 > 0.0, h2 = v2 > 0.0, h3 = v3 > 0.0;
  const int np = (int)h0 + (int)h1 + (int)h2 + (int)h3;
  const bool three = np == 3, two = np == 2;
  // the set vertices: the hot ones, or the cold one of three hot
  const bool b0 = h0 != three, b1 = h1 != three, b2 = h2 != three, b3 = h3 != three;
  const double x0 = fabs(v0), x1 = fabs(v1), x2 = fabs(v2), x3 = fabs(v3);
  const double s0 = b0 ? x0 : (b1 ? x1 : (b2 ? x2 : x3));  // first set
  const double s1 = b3 ? x3 : (b2 ? x2 : x1);              // last set
  const double r0 = !b0 ? x0 : (!b1 ? x1 : x2);            // first not set
  const double rl = !b3 ? x3 : (!b2 ? x2 : x1);            // last not set
  const double r1 = two ? rl : (b0 || b1 ? x2 : x1);       // second not set
  const double num = s0 * s0 * s1 * s1 + s0 * s1 * (s0 + s1) * (r0 + r1) +
                     r0 * r1 * (s0 * s0 + s0 * s1 + s1 * s1);
  const double den = (s0 + r0) * (s0 + r1) * (s1 + r0) * (s1 + r1);
  const double q = (two ? num : s0) / (two ? den : s0 + r0);
  const double c = q * (s0 / (s0 + r1)) * (s0 / (s0 + rl));
  const double f = two ? q : (three ? 1.0 - c : c);
  return np == 0 ? 0.0 : (np == 4 ? 1.0 : f);
}

// Hot fraction of a 3-cube with corner values w[4 b0 + 2 b1 + b2]: mean over the
// Kuhn tetrahedra 000 -> +e_p -> +e_q -> 111 for the axis orders
// (0,1,2), (0,2,1), (1,0,2), (1,2,0), (2,0,1), (2,1,0).
__device__ __forceinline__ double cube_hot(const double w[8]) {
  double s = 0.0;
  s += tet_hot(w[0], w[4], w[6], w[7]);  // 0,1,2
  s += tet_hot(w[0], w[4], w[5], w[7]);  // 0,2,1
  s += tet_hot(w[0], w[2], w[6], w[7]);  // 1,0,2
  s += tet_hot(w[0], w[2], w[3], w[7]);  // 1,2,0
  s += tet_hot(w[0], w[1], w[5], w[7]);  // 2,0,1
  s += tet_hot(w[0], w[1], w[3], w[7]);  // 2,1,0
  return s / 6.0;
}

// Corner index of the hypercube (8 b_tau + 4 b_x + 2 b_y + b_eta) of bit b of
// the face normal to axis mu on side `side` (the face's bits run over the other
// three axes in increasing order).
__host__ __device__ constexpr int face_corner(int mu, int side, int b) {
  int c = 0, t = 0;
  for (int ax = 0; ax < 4; ++ax) {
    int bit = 0;
    if (ax == mu) {
      bit = side;
    } else {
      bit = (b >> (2 - t)) & 1;
      ++t;
    }
    c |= bit << (3 - ax);
  }
  return c;
}

// Hypercube index -> (i, j, k) and the flat cell index of its 8 spatial corners
// (grids hold fewer than 2^31 cells).
struct Cube {
  int i, j, k;
  int cell[8];
};

__device__ __forceinline__ Cube cube_of(const SurfaceArgs& a, int id) {
  const int cy = a.ny > 1 ? a.ny - 1 : 1, cz = a.ne > 1 ? a.ne - 1 : 1;
  Cube q;
  const int r = id / cz;
  q.k = id - r * cz;
  q.i = r / cy;
  q.j = r - q.i * cy;
  const int ii[2] = {q.i, a.nx > 1 ? q.i + 1 : q.i};
  const int jj[2] = {q.j, a.ny > 1 ? q.j + 1 : q.j};
  const int kk[2] = {q.k, a.ne > 1 ? q.k + 1 : q.k};
#pragma unroll
  for (int b = 0; b < 8; ++b) q.cell[b] = (ii[(b >> 2) & 1] * a.ny + jj[(b >> 1) & 1]) * a.ne + kk[b & 1];
  return q;
}

__host__ __device__ __forceinline__ long cube_count(long nx, long ny, long ne) {
  return (nx > 1 ? nx - 1 : 1) * (ny > 1 ? ny - 1 : 1) * (ne > 1 ? ne - 1 : 1);
}

// Every count / compaction workgroup covers kSpan consecutive hypercubes: kIt
// rounds of kSurfBlock threads.  Scratch layout (words): [0, nblk) counts per
// workgroup, then exclusive offsets in place; [nblk, nblk + kIt kWaves nblk) the
// straddle mask of every (workgroup, round, wave).
constexpr int kWaves = kSurfBlock / 64;
constexpr int kIt = 16;
constexpr long kSpan = (long)kIt * kSurfBlock;

// Workgroup b of a launch of G runs on XCD b % 8; the span it takes is
// xcd_span(b, G): the spans [k G/8, (k+1) G/8) (remainder spread over the first
// XCDs) go to XCD k in order, so the planes a workgroup shares with the next
// span stay in one XCD's L2.  A bijection on [0, G).
__device__ __forceinline__ long xcd_span(long b, long G) {
  const long per = G / 8, rem = G % 8, k = b % 8;
  return k * per + (k < rem ? k : rem) + b / 8;
}

// Pass 1: straddle masks (some of the 16 corners > e_f, some not) and straddling
// hypercubes per workgroup.  The lower corners of a span's hypercubes lie in one run of
// cells (the next row's and the next eta included), the upper ones in another: the
// workgroup reads both runs of both slices once, in order, keeps a bit per cell (e > e_f)
// in LDS, and takes the 16 corners from there.  Bound by reading e, 2.1 times, against 8
// loads per hypercube through the caches and a wait for each of 16 rounds of them before
// (201x201x105: 37 -> 24 us).
// Runs too long for the LDS (ne of thousands) are read corner by corner.
constexpr int kCountBlock = 1024;
constexpr int kRunWords = 288;  // 64-cell words of a run

__global__ __launch_bounds__(kCountBlock) void k_surface_count(SurfaceArgs a, int nblk) {
  constexpr int W = kCountBlock / 64;
  __shared__ int wc[W];
  __shared__ unsigned long long run[4][kRunWords + 1];
  const long ncube = cube_count(a.nx, a.ny, a.ne);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const gdouble* A = (const gdouble*)a.A;
  const gdouble* B = (const gdouble*)a.B;
  gullong* blk = (gullong*)a.blocks;
  const long sb = xcd_span(blockIdx.x, nblk);
  gullong* masks = blk + nblk + sb * kIt * kWaves;
  const unsigned cy = a.ny > 1 ? a.ny - 1 : 1, cz = a.ne > 1 ? a.ne - 1 : 1;
  const int sx = a.nx > 1 ? a.ny * a.ne : 0, sy = a.ny > 1 ? a.ne : 0, sz = a.ne > 1;
  auto first_corner = [&](long id) {
    const unsigned u = (unsigned)(id < ncube ? id : ncube - 1);
    const unsigned r = u / cz, k = u - r * cz, i = r / cy;
    return (int)((r + i * (a.ny - cy)) * a.ne + k);  // (i ny + j) ne + k
  };
  const int c0 = first_corner(sb * kSpan);
  const int len = first_corner(sb * kSpan + kSpan - 1) - c0 + sy + sz + 1;
  const bool fits = len <= 64 * kRunWords;
  if (fits) {
    const gdouble* S[4] = {A + c0, A + c0 + sx, B + c0, B + c0 + sx};
    for (int t = threadIdx.x; t - lane < len; t += 2 * kCountBlock) {
      double v[2][4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = t + h * kCountBlock;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[h][q] = c < len ? S[q][c] : a.eps_f;
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int w = (t - lane + h * kCountBlock) >> 6;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const unsigned long long m = __ballot(v[h][q] > a.eps_f);
          if (lane == 0 && w < kRunWords) run[q][w] = m;
        }
      }
    }
    __syncthreads();
  }
  int nw = 0;
  for (int it = 0; it < kSpan / kCountBlock; ++it) {
    const long id = sb * kSpan + (long)it * kCountBlock + threadIdx.x;
    unsigned long long mask = 0;
    if (id - lane < ncube) {  // (waves past the end of a small grid have nothing to look at)
      const int c = first_corner(id);
      unsigned any = 0, all = 3;  // of the corners on the lower and the upper eta
      auto corners = [&](unsigned two) {
        any |= two;
        all &= two;
      };
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          if (fits) {
            const int b = c - c0 + (r ? sy : 0);
            const unsigned* w = (const unsigned*)run[q] + (b >> 5);
            const unsigned two = __builtin_amdgcn_alignbit(w[1], w[0], b & 31);
            corners(sz ? two & 3 : 3 * (two & 1));
          } else {
            const gdouble* e = (q & 2 ? B : A) + (q & 1 ? sx : 0) + (r ? sy : 0) + c;
            corners((e[0] > a.eps_f ? 1u : 0u) | (e[sz] > a.eps_f ? 2u : 0u));
          }
        }
      mask = __ballot(id < ncube && any != 0 && all != 3);
    }
    if (lane == 0) masks[it * W + wave] = mask;
    nw += __popcll(mask);
  }
  if (lane == 0) wc[wave] = nw;
  __syncthreads();
  if (threadIdx.x == 0) {
    int n = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) n += wc[w];
    blk[sb] = (unsigned long long)n;
  }
}

// Pass 2 (one workgroup of 1024): exclusive prefix sums of the counts, in place
// (each thread sums a run of consecutive counts, one workgroup-wide scan of the
// run totals, then each thread writes its run), and the total into *count.
__global__ __launch_bounds__(1024) void k_surface_offsets(SurfaceArgs a, int nblk) {
  __shared__ long long part[16];
  gullong* blk = (gullong*)a.blocks;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (nblk + 1023) / 1024;
  const int i0 = tid * per;
  long long loc = 0;
  for (int q = 0; q < per; ++q)
    if (i0 + q < nblk) loc += (long long)blk[i0 + q];
  long long x = loc;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const long long y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) part[wave] = x;
  __syncthreads();
  if (wave == 0) {
    long long p = lane < 16 ? part[lane] : 0;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const long long y = __shfl_up(p, o);
      if (lane >= o) p += y;
    }
    if (lane < 16) part[lane] = p;
  }
  __syncthreads();
  long long run = x - loc + (wave ? part[wave - 1] : 0);  // exclusive
  for (int q = 0; q < per; ++q)
    if (i0 + q < nblk) {
      const long long v = (long long)blk[i0 + q];
      blk[i0 + q] = (unsigned long long)run;
      run += v;
    }
  if (tid == 1023) *(gullong*)a.count = (unsigned long long)run;
}

// Pass 3: every straddling hypercube writes its index to its slot, in hypercube
// order (workgroup offset, then round, wave and lane), from the pass-1 masks.
__global__ __launch_bounds__(kSurfBlock) void k_surface_compact(SurfaceArgs a, int nblk) {
  __shared__ long long moff[kIt * kWaves];
  const gullong* blk = (const gullong*)a.blocks;
  const long sb = xcd_span(blockIdx.x, nblk);
  const gullong* masks = blk + nblk + sb * kIt * kWaves;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (wave == 0) {  // exclusive offsets of the kIt * kWaves masks (one wave, 64 masks)
    static_assert(kIt * kWaves == 64, "one mask per lane");
    const long long c = __popcll(masks[lane]);
    long long x = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const long long y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    moff[lane] = (long long)blk[sb] + x - c;
  }
  __syncthreads();
  for (int it = 0; it < kIt; ++it) {
    const unsigned long long mask = masks[it * kWaves + wave];
    if (!((mask >> lane) & 1ull)) continue;
    const long long slot = moff[it * kWaves + wave] + __popcll(mask & ((1ull << lane) - 1ull));
    const long id = sb * kSpan + (long)it * kSurfBlock + threadIdx.x;
    if (slot < (long long)a.capacity) ((gdouble*)a.out)[slot * kSurfRec] = (double)id;
  }
}

// Pass 4: the element of every claimed slot below min(count, capacity).  Eight
// lanes share one element: the 16 corner values go through LDS, lane t
// evaluates the hot fraction of the 3-face normal to axis t/2 on side t%2 (its
// six tetrahedra) and the even lane of each pair forms S_mu; lane t divides out 4 of
// the 32 edges' sign changes and sums the centre along axis t % 4; every lane forms
// the corner weights (the same arithmetic in each); lane t interpolates fields t and
// t + 8.  Grid-stride over groups of elements; the
// loop bound is block-uniform, so every thread reaches each barrier.  Bound by its
// arithmetic (20 us of 33 for the 201x201x105 event's surface; 44 with the divisions of
// every tetrahedron's case and every edge in each lane), then by the corners' fields; 166
// VGPRs, three waves per SIMD (four or five spill: 42 and 67 us).
constexpr int kGroup = 8;
constexpr int kElemPerBlock = kSurfBlock / kGroup;

__global__ __launch_bounds__(kSurfBlock) __attribute__((amdgpu_waves_per_eu(3))) void k_surface_elem(SurfaceArgs a) {
  __shared__ double sphi[kElemPerBlock][17], sedge[kElemPerBlock][4][17];  // (17: banks)
  const gdouble* A = (const gdouble*)a.A;
  const gdouble* B = (const gdouble*)a.B;
  gdouble* outp = (gdouble*)a.out;
  const unsigned long long found = *(const gullong*)a.count;
  const long n = (long)(found < (unsigned long long)a.capacity ? found
                                                                : (unsigned long long)a.capacity);
  const int t = threadIdx.x & (kGroup - 1), g = threadIdx.x / kGroup;
  const int mu = t >> 1, side = t & 1;
  const double ext[4] = {a.tauB - a.tauA, a.dx, a.dy, a.de};
  const long ncell = (long)a.nx * a.ny * a.ne;
  // contiguous runs of element groups per workgroup, the runs of one XCD adjacent
  // (neighbouring elements share corner cells); the first min(grid, groups)
  // workgroups share the groups, so every XCD gets work
  const long ngrp = (n + kElemPerBlock - 1) / kElemPerBlock;
  const long G = (long)gridDim.x < ngrp ? (long)gridDim.x : ngrp;
  if ((long)blockIdx.x >= G) return;  // whole workgroup: before any barrier
  const long per = (ngrp + G - 1) / G, g0 = xcd_span(blockIdx.x, G) * per;
  const long g1 = g0 + per < ngrp ? g0 + per : ngrp;
  for (long base = g0 * kElemPerBlock; base < g1 * kElemPerBlock; base += kElemPerBlock) {
    const long slot = base + g;
    const bool act = slot < n;
    gdouble* r = outp + (act ? slot : 0) * kSurfRec;
    const int id = act ? (int)r[0] : 0;
    const Cube q = cube_of(a, id);
    double v2[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int c = 2 * t + u;
      const gdouble* S = (c & 8) ? B : A;
      v2[u] = S[q.cell[c & 7]] - a.eps_f;
      sphi[g][c] = v2[u];
    }
    __syncthreads();
    double w[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) w[b] = sphi[g][face_corner(mu, side, b)];
    const double f = cube_hot(w);
    const double f_other = __shfl_xor(f, 1);
    // the sign change along each edge (corner c, axis): lane t those of axis t % 4 from the
    // corners 4 (t / 4) ... of the 8 without that axis' bit
    const int ax0 = t & 3, low = (8 >> ax0) - 1;
#pragma unroll
    for (int n4 = 0; n4 < 4; ++n4) {
      const int b = 4 * (t >> 2) + n4, c = ((b & ~low) << 1) | (b & low);
      const double p1 = sphi[g][c], p2 = sphi[g][c | (low + 1)];
      sedge[g][ax0][c] = p1 / (p1 - p2);
    }
    // hot corners of the element (bit c), and per axis the edges that cross
    const int sh = (int)(threadIdx.x & 63 & ~(kGroup - 1));
    auto spread = [](unsigned x) {  // bit i -> bit 2 i
      x = (x | x << 4) & 0x0f0fu;
      x = (x | x << 2) & 0x3333u;
      return (x | x << 1) & 0x5555u;
    };
    const unsigned hot = spread((unsigned)(__ballot(v2[0] > 0.0) >> sh) & 0xffu) |
                         spread((unsigned)(__ballot(v2[1] > 0.0) >> sh) & 0xffu) << 1;
    const unsigned cr[4] = {(hot ^ hot >> 8) & 0x00ffu, (hot ^ hot >> 4) & 0x0f0fu,
                            (hot ^ hot >> 2) & 0x3333u, (hot ^ hot >> 1) & 0x5555u};
    const int ncross = __popc(cr[0]) + __popc(cr[1]) + __popc(cr[2]) + __popc(cr[3]);
    __syncthreads();
    // the centre along axis t % 4: the edges in order of corner, then axis
    double cm = 0.0;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const double s = sedge[g][ax0][c], bit = (double)((c >> (3 - ax0)) & 1);
#pragma unroll
      for (int ax = 0; ax < 4; ++ax)
        if (!(c & (8 >> ax))) cm += (cr[ax] >> c) & 1 ? (ax == ax0 ? s : bit) : 0.0;
    }
    cm /= (double)ncross;
    double cen[4];
#pragma unroll
    for (int a2 = 0; a2 < 4; ++a2) cen[a2] = __shfl(cm, sh + a2);
    const double tc = a.tauA + cen[0] * ext[0];
    if (act) {
      if (side == 0) {  // S_mu = V_mu (f_lo - f_hi), V_mu over the other axes in order
        double V = 1.0;
#pragma unroll
        for (int ax = 0; ax < 4; ++ax)
          if (ax != mu) V *= ext[ax];
        r[5 + mu] = (a.cart ? 1.0 : tc) * (V * (f - f_other));
      }
      if (t == 0) {
        r[1] = tc;
        r[2] = ((double)q.i - 0.5 * (a.nx - 1)) * a.dx + (a.nx > 1 ? cen[1] * a.dx : 0.0);
        r[3] = ((double)q.j - 0.5 * (a.ny - 1)) * a.dy + (a.ny > 1 ? cen[2] * a.dy : 0.0);
        r[4] = ((double)q.k - 0.5 * (a.ne - 1)) * a.de + (a.ne > 1 ? cen[3] * a.de : 0.0);
        r[23] = 0.0;
      }
      double wgt[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        double wv = 1.0;
#pragma unroll
        for (int a2 = 0; a2 < 4; ++a2) {
          const int bb = (c >> (3 - a2)) & 1;
          wv *= bb ? cen[a2] : 1.0 - cen[a2];
        }
        wgt[c] = wv;
      }
#pragma unroll 1  // (both at once spill)
      for (int h2 = 0; h2 < 2; ++h2) {
        const int fld = t + kGroup * h2;
        if (fld >= 14) continue;
        double v = 0.0;
        if (fld < a.nf) {
#pragma unroll
          for (int c = 0; c < 16; ++c) {
            const gdouble* S = (c & 8) ? B : A;
            v += wgt[c] * S[(long)fld * ncell + (long)q.cell[c & 7]];
          }
        }
        if (fld == 0)
          r[22] = v;
        else
          r[8 + fld] = v;  // u~ at 9..11, pi~ at 12..21
      }
    }
    __syncthreads();
  }
}

}  // namespace

size_t surface_scratch_words(long nx, long ny, long ne) {
  return (size_t)((cube_count(nx, ny, ne) + kSpan - 1) / kSpan) * (1 + kIt * kWaves) + 1;
}

int launch_surface(const SurfaceArgs& a, hipStream_t s) {
  const long nblk = (cube_count(a.nx, a.ny, a.ne) + kSpan - 1) / kSpan;
  hipLaunchKernelGGL(k_surface_count, dim3((unsigned)nblk), dim3(kCountBlock), 0, s, a, (int)nblk);
  hipLaunchKernelGGL(k_surface_offsets, dim3(1), dim3(1024), 0, s, a, (int)nblk);
  if (a.capacity > 0) {
    hipLaunchKernelGGL(k_surface_compact, dim3((unsigned)nblk), dim3(kSurfBlock), 0, s, a,
                       (int)nblk);
    // enough workgroups for the buffer, at most 16 per CU's worth of the chip
    const long eb = std::min<long>((a.capacity + kElemPerBlock - 1) / kElemPerBlock, 4096);
    hipLaunchKernelGGL(k_surface_elem, dim3((unsigned)eb), dim3(kSurfBlock), 0, s, a);
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ktmi
