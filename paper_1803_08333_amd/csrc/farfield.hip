// Far field and radar cross section of RWG currents (Sec. 4), FP64.
//
// F_r(d) = int j_r exp(-i k dhat_d . x) dS: on cell c the RWG current is
// sum_i j_m sigma_i (x - v_i)/(2 A_c) (v_i opposite local edge i) and the
// rule's weights sum to one, so F = sum_p J_r(p) exp(-i k dhat . x_p) over the
// 7 C quadrature points, J_r(p) = w_q/2 sum_i sigma_i j_m (x_q - v_i), and
// sigma_r(d) = k^2/(4 pi) |F - dhat (dhat . F)|^2 (unit incident amplitude).
// With js != nullptr, j is the loop (divergence-free) part of the current and
// js its star part: a loop current carries no net current, so its phase
// factor is taken as exp(-i t) - 1 = -2 sin^2(t/2) - i sin t, without
// cancellation at any k; js takes the plain phase.
//
// The sum is a product of the phases (directions x points) with the point
// currents (points x 6 real columns per right-hand side) on the FP64 matrix
// cores (v_mfma_f64_16x16x4): each lane forms the sine and cosine of one
// direction and point, which is its own operand entry, and every right-hand
// side shares them.  The current of a point is formed once per call
// (k_ff_current) instead of once per direction.
//
// Bound: FP64 arithmetic, about 40 operations per sine and cosine and 24 per
// right-hand side (6 columns, twice, as MFMA; padded to 16 columns), 7 C ndir
// of each.  One workgroup takes 16 directions, a slice of the points and up to
// 8 of the column groups; its four waves take every fourth group of four
// points.  Level 4 (C = 5120), 362 directions, 4 currents: 61 us for the sums
// and 14 for the two small kernels around them, 100 us a call (306 with one
// workgroup per direction and right-hand side, each forming every phase and
// every point current again).  A body of 80 to 320 cells takes 36 to 40 us, most
// of them the call's own.
#include <algorithm>
#include <cmath>

#include "farpair.h"
#include "internal.h"

namespace rfcmp {
namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int kFfDirs = 16;         // directions per workgroup (an MFMA operand)
// workgroups of a launch: what the chip holds at once (registers: 4, 3 or 2
// per compute unit), since a second round would run nearly empty
constexpr int ff_waves(int ng) { return ng == 1 ? 4 : ng == 2 ? 3 : 2; }
constexpr int kFfWidest = 8;        // column groups per workgroup, at most
constexpr int kFfDirChunk = 16384;  // directions per launch (bounds the partial sums)

// sin and cos of t.  Up to |t| = 1e5 (a body of 16 000 wavelengths) the
// nearest multiple n of pi/2 is taken off with pi/2 as the sum of two doubles
// (Cody and Waite's reduction; n times what the two leave out is below 1e-27),
// which leaves |r| <= pi/4 rounded once to double, by at most 2^-54.  r goes
// through the Taylor series of both functions (the terms left out are below
// 2^-58 of either), the cosine's as w = 1 - r^2/2 with what rounding took from w
// added back to the rest of the series, as fdlibm does.  In all 1.2e-16 absolute,
// 2.2e-16 relative (against 64-bit values over |t| <= 1e5).  Beyond, the
// library's.  About 35 operations where the library's takes over 100.
constexpr double kPio2Hi = 1.57079632679489655800e+00;
constexpr double kPio2Lo = 6.12323399573676603587e-17;
__device__ inline void ff_sincos(double t, double& sn, double& cs) {
  if (!(fabs(t) <= 1e5)) {
    sincos(t, &sn, &cs);
    return;
  }
  const double n = rint(t * 0.63661977236758134308);
  const double r = fma(-n, kPio2Lo, fma(-n, kPio2Hi, t));
  const double z = r * r;
  double a = 1.0 / 355687428096000.0;         // 1/17!
  a = fma(a, z, -1.0 / 1307674368000.0);      // 1/15!
  a = fma(a, z, 1.0 / 6227020800.0);          // 1/13!
  a = fma(a, z, -1.0 / 39916800.0);           // 1/11!
  a = fma(a, z, 1.0 / 362880.0);              // 1/9!
  a = fma(a, z, -1.0 / 5040.0);               // 1/7!
  a = fma(a, z, 1.0 / 120.0);
  a = fma(a, z, -1.0 / 6.0);
  const double s = fma(r * z, a, r);
  double b = -1.0 / 6402373705728000.0;       // 1/18!
  b = fma(b, z, 1.0 / 20922789888000.0);      // 1/16!
  b = fma(b, z, -1.0 / 87178291200.0);        // 1/14!
  b = fma(b, z, 1.0 / 479001600.0);           // 1/12!
  b = fma(b, z, -1.0 / 3628800.0);            // 1/10!
  b = fma(b, z, 1.0 / 40320.0);               // 1/8!
  b = fma(b, z, -1.0 / 720.0);
  b = fma(b, z, 1.0 / 24.0);
  const double hz = 0.5 * z, w = 1.0 - hz;
  const double c = w + fma(z * z, b, (1.0 - w) - hz);
  const int q = (int)n;
  const double u = (q & 1) ? c : s, v = (q & 1) ? s : c;
  sn = (q & 2) ? -u : u;
  cs = ((q + 1) & 2) ? -v : v;
}

// Up to kFfDirArgs directions ride in the arguments of the call's first kernel
// (a copy from the caller's pageable memory takes longer than the kernel).
constexpr int kFfDirArgs = 128;
struct DirArgs {
  int n = 0;
  double d[3 * kFfDirArgs];
};

struct FfMesh {
  int N;
  const int* cell_edge;
  const float* sgn;
  const double* vtx;
  RuleArgs rule;
};
// Component k of the position of quadrature point q of the cell with vertices P.
__device__ inline double ff_position(const FfMesh& m, const double* P, int q, int k) {
  return fma(m.rule.bary[q][2], P[6 + k], fma(m.rule.bary[q][1], P[3 + k], m.rule.bary[q][0] * P[k]));
}
// Component k of the current there (less its weight) of the three edges' values,
// rounded alike wherever it is formed.
__device__ inline double ff_current(const double* P, const double (&sg)[3], double xk, int k, double j0, double j1,
                                    double j2) {
  return fma(sg[2] * (xk - P[6 + k]), j2, fma(sg[1] * (xk - P[3 + k]), j1, sg[0] * (xk - P[k]) * j0));
}

// Positions x [n][3] and point currents J [n][ld] of the points p0 .. p0 + n - 1
// (7 c + q), column 6 r + 2 k + (0: real, 1: imaginary) of component k of
// right-hand side r; js (nullable) into Js.
__global__ __launch_bounds__(256) void k_ff_current(int p0, int n, int nr, int ld, const FfMesh m,
                                                    const double2* __restrict__ j, const double2* __restrict__ js,
                                                    double* __restrict__ x, double* __restrict__ J,
                                                    double* __restrict__ Js, DirArgs da, double* __restrict__ dirs) {
  if (blockIdx.x == 0)
    for (int e = threadIdx.x; e < 3 * da.n; e += 256) dirs[e] = da.d[e];
  const unsigned t = blockIdx.x * 256u + threadIdx.x;  // n nr < 2^26 (1 GB of point currents)
  if (t >= (unsigned)n * (unsigned)nr) return;
  const int r = (int)(t % (unsigned)nr), pt = (int)(t / (unsigned)nr);
  const long p = pt;
  const int c = (p0 + pt) / kQ, q = (p0 + pt) % kQ;
  double P[9], sg[3];
  for (int k = 0; k < 9; ++k) P[k] = m.vtx[(long)c * 9 + k];
  double2 jc[3], jsc[3];
  for (int i = 0; i < 3; ++i) {
    const long e = (long)r * m.N + m.cell_edge[3 * c + i];
    jc[i] = j[e];
    jsc[i] = js ? js[e] : make_double2(0.0, 0.0);
    sg[i] = 0.5 * (double)m.sgn[3 * c + i];
  }
  const double wq = m.rule.wd[q];
  for (int k = 0; k < 3; ++k) {
    const double xk = ff_position(m, P, q, k);
    if (r == 0) x[3 * p + k] = xk;
    const long o = p * ld + 6 * r + 2 * k;
    *reinterpret_cast<double2*>(J + o) = make_double2(wq * ff_current(P, sg, xk, k, jc[0].x, jc[1].x, jc[2].x),
                                                      wq * ff_current(P, sg, xk, k, jc[0].y, jc[1].y, jc[2].y));
    if (js)
      *reinterpret_cast<double2*>(Js + o) = make_double2(wq * ff_current(P, sg, xk, k, jsc[0].x, jsc[1].x, jsc[2].x),
                                                         wq * ff_current(P, sg, xk, k, jsc[0].y, jsc[1].y, jsc[2].y));
  }
}

// Partial sums of a slice of `ps` points (a multiple of 32) for 16 directions
// and NG of the ng 16-column groups:
// part[slice][tile][cos, sin][group][direction][column].  The columns of J
// beyond 6 nr hold anything: a column only reaches itself.
template <int NG, bool SPLIT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(ff_waves(NG))))
void k_ff_sum(int P, int ndir, int ps, int ng, double kk, const double* __restrict__ dirs, const double* __restrict__ x,
              const double* __restrict__ J, const double* __restrict__ Js, double* __restrict__ part) {
  const int ld = 16 * ng, g0 = blockIdx.z * NG;
  J += 16 * g0;
  Js += 16 * g0;
  __shared__ double red[2][2 * NG * 4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, col = lane & 15;
  const int d = min(blockIdx.x * kFfDirs + col, (unsigned)ndir - 1);
  const double d0 = dirs[3 * d], d1 = dirs[3 * d + 1], d2 = dirs[3 * d + 2];
  dbl4 ac[NG], as[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) ac[g] = as[g] = dbl4{0.0, 0.0, 0.0, 0.0};
  const int p_end = min(P, (int)(blockIdx.y + 1) * ps);
  // the operands of the next group are loaded while this one's phases and
  // products run (a round trip to memory per group otherwise)
  struct Operands {
    double b[NG], bs[SPLIT ? NG : 1], x0, x1, x2;
  };
  auto load = [&](Operands& o, int p0) {
    const long pc = min(p0 + (lane >> 4), P - 1);
    o.x0 = x[3 * pc];
    o.x1 = x[3 * pc + 1];
    o.x2 = x[3 * pc + 2];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      o.b[g] = J[pc * ld + 16 * g + col];
      if (SPLIT) o.bs[g] = Js[pc * ld + 16 * g + col];
    }
  };
  auto products = [&](const Operands& o, int p0) {
    const double ph = kk * fma(d2, o.x2, fma(d1, o.x1, d0 * o.x0));  // rounded alike in every instantiation
    double sn, cs;
    ff_sincos(ph, sn, cs);
    double lc = cs;
    if (SPLIT) {
      double h, unused;
      ff_sincos(0.5 * ph, h, unused);
      lc = -2.0 * h * h;
    }
    if (p0 + (lane >> 4) >= p_end) sn = cs = lc = 0.0;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      ac[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(lc, o.b[g], ac[g], 0, 0, 0);
      as[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(sn, o.b[g], as[g], 0, 0, 0);
      if (SPLIT) {
        ac[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(cs, o.bs[g], ac[g], 0, 0, 0);
        as[g] = __builtin_amdgcn_mfma_f64_16x16x4f64(sn, o.bs[g], as[g], 0, 0, 0);
      }
    }
  };
  Operands oa, ob;
  int p0 = blockIdx.y * ps + 4 * w;
  load(oa, p0);
  for (; p0 < p_end; p0 += 32) {
    load(ob, p0 + 16);
    products(oa, p0);
    load(oa, p0 + 32);
    products(ob, p0 + 16);
  }
  // the four waves' sums, (0 + 1) + (2 + 3); wave 0 ends with the cosines', wave
  // 2 with the sines'.  Value v of lane l: direction 4 v + l / 16, column l % 16
  auto put = [&](double(*dst)[64], const dbl4(&a)[NG]) {
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) dst[4 * g + v][lane] = a[g][v];
  };
  auto add = [&](dbl4(&a)[NG], const double(*src)[64]) {
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) a[g][v] += src[4 * g + v][lane];
  };
  double(*mine)[64] = red[w >> 1];
  if (w & 1) {
    put(mine, ac);
    put(mine + 4 * NG, as);
  }
  __syncthreads();
  if (!(w & 1)) {
    add(ac, mine);
    add(as, mine + 4 * NG);
    put(mine, w == 0 ? as : ac);
  }
  __syncthreads();
  if (w & 1) return;
  double* o = part + ((long)blockIdx.y * gridDim.x + blockIdx.x) * (2 * ng * 256) + g0 * 256;
  auto out = [&](dbl4(&a)[NG], const double(*src)[64], double* dst) {
    add(a, src);
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) dst[g * 256 + (4 * v + (lane >> 4)) * 16 + col] = a[g][v];
  };
  if (w == 0)
    out(ac, red[1], o);
  else
    out(as, red[0], o + ng * 256);
}

// The slices' sums in order (five interleaved sums, added in order), then
// Re F = C_re + S_im, Im F = C_im - S_re (exp(-i t) = cos t - i sin t) and the
// RCS.  One workgroup per 16 directions and R right-hand sides: threads (part,
// sum), R sums (cos or sin, direction, column) each.  F [nr][ndir_all][3], rcs
// [nr][ndir_all] from direction dir0 on.  Bound: the partial sums' bytes.  One
// right-hand side takes 48 bytes of a 128-byte line, so with R = 1 the line is
// fetched for each of the three it holds, by as many XCDs; eight take whole
// lines.
constexpr int kFfParts = 5, kFfSums = 2 * kFfDirs * 6;
template <int R>
constexpr int kFfAhead = R == 1 ? 16 : 2;  // slices in flight
template <int R>
__global__ __launch_bounds__(kFfParts * kFfSums) void k_ff_finish(int ndir, int nr, int ng, int nslice, double kk,
                                                                  const double* __restrict__ dirs,
                                                                  const double* __restrict__ part, long ndir_all,
                                                                  long dir0, double2* __restrict__ F,
                                                                  double* __restrict__ rcs) {
  __shared__ double red[kFfParts][kFfSums * R];
  const int t = threadIdx.x, q = t / kFfSums, t0 = t % kFfSums, r0 = blockIdx.y * R;
  const long stride = (long)gridDim.x * (2 * ng * 256);
  const double* src = part + (long)blockIdx.x * (2 * ng * 256);
  int off[R];
  double v[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int e = t0 + kFfSums * k, c = min(6 * r0 + e % (6 * R), 6 * nr - 1);  // column of the pass
    off[k] = (e / (6 * R * kFfDirs) * ng + c / 16) * 256 + e / (6 * R) % kFfDirs * 16 + c % 16;
    v[k] = 0.0;
  }
#pragma unroll kFfAhead<R>
  for (int u = q; u < nslice; u += kFfParts)
#pragma unroll
    for (int k = 0; k < R; ++k) v[k] += src[u * stride + off[k]];
#pragma unroll
  for (int k = 0; k < R; ++k) red[q][t0 + kFfSums * k] = v[k];
  __syncthreads();
  if (q == 0)
#pragma unroll
    for (int k = 0; k < R; ++k) {
      for (int u = 1; u < kFfParts; ++u) v[k] += red[u][t0 + kFfSums * k];
      red[0][t0 + kFfSums * k] = v[k];
    }
  __syncthreads();
  const int row = t % kFfDirs, d = blockIdx.x * kFfDirs + row, r = r0 + t / kFfDirs;
  if (t >= kFfDirs * R || d >= ndir || r >= nr) return;
  const double* c = &red[0][6 * (R * row + t / kFfDirs)];
  const double* sn = c + 6 * R * kFfDirs;
  double f[6];
  for (int k = 0; k < 3; ++k) {
    f[2 * k] = c[2 * k] + sn[2 * k + 1];
    f[2 * k + 1] = c[2 * k + 1] - sn[2 * k];
  }
  const long o = (long)r * ndir_all + dir0 + d;
  for (int k = 0; k < 3; ++k) F[3 * o + k] = make_double2(f[2 * k], f[2 * k + 1]);
  if (rcs) {
    const double dh[3] = {dirs[3 * d], dirs[3 * d + 1], dirs[3 * d + 2]};
    const double pr = dh[0] * f[0] + dh[1] * f[2] + dh[2] * f[4];  // dhat . F
    const double pi = dh[0] * f[1] + dh[1] * f[3] + dh[2] * f[5];
    double s = 0.0;
    for (int k = 0; k < 3; ++k) {
      const double tr = f[2 * k] - dh[k] * pr, ti = f[2 * k + 1] - dh[k] * pi;
      s += tr * tr + ti * ti;
    }
    rcs[o] = kk * kk / (4.0 * M_PI) * s;
  }
}

template <int NG>
void ff_launch(bool split, dim3 grid, hipStream_t s, int P, int ndir, int ps, int ng, double kk, const double* dirs,
               const double* x, const double* J, const double* Js, double* part) {
  if (split)
    hipLaunchKernelGGL((k_ff_sum<NG, true>), grid, dim3(256), 0, s, P, ndir, ps, ng, kk, dirs, x, J, Js, part);
  else
    hipLaunchKernelGGL((k_ff_sum<NG, false>), grid, dim3(256), 0, s, P, ndir, ps, ng, kk, dirs, x, J, J, part);
}

// Points per slice.  It depends on the body alone, and so does the order in
// which a current's points are summed: its far field has the same bits whichever
// currents and directions share the call.  Long slices leave a call of few
// directions few workgroups, short ones one of many directions much to write
// and add up: in proportion to the root of the points both stay small (of 1.4
// to 4.6 times the root, over bodies of 80 to 20 480 cells, 1 to 37 currents and
// 1 to 720 directions, 2.0 to 3.6 were within 2 % on the mean, 1.4 and 4.6 slower).
int ff_slice(int64_t P) { return 32 * (int)std::ceil(2.8 * std::sqrt((double)P) / 32.0); }

// Column groups per workgroup: the phases, about five groups' worth of products,
// are formed once per workgroup, so the width that pads least does the least
// work; but a small body gives few workgroups, which run at about two thirds of a
// full chip's rate.  The width whose larger bound is least: at 5120 cells, 181
// directions and 16 currents (6 groups) w = 6, 132 us a call (148 with w = 8),
// with 37 directions and 4 currents w = 2, 58 us (68 with w = 8).
int ff_width(int need, int tiles, int slices) {
  int w = 1;
  double least = 0.0;
  for (int c = 1; c <= kFfWidest; ++c) {
    const double cost = (5.0 + c) * std::max((double)tiles * ((need + c - 1) / c) * slices / 256.0, 1.4);
    if (c == 1 || cost <= least) {
      least = cost;
      w = c;
    }
  }
  return w;
}

// One call's passes and memory: `per` right-hand sides, `dch` directions (a
// multiple of 16) and `sch` slices at a time, in at most about `budget` bytes.
// The order of the sums is the same in every plan.  Fewer slices at a time cost
// nothing while the launches fill the chip, fewer right-hand sides form the
// phases again.
struct FfPlan {
  int per, dch, sch, w, nz;
  size_t nj, npart, bytes;  // doubles of the point currents and of the partial sums; all bytes
  bool least;               // nothing left to shrink
};
FfPlan ff_plan(int64_t P, int ps, int ns, int nrhs, int ndir, bool split, size_t budget) {
  FfPlan p{std::min(nrhs, 4096), (int)round_up(std::min(ndir, kFfDirChunk), kFfDirs), ns, 1, 1, 0, 0, 0, false};
  for (;;) {
    const int need = (6 * p.per + 15) / 16, tiles = p.dch / kFfDirs;
    p.w = ff_width(need, tiles, p.sch);
    p.nz = (need + p.w - 1) / p.w;
    const size_t points = (size_t)std::min<int64_t>(P, (int64_t)p.sch * ps), ng = (size_t)p.nz * p.w;
    p.nj = points * 16 * ng * (split ? 2 : 1);
    p.npart = (size_t)ns * tiles * 2 * ng * 256;
    p.bytes = sizeof(double) * (3 * (size_t)ndir + 3 * points + p.nj + p.npart);
    p.least = p.per == 1 && p.dch == kFfDirs && p.sch == 1;
    if (p.bytes <= budget || p.least) return p;
    if (p.npart > p.nj && p.dch > kFfDirs)
      p.dch = (int)round_up(p.dch / 2, kFfDirs);
    else if (p.sch > 1 && ((int64_t)p.sch * tiles * p.nz >= 2048 || p.per == 1))
      p.sch = (p.sch + 1) / 2;
    else if (p.per > 1)
      p.per = (p.per + 1) / 2;
    else
      p.dch = (int)round_up(p.dch / 2, kFfDirs);
  }
}

}  // namespace

rfcmp_status far_field(rfcmp_op op, const double2* j, const double2* js, int nrhs, const double* dirs, int ndir,
                       double2* F, double* rcs, hipStream_t s) {
  rfcmp_mesh mesh = op->mesh;
  const MeshDev& D = mesh->d;
  const int64_t N = mesh->h.N, P = mesh->h.C * kQ;
  const int ps = ff_slice(P), ns = (int)((P + ps - 1) / ps);
  DevBuf buf;
  FfPlan pl;
  // 1 GB at most, a quarter of it at a time where that is refused
  for (size_t budget = (size_t)1 << 30;; budget /= 4) {
    pl = ff_plan(P, ps, ns, nrhs, ndir, js != nullptr, budget);
    const rfcmp_status st = buf.alloc(pl.bytes);
    if (st == RFCMP_OK) break;
    if (st != RFCMP_E_OOM || pl.least) return st;
  }
  const int ng = pl.nz * pl.w;
  double* part = buf.as<double>();
  double* J = part + pl.npart;
  double* Js = J + pl.nj / 2;
  double* x = J + pl.nj;
  double* dd = x + 3 * std::min<int64_t>(P, (int64_t)pl.sch * ps);
  DirArgs da;
  if (ndir <= kFfDirArgs) {
    da.n = ndir;
    std::copy(dirs, dirs + 3 * ndir, da.d);
  } else {
    RF_HIP(hipMemcpyAsync(dd, dirs, sizeof(double) * 3 * ndir, hipMemcpyHostToDevice, s));
  }
  const FfMesh fm{(int)N, D.cell_edge.as<int>(), D.sgn.as<float>(), D.vtx.as<double>(), rule_args()};
  using Sums = decltype(&ff_launch<1>);
  constexpr Sums kSums[kFfWidest] = {ff_launch<1>, ff_launch<2>, ff_launch<3>, ff_launch<4>,
                                     ff_launch<5>, ff_launch<6>, ff_launch<7>, ff_launch<8>};
  constexpr const char* kTags[kFfWidest] = {"farfield_w1", "farfield_w2", "farfield_w3", "farfield_w4",
                                            "farfield_w5", "farfield_w6", "farfield_w7", "farfield_w8"};
  const Sums sums = kSums[pl.w - 1];
  for (int r0 = 0; r0 < nrhs; r0 += pl.per) {
    const int nr = std::min(pl.per, nrhs - r0);
    for (int q0 = 0; q0 < ndir; q0 += pl.dch) {
      const int nd = std::min(pl.dch, ndir - q0);
      const unsigned nt = (unsigned)((nd + kFfDirs - 1) / kFfDirs);
      for (int s0 = 0; s0 < ns; s0 += pl.sch) {
        const int slices = std::min(pl.sch, ns - s0);
        const int64_t p0 = (int64_t)s0 * ps, points = std::min<int64_t>(P - p0, (int64_t)slices * ps);
        if (pl.sch < ns || q0 == 0)  // else the point currents are there
          hipLaunchKernelGGL(k_ff_current, dim3((unsigned)((points * nr + 255) / 256)), dim3(256), 0, s, (int)p0,
                             (int)points, nr, 16 * ng, fm, j + (int64_t)r0 * N,
                             js ? js + (int64_t)r0 * N : nullptr, x, J, Js, da, dd);
        ProfScope prof(kTags[pl.w - 1], s);
        sums(js != nullptr, dim3(nt, (unsigned)slices, (unsigned)pl.nz), s, (int)points, nd, ps, ng, op->k,
             dd + 3L * q0, x, J, Js, part + (size_t)s0 * nt * (2 * ng * 256));
      }
      // eight right-hand sides a workgroup where that leaves 16 of them
      const bool wide = nr >= 8 && (int64_t)nt * ((nr + 7) / 8) >= 16;
      const auto finish = wide ? k_ff_finish<8> : k_ff_finish<1>;
      hipLaunchKernelGGL(finish, dim3(nt, (unsigned)(wide ? (nr + 7) / 8 : nr)), dim3(kFfParts * kFfSums), 0, s, nd,
                         nr, ng, ns, op->k, dd + 3L * q0, part, (long)ndir, (long)q0, F + (int64_t)r0 * ndir * 3,
                         rcs ? rcs + (int64_t)r0 * ndir : nullptr);
    }
  }
  RF_HIP(hipGetLastError());
  RF_HIP(hipStreamSynchronize(s));
  return RFCMP_OK;
}

}  // namespace rfcmp
