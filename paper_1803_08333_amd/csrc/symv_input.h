// Device-side formation of a product input x[r][g] from a SymvInput (the
// fused gathers of the operator), shared by the dense symmetric products
// (symv.hip) and the sparse projector solves (spsolve.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "symv.h"

namespace rfcmp {

__device__ inline double2 csub2(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// x[r][g] of a SymvInput (g < n).
__device__ inline double2 input_entry(const SymvInput& in, int r, int g) {
  const double2* p0 = in.p[0] + r * in.stride[0];
  switch (in.mode) {
    case SymvInput::kSigmaT: {
      double sr = 0.0, si = 0.0;
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        const double2 v = p0[in.idx0[3 * g + l]];
        const double sg = in.sgn[3 * g + l];
        sr = fma(sg, v.x, sr);
        si = fma(sg, v.y, si);
      }
      return make_double2(sr, si);
    }
    case SymvInput::kLambdaT: {
      double sr = 0.0, si = 0.0;
      for (int q = in.idx0[g]; q < in.idx0[g + 1]; ++q) {
        const double2 v = p0[in.idx1[q]];
        const double sg = in.sgn[q];
        sr = fma(sg, v.x, sr);
        si = fma(sg, v.y, si);
      }
      return make_double2(sr, si);
    }
    case SymvInput::kVin: {
      const int cp = in.idx0[2 * g], cm = in.idx0[2 * g + 1];
      const double2* p1 = in.p[1] + r * in.stride[1];
      const double2* p2 = in.p[2] + r * in.stride[2];
      const double2 ul = csub2(p0[g], csub2(p1[cp], p1[cm]));
      const double2 ug = csub2(p2[cp], p2[cm]);
      const double ka = in.c[0], kb = in.c[1];
      return make_double2(-ka * ul.y - kb * ug.x, ka * ul.x - kb * ug.y);
    }
    case SymvInput::kMiddleW: {
      const int cp = in.idx0[2 * g], cm = in.idx0[2 * g + 1];
      const double2* p1 = in.p[1] + r * in.stride[1];
      const double2* p2 = in.p[2] + r * in.stride[2];
      const double2* p3 = in.p[3] + r * in.stride[3];
      const double2 lh = csub2(p0[in.idx1[2 * g]], p0[in.idx1[2 * g + 1]]);
      const double2 pl = csub2(p1[g], csub2(p2[cp], p2[cm]));
      const double2 ss = csub2(p3[cp], p3[cm]);
      return make_double2(in.c[0] * lh.x + in.c[1] * pl.x + in.c[2] * ss.x,
                          in.c[0] * lh.y + in.c[1] * pl.y + in.c[2] * ss.y);
    }
    case SymvInput::kProjLH: {
      const int cp = in.idx0[2 * g], cm = in.idx0[2 * g + 1];
      const double2* p1 = in.p[1] + r * in.stride[1];
      return csub2(p0[g], csub2(p1[cp], p1[cm]));
    }
    default:
      return p0[g];
  }
}

// x[r0 + u][g], u < NU, of a SymvInput, each in input_entry's order; 0 from nr
// on.  The loads of all are in flight together.
template <int NU>
__device__ inline void input_entries(const SymvInput& in, int r0, int nr, int g, double2 (&x)[NU]) {
  long o[NU];  // right-hand sides from nr on repeat the last one
#pragma unroll
  for (int u = 0; u < NU; ++u) o[u] = min(r0 + u, nr - 1);
  const double2* p0 = in.p[0];
  switch (in.mode) {
    case SymvInput::kSigmaT: {
      int e[3];
      double sg[3];
      double2 v[3][NU];
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        e[l] = in.idx0[3 * g + l];
        sg[l] = in.sgn[3 * g + l];
      }
#pragma unroll
      for (int l = 0; l < 3; ++l)
#pragma unroll
        for (int u = 0; u < NU; ++u) v[l][u] = p0[o[u] * in.stride[0] + e[l]];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        x[u] = make_double2(0.0, 0.0);
#pragma unroll
        for (int l = 0; l < 3; ++l) {
          x[u].x = fma(sg[l], v[l][u].x, x[u].x);
          x[u].y = fma(sg[l], v[l][u].y, x[u].y);
        }
      }
      break;
    }
    case SymvInput::kLambdaT: {
#pragma unroll
      for (int u = 0; u < NU; ++u) x[u] = make_double2(0.0, 0.0);
      const int q1 = in.idx0[g + 1];
      for (int q = in.idx0[g]; q < q1; ++q) {
        const int e = in.idx1[q];
        const double sg = in.sgn[q];
        double2 v[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) v[u] = p0[o[u] * in.stride[0] + e];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          x[u].x = fma(sg, v[u].x, x[u].x);
          x[u].y = fma(sg, v[u].y, x[u].y);
        }
      }
      break;
    }
    case SymvInput::kVin: {
      const int cp = in.idx0[2 * g], cm = in.idx0[2 * g + 1];
      const double ka = in.c[0], kb = in.c[1];
      double2 v[5][NU];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const double2 *p1 = in.p[1] + o[u] * in.stride[1], *p2 = in.p[2] + o[u] * in.stride[2];
        v[0][u] = p0[o[u] * in.stride[0] + g];
        v[1][u] = p1[cp];
        v[2][u] = p1[cm];
        v[3][u] = p2[cp];
        v[4][u] = p2[cm];
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const double2 ul = csub2(v[0][u], csub2(v[1][u], v[2][u])), ug = csub2(v[3][u], v[4][u]);
        x[u] = make_double2(-ka * ul.y - kb * ug.x, ka * ul.x - kb * ug.y);
      }
      break;
    }
    case SymvInput::kMiddleW: {
      const int cp = in.idx0[2 * g], cm = in.idx0[2 * g + 1], vp = in.idx1[2 * g], vm = in.idx1[2 * g + 1];
      double2 v[7][NU];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const double2 *q0 = p0 + o[u] * in.stride[0], *p2 = in.p[2] + o[u] * in.stride[2],
                      *p3 = in.p[3] + o[u] * in.stride[3];
        v[0][u] = q0[vp];
        v[1][u] = q0[vm];
        v[2][u] = in.p[1][o[u] * in.stride[1] + g];
        v[3][u] = p2[cp];
        v[4][u] = p2[cm];
        v[5][u] = p3[cp];
        v[6][u] = p3[cm];
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const double2 lh = csub2(v[0][u], v[1][u]), pl = csub2(v[2][u], csub2(v[3][u], v[4][u])),
                      ss = csub2(v[5][u], v[6][u]);
        x[u] = make_double2(in.c[0] * lh.x + in.c[1] * pl.x + in.c[2] * ss.x,
                            in.c[0] * lh.y + in.c[1] * pl.y + in.c[2] * ss.y);
      }
      break;
    }
    case SymvInput::kProjLH: {
      const int cp = in.idx0[2 * g], cm = in.idx0[2 * g + 1];
      double2 v[3][NU];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const double2* p1 = in.p[1] + o[u] * in.stride[1];
        v[0][u] = p0[o[u] * in.stride[0] + g];
        v[1][u] = p1[cp];
        v[2][u] = p1[cm];
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) x[u] = csub2(v[0][u], csub2(v[1][u], v[2][u]));
      break;
    }
    default: {
#pragma unroll
      for (int u = 0; u < NU; ++u) x[u] = p0[o[u] * in.stride[0] + g];
    }
  }
#pragma unroll
  for (int u = 0; u < NU; ++u)
    if (r0 + u >= nr) x[u] = make_double2(0.0, 0.0);
}

}  // namespace rfcmp
