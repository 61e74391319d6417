// Galerkin assembly of the EFIE blocks (Sec. 2 of the paper):
//   T_A[m,n] = int int f_m(r).f_n(r') G_k dS dS',
//   V[c,c']  = (A_c A_c')^-1 int_c int_c' G_k,     G_k = exp(ikR)/(4 pi R),
// with RWG pieces f_m|_c = sigma (r - r_m^c)/(2 A_c) (eq. RWGdef).
//
// Cell-pair formulation.  For the 3 x 3 local edges (i of c, j of c') the
// pair contributes
//   B[(c,i),(c',j)] = sigma_i sigma_j / (4 A_c A_c') int int (r - r_i).(r' - r_j) G_k,
// and T_A[m,n] sums the four B entries of the cell slots of m and n.
//
// Far pairs (FP32, 7 x 7 points): with r = x_c + rho, r' = x_c' + rho' and
// q_i = r_i - x_c (all O(h)), the block is
//   B = sigma sigma'/4 (I_rr' - q_i.I_r' - q'_j.I_r + q_i.q'_j I_0)
// over the normalised moments I_0 = sum w w' G, I_r = sum w w' rho G,
// I_r' = sum w w' rho' G, I_rr' = sum w w' rho.rho' G.  The centroid offset is
// formed in FP64 and every other length is O(h), so FP32 keeps its relative
// precision instead of losing (1/h)^2 to cancellation of O(1) coordinates.
//
// Near pairs (FP64): singular extraction G = 1/(4 pi R) + (exp(ikR) - 1)/(4 pi R);
// the 1/R part is integrated over the inner cell in closed form (Wilton et al.,
// IEEE TAP 1984; Graglia, IEEE TAP 1993), the bounded rest with 7 x 7 points,
// the outer cell is the lower-indexed one and self blocks are symmetrised.
#include <algorithm>
#include <climits>
#include <cmath>
#include <mutex>
#include <thread>
#include <vector>

#include "farpair.h"
#include "hmat.h"
#include "internal.h"

namespace rfcmp {

namespace {

// ------------------------------------------------------- cell pairs, dense T_A
// The dense blocks are formed in two passes over pairs (s <= t) of large edge
// tiles (asm_tile consecutive edges each).  k_cell_pairs forms the 3 x 3 block
// B[(a,i),(b,j)] of every cell pair (a, b) that the two tiles touch, into
// scratch, and k_gather_ta sums T_A[m,n] = (B[m+,n+] + B[m-,n-]) +
// (B[m+,n-] + B[m-,n+]) from it, for m in s and n in t, and writes both
// triangles: T_A is stored whole and exactly symmetric.  Between two different
// 64-edge tiles the cell of the lower one is the first cell of every pair;
// inside one tile the lower-indexed cell is, for (m, n) and (n, m) alike.
//
// A cell that two tiles touch is formed once for each, so the pass forms
// 1.1-1.2 times the unordered cell pairs at 2048-edge tiles, where 64-edge tiles
// (whose sums fit LDS, the form of k_assemble_list) take 1.9 on the spheres and
// 2.3 on the 96 x 48 torus.  Bound: FP32 VALU, about 28 instructions and three
// transcendentals per point pair and a fifth of that per cell pair for its
// entries (about 14 ms of the 17.4 at level 5); k_gather_ta streams the
// scratch, which is kept small so that it comes from the memory-side cache.
// Both passes: level 5 26.3 -> 17.4 ms, the torus 6.3 -> 3.5, level 2 0.074 ->
// 0.026.  One launch that formed a batch and summed the one before it was slower
// (its waves of the second kind took the places of the first).
//
// Near cell pairs (the self pairs among them) take their blocks from
// k_near_pairs (NB, FP64 singular extraction, run first) instead of the far
// rule: a tile pair that has near cell pairs (tile_near) looks each of its cell
// pairs up in the sorted near partners of its first cell.  V[c, c'] = I_0 of a
// far pair is written, with its mirror, where the tiles are those of the two
// cells' home edges and c is the first (k_near_pairs writes the near ones).
struct PairArgs {
  const int* st_ptr;    // cells of each tile: st_cell[st_ptr[t] ..], ascending
  const int* st_cell;
  const int* st_span;   // per entry of st_cell: lowest | highest << 16 of the 64-edge tiles of its edges in the tile
  const int2* st_pos;   // [N]: the slot 3 c + i of each edge in its c+ and c-, c counted in its tile
  const int* cell_home; // 64-edge tile of each cell's local edge 0
  const int4* pair;     // tile pairs (s, t)
  const long* off;      // their blocks in the scratch (entries)
  const uint8_t* near;  // tile pair t (t + 1)/2 + s has near cell pairs
  const int* np_ptr;
  const int* np_other;
  const int* np_code;
  const float2* NB;
  const double* cen;
  const float4* qoff;
  const float4* fvoff;
  const float* sgn;
  RuleArgs rule;
  float kk;
  int N;
  int hshift;           // 64-edge tiles per tile, as a shift
  int p0;               // first tile pair of the launch
  int rows;             // first cells per wave
};

constexpr int64_t kAsmScratch = 3 << 23;  // complex64 entries of a batch's blocks (192 MB)
constexpr int64_t kAsmBatch = 4096;       // tile pairs of a batch
constexpr int kAsmMinShift = 2;           // the smallest tiles, for want of memory: 256 edges

__global__ __launch_bounds__(256) void k_cell_pairs(const PairArgs g, float2* __restrict__ B, float2* __restrict__ Vm,
                                                    long ldV) {
  const int pi = g.p0 + blockIdx.z, bx = blockIdx.x, by = blockIdx.y;
  const int4 pr = g.pair[pi];
  const int s = pr.x, t = pr.y;
  const int a0 = g.st_ptr[s], na = g.st_ptr[s + 1] - a0, b0 = g.st_ptr[t], nb = g.st_ptr[t + 1] - b0;
  const int b = bx * 64 + (threadIdx.x & 63);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = (by * 4 + w) * g.rows, r1 = min(r0 + g.rows, na);
  if (bx * 64 >= nb || r0 >= na) return;
  float2* out = B + g.off[pi];
  const long ld = 3L * nb;
  const int cb = g.st_cell[b0 + min(b, nb - 1)];
  float4 qb[kQ], fb[3];
  float sb[3];
  double xb[3];
#pragma unroll
  for (int q = 0; q < kQ; ++q) qb[q] = g.qoff[(long)cb * kQ + q];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    fb[i] = g.fvoff[(long)cb * 3 + i];
    sb[i] = g.sgn[(long)cb * 3 + i];
    xb[i] = g.cen[(long)cb * 3 + i];
  }
  const int hb = g.cell_home[cb];
  const bool near = g.near[(long)t * (t + 1) / 2 + s] != 0;
  const bool in = b < nb, home_b = hb >> g.hshift == t;
  const int hi_b = g.st_span[b0 + min(b, nb - 1)] >> 16;
  for (int r = r0; r < r1; ++r) {
    const int ca = g.st_cell[a0 + r];
    // inside one tile a pair whose first cell has the higher index serves only
    // edges of a lower 64-edge tile with edges of a higher one
    if (s == t && r > b && (g.st_span[a0 + r] & 0xFFFF) >= hi_b) continue;
    float2* row = out + (3L * r) * ld + 3L * b;
    int code = -1;
    if (near) {  // binary search of cb among ca's near partners
      int lo = g.np_ptr[ca], hi = g.np_ptr[ca + 1];
      const int end = hi;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (g.np_other[mid] < cb)
          lo = mid + 1;
        else
          hi = mid;
      }
      if (lo < end && g.np_other[lo] == cb) code = g.np_code[lo];
    }
    if (code >= 0) {
      // near: B[(ca,i),(cb,j)] of the pair stored as (ca, cb) (code even) or (cb, ca)
      const float2* nbk = g.NB + (long)(code >> 1) * 9;
      if (in)
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int j = 0; j < 3; ++j) row[i * ld + j] = nbk[(code & 1) ? 3 * j + i : 3 * i + j];
      continue;
    }
    const double* xa = g.cen + 3L * ca;
    Moments M;
    far_moments(g.qoff + (long)ca * kQ, qb, (float)(xa[0] - xb[0]), (float)(xa[1] - xb[1]), (float)(xa[2] - xb[2]),
                g.rule, g.kk, M);
    const int ha = g.cell_home[ca];
    if (in && home_b && ha >> g.hshift == s && (ha < hb || (ha == hb && ca <= cb))) {
      const float2 v = make_float2(M.i0r, M.i0i);
      Vm[(long)ca * ldV + cb] = v;
      Vm[(long)cb * ldV + ca] = v;
    }
    if (in)
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
          row[i * ld + j] = b_entry(M, g.fvoff[3L * ca + i], fb[j], g.sgn[3L * ca + i], sb[j]);
  }
}

// One workgroup per pair of 64-edge tiles (I <= J) of a tile pair.  Workgroups
// go round robin to the 8 XCDs: an XCD takes whole rows of 64-edge tiles, so
// that the tiles that share B rows share an L2 (level 5: 6.4 -> 2.9 ms in all).
__global__ __launch_bounds__(256) void k_gather_ta(const PairArgs g, const float2* __restrict__ Bs,
                                                   float2* __restrict__ TA, long ldA) {
  __shared__ float2 tile[kEdgeTile][kEdgeTile + 1];
  const int per = 1 << (2 * g.hshift - 3), e0 = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  const int qi = g.p0 + blockIdx.y;
  const int4 pr = g.pair[qi];
  const int N = g.N;
  const long m0 = ((long)(pr.x << g.hshift) + (e0 >> g.hshift)) * kEdgeTile;
  const long n0 = ((long)(pr.y << g.hshift) + (e0 & ((1 << g.hshift) - 1))) * kEdgeTile;
  if (m0 > n0 || n0 >= N) return;
  const long ld = 3L * (g.st_ptr[pr.y + 1] - g.st_ptr[pr.y]);
  const float2* B = Bs + g.off[qi];
  const int2* pos = g.st_pos;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long n = n0 + lane;
  const int2 c = pos[min(n, (long)N - 1)];
  const bool diag = m0 == n0;
  for (int u = 0; u < 16; u += 4) {
    float2 pp[4], mm[4], pm[4], mp[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int2 r = pos[min(m0 + 16 * w + u + e, (long)N - 1)];
      // the lower cell first inside one tile
      auto at = [&](int a, int b) { return diag && a / 3 > b / 3 ? B[(long)b * ld + a] : B[(long)a * ld + b]; };
      pp[e] = at(r.x, c.x);
      mm[e] = at(r.y, c.y);
      pm[e] = at(r.x, c.y);
      mp[e] = at(r.y, c.x);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = 16 * w + u + e;
      const float2 v = make_float2((pp[e].x + mm[e].x) + (pm[e].x + mp[e].x), (pp[e].y + mm[e].y) + (pm[e].y + mp[e].y));
      if (m0 + row < N && n < N) TA[(m0 + row) * ldA + n] = v;
      tile[row][lane] = v;
    }
  }
  if (diag) return;
  __syncthreads();
  for (int row = w; row < kEdgeTile; row += 4)
    if (n0 + row < N && m0 + lane < N) TA[(n0 + row) * ldA + m0 + lane] = tile[lane][row];
}

// ------------------------------------------- dense tiles of a compressed T_A
// One workgroup per listed pair of 64-edge tiles (I <= J) forms the T_A entries
// (m in I, n in J) straight from the cell pairs of the cells the two tiles
// touch, and adds its B entries to the entries of its edges that lie in the
// tiles.  The sums run in LDS in a fixed order without atomics: t1 = B[m+,n+] +
// B[m-,n-], t2 = B[m+,n-] + B[m-,n+], the contributions whose row cell is c+
// added in a first phase and those whose row cell is c- in a second (each entry
// of t1 or t2 has one contribution per phase), and T_A = t1 + t2 -- the same
// pairing whatever the order of the cell pairs.  A diagonal tile takes each
// unordered cell pair once and adds it to (m, n) and (n, m) from the same
// registers.  V entries of the home cells of I and J go into the block's own
// dense V block.
constexpr int kAsmThreads = 1024;
struct CellL {
  float4 q[kQ];   // quadrature points minus centroid
  float4 fv[3];   // vertices minus centroid
  double cen[3];
  float sg[3];
  int rows;       // rows of the three local edges in this tile (8 bits each)
  int gid;        // cell index
  int home;       // home tile
};

__global__ __launch_bounds__(kAsmThreads) void k_assemble_list(const int* __restrict__ et_ptr,
                                                             const int* __restrict__ et_cell,
                                                             const int* __restrict__ et_rows,
                                                             const int* __restrict__ cell_home,
                                                             const double* __restrict__ cen,
                                                             const float4* __restrict__ qoff,
                                                             const float4* __restrict__ fvoff,
                                                             const float* __restrict__ sgn, float kk,
                                                             RuleArgs rule,
                                                             const int* __restrict__ np_ptr,
                                                             const int* __restrict__ np_other,
                                                             const int* __restrict__ np_code,
                                                             const float2* __restrict__ NB,
                                                             float2* __restrict__ TA,
                                                             float2* __restrict__ Vm,
                                                             const int2* __restrict__ lst,
                                                             const long* __restrict__ vdoff,
                                                             const int* __restrict__ cstart,
                                                             const int* __restrict__ ipc,
                                                             const float2* __restrict__ NV) {
  const long t = blockIdx.x;
  const int I = lst[t].x, Jt = lst[t].y;
  extern __shared__ __align__(16) unsigned char smem[];
  float2(*t1)[kEdgeTile] = reinterpret_cast<float2(*)[kEdgeTile]>(smem);
  float2(*t2)[kEdgeTile] = reinterpret_cast<float2(*)[kEdgeTile]>(smem + sizeof(float2) * kEdgeTile * kEdgeTile);
  CellL* cl = reinterpret_cast<CellL*>(smem + 2 * sizeof(float2) * kEdgeTile * kEdgeTile);
  const bool diag = I == Jt;
  const int i0 = et_ptr[I], nI = et_ptr[I + 1] - i0, j0 = et_ptr[Jt], nJ = et_ptr[Jt + 1] - j0;
  const int ncell = diag ? nI : nI + nJ;
  const int tid = threadIdx.x;
  for (int e = tid; e < 2 * kEdgeTile * kEdgeTile; e += kAsmThreads)
    reinterpret_cast<float2*>(smem)[e] = make_float2(0.f, 0.f);
  for (int e = tid; e < ncell * kQ; e += kAsmThreads) {
    const int k = e / kQ, q = e % kQ;
    const int g = k < nI ? et_cell[i0 + k] : et_cell[j0 + k - nI];
    cl[k].q[q] = qoff[(long)g * kQ + q];
  }
  for (int k = tid; k < ncell; k += kAsmThreads) {
    const int g = k < nI ? et_cell[i0 + k] : et_cell[j0 + k - nI];
    CellL& c = cl[k];
    c.rows = k < nI ? et_rows[i0 + k] : et_rows[j0 + k - nI];
    c.gid = g;
    c.home = cell_home[g];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      c.fv[i] = fvoff[(long)g * 3 + i];
      c.sg[i] = sgn[(long)g * 3 + i];
      c.cen[i] = cen[(long)g * 3 + i];
    }
  }
  __syncthreads();
  const CellL* cI = cl;
  const CellL* cJ = diag ? cl : cl + nI;
  const long vbase = vdoff[t];
  const int vcI = cstart[I], vcJ = cstart[Jt], vnJ = cstart[Jt + 1] - vcJ;
  const int total = nI * nJ;
  for (int base = 0; base < total; base += kAsmThreads) {
    const int p = base + tid;
    const int a = p / nJ, b = p % nJ;
    // a diagonal tile takes each unordered pair once, the self pairs too
    const bool act = p < total && (!diag || a <= b);
    float2 bv[3][3];
    int ra = 0, rb = 0;
    float sa[3] = {0, 0, 0}, sb[3] = {0, 0, 0};
    bool self = false;
    if (act) {
      const CellL& A = cI[a];
      const CellL& Bc = cJ[b];
      self = A.gid == Bc.gid;
      int code = -1;
      {  // binary search of Bc among A's near partners
        int lo = np_ptr[A.gid], hi = np_ptr[A.gid + 1];
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (np_other[mid] < Bc.gid)
            lo = mid + 1;
          else
            hi = mid;
        }
        if (lo < np_ptr[A.gid + 1] && np_other[lo] == Bc.gid) code = np_code[lo];
      }
      if (code >= 0) {
        // near: B[(A,i),(Bc,j)] of the pair stored as (A, Bc) (t = 0) or (Bc, A)
        const float2* nb = NB + (long)(code >> 1) * 9;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int j = 0; j < 3; ++j) bv[i][j] = nb[(code & 1) ? 3 * j + i : 3 * i + j];
        if (A.home == I && Bc.home == Jt) {
          const float2 v = NV[code >> 1];
          const int la = ipc[A.gid] - vcI, lb = ipc[Bc.gid] - vcJ;
          Vm[vbase + (long)la * vnJ + lb] = v;
          if (diag) Vm[vbase + (long)lb * vnJ + la] = v;
        }
      } else {
        Moments M;
        far_moments(A.q, Bc.q, (float)(A.cen[0] - Bc.cen[0]), (float)(A.cen[1] - Bc.cen[1]),
                        (float)(A.cen[2] - Bc.cen[2]), rule, kk, M);
        if (A.home == I && Bc.home == Jt) {
          const float2 v = make_float2(M.i0r, M.i0i);
          const int la = ipc[A.gid] - vcI, lb = ipc[Bc.gid] - vcJ;
          Vm[vbase + (long)la * vnJ + lb] = v;
          if (diag) Vm[vbase + (long)lb * vnJ + la] = v;
        }
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int j = 0; j < 3; ++j) bv[i][j] = b_entry(M, A.fv[i], Bc.fv[j], A.sg[i], Bc.sg[j]);
      }
      ra = A.rows;
      rb = Bc.rows;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        sa[i] = A.sg[i];
        sb[i] = Bc.sg[i];
      }
    }
    // phase 0: contributions whose row cell is the edge's c+, phase 1: c-
#pragma unroll
    for (int phase = 0; phase < 2; ++phase) {
      if (act) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const int r = (ra >> (8 * i)) & 0xFF;
          if (r == 0xFF) continue;
          const bool pa = sa[i] > 0.f;
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            const int c = (rb >> (8 * j)) & 0xFF;
            if (c == 0xFF) continue;
            const bool pb = sb[j] > 0.f;
            float2(*T)[kEdgeTile] = pa == pb ? t1 : t2;
            if ((phase == 0) == pa) {
              T[r][c].x += bv[i][j].x;
              T[r][c].y += bv[i][j].y;
            }
            if (diag && !self && (phase == 0) == pb) {
              T[c][r].x += bv[i][j].x;
              T[c][r].y += bv[i][j].y;
            }
          }
        }
      }
      __syncthreads();
    }
  }
  // the tile as it is (both triangles for a diagonal tile; zero beyond N)
  float2* out = TA + t * (long)(kEdgeTile * kEdgeTile);
  for (int e = tid; e < kEdgeTile * kEdgeTile; e += kAsmThreads) {
    const int r = e / kEdgeTile, c = e % kEdgeTile;
    out[e] = make_float2(t1[r][c].x + t2[r][c].x, t1[r][c].y + t2[r][c].y);
  }
}

// ---------------------------------------------------------------- near pairs
struct Pot {
  double S;       // int 1/R
  double W[3];    // int (r' - r)/R
};

// Closed-form potentials of the flat triangle P (CCW about its normal) at r.
__device__ Pot tri_potentials(const double P[3][3], const double r[3]) {
  double u0[3], v0[3], nr[3];
  for (int d = 0; d < 3; ++d) {
    u0[d] = P[1][d] - P[0][d];
    v0[d] = P[2][d] - P[0][d];
  }
  nr[0] = u0[1] * v0[2] - u0[2] * v0[1];
  nr[1] = u0[2] * v0[0] - u0[0] * v0[2];
  nr[2] = u0[0] * v0[1] - u0[1] * v0[0];
  const double nl = sqrt(nr[0] * nr[0] + nr[1] * nr[1] + nr[2] * nr[2]);
  for (int d = 0; d < 3; ++d) nr[d] /= nl;
  const double h = (r[0] - P[0][0]) * nr[0] + (r[1] - P[0][1]) * nr[1] + (r[2] - P[0][2]) * nr[2];
  const double ah = fabs(h);
  double rho[3];
  for (int d = 0; d < 3; ++d) rho[d] = r[d] - h * nr[d];
  Pot out{0.0, {0.0, 0.0, 0.0}};
  for (int e = 0; e < 3; ++e) {
    const double* a = P[e];
    const double* b = P[(e + 1) % 3];
    double lv[3];
    for (int d = 0; d < 3; ++d) lv[d] = b[d] - a[d];
    const double L = sqrt(lv[0] * lv[0] + lv[1] * lv[1] + lv[2] * lv[2]);
    for (int d = 0; d < 3; ++d) lv[d] /= L;
    // outward in-plane edge normal u = l x n
    const double uu[3] = {lv[1] * nr[2] - lv[2] * nr[1], lv[2] * nr[0] - lv[0] * nr[2],
                          lv[0] * nr[1] - lv[1] * nr[0]};
    double ta = 0, lm = 0, lp = 0, Rm2 = 0, Rp2 = 0;
    for (int d = 0; d < 3; ++d) {
      ta += (a[d] - rho[d]) * uu[d];
      lm += (a[d] - rho[d]) * lv[d];
      lp += (b[d] - rho[d]) * lv[d];
      Rm2 += (r[d] - a[d]) * (r[d] - a[d]);
      Rp2 += (r[d] - b[d]) * (r[d] - b[d]);
    }
    const double Rm = sqrt(Rm2), Rp = sqrt(Rp2);
    const double R02 = ta * ta + h * h;
    double f = 0.0;
    if (R02 > 1e-30 * L * L) {
      // ln((R+ + l+)/(R- + l-)) = ln((R- - l-)/(R+ - l+)); pick the form without cancellation
      f = (lp + lm >= 0.0) ? log((Rp + lp) / (Rm + lm)) : log((Rm - lm) / (Rp - lp));
    }
    double at = 0.0;
    if (ah > 0.0) at = atan(ta * lp / (R02 + ah * Rp)) - atan(ta * lm / (R02 + ah * Rm));
    out.S += ta * f - ah * at;
    const double wcoef = 0.5 * (R02 * f + lp * Rp - lm * Rm);
    for (int d = 0; d < 3; ++d) out.W[d] += wcoef * uu[d];
  }
  for (int d = 0; d < 3; ++d) out.W[d] -= h * out.S * nr[d];
  return out;
}

// Near pairs (c <= c'): outer cell c, inner cell c'.  A workgroup takes
// kNearPairs pairs: first one thread per (pair, outer point) forms the
// closed-form potentials and one per (pair, point pair) the bounded part's
// kernel, into LDS; then one thread per (pair, block entry) adds its terms in
// the order of the points.  (One thread per pair doing all of it left a few
// hundred waves on the chip, each a chain of 10^4 FP64 operations: 60 us at
// level 2 and 124 at level 4, now 18 and 102.)  31 pairs fill the rounds of
// every phase and leave room for three workgroups (level 4: 128 us with 15
// pairs, 105 with 26, 117 with 36).
constexpr int kNearPairs = 31;
__global__ __launch_bounds__(256) void k_near_pairs(long npairs, const int* __restrict__ pairs,
                                                    const double* __restrict__ vtx,
                                                    const double* __restrict__ area,
                                                    const float* __restrict__ sgn, double kk,
                                                    RuleArgs rule, float2* __restrict__ NB,
                                                    float2* __restrict__ Vm, long ldV,
                                                    float2* __restrict__ NV) {
  __shared__ double geo[kNearPairs][2][9];             // vertices of the outer and the inner cell
  __shared__ double pts[kNearPairs][2][kQ][3];         // their quadrature points
  __shared__ double pot[kNearPairs][kQ][4];            // S, W of the inner cell at the outer points
  __shared__ double gk[kNearPairs][kQ * kQ][2];        // (exp(ikR) - 1)/R
  __shared__ double blk[kNearPairs][9][2];
  const long t0 = (long)blockIdx.x * kNearPairs;
  const int np = (int)min((long)kNearPairs, npairs - t0), tid = threadIdx.x;
  for (int e = tid; e < np * 18; e += 256) {
    const int u = e / 18, k = e % 18, c = pairs[2 * (t0 + u) + k / 9];
    geo[u][k / 9][k % 9] = vtx[(long)c * 9 + k % 9];
  }
  __syncthreads();
  for (int e = tid; e < np * 2 * kQ * 3; e += 256) {
    const int u = e / (2 * kQ * 3), side = e / (kQ * 3) % 2, q = e / 3 % kQ, d = e % 3;
    const double* P = geo[u][side];
    pts[u][side][q][d] = rule.bary[q][0] * P[d] + rule.bary[q][1] * P[3 + d] + rule.bary[q][2] * P[6 + d];
  }
  __syncthreads();
  for (int e = tid; e < np * kQ; e += 256) {
    const int u = e / kQ, p = e % kQ;
    const Pot v = tri_potentials(reinterpret_cast<const double(*)[3]>(geo[u][1]), pts[u][0][p]);
    pot[u][p][0] = v.S;
    for (int d = 0; d < 3; ++d) pot[u][p][1 + d] = v.W[d];
  }
  // bounded part: (exp(ikR) - 1)/R = (-2 sin^2(kR/2) + i sin(kR))/R, ik at R = 0
  for (int e = (tid + 128) % 256; e < np * kQ * kQ; e += 256) {
    const int u = e / (kQ * kQ), p = e / kQ % kQ, q = e % kQ;
    double rr[3];
    for (int d = 0; d < 3; ++d) rr[d] = pts[u][0][p][d] - pts[u][1][q][d];
    const double R = sqrt(rr[0] * rr[0] + rr[1] * rr[1] + rr[2] * rr[2]);
    double gr, gi;
    if (R > 0.0) {
      const double sh = sin(0.5 * kk * R);
      gr = -2.0 * sh * sh / R;
      gi = sin(kk * R) / R;
    } else {
      gr = 0.0;
      gi = kk;
    }
    gk[u][p * kQ + q][0] = gr;
    gk[u][p * kQ + q][1] = gi;
  }
  __syncthreads();
  // entries 0..8: (i, j) = (e / 3, e % 3) of the block; entry 9: V
  for (int f = tid; f < np * 10; f += 256) {
    const int u = f / 10, e = f % 10, i = e / 3, j = e % 3;
    const int c = pairs[2 * (t0 + u)], cp = pairs[2 * (t0 + u) + 1];
    const double Ain = area[cp];
    const double inv4pi = 0.25 / M_PI;
    double ar = 0.0, ai = 0.0;
    if (e < 9) {
      const double* Po = geo[u][0] + 3 * i;
      const double* Pi = geo[u][1] + 3 * j;
      for (int p = 0; p < kQ; ++p) {
        const double wp = rule.wd[p];
        const double* xo = pts[u][0][p];
        // singular part: int_c' (r' - r_j)/R = W + (x_p - r_j) S
        double arm[3], inner[3];
        for (int d = 0; d < 3; ++d) arm[d] = xo[d] - Po[d];
        for (int d = 0; d < 3; ++d) inner[d] = pot[u][p][1 + d] + (xo[d] - Pi[d]) * pot[u][p][0];
        ar += wp * (arm[0] * inner[0] + arm[1] * inner[1] + arm[2] * inner[2]) / Ain;
        for (int q = 0; q < kQ; ++q) {
          const double ww = wp * rule.wd[q];
          double dot = 0.0;
          for (int d = 0; d < 3; ++d) dot += (xo[d] - Po[d]) * (pts[u][1][q][d] - Pi[d]);
          ar += ww * dot * gk[u][p * kQ + q][0];
          ai += ww * dot * gk[u][p * kQ + q][1];
        }
      }
      const double s = 0.25 * sgn[c * 3 + i] * sgn[cp * 3 + j] * inv4pi;
      blk[u][e][0] = ar * s;
      blk[u][e][1] = ai * s;
    } else {
      for (int p = 0; p < kQ; ++p) {
        const double wp = rule.wd[p];
        ar += wp * pot[u][p][0] / Ain;
        for (int q = 0; q < kQ; ++q) {
          const double ww = wp * rule.wd[q];
          ar += ww * gk[u][p * kQ + q][0];
          ai += ww * gk[u][p * kQ + q][1];
        }
      }
      ar *= inv4pi;
      ai *= inv4pi;
      const float2 v = make_float2((float)ar, (float)ai);
      if (NV) {  // compressed operator: V of the pair, placed by the tile kernel
        NV[t0 + u] = v;
      } else {
        Vm[(long)c * ldV + cp] = v;
        Vm[(long)cp * ldV + c] = v;
      }
    }
  }
  __syncthreads();
  for (int f = tid; f < np * 9; f += 256) {
    const int u = f / 9, e = f % 9, m = 3 * (e % 3) + e / 3;
    double br = blk[u][e][0], bi = blk[u][e][1];
    if (e != m && pairs[2 * (t0 + u)] == pairs[2 * (t0 + u) + 1]) {  // a self block is symmetrised
      br = 0.5 * (br + blk[u][m][0]);
      bi = 0.5 * (bi + blk[u][m][1]);
    }
    NB[(t0 + u) * 9 + e] = make_float2((float)br, (float)bi);
  }
}

// ---------------------------------------------------------------- excitation
// e[r][m] = sum over the two cells of m: sigma/2 sum_q w_q (x_q - r_m).pol exp(ik khat.x_q).
// split = 1: e1 = e - Sigma s, the plane wave less its static part pol
// (whose excitation Sigma s, s_c = -pol . x_c, lies in the range of Sigma):
// exp(i t) - 1 = -2 sin^2(t/2) + i sin t keeps e1's O(k) loop part at any k.
__global__ void k_rhs(int N, int nrhs, const int* __restrict__ edge_cell, const int* __restrict__ edge_slot,
                      const double* __restrict__ vtx, double kk, const double* __restrict__ khat,
                      const double* __restrict__ pol, RuleArgs rule, double2* __restrict__ e, int split = 0) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long)N * nrhs) return;
  const int r = int(t / N), m = int(t % N);
  const double kh[3] = {khat[3 * r], khat[3 * r + 1], khat[3 * r + 2]};
  const double po[3] = {pol[3 * r], pol[3 * r + 1], pol[3 * r + 2]};
  double sr = 0.0, si = 0.0;
  for (int side = 0; side < 2; ++side) {
    const int c = edge_cell[2 * m + side], l = edge_slot[2 * m + side] - 3 * c;
    const double sg = side == 0 ? 0.5 : -0.5;
    const double* P = vtx + (long)c * 9;
    double accr = 0.0, acci = 0.0;
    for (int q = 0; q < kQ; ++q) {
      double x[3];
      for (int d = 0; d < 3; ++d)
        x[d] = rule.bary[q][0] * P[d] + rule.bary[q][1] * P[3 + d] + rule.bary[q][2] * P[6 + d];
      const double proj = (x[0] - P[3 * l]) * po[0] + (x[1] - P[3 * l + 1]) * po[1] + (x[2] - P[3 * l + 2]) * po[2];
      double sn, cs;
      const double ph = kk * (kh[0] * x[0] + kh[1] * x[1] + kh[2] * x[2]);
      sincos(ph, &sn, &cs);
      if (split) {
        const double h = sin(0.5 * ph);
        cs = -2.0 * h * h;
      }
      accr += rule.wd[q] * proj * cs;
      acci += rule.wd[q] * proj * sn;
    }
    sr += sg * accr;
    si += sg * acci;
  }
  e[t] = make_double2(sr, si);
}

// s[r][c] = -pol_r . x_c (x_c the centroid): the static part Sigma s of the
// plane-wave excitation (int f_m . pol = -int div(f_m) pol . r).
__global__ void k_rhs_static(int C, int nrhs, const double* __restrict__ cen, const double* __restrict__ pol,
                             double2* __restrict__ sv) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long)C * nrhs) return;
  const int r = int(t / C), c = int(t % C);
  const double v = pol[3 * r] * cen[3 * c] + pol[3 * r + 1] * cen[3 * c + 1] + pol[3 * r + 2] * cen[3 * c + 2];
  sv[t] = make_double2(-v, 0.0);
}

}  // namespace

RuleArgs rule_args() {
  static const Rule r = make_rule();
  RuleArgs a;
  for (int q = 0; q < kQ; ++q) {
    a.wf[q] = (float)r.w[q];
    a.wd[q] = r.w[q];
    for (int d = 0; d < 3; ++d) a.bary[q][d] = r.bary[q][d];
  }
  return a;
}

// The mesh's edge tiles for the dense assembly.
static rfcmp_status asm_upload(rfcmp_mesh m, int shift, int64_t cap, hipStream_t s) {
  MeshDev& d = m->d;
  AsmTiles at;
  asm_tiles(m->h, shift, cap, at);
  d.asm_hshift = -1;
  auto up = [&](DevBuf& b, const void* src, size_t bytes) -> rfcmp_status {
    RF_TRY(b.alloc(bytes));
    RF_HIP(hipMemcpyAsync(b.p, src, bytes, hipMemcpyHostToDevice, s));
    return RFCMP_OK;
  };
  RF_TRY(up(d.st_ptr, at.ptr.data(), sizeof(int) * at.ptr.size()));
  RF_TRY(up(d.st_cell, at.cell.data(), sizeof(int) * at.cell.size()));
  RF_TRY(up(d.st_span, at.span.data(), sizeof(int) * at.span.size()));
  RF_TRY(up(d.st_pos, at.pos.data(), sizeof(int) * at.pos.size()));
  RF_TRY(up(d.asm_pair, at.pair.data(), sizeof(int) * at.pair.size()));
  RF_TRY(up(d.asm_off, at.off.data(), sizeof(long) * at.off.size()));
  RF_HIP(hipStreamSynchronize(s));  // the host vectors go out of scope
  d.asm_npair = (int64_t)at.off.size();
  d.asm_batch = at.batch;
  d.asm_scratch = at.scratch;
  d.asm_cells_max = at.cmax;
  d.asm_hshift = shift;
  return RFCMP_OK;
}

rfcmp_status mesh_upload(rfcmp_mesh m, hipStream_t s) {
  const MeshHost& h = m->h;
  MeshDev& d = m->d;
  const int64_t C = h.C, N = h.N, V = h.V;
  const Rule rule = make_rule();
  std::vector<double> vtx(9 * C);
  std::vector<float> qoff(4 * kQ * C), fvoff(12 * C), sg(3 * C);
  std::vector<int> slot(2 * N);
  for (int64_t c = 0; c < C; ++c) {
    const double* x = &h.centroid[3 * c];
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < 3; ++k) vtx[9 * c + 3 * i + k] = h.xyz[3 * h.tri[3 * c + i] + k];
    for (int q = 0; q < kQ; ++q)
      for (int k = 0; k < 3; ++k) {
        double p = 0.0;
        for (int i = 0; i < 3; ++i) p += rule.bary[q][i] * vtx[9 * c + 3 * i + k];
        qoff[4 * (kQ * c + q) + k] = (float)(p - x[k]);
      }
    for (int i = 0; i < 3; ++i) {
      for (int k = 0; k < 3; ++k) fvoff[12 * c + 4 * i + k] = (float)(vtx[9 * c + 3 * i + k] - x[k]);
      sg[3 * c + i] = (float)h.cell_sign[3 * c + i];
    }
  }
  for (int64_t n = 0; n < N; ++n) {
    slot[2 * n] = 3 * h.edge_cell[2 * n] + h.edge_local[2 * n];
    slot[2 * n + 1] = 3 * h.edge_cell[2 * n + 1] + h.edge_local[2 * n + 1];
  }
  auto up = [&](DevBuf& b, const void* src, size_t bytes) -> rfcmp_status {
    RF_TRY(b.alloc(bytes));
    RF_HIP(hipMemcpyAsync(b.p, src, bytes, hipMemcpyHostToDevice, s));
    return RFCMP_OK;
  };
  RF_TRY(up(d.cen, h.centroid.data(), sizeof(double) * 3 * C));
  RF_TRY(up(d.vtx, vtx.data(), sizeof(double) * 9 * C));
  RF_TRY(up(d.area, h.area.data(), sizeof(double) * C));
  RF_TRY(up(d.qoff, qoff.data(), sizeof(float) * qoff.size()));
  RF_TRY(up(d.fvoff, fvoff.data(), sizeof(float) * fvoff.size()));
  RF_TRY(up(d.sgn, sg.data(), sizeof(float) * sg.size()));
  RF_TRY(up(d.cell_edge, h.cell_edge.data(), sizeof(int) * 3 * C));
  RF_TRY(up(d.edge_cell, h.edge_cell.data(), sizeof(int) * 2 * N));
  RF_TRY(up(d.edge_slot, slot.data(), sizeof(int) * 2 * N));
  RF_TRY(up(d.edge_vtx, h.edge_vtx.data(), sizeof(int) * 2 * N));
  RF_TRY(up(d.ve_ptr, h.vtx_edge_ptr.data(), sizeof(int) * (V + 1)));
  RF_TRY(up(d.ve_idx, h.vtx_edge_idx.data(), sizeof(int) * 2 * N));
  std::vector<float> vs(h.vtx_edge_sgn.begin(), h.vtx_edge_sgn.end());
  RF_TRY(up(d.ve_sgn, vs.data(), sizeof(float) * 2 * N));
  std::vector<int> home(C);
  for (int64_t c = 0; c < C; ++c) home[c] = int(h.cell_edge[3 * c] / kEdgeTile);
  RF_TRY(up(d.cell_home, home.data(), sizeof(int) * C));
  RF_HIP(hipStreamSynchronize(s));  // host staging vectors die here
  return asm_upload(m, asm_shift(h.N), kAsmScratch, s);
}

// Where the blocks of a batch go: into the operator's slots of the symmetric
// products, which nothing uses yet, where those are large enough (from about
// 16 700 edges on, cells in order), else into `scratch`.  Where there is no
// memory for that, the mesh takes tiles of half the edges, down to 256 (a pair
// of them takes 3.5 MB, for cells in random order 16), in batches that fit the
// slots or 12 MB: the same bits, an operator at level 4 in 1.74 ms instead of
// 1.34.
static rfcmp_status asm_room(rfcmp_op op, DevBuf& scratch, hipStream_t s, float2** B) {
  rfcmp_mesh m = op->mesh;
  MeshDev& d = m->d;
  for (;;) {
    if (d.asm_hshift < 0) RF_TRY(asm_upload(m, asm_shift(m->h.N), kAsmScratch, s));
    if (d.near_host.hshift != d.asm_hshift) {
      RF_HIP(hipStreamSynchronize(s));  // the map may still be on its way to the device
      d.near_host.hshift = -1;
      near_tiles(m->h, d.near_host.pairs, d.asm_hshift, d.near_host.tile_near);
      RF_TRY(d.tile_near.alloc(d.near_host.tile_near.size()));
      RF_HIP(hipMemcpyAsync(d.tile_near.p, d.near_host.tile_near.data(), d.near_host.tile_near.size(),
                            hipMemcpyHostToDevice, s));
      d.near_host.hshift = d.asm_hshift;
    }
    const size_t need = sizeof(float2) * (size_t)d.asm_scratch;
    if (op->symv_scratch.bytes >= need) {
      *B = op->symv_scratch.as<float2>();
      return RFCMP_OK;
    }
    const rfcmp_status st = scratch.bytes >= need ? RFCMP_OK : scratch.alloc(need);
    *B = scratch.as<float2>();
    if (st != RFCMP_E_OOM || d.asm_hshift == kAsmMinShift) return st;
    const int64_t cap = std::max<int64_t>(3 << 19, (int64_t)(op->symv_scratch.bytes / sizeof(float2)));
    RF_TRY(asm_upload(m, d.asm_hshift - 1, cap, s));
  }
}

rfcmp_status assemble_blocks(rfcmp_op op, DevBuf& scratch, hipStream_t s) {
  rfcmp_mesh m = op->mesh;
  const MeshHost& h = m->h;
  MeshDev& d = m->d;
  const int64_t N = h.N;
  const RuleArgs ra = rule_args();
  HmOp* hm = op->hm.get();
  // the near pairs (computed on a host thread from mesh creation on): their
  // blocks first, which the T_A tiles read
  if (d.near_factor != op->opt.near_factor) {
    NearData nd;
    if (m->near_async.valid() && m->near_async_factor == op->opt.near_factor)
      nd = m->near_async.get();
    else
      near_data(h, op->opt.near_factor, nd);
    const int64_t np = (int64_t)nd.pairs.size() / 2;
    d.near_factor = -1.0;  // none cached until every array below is in place
    RF_TRY(d.near.alloc(sizeof(int) * std::max<int64_t>(2 * np, 2)));
    RF_TRY(d.nearB.alloc(sizeof(float2) * 9 * std::max<int64_t>(np, 1)));
    RF_TRY(d.np_ptr.alloc(sizeof(int) * nd.ptr.size()));
    RF_TRY(d.np_other.alloc(sizeof(int) * std::max<size_t>(nd.other.size(), 1)));
    RF_TRY(d.np_code.alloc(sizeof(int) * std::max<size_t>(nd.code.size(), 1)));
    RF_TRY(d.tile_near.alloc(std::max<size_t>(nd.tile_near.size(), 1)));
    d.near_host = std::move(nd);  // the sources stay alive with the mesh
    const NearData& q = d.near_host;
    auto copy = [&](DevBuf& dst, const void* src, size_t bytes) -> rfcmp_status {
      if (bytes) RF_HIP(hipMemcpyAsync(dst.p, src, bytes, hipMemcpyHostToDevice, s));
      return RFCMP_OK;
    };
    RF_TRY(copy(d.near, q.pairs.data(), sizeof(int) * q.pairs.size()));
    RF_TRY(copy(d.np_ptr, q.ptr.data(), sizeof(int) * q.ptr.size()));
    RF_TRY(copy(d.np_other, q.other.data(), sizeof(int) * q.other.size()));
    RF_TRY(copy(d.np_code, q.code.data(), sizeof(int) * q.code.size()));
    RF_TRY(copy(d.tile_near, q.tile_near.data(), q.tile_near.size()));
    d.npairs = np;
    d.near_factor = op->opt.near_factor;
  }
  const long npairs = (long)d.npairs;
  if (hm) RF_TRY(hm->NV.alloc(sizeof(float2) * std::max<long>(npairs, 1)));
  if (npairs > 0) {
    ProfScope prof("near_pairs", s);
    hipLaunchKernelGGL(k_near_pairs, dim3((unsigned)((npairs + kNearPairs - 1) / kNearPairs)), dim3(256), 0, s,
                       npairs,
                       d.near.as<int>(), d.vtx.as<double>(), d.area.as<double>(), d.sgn.as<float>(), op->k, ra,
                       d.nearB.as<float2>(), hm ? nullptr : op->Vb.as<float2>(), (long)op->ldV,
                       hm ? hm->NV.as<float2>() : nullptr);
    RF_HIP(hipGetLastError());
  }
  if (hm) {
    // compressed: the dense blocks (pairs of tiles of the permuted order),
    // then ACA of the low-rank blocks
    const HmMesh& H = *m->hm;
    const int64_t nd = (int64_t)H.t.dense_I.size();
    RF_TRY(hm->TAd.alloc(sizeof(float2) * kEdgeTile * kEdgeTile * std::max<int64_t>(nd, 1)));
    RF_TRY(hm->Vd.alloc(sizeof(float2) * std::max<int64_t>(H.vd_total, 1)));
    RF_HIP(hipMemsetAsync(hm->Vd.p, 0, hm->Vd.bytes, s));
    if (nd > 0) {
      ProfScope prof("hm_dense", s);
      const size_t lds = 2 * sizeof(float2) * kEdgeTile * kEdgeTile + 2 * sizeof(CellL) * (size_t)H.t.et_cells_max;
      hipLaunchKernelGGL(k_assemble_list, dim3((unsigned)nd), dim3(kAsmThreads),
                         lds, s, H.et_ptr.as<int>(), H.et_cell.as<int>(), H.et_rows.as<int>(),
                         H.home.as<int>(), d.cen.as<double>(), d.qoff.as<float4>(), d.fvoff.as<float4>(),
                         d.sgn.as<float>(), (float)op->k, ra, d.np_ptr.as<int>(),
                         d.np_other.as<int>(), d.np_code.as<int>(), d.nearB.as<float2>(), hm->TAd.as<float2>(),
                         hm->Vd.as<float2>(), H.dense_ij.as<int2>(), H.vd_off.as<long>(),
                         H.cell_start.as<int>(), H.iperm_c.as<int>(), hm->NV.as<float2>());
      RF_HIP(hipGetLastError());
    }
    hm->dense_entries[0] = nd * kEdgeTile * kEdgeTile;
    hm->dense_entries[1] = H.vd_total;
    return hm_aca(op, s);
  }
  float2* B = nullptr;
  RF_TRY(asm_room(op, scratch, s, &B));
  ProfScope prof("assemble_ta", s);
  PairArgs g;
  g.st_ptr = d.st_ptr.as<int>();
  g.st_cell = d.st_cell.as<int>();
  g.cell_home = d.cell_home.as<int>();
  g.pair = d.asm_pair.as<int4>();
  g.off = d.asm_off.as<long>();
  g.near = d.tile_near.as<uint8_t>();
  g.np_ptr = d.np_ptr.as<int>();
  g.np_other = d.np_other.as<int>();
  g.np_code = d.np_code.as<int>();
  g.NB = d.nearB.as<float2>();
  g.cen = d.cen.as<double>();
  g.qoff = d.qoff.as<float4>();
  g.fvoff = d.fvoff.as<float4>();
  g.sgn = d.sgn.as<float>();
  g.rule = ra;
  g.kk = (float)op->k;
  g.st_span = d.st_span.as<int>();
  g.st_pos = d.st_pos.as<int2>();
  g.N = (int)N;
  g.hshift = d.asm_hshift;
  const unsigned cmax = (unsigned)d.asm_cells_max, ncol = (cmax + 63) / 64;
  for (size_t q = 0; q + 1 < d.asm_batch.size(); ++q) {
    const unsigned np = (unsigned)(d.asm_batch[q + 1] - d.asm_batch[q]);
    g.p0 = (int)d.asm_batch[q];
    // first cells per wave: 2 once that leaves the launch 8192 waves (a wave's
    // work is the launch's tail: level 5 17.4 ms with 2, 18.1 with 4)
    g.rows = (long)ncol * cmax * np >= 16384 ? 2 : 1;
    hipLaunchKernelGGL(k_cell_pairs, dim3(ncol, (cmax + 4 * g.rows - 1) / (4 * g.rows), np), dim3(256), 0, s, g,
                       B, op->Vb.as<float2>(), (long)op->ldV);
    hipLaunchKernelGGL(k_gather_ta, dim3(1u << (2 * g.hshift), np), dim3(256), 0, s, g, B,
                       op->TA.as<float2>(), (long)op->ldA);
  }
  RF_HIP(hipGetLastError());
  return RFCMP_OK;
}

// Edge tiles of the dense assembly: 2048 edges above 6144, 1024 and 512 below,
// where a larger tile leaves too few pairs of tiles (level 5: 17.4 ms at 2048,
// 18.1 at 1024, 19.8 at 512; level 2: 0.027 ms at 512, 0.040 at 2048).
int asm_shift(int64_t N) { return N > 6144 ? 5 : N > 1536 ? 4 : 3; }

void asm_tiles(const MeshHost& h, int shift, int64_t cap, AsmTiles& out) {
  const int64_t N = h.N, E = (int64_t)kEdgeTile << shift, nt = (N + E - 1) / E;
  out.ptr.assign(nt + 1, 0);
  out.pos.resize(2 * N);
  std::vector<int> cells;
  std::vector<int> local(h.C, 0);
  for (int64_t t = 0; t < nt; ++t) {
    const int64_t e0 = t * E, e1 = std::min<int64_t>(N, e0 + E);
    cells.assign(h.edge_cell.begin() + 2 * e0, h.edge_cell.begin() + 2 * e1);
    std::sort(cells.begin(), cells.end());
    cells.erase(std::unique(cells.begin(), cells.end()), cells.end());
    for (size_t i = 0; i < cells.size(); ++i) local[cells[i]] = (int)i;
    for (int64_t e = e0; e < e1; ++e)
      for (int k = 0; k < 2; ++k) out.pos[2 * e + k] = 3 * local[h.edge_cell[2 * e + k]] + h.edge_local[2 * e + k];
    out.cell.insert(out.cell.end(), cells.begin(), cells.end());
    for (int c : cells) {
      int lo = INT_MAX, hi = 0;
      for (int i = 0; i < 3; ++i) {
        const int64_t e = h.cell_edge[3 * c + i];
        if (e < e0 || e >= e1) continue;
        lo = std::min(lo, (int)((e - e0) / kEdgeTile));
        hi = std::max(hi, (int)((e - e0) / kEdgeTile));
      }
      out.span.push_back(lo | hi << 16);
    }
    out.ptr[t + 1] = (int)out.cell.size();
    out.cmax = std::max(out.cmax, (int)cells.size());
  }
  // tile pairs s <= t in batches whose blocks fit the scratch
  int64_t used = 0;
  out.batch.assign(1, 0);
  for (int64_t t = 0; t < nt; ++t)
    for (int64_t s = 0; s <= t; ++s) {
      const int64_t need = 9 * (int64_t)(out.ptr[s + 1] - out.ptr[s]) * (out.ptr[t + 1] - out.ptr[t]);
      const int64_t p = (int64_t)out.off.size();
      if (used > 0 && (used + need > cap || p - out.batch.back() >= kAsmBatch)) {
        out.batch.push_back(p);
        used = 0;
      }
      const int q[4] = {(int)s, (int)t, 0, 0};
      out.pair.insert(out.pair.end(), q, q + 4);
      out.off.push_back((long)used);
      used += need;
      out.scratch = std::max(out.scratch, used);
    }
  if (!out.off.empty()) out.batch.push_back((int64_t)out.off.size());
}

static size_t near_tile_count(const MeshHost& h, int shift) {
  const int64_t E = (int64_t)kEdgeTile << shift, nt = (h.N + E - 1) / E;
  return (size_t)(nt * (nt + 1) / 2);
}
// Marks the pairs of edge tiles (s <= t, index t (t + 1)/2 + s) that the near
// pairs p0 .. p1 - 1 of the list touch.
static void mark_near_tiles(const MeshHost& h, const int32_t* pr, int64_t p0, int64_t p1, int shift,
                            std::vector<uint8_t>& map) {
  const int64_t E = (int64_t)kEdgeTile << shift;
  for (int64_t p = p0; p < p1; ++p) {
    int64_t ta[3], tb[3];
    for (int i = 0; i < 3; ++i) {
      ta[i] = h.cell_edge[3 * pr[2 * p] + i] / E;
      tb[i] = h.cell_edge[3 * pr[2 * p + 1] + i] / E;
    }
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j) {
        const int64_t I = std::min(ta[i], tb[j]), J = std::max(ta[i], tb[j]);
        map[(size_t)(J * (J + 1) / 2 + I)] = 1;
      }
  }
}
void near_tiles(const MeshHost& h, const std::vector<int32_t>& pairs, int shift, std::vector<uint8_t>& out) {
  out.assign(near_tile_count(h, shift), 0);
  mark_near_tiles(h, pairs.data(), 0, (int64_t)pairs.size() / 2, shift, out);
}

void near_data(const MeshHost& h, double factor, NearData& out) {
  near_pairs(h, factor, out.pairs);
  const int64_t np = (int64_t)out.pairs.size() / 2, C = h.C;
  const int32_t* pr = out.pairs.data();
  out.hshift = asm_shift(h.N);
  const size_t ntp = near_tile_count(h, out.hshift);
  // Contiguous chunks of the pair list on a few threads.  Pass 1 counts each
  // chunk's occurrences of every cell; pass 2 places them, chunk by chunk in
  // list order (the offsets of a chunk follow the earlier chunks' counts), so
  // the result is the one of a single thread, and marks the chunk's tile
  // pairs in a map of its own (or-ed together afterwards).
  const int nthr = np >= 65536 ? (int)std::min<int64_t>(8, std::max(1u, std::thread::hardware_concurrency())) : 1;
  std::vector<std::vector<int32_t>> cnt(nthr, std::vector<int32_t>(C, 0));
  std::vector<std::vector<uint8_t>> tmap(nthr);
  auto chunk = [&](int t, int64_t& p0, int64_t& p1) {
    p0 = np * t / nthr;
    p1 = np * (t + 1) / nthr;
  };
  auto count = [&](int t) {
    int64_t p0, p1;
    chunk(t, p0, p1);
    std::vector<int32_t>& c = cnt[t];
    for (int64_t p = p0; p < p1; ++p) {
      ++c[pr[2 * p]];
      if (pr[2 * p] != pr[2 * p + 1]) ++c[pr[2 * p + 1]];
    }
  };
  auto place = [&](int t) {
    int64_t p0, p1;
    chunk(t, p0, p1);
    std::vector<int32_t>& fill = cnt[t];  // the chunk's offsets by now
    for (int64_t p = p0; p < p1; ++p) {
      const int32_t a = pr[2 * p], b = pr[2 * p + 1];
      out.other[fill[a]] = b;
      out.code[fill[a]++] = int32_t(2 * p);
      if (a != b) {
        out.other[fill[b]] = a;
        out.code[fill[b]++] = int32_t(2 * p + 1);
      }
    }
    std::vector<uint8_t>& m = tmap[t];
    m.assign(ntp, 0);
    mark_near_tiles(h, pr, p0, p1, out.hshift, m);
  };
  auto run = [&](auto&& fn) {
    std::vector<std::thread> pool;
    try {
      for (int t = 1; t < nthr; ++t) pool.emplace_back(fn, t);
    } catch (const std::system_error&) {
      for (int t = (int)pool.size() + 1; t < nthr; ++t) fn(t);  // no threads to be had: here
    }
    fn(0);
    for (auto& th : pool) th.join();
  };
  run(count);
  // the near partners of every cell, ascending, with 2 p + t.  The list runs
  // in order of its first cell, partners ascending, so placing in list order
  // puts cell c's partners a < c (from the pairs (a, c), in order of a)
  // before its own pairs (c, b), b >= c ascending: already sorted.
  out.ptr.assign(C + 1, 0);
  for (int64_t c = 0; c < C; ++c) {
    int32_t o = out.ptr[c];
    for (int t = 0; t < nthr; ++t) {
      const int32_t k = cnt[t][c];
      cnt[t][c] = o;
      o += k;
    }
    out.ptr[c + 1] = o;
  }
  out.other.resize(out.ptr[C]);
  out.code.resize(out.ptr[C]);
  run(place);
  // edge-tile pairs (I <= J) that hold a near cell pair
  out.tile_near.assign(ntp, 0);
  for (int t = 0; t < nthr; ++t)
    for (size_t q = 0; q < ntp; ++q) out.tile_near[q] |= tmap[t][q];
}

namespace {
// Voltage-gap excitation: element t = r N + m of e takes the summed gap
// voltage of flat index t from the sorted, duplicate-free list idx/val, found
// by binary search, else 0.
__global__ void k_rhs_gap(long total, const long* __restrict__ idx, const double2* __restrict__ val, int P,
                          double2* __restrict__ e) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= total) return;
  int lo = 0, hi = P;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (idx[mid] < t) lo = mid + 1;
    else hi = mid;
  }
  e[t] = (lo < P && idx[lo] == t) ? val[lo] : make_double2(0.0, 0.0);
}
}  // namespace

rfcmp_status rhs_planewave(rfcmp_op op, const double* khat, const double* pol, int nrhs, double2* e,
                           hipStream_t s, double2* sv) {
  rfcmp_mesh m = op->mesh;
  const int64_t N = m->h.N, C = m->h.C;
  DevBuf dk;
  RF_TRY(dk.alloc(sizeof(double) * 6 * nrhs));
  RF_HIP(hipMemcpyAsync(dk.p, khat, sizeof(double) * 3 * nrhs, hipMemcpyHostToDevice, s));
  RF_HIP(hipMemcpyAsync(dk.as<double>() + 3 * nrhs, pol, sizeof(double) * 3 * nrhs, hipMemcpyHostToDevice, s));
  const long total = (long)N * nrhs;
  hipLaunchKernelGGL(k_rhs, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, (int)N, nrhs,
                     m->d.edge_cell.as<int>(), m->d.edge_slot.as<int>(), m->d.vtx.as<double>(), op->k, dk.as<double>(),
                     dk.as<double>() + 3 * nrhs, rule_args(), e, sv ? 1 : 0);
  RF_HIP(hipGetLastError());
  if (sv) {
    const long tc = (long)C * nrhs;
    hipLaunchKernelGGL(k_rhs_static, dim3((unsigned)((tc + 255) / 256)), dim3(256), 0, s, (int)C, nrhs,
                       m->d.cen.as<double>(), dk.as<double>() + 3 * nrhs, sv);
    RF_HIP(hipGetLastError());
  }
  RF_HIP(hipStreamSynchronize(s));
  return RFCMP_OK;
}

// Staging of rfcmp_rhs_planewave_noalloc: the directions and polarisations of
// at most RFCMP_RHS_NOALLOC_MAX plane waves (khat [nrhs][3], then pol
// [nrhs][3]), in a fixed array of each device instead of a buffer allocated
// per call.  Host code never uses the array's name as an address: its device
// address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) double rhs_stage[6 * RFCMP_RHS_NOALLOC_MAX];

namespace {
constexpr int kMaxDevices = 64;

rfcmp_status rhs_stage_address(double** out) {
  static std::mutex mu;
  static double* addr[kMaxDevices] = {};
  int dev = 0;
  RF_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) {
    set_error("device %d beyond the %d devices the staging array is set up for", dev, kMaxDevices);
    return RFCMP_E_STATE;
  }
  std::lock_guard<std::mutex> g(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    RF_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(rhs_stage)));
    addr[dev] = static_cast<double*>(p);
  }
  *out = addr[dev];
  return RFCMP_OK;
}
}  // namespace

rfcmp_status rhs_planewave_noalloc(rfcmp_op op, const double* khat, const double* pol, int nrhs, double2* e,
                                   hipStream_t s) {
  if (nrhs > RFCMP_RHS_NOALLOC_MAX) {
    set_error("rfcmp_rhs_planewave_noalloc: %d plane waves, at most %d", nrhs, RFCMP_RHS_NOALLOC_MAX);
    return RFCMP_E_ARG;
  }
  rfcmp_mesh m = op->mesh;
  const int64_t N = m->h.N;
  double* stage = nullptr;
  RF_TRY(rhs_stage_address(&stage));
  RF_HIP(hipMemcpyAsync(stage, khat, sizeof(double) * 3 * nrhs, hipMemcpyHostToDevice, s));
  RF_HIP(hipMemcpyAsync(stage + 3 * nrhs, pol, sizeof(double) * 3 * nrhs, hipMemcpyHostToDevice, s));
  const long total = (long)N * nrhs;
  hipLaunchKernelGGL(k_rhs, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, (int)N, nrhs,
                     m->d.edge_cell.as<int>(), m->d.edge_slot.as<int>(), m->d.vtx.as<double>(), op->k, stage,
                     stage + 3 * nrhs, rule_args(), e);
  RF_HIP(hipGetLastError());
  // the next call on this device overwrites the stage
  RF_HIP(hipStreamSynchronize(s));
  return RFCMP_OK;
}

rfcmp_status rhs_gap(rfcmp_mesh m, const int32_t* edges, const double2* volts, int ngap, int nrhs, double2* e,
                     hipStream_t s) {
  const int64_t N = m->h.N;
  // Flat indices r N + m in order, gaps on one edge summed in the order given.
  std::vector<std::pair<long, double2>> g;
  g.reserve((size_t)ngap * nrhs);
  for (int r = 0; r < nrhs; ++r)
    for (int q = 0; q < ngap; ++q) g.push_back({(long)r * N + edges[(long)r * ngap + q], volts[(long)r * ngap + q]});
  std::stable_sort(g.begin(), g.end(), [](const auto& a, const auto& b) { return a.first < b.first; });
  std::vector<long> idx;
  std::vector<double2> val;
  for (const auto& x : g) {
    if (!idx.empty() && idx.back() == x.first) {
      val.back().x += x.second.x;
      val.back().y += x.second.y;
    } else {
      idx.push_back(x.first);
      val.push_back(x.second);
    }
  }
  const int P = (int)idx.size();
  DevBuf di, dv;
  if (P) {
    RF_TRY(di.alloc(sizeof(long) * P));
    RF_TRY(dv.alloc(sizeof(double2) * P));
    RF_HIP(hipMemcpyAsync(di.p, idx.data(), sizeof(long) * P, hipMemcpyHostToDevice, s));
    RF_HIP(hipMemcpyAsync(dv.p, val.data(), sizeof(double2) * P, hipMemcpyHostToDevice, s));
  }
  const long total = (long)N * nrhs;
  hipLaunchKernelGGL(k_rhs_gap, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, total,
                     P ? di.as<long>() : nullptr, P ? dv.as<double2>() : nullptr, P, e);
  RF_HIP(hipGetLastError());
  RF_HIP(hipStreamSynchronize(s));
  return RFCMP_OK;
}

}  // namespace rfcmp
