// Compressed EFIE blocks on the device (see hmat.h): the tree's upload,
// adaptive cross approximation of the low-rank blocks, the compressed product
// and the dense write-out.
//
// ACA (one workgroup per block, partial pivoting): the residual of pivot row
// i is formed from the block's entries less the terms so far, its largest
// entry (first on ties) is the column pivot j, v = row / row[j], the residual
// column j is u, and the next pivot row is the largest entry of u among the
// rows not yet taken.  The Frobenius norm of the approximation S_k is updated
// exactly, |S_k|^2 = |S_k-1|^2 + 2 Re sum_l<k (u_l^H u_k)(v_l^H v_k) +
// |u_k|^2 |v_k|^2, and the iteration stops when |u_k| |v_k| <= tol |S_k|.
// Entries are formed on the fly in FP32 by the far-pair rule (an admissible
// block holds no near cell pair): a T_A entry sums the four cell pairs of its
// two edges, (B++ + B--) + (B+- + B-+), a V entry is I_0 of its cell pair.
// Factors are complex64; each thread owns the rows (columns) i = tid mod 256
// of its block's factors, so the only values it reads from other threads are
// the pivots, staged in LDS after a barrier.
//
// Product y = M x (M = T_A or V, x [nr][n] complex128, FP64 accumulation on the
// FP64 matrix cores, 8 right-hand sides at a time): the input in the permuted
// order; per low-rank block z = V^T x_cols and w = U^T x_rows (k_hm_proj); per
// tile of output rows the sum, in a fixed order, of its dense blocks (and the
// transposes of those it is the column of), U z of the low-rank blocks it is a
// row of and V w of those it is a column of (k_hm_tile), written back in the
// mesh's numbering.
#include <algorithm>
#include <climits>
#include <cmath>
#include <numeric>

#include "farpair.h"
#include "hmat.h"
#include "internal.h"

rfcmp_mesh_s::rfcmp_mesh_s() = default;
rfcmp_mesh_s::~rfcmp_mesh_s() = default;

namespace rfcmp {
namespace {

constexpr int kAcaThreads = 256;
constexpr int kAcaWaves = kAcaThreads / 64;

struct AcaArgs {
  const int* perm;        // position -> edge (T_A) or cell (V)
  const int* edge_slot;   // [N][2]: 3 c + local index of each edge in c+ and c-
  const double* cen;
  const float4* qoff;
  const float4* fvoff;
  const float* sgn;
  RuleArgs rule;
  float kk;
  float tol;
  int kmax;
  const HmLr* blk;
  const long* uoff;       // pool offsets (complex64 entries) of U and V
  const long* voff;
  const long* toff;       // offsets of the taken-row flags
  float2* pool;
  unsigned char* taken;
  int* rank;
  int* flag;              // 1: stopped at kmax above the tolerance
};

__device__ float2 ta_entry(const AcaArgs& a, int m, int n) {
  float2 b00, b01, b10, b11;
#pragma unroll 1
  for (int pq = 0; pq < 4; ++pq) {
    const int p = pq >> 1, q = pq & 1;
    const int sa = a.edge_slot[2 * m + p], sb = a.edge_slot[2 * n + q];
    const int ca = sa / 3, la = sa - 3 * ca, cb = sb / 3, lb = sb - 3 * cb;
    Moments M;
    far_moments(a.qoff + (long)ca * kQ, a.qoff + (long)cb * kQ, (float)(a.cen[3 * ca] - a.cen[3 * cb]),
                    (float)(a.cen[3 * ca + 1] - a.cen[3 * cb + 1]), (float)(a.cen[3 * ca + 2] - a.cen[3 * cb + 2]),
                    a.rule, a.kk, M);
    const float2 v = b_entry(M, a.fvoff[3 * ca + la], a.fvoff[3 * cb + lb], a.sgn[3 * ca + la], a.sgn[3 * cb + lb]);
    if (pq == 0)
      b00 = v;
    else if (pq == 1)
      b01 = v;
    else if (pq == 2)
      b10 = v;
    else
      b11 = v;
  }
  return make_float2((b00.x + b11.x) + (b01.x + b10.x), (b00.y + b11.y) + (b01.y + b10.y));
}

__device__ float2 v_entry(const AcaArgs& a, int c, int cp) {
  return far_i0(a.qoff + (long)c * kQ, a.qoff + (long)cp * kQ, (float)(a.cen[3 * c] - a.cen[3 * cp]),
                    (float)(a.cen[3 * c + 1] - a.cen[3 * cp + 1]), (float)(a.cen[3 * c + 2] - a.cen[3 * cp + 2]),
                    a.rule, a.kk);
}

struct AcaLds {
  float v[kAcaWaves];
  int i[kAcaWaves];
  double d[kAcaWaves][2];
  float c[kAcaWaves][32];
};

// Largest value, smallest index on ties, over the workgroup; every thread
// receives it.
__device__ inline void block_argmax(float& v, int& idx, AcaLds& L) {
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(v, o);
    const int oi = __shfl_xor(idx, o);
    if (ov > v || (ov == v && oi < idx)) {
      v = ov;
      idx = oi;
    }
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    L.v[w] = v;
    L.i[w] = idx;
  }
  __syncthreads();
  v = L.v[0];
  idx = L.i[0];
  for (int q = 1; q < kAcaWaves; ++q)
    if (L.v[q] > v || (L.v[q] == v && L.i[q] < idx)) {
      v = L.v[q];
      idx = L.i[q];
    }
  __syncthreads();
}

// Sums of two doubles over the workgroup in a fixed order (lane 0 of each
// wave, then the waves in order).
__device__ inline void block_sum2(double& x, double& y, AcaLds& L) {
  for (int o = 32; o > 0; o >>= 1) {
    x += __shfl_xor(x, o);
    y += __shfl_xor(y, o);
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    L.d[w][0] = x;
    L.d[w][1] = y;
  }
  __syncthreads();
  x = L.d[0][0];
  y = L.d[0][1];
  for (int q = 1; q < kAcaWaves; ++q) {
    x += L.d[q][0];
    y += L.d[q][1];
  }
  __syncthreads();
}

__device__ inline void block_sum32(float (&v)[32], AcaLds& L) {
#pragma unroll
  for (int q = 0; q < 32; ++q)
    for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_xor(v[q], o);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int q = 0; q < 32; ++q) L.c[w][q] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 32; ++q) {
    float s = L.c[0][q];
    for (int u = 1; u < kAcaWaves; ++u) s += L.c[u][q];
    v[q] = s;
  }
  __syncthreads();
}

template <int KIND>
__global__ __launch_bounds__(kAcaThreads) void k_aca(const AcaArgs a, int b0) {
  const int b = b0 + blockIdx.x;
  const HmLr B = a.blk[b];
  const int m = B.m, n = B.n;
  float2* U = a.pool + a.uoff[b];
  float2* V = a.pool + a.voff[b];
  unsigned char* taken = a.taken + a.toff[b];
  const int kcap = min(a.kmax, min(m, n));
  const int tid = threadIdx.x;
  __shared__ float2 sU[kHmKmax], sV[kHmKmax + 1];
  __shared__ AcaLds L;
  for (int i = tid; i < m; i += kAcaThreads) taken[i] = 0;
  __syncthreads();
  auto entry = [&](int pi, int pj) -> float2 {
    const int x = a.perm[B.r0 + pi], y = a.perm[B.c0 + pj];
    return KIND == 0 ? ta_entry(a, x, y) : v_entry(a, x, y);
  };
  double S2 = 0.0;
  int k = 0, i = 0, tries = 0;
  bool conv = false;
  while (k < kcap) {
    for (int l = tid; l < k; l += kAcaThreads) sU[l] = U[(long)l * m + i];
    __syncthreads();
    // residual of row i into V[k]
    float2* Vk = V + (long)k * n;
    float best = -1.f;
    int bj = INT_MAX;
    for (int j = tid; j < n; j += kAcaThreads) {
      float2 e = entry(i, j);
      for (int l = 0; l < k; ++l) {
        const float2 v = V[(long)l * n + j], u = sU[l];
        e.x -= u.x * v.x - u.y * v.y;
        e.y -= u.x * v.y + u.y * v.x;
      }
      Vk[j] = e;
      const float mg = e.x * e.x + e.y * e.y;
      if (mg > best) {
        best = mg;
        bj = j;
      }
    }
    block_argmax(best, bj, L);
    if (tid == 0) taken[i] = 1;
    __syncthreads();
    if (!(best > 0.f)) {
      // row i is represented already: the first row not yet taken
      int cand = INT_MAX;
      for (int ii = tid; ii < m; ii += kAcaThreads)
        if (!taken[ii]) {
          cand = ii;
          break;
        }
      float cv = cand < INT_MAX ? 0.f : -1.f;
      block_argmax(cv, cand, L);
      if (cand == INT_MAX || ++tries > m) break;
      i = cand;
      continue;
    }
    const float2 piv = Vk[bj];
    __syncthreads();  // every thread has the pivot before its owner scales it
    const float dd = piv.x * piv.x + piv.y * piv.y;
    const float2 inv = make_float2(piv.x / dd, -piv.y / dd);
    double nv = 0.0, nu = 0.0;
    for (int j = tid; j < n; j += kAcaThreads) {
      const float2 e = Vk[j];
      const float2 v = make_float2(e.x * inv.x - e.y * inv.y, e.x * inv.y + e.y * inv.x);
      Vk[j] = v;
      nv += (double)v.x * v.x + (double)v.y * v.y;
    }
    __syncthreads();
    for (int l = tid; l <= k; l += kAcaThreads) sV[l] = V[(long)l * n + bj];
    __syncthreads();
    // residual of column bj into U[k]
    float2* Uk = U + (long)k * m;
    float bu = -1.f;
    int bi = INT_MAX;
    for (int ii = tid; ii < m; ii += kAcaThreads) {
      float2 e = entry(ii, bj);
      for (int l = 0; l < k; ++l) {
        const float2 u = U[(long)l * m + ii], v = sV[l];
        e.x -= u.x * v.x - u.y * v.y;
        e.y -= u.x * v.y + u.y * v.x;
      }
      Uk[ii] = e;
      nu += (double)e.x * e.x + (double)e.y * e.y;
      if (!taken[ii]) {
        const float mg = e.x * e.x + e.y * e.y;
        if (mg > bu) {
          bu = mg;
          bi = ii;
        }
      }
    }
    // cross terms with the earlier terms, eight at a time
    double cr = 0.0;
    for (int l0 = 0; l0 < k; l0 += 8) {
      float pp[32];
#pragma unroll
      for (int q = 0; q < 32; ++q) pp[q] = 0.f;
      for (int ii = tid; ii < m; ii += kAcaThreads) {
        const float2 u = Uk[ii];
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (l0 + q < k) {
            const float2 w = U[(long)(l0 + q) * m + ii];
            pp[2 * q] += w.x * u.x + w.y * u.y;
            pp[2 * q + 1] += w.x * u.y - w.y * u.x;
          }
      }
      for (int j = tid; j < n; j += kAcaThreads) {
        const float2 v = Vk[j];
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (l0 + q < k) {
            const float2 w = V[(long)(l0 + q) * n + j];
            pp[16 + 2 * q] += w.x * v.x + w.y * v.y;
            pp[16 + 2 * q + 1] += w.x * v.y - w.y * v.x;
          }
      }
      block_sum32(pp, L);
#pragma unroll
      for (int q = 0; q < 8; ++q)
        cr += (double)pp[2 * q] * pp[16 + 2 * q] - (double)pp[2 * q + 1] * pp[16 + 2 * q + 1];
    }
    block_sum2(nu, nv, L);
    S2 += 2.0 * cr + nu * nv;
    ++k;
    if (nu * nv <= (double)a.tol * (double)a.tol * S2) {
      conv = true;
      break;
    }
    block_argmax(bu, bi, L);
    if (bi == INT_MAX) {  // every row taken: the block is exact
      conv = true;
      break;
    }
    i = bi;
  }
  if (k >= min(m, n)) conv = true;
  if (tid == 0) {
    a.rank[b] = k;
    a.flag[b] = conv ? 0 : 1;
  }
}

// The first rank[b] columns of each block's factors, from the pool to their
// own storage.
__global__ __launch_bounds__(256) void k_aca_compact(int b0, const HmLr* blk, const int* rank, const long* uoff,
                                                     const long* voff, const float2* pool, float2* const* ud,
                                                     float2* const* vd) {
  const int b = b0 + blockIdx.x;
  const long k = rank[b];
  const long nu = k * blk[b].m, nv = k * blk[b].n;
  const float2* su = pool + uoff[b];
  const float2* sv = pool + voff[b];
  float2* du = ud[b];
  float2* dv = vd[b];
  for (long e = threadIdx.x; e < nu; e += 256) du[e] = su[e];
  for (long e = threadIdx.x; e < nv; e += 256) dv[e] = sv[e];
}

// The product's vectors in the permuted order hold kHmR = 8 right-hand sides
// per position, real and imaginary parts apart: 16 doubles, the columns of one
// FP64 matrix-core operand (v_mfma_f64_16x16x4; right-hand sides beyond the
// call's are zero).  A complex matrix times such a block takes two products,
// P = Re(M) X and Q = Im(M) X, combined once at the end: Re Y = P_re - Q_im,
// Im Y = P_im + Q_re, with Q negated for conj(M).
typedef double dbl4 __attribute__((ext_vector_type(4)));
constexpr int kHmCols = 2 * kHmR;
static_assert(kHmCols == 16, "one operand of 16 columns");

// Operand entries: rows i = lane % 16, columns (and X rows) lane / 16 of each
// step of four.
struct HmAcc {
  dbl4 p = dbl4{0.0, 0.0, 0.0, 0.0}, q = dbl4{0.0, 0.0, 0.0, 0.0};
  __device__ inline void add(float2 m, double x) {
    p = __builtin_amdgcn_mfma_f64_16x16x4f64((double)m.x, x, p, 0, 0, 0);
    q = __builtin_amdgcn_mfma_f64_16x16x4f64((double)m.y, x, q, 0, 0, 0);
  }
};
// Four neighbouring entries (8-byte aligned) in two loads.
__device__ inline void hm_load4(const float2* p, float2 (&m)[4]) {
  typedef float vf4 __attribute__((ext_vector_type(4), aligned(8)));
  const vf4 a = *reinterpret_cast<const vf4*>(p), b = *reinterpret_cast<const vf4*>(p + 2);
  m[0] = make_float2(a.x, a.y);
  m[1] = make_float2(a.z, a.w);
  m[2] = make_float2(b.x, b.y);
  m[3] = make_float2(b.z, b.w);
}
// Value v of lane l: row 4 v + l / 16, column l % 16; the real (even) and
// imaginary (odd) columns exchange their Q.
__device__ inline double hm_combine(double p, double q, int lane, double sgn) {
  const double other = __shfl_xor(q, 1);
  return (lane & 1) ? p + sgn * other : p - sgn * other;
}

// xp[p][r] = x[r][perm[p]]
__global__ void k_hm_gather(int n, int nr, const int* __restrict__ perm, const double2* __restrict__ x,
                            double2* __restrict__ xp) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long)n * kHmR) return;
  const int r = (int)(e % kHmR), p = (int)(e / kHmR);
  xp[e] = r < nr ? x[(long)r * n + perm[p]] : make_double2(0.0, 0.0);
}

// z = V^T x_cols (part 0) and w = U^T x_rows (part 1) of every low-rank block
// (conj: of the conjugated factors): 16 factor columns at a time are the
// operand's rows, four waves take every fourth chunk of 16 positions, a lane
// four neighbouring ones, and their sums are added in order.  Bound: memory,
// the factors once and 128 bytes of input per position and block (level 6, tol
// 1e-4: T_A 0.55 ms, V 0.24, where sums of FP64 FMAs over staged chunks took 1.5
// and 0.7).  Nontemporal loads of the factors were slower (0.59 against 0.46 on
// the mean of both).
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
void k_hm_proj(const HmLr* __restrict__ blk, const int* __restrict__ rank,
                                                 float2* const* __restrict__ Up, float2* const* __restrict__ Vp,
                                                 const long* __restrict__ zoff, const double* __restrict__ xp,
                                                 double sgn, double* __restrict__ zw) {
  __shared__ double red[3][8][64];
  const int b = blockIdx.x, part = blockIdx.y;
  const int k = rank[b];
  const HmLr B = blk[b];
  const float2* M = part == 0 ? Vp[b] : Up[b];
  const int len = part == 0 ? B.n : B.m, off = part == 0 ? B.c0 : B.r0;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4, col = lane & 15;
  double* out = zw + (zoff[b] + (long)part * k * kHmR) * 2;
  for (int l0 = 0; l0 < k; l0 += 16) {
    const float2* row = M + (long)min(l0 + col, k - 1) * len;
    HmAcc acc;
    int j0 = 16 * w;
#pragma unroll 4
    for (; j0 + 16 <= len; j0 += 64) {
      const int j = j0 + 4 * g;
      float2 m[4];
      double x[4];
      hm_load4(row + j, m);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = xp[(long)(off + j + e) * kHmCols + col];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc.add(m[e], x[e]);
    }
    if (j0 < len) {  // the last, short chunk
      const int j = j0 + 4 * g;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int je = min(j + e, len - 1);
        float2 m = row[je];
        if (j + e >= len) m = make_float2(0.f, 0.f);
        acc.add(m, xp[(long)(off + je) * kHmCols + col]);
      }
    }
    if (w > 0)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        red[w - 1][v][lane] = acc.p[v];
        red[w - 1][4 + v][lane] = acc.q[v];
      }
    __syncthreads();
    if (w == 0)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double p = acc.p[v], q = acc.q[v];
        for (int u = 0; u < 3; ++u) {
          p += red[u][v][lane];
          q += red[u][4 + v][lane];
        }
        const int l = l0 + 4 * v + g;
        const double z = hm_combine(p, q, lane, sgn);
        if (l < k) out[(long)l * kHmCols + col] = z;
      }
    __syncthreads();
  }
}

struct TileArgs {
  int n;                // N or C
  const int* perm;      // position -> mesh index
  const int* row0;      // KIND 1: cell_start (rows of tile T: [row0[T], row0[T + 1]))
  const int* list_ptr;
  const HmEnt* ent;     // the list entries, resolved
  const double* zw;
  const double* xp;
  int nr;
  double sgn;
};

// One wave per 16 output rows of a tile (four waves a workgroup): it walks the
// tile's list and adds each block's rows times its input, straight from memory
// (the four waves share the input through L1), into the same two accumulators;
// nothing is staged and no wave waits for another.  Entries: a dense block as
// it is (kind 0) or transposed (1), or the rows of a low-rank block's factor
// (2, 3) times its projections.  Eight waves a SIMD hold every wave of level 6
// at once.  Bound: memory, dense blocks twice and the factor rows once (level 6,
// tol 1e-4: T_A 0.81 ms = 3.5 TB/s, V 0.48, where blocks staged in LDS took 2.20
// and 1.45).
template <int KIND>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8)))
void k_hm_tile(const TileArgs a, double* __restrict__ y) {
  const int T = blockIdx.x;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, col = lane & 15;
  const int p0 = KIND == 0 ? T * kEdgeTile : a.row0[T];
  const int nrow = KIND == 0 ? min(kEdgeTile, a.n - p0) : a.row0[T + 1] - p0;
  const int e0 = a.list_ptr[T], e1 = a.list_ptr[T + 1];
  for (int base = 16 * w; base < nrow; base += 64) {
    const int i = min(base + col, nrow - 1);
    HmAcc acc;
    HmEnt next = a.ent[min(e0, e1 - 1)];
    for (int e = e0; e < e1; ++e) {
      const HmEnt E = next;
      next = a.ent[min(e + 1, e1 - 1)];
      const int kind = E.code & 3, k = E.k;
      if (kind < 2) {  // k input rows from position `start` on; `len` entries between the block's rows
        const float2* D = E.F + (kind == 0 ? (long)i * E.len : (long)i);
        const double* x0 = a.xp + (long)E.start * kHmCols + col;
        int c0 = 0;
        if (kind == 0) {
#pragma unroll 2
          for (; c0 + 16 <= k; c0 += 16) {
            const int c = c0 + 4 * g;
            float2 m[4];
            double x[4];
            hm_load4(D + c, m);
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = x0[(c + u) * kHmCols];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc.add(m[u], x[u]);
          }
        } else {
#pragma unroll 2
          for (; c0 + 16 <= k; c0 += 16) {
            const int c = c0 + 4 * g;
            float2 m[4];
            double x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              m[u] = D[(c + u) * (long)E.len];
              x[u] = x0[(c + u) * kHmCols];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) acc.add(m[u], x[u]);
          }
        }
        if (c0 < k) {  // the last, short chunk
          const int c = c0 + 4 * g;
          const long step = kind == 0 ? 1 : E.len;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int cu = min(c + u, k - 1);
            float2 m = D[cu * step];
            if (c + u >= k) m = make_float2(0.f, 0.f);
            acc.add(m, x0[cu * kHmCols]);
          }
        }
      } else {
        const float2* F = E.F + (p0 + i - E.start);
        const double* z = a.zw + E.zb * 2 + col;
        for (int l0 = 0; l0 < k; l0 += 16) {
          float2 m[4];
          double x[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int l = min(l0 + 4 * u + g, k - 1);
            m[u] = F[(long)l * E.len];
            x[u] = z[(long)l * kHmCols];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (l0 + 4 * u >= k) break;
            if (l0 + 4 * u + g >= k) m[u] = make_float2(0.f, 0.f);
            acc.add(m[u], x[u]);
          }
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double s = hm_combine(acc.p[v], acc.q[v], lane, a.sgn);
      const int row = base + 4 * v + g;
      if (row < nrow && (col >> 1) < a.nr) y[((long)(col >> 1) * a.n + a.perm[p0 + row]) * 2 + (col & 1)] = s;
    }
  }
}

// Dense write-out (complex64, the mesh's numbering): dense blocks and their
// transposes, low-rank blocks U V^T and their transposes.
template <int KIND>
__global__ __launch_bounds__(256) void k_hm_out_dense(int n, const int* __restrict__ perm, const int* __restrict__ row0,
                                                      const int2* __restrict__ ij, const float2* __restrict__ D,
                                                      const long* __restrict__ doff, float2* __restrict__ out) {
  const int b = blockIdx.x;
  const int I = ij[b].x, J = ij[b].y;
  int qI, nI, qJ, nJ;
  const float2* Db;
  if (KIND == 0) {
    qI = I * kEdgeTile;
    qJ = J * kEdgeTile;
    nI = min(kEdgeTile, n - qI);
    nJ = min(kEdgeTile, n - qJ);
    Db = D + (long)b * kEdgeTile * kEdgeTile;
  } else {
    qI = row0[I];
    nI = row0[I + 1] - qI;
    qJ = row0[J];
    nJ = row0[J + 1] - qJ;
    Db = D + doff[b];
  }
  const int ld = KIND == 0 ? kEdgeTile : nJ;
  for (int e = threadIdx.x; e < nI * nJ; e += 256) {
    const int r = e / nJ, c = e % nJ;
    const float2 v = Db[(long)r * ld + c];
    const long pr = perm[qI + r], pc = perm[qJ + c];
    out[pr * n + pc] = v;
    if (I != J) out[pc * n + pr] = v;
  }
}

__global__ __launch_bounds__(256) void k_hm_out_lr(int n, const int* __restrict__ perm, const HmLr* __restrict__ blk,
                                                   const int* __restrict__ rank, float2* const* __restrict__ Up,
                                                   float2* const* __restrict__ Vp, float2* __restrict__ out) {
  const int b = blockIdx.x;
  const HmLr B = blk[b];
  const int k = rank[b];
  const float2* U = Up[b];
  const float2* V = Vp[b];
  for (long e = threadIdx.x; e < (long)B.m * B.n; e += 256) {
    const int i = (int)(e / B.n), j = (int)(e % B.n);
    double sr = 0.0, si = 0.0;
    for (int l = 0; l < k; ++l) {
      const float2 u = U[(long)l * B.m + i], v = V[(long)l * B.n + j];
      sr += (double)u.x * v.x - (double)u.y * v.y;
      si += (double)u.x * v.y + (double)u.y * v.x;
    }
    const float2 val = make_float2((float)sr, (float)si);
    const long pr = perm[B.r0 + i], pc = perm[B.c0 + j];
    out[pr * n + pc] = val;
    out[pc * n + pr] = val;
  }
}

template <class T>
rfcmp_status upload(DevBuf& b, const std::vector<T>& v, hipStream_t s) {
  RF_TRY(b.alloc(sizeof(T) * std::max<size_t>(v.size(), 1)));
  if (!v.empty()) RF_HIP(hipMemcpyAsync(b.p, v.data(), sizeof(T) * v.size(), hipMemcpyHostToDevice, s));
  return RFCMP_OK;
}

}  // namespace

rfcmp_status hm_mesh_setup(rfcmp_mesh m, hipStream_t s) {
  if (m->hm) return RFCMP_OK;
  auto H = std::make_unique<HmMesh>();
  HmTree& t = H->t;
  hm_build_tree(m->h, t);
  const int64_t nd = (int64_t)t.dense_I.size(), nlr = (int64_t)t.lr_a.size();
  std::vector<int2> ij(nd);
  std::vector<long> voff(nd);
  int64_t vt = 0;
  for (int64_t b = 0; b < nd; ++b) {
    ij[b] = make_int2(t.dense_I[b], t.dense_J[b]);
    voff[b] = vt;
    vt += (int64_t)(t.cell_start[t.dense_I[b] + 1] - t.cell_start[t.dense_I[b]]) *
          (t.cell_start[t.dense_J[b] + 1] - t.cell_start[t.dense_J[b]]);
  }
  H->vd_total = vt;
  std::vector<HmLr> la(nlr), lv(nlr);
  for (int64_t b = 0; b < nlr; ++b) {
    const HmNode& A = t.nodes[t.lr_a[b]];
    const HmNode& B = t.nodes[t.lr_b[b]];
    la[b] = HmLr{(int)A.e0, (int)(A.e1 - A.e0), (int)B.e0, (int)(B.e1 - B.e0)};
    lv[b] = HmLr{(int)A.c0, (int)(A.c1 - A.c0), (int)B.c0, (int)(B.c1 - B.c0)};
  }
  // per tile, the blocks its rows meet (dense first, then low-rank, each in
  // block order)
  std::vector<std::vector<int>> lists(t.ntiles);
  for (int64_t b = 0; b < nd; ++b) {
    lists[t.dense_I[b]].push_back((int)(4 * b + 0));
    if (t.dense_I[b] != t.dense_J[b]) lists[t.dense_J[b]].push_back((int)(4 * b + 1));
  }
  for (int64_t b = 0; b < nlr; ++b) {
    const HmNode& A = t.nodes[t.lr_a[b]];
    const HmNode& B = t.nodes[t.lr_b[b]];
    for (int q = A.t0; q < A.t1; ++q) lists[q].push_back((int)(4 * b + 2));
    for (int q = B.t0; q < B.t1; ++q) lists[q].push_back((int)(4 * b + 3));
  }
  std::vector<int> lp(t.ntiles + 1, 0), le;
  for (int64_t q = 0; q < t.ntiles; ++q) {
    le.insert(le.end(), lists[q].begin(), lists[q].end());
    lp[q + 1] = (int)le.size();
  }
  RF_TRY(upload(H->perm_e, t.perm_e, s));
  RF_TRY(upload(H->perm_c, t.perm_c, s));
  RF_TRY(upload(H->iperm_c, t.iperm_c, s));
  RF_TRY(upload(H->cell_start, t.cell_start, s));
  RF_TRY(upload(H->et_ptr, t.et_ptr, s));
  RF_TRY(upload(H->et_cell, t.et_cell, s));
  RF_TRY(upload(H->et_rows, t.et_rows, s));
  RF_TRY(upload(H->home, t.home, s));
  RF_TRY(upload(H->dense_ij, ij, s));
  RF_TRY(upload(H->vd_off, voff, s));
  RF_TRY(upload(H->lrA, la, s));
  RF_TRY(upload(H->lrV, lv, s));
  RF_TRY(upload(H->list_ptr, lp, s));
  RF_HIP(hipStreamSynchronize(s));  // the host vectors go out of scope
  H->list_host = std::move(le);
  H->vd_host = std::move(voff);
  m->hm = std::move(H);
  return RFCMP_OK;
}

rfcmp_status hm_aca(rfcmp_op op, hipStream_t s) {
  rfcmp_mesh m = op->mesh;
  const MeshDev& d = m->d;
  const HmMesh& H = *m->hm;
  HmOp& P = *op->hm;
  const HmTree& t = H.t;
  const int64_t nlr = (int64_t)t.lr_a.size();
  P.lr_entries[0] = P.lr_entries[1] = 0;
  P.unconverged = 0;
  std::vector<long> zoff_all[2];
  int64_t zw_need = 0;
  for (int kind = 0; kind < 2; ++kind) {
    std::vector<HmLr> blk(nlr);
    for (int64_t b = 0; b < nlr; ++b) {
      const HmNode& A = t.nodes[t.lr_a[b]];
      const HmNode& B = t.nodes[t.lr_b[b]];
      blk[b] = kind == 0 ? HmLr{(int)A.e0, (int)(A.e1 - A.e0), (int)B.e0, (int)(B.e1 - B.e0)}
                         : HmLr{(int)A.c0, (int)(A.c1 - A.c0), (int)B.c0, (int)(B.c1 - B.c0)};
    }
    // passes over the blocks whose working factors (kmax columns) fit a
    // bounded pool
    std::vector<long> uoff(nlr), voff(nlr), toff(nlr);
    std::vector<int64_t> pass_start{0};
    const long pool_cap = 1L << 29;  // complex64 entries (4 GB)
    long used = 0, tused = 0, pool_max = 1, taken_max = 1;
    for (int64_t b = 0; b < nlr; ++b) {
      const long kc = std::min<long>(kHmKmax, std::min(blk[b].m, blk[b].n));
      const long need = kc * (blk[b].m + blk[b].n);
      if (b > pass_start.back() && used + need > pool_cap) {
        pass_start.push_back(b);
        used = 0;
        tused = 0;
      }
      uoff[b] = used;
      voff[b] = used + kc * blk[b].m;
      toff[b] = tused;
      used += need;
      tused += blk[b].m;
      pool_max = std::max(pool_max, used);
      taken_max = std::max(taken_max, tused);
    }
    pass_start.push_back(nlr);
    DevBuf dblk, duoff, dvoff, dtoff, drank, dflag, pool, taken;
    DevBuf& up = kind == 0 ? P.uA : P.uV;
    DevBuf& vp = kind == 0 ? P.vA : P.vV;
    DevBuf& rk = kind == 0 ? P.rankA : P.rankV;
    RF_TRY(upload(dblk, blk, s));
    RF_TRY(upload(duoff, uoff, s));
    RF_TRY(upload(dvoff, voff, s));
    RF_TRY(upload(dtoff, toff, s));
    RF_TRY(rk.alloc(sizeof(int) * std::max<int64_t>(nlr, 1)));
    RF_TRY(dflag.alloc(sizeof(int) * std::max<int64_t>(nlr, 1)));
    RF_TRY(up.alloc(sizeof(float2*) * std::max<int64_t>(nlr, 1)));
    RF_TRY(vp.alloc(sizeof(float2*) * std::max<int64_t>(nlr, 1)));
    RF_TRY(pool.alloc(sizeof(float2) * pool_max));
    RF_TRY(taken.alloc((size_t)taken_max));
    AcaArgs a;
    a.perm = kind == 0 ? H.perm_e.as<int>() : H.perm_c.as<int>();
    a.edge_slot = d.edge_slot.as<int>();
    a.cen = d.cen.as<double>();
    a.qoff = d.qoff.as<float4>();
    a.fvoff = d.fvoff.as<float4>();
    a.sgn = d.sgn.as<float>();
    a.rule = rule_args();
    a.kk = (float)op->k;
    a.tol = (float)P.tol;
    a.kmax = kHmKmax;
    a.blk = dblk.as<HmLr>();
    a.uoff = duoff.as<long>();
    a.voff = dvoff.as<long>();
    a.toff = dtoff.as<long>();
    a.pool = pool.as<float2>();
    a.taken = taken.as<unsigned char>();
    a.rank = rk.as<int>();
    a.flag = dflag.as<int>();
    std::vector<int>& hr = kind == 0 ? P.hrankA : P.hrankV;
    hr.assign(nlr, 0);
    std::vector<float2*> hu(nlr, nullptr), hv(nlr, nullptr);
    {
      ProfScope prof(kind == 0 ? "hm_aca_ta" : "hm_aca_v", s);
      for (size_t q = 0; q + 1 < pass_start.size(); ++q) {
        const int64_t b0 = pass_start[q], b1 = pass_start[q + 1];
        if (b1 <= b0) continue;
        void (*kern)(const AcaArgs, int) = kind == 0 ? k_aca<0> : k_aca<1>;
        hipLaunchKernelGGL(kern, dim3((unsigned)(b1 - b0)), dim3(kAcaThreads), 0, s, a, (int)b0);
        RF_HIP(hipGetLastError());
        RF_HIP(hipMemcpyAsync(hr.data() + b0, rk.as<int>() + b0, sizeof(int) * (b1 - b0), hipMemcpyDeviceToHost, s));
        RF_HIP(hipStreamSynchronize(s));
        long tot = 0;
        for (int64_t b = b0; b < b1; ++b) tot += (long)hr[b] * (blk[b].m + blk[b].n);
        P.store.push_back(std::make_unique<DevBuf>());
        DevBuf& st = *P.store.back();
        RF_TRY(st.alloc(sizeof(float2) * std::max<long>(tot, 1)));
        long o = 0;
        for (int64_t b = b0; b < b1; ++b) {
          hu[b] = st.as<float2>() + o;
          o += (long)hr[b] * blk[b].m;
          hv[b] = st.as<float2>() + o;
          o += (long)hr[b] * blk[b].n;
        }
        P.lr_entries[kind] += tot;
        RF_HIP(hipMemcpyAsync(up.as<float2*>() + b0, hu.data() + b0, sizeof(float2*) * (b1 - b0),
                              hipMemcpyHostToDevice, s));
        RF_HIP(hipMemcpyAsync(vp.as<float2*>() + b0, hv.data() + b0, sizeof(float2*) * (b1 - b0),
                              hipMemcpyHostToDevice, s));
        hipLaunchKernelGGL(k_aca_compact, dim3((unsigned)(b1 - b0)), dim3(256), 0, s, (int)b0, dblk.as<HmLr>(),
                           rk.as<int>(), duoff.as<long>(), dvoff.as<long>(), pool.as<float2>(),
                           up.as<float2*>(), vp.as<float2*>());
        RF_HIP(hipGetLastError());
        RF_HIP(hipStreamSynchronize(s));  // the pool is reused by the next pass
      }
    }
    std::vector<int> hf(nlr, 0);
    if (nlr > 0)
      RF_HIP(hipMemcpyAsync(hf.data(), dflag.p, sizeof(int) * nlr, hipMemcpyDeviceToHost, s));
    RF_HIP(hipStreamSynchronize(s));
    for (int64_t b = 0; b < nlr; ++b) P.unconverged += hf[b];
    // offsets of the projections z, w (2 k kHmR complex128 per block)
    std::vector<long>& zo = zoff_all[kind];
    zo.assign(nlr, 0);
    long zt = 0;
    for (int64_t b = 0; b < nlr; ++b) {
      zo[b] = zt;
      zt += 2L * hr[b] * kHmR;
    }
    zw_need = std::max<int64_t>(zw_need, zt);
    // the tile lists' entries resolved for this operator
    std::vector<HmEnt> ent(H.list_host.size());
    for (size_t e = 0; e < ent.size(); ++e) {
      const int code = H.list_host[e], b = code >> 2;
      HmEnt E{nullptr, 0, 0, 0, 0, code};
      if ((code & 3) >= 2) {
        const bool rows = (code & 3) == 2;
        E.F = rows ? hu[b] : hv[b];
        E.start = rows ? blk[b].r0 : blk[b].c0;
        E.len = rows ? blk[b].m : blk[b].n;
        E.k = hr[b];
        E.zb = zo[b] + (rows ? 0 : (long)hr[b] * kHmR);
      } else {
        const bool rows = (code & 3) == 0;   // else its transpose
        const int I = t.dense_I[b], J = t.dense_J[b];
        const int qI = kind == 0 ? I * kEdgeTile : t.cell_start[I], qJ = kind == 0 ? J * kEdgeTile : t.cell_start[J];
        const int nI = kind == 0 ? (int)std::min<int64_t>(kEdgeTile, t.N - qI) : t.cell_start[I + 1] - qI;
        const int nJ = kind == 0 ? (int)std::min<int64_t>(kEdgeTile, t.N - qJ) : t.cell_start[J + 1] - qJ;
        E.F = kind == 0 ? P.TAd.as<float2>() + (long)b * kEdgeTile * kEdgeTile : P.Vd.as<float2>() + H.vd_host[b];
        E.start = rows ? qJ : qI;
        E.k = rows ? nJ : nI;
        E.len = kind == 0 ? kEdgeTile : nJ;
      }
      ent[e] = E;
    }
    RF_TRY(upload(kind == 0 ? P.entA : P.entV, ent, s));
    RF_HIP(hipStreamSynchronize(s));  // ent goes out of scope
  }
  RF_TRY(upload(P.zwA, zoff_all[0], s));
  RF_TRY(upload(P.zwV, zoff_all[1], s));
  P.zw_total = zw_need;
  RF_TRY(P.zw.alloc(sizeof(double2) * std::max<int64_t>(zw_need, 1)));
  RF_TRY(P.xp.alloc(sizeof(double2) * kHmR * std::max<int64_t>(std::max(t.N, t.C), 1)));
  RF_HIP(hipStreamSynchronize(s));
  if (P.unconverged > 0) {
    set_error("ACA: %d low-rank blocks reached rank %d above the tolerance %g", P.unconverged, kHmKmax, P.tol);
    return RFCMP_E_STATE;
  }
  return RFCMP_OK;
}

rfcmp_status hm_matvec(rfcmp_op op, int which, bool conj, const double2* x, double2* y, int nr, hipStream_t s) {
  const HmMesh& H = *op->mesh->hm;
  HmOp& P = *op->hm;
  const HmTree& t = H.t;
  const int n = (int)(which == 0 ? t.N : t.C);
  const int64_t nlr = (int64_t)t.lr_a.size();
  if (n == 0 || nr <= 0) return RFCMP_OK;
  ProfScope prof(profiling_enabled() ? profile_tag_suffix(which == 0 ? "hm_matvec_ta" : "hm_matvec_v", nr) : "hm", s);
  TileArgs ta;
  ta.n = n;
  ta.perm = which == 0 ? H.perm_e.as<int>() : H.perm_c.as<int>();
  ta.row0 = H.cell_start.as<int>();
  ta.list_ptr = H.list_ptr.as<int>();
  ta.ent = which == 0 ? P.entA.as<HmEnt>() : P.entV.as<HmEnt>();
  ta.zw = P.zw.as<double>();
  ta.xp = P.xp.as<double>();
  ta.sgn = conj ? -1.0 : 1.0;
  const long tot = (long)n * kHmR;
  for (int r0 = 0; r0 < nr; r0 += kHmR) {
    ta.nr = std::min(kHmR, nr - r0);
    hipLaunchKernelGGL(k_hm_gather, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, n, ta.nr, ta.perm,
                       x + (long)r0 * n, P.xp.as<double2>());
    if (nlr > 0)
      hipLaunchKernelGGL(k_hm_proj, dim3((unsigned)nlr, 2), dim3(256), 0, s,
                         which == 0 ? H.lrA.as<HmLr>() : H.lrV.as<HmLr>(),
                         which == 0 ? P.rankA.as<int>() : P.rankV.as<int>(),
                         which == 0 ? P.uA.as<float2*>() : P.uV.as<float2*>(),
                         which == 0 ? P.vA.as<float2*>() : P.vV.as<float2*>(),
                         which == 0 ? P.zwA.as<long>() : P.zwV.as<long>(), ta.xp, ta.sgn, P.zw.as<double>());
    void (*tile)(const TileArgs, double*) = which == 0 ? k_hm_tile<0> : k_hm_tile<1>;
    hipLaunchKernelGGL(tile, dim3((unsigned)t.ntiles), dim3(256), 0, s, ta, reinterpret_cast<double*>(y + (long)r0 * n));
    RF_HIP(hipGetLastError());
  }
  return RFCMP_OK;
}

rfcmp_status hm_export(rfcmp_op op, float2* TA, float2* V, hipStream_t s) {
  const HmMesh& H = *op->mesh->hm;
  const HmOp& P = *op->hm;
  const HmTree& t = H.t;
  const int64_t nd = (int64_t)t.dense_I.size(), nlr = (int64_t)t.lr_a.size();
  if (TA) {
    RF_HIP(hipMemsetAsync(TA, 0, sizeof(float2) * t.N * t.N, s));
    if (nd > 0)
      hipLaunchKernelGGL(k_hm_out_dense<0>, dim3((unsigned)nd), dim3(256), 0, s, (int)t.N, H.perm_e.as<int>(),
                         H.cell_start.as<int>(), H.dense_ij.as<int2>(), P.TAd.as<float2>(), H.vd_off.as<long>(), TA);
    if (nlr > 0)
      hipLaunchKernelGGL(k_hm_out_lr, dim3((unsigned)nlr), dim3(256), 0, s, (int)t.N, H.perm_e.as<int>(),
                         H.lrA.as<HmLr>(), P.rankA.as<int>(), P.uA.as<float2*>(), P.vA.as<float2*>(), TA);
    RF_HIP(hipGetLastError());
  }
  if (V) {
    RF_HIP(hipMemsetAsync(V, 0, sizeof(float2) * t.C * t.C, s));
    if (nd > 0)
      hipLaunchKernelGGL(k_hm_out_dense<1>, dim3((unsigned)nd), dim3(256), 0, s, (int)t.C, H.perm_c.as<int>(),
                         H.cell_start.as<int>(), H.dense_ij.as<int2>(), P.Vd.as<float2>(), H.vd_off.as<long>(), V);
    if (nlr > 0)
      hipLaunchKernelGGL(k_hm_out_lr, dim3((unsigned)nlr), dim3(256), 0, s, (int)t.C, H.perm_c.as<int>(),
                         H.lrV.as<HmLr>(), P.rankV.as<int>(), P.uV.as<float2*>(), P.vV.as<float2*>(), V);
    RF_HIP(hipGetLastError());
  }
  return RFCMP_OK;
}

}  // namespace rfcmp
