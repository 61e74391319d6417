// Complex products Y = M X (or conj(M) X) of a complex64 matrix stored whole
// with many complex128 right-hand sides, accumulated in FP64 on the FP64
// matrix cores (v_mfma_f64_16x16x4).  They serve the FP64-accumulated
// products of T_A and V (the refinement residual, the right-hand side, the
// FP32-path iterations) once there are enough right-hand sides that the
// products are bound by FP64 arithmetic rather than by the matrix stream:
// with 32 right-hand sides a pass does 192 flops per matrix entry (8 bytes),
// where the symmetric streaming product (symv.hip) can take 8.
//
// Three real products per complex one (Gauss): with M = Mr + i Mi and
// X = Xr + i Xi,
//   P1 = Mr Xr,  P2 = Mi Xi,  P3 = (Mr + Mi)(Xr + Xi),
//   Re Y = P1 - P2,  Im Y = P3 - P1 - P2,
// so 16 right-hand sides take three 16-column MFMA operands where the
// four-product form takes four.  In FP64 the extra rounding of the sums is
// of order 1e-16 relative to |M| |X|, far below the complex64 storage of M.
// A launch serves NG groups of 16 right-hand sides (NG = 2 from 17 on), so
// that each pass over the matrix does 3 NG MFMAs per K step and 16 rows.
//
// A workgroup (4 waves) owns 128 rows over one K slice, a wave 32 rows in two
// 16-row tiles (64 and one where those would leave the chip idle, zgemm_wide).
// M is symmetric and stored whole, so the operand M[i][k] is read as M[k][i]: 16
// neighbouring lanes take 256 contiguous bytes of row k, a workgroup 1 KB (read
// along its own row, a lane's 16 bytes stood 64 apart and every load touched 64
// lines).  The accumulators live in plain VGPRs (at
// least two waves per SIMD are asked for, else the compiler takes AGPRs).  The
// X chunk of 32 columns sits in LDS in operand order, one 512-byte wave read
// per operand, the next step's read while this step's products run.  Partial
// sums of the K slices go to a buffer [slice][32][n] (complex128); a second
// kernel adds the slices in order (the result does not depend on timing).
//
// Bound: the FP64 matrix cores, 77.8 TFLOP/s in a register-only probe.  At
// n = 30720 with 32 right-hand sides 3.02 ms (4.03 before, with one 16-row
// tile per wave read along the rows): 60 TFLOP/s of executed flops, 80 of
// algorithmic ones.  The conversions and sums of the operands take issue slots
// of the matrix cores (8 FP64 operations per 12 MFMAs), the rest is the wait
// at the chunk's barrier.  With 16 right-hand sides 1.74 ms (2.60 before), 4.3
// TB/s of the matrix: there the stream weighs as much as the products.
#include <type_traits>

#include "internal.h"
#include "gemm.h"

namespace rfcmp {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int kZThreads = 256;
template <int TILES>
constexpr int kZRows = 64 * TILES;             // rows per workgroup, TILES 16-row tiles a wave
constexpr int kZK = 32;                        // K chunk
constexpr int kZRhs = 32;                      // right-hand sides per launch (at most)
constexpr int kZLd = 66;                       // padded lane row of a stage

// lds[g][b][e][l]: operand b (0: Xr, 1: Xi) of group g at step e for lane l
// (chunk column 8 (l / 16) + e, right-hand side 16 g + l % 16).  A step's lanes
// are padded to 66 entries, so that the stores of neighbouring columns spread
// over the banks.
template <int NG>
struct ZStage {
  double v[NG][2][8][kZLd];
};

// X chunk into the operand order, 32 consecutive columns of a right-hand side
// per half wave.  The loads go to registers first (z_load_x, before the
// products of the current chunk) and to LDS after them (z_store_x, which
// zeroes what lies beyond the slice or the right-hand sides: the loads
// themselves are never conditional, so that the wait counts stay exact).
template <int NG>
__device__ inline void z_load_x(double2 (&xr)[2 * NG], const double2* __restrict__ X, int n, int nr, int kc, int tid) {
#pragma unroll
  for (int u = 0; u < 2 * NG; ++u) {
    const int idx = tid + u * kZThreads;
    const int k = min(kc + idx % kZK, n - 1), r = min(idx / kZK, nr - 1);
    xr[u] = X[(long)r * n + k];
  }
}
template <int NG>
__device__ inline void z_store_x(ZStage<NG>& st, const double2 (&xr)[2 * NG], int kc, int k_end, int nr, int tid) {
#pragma unroll
  for (int u = 0; u < 2 * NG; ++u) {
    const int idx = tid + u * kZThreads;
    const int k = idx % kZK, r = idx / kZK;
    const int g = r / 16, e = k % 8, ll = (k / 8) * 16 + r % 16;
    const bool in = kc + k < k_end && r < nr;
    st.v[g][0][e][ll] = in ? xr[u].x : 0.0;
    st.v[g][1][e][ll] = in ? xr[u].y : 0.0;
  }
}

// the matrix: M is symmetric, so operand row i, column k is read as M[k][i],
// along the rows of the store: a lane takes one operand row per tile, neighbours
// in the store, 16 lanes 256 (128 with one tile) contiguous bytes of one k.
// Columns beyond the slice repeat the last one (their X entries are zero).
template <int TILES>
struct ZFrag {
  typedef float Entries __attribute__((ext_vector_type(2 * TILES)));
  Entries e[kZK / 4];
};
template <int TILES>
__device__ inline void z_load_m(ZFrag<TILES>& av, const float2* __restrict__ src, long ld, int kc, int n, int lane) {
#pragma unroll
  for (int e = 0; e < kZK / 4; ++e) {
    const int k = min(kc + 8 * (lane >> 4) + e, n - 1);
    av.e[e] =
        __builtin_nontemporal_load(reinterpret_cast<const typename ZFrag<TILES>::Entries*>(src + (long)k * ld));
  }
}

template <int NG>
__device__ inline void z_operands(double (&xb)[NG][2], const ZStage<NG>& st, int e, int lane) {
#pragma unroll
  for (int g = 0; g < NG; ++g)
#pragma unroll
    for (int b = 0; b < 2; ++b) xb[g][b] = st.v[g][b][e][lane];
}

template <bool CONJ, int NG, int TILES>
__device__ inline void z_mfma(dbl4 (&acc)[TILES][NG][3], const ZFrag<TILES>& av, const ZStage<NG>& st, int lane) {
  double xb[2][NG][2];
  z_operands<NG>(xb[0], st, 0, lane);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    // the next step's operands leave LDS while this step's products run
    if (e + 1 < 8) z_operands<NG>(xb[(e + 1) & 1], st, e + 1, lane);
    double mb[3][TILES], xs[NG][3];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      xs[g][0] = xb[e & 1][g][0];
      xs[g][1] = xb[e & 1][g][1];
      xs[g][2] = xs[g][0] + xs[g][1];
    }
#pragma unroll
    for (int a = 0; a < TILES; ++a) {
      mb[0][a] = (double)av.e[e][2 * a];
      mb[1][a] = CONJ ? -(double)av.e[e][2 * a + 1] : (double)av.e[e][2 * a + 1];
      mb[2][a] = mb[0][a] + mb[1][a];
    }
    // each accumulator is taken once per step, 3 NG TILES instructions apart
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int a = 0; a < TILES; ++a)
#pragma unroll
        for (int g = 0; g < NG; ++g)
          acc[a][g][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(mb[b][a], xs[g][b], acc[a][g][b], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);  // later steps' conversions stay behind (registers)
  }
}

// Two chunks in flight: the loads of chunk c + 1 (matrix into registers, X
// into the other LDS stage) are issued before the products of chunk c.  With two
// tiles the chunks run in pairs without an exit between them (a slice of an odd
// count takes one of zeros): with one, the accumulators had two homes and were
// copied between them.  With one tile, whose slices are a few chunks, the chunk
// of zeros costs more.
template <bool CONJ, int NG, int TILES>
__global__ __launch_bounds__(kZThreads) __attribute__((amdgpu_waves_per_eu(NG == 1 ? 3 : 2, NG == 1 ? 3 : 2)))
void k_zgemm(const float2* __restrict__ M, int n, long ld, const double2* __restrict__ X, int nr, int kslice,
             double2* __restrict__ part) {
  __shared__ ZStage<NG> st[2];
  const int rb = blockIdx.x, ks = blockIdx.y;
  const int k_begin = ks * kslice, k_end = min(n, k_begin + kslice);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int row0 = rb * kZRows<TILES> + w * 16 * TILES;
  const float2* src = M + min((long)row0 + TILES * (lane & 15), ld - TILES);
  dbl4 acc[TILES][NG][3];
#pragma unroll
  for (int a = 0; a < TILES; ++a)
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int b = 0; b < 3; ++b) acc[a][g][b] = dbl4{0.0, 0.0, 0.0, 0.0};
  ZFrag<TILES> va, vb;
  double2 xr[2 * NG];
  z_load_m(va, src, ld, k_begin, n, lane);
  z_load_x<NG>(xr, X, n, nr, k_begin, tid);
  z_store_x<NG>(st[0], xr, k_begin, k_end, nr, tid);
  __syncthreads();
  for (int kc = k_begin; kc < k_end; kc += 2 * kZK) {
    const int k1 = kc + kZK, k2 = kc + 2 * kZK;
    z_load_x<NG>(xr, X, n, nr, k1, tid);
    z_load_m(vb, src, ld, k1, n, lane);
    __builtin_amdgcn_sched_barrier(0);
    z_mfma<CONJ, NG, TILES>(acc, va, st[0], lane);
    if (TILES == 1 && k1 >= k_end) break;
    z_store_x<NG>(st[1], xr, k1, k_end, nr, tid);  // waits for its loads here, after the products
    __syncthreads();                               // stage 1 written, stage 0 read
    z_load_x<NG>(xr, X, n, nr, k2, tid);
    z_load_m(va, src, ld, k2, n, lane);
    __builtin_amdgcn_sched_barrier(0);
    z_mfma<CONJ, NG, TILES>(acc, vb, st[1], lane);
    z_store_x<NG>(st[0], xr, k2, k_end, nr, tid);
    __syncthreads();  // stage 0 written, stage 1 read
  }
  // accumulator value v of lane l: operand row 4 v + l / 16 (tile a holds the
  // wave's rows TILES i + a), right-hand side 16 g + l % 16
  double2* pd = part + (long)ks * kZRhs * n;
#pragma unroll
  for (int a = 0; a < TILES; ++a)
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = row0 + TILES * (4 * v + (lane >> 4)) + a;
        const int r = 16 * g + (lane & 15);
        const double p1 = acc[a][g][0][v], p2 = acc[a][g][1][v], p3 = acc[a][g][2][v];
        if (row < n && r < nr) pd[(long)r * n + row] = make_double2(p1 - p2, p3 - p1 - p2);
      }
}

// Y[r][i] = sum over the slices, in order, of part[s][r][i]
__global__ __launch_bounds__(256) void k_zgemm_sum(const double2* __restrict__ part, int n, int nr, int nslice,
                                                   double2* __restrict__ Y) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long)nr * n) return;
  const int r = (int)(t / n), i = (int)(t % n);
  double2 s = make_double2(0.0, 0.0);
  for (int q = 0; q < nslice; ++q) {
    const double2 v = part[((long)q * kZRhs + r) * n + i];
    s.x += v.x;
    s.y += v.y;
  }
  Y[(long)r * n + i] = s;
}

// K slices of a launch, at most 16 (8 at n = 30720, 12 at 20480).  The slices
// and the order of the columns inside a chunk fix the order of the sums, which
// the solves' iterates follow bit for bit.  Measured with 32 right-hand sides
// at n = 30720: 8 slices (3.75 rounds of 512 workgroups, two per compute unit)
// 3.02 ms, 17 slices (7.97 rounds) 2.89, 2 slices 3.05, 15 slices 3.05.
int zgemm_slices(int64_t n) {
  const int64_t rbs = (n + 63) / 64;
  return (int)std::min<int64_t>(16, std::max<int64_t>(1, (3840 + rbs / 2) / rbs));
}

// Two tiles a wave, or one where the launch leaves compute units short: by the
// chunks that the fullest compute unit walks (pairs of them with two tiles, each
// of twice the rows), one tile at 1.15 times its share (with nearly equal ones it
// is 3 to 7 % slower: n = 7680 237 us to 222, 10 368 411 to 397).  The same bits either way.  With 32 right-hand
// sides n = 320: 13.6 us with one tile, 15.8 with two; 480 13.5 and 17.1; 2352 41
// and 54; 4608 99 and 112; 4056, where the shares are equal, 75 and 69.
bool zgemm_wide(int64_t n, int kslice, int nsl) {
  auto share = [&](int64_t rows) { return ((n + rows - 1) / rows * nsl + 255) / 256; };
  const int64_t chunks = kslice / kZK;
  return 2.0 * (chunks + chunks % 2) * share(kZRows<2>) <= 1.15 * chunks * share(kZRows<1>);
}

}  // namespace

size_t zgemm_scratch_bytes(int64_t n) { return sizeof(double2) * (size_t)zgemm_slices(n) * kZRhs * (size_t)n; }

rfcmp_status zgemm_c64(const float2* M, int64_t n, int64_t ld, bool conj, const double2* X, double2* Y, int nrhs,
                       void* scratch, size_t scratch_bytes, hipStream_t s, const char* tag) {
  if (n <= 0 || nrhs <= 0) return RFCMP_OK;
  if (ld < (n + kZK - 1) / kZK * kZK || ld % 4 != 0 || n > INT32_MAX / 2) {
    set_error("zgemm: n = %lld, ld = %lld (ld >= n rounded up to %d, a multiple of 4)", (long long)n, (long long)ld, kZK);
    return RFCMP_E_ARG;
  }
  if (scratch_bytes < zgemm_scratch_bytes(n)) {
    set_error("zgemm: needs %zu bytes of scratch, %zu given", zgemm_scratch_bytes(n), scratch_bytes);
    return RFCMP_E_ARG;
  }
  const int ns = zgemm_slices(n);
  const int kslice = (int)(((n + ns - 1) / ns + kZK - 1) / kZK * kZK);
  const int nsl = (int)((n + kslice - 1) / kslice);
  const bool wide = zgemm_wide(n, kslice, nsl);
  const int64_t rows = wide ? kZRows<2> : kZRows<1>;
  const dim3 grid((unsigned)((n + rows - 1) / rows), (unsigned)nsl);
  double2* part = static_cast<double2*>(scratch);
  for (int r0 = 0; r0 < nrhs; r0 += kZRhs) {
    const int nr = std::min(kZRhs, nrhs - r0);
    ProfScope prof(profile_tag_suffix(tag, nr), s);
    auto pick = [&](auto c) {
      constexpr bool C = decltype(c)::value;
      return nr > 16 ? (wide ? k_zgemm<C, 2, 2> : k_zgemm<C, 2, 1>) : (wide ? k_zgemm<C, 1, 2> : k_zgemm<C, 1, 1>);
    };
    const auto kern = conj ? pick(std::true_type()) : pick(std::false_type());
    hipLaunchKernelGGL(kern, grid, dim3(kZThreads), 0, s, M, (int)n, (long)ld, X + (long)r0 * n, nr, kslice, part);
    hipLaunchKernelGGL(k_zgemm_sum, dim3((unsigned)(((long)nr * n + 255) / 256)), dim3(256), 0, s, part, (int)n, nr,
                       nsl, Y + (long)r0 * n);
  }
  RF_HIP(hipGetLastError());
  return RFCMP_OK;
}

}  // namespace rfcmp
