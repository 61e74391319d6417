// Symmetric streaming matrix-vector products.
//
// Every dense matrix the operator applies is symmetric: T_A and V are
// complex-symmetric Galerkin blocks (T_A = T_A^T, V = V^T), and L^+, G_ll^-1
// and G_tp^-1 are real symmetric.  The products are HBM-bound (about one flop
// per byte), so reading each off-diagonal entry once and using it for two
// outputs halves the time:  with the matrix cut into S x S blocks,
//   block (P, Q), P < Q:  y_P += M_PQ x_Q   and   y_Q += M_PQ^T x_P,
//   block (P, P):         y_P += M_PP x_P   (read whole),
// only blocks with Q >= P are read.  Each workgroup owns one block and writes
// its two partial outputs to a slot of a partial buffer, part[K][L] = the
// contribution to output block K from the block pairing K with L; a second
// kernel sums the slots of each output block in a fixed order.  The result
// is deterministic (no atomics) and the matrix is read from its upper block
// triangle only.
//
// A block is streamed in sub-tiles of 32 rows x S columns: each thread loads
// 16-byte column pairs of several rows into registers (coalesced: a wave
// reads a whole row), accumulates the transposed product M^T x_P for its
// column pair straight from registers, and stores the sub-tile to LDS, from
// where eight threads per row form the row sums M x_Q (thread s of a row
// takes pairs s, s + 8, ..., so a row's threads read adjacent LDS words; the
// eight partial sums meet through DPP lane moves).
// Two sub-tiles are in flight per workgroup: the loads of sub-tile t + 2 are
// issued as soon as sub-tile t sits in LDS, without a condition, so that the
// wait for a sub-tile leaves the other one in flight.  Products are formed
// and accumulated in FP64 (complex64 entries are widened), x and y are
// complex128.
//
// The input x is formed while it is staged (SymvInput): a plain vector, or a
// sparse incidence product (Sigma^T, Lambda^T) or fused operator line of
// vectors already in HBM.  Each workgroup forms only the 2 x 128 entries it
// needs, reading a few source entries per entry from L2.  One launch can
// carry two products of the same element type (their blocks side by side in
// the grid), so a small matrix rides along with a large one.
//
// Bound: the stream, together with the partial sums written beside it.  T_A at
// N = 30720 takes 650 us (5.8 TB/s) with one right-hand side; the same blocks
// read without any sums take 545 us, with the 59 MB of slot writes alone 650.
#include "symv.h"
#include "symv_input.h"

namespace rfcmp {

namespace {

typedef float vf4 __attribute__((ext_vector_type(4)));
typedef double vd2 __attribute__((ext_vector_type(2)));
typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
// rows per sub-tile for block size S: the sub-tile is 4 KB of pairs per 256 threads
template <int S>
constexpr int rows_sub() { return S == 128 ? 32 : 16; }
// Pairs per LDS tile row: a 16-lane pass of the row sums covers 256 / S rows
// (two at S = 128), so rows are padded to start 128 bytes apart in the banks.
template <int S>
constexpr int tile_ld() { return S / 2 + 8; }

// Entry e (0, 1) of a 16-byte column pair, widened to FP64 (re, im).
struct C64 {
  typedef vf4 Pair;
  static constexpr bool kComplex = true;
  // operand h of the transposed sums for column e of a load: (im, re) of its
  // rows 2 h, 2 h + 1, by an exchange of the odd rows of lanes of im with the
  // even ones of re
  __device__ static inline double col_operand(const Pair& v, int e, int h) {
    const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(e ? v.w : v.y), __float_as_uint(e ? v.z : v.x),
                                                    false, false);
    return (double)__uint_as_float(t[h]);
  }
  typedef float Row;
  __device__ static inline void mac(double ar, double ai, const double2& x, double& re, double& im) {
    re = fma(ar, x.x, fma(-ai, x.y, re));
    im = fma(ar, x.y, fma(ai, x.x, im));
  }
  __device__ static inline Pair first_only(Pair v) {
    v.z = 0.0f;
    v.w = 0.0f;
    return v;
  }
  template <bool CONJ>
  __device__ static inline void entry(const Pair& v, int e, double& re, double& im) {
    re = e ? (double)v.z : (double)v.x;
    const double t = e ? (double)v.w : (double)v.y;
    im = CONJ ? -t : t;
  }
};
struct F64 {
  typedef vd2 Pair;
  static constexpr bool kComplex = false;
  __device__ static inline double col_operand(const Pair& v, int e, int) { return e ? v.y : v.x; }
  typedef double Row;
  __device__ static inline void mac(double ar, double, const double2& x, double& re, double& im) {
    re = fma(ar, x.x, re);
    im = fma(ar, x.y, im);
  }
  __device__ static inline Pair first_only(Pair v) {
    v.y = 0.0;
    return v;
  }
  template <bool CONJ>
  __device__ static inline void entry(const Pair& v, int e, double& re, double& im) {
    re = e ? v.y : v.x;
    im = 0.0;
  }
};

template <class T>
__device__ inline typename T::Pair zero_pair() {
  typename T::Pair z;
  z = 0;
  return z;
}

__global__ void k_form_input(const SymvInput in, int n, double2* __restrict__ out) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  if (g < n) out[(long)r * n + g] = input_entry(in, r, g);
}

// Kernel arguments: up to two products; blocks [0, nblk0) belong to job 0.
struct JobArg {
  const void* M;
  int n;
  long ldp;  // row length in 16-byte pairs
  int nsb;
  SymvInput in;
  double2* part;
  double2* y;
};
struct JobsArg {
  JobArg j[2];
  int nblk0;
  int nsb0;
  int nr;   // right-hand sides of job 0
  int nr1;  // of job 1
};

// DPP move of a double: lane i takes the value of the lane CTRL selects
// (quad_perm or row shift); lanes without a source get 0.
template <int CTRL>
__device__ inline double dpp_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Sum over each aligned group of TPR (8 or 16) lanes; lanes TPR - 4 .. TPR - 1
// of a group hold it.
template <int TPR>
__device__ inline double sum_lanes(double v) {
  static_assert(TPR == 8 || TPR == 16, "group size");
  v += dpp_move<0xB1>(v);   // quad_perm [1,0,3,2]: lane ^ 1
  v += dpp_move<0x4E>(v);   // quad_perm [2,3,0,1]: lane ^ 2
  v += dpp_move<0x114>(v);  // row_shr:4: lanes 4..7 (of 8) add lanes 0..3
  if (TPR == 16) v += dpp_move<0x118>(v);  // row_shr:8: lanes 12..15 add lanes 4..7
  return v;
}

// One block (P, Q) of a product.  EDGE: the block reaches past n, so loads
// are masked (rows beyond n are not read, columns beyond n read as zero).
// The block's rows start at the uniform address `strip`; each thread
// addresses its 16-byte pairs by 32-bit offsets from it.
template <class T, int S, int NR, bool CONJ, bool EDGE>
__device__ void symv_block(const char* __restrict__ strip, int n, int ldp, int P, int Q,
                           const SymvInput& in, double2* __restrict__ part, int nsb,
                           typename T::Pair (*tile)[tile_ld<S>()], double2 (*xs)[NR][S]) {
  typedef typename T::Pair Pair;
  constexpr int kRowsSub = rows_sub<S>();
  constexpr int PP = S / 2;                       // column pairs per row
  constexpr int G = kThreads / PP;                // row groups in the load layout
  constexpr int LPT = kRowsSub / G;               // loads per thread per sub-tile
  constexpr int NSUB = S / kRowsSub;              // sub-tiles per block
  constexpr int TPR = kThreads / kRowsSub;        // threads per row in the row sums
  constexpr int PPT = PP / TPR;                   // pairs per thread in the row sums
  static_assert(kRowsSub % G == 0 && PP % TPR == 0 && NSUB % 2 == 0, "block shape");
  const bool diag = (P == Q);
  const int tid = threadIdx.x;

  // load layout: column pair p, rows g0 + G q of each sub-tile
  const int p = tid % PP, g0 = tid / PP;
  const int gc = Q * S + 2 * p;  // first global column of the pair
  const bool c0 = gc < n, c1 = gc + 1 < n;
  const unsigned ldb = (unsigned)ldp * 16u;
  const unsigned offc = (unsigned)((!EDGE || c0 ? gc : 0) >> 1) * 16u;
  Pair ra[LPT], rb[LPT];  // two sub-tiles in flight

  // The loads are never conditional, so that a wait for one sub-tile leaves
  // the other in flight: EDGE blocks read what lies beyond the matrix from a
  // place inside it, and SYMV_MASK clears it once it is used.
#define SYMV_LOAD(REG, SUB)                                                                        \
  _Pragma("unroll") for (int q = 0; q < LPT; ++q) {                                                \
    const int lr = (SUB) * kRowsSub + g0 + G * q;                                                  \
    const unsigned row = EDGE ? (unsigned)min(lr, n - 1 - P * S) : (unsigned)lr;                   \
    REG[q] = __builtin_nontemporal_load(reinterpret_cast<const Pair*>(strip + offc + row * ldb));  \
  }
#define SYMV_MASK(REG, SUB)                                                                        \
  if (EDGE) {                                                                                      \
    _Pragma("unroll") for (int q = 0; q < LPT; ++q) {                                              \
      const bool in = P * S + (SUB) * kRowsSub + g0 + G * q < n && c0;                             \
      const Pair v = in ? REG[q] : zero_pair<T>();                                                 \
      REG[q] = c1 ? v : T::first_only(v);                                                          \
    }                                                                                              \
  }
  SYMV_LOAD(ra, 0)
  SYMV_LOAD(rb, 1)
#pragma unroll
  for (int t = tid; t < 2 * S; t += kThreads) {
    const int side = t / S, i = t % S;
    const int g = (side == 0 ? P : Q) * S + i;
    // x_Q is stored even columns first, then odd ones, so that the row sums
    // (neighbouring threads, neighbouring pairs) read it without bank conflicts
    const int slot = side ? (i & 1) * (S / 2) + (i >> 1) : i;
    double2 v[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) v[r] = make_double2(0.0, 0.0);
    if (!EDGE || g < n) input_entries(in, 0, NR, g, v);
#pragma unroll
    for (int r = 0; r < NR; ++r) xs[side][r][slot] = v[r];
  }

  double cr[2][NR], ci[2][NR];  // transposed sums of the two columns
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int r = 0; r < NR; ++r) cr[e][r] = ci[e][r] = 0.0;
  const int rrow = tid / TPR, seg = tid % TPR;  // row-sum layout
  __syncthreads();  // xs ready

#define SYMV_CONSUME(REG, SUB, MORE)                                                               \
  {                                                                                                \
    SYMV_MASK(REG, SUB)                                                                            \
    if (!diag) {                                                                                   \
      _Pragma("unroll") for (int q = 0; q < LPT; ++q) {                                            \
        const int lr = (SUB) * kRowsSub + g0 + G * q;                                              \
        _Pragma("unroll") for (int e = 0; e < 2; ++e) {                                            \
          double ar, ai;                                                                           \
          T::template entry<CONJ>(REG[q], e, ar, ai);                                              \
          _Pragma("unroll") for (int r = 0; r < NR; ++r) {                                         \
            T::mac(ar, ai, xs[0][r][lr], cr[e][r], ci[e][r]);                                      \
          }                                                                                        \
        }                                                                                          \
      }                                                                                            \
    }                                                                                              \
    __syncthreads(); /* the previous row sums are done with the tile */                            \
    _Pragma("unroll") for (int q = 0; q < LPT; ++q) tile[g0 + G * q][p] = REG[q];                  \
    if (MORE) { SYMV_LOAD(REG, (SUB) + 2) }                                                        \
    __syncthreads();                                                                               \
    double rr[NR], ri[NR];                                                                         \
    _Pragma("unroll") for (int r = 0; r < NR; ++r) rr[r] = ri[r] = 0.0;                            \
    _Pragma("unroll") for (int u = 0; u < PPT; ++u) {                                              \
      const int pc = seg + TPR * u; /* neighbouring threads read neighbouring pairs */             \
      const Pair v = tile[rrow][pc];                                                               \
      _Pragma("unroll") for (int e = 0; e < 2; ++e) {                                              \
        double ar, ai;                                                                             \
        T::template entry<CONJ>(v, e, ar, ai);                                                     \
        _Pragma("unroll") for (int r = 0; r < NR; ++r) {                                           \
          T::mac(ar, ai, xs[1][r][e * (S / 2) + pc], rr[r], ri[r]);                                \
        }                                                                                          \
      }                                                                                            \
    }                                                                                              \
    _Pragma("unroll") for (int r = 0; r < NR; ++r) {                                               \
      rr[r] = sum_lanes<TPR>(rr[r]);                                                               \
      ri[r] = sum_lanes<TPR>(ri[r]);                                                               \
    }                                                                                              \
    if (seg == TPR - 4) {                                                                          \
      const int i = (SUB) * kRowsSub + rrow; /* x_P of these rows has been read */                 \
      _Pragma("unroll") for (int r = 0; r < NR; ++r) xs[0][r][i] = make_double2(rr[r], ri[r]);     \
    }                                                                                              \
  }
#pragma unroll 1
  for (int sub = 0; sub < NSUB - 2; sub += 2) {
    SYMV_CONSUME(ra, sub, true)
    SYMV_CONSUME(rb, sub + 1, true)
  }
  SYMV_CONSUME(ra, NSUB - 2, false)
  SYMV_CONSUME(rb, NSUB - 1, false)
#undef SYMV_CONSUME
#undef SYMV_MASK
#undef SYMV_LOAD

  // The row sums leave at the end: a store between the loads of a sub-tile
  // would have to be complete before later loads count as arrived.
  __syncthreads();
  for (int t = tid; t < S * NR; t += kThreads)
    part[(((long)P * nsb + Q) * NR + t / S) * S + t % S] = xs[0][t / S][t % S];
  if (!diag) {
    // reduce the transposed sums over the G row groups through LDS
    double2* red = reinterpret_cast<double2*>(&tile[0][0]);  // [G][S][NR]
    static_assert(sizeof(double2) * G * S * NR <= sizeof(Pair) * kRowsSub * tile_ld<S>(), "reduction fits the tile");
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int r = 0; r < NR; ++r) red[(g0 * S + 2 * p + e) * NR + r] = make_double2(cr[e][r], ci[e][r]);
    __syncthreads();
    for (int t = tid; t < S * NR; t += kThreads) {
      const int c = t % S, r = t / S;
      double sr = 0.0, si = 0.0;
      for (int g = 0; g < G; ++g) {
        const double2 v = red[(g * S + c) * NR + r];
        sr += v.x;
        si += v.y;
      }
      part[(((long)Q * nsb + P) * NR + r) * S + c] = make_double2(sr, si);
    }
  }
}

// Partial buffer layout: part[((K * nsb + L) * NR + r) * S + i], complex128.
// Job 0 has NR0 right-hand sides, job 1 NR1.
template <class T, int S, int NR0, int NR1, bool CONJ>
__global__ __launch_bounds__(kThreads) void k_symv(const JobsArg args) {
  typedef typename T::Pair Pair;
  constexpr int NRM = NR0 > NR1 ? NR0 : NR1;
  const int job = (int)blockIdx.x < args.nblk0 ? 0 : 1;
  const JobArg& ja = args.j[job];
  const int n = ja.n, nsb = ja.nsb;

  // block (P, Q), Q >= P, from the linear upper-triangle index
  int P = 0, rem = (int)blockIdx.x - (job ? args.nblk0 : 0);
  while (rem >= nsb - P) {
    rem -= nsb - P;
    ++P;
  }
  const int Q = P + rem;
  __shared__ Pair tile[rows_sub<S>()][tile_ld<S>()];
  __shared__ double2 xs[2][NRM][S];  // x_P (rows), x_Q (columns)
  const char* strip = static_cast<const char*>(ja.M) + (size_t)P * S * (size_t)ja.ldp * 16;
  const bool edge = (Q + 1) * S > n;  // else (P + 1) S <= n as well
  if (job == 0 || NR0 == NR1) {
    auto x0 = reinterpret_cast<double2(*)[NR0][S]>(&xs[0][0][0]);
    if (!edge)
      symv_block<T, S, NR0, CONJ, false>(strip, n, (int)ja.ldp, P, Q, ja.in, ja.part, nsb, tile, x0);
    else
      symv_block<T, S, NR0, CONJ, true>(strip, n, (int)ja.ldp, P, Q, ja.in, ja.part, nsb, tile, x0);
  } else {
    auto x1 = reinterpret_cast<double2(*)[NR1][S]>(&xs[0][0][0]);
    if (!edge)
      symv_block<T, S, NR1, CONJ, false>(strip, n, (int)ja.ldp, P, Q, ja.in, ja.part, nsb, tile, x1);
    else
      symv_block<T, S, NR1, CONJ, true>(strip, n, (int)ja.ldp, P, Q, ja.in, ja.part, nsb, tile, x1);
  }
}

// ---- three to eight right-hand sides: the FP64 matrix cores
//
// With several right-hand sides the vector form above is bound by its LDS
// reads of x (three 16-byte reads per right-hand side and matrix pair).  Here
// both sums of a block are products with a 16-column operand, 8 right-hand
// sides by (re, im), on v_mfma_f64_16x16x4, which adds its four terms to the
// accumulator as a chain of fused multiply-adds in the order k = 0..3.  Each
// chain of the vector form (a row group of a column, a thread's pairs of a
// row) is therefore kept as the K dimension of an accumulator of its own, and
// the chains meet in the same tree: a right-hand side has the same bits
// whichever others go with it.
//
// A workgroup of four waves owns a block.  It walks stages of 32 KB (32 rows at
// S = 128, 16 at S = 256), one in flight while the one before is in LDS: a wave
// loads its S / 4 columns (four rows a load, in operand order: lane l takes
// column pair l % 16 of row l / 16), takes the transposed sums M^T x_P straight
// from the registers (tiles of 16 columns by G row groups), and stores the stage
// to LDS, from where it forms four of the chains of 16 rows of M x_Q.  For
// complex64 K holds (im, re) of two entries; in the transposed sums an exchange
// between neighbouring rows of 16 lanes turns a load into the operands of its
// first and its last two rows.  x sits in LDS as [entry][right-hand side][re,
// im], the right-hand sides of an entry exchanged by its number, so that neither
// the stores nor the operand reads meet in a bank.
//
// Bound: with FP64 entries the stream (8 right-hand sides do 32 flops a byte
// at half the rate of the matrix cores), with complex64 the matrix cores,
// which do 8 columns' work for 5.  At n = 9216 with 8 right-hand sides FP64
// 100 us (two vector passes 210), with 4 90 us (102); complex64 with 7 135 us
// (two passes 175).  At n <= 2000, where a product is one block's latency,
// 4 right-hand sides 12-16 us (21-27), most of it the inputs, which are
// gathered for all columns at once.
constexpr int kMfmaNR = 8;  // right-hand sides per pass
// From three FP64 columns on one pass here is the faster one (n = 9216: 86 us
// to 95); a complex64 block needs two operands where FP64 needs one, so up to
// four columns the vector form is (n = 9216: 117 us to 140).
template <class T>
constexpr int kMfmaMinNR = T::kComplex ? 5 : 3;
template <int S>
struct MfmaLds {
  static constexpr int kRows = 4096 / S;  // rows per stage: 32 KB
  static constexpr int kQuads = S / 64;   // groups of four chains of a row
  struct Work {
    vf4 tile[kRows][S / 2 + 1];        // rows start 16 bytes apart in the banks
    double2 rowsum[kQuads][kRows][9];  // chains summed by fours
    double2 xp[kRows][kMfmaNR];        // x_P of a stage, grouped by row % G
    double2 xq[S][kMfmaNR];
  };
  union {
    Work wk;
    double2 col[S][9];  // transposed sums on their way out
  };
};

__device__ inline double xor_sign(double v, unsigned mask) {
  return __hiloint2double(__double2hiint(v) ^ (int)mask, __double2loint(v));
}

template <class T, int S, bool CONJ, bool EDGE>
__device__ void symv_block_mfma(const char* __restrict__ strip, int n, int ldp, int P, int Q, int nr,
                                const SymvInput& in, double2* __restrict__ part, int nsb, MfmaLds<S>& lds) {
  typedef typename T::Pair Pair;
  constexpr bool kComplex = T::kComplex;
  constexpr int kQuads = MfmaLds<S>::kQuads;
  constexpr int G = kThreads / (S / 2);          // row groups of the transposed sums
  constexpr int TPR = kThreads / rows_sub<S>();  // chains of a row
  constexpr int kRows = MfmaLds<S>::kRows;
  constexpr int ML = kRows / (4 * G);            // loads per row group, column pair and stage
  constexpr int NST = S / kRows;
  constexpr int NP = S / 128;                    // column pairs per lane
  constexpr int RT = kRows / 16;                 // row tiles per stage
  static_assert(ML == 2 && kQuads * RT == 4, "a wave forms four chains of 16 rows");
  static_assert(TPR == 4 * kQuads && S / 2 == 8 * TPR, "four chains of eight pairs a wave");
  const bool diag = (P == Q);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, k = lane >> 4;
  // row of a load's lane group: complex rows 1 and 2 change places for the
  // lane exchange
  const int kr = kComplex ? ((k & 1) << 1 | k >> 1) : k;

  const int gc = Q * S + 32 * NP * w + 2 * li;  // first pair; the second 32 columns on
  const unsigned ldb = (unsigned)ldp * 16u;
  Pair ra[G][ML][NP];
  auto load = [&](Pair(&reg)[G][ML][NP], int st) {
#pragma unroll
    for (int m = 0; m < ML; ++m)
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          const int lr = st * kRows + 4 * G * m + g + G * kr, c = gc + 32 * q;
          const unsigned row = EDGE ? (unsigned)min(lr, n - 1 - P * S) : (unsigned)lr;
          const unsigned off = row * ldb + (unsigned)((EDGE && c >= n ? 0 : c) >> 1) * 16u;
          reg[g][m][q] = __builtin_nontemporal_load(reinterpret_cast<const Pair*>(strip + off));
        }
  };
  auto mask = [&](Pair(&reg)[G][ML][NP], int st) {  // clears what lies beyond the matrix
#pragma unroll
    for (int m = 0; m < ML; ++m)
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          const int c = gc + 32 * q;
          const bool in = P * S + st * kRows + 4 * G * m + g + G * kr < n && c < n;
          const Pair v = in ? reg[g][m][q] : zero_pair<T>();
          reg[g][m][q] = c + 1 < n ? v : T::first_only(v);
        }
  };
  load(ra, 0);
  // x_Q goes to LDS whole; x_P stays with the thread of its row until the
  // stage before its own
  double2 xr[kMfmaNR];
  auto form = [&](int g) {
#pragma unroll
    for (int r0 = 0; r0 < kMfmaNR; r0 += 4) {
      double2 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = make_double2(0.0, 0.0);
      if ((!EDGE || g < n) && r0 < nr) input_entries(in, r0, nr, g, v);
#pragma unroll
      for (int u = 0; u < 4; ++u) xr[r0 + u] = v[u];
    }
  };
  auto put = [&](double2(*dst)[kMfmaNR], int slot) {
#pragma unroll
    for (int r = 0; r < kMfmaNR; ++r) dst[slot][r ^ (slot & 7)] = xr[r];
  };
  const int xi = tid % S;
  if (S == kThreads || tid >= S) {
    form(Q * S + xi);
    put(lds.wk.xq, xi);
  }
  if (S == kThreads || tid < S) form(P * S + xi);
  auto put_xp = [&](int st) {
    if (tid / kRows == st) put(lds.wk.xp, (xi % G) * (kRows / G) + (xi % kRows) / G);
  };
  put_xp(0);

  // operand columns: right-hand side li / 2, its re or im by li & 1; against
  // an imaginary part (complex, even k) the other part of x with its sign
  const bool im_k = kComplex && !(k & 1);
  const int rr = li >> 1, cc = im_k ? (li & 1) ^ 1 : li & 1;
  const unsigned sgn = im_k && (li & 1) == (CONJ ? 1 : 0) ? 0x80000000u : 0u;
  // the entry this lane holds of an operand of the transposed sums, ...
  const int kx = kComplex ? k >> 1 : k;
  const char* xp = reinterpret_cast<const char*>(&lds.wk.xp[kx][0]) + cc * 8;
  const int xp_rot = (rr ^ kx) << 4;
  // ... and of the rows (pair kp, column ke of it): the wave forms chains
  // 4 quad .. + 3 of rows 16 rt .. + 15
  const int quad = w / RT, rt = w % RT;
  const int ke = kComplex ? k >> 1 : k & 1, kp = kComplex ? 0 : k >> 1;
  const char* xq = reinterpret_cast<const char*>(&lds.wk.xq[2 * (4 * quad + TPR * kp) + ke][0]) + cc * 8;
  const int xq_rot = (rr ^ ke) << 4;
  const char* at = reinterpret_cast<const char*>(&lds.wk.tile[16 * rt + li][4 * quad + TPR * kp]) +
                   (kComplex ? (k ^ 1) * 4 : (k & 1) * 8);

  dbl4 col[G][2 * NP];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < 2 * NP; ++e) col[g][e] = dbl4{0.0, 0.0, 0.0, 0.0};
  __syncthreads();  // x ready

  constexpr int kH = kComplex ? 2 : 1;  // operands per load
  auto columns = [&](const Pair(&reg)[G][ML][NP]) {
    double b[ML][kH][G];
#pragma unroll
    for (int m = 0; m < ML; ++m)
#pragma unroll
      for (int h = 0; h < kH; ++h) {
        // slot of the lane's entry: a multiple of 8, + 4 m + 2 h + kx
        const char* xm = xp + (4 * m + 2 * h) * 128 + (xp_rot ^ ((4 * m + 2 * h) << 4));
#pragma unroll
        for (int g = 0; g < G; ++g) b[m][h][g] = *reinterpret_cast<const double*>(xm + g * (kRows / G) * 128);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < ML; ++m)
#pragma unroll
      for (int h = 0; h < kH; ++h)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int e = 0; e < 2 * NP; ++e)
            col[g][e] = __builtin_amdgcn_mfma_f64_16x16x4f64(T::col_operand(reg[g][m][e / 2], e & 1, h),
                                                             xor_sign(b[m][h][g], sgn), col[g][e], 0, 0, 0);
  };
  auto rows = [&]() {
    dbl4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = dbl4{0.0, 0.0, 0.0, 0.0};
    constexpr int kStep = kComplex ? 1 : 2;  // pairs of a chain per operand
    typename T::Row a[2][4];
    double b[2][4];
    auto operands = [&](int u) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        a[u & 1][j] = *reinterpret_cast<const typename T::Row*>(at + (TPR * kStep * u + j) * 16);
        b[u & 1][j] =
            *reinterpret_cast<const double*>(xq + 2 * (TPR * kStep * u + j) * 128 + (xq_rot ^ (2 * j << 4)));
      }
    };
    operands(0);
#pragma unroll
    for (int u = 0; u < 8 / kStep; ++u) {
      if (u + 1 < 8 / kStep) operands(u + 1);  // leave LDS while this step's products run
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[u & 1][j], xor_sign(b[u & 1][j], sgn), acc[j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    double* out = &lds.wk.rowsum[quad][16 * rt + k][0].x + li;
#pragma unroll
    for (int v = 0; v < 4; ++v) out[4 * v * 18] = (acc[0][v] + acc[1][v]) + (acc[2][v] + acc[3][v]);
  };
  // the sums of four chains meet across the waves: (Q1 + Q0), at S = 256
  // (Q3 + Q2) + (Q1 + Q0)
  auto finish_rows = [&](int st) {
    const int r = tid / kRows, i = tid % kRows;
    if (r >= nr) return;
    const double2 a0 = lds.wk.rowsum[0][i][r], a1 = lds.wk.rowsum[1][i][r];
    double2 t = make_double2(a1.x + a0.x, a1.y + a0.y);
    if (kQuads == 4) {
      const double2 a2 = lds.wk.rowsum[kQuads - 2][i][r], a3 = lds.wk.rowsum[kQuads - 1][i][r];
      t = make_double2((a3.x + a2.x) + t.x, (a3.y + a2.y) + t.y);
    }
    part[(((long)P * nsb + Q) * nr + r) * S + st * kRows + i] = t;
  };
  auto stage = [&](Pair(&reg)[G][ML][NP], int st, auto more) {
    if (EDGE) mask(reg, st);
    if (!diag) columns(reg);
    __syncthreads();  // the rows of the stage before are done with the tile, their sums are in LDS
#pragma unroll
    for (int m = 0; m < ML; ++m)
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int q = 0; q < NP; ++q)
          *reinterpret_cast<Pair*>(&lds.wk.tile[G * (4 * m + kr) + g][16 * (NP * w + q) + li]) = reg[g][m][q];
    if (more) load(reg, st + 1);
    put_xp(st + 1);
    if (st > 0) finish_rows(st - 1);
    __syncthreads();
    rows();
  };
#pragma unroll 1
  for (int st = 0; st < NST - 1; ++st) stage(ra, st, std::true_type());
  stage(ra, NST - 1, std::false_type());
  __syncthreads();
  finish_rows(NST - 1);
  if (diag) return;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 2 * NP; ++e)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double t = 0.0;
#pragma unroll
      for (int g = 0; g < G; ++g) t += col[g][e][v];
      (&lds.col[32 * (NP * w + e / 2) + 2 * (4 * v + k) + (e & 1)][0].x)[li] = t;
    }
  __syncthreads();
  for (int t = tid; t < S * nr; t += kThreads)
    part[(((long)Q * nsb + P) * nr + t / S) * S + t % S] = lds.col[t % S][t / S];
}

template <class T, int S, bool CONJ>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_symv_mfma(const JobsArg args) {
  const int job = (int)blockIdx.x < args.nblk0 ? 0 : 1;
  const JobArg& ja = args.j[job];
  const int n = ja.n, nsb = ja.nsb;
  int P = 0, rem = (int)blockIdx.x - (job ? args.nblk0 : 0);
  while (rem >= nsb - P) {
    rem -= nsb - P;
    ++P;
  }
  const int Q = P + rem;
  __shared__ MfmaLds<S> lds;
  const char* strip = static_cast<const char*>(ja.M) + (size_t)P * S * (size_t)ja.ldp * 16;
  if ((Q + 1) * S <= n)
    symv_block_mfma<T, S, CONJ, false>(strip, n, (int)ja.ldp, P, Q, args.nr, ja.in, ja.part, nsb, lds);
  else
    symv_block_mfma<T, S, CONJ, true>(strip, n, (int)ja.ldp, P, Q, args.nr, ja.in, ja.part, nsb, lds);
}

// y[r][K S + i] = sum over L (in order) of part[K][L][r][i].  Workgroup
// (K, r): eight threads per row each add an eighth of the slots (all loads
// issued before the adds, so they overlap), then the eighths are added in
// order through LDS.  Blocks [0, nsb0) of the grid reduce job 0, the rest
// job 1.
template <int S>
constexpr int red_parts() { return 1024 / S; }
template <int S>
__global__ __launch_bounds__(1024) void k_symv_reduce(const JobsArg args) {
  constexpr int kRedParts = red_parts<S>();
  __shared__ double2 q8[kRedParts][S];
  const int job = (int)blockIdx.x < args.nsb0 ? 0 : 1;
  const JobArg& ja = args.j[job];
  const int n = ja.n, nsb = ja.nsb;
  const int NR = job ? args.nr1 : args.nr;
  const int K = (int)blockIdx.x - (job ? args.nsb0 : 0), r = blockIdx.y;
  if (r >= NR) return;
  const int i = threadIdx.x % S, qt = threadIdx.x / S;
  const int per = (nsb + kRedParts - 1) / kRedParts;
  const int L0 = qt * per;
  const double2* src = ja.part + (((long)K * nsb) * NR + r) * S + i;
  double sr = 0.0, si = 0.0;
  for (int b0 = 0; b0 < per; b0 += 8) {
    double2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int L = L0 + b0 + u;
      v[u] = (b0 + u < per && L < nsb) ? src[(long)L * NR * S] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      sr += v[u].x;
      si += v[u].y;
    }
  }
  q8[qt][i] = make_double2(sr, si);
  __syncthreads();
  const int row = K * S + i;
  if (qt == 0 && row < n) {
    double2 t = q8[0][i];
    for (int u = 1; u < kRedParts; ++u) {
      t.x += q8[u][i].x;
      t.y += q8[u][i].y;
    }
    ja.y[(long)r * n + row] = t;
  }
}

constexpr int kSmax = 256, kSmin = 128;

// The product kernel is timed under `tag` (one right-hand side) or
// "<tag>_nr<k>" (k right-hand sides), the slot sums under "symv_reduce".
template <int S, class F>
void launch(const JobsArg& a, int nsbsum, hipStream_t s, const char* tag, F product) {
  {
    ProfScope prof(a.nr == 1 ? tag : profile_tag_suffix(tag, a.nr), s);
    product();
  }
  ProfScope prof("symv_reduce", s);
  hipLaunchKernelGGL(k_symv_reduce<S>, dim3((unsigned)nsbsum, (unsigned)a.nr), dim3(1024), 0, s, a);
}
template <class T, int S, int NR0, int NR1, bool CONJ>
void launch_vec(const JobsArg& a, int nblk, hipStream_t s) {
  hipLaunchKernelGGL((k_symv<T, S, NR0, NR1, CONJ>), dim3((unsigned)nblk), dim3(kThreads), 0, s, a);
}
template <class T, int S, bool CONJ>
void launch_any(const JobsArg& a, int nblk, int nsbsum, hipStream_t s, const char* tag) {
  launch<S>(a, nsbsum, s, tag, [&] {
    if (a.nr >= kMfmaMinNR<T>) {
      hipLaunchKernelGGL((k_symv_mfma<T, S, CONJ>), dim3((unsigned)nblk), dim3(kThreads), 0, s, a);
    } else if (a.nr == 1) {
      launch_vec<T, S, 1, 1, CONJ>(a, nblk, s);
    } else if (a.nr == 2) {
      if (a.nr1 == 1)
        launch_vec<T, S, 2, 1, CONJ>(a, nblk, s);
      else
        launch_vec<T, S, 2, 2, CONJ>(a, nblk, s);
    } else if constexpr (T::kComplex) {
      if (a.nr == 3)
        launch_vec<T, S, 3, 3, CONJ>(a, nblk, s);
      else
        launch_vec<T, S, 4, 4, CONJ>(a, nblk, s);
    }
  });
}

// Block size: 256 x 256 blocks (longer streams per workgroup, fewer slots)
// once they still give the grid a few hundred workgroups, else 128 x 128.
constexpr int kMinBlocks256 = 400;
long blocks_of(int64_t n, int S) {
  const long nb = (n + S - 1) / S;
  return nb * (nb + 1) / 2;
}
size_t part_bytes(int64_t n, int nr, int S) {
  const int64_t nsb = (n + S - 1) / S;
  return sizeof(double2) * (size_t)(nsb * nsb * nr * S);
}

// Advance every source pointer of an input by r0 right-hand sides.
SymvInput shift_input(SymvInput in, int r0) {
  for (int q = 0; q < 4; ++q)
    if (in.p[q]) in.p[q] += (long)r0 * in.stride[q];
  return in;
}

template <class T, bool CONJ>
rfcmp_status symv_any(const SymvJob* jobs, int njobs, int nrhs, void* scratch, size_t scratch_bytes,
                      hipStream_t s, const char* tag) {
  if (njobs < 1 || njobs > 2) {
    set_error("symv: %d jobs (1 or 2 allowed)", njobs);
    return RFCMP_E_ARG;
  }
  if (nrhs <= 0) return RFCMP_OK;
  // right-hand sides of each job: nrhs, or 1 of 2 for job 1 (a product riding
  // along with fewer columns)
  int jn[2] = {nrhs, nrhs};
  if (njobs == 2 && jobs[1].nrhs > 0 && jobs[1].nrhs < nrhs) {
    if (!(nrhs == 2 && jobs[1].nrhs == 1)) {
      set_error("symv: job 1 with %d of %d right-hand sides is not supported", jobs[1].nrhs, nrhs);
      return RFCMP_E_ARG;
    }
    jn[1] = jobs[1].nrhs;
  }
  long blocks_big = 0;
  for (int q = 0; q < njobs; ++q) {
    if (jobs[q].n <= 0 || jobs[q].ld % 2 != 0 || jobs[q].ld < jobs[q].n) {
      set_error("symv: job %d has n = %lld, ld = %lld", q, (long long)jobs[q].n, (long long)jobs[q].ld);
      return RFCMP_E_ARG;
    }
    blocks_big += blocks_of(jobs[q].n, kSmax);
  }
  const int S = blocks_big >= kMinBlocks256 ? kSmax : kSmin;
  // right-hand sides per pass: what the scratch holds, at least 4 (their
  // sums do not depend on it)
  auto need = [&](int per) {
    size_t b = 0;
    for (int q = 0; q < njobs; ++q) b += part_bytes(jobs[q].n, std::min(jn[q], per), S);
    return b;
  };
  int per = kMfmaNR;
  while (per > 4 && need(per) > scratch_bytes) --per;
  if (need(per) > scratch_bytes) {
    set_error("symv: needs %zu bytes of scratch, %zu given", need(per), scratch_bytes);
    return RFCMP_E_ARG;
  }
  for (int r0 = 0, nr = 0; r0 < nrhs; r0 += nr) {
    nr = std::min(per, nrhs - r0);
    const bool split = jn[1] != nrhs;  // job 1: one column (nr == 2 here)
    JobsArg a{};
    a.nr = nr;
    a.nr1 = split ? 1 : nr;
    char* sp = static_cast<char*>(scratch);
    int nblk = 0, nsbsum = 0;
    for (int q = 0; q < njobs; ++q) {
      const SymvJob& jb = jobs[q];
      JobArg& ja = a.j[q];
      ja.M = jb.M;
      ja.n = (int)jb.n;
      ja.ldp = (long)(jb.ld / 2);
      ja.nsb = int((jb.n + S - 1) / S);
      ja.in = shift_input(jb.in, r0);
      ja.part = reinterpret_cast<double2*>(sp);
      ja.y = jb.y + (long)r0 * jb.n;
      sp += part_bytes(jb.n, q == 1 ? a.nr1 : nr, S);
      if (q == 0) {
        a.nblk0 = ja.nsb * (ja.nsb + 1) / 2;
        a.nsb0 = ja.nsb;
      }
      nblk += ja.nsb * (ja.nsb + 1) / 2;
      nsbsum += ja.nsb;
    }
    if (S == kSmax)
      launch_any<T, kSmax, CONJ>(a, nblk, nsbsum, s, tag);
    else
      launch_any<T, kSmin, CONJ>(a, nblk, nsbsum, s, tag);
  }
  RF_HIP(hipGetLastError());
  return RFCMP_OK;
}

}  // namespace

size_t symv_scratch_bytes(int64_t n, int nrhs) {
  // the smaller block size needs the most slots; a matrix that fills the chip
  // with the larger one alone never takes it
  return part_bytes(n, std::min(std::max(nrhs, 1), kMfmaNR), blocks_of(n, kSmax) >= kMinBlocks256 ? kSmax : kSmin);
}

rfcmp_status symv_form_input(const SymvInput& in, int64_t n, int nrhs, double2* out, hipStream_t s) {
  if (n <= 0 || nrhs <= 0) return RFCMP_OK;
  hipLaunchKernelGGL(k_form_input, dim3((unsigned)((n + 255) / 256), nrhs), dim3(256), 0, s, in, (int)n, out);
  RF_HIP(hipGetLastError());
  return RFCMP_OK;
}

rfcmp_status csymv_jobs(const SymvJob* jobs, int njobs, bool conj, int nrhs, void* scratch, size_t scratch_bytes,
                        hipStream_t s, const char* tag) {
  if (conj) return symv_any<C64, true>(jobs, njobs, nrhs, scratch, scratch_bytes, s, tag);
  return symv_any<C64, false>(jobs, njobs, nrhs, scratch, scratch_bytes, s, tag);
}

rfcmp_status dsymv_jobs(const SymvJob* jobs, int njobs, int nrhs, void* scratch, size_t scratch_bytes,
                        hipStream_t s, const char* tag) {
  return symv_any<F64, false>(jobs, njobs, nrhs, scratch, scratch_bytes, s, tag);
}

rfcmp_status csymv(const float2* M, int64_t n, int64_t ld, bool conj, const double2* x, double2* y, int nrhs,
                   void* scratch, size_t scratch_bytes, hipStream_t s, const char* tag) {
  SymvJob j;
  j.M = M;
  j.n = n;
  j.ld = ld;
  j.in.p[0] = x;
  j.in.stride[0] = n;
  j.y = y;
  return csymv_jobs(&j, 1, conj, nrhs, scratch, scratch_bytes, s, tag);
}

rfcmp_status dsymv(const double* M, int64_t n, int64_t ld, const double2* x, double2* y, int nrhs,
                   void* scratch, size_t scratch_bytes, hipStream_t s, const char* tag) {
  SymvJob j;
  j.M = M;
  j.n = n;
  j.ld = ld;
  j.in.p[0] = x;
  j.in.stride[0] = n;
  j.y = y;
  return dsymv_jobs(&j, 1, nrhs, scratch, scratch_bytes, s, tag);
}

}  // namespace rfcmp
