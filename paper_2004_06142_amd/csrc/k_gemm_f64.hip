// Float64 matrix-core (v_mfma_f64_16x16x4) products, and the three-index contractions in float64 and float32.
//
// The products: block tile 64 x 64 x 16, 256 threads = 4 waves in a 2 x 2 arrangement, each wave owning a
// 32 x 32 sub-tile = 2 x 2 MFMA blocks of 16 x 16.  Operands are staged through LDS stored
// k-major ([k][m] and [k][n]), which is the order in which the f64 MFMA consumes them (lane l
// supplies A[m = l%16][k = l/16] and B[k = l/16][n = l%16]; the result element (l/16 + 4*j, l%16)
// sits in component j of lane l).  Register prefetch of the next k-slab overlaps global loads
// with the matrix-core work.
#include <type_traits>

#include "common.h"
#include "f64_tile.h"

namespace pnof {
namespace {

using namespace f64t;

template <bool AM, bool BN>
__global__ __launch_bounds__(256) void gemm_f64_kernel(int M, int N, int K, double alpha,
                                                       const double* __restrict__ A, long long sam,
                                                       long long sak, long long sab,
                                                       const double* __restrict__ B, long long sbk,
                                                       long long sbn, long long sbb, double beta,
                                                       double* __restrict__ C, long long scm,
                                                       long long scn, long long scb) {
  __shared__ F64Smem sm;
  const int tiles_n = (N + TN - 1) / TN;
  const int m0 = (blockIdx.x / tiles_n) * TM, n0 = (blockIdx.x % tiles_n) * TN;
  const long long b = blockIdx.y;
  f64x4 acc[2][2];
  zero_acc(acc);
  tile_f64<AM, BN>(sm, A + b * sab, sam, sak, B + b * sbb, sbk, sbn, M, N, 0, K, m0, n0, acc);
  double* Cb = C + b * scb;
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int m = m0 + acc_row(mi, j), n = n0 + acc_col(ni);
        if (m < M && n < N) {
          double* c = Cb + (long long)m * scm + (long long)n * scn;
          *c = alpha * acc[mi][ni][j] + (beta != 0.0 ? beta * *c : 0.0);
        }
      }
}

// Single products (the step's float64 products: H C_A, lambda = C^T Y, J = D^T D, Q Z and C U) on a
// finer grid: block tile 64 x 32 (4 waves of 32 x 16, each two 16 x 16 MFMA blocks), so that a
// 1200 x 1200 product makes 722 blocks, about 2.8 per compute unit, where 64 x 64 tiles made 361,
// about 1.4, and the units holding two of them set the time.  k-slabs of 16 go through two LDS
// stages, loaded into registers two slabs ahead of their multiplication; one barrier per slab
// separates the writes of one stage from the reads of the other (1200^3: 94-101 us, against
// 103-113 us with slabs of 32 one ahead and 117-130 us with 64 x 64 tiles).
// KG groups of 4 waves share a tile's slabs between them (their sums are added in LDS, in order): a slab takes a
// block about 0.8 us, most of it waiting for its loads, so a product whose tiles do not fill the chip is bound by
// the length of k (gemm_f64_groups; with 4 groups J of 300 orbitals over 2000 rows 109 -> 65 us, lambda of 500
// functions 33 -> 20; at 24 functions, whose five products have two slabs, one group each).
template <bool AM, bool BN, int KG>
__global__ __launch_bounds__(256 * KG, KG == 1 ? 3 : 1) void gemm_f64_wide_kernel(int M, int N, int K, double alpha,
                                                              const double* __restrict__ A, long long sam,
                                                              long long sak, const double* __restrict__ B,
                                                              long long sbk, long long sbn, double beta,
                                                              double* __restrict__ C, long long scm, long long scn) {
  using namespace wide;
  __shared__ Smem sm[KG];
  const int tn_n = (N + BNT - 1) / BNT, grp = KG == 1 ? 0 : threadIdx.x >> 8;
  const int m0 = (blockIdx.x / tn_n) * BM, n0 = (blockIdx.x % tn_n) * BNT;
  const int ns = ((K + BK - 1) / BK + KG - 1) / KG;
  f64x4 acc[2];
  wide_tile<AM, BN>(sm[grp], A, sam, sak, B, sbk, sbn, M, N, K, grp * ns * BK, ns, m0, n0, acc);
  if constexpr (KG > 1) {
    static_assert(sizeof(Smem) >= 256 * 8 * sizeof(double), "a group's sums in its stages");
    double* own = reinterpret_cast<double*>(&sm[grp]) + (threadIdx.x & 255);
    if (grp > 0)
#pragma unroll
      for (int e = 0; e < 8; ++e) own[256 * e] = acc[e >> 2][e & 3];
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g = 1; g < KG; ++g)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e >> 2][e & 3] += reinterpret_cast<const double*>(&sm[g])[threadIdx.x + 256 * e];
  }
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = m0 + wide_row(mi, j), n = n0 + wide_col();
      if (m < M && n < N) {
        double* c = C + (long long)m * scm + (long long)n * scn;
        *c = alpha * acc[mi][j] + (beta != 0.0 ? beta * *c : 0.0);
      }
    }
}
// Groups for a product: 4 while its tiles make one block per compute unit, 2 while they make two, if each group
// has at least two slabs.
int gemm_f64_groups(int M, int N, int K) {
  const long long tiles = (long long)cdiv(M, wide::BM) * cdiv(N, wide::BNT);
  const int ns = cdiv(K, wide::BK);
  return tiles <= 256 && ns >= 8 ? 4 : tiles <= 512 && ns >= 4 ? 2 : 1;
}

// One product of a grouped launch per blockIdx.y; blocks beyond that product's tiles exit.
template <bool AM, bool BN>
__global__ __launch_bounds__(256) void gemm_f64_grouped_kernel(const F64Gemm* __restrict__ tab) {
  __shared__ F64Smem sm;
  grouped_tile<AM, BN>(tab[blockIdx.y], blockIdx.x, sm);
}

// Split-K form for products with few output tiles: block (tile, s) sums k in the s-th of ks equal
// ranges and writes its partial to slab s of Cpart (ks dense M x N slabs, row-major).  The caller
// adds the slabs in slab order, so the result does not depend on the schedule.
template <bool AM, bool BN>
__global__ __launch_bounds__(256) void gemm_f64_splitk_kernel(int M, int N, int K, int ks, const double* __restrict__ A,
                                                              long long sam, long long sak,
                                                              const double* __restrict__ B, long long sbk,
                                                              long long sbn, double* __restrict__ Cpart) {
  __shared__ F64Smem sm;
  const int tiles_n = (N + TN - 1) / TN;
  const int tile = blockIdx.x / ks, sidx = blockIdx.x % ks;
  const int m0 = (tile / tiles_n) * TM, n0 = (tile % tiles_n) * TN;
  const int kb = (int)((long long)K * sidx / ks), ke = (int)((long long)K * (sidx + 1) / ks);
  f64x4 acc[2][2];
  zero_acc(acc);
  tile_f64<AM, BN>(sm, A, sam, sak, B, sbk, sbn, M, N, kb, ke, m0, n0, acc);
  double* Cs = Cpart + (long long)sidx * M * N;
#pragma unroll
  for (int mi = 0; mi < 2; ++mi)
#pragma unroll
    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int m = m0 + acc_row(mi, j), n = n0 + acc_col(ni);
        if (m < M && n < N) Cs[(long long)m * N + n] = acc[mi][ni][j];
      }
}

// ------------------------------------------------------------------------------------------------
// The three-index contractions in float64 (v_mfma_f64_16x16x4) and float32 (v_mfma_f32_16x16x4f32).
//
// Block tile BM x BN, 256 threads = 4 waves in 2 x 2, k-slabs of 16.  The next slab travels in registers
// while the current one is multiplied from LDS (two stages, one barrier per slab); a block's slabs run on
// over all its P, so the pipeline is filled once.  An operand slab is "row" (rows of the output index,
// contiguous in k) or "col" (rows of k, contiguous in the output index):
//   row  LDS [r][16], 16-byte chunks swizzled so that the fragment reads of 16 rows meet distinct banks;
//   col  LDS [k][R + pad].
// Rows past the operand's end repeat its last row and columns past it read what follows in the row (both
// only reach output elements that are not stored); past the end of k the loaders put zeros.
// Sums run over k in ascending slabs; within a slab float32 takes k = 4 s + lane / 16 in step s (the order
// of its rounding is part of the results), float64 k = 8 h + 2 (lane / 16) + s, so that a lane's two
// values of a row operand are one 16-byte read.
// What bounds them: the matrix cores (64 cycles a float64 product, 32 a float32 one), once the address
// arithmetic is out of the loop.  500 functions, 300 active, 2000 rows of bf16 B in float64: X 7.08 + 1.22 ms
// (B widened to float64 in a pass of its own), b 5.22, Y 4.68 ms with 64 x 64 tiles and strided element
// loads; X 5.57, b 2.67, Y 4.1 ms here (X 73 % of the card's float64 matrix rate).  301 functions, 170 active,
// 1200 rows in float32: X 1.00 -> 0.51, b 0.79 -> 0.38, Y 0.43 -> 0.44 ms.
typedef double f64x2 __attribute__((ext_vector_type(2)));
constexpr int SK = 16;   // k per slab

template <typename T>
struct Fp;
template <>
struct Fp<double> {
  typedef f64x4 acc;
  static constexpr int CH = 2;   // elements of a 16-byte chunk
  static __device__ __forceinline__ acc mma(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  static __device__ __forceinline__ int row(int j) { return ((threadIdx.x & 63) >> 4) + 4 * j; }
  static __device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }
  static constexpr int pad = 8;
};
template <>
struct Fp<float> {
  typedef f32x4 acc;
  static constexpr int CH = 4;
  static __device__ __forceinline__ acc mma(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  static __device__ __forceinline__ int row(int j) { return 4 * ((threadIdx.x & 63) >> 4) + j; }
  static __device__ __forceinline__ int swz(int r) { return (r >> 2) & 3; }
  static constexpr int pad = 16;
};

template <typename T>
__device__ __forceinline__ T fp_from(double v) { return (T)v; }
template <typename T>
__device__ __forceinline__ T fp_from(float v) { return (T)v; }
template <typename T>
__device__ __forceinline__ T fp_from(u16 v) { return (T)bf16_bits_to_f32(v); }

// One thread's share of a slab of R rows (R = 64 or 128): NC pieces of E elements, contiguous in k ("row") or in
// the output index ("col").  Pieces are 16 bytes (bf16: 8 elements, the two halves of a slab's row), dealt so
// that neighbouring threads take neighbouring pieces, in memory and in LDS.
template <typename S, int R>
struct FpPart {
  static constexpr int E = sizeof(S) == 8 ? 2 : sizeof(S) == 4 ? 4 : 8, NC = R * SK / E / 256;
  static_assert(NC >= 1, "whole pieces per thread");
  S v[NC][E];
};
// Byte offsets of a thread's pieces from the slab's first element (row: element (r0, k0); col: row k0 of
// the storage), the same for every slab, so that the loop advances one uniform pointer.  Rows are clamped to
// the last valid one (row), columns to the last whole piece of the storage row (col).
template <bool COL, typename S, int R, int NC>
__device__ __forceinline__ void fp_offsets(unsigned (&off)[NC], long long ld, int nrows, int r0) {
  constexpr int E = FpPart<S, R>::E, PR = (COL ? R : SK) / E;
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int q = t / PR + i * (256 / PR);   // row, or k
    if constexpr (COL) off[i] = (unsigned)((q * ld + min(r0 + (t % PR) * E, (int)ld - E)) * sizeof(S));
    else off[i] = (unsigned)((min(q, nrows - 1 - r0) * ld + (t % PR) * E) * sizeof(S));
  }
}
// slab: its first element (see fp_offsets); kleft: values of k from there on
template <bool COL, typename S, int R, int NC>
__device__ __forceinline__ void fp_load(FpPart<S, R>& p, const S* __restrict__ slab, const unsigned (&off)[NC], int kleft) {
  constexpr int E = FpPart<S, R>::E, PR = (COL ? R : SK) / E;
  const char* __restrict__ base = reinterpret_cast<const char*>(slab);
  if (kleft >= SK) {
#pragma unroll
    for (int i = 0; i < NC; ++i) __builtin_memcpy(p.v[i], base + off[i], 16);
    return;
  }
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const S* __restrict__ src = reinterpret_cast<const S*>(base + off[i]);
#pragma unroll
    for (int e = 0; e < E; ++e) p.v[i][e] = (COL ? t / PR + i * (256 / PR) : (t % PR) * E + e) < kleft ? src[e] : S(0);
  }
}
template <typename T, int R>
struct FpSlab {   // LDS of one stage of one operand, either layout
  static constexpr int PITCH = R + Fp<T>::pad;
  static constexpr int SIZE = R * SK > SK * PITCH ? R * SK : SK * PITCH;
  __align__(16) T v[SIZE];
};
template <bool COL, typename T, typename S, int R>
__device__ __forceinline__ void fp_store(FpSlab<T, R>& sm, const FpPart<S, R>& p) {
  constexpr int E = FpPart<S, R>::E, NC = FpPart<S, R>::NC, CH = Fp<T>::CH, PR = (COL ? R : SK) / E;
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    T x[E];
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = fp_from<T>(p.v[i][e]);
    const int q = t / PR + i * (256 / PR), c0 = (t % PR) * E;   // row and k of the piece, or k and column
    if constexpr (E < CH) {   // float64 elements rounded to float: half a chunk
      static_assert(!COL, "B of the float32 X");
      __builtin_memcpy(__builtin_assume_aligned(sm.v + q * SK + ((c0 / CH) ^ Fp<T>::swz(q)) * CH + c0 % CH, E * sizeof(T)), x,
                       E * sizeof(T));
    } else {
#pragma unroll
      for (int c = 0; c < E / CH; ++c) {
        T* dst = COL ? sm.v + q * FpSlab<T, R>::PITCH + c0 + c * CH : sm.v + q * SK + ((c0 / CH + c) ^ Fp<T>::swz(q)) * CH;
        __builtin_memcpy(__builtin_assume_aligned(dst, 16), x + c * CH, 16);
      }
    }
  }
}
// The four k-steps of a slab for the 16 rows starting at r: f[s] is this lane's element of step s.
template <typename T, int R>
__device__ __forceinline__ void fp_frag(const FpSlab<T, R>& sm, bool col, int r, T (&f)[4]) {
  const int lane = threadIdx.x & 63, g = lane >> 4, rr = r + (lane & 15);
  constexpr int CH = Fp<T>::CH, PITCH = FpSlab<T, R>::PITCH;
  if (!col) {
    if constexpr (CH == 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f64x2 x = *reinterpret_cast<const f64x2*>(sm.v + rr * SK + ((4 * h + g) ^ Fp<T>::swz(rr)) * CH);
        f[2 * h] = x.x;
        f[2 * h + 1] = x.y;
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) f[s] = sm.v[rr * SK + ((s ^ Fp<T>::swz(rr)) * CH) + g];
    }
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s) f[s] = sm.v[(CH == 2 ? 8 * (s >> 1) + 2 * g + (s & 1) : 4 * s + g) * PITCH + rr];
  }
}

// The block's main loop: segments seg = 0 .. nseg-1 of K each.  A(seg) / B(seg): base pointers of the operands
// (uniform); with MIXED the view of B changes from slab to slab (col where bcol(k0)), otherwise it is row.
// epi(seg, acc) at the end of each segment, acc cleared after it when RESET.
template <typename T, typename SB, int BM, int BN, bool ACOL, bool MIXED, bool RESET, typename FA, typename FB, typename FC,
          typename EPI>
__device__ __forceinline__ void fp_mainloop(FpSlab<T, BM> (&sa)[2], FpSlab<T, BN> (&sb)[2], int nseg, int K, FA A,
                                            long long lda, int arows, int m0, FB B, long long ldb, int brows, int n0, FC bcol,
                                            typename Fp<T>::acc (&acc)[BM / 32][BN / 32], EPI epi) {
  constexpr int MI = BM / 32, NI = BN / 32;
  const int wave = threadIdx.x >> 6, wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
  const int ns = (K + SK - 1) / SK, total = nseg * ns;
  if (total <= 0) return;
  FpPart<T, BM> pa;
  FpPart<SB, BN> pb;
  unsigned oa[FpPart<T, BM>::NC], ob[FpPart<SB, BN>::NC], oc[FpPart<SB, BN>::NC];
  fp_offsets<ACOL, T, BM>(oa, lda, arows, m0);
  fp_offsets<false, SB, BN>(ob, ldb, brows, n0);
  if constexpr (MIXED) fp_offsets<true, SB, BN>(oc, ldb, brows, n0);
  const long long a0 = ACOL ? 0 : (long long)m0 * lda, b0 = (long long)n0 * ldb;
  int lseg = 0, lk = 0;
  auto load = [&]() {
    fp_load<ACOL>(pa, A(lseg) + (ACOL ? lk * lda : a0 + lk), oa, K - lk);
    if constexpr (MIXED)
      if (bcol(lk)) {
        fp_load<true>(pb, B(lseg) + lk * ldb, oc, K - lk);
        return;
      }
    fp_load<false>(pb, B(lseg) + b0 + lk, ob, K - lk);
  };
  auto store = [&](int st, int k0) {
    fp_store<ACOL>(sa[st], pa);
    if constexpr (MIXED)
      if (bcol(k0)) {
        fp_store<true>(sb[st], pb);
        return;
      }
    fp_store<false>(sb[st], pb);
  };
  auto advance = [&]() {
    lk += SK;
    if (lk >= K) {
      lk = 0;
      ++lseg;
    }
  };
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = typename Fp<T>::acc{0, 0, 0, 0};
  };
  load();
  store(0, lk);
  advance();
  if (total > 1) load();
  clear();
  __syncthreads();
  int it = 0;
  for (int seg = 0; seg < nseg; ++seg) {
    for (int k0 = 0; k0 < K; k0 += SK, ++it) {
      const int st = it & 1;
      if (it + 1 < total) {   // slab it + 1 to the other stage, slab it + 2 on its way
        store(st ^ 1, lk);
        advance();
        if (it + 2 < total) load();
      }
      T fa[MI][4], fb[NI][4];
#pragma unroll
      for (int i = 0; i < MI; ++i) fp_frag(sa[st], ACOL, wm + 16 * i, fa[i]);
      const bool bc = MIXED && bcol(k0);
#pragma unroll
      for (int j = 0; j < NI; ++j) fp_frag(sb[st], bc, wn + 16 * j, fb[j]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = Fp<T>::mma(fa[i][s], fb[j][s], acc[i][j]);
      __syncthreads();
    }
    epi(seg, acc);
    if (RESET) clear();
  }
}
template <int BM>
__device__ __forceinline__ int fp_row0(int i) { return (threadIdx.x >> 7) * (BM / 2) + 16 * i; }
template <int BN>
__device__ __forceinline__ int fp_col(int j) { return ((threadIdx.x >> 6) & 1) * (BN / 2) + 16 * j + (threadIdx.x & 15); }

// Lower-triangle tile index t -> (tm, tn) with tn <= tm.
__device__ __forceinline__ void tri_tile(int t, int& tm, int& tn) {
  int r = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
  while ((r + 1) * (r + 2) / 2 <= t) ++r;
  while (r * (r + 1) / 2 > t) --r;
  tm = r;
  tn = t - r * (r + 1) / 2;
}
constexpr int XM = 64;             // X: active orbitals x 128 or 64 stacked rows (P, mu)
constexpr int BT = 64;             // b: square tiles on and below the diagonal
constexpr int YN = 64;             // Y: 128 or 64 mu x 64 active orbitals

// gemm1: XT[P][p][mu] = sum_nu Ct[p][nu] B_P[mu][nu] over the stacked rows (P, mu) of the chunk, B read as
// stored (bf16 or float64) and rounded to T.
template <typename T, typename SB, int XN>
__global__ __launch_bounds__(256, 3) void df_x_kernel(int nbf, int nact, int np, const T* __restrict__ Ct, int ldk,
                                                   const SB* __restrict__ Bc, T* __restrict__ XT, int ldx) {
  __shared__ FpSlab<T, XM> sa[2];
  __shared__ FpSlab<T, XN> sb[2];
  const int nrows = np * nbf, tm_n = (nact + XM - 1) / XM;
  const int w = xcd_item(tm_n * ((nrows + XN - 1) / XN));
  if (w < 0) return;
  const int m0 = (w % tm_n) * XM, n0 = (w / tm_n) * XN;
  typename Fp<T>::acc acc[XM / 32][XN / 32];
  auto A = [&](int) { return Ct; };
  auto B = [&](int) { return Bc; };
  auto bcol = [](int) { return false; };
  auto epi = [&](int, typename Fp<T>::acc(&a)[XM / 32][XN / 32]) {
#pragma unroll
    for (int j = 0; j < XN / 32; ++j) {
      const int c = n0 + fp_col<XN>(j);
      if (c >= nrows) continue;
      const int P = c / nbf, mu = c - P * nbf;
      T* X = XT + (long long)P * nact * ldx;
#pragma unroll
      for (int i = 0; i < XM / 32; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int p = m0 + fp_row0<XM>(i) + Fp<T>::row(q);
          if (p >= nact) continue;
          X[(long long)p * ldx + mu] = a[i][j][q];
        }
    }
  };
  fp_mainloop<T, SB, XM, XN, false, false, false>(sa, sb, 1, nbf, A, ldk, nact, m0, B, nbf, nrows, n0, bcol, acc, epi);
}

// gemm2: b_P = Ct XT_P^T on the tiles on and below the diagonal, P in the block's split; K partials (float64
// sums of b^2; added to Kpart, or stored with kset), D, and W = b o beta: a tile below the diagonal is
// stored once, W[p][q] with p the larger block, a diagonal tile in full (its upper half mirrored from the
// lower).
template <typename T>
__global__ __launch_bounds__(256, 3) void df_b_kernel(int nbf, int nact, int np, int nsplit, const T* __restrict__ Ct, int ldk,
                                                   const T* __restrict__ XT, int ldx, const T* __restrict__ beta, int ldbeta,
                                                   double* __restrict__ Kpart, int kset, double* __restrict__ Dc,
                                                   T* __restrict__ W, int ldw) {
  __shared__ FpSlab<T, BT> sa[2], sb[2];
  const int t = (nact + BT - 1) / BT, ntri = t * (t + 1) / 2;
  const int w = xcd_item(ntri * nsplit);
  if (w < 0) return;
  int tm, tn;
  tri_tile(w % ntri, tm, tn);
  const int m0 = tm * BT, n0 = tn * BT, s = w / ntri;
  const int pb = (int)((long long)np * s / nsplit), pe = (int)((long long)np * (s + 1) / nsplit);
  typename Fp<T>::acc acc[2][2];
  f64x4 kacc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) kacc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  auto A = [&](int) { return Ct; };
  auto B = [&](int seg) { return XT + (long long)(pb + seg) * nact * ldx; };
  auto bcol = [](int) { return false; };
  const int p0 = m0 + fp_row0<BT>(0), q0 = n0 + fp_col<BT>(0);
  auto epi = [&](int seg, typename Fp<T>::acc(&a)[2][2]) {
    const long long P = pb + seg;
    T* Wp = W + P * nact * ldw;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int p = p0 + 16 * i + Fp<T>::row(e);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int q = q0 + 16 * j;
          const T b = a[i][j][e];
          kacc[i][j][e] += (double)b * (double)b;
          if (p < nact && q <= p) {
            const T wv = b * beta[p * ldbeta + q];
            Wp[p * ldw + q] = wv;
            if (tm == tn) {
              Wp[q * ldw + p] = wv;
              if (p == q) Dc[P * nact + p] = (double)b;
            }
          }
        }
      }
  };
  fp_mainloop<T, T, BT, BT, false, false, true>(sa, sb, pe - pb, nbf, A, ldk, nact, m0, B, ldx, nact, n0, bcol, acc, epi);
  double* Kp = Kpart + (long long)s * nact * nact;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int p = m0 + fp_row0<BT>(i) + Fp<T>::row(e), q = n0 + fp_col<BT>(j);
        if (p < nact && q <= p) {
          double* k = Kp + (long long)p * nact + q;
          *k = kset ? kacc[i][j][e] : *k + kacc[i][j][e];
        }
      }
}

// gemm3: Ypart[s][mu][q] = sum_{P in split s} sum_r XT_P[r][mu] W_P[r][q].  W_P is symmetric and each of its
// 64 x 64 blocks is read in the orientation that gemm2 stored: rows r when r's block is q's or a later one,
// rows q otherwise.
template <typename T, int YM>
__global__ __launch_bounds__(256, 3) void df_y_kernel(int nbf, int nact, int np, int nsplit, const T* __restrict__ XT, int ldx,
                                                   const T* __restrict__ W, int ldw, T* __restrict__ Ypart) {
  static_assert(YN == BT && BT % SK == 0, "one block column of W per tile, whole slabs per block");
  __shared__ FpSlab<T, YM> sa[2];
  __shared__ FpSlab<T, YN> sb[2];
  const int tn_n = (nact + YN - 1) / YN, tiles = ((nbf + YM - 1) / YM) * tn_n;
  const int w = xcd_item(tiles * nsplit);
  if (w < 0) return;
  const int s = w / tiles, m0 = (w % tiles) / tn_n * YM, n0 = (w % tn_n) * YN;
  const int pb = (int)((long long)np * s / nsplit), pe = (int)((long long)np * (s + 1) / nsplit);
  typename Fp<T>::acc acc[YM / 32][YN / 32];
#pragma unroll
  for (int i = 0; i < YM / 32; ++i)
#pragma unroll
    for (int j = 0; j < YN / 32; ++j) acc[i][j] = typename Fp<T>::acc{0, 0, 0, 0};
  auto A = [&](int seg) { return XT + (long long)(pb + seg) * nact * ldx; };
  auto B = [&](int seg) { return W + (long long)(pb + seg) * nact * ldw; };
  auto bcol = [&](int k0) { return k0 / BT >= n0 / BT; };
  auto epi = [](int, typename Fp<T>::acc(&)[YM / 32][YN / 32]) {};
  fp_mainloop<T, T, YM, YN, true, true, false>(sa, sb, pe - pb, nact, A, ldx, nact, m0, B, ldw, nact, n0, bcol, acc, epi);
  T* Y = Ypart + (long long)s * nbf * nact;
#pragma unroll
  for (int i = 0; i < YM / 32; ++i)
#pragma unroll
    for (int j = 0; j < YN / 32; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + fp_row0<YM>(i) + Fp<T>::row(e), n = n0 + fp_col<YN>(j);
        if (m < nbf && n < nact) Y[(long long)m * nact + n] = acc[i][j][e];
      }
}

}  // namespace

hipError_t gemm_f64(hipStream_t s, int M, int N, int K, int batch, double alpha, const double* A,
                    long long sam, long long sak, long long sab, const double* B, long long sbk,
                    long long sbn, long long sbb, double beta, double* C, long long scm, long long scn,
                    long long scb) {
  if (M <= 0 || N <= 0 || batch <= 0) return hipSuccess;
  const bool am = (sam == 1), bn = (sbn == 1);
  if (batch == 1) {
    const dim3 g1((unsigned)(cdiv(M, wide::BM) * cdiv(N, wide::BNT)));
    auto go = [&](auto kern, int kg) {
      hipLaunchKernelGGL(kern, g1, dim3(256 * kg), 0, s, M, N, K, alpha, A, sam, sak, B, sbk, sbn, beta, C, scm, scn);
    };
    auto pick = [&](auto am_, auto bn_) {
      constexpr bool AM = decltype(am_)::value, BN = decltype(bn_)::value;
      switch (gemm_f64_groups(M, N, K)) {
        case 4: go(gemm_f64_wide_kernel<AM, BN, 4>, 4); break;
        case 2: go(gemm_f64_wide_kernel<AM, BN, 2>, 2); break;
        default: go(gemm_f64_wide_kernel<AM, BN, 1>, 1); break;
      }
    };
    if (am && bn) pick(std::true_type{}, std::true_type{});
    else if (am) pick(std::true_type{}, std::false_type{});
    else if (bn) pick(std::false_type{}, std::true_type{});
    else pick(std::false_type{}, std::false_type{});
    return hipGetLastError();
  }
  dim3 grid(cdiv(M, TM) * cdiv(N, TN), batch);
  if (am && bn)
    hipLaunchKernelGGL((gemm_f64_kernel<true, true>), grid, dim3(256), 0, s, M, N, K, alpha, A, sam, sak, sab, B, sbk, sbn, sbb, beta, C, scm, scn, scb);
  else if (am && !bn)
    hipLaunchKernelGGL((gemm_f64_kernel<true, false>), grid, dim3(256), 0, s, M, N, K, alpha, A, sam, sak, sab, B, sbk, sbn, sbb, beta, C, scm, scn, scb);
  else if (!am && bn)
    hipLaunchKernelGGL((gemm_f64_kernel<false, true>), grid, dim3(256), 0, s, M, N, K, alpha, A, sam, sak, sab, B, sbk, sbn, sbb, beta, C, scm, scn, scb);
  else
    hipLaunchKernelGGL((gemm_f64_kernel<false, false>), grid, dim3(256), 0, s, M, N, K, alpha, A, sam, sak, sab, B, sbk, sbn, sbb, beta, C, scm, scn, scb);
  return hipGetLastError();
}

int gemm_f64_ksplit(int M, int N, int K) {
  const int tiles = cdiv(M, TM) * cdiv(N, TN);
  int ks = cdiv(512, tiles);                   // about two blocks per compute unit
  ks = ks < F64_KSPLIT_MAX ? ks : F64_KSPLIT_MAX;
  const int kmax = cdiv(K, 4 * TK);            // at least four k-slabs per block
  return ks < kmax ? ks : (kmax > 0 ? kmax : 1);
}

hipError_t gemm_f64_splitk(hipStream_t s, int M, int N, int K, int ks, const double* A, long long sam, long long sak,
                           const double* B, long long sbk, long long sbn, double* Cpart) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (ks < 1 || ks > F64_KSPLIT_MAX) return hipErrorInvalidValue;
  const dim3 grid(cdiv(M, TM) * cdiv(N, TN) * ks);
  const bool am = (sam == 1), bn = (sbn == 1);
  if (am && bn)
    hipLaunchKernelGGL((gemm_f64_splitk_kernel<true, true>), grid, dim3(256), 0, s, M, N, K, ks, A, sam, sak, B, sbk, sbn, Cpart);
  else if (am)
    hipLaunchKernelGGL((gemm_f64_splitk_kernel<true, false>), grid, dim3(256), 0, s, M, N, K, ks, A, sam, sak, B, sbk, sbn, Cpart);
  else if (bn)
    hipLaunchKernelGGL((gemm_f64_splitk_kernel<false, true>), grid, dim3(256), 0, s, M, N, K, ks, A, sam, sak, B, sbk, sbn, Cpart);
  else
    hipLaunchKernelGGL((gemm_f64_splitk_kernel<false, false>), grid, dim3(256), 0, s, M, N, K, ks, A, sam, sak, B, sbk, sbn, Cpart);
  return hipGetLastError();
}

hipError_t gemm_f64_grouped(hipStream_t s, int ngemm, int maxM, int maxN, bool a_unit_m, bool b_unit_n,
                            const F64Gemm* tab) {
  if (ngemm <= 0 || maxM <= 0 || maxN <= 0) return hipSuccess;
  dim3 grid(cdiv(maxM, TM) * cdiv(maxN, TN), ngemm);
  if (a_unit_m && b_unit_n) hipLaunchKernelGGL((gemm_f64_grouped_kernel<true, true>), grid, dim3(256), 0, s, tab);
  else if (a_unit_m) hipLaunchKernelGGL((gemm_f64_grouped_kernel<true, false>), grid, dim3(256), 0, s, tab);
  else if (b_unit_n) hipLaunchKernelGGL((gemm_f64_grouped_kernel<false, true>), grid, dim3(256), 0, s, tab);
  else hipLaunchKernelGGL((gemm_f64_grouped_kernel<false, false>), grid, dim3(256), 0, s, tab);
  return hipGetLastError();
}

// Height of Y's tile: the one whose launch ends sooner, counted as blocks on the fullest of 256 compute units
// times the rows of one (128 on a tie: it reads W half as often).
int df_fp_y_tile(int nbf, int nact, int nsplit) {
  const long long n = (long long)cdiv(nact, YN) * nsplit;
  return 128LL * cdiv(n * cdiv(nbf, 128), 256) <= 64LL * cdiv(n * cdiv(nbf, 64), 256) ? 128 : 64;
}

namespace {
inline dim3 xcd_grid(long long items) { return dim3((unsigned)(cdiv(items, 8) * 8)); }
}  // namespace

// float64 B: tiles of 64 rows while those of 128 make at most two blocks per compute unit, of the three that fit (600
// functions, 300 active, 12 rows of B, which are 285 tiles of 128: 93 us, 71 with tiles of 64).
constexpr int X_WIDE = 512;
template <typename T>
hipError_t df_fp_gemm1(hipStream_t s, int nbf, int nact, int np, const T* Ct, int ldk, const void* Bchunk, int b_is_bf16,
                       T* XT, int ldx) {
  if (np <= 0) return hipSuccess;
  if ((long long)np * nbf >= (1LL << 31)) return hipErrorInvalidValue;
  const long long rows = (long long)np * nbf, wide = cdiv(nact, XM) * (long long)cdiv(rows, 128);
  if (b_is_bf16)
    hipLaunchKernelGGL((df_x_kernel<T, u16, 128>), xcd_grid(wide), dim3(256), 0, s, nbf, nact, np, Ct, ldk,
                       static_cast<const u16*>(Bchunk), XT, ldx);
  else if (wide > X_WIDE)
    hipLaunchKernelGGL((df_x_kernel<T, double, 128>), xcd_grid(wide), dim3(256), 0, s, nbf, nact, np, Ct, ldk,
                       static_cast<const double*>(Bchunk), XT, ldx);
  else
    hipLaunchKernelGGL((df_x_kernel<T, double, 64>), xcd_grid((long long)cdiv(nact, XM) * cdiv(rows, 64)), dim3(256), 0, s, nbf,
                       nact, np, Ct, ldk, static_cast<const double*>(Bchunk), XT, ldx);
  return hipGetLastError();
}
template <typename T>
hipError_t df_fp_gemm2(hipStream_t s, int nbf, int nact, int np, int nsplit, const T* Ct, int ldk, const T* XT, int ldx,
                       const T* beta, int ldbeta, double* Kpart, bool kset, double* Dchunk, T* W, int ldw) {
  if (np <= 0) return hipSuccess;
  const long long t = cdiv(nact, BT);
  hipLaunchKernelGGL(df_b_kernel<T>, xcd_grid(t * (t + 1) / 2 * nsplit), dim3(256), 0, s, nbf, nact, np, nsplit, Ct, ldk, XT,
                     ldx, beta, ldbeta, Kpart, kset ? 1 : 0, Dchunk, W, ldw);
  return hipGetLastError();
}
template <typename T>
hipError_t df_fp_gemm3(hipStream_t s, int nbf, int nact, int np, int nsplit, const T* XT, int ldx, const T* W, int ldw,
                       T* Ypart) {
  if (np <= 0) return hipSuccess;
  if (df_fp_y_tile(nbf, nact, nsplit) == 128)
    hipLaunchKernelGGL((df_y_kernel<T, 128>), xcd_grid((long long)cdiv(nbf, 128) * cdiv(nact, YN) * nsplit), dim3(256), 0, s,
                       nbf, nact, np, nsplit, XT, ldx, W, ldw, Ypart);
  else
    hipLaunchKernelGGL((df_y_kernel<T, 64>), xcd_grid((long long)cdiv(nbf, 64) * cdiv(nact, YN) * nsplit), dim3(256), 0, s,
                       nbf, nact, np, nsplit, XT, ldx, W, ldw, Ypart);
  return hipGetLastError();
}
#define DF_FP(T)                                                                                                            \
  template hipError_t df_fp_gemm1<T>(hipStream_t, int, int, int, const T*, int, const void*, int, T*, int);                 \
  template hipError_t df_fp_gemm2<T>(hipStream_t, int, int, int, int, const T*, int, const T*, int, const T*, int, double*,  \
                                     bool, double*, T*, int);                                                               \
  template hipError_t df_fp_gemm3<T>(hipStream_t, int, int, int, int, const T*, int, const T*, int, T*)
DF_FP(double);
DF_FP(float);

}  // namespace pnof
