// Element-wise, reduction and small-matrix kernels of the PNOF step (float64 throughout).
#include <algorithm>

#include "common.h"

namespace pnof {
namespace {

constexpr int NT = 256;

inline dim3 grid1(long long n, int per = NT) {
  long long b = (n + per - 1) / per;
  if (b < 1) b = 1;
  if (b > 65535LL * 16) b = 65535LL * 16;
  return dim3((unsigned)b);
}

#define GRID_STRIDE(i, n) \
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += (long long)gridDim.x * blockDim.x)

__global__ void fill_f64_k(double* p, long long n, double v) { GRID_STRIDE(i, n) p[i] = v; }

// alpha, beta of E_2 = sum_pq alpha_pq J_pq + beta_pq K_pq (Eqs. Eg, Efg, Efg_s); beta32: ld32 x ld32, zero past
// nact.
__global__ void coeffs_k(int nact, int ld32, int npairs, int ncwo, int nsingle, int functional, const double* __restrict__ n,
                         double* __restrict__ alpha, double* __restrict__ beta, float* __restrict__ beta32) {
  const int w = beta32 ? ld32 : nact;
  GRID_STRIDE(i, (long long)w * w) {
    const int p = (int)(i / w), q = (int)(i % w);
    double a, b = 0.0;
    if (p < nact && q < nact) {
      pnof_coeff(p, q, n[p], n[q], npairs, ncwo, nsingle, functional, a, b);
      alpha[(long long)p * nact + q] = a;
      beta[(long long)p * nact + q] = b;
    }
    if (beta32) beta32[i] = (float)b;
  }
}

template <typename T>
__global__ void transpose_ca_k(int nbf, int nact, const double* __restrict__ C, T* __restrict__ Ct, int ldk) {
  GRID_STRIDE(i, (long long)nact * nbf) {
    const int p = (int)(i / nbf), mu = (int)(i % nbf);
    Ct[(long long)p * ldk + mu] = (T)C[(long long)mu * nbf + p];
  }
}

// C_A^T as bf16: one value (terms 1), or the compact bf16 pair C~ = hi + lo of X's contraction plus
// the exact fp16 pair of C~ sC for the b contraction (and X from a float64 B); zeros in the padding
// (rows nact to `rows`, columns nbf to ldk).
__global__ void split_ca_k(int nbf, int nact, int rows, int terms, const double* __restrict__ C, u16* __restrict__ hi,
                           u16* __restrict__ lo, u16* __restrict__ h16, u16* __restrict__ l16, int ldk,
                           const uint32_t* __restrict__ bnd) {
  const float sC = terms > 1 ? chunk_scales(bnd, 0, false).sC : 1.0f;
  GRID_STRIDE(o, (long long)rows * ldk) {
    const int p = (int)(o / ldk), mu = (int)(o % ldk);
    const double x = p < nact && mu < nbf ? C[(long long)mu * nbf + p] : 0.0;
    if (terms == 1) {
      hi[o] = f32_to_bf16_bits((float)x);
      continue;
    }
    u16 h, l;
    split_compact(x, h, l);
    hi[o] = h;
    lo[o] = l;
    // hi + lo spans at most 22 bits: exact in float32, and its fp16 pair is exact (split_compact)
    const float xs = (bf16_bits_to_f32(h) + bf16_bits_to_f32(l)) * sC;
    u16 a, b;
    split_f16(xs, a, b);
    h16[o] = a;
    l16[o] = b;
  }
}

// Rows of float64 B (n elements each) as the fp16 pair of B sB (sB of the chunk), or as one bf16 value
// when bnd is null, in rows of ldo (a multiple of 8) with zeros from n on; ldo == n: one run of
// nrows n elements, whatever n is.  One thread per 8 elements: four 16-byte loads, one 16-byte store
// of each part.
__global__ __launch_bounds__(NT) void split_b_k(long long tot, uint32_t pieces, int n, const double* __restrict__ B,
                                                u16* __restrict__ hi, u16* __restrict__ lo, int ldo,
                                                const uint32_t* __restrict__ bnd, int chunk) {
  const double sB = bnd ? (double)chunk_scales(bnd, chunk, true).sB : 1.0;
  const uint32_t per = (uint32_t)(ldo / 8);
  for (uint32_t i = blockIdx.x * NT + threadIdx.x; i < pieces; i += gridDim.x * NT) {
    long long so = 8LL * i, o = so;   // first element read and written
    int valid = (int)min(8LL, tot - so);
    if (ldo != n) {
      const uint32_t r = i / per;
      const int c = 8 * (int)(i - r * per);
      so = (long long)r * n + c;
      valid = min(8, n - c);
    }
    double x[8];
    if (valid == 8) {
      __builtin_memcpy(x, B + so, 64);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) x[k] = k < valid ? B[so + k] : 0.0;
    }
    u16 h[8], l[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (bnd) {
        const double xs = x[k] * sB;
        h[k] = f32_to_f16_bits((float)xs);
        l[k] = f32_to_f16_bits((float)(xs - (double)f16_bits_to_f32(h[k])));
      } else {
        h[k] = f32_to_bf16_bits((float)x[k]);
        l[k] = 0;
      }
    }
    if (valid == 8 || ldo != n) {
      uint4 v;
      __builtin_memcpy(&v, h, 16);
      *reinterpret_cast<uint4*>(hi + o) = v;
      if (bnd) {
        __builtin_memcpy(&v, l, 16);
        *reinterpret_cast<uint4*>(lo + o) = v;
      }
    } else {
      for (int k = 0; k < valid; ++k) {
        hi[o + k] = h[k];
        if (bnd) lo[o + k] = l[k];
      }
    }
  }
}

// Scale bounds, stage 1: one wavefront per active orbital q writes col[4q..4q+3] = sum_mu |C_mu q|,
// max_mu |C_mu q|, sum_r |alpha_qr|, max_r |beta_qr| (alpha, beta of Eqs. Eg, Efg from n; zero when
// n is absent).
__global__ void col_bounds_k(int nbf, int nact, const double* __restrict__ C, const double* __restrict__ n,
                             int npairs, int ncwo, int nsingle, int functional, float* __restrict__ col) {
  const int lane = threadIdx.x & 63;
  const int q = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (q >= nact) return;
  double s1 = 0.0, cm = 0.0, sa = 0.0, bm = 0.0;
  for (int mu = lane; mu < nbf; mu += 64) {
    const double c = fabs(C[(long long)mu * nbf + q]);
    s1 += c;
    cm = fmax(cm, c);
  }
  if (n) {
    for (int r = lane; r < nact; r += 64) {
      double a, b;
      pnof_coeff(q, r, n[q], n[r], npairs, ncwo, nsingle, functional, a, b);
      sa += fabs(a);
      bm = fmax(bm, fabs(b));
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    s1 += __shfl_down(s1, off, 64);
    sa += __shfl_down(sa, off, 64);
    cm = fmax(cm, __shfl_down(cm, off, 64));
    bm = fmax(bm, __shfl_down(bm, off, 64));
  }
  if (lane == 0) {
    col[4 * q + 0] = (float)s1;
    col[4 * q + 1] = (float)cm;
    col[4 * q + 2] = (float)sa;
    col[4 * q + 3] = (float)bm;
  }
}

// Scale bounds, stage 2 (one block): the call-level words of bnd, and the per-chunk words cleared.
__global__ void bounds_reduce_k(int nact, const float* __restrict__ col, uint32_t* __restrict__ bnd, int nclear) {
  __shared__ float red[4][NT / 64];
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int q = threadIdx.x; q < nact; q += blockDim.x)
    for (int k = 0; k < 4; ++k) v[k] = fmaxf(v[k], col[4 * q + k]);
  for (int off = 32; off > 0; off >>= 1)
    for (int k = 0; k < 4; ++k) v[k] = fmaxf(v[k], __shfl_down(v[k], off, 64));
  if ((threadIdx.x & 63) == 0)
    for (int k = 0; k < 4; ++k) red[k][threadIdx.x >> 6] = v[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 0; k < 4; ++k)
      for (int w = 1; w < NT / 64; ++w) red[k][0] = fmaxf(red[k][0], red[k][w]);
    bnd[0] = __float_as_uint(red[1][0]);                 // max |C|
    bnd[1] = __float_as_uint(red[0][0]);                 // max column 1-norm
    bnd[2] = __float_as_uint(red[3][0] + red[2][0]);     // max |beta| + max row 1-norm of alpha
    bnd[3] = 0u;
  }
  for (int i = threadIdx.x; i < nclear; i += blockDim.x) bnd[SCL_CALL + i] = 0u;
}

// One pass over rows of B (rows of n elements, densely stored): the bounds that fix a chunk's scales
// and / or a copy with 16-byte aligned rows.  blockIdx.y is the chunk of rows_per_chunk consecutive
// rows; LPR lanes share a row, each taking 16-byte pieces of it (whatever the row's alignment: the
// row's last piece is loaded so that it ends with the row and shifted down, so nothing past the row
// is read), RU rows of a group in flight.
//   BND   the largest row 1-norm and the largest |B| of the chunk, raised into slot[2c], slot[2c + 1]
//         with integer atomic maxima on the bits of the non-negative floats, once per block;
//   PACK  (bf16) row r copied to out + r ldo, zero from n to ldo (a multiple of 8).
// Memory-bound.  2000 x 500 rows of 500 bf16 (1 GB): the bounds alone 752 us with one wavefront walking
// 2-byte elements of one row at a time, 217 us here (4.6 TB/s); the copy of bf16 rows in six chunks 391 us (5.1 TB/s read and written).
// 800 x 200 rows of 200 float64 (256 MB): 405 us before, 99 us here.
constexpr int RU = 4;
// The 16 bytes at element c of a row of n (zeros from n on), as loaded from element min(c, n - E) and
// moved down by c minus that; rows shorter than one piece element by element.
template <typename T>
__device__ __forceinline__ unsigned __int128 row_load(const T* __restrict__ row, int c, int n) {
  constexpr int E = 16 / sizeof(T);
  unsigned __int128 x = 0;
  if (n >= E) {
    __builtin_memcpy(&x, row + (c < n - E ? c : n - E), 16);
  } else {
    T v[E] = {};
    for (int k = 0; k < E; ++k)
      if (c + k < n) v[k] = row[c + k];
    __builtin_memcpy(&x, v, 16);
  }
  return x;
}
template <typename T>
__device__ __forceinline__ unsigned __int128 row_shift(unsigned __int128 x, int c, int n) {
  constexpr int E = 16 / sizeof(T);
  const int d = n >= E && c > n - E ? c - (n - E) : 0;
  return d >= E ? 0 : x >> (8 * (int)sizeof(T) * d);
}
__device__ __forceinline__ void piece_abs(unsigned __int128 x, float (&v)[8]) {
  uint32_t w[4];
  __builtin_memcpy(w, &x, 16);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[2 * k] = fabsf(__uint_as_float(w[k] << 16));
    v[2 * k + 1] = fabsf(__uint_as_float(w[k] & 0xFFFF0000u));
  }
}
__device__ __forceinline__ void piece_abs(unsigned __int128 x, float (&v)[2]) {
  double d[2];
  __builtin_memcpy(d, &x, 16);
  v[0] = (float)fabs(d[0]);
  v[1] = (float)fabs(d[1]);
}
template <typename T, int LPR, bool BND, bool PACK>
__global__ __launch_bounds__(NT) void b_rows_k(const T* __restrict__ B, long long nrows, int n, long long rows_per_chunk,
                                               uint32_t* __restrict__ slot, u16* __restrict__ out, int ldo) {
  constexpr int E = 16 / sizeof(T), RB = NT / LPR;   // elements per piece, rows of a block at a time
  const long long c0 = blockIdx.y * rows_per_chunk, c1 = c0 + rows_per_chunk < nrows ? c0 + rows_per_chunk : nrows;
  const int g = threadIdx.x / LPR, l = threadIdx.x % LPR;
  const int width = PACK ? ldo : n;
  float rmax = 0.f, amax = 0.f;
  for (long long r0 = c0 + (long long)blockIdx.x * (RB * RU); r0 < c1; r0 += (long long)gridDim.x * (RB * RU)) {
    float s[RU];
#pragma unroll
    for (int u = 0; u < RU; ++u) s[u] = 0.f;
    for (int c = E * l; c < width; c += E * LPR) {
      unsigned __int128 x[RU];
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        const long long r = r0 + u * RB + g;
        x[u] = row_load(B + (r < c1 ? r : c1 - 1) * n, c, n);
      }
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        const long long r = r0 + u * RB + g;
        x[u] = r < c1 ? row_shift<T>(x[u], c, n) : 0;
        if constexpr (PACK) {
          uint4 w;
          __builtin_memcpy(&w, &x[u], 16);
          if (r < c1) *reinterpret_cast<uint4*>(out + r * ldo + c) = w;
        }
        if constexpr (BND) {
          float v[E];
          piece_abs(x[u], v);
#pragma unroll
          for (int k = 0; k < E; ++k) {
            s[u] += v[k];
            amax = fmaxf(amax, v[k]);
          }
        }
      }
    }
    if constexpr (BND) {
#pragma unroll
      for (int u = 0; u < RU; ++u) {
#pragma unroll
        for (int m = LPR / 2; m >= 1; m >>= 1) s[u] += __shfl_xor(s[u], m, 64);
        rmax = fmaxf(rmax, s[u]);
      }
    }
  }
  if constexpr (BND) {
    __shared__ float red[2][NT / 64];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      rmax = fmaxf(rmax, __shfl_xor(rmax, m, 64));
      amax = fmaxf(amax, __shfl_xor(amax, m, 64));
    }
    if ((threadIdx.x & 63) == 0) {
      red[0][threadIdx.x >> 6] = rmax;
      red[1][threadIdx.x >> 6] = amax;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
      float m = 0.f;
      for (int w = 0; w < NT / 64; ++w) m = fmaxf(m, red[threadIdx.x][w]);
      if (m > 0.f) atomicMax(slot + 2 * blockIdx.y + threadIdx.x, __float_as_uint(m));
    }
  }
}

// Hpp[p] = sum_mu C[mu][p] HC[mu][p]: one wavefront per orbital, fixed reduction order.
__global__ void hpp_k(int nbf, int nact, const double* __restrict__ C, const double* __restrict__ HC,
                      double* __restrict__ Hpp) {
  const int p = blockIdx.x;
  const int lane = threadIdx.x;
  double s = 0.0;
  for (int mu = lane; mu < nbf; mu += 64) s += C[(long long)mu * nbf + p] * HC[(long long)mu * nact + p];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) Hpp[p] = s;
}

// W_P[p][p] += d[P][p], with d = D alpha (d_Pp = sum_q D_Pq alpha_qp) computed beforehand as ks
// partial slabs over ranges of q, added here in slab order.
__device__ __forceinline__ double sum_slabs(const double* __restrict__ d, int ks, long long slab, long long i) {
  double v = 0.0;
  for (int s = 0; s < ks; ++s) v += d[s * slab + i];
  return v;
}

// d[P][q] = sum_p D[P][p] alpha_pq.  The Coulomb coefficients are alpha_pq = 2 n_p n_q between
// different subspaces and 0 within one (Eqs. Eg, Efg), so d = 2 n_q (s_P - S_P,g(q)) with
// s_P = sum_p n_p D[P][p] and S_P,g the same sum over q's own subspace (a strong orbital and its weak
// ones, or one singly occupied orbital): O(nact) per row instead of a product with alpha.  One
// workgroup per row P; the row sum is reduced in a fixed order.
__global__ void d_alpha_k(int nact, int npairs, int ncwo, int nsingle, const double* __restrict__ n,
                          const double* __restrict__ Dc, double* __restrict__ d) {
  const int P = blockIdx.x, tid = threadIdx.x;
  const double* Dr = Dc + (long long)P * nact;
  __shared__ double red[NT / 64];
  double v = 0.0;
  for (int p = tid; p < nact; p += NT) v += n[p] * Dr[p];
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  double sP = 0.0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) sP += red[w];
  for (int q = tid; q < nact; q += NT) {
    const int g = pair_of(q, npairs, ncwo, nsingle);
    double Sg;
    if (g < npairs) {
      Sg = n[g] * Dr[g];
      for (int k = 0; k < ncwo; ++k) {
        const int w = weak_index(g, k, npairs, ncwo, nsingle);
        Sg += n[w] * Dr[w];
      }
    } else {
      Sg = n[q] * Dr[q];
    }
    d[(long long)P * nact + q] = 2.0 * n[q] * (sP - Sg);
  }
}

__global__ void add_diag_f64_k(int nact, int np, int ks, const double* __restrict__ d, double* __restrict__ W,
                               int ldw) {
  const long long slab = (long long)np * nact;
  GRID_STRIDE(i, slab) {
    const long long P = i / nact;
    const int p = (int)(i % nact);
    W[P * nact * ldw + (long long)p * ldw + p] += sum_slabs(d, ks, slab, i);
  }
}

__global__ void add_diag_f32_k(int nact, int np, int ks, const double* __restrict__ d, float* __restrict__ W, int ldw) {
  const long long slab = (long long)np * nact;
  GRID_STRIDE(i, slab) {
    const long long P = i / nact;
    const int p = (int)(i % nact);
    float* w = W + P * nact * ldw + (long long)p * ldw + p;
    *w = (float)((double)*w + sum_slabs(d, ks, slab, i));
  }
}

__global__ void add_diag_bf16_k(int nact, int np, int ks, const double* __restrict__ d, const double* __restrict__ Dc,
                                const float* __restrict__ beta32, u16* __restrict__ Wh, u16* __restrict__ Wl, int ldw,
                                long long pstride, const uint32_t* __restrict__ bnd, int chunk) {
  const long long slab = (long long)np * nact;
  const float sW = Wl ? chunk_scales(bnd, chunk, false).sW : 1.0f;
  GRID_STRIDE(i, slab) {
    const long long P = i / nact;
    const int p = (int)(i % nact);
    const long long o = P * pstride + (long long)p * ldw + p;
    const float wv = (float)Dc[i] * beta32[(long long)p * ldw + p];
    const double w = (double)wv + sum_slabs(d, ks, slab, i);
    if (Wl) {   // split mode: the fp16 pair of W sW
      u16 h, l;
      split_f16((float)(w * (double)sW), h, l);
      Wh[o] = h;
      Wl[o] = l;
    } else {
      Wh[o] = f32_to_bf16_bits((float)w);
    }
  }
}

// K[p][q] = sum_s Kpart[s][max][min], mirrored: each lower-triangle position is read along rows
// (coalesced) and written to both halves.
// Sums of split partials.  PARTS groups of threads share an element's splits between them, so that many splits do not
// wait one behind the other (each group reads its own with eight loads in flight; the groups' sums meet in LDS, in
// order; K of 75 functions 17.5 -> 6.0 us).
constexpr int RED_PARTS = 8, RED_SPLITS = 24;   // from RED_SPLITS splits on
template <int PARTS, typename T>
__device__ __forceinline__ double sum_parts(const T* __restrict__ p, bool valid, int nsplit, long long stride) {
  if constexpr (PARTS == 1) {
    return valid ? sum_strided(p, nsplit, stride) : 0.0;
  } else {
    __shared__ double red[PARTS - 1][64];
    const int part = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int b = nsplit * part / PARTS, e = nsplit * (part + 1) / PARTS;
    double s = valid ? sum_strided(p + b * stride, e - b, stride) : 0.0;
    __syncthreads();
    if (part > 0) red[part - 1][lane] = s;
    __syncthreads();
    if (part == 0)
      for (int k = 0; k < PARTS - 1; ++k) s += red[k][lane];
    return s;
  }
}
// Elements [64 b, 64 b + 64) (PARTS > 1) or [NT b, ..) of block b.
template <int PARTS>
__global__ void reduce_k_k(int nact, int nsplit, const double* __restrict__ Kpart, double* __restrict__ K) {
  const long long n2 = (long long)nact * nact, i = (long long)blockIdx.x * (PARTS > 1 ? 64 : NT) + (PARTS > 1 ? threadIdx.x & 63 : threadIdx.x);
  const int p = (int)(i / nact), q = (int)(i % nact);
  const bool valid = i < n2 && q <= p;
  const double s = sum_parts<PARTS>(Kpart + (valid ? i : 0), valid, nsplit, n2);
  if (!valid || (PARTS > 1 && threadIdx.x >= 64)) return;
  K[i] = s;
  if (q != p) K[(long long)q * nact + p] = s;
}

template <int PARTS, typename T>
__global__ void reduce_y_k(long long n, int nsplit, int first, const T* __restrict__ Yp, double* __restrict__ Y) {
  const long long i = (long long)blockIdx.x * (PARTS > 1 ? 64 : NT) + (PARTS > 1 ? threadIdx.x & 63 : threadIdx.x);
  const bool valid = i < n;
  const double y = sum_parts<PARTS>(Yp + (valid ? i : 0), valid, nsplit, n);
  if (!valid || (PARTS > 1 && threadIdx.x >= 64)) return;
  Y[i] = first ? y : Y[i] + y;
}

// Energy (Eqs. EPNOF7, Eg, Efg) and, for split arithmetic, the first-order correction
// 4 <Y2e, C_A - C~_A>.  Stage 1: fixed-range block partial sums; stage 2: one block.
__device__ inline double block_sum(double v) {
  __shared__ double red[NT / 64];
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < NT / 64; ++i) s += red[i];
  return s;
}

struct EnergyArgs {
  int nbf, nact;
  const double *n, *Hpp, *alpha, *beta, *J, *K, *Y2e, *C;
  const u16 *cth, *ctl;
  const float* ct32;
  int ldk, corr_terms;
};
// Block `part` of `parts`: its range of the terms of E.
__device__ inline double energy_part(const EnergyArgs& a, int part, int parts) {
  const int nact = a.nact;
  const long long n2 = (long long)nact * nact;
  const long long ncorr = a.corr_terms > 0 ? (long long)a.nbf * nact : 0;
  const long long total = nact + n2 + ncorr;
  const long long per = (total + parts - 1) / parts;
  const long long b0 = part * per, b1 = min(total, b0 + per);
  double s = 0.0;
  for (long long i = b0 + threadIdx.x; i < b1; i += blockDim.x) {
    if (i < nact) s += 2.0 * a.n[i] * a.Hpp[i];
    else if (i < nact + n2) { const long long k = i - nact; s += a.alpha[k] * a.J[k] + a.beta[k] * a.K[k]; }
    else {
      const long long k = i - nact - n2;
      const int mu = (int)(k / nact), p = (int)(k % nact);
      double ct;
      if (a.ct32) ct = (double)a.ct32[(long long)p * a.ldk + mu];
      else {
        ct = (double)bf16_bits_to_f32(a.cth[(long long)p * a.ldk + mu]);
        if (a.corr_terms > 1) ct += (double)bf16_bits_to_f32(a.ctl[(long long)p * a.ldk + mu]);
      }
      s += 4.0 * a.Y2e[k] * (a.C[(long long)mu * a.nbf + p] - ct);
    }
  }
  return block_sum(s);
}
__global__ void energy_stage1_k(EnergyArgs a, double* __restrict__ partials) {
  const double s = energy_part(a, blockIdx.x, gridDim.x);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

__global__ void sum_partials_k(int nparts, const double* __restrict__ partials, double* __restrict__ out) {
  double s = 0.0;
  for (int i = threadIdx.x; i < nparts; i += blockDim.x) s += partials[i];
  s = block_sum(s);
  if (threadIdx.x == 0) *out = s;
}

// NOF-MP2 reference terms (Eqs. HFL, Esta): block partial sums of E_hf and E_sta over a fixed
// range of the index space [0, nom) + [0, nom^2) + [0, nact^2), nom = npairs + nsingle (the
// subspace-defining orbitals, weight A = 1 strong, 1/2 single); stage 2 adds the partials in order.
__global__ void nofmp2_stage1_k(int nact, int npairs, int ncwo, int nsingle, const double* __restrict__ n,
                                const double* __restrict__ Hpp, const double* __restrict__ J,
                                const double* __restrict__ K, double* __restrict__ partials) {
  const long long n2 = (long long)nact * nact;
  const int nom = npairs + nsingle;
  const long long total = nom + (long long)nom * nom + n2;
  const long long per = (total + gridDim.x - 1) / gridDim.x;
  const long long b0 = blockIdx.x * per, b1 = min(total, b0 + per);
  double hf = 0.0, sta = 0.0;
  for (long long i = b0 + threadIdx.x; i < b1; i += blockDim.x) {
    if (i < nom) {
      const int g = (int)i;
      // 2 A_g H_gg, and minus the self-Coulomb J_gg / 4 of a single orbital
      hf += g < npairs ? 2.0 * Hpp[g] : Hpp[g] - 0.25 * J[(long long)g * nact + g];
    } else if (i < nom + (long long)nom * nom) {
      const long long k = i - nom;
      const int f = (int)(k / nom), g = (int)(k % nom);
      const double af = f < npairs ? 1.0 : 0.5, ag = g < npairs ? 1.0 : 0.5;
      hf += af * ag * (2.0 * J[(long long)f * nact + g] - K[(long long)f * nact + g]);
    } else {
      const long long k = i - nom - (long long)nom * nom;
      const int p = (int)(k / nact), q = (int)(k % nact);
      if (p == q) continue;
      const double np_ = n[p], nq = n[q];
      if (pair_of(p, npairs, ncwo, nsingle) == pair_of(q, npairs, ncwo, nsingle)) {
        const double lp = 1.0 - fabs(1.0 - 2.0 * np_), lq = 1.0 - fabs(1.0 - 2.0 * nq);
        const double sg = (p < npairs || q < npairs) ? -1.0 : 1.0;
        sta += sqrt(lp * lq) * sg * sqrt(np_ * nq) * K[k];
      } else {
        sta += -4.0 * (nq * (1.0 - nq)) * (np_ * (1.0 - np_)) * K[k];
      }
    }
  }
  hf = block_sum(hf);
  sta = block_sum(sta);
  if (threadIdx.x == 0) {
    partials[2 * blockIdx.x] = hf;
    partials[2 * blockIdx.x + 1] = sta;
  }
}

__global__ void sum2_partials_k(int nparts, const double* __restrict__ partials, double* __restrict__ a,
                                double* __restrict__ b) {
  double x = 0.0, y = 0.0;
  for (int i = threadIdx.x; i < nparts; i += blockDim.x) {
    x += partials[2 * i];
    y += partials[2 * i + 1];
  }
  x = block_sum(x);
  y = block_sum(y);
  if (threadIdx.x == 0) {
    *a = x;
    *b = y;
  }
}

__device__ inline double block_max(double v) {
  __shared__ double red[NT / 64];
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_down(v, off, 64));
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < NT / 64; ++i) s = fmax(s, red[i]);
  return s;
}

// dE/dn_p (derivative of Eqs. Eg, Efg at fixed J, K, H_pp), by one wavefront.
__device__ inline void grad_n_row(int p, int nact, int npairs, int ncwo, int nsingle, int functional, const double* __restrict__ n,
                                  const double* __restrict__ Hpp, const double* __restrict__ J, const double* __restrict__ K,
                                  double* __restrict__ g) {
  const int lane = threadIdx.x & 63;
  const double np_ = n[p];
  const double php = sqrt(np_ * (1.0 - np_));
  double s = 0.0;
  for (int q = lane; q < nact; q += 64) {
    if (q == p) continue;
    s += grad_n_term(p, q, np_, n[q], php, J[(long long)p * nact + q], K[(long long)p * nact + q], npairs, ncwo,
                     nsingle, functional);
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  // a singly occupied orbital has no K_pp term (beta_pp = 0); its n is fixed at 1/2
  if (lane == 0) g[p] = 2.0 * Hpp[p] + (is_single(p, npairs, nsingle) ? 0.0 : K[(long long)p * nact + p]) + s;
}

// What the step forms between the contractions and lambda = C^T Y, in one launch: blocks [0, ne) the partial sums of
// E; the next ng dE/dn, a wave per orbital; the rest element by element Y = n o (H C_A) + Y2e, the zero columns of
// lambda past nact, and the zero from which step_end_k raises the asymmetry.
struct TailArgs {
  EnergyArgs e;
  int ne, ng, npairs, ncwo, nsingle, functional;
  const double* HC;
  double *partials, *dEdn, *Y, *lam, *asym;
};
__global__ void step_tail_k(TailArgs a) {
  const int nbf = a.e.nbf, nact = a.e.nact;
  int b = blockIdx.x;
  if (b < a.ne) {
    const double s = energy_part(a.e, b, a.ne);
    if (threadIdx.x == 0) a.partials[b] = s;
    return;
  }
  b -= a.ne;
  if (b < a.ng) {
    const int p = b * (NT / 64) + (threadIdx.x >> 6);
    if (p < nact) grad_n_row(p, nact, a.npairs, a.ncwo, a.nsingle, a.functional, a.e.n, a.e.Hpp, a.e.J, a.e.K, a.dEdn);
    return;
  }
  b -= a.ng;
  if (b == 0 && threadIdx.x == 0 && a.asym) *a.asym = 0.0;
  const int w = a.lam ? nbf : nact;
  const long long stride = (long long)(gridDim.x - a.ne - a.ng) * NT;
  for (long long i = (long long)b * NT + threadIdx.x; i < (long long)nbf * w; i += stride) {
    const long long mu = i / w;
    const int q = (int)(i - mu * w);
    const long long o = mu * nact + q;
    if (q < nact) a.Y[o] = a.e.n[q] * a.HC[o] + a.e.Y2e[o];
    else a.lam[i] = 0.0;
  }
}
// After lambda: block 0 adds the partial sums of E, the next na raise max |lambda - lambda^T| (not negative, so its
// bits order as its value), the rest write dE/dC = 4 Y, zero past nact (it may take the place of C, which E and
// lambda are formed from).
__global__ void step_end_k(int ne, int na, const double* __restrict__ partials, double* __restrict__ E, int nbf, int nact,
                           const double* __restrict__ lam, double* __restrict__ asym, const double* __restrict__ Y,
                           double* __restrict__ dEdC) {
  if (blockIdx.x == 0) {
    double s = 0.0;
    for (int i = threadIdx.x; i < ne; i += blockDim.x) s += partials[i];
    s = block_sum(s);
    if (threadIdx.x == 0 && ne > 0) *E = s;
    return;
  }
  if ((int)blockIdx.x > na) {
    const long long stride = (long long)(gridDim.x - 1 - na) * NT;
    for (long long i = (long long)(blockIdx.x - 1 - na) * NT + threadIdx.x; i < (long long)nbf * nbf; i += stride) {
      const long long mu = i / nbf;
      const int q = (int)(i - mu * nbf);
      dEdC[i] = q < nact ? 4.0 * Y[mu * nact + q] : 0.0;
    }
    return;
  }
  double m = 0.0;
  for (long long i = (long long)(blockIdx.x - 1) * NT + threadIdx.x; i < (long long)nbf * nbf; i += (long long)na * NT) {
    const long long p = i / nbf, q = i % nbf;
    m = fmax(m, fabs(lam[i] - lam[q * nbf + p]));
  }
  m = block_max(m);
  if (threadIdx.x == 0) atomicMax(reinterpret_cast<unsigned long long*>(asym), (unsigned long long)__double_as_longlong(m));
}

// ON maps, one thread per pair (Section 3.1); singly occupied orbitals get n = 1/2 (their rows of
// the Jacobian stay zero).
__global__ void on_map_k(int kind, int npairs, int ncwo, int nsingle, const double* __restrict__ gamma,
                         double* __restrict__ n, double* __restrict__ jac) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g < nsingle) n[npairs + g] = 0.5;
  if (g >= npairs) return;
  const int nact = npairs * (ncwo + 1) + nsingle;
  const int ngam = kind == 0 ? nact : npairs * ncwo;
  if (kind == 0) {
    double S = sigm(gamma[g]);
    for (int k = 0; k < ncwo; ++k) S += sigm(gamma[weak_index(g, k, npairs, ncwo, nsingle)]);
    for (int a = -1; a < ncwo; ++a) {
      const int p = a < 0 ? g : weak_index(g, a, npairs, ncwo, nsingle);
      const double sp = sigm(gamma[p]);
      n[p] = sp / S;
      if (jac) {
        for (int b = -1; b < ncwo; ++b) {
          const int r = b < 0 ? g : weak_index(g, b, npairs, ncwo, nsingle);
          const double sr = sigm(gamma[r]);
          const double dsr = sr * (1.0 - sr);
          jac[(long long)p * ngam + r] = ((p == r ? dsr : 0.0) * S - sp * dsr) / (S * S);
        }
      }
    }
  } else {
    const double gs = gamma[g];
    const double cg = cos(gs), sg = sin(gs);
    n[g] = 0.5 * (1.0 + cg * cg);
    const double h = 0.5 * sg * sg, dh = sg * cg;
    if (jac) jac[(long long)g * ngam + g] = -cg * sg;
    double prod = 1.0;
    for (int i = 0; i < ncwo; ++i) {
      const int p = weak_index(g, i, npairs, ncwo, nsingle);
      const bool last = (i == ncwo - 1);
      const double gi = last ? 0.0 : gamma[npairs + g * (ncwo - 1) + i];
      const double si2 = last ? 1.0 : sin(gi) * sin(gi);
      n[p] = h * prod * si2;
      if (jac) {
        jac[(long long)p * ngam + g] = dh * prod * si2;
        // derivative w.r.t. the earlier weak variables j < i (cos^2 factors)
        for (int j = 0; j < i && j < ncwo - 1; ++j) {
          const double gj = gamma[npairs + g * (ncwo - 1) + j];
          double other = h * si2;
          for (int k = 0; k < i && k < ncwo - 1; ++k) {
            if (k == j) continue;
            const double gk = gamma[npairs + g * (ncwo - 1) + k];
            other *= cos(gk) * cos(gk);
          }
          jac[(long long)p * ngam + npairs + g * (ncwo - 1) + j] = other * (-2.0 * cos(gj) * sin(gj));
        }
        if (!last) jac[(long long)p * ngam + npairs + g * (ncwo - 1) + i] = h * prod * 2.0 * sin(gi) * cos(gi);
      }
      if (!last) prod *= cos(gi) * cos(gi);
    }
  }
}

// dE/dgamma = (dn/dgamma)^T dE/dn, pair by pair (the sigmoid variables of singly occupied orbitals
// do not enter: zero).
__global__ void on_map_vjp_k(int kind, int npairs, int ncwo, int nsingle, const double* __restrict__ gamma,
                             const double* __restrict__ dEdn, double* __restrict__ out) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g < npairs + nsingle) on_map_vjp_subspace(kind, npairs, ncwo, nsingle, gamma, dEdn, out, g);
}

// E(n(gamma)) and dE/dgamma at fixed H_pp, J, K.  Every block forms all of n itself (in LDS; from nglob where that
// does not fit); a wave sums dE/dn of a row p, and the terms of E are summed in energy_part's ON_EVAL_PARTS ranges, by a
// wave each where a range has at most 64 terms, otherwise by a block; the block that finishes last adds the ranges and
// takes dE/dn back through the map.  (Every sum runs in the order of the separate kernels: the optimisation amplifies a
// change in the last bits.)  Bound by its own latency and the launch: as a map, coefficients, two stages of the
// energy, gradient and adjoint launch by launch, with three copies, an evaluation at 24 orbitals took 60 us more.
constexpr int ON_EVAL_PARTS = 256;
__global__ __launch_bounds__(NT) void on_eval_k(int kind, int nact, int npairs, int ncwo, int nsingle, int functional, int ngam,
                                                const double* __restrict__ gamma, const double* __restrict__ nglob,
                                                const double* __restrict__ Hpp, const double* __restrict__ J,
                                                const double* __restrict__ K, double* __restrict__ epart,
                                                double* __restrict__ dEdn, unsigned* __restrict__ counter,
                                                double* __restrict__ out) {
  extern __shared__ double sh[];
  __shared__ bool s_last;
  const int t = threadIdx.x, lane = t & 63, wave = blockIdx.x * (NT / 64) + (t >> 6);
  const double *n = nglob, *gam = gamma;
  if (!nglob) {
    double* sg = sh + nact;
    for (int i = t; i < ngam; i += NT) sg[i] = gamma[i];
    for (int i = t; i < nsingle; i += NT) sh[npairs + i] = 0.5;
    __syncthreads();
    for (int g = t; g < npairs; g += NT) on_map_pair(kind, npairs, ncwo, nsingle, sg, sh, g);
    __syncthreads();
    n = sh;
    gam = sg;
  }
  if (wave < nact) grad_n_row(wave, nact, npairs, ncwo, nsingle, functional, n, Hpp, J, K, dEdn);
  const long long total = nact + (long long)nact * nact, per = (total + ON_EVAL_PARTS - 1) / ON_EVAL_PARTS;
  auto term = [&](long long i) {
    if (i < nact) return 2.0 * n[i] * Hpp[i];
    const long long k = i - nact;
    const int p = (int)(k / nact), q = (int)(k % nact);
    double a, b;
    pnof_coeff(p, q, n[p], n[q], npairs, ncwo, nsingle, functional, a, b);
    return a * J[k] + b * K[k];
  };
  if (per <= 64) {
    for (int part = wave; part < ON_EVAL_PARTS; part += gridDim.x * (NT / 64)) {
      const long long i = part * per + lane;
      double s = lane < per && i < total ? term(i) : 0.0;
      for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
      if (lane == 0) epart[part] = s;
    }
  } else {
    for (int part = blockIdx.x; part < ON_EVAL_PARTS; part += gridDim.x) {
      double s = 0.0;
      for (long long i = part * per + t; i < min(total, (part + 1) * per); i += NT) s += term(i);
      s = block_sum(s);
      if (t == 0) epart[part] = s;
    }
  }
  if (lane == 0) __threadfence();
  __syncthreads();
  if (t == 0) s_last = atomicAdd(counter, 1u) == gridDim.x - 1;
  __syncthreads();
  if (!s_last) return;
  __threadfence();
  double e = 0.0;
  for (int i = t; i < ON_EVAL_PARTS; i += NT) e += epart[i];
  e = block_sum(e);
  if (t == 0) {
    out[0] = e;
    *counter = 0;
  }
  for (int g = t; g < npairs + nsingle; g += NT) on_map_vjp_subspace(kind, npairs, ncwo, nsingle, gam, dEdn, out + 1, g);
}

// dst = src with a zero diagonal (the error vector of the DIIS extrapolation).
__global__ void offdiag_k(int nbf, const double* __restrict__ src, double* __restrict__ dst) {
  GRID_STRIDE(i, (long long)nbf * nbf) dst[i] = (i / nbf == i % nbf) ? 0.0 : src[i];
}

// Matrix diagonalised by the orbital step, and a copy of it in `keep` unless that is null.
__global__ void build_s_k(int nbf, const double* __restrict__ lam, const double* __restrict__ dprev, double zeta,
                          double* __restrict__ S, double* __restrict__ keep) {
  GRID_STRIDE(i, (long long)nbf * nbf) {
    const long long p = i / nbf, q = i % nbf;
    const double a = lam[p * nbf + q], b = lam[q * nbf + p];
    double v;
    if (!dprev) v = 0.5 * (a + b);
    else if (p == q) v = dprev[p];
    else {
      v = (p < q) ? (b - a) : (a - b);   // S_pq = lambda_qp - lambda_pq for p < q, mirrored
      if (zeta > 0.0)
        while (fabs(v) > zeta && isfinite(v)) v /= 10.0;
    }
    S[i] = v;
    if (keep) keep[i] = v;
  }
}

// Column j of the column-major eigenvector matrix: make its largest-|.| entry (lowest index on
// ties) positive.  One block per column.
__global__ void sign_fix_k(int nbf, double* __restrict__ U) {
  const int j = blockIdx.x;
  double* col = U + (long long)j * nbf;
  __shared__ double bv[NT];
  __shared__ int bi[NT];
  double best = -1.0;
  int idx = 0;
  for (int i = threadIdx.x; i < nbf; i += blockDim.x) {
    const double a = fabs(col[i]);
    if (a > best) { best = a; idx = i; }
  }
  bv[threadIdx.x] = best;
  bi[threadIdx.x] = idx;
  __syncthreads();
  for (int off = NT / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) {
      const double o = bv[threadIdx.x + off];
      const int oi = bi[threadIdx.x + off];
      if (o > bv[threadIdx.x] || (o == bv[threadIdx.x] && oi < bi[threadIdx.x])) {
        bv[threadIdx.x] = o;
        bi[threadIdx.x] = oi;
      }
    }
    __syncthreads();
  }
  const bool neg = col[bi[0]] < 0.0;
  __syncthreads();
  if (neg)
    for (int i = threadIdx.x; i < nbf; i += blockDim.x) col[i] = -col[i];
}

__global__ void nonfinite_k(const void* p, long long n, int is_bf16, int* flag) {
  int bad = 0;
  GRID_STRIDE(i, n) {
    double v = is_bf16 ? (double)bf16_bits_to_f32(reinterpret_cast<const u16*>(p)[i])
                       : reinterpret_cast<const double*>(p)[i];
    if (!isfinite(v)) bad = 1;
  }
  if (bad) atomicOr(flag, 1);
}

__global__ void gather_ao_k(int nbf, int nq, const int32_t* __restrict__ q_idx, const double* __restrict__ src,
                            double* __restrict__ dst) {
  const long long n2 = (long long)nbf * nbf;
  GRID_STRIDE(i, (long long)nq * n2) {
    const int k = (int)(i / n2);
    dst[i] = src[(long long)q_idx[k] * n2 + i % n2];
  }
}

__global__ void eri_fock_ao_k(int nbf, int nact, int nq, const int32_t* __restrict__ q_idx,
                              const double* __restrict__ n, const double* __restrict__ H,
                              const double* __restrict__ alpha, const double* __restrict__ beta,
                              const double* __restrict__ Jr, const double* __restrict__ Kr,
                              double* __restrict__ Fq) {
  const long long n2 = (long long)nbf * nbf;
  GRID_STRIDE(i, (long long)nq * n2) {
    const int k = (int)(i / n2);
    const long long e = i % n2;
    const int q = q_idx[k];
    double s = n[q] * H[e];
    for (int r = 0; r < nact; ++r)
      s += alpha[(long long)q * nact + r] * Jr[(long long)r * n2 + e] + beta[(long long)q * nact + r] * Kr[(long long)r * n2 + e];
    Fq[i] = s;
  }
}

__global__ void fock_ao_h_k(int nbf, int nq, const int32_t* __restrict__ q_idx, const double* __restrict__ n,
                            const double* __restrict__ H, double* __restrict__ Fq) {
  const long long n2 = (long long)nbf * nbf;
  GRID_STRIDE(i, (long long)nq * n2) {
    const int k = (int)(i / n2);
    Fq[i] += n[q_idx[k]] * H[i % n2];
  }
}

}  // namespace

#define LAUNCH(kern, grid, block, ...)                              \
  do {                                                              \
    hipLaunchKernelGGL(kern, grid, block, 0, s, __VA_ARGS__);       \
    return hipGetLastError();                                       \
  } while (0)

hipError_t fill_f64(hipStream_t s, double* p, long long n, double v) {
  if (n <= 0) return hipSuccess;
  LAUNCH(fill_f64_k, grid1(n), dim3(NT), p, n, v);
}
hipError_t on_eval(hipStream_t s, int kind, int nact, int npairs, int ncwo, int nsingle, int functional, int ngam,
                   const double* gamma, const double* Hpp, const double* J, const double* K, double* nbuf, double* epart,
                   double* dEdn, unsigned* counter, double* out) {
  const size_t lds = sizeof(double) * (size_t)(nact + ngam);
  const bool fits = lds <= 60 * 1024;
  if (!fits) {
    const hipError_t e = on_map(s, kind, npairs, ncwo, nsingle, gamma, nbuf, nullptr);
    if (e != hipSuccess) return e;
  }
  // a wave per row of dE/dn, and per range of E
  const int nb = std::max((int)cdiv(nact, NT / 64), ON_EVAL_PARTS / (NT / 64));
  hipLaunchKernelGGL(on_eval_k, dim3((unsigned)nb), dim3(NT), fits ? lds : 0, s, kind, nact, npairs, ncwo,
                     nsingle, functional, ngam, gamma, fits ? nullptr : nbuf, Hpp, J, K, epart, dEdn, counter, out);
  return hipGetLastError();
}
hipError_t coeffs(hipStream_t s, int nact, int npairs, int ncwo, int nsingle, int functional, const double* n,
                  double* alpha, double* beta, float* beta32, int ld32) {
  const long long w = beta32 ? ld32 : nact;
  LAUNCH(coeffs_k, grid1(w * w), dim3(NT), nact, ld32, npairs, ncwo, nsingle, functional, n, alpha, beta, beta32);
}
template <typename T>
hipError_t transpose_ca(hipStream_t s, int nbf, int nact, const double* C, T* Ct, int ldk) {
  LAUNCH(transpose_ca_k<T>, grid1((long long)nbf * nact), dim3(NT), nbf, nact, C, Ct, ldk);
}
template hipError_t transpose_ca<double>(hipStream_t, int, int, const double*, double*, int);
template hipError_t transpose_ca<float>(hipStream_t, int, int, const double*, float*, int);
hipError_t add_diag_f32(hipStream_t s, int nact, int np, const double* Dc, const OccLayout& oc, double* dbuf, float* W,
                        int ldw) {
  if (np <= 0) return hipSuccess;
  hipLaunchKernelGGL(d_alpha_k, dim3(np), dim3(NT), 0, s, nact, oc.npairs, oc.ncwo, oc.nsingle, oc.n, Dc, dbuf);
  LAUNCH(add_diag_f32_k, grid1((long long)np * nact), dim3(NT), nact, np, 1, dbuf, W, ldw);
}
hipError_t split_ca(hipStream_t s, int nbf, int nact, int rows, int terms, const double* C, u16* hi, u16* lo, u16* h16,
                    u16* l16, int ldk, const uint32_t* bnd) {
  LAUNCH(split_ca_k, grid1((long long)rows * ldk), dim3(NT), nbf, nact, rows, terms, C, hi, lo, h16, l16, ldk, bnd);
}
hipError_t split_b(hipStream_t s, long long nrows, int n, const double* B, u16* hi, u16* lo, int ldo, const uint32_t* bnd,
                   int chunk) {
  if (nrows <= 0) return hipSuccess;
  if (ldo != n && ldo % 8 != 0) return hipErrorInvalidValue;
  // 32-bit piece counts: rows in parts of at most 2^29 pieces, each starting on a whole piece
  const long long part = std::max(1LL, (1LL << 29) / (ldo / 8 + 1)) & ~7LL;
  if (part == 0) return hipErrorInvalidValue;
  for (long long r0 = 0; r0 < nrows; r0 += part) {
    const long long nr = std::min(part, nrows - r0), pieces = (nr * ldo + 7) / 8;
    hipLaunchKernelGGL(split_b_k, dim3((unsigned)std::min<long long>(cdiv(pieces, NT), 16384)), dim3(NT), 0, s, nr * n,
                       (uint32_t)pieces, n, B + r0 * n, hi + r0 * ldo, lo ? lo + r0 * ldo : nullptr, ldo, bnd, chunk);
  }
  return hipGetLastError();
}
hipError_t scale_bounds(hipStream_t s, int nbf, int nact, const double* C, const double* n, int npairs, int ncwo,
                        int nsingle, int functional, float* col, uint32_t* bnd, int nclear) {
  hipLaunchKernelGGL(col_bounds_k, dim3((unsigned)cdiv(nact, NT / 64)), dim3(NT), 0, s, nbf, nact, C, n, npairs, ncwo,
                     nsingle, functional, col);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  LAUNCH(bounds_reduce_k, dim3(1), dim3(NT), nact, col, bnd, nclear);
}
// Lanes per row: the fewest (8 to 64) whose 16-byte pieces cover the row in one go.
template <typename T, bool BND, bool PACK>
static hipError_t b_rows(hipStream_t s, const T* B, long long nrows, int n, long long rows_per_chunk, uint32_t* slot,
                         u16* out, int ldo) {
  const int pieces = cdiv(PACK ? ldo : n, 16 / (int)sizeof(T));
  const int lpr = pieces <= 8 ? 8 : pieces <= 16 ? 16 : pieces <= 32 ? 32 : 64;
  const long long nch = cdiv(nrows, rows_per_chunk);
  if (nch > 65535) return hipErrorInvalidValue;
  // about 4096 blocks over the chunks, each with whole passes of its rows
  const long long per = std::min(nrows, rows_per_chunk);
  const long long bx = std::min<long long>(cdiv(per, (NT / lpr) * RU), std::max(1LL, 4096 / nch));
  const dim3 g((unsigned)bx, (unsigned)nch);
  if (lpr == 8) hipLaunchKernelGGL((b_rows_k<T, 8, BND, PACK>), g, dim3(NT), 0, s, B, nrows, n, rows_per_chunk, slot, out, ldo);
  else if (lpr == 16) hipLaunchKernelGGL((b_rows_k<T, 16, BND, PACK>), g, dim3(NT), 0, s, B, nrows, n, rows_per_chunk, slot, out, ldo);
  else if (lpr == 32) hipLaunchKernelGGL((b_rows_k<T, 32, BND, PACK>), g, dim3(NT), 0, s, B, nrows, n, rows_per_chunk, slot, out, ldo);
  else hipLaunchKernelGGL((b_rows_k<T, 64, BND, PACK>), g, dim3(NT), 0, s, B, nrows, n, rows_per_chunk, slot, out, ldo);
  return hipGetLastError();
}
hipError_t b_bounds(hipStream_t s, const void* B, int is_f64, long long nrows, int n, long long rows_per_chunk,
                    uint32_t* slot) {
  if (nrows <= 0) return hipSuccess;
  // the grid's second dimension holds at most 65535 chunks
  const long long part = 65535 * rows_per_chunk;
  for (long long r0 = 0; r0 < nrows; r0 += part) {
    const long long nr = std::min(part, nrows - r0);
    const hipError_t e = is_f64 ? b_rows<double, true, false>(s, static_cast<const double*>(B) + r0 * n, nr, n,
                                                              rows_per_chunk, slot, nullptr, 0)
                                : b_rows<u16, true, false>(s, static_cast<const u16*>(B) + r0 * n, nr, n, rows_per_chunk,
                                                           slot, nullptr, 0);
    if (e != hipSuccess) return e;
    slot += 2 * 65535;
  }
  return hipSuccess;
}
hipError_t pack_b(hipStream_t s, long long nrows, int n, const u16* B, u16* out, int ldo, uint32_t* slot) {
  if (nrows <= 0) return hipSuccess;
  return slot ? b_rows<u16, true, true>(s, B, nrows, n, nrows, slot, out, ldo)
              : b_rows<u16, false, true>(s, B, nrows, n, nrows, slot, out, ldo);
}
hipError_t hpp_from_hc(hipStream_t s, int nbf, int nact, const double* C, const double* HC, double* Hpp) {
  LAUNCH(hpp_k, dim3(nact), dim3(64), nbf, nact, C, HC, Hpp);
}
hipError_t add_diag_f64(hipStream_t s, int nact, int np, const double* Dc, const OccLayout& oc, double* dbuf,
                        double* W, int ldw) {
  if (np <= 0) return hipSuccess;
  hipLaunchKernelGGL(d_alpha_k, dim3(np), dim3(NT), 0, s, nact, oc.npairs, oc.ncwo, oc.nsingle, oc.n, Dc, dbuf);
  LAUNCH(add_diag_f64_k, grid1((long long)np * nact), dim3(NT), nact, np, 1, dbuf, W, ldw);
}
hipError_t add_diag_bf16(hipStream_t s, int nact, int np, const double* Dc, const OccLayout& oc, const float* beta32,
                         double* dbuf, u16* Wh, u16* Wl, int ldw, long long pstride, const uint32_t* bnd, int chunk) {
  if (np <= 0) return hipSuccess;
  hipLaunchKernelGGL(d_alpha_k, dim3(np), dim3(NT), 0, s, nact, oc.npairs, oc.ncwo, oc.nsingle, oc.n, Dc, dbuf);
  LAUNCH(add_diag_bf16_k, grid1((long long)np * nact), dim3(NT), nact, np, 1, dbuf, Dc, beta32, Wh, Wl, ldw, pstride,
         bnd, chunk);
}
hipError_t nofmp2_terms(hipStream_t s, int nact, int npairs, int ncwo, int nsingle, const double* n,
                        const double* Hpp, const double* J, const double* K, double* partials, double* E_hf,
                        double* E_sta) {
  const int nb = 128;   // partials holds 2 * nb doubles
  hipLaunchKernelGGL(nofmp2_stage1_k, dim3(nb), dim3(NT), 0, s, nact, npairs, ncwo, nsingle, n, Hpp, J, K, partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  LAUNCH(sum2_partials_k, dim3(1), dim3(NT), nb, partials, E_hf, E_sta);
}
hipError_t offdiag_copy(hipStream_t s, int nbf, const double* src, double* dst) {
  LAUNCH(offdiag_k, grid1((long long)nbf * nbf), dim3(NT), nbf, src, dst);
}
hipError_t reduce_k(hipStream_t s, int nact, int nsplit, const double* Kpart, double* K) {
  const long long n2 = (long long)nact * nact;
  if (nsplit >= RED_SPLITS) LAUNCH(reduce_k_k<RED_PARTS>, dim3((unsigned)cdiv(n2, 64)), dim3(64 * RED_PARTS), nact, nsplit, Kpart, K);
  LAUNCH(reduce_k_k<1>, dim3((unsigned)cdiv(n2, NT)), dim3(NT), nact, nsplit, Kpart, K);
}
template <typename T>
static hipError_t reduce_y(hipStream_t s, long long n, int nsplit, int first, const T* Yp, double* Y) {
  if (nsplit >= RED_SPLITS)
    LAUNCH((reduce_y_k<RED_PARTS, T>), dim3((unsigned)cdiv(n, 64)), dim3(64 * RED_PARTS), n, nsplit, first, Yp, Y);
  LAUNCH((reduce_y_k<1, T>), dim3((unsigned)cdiv(n, NT)), dim3(NT), n, nsplit, first, Yp, Y);
}
hipError_t reduce_y_f64(hipStream_t s, long long n, int nsplit, int first, const double* Yp, double* Y) {
  return reduce_y(s, n, nsplit, first, Yp, Y);
}
hipError_t reduce_y_f32(hipStream_t s, long long n, int nsplit, int first, const float* Yp, double* Y) {
  return reduce_y(s, n, nsplit, first, Yp, Y);
}
hipError_t energy(hipStream_t s, int nbf, int nact, const double* n, const double* Hpp,
                  const double* alpha, const double* beta, const double* J, const double* K,
                  const double* Y2e, const double* C, const u16* cth, const u16* ctl, const float* ct32, int ldk,
                  int corr_terms, double* partials, double* E) {
  const int nb = 256;
  const EnergyArgs a{nbf, nact, n, Hpp, alpha, beta, J, K, Y2e, C, cth, ctl, ct32, ldk, corr_terms};
  hipLaunchKernelGGL(energy_stage1_k, dim3(nb), dim3(NT), 0, s, a, partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  LAUNCH(sum_partials_k, dim3(1), dim3(NT), nb, partials, E);
}
static int tail_parts(int nbf, int nact, int corr_terms) {   // 256 blocks at most, of 1024 terms at least
  const long long total = nact + (long long)nact * nact + (corr_terms > 0 ? (long long)nbf * nact : 0);
  return (int)std::min(256LL, (total + 1023) / 1024);
}
hipError_t step_tail(hipStream_t s, int nbf, int nact, int npairs, int ncwo, int nsingle, int functional, const double* n,
                     const double* Hpp, const double* alpha, const double* beta, const double* J, const double* K,
                     const double* HC, const double* Y2e, const double* C, const u16* cth, const u16* ctl, const float* ct32,
                     int ldk, int corr_terms, double* partials, double* Y, double* dEdn, double* lam, double* asym) {
  TailArgs a{{nbf, nact, n, Hpp, alpha, beta, J, K, Y2e, C, cth, ctl, ct32, ldk, corr_terms}, 0, 0, npairs, ncwo, nsingle,
             functional, HC, partials, dEdn, Y, lam, asym};
  a.ne = partials ? tail_parts(nbf, nact, corr_terms) : 0;
  a.ng = dEdn ? cdiv(nact, NT / 64) : 0;
  const unsigned nel = Y ? grid1((long long)nbf * (lam ? nbf : nact)).x : 0;
  if (a.ne + a.ng + nel == 0) return hipSuccess;
  LAUNCH(step_tail_k, dim3(a.ne + a.ng + nel), dim3(NT), a);
}
hipError_t step_end(hipStream_t s, int nbf, int nact, int corr_terms, const double* partials, double* E, const double* lam,
                    double* asym, const double* Y, double* dEdC) {
  const int ne = partials ? tail_parts(nbf, nact, corr_terms) : 0;
  const unsigned na = asym ? (unsigned)std::min(256LL, ((long long)nbf * nbf + NT - 1) / NT) : 0;
  const unsigned nd = dEdC ? grid1((long long)nbf * nbf).x : 0;
  if (ne + na + nd == 0) return hipSuccess;
  LAUNCH(step_end_k, dim3(1 + na + nd), dim3(NT), ne, (int)na, partials, E, nbf, nact, lam, asym, Y, dEdC);
}
hipError_t on_map(hipStream_t s, int kind, int npairs, int ncwo, int nsingle, const double* gamma, double* n,
                  double* jac) {
  LAUNCH(on_map_k, dim3(cdiv(std::max(npairs, nsingle), 64)), dim3(64), kind, npairs, ncwo, nsingle, gamma, n, jac);
}
hipError_t on_map_vjp(hipStream_t s, int kind, int npairs, int ncwo, int nsingle, const double* gamma,
                      const double* dEdn, double* out) {
  LAUNCH(on_map_vjp_k, dim3(cdiv(npairs + nsingle, 64)), dim3(64), kind, npairs, ncwo, nsingle, gamma, dEdn, out);
}
hipError_t build_s(hipStream_t s, int nbf, const double* lam, const double* dprev, double zeta, double* S, double* keep) {
  LAUNCH(build_s_k, grid1((long long)nbf * nbf), dim3(NT), nbf, lam, dprev, zeta, S, keep);
}
hipError_t sign_fix_cols(hipStream_t s, int nbf, double* U) {
  LAUNCH(sign_fix_k, dim3(nbf), dim3(NT), nbf, U);
}
hipError_t count_nonfinite(hipStream_t s, const void* p, long long n, int is_bf16, int* flag) {
  if (n <= 0) return hipSuccess;
  LAUNCH(nonfinite_k, grid1(n), dim3(NT), p, n, is_bf16, flag);
}
hipError_t gather_ao(hipStream_t s, int nbf, int nq, const int32_t* q_idx, const double* src, double* dst) {
  if (nq <= 0) return hipSuccess;
  LAUNCH(gather_ao_k, grid1((long long)nq * nbf * nbf), dim3(NT), nbf, nq, q_idx, src, dst);
}
hipError_t eri_fock_ao(hipStream_t s, int nbf, int nact, int nq, const int32_t* q_idx, const double* n,
                       const double* H, const double* alpha, const double* beta, const double* Jr,
                       const double* Kr, double* Fq) {
  if (nq <= 0) return hipSuccess;
  LAUNCH(eri_fock_ao_k, grid1((long long)nq * nbf * nbf), dim3(NT), nbf, nact, nq, q_idx, n, H, alpha, beta, Jr, Kr, Fq);
}
hipError_t fock_ao_h(hipStream_t s, int nbf, int nq, const int32_t* q_idx, const double* n, const double* H,
                     double* Fq) {
  if (nq <= 0) return hipSuccess;
  LAUNCH(fock_ao_h_k, grid1((long long)nq * nbf * nbf), dim3(NT), nbf, nq, q_idx, n, H, Fq);
}

}  // namespace pnof
