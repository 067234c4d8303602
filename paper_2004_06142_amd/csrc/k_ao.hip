// Per-orbital AO matrices (float64): J^r and K^r of explicit four-index integrals (at most 64 functions) with what
// the step forms from them, and J^q, K^q, F^q of the requested orbitals from density-fitted chunks.
#include "common.h"

namespace pnof {
namespace {

constexpr int NT = 256;

// ---- explicit four-index integrals ----
// Jr[r][m][n] = sum_ls (mn|ls) C_lr C_sr ; Kr[r][m][n] = sum_ls (ml|ns) C_lr C_sr (Eq. Gpmn), from the half
// transformation T[a][b] = sum_s (ma|bs) C_sr of one m: J^r_mn = sum_l T[n][l] C_lr, K^r_mn = sum_l T[l][n] C_lr.
// One block per m and two r; (ma|..) goes through LDS in tiles of 128 pairs (a, b), the next tile's loads in
// flight.  Bound by the latency of its five tiles at 24 functions.  As one thread per (r, m, n), each with the
// whole double sum, 24 functions took 130 us; here 11.5.
template <int MX>
__global__ __launch_bounds__(NT) void eri_jk_ao_k(int nbf, int nact, const double* __restrict__ ERI,
                                                  const double* __restrict__ C, double* __restrict__ Jr,
                                                  double* __restrict__ Kr) {
  constexpr int TP = 128, PER = TP * MX / NT;
  __shared__ double T[2][MX * (MX + 1)], st[TP * (MX + 1)], c[2][MX];
  const int t = threadIdx.x, m = blockIdx.x, r0 = 2 * blockIdx.y, pitch = nbf + 1 - (nbf & 1);   // odd
  const int pairs = nbf * nbf;
  if (t < 2 * nbf) {
    const int k = t / nbf, s = t % nbf;
    c[k][s] = r0 + k < nact ? C[(long long)s * nbf + r0 + k] : 0.0;
  }
  const double* __restrict__ src = ERI + (long long)m * pairs * nbf;
  const int rstep = NT / nbf, row0 = t / nbf, col = t % nbf;   // rows of a tile that one pass of the block takes
  double v[PER + 1];
  auto load = [&](int p0) {
#pragma unroll
    for (int j = 0; j <= PER; ++j) {
      const int row = row0 + j * rstep;
      v[j] = row0 < rstep && row < TP && p0 + row < pairs ? src[(long long)(p0 + row) * nbf + col] : 0.0;
    }
  };
  load(0);
  for (int p0 = 0; p0 < pairs; p0 += TP) {
#pragma unroll
    for (int j = 0; j <= PER; ++j) {
      const int row = row0 + j * rstep;
      if (row0 < rstep && row < TP) st[row * pitch + col] = v[j];
    }
    __syncthreads();
    if (p0 + TP < pairs) load(p0 + TP);
    const int row = t & (TP - 1), k = t / TP;
    if (p0 + row < pairs) {
      double s = 0.0;
      for (int u = 0; u < nbf; ++u) s += st[row * pitch + u] * c[k][u];
      T[k][(p0 + row) / nbf * pitch + (p0 + row) % nbf] = s;
    }
    __syncthreads();
  }
  for (int o = t; o < 4 * nbf; o += NT) {
    const int n = o % nbf, k = (o / nbf) & 1, ex = o / (2 * nbf);
    if (r0 + k >= nact) continue;
    const double* x = T[k] + (ex ? n : n * pitch);
    const int step = ex ? pitch : 1;
    double s = 0.0;
    for (int l = 0; l < nbf; ++l) s += c[k][l] * x[l * step];
    (ex ? Kr : Jr)[((long long)(r0 + k) * nbf + m) * nbf + n] = s;
  }
}

// Blocks q < nact: J_pq = c_p^T J^q c_p, K_pq = c_p^T K^q c_p (Eq. JKpq).  Blocks nact + m: row m of
// Y2e[m][q] = sum_r (alpha_qr J^r + beta_qr K^r) c_q.  Matrices in LDS; the threads of one p (or q) share the
// rows (or r) between them, and one adds their products in order (an optimisation of the occupations amplifies
// a change in the last bits of J and K).  As one thread per element 24 functions took 77 + 27 us; here 4.4.
template <int MX>
__global__ __launch_bounds__(NT) void eri_no_k(int nbf, int nact, const double* __restrict__ C, const double* __restrict__ alpha,
                                               const double* __restrict__ beta, const double* __restrict__ Jr,
                                               const double* __restrict__ Kr, double* __restrict__ J, double* __restrict__ K,
                                               double* __restrict__ Y2e) {
  __shared__ double js[MX * MX], ks[MX * MX], cs[MX * MX], tj_[MX * MX], tk_[MX * MX];
  const int t = threadIdx.x;
  const bool no = (int)blockIdx.x < nact;
  const int id = no ? blockIdx.x : blockIdx.x - nact, rows = no ? nbf : nact;   // js: rows of nbf
  for (int i = t; i < rows * nbf; i += NT) {
    const long long o = no ? (long long)id * nbf * nbf + i : ((long long)(i / nbf) * nbf + id) * nbf + i % nbf;
    js[i] = Jr[o];
    ks[i] = Kr[o];
  }
  for (int i = t; i < nbf * nact; i += NT) cs[i] = C[(long long)(i / nact) * nbf + i % nact];
  __syncthreads();
  const int parts = NT / nact, p = t % nact, part = t / nact;
  if (part < parts)
    for (int m = part; m < rows; m += parts) {
      double tj = 0.0, tk = 0.0;
      for (int n = 0; n < nbf; ++n) {
        tj += js[m * nbf + n] * cs[n * nact + p];
        tk += ks[m * nbf + n] * cs[n * nact + p];
      }
      tj_[m * nact + p] = tj;
      tk_[m * nact + p] = tk;
    }
  __syncthreads();
  if (t >= nact) return;
  double sj = 0.0, sk = 0.0;
  for (int m = 0; m < rows; ++m) {
    const double tj = tj_[m * nact + t], tk = tk_[m * nact + t];
    if (no) {
      sj += cs[m * nact + t] * tj;
      sk += cs[m * nact + t] * tk;
    } else {
      sj += alpha[(long long)t * nact + m] * tj + beta[(long long)t * nact + m] * tk;
    }
  }
  if (no) {
    J[(long long)t * nact + id] = sj;
    K[(long long)t * nact + id] = sk;
  } else Y2e[(long long)id * nact + t] = sj;
}

// ---- density-fitted chunks ----
// J^q += sum_P D_Pq B_P,  K^q += sum_P x_Pq x_Pq^T,  F^q += sum_P [d_Pq B_P + sum_r beta_qr x_Pr x_Pr^T] with
// x_Pr[mu] = XT[P][r][mu], d_Pq = sum_r alpha_qr D_Pr (first: = in place of +=).
struct Xt {   // XT as float64, float32, one bf16 value, or the fp16 pair of X sX (invX = 1 / sX)
  const double* d;
  const float* f;
  const u16* hi;
  const u16* lo;
  double invX;
  __device__ __forceinline__ double at(long long o) const {
    if (d) return d[o];
    if (f) return (double)f[o];
    if (!lo) return (double)bf16_bits_to_f32(hi[o]);
    return ((double)f16_bits_to_f32(hi[o]) + (double)f16_bits_to_f32(lo[o])) * invX;
  }
  // v = x[o .. o + 3], zero from `left` on
  __device__ __forceinline__ void at4(long long o, int left, double (&v)[4]) const {
    if (d && left >= 4) {
      __builtin_memcpy(v, d + o, 32);
      return;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = u < left ? at(o + u) : 0.0;
  }
};

// The B_P terms of up to 8 sums (k: J of request k, nq + k: F of request k).  A wave sums every eighth row over 128
// elements of B, so that B is read once, in whole lines, by enough waves; the waves' sums meet in LDS.  Bound by
// reading B: J of 8 orbitals, 400 rows of 200 functions in float64 (128 MB) 46 us; as one thread per element and
// orbital, with K, 248 us.
constexpr int AO_W = 8, AO_P = 128, AO_NW = 8;
template <typename SB>
__global__ __launch_bounds__(64 * AO_NW) void ao_b_k(int nbf, int nact, int np, int nq, const int32_t* __restrict__ q_idx, int w0,
                                             int nw, const SB* __restrict__ Bc, const double* __restrict__ Dc,
                                             const double* __restrict__ alpha, double* __restrict__ Jq,
                                             double* __restrict__ Fq, int first) {
  __shared__ double w[AO_P][AO_W], red[AO_NW - 1][64][2 * AO_W];
  const long long n2 = (long long)nbf * nbf;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const long long e = (long long)blockIdx.x * 128 + 2 * lane;
  double acc[AO_W][2] = {};
  for (int p0 = 0; p0 < np; p0 += AO_P) {
    const int pc = min(AO_P, np - p0);
    __syncthreads();
    for (int i = t; i < pc * AO_W; i += 64 * AO_NW) {
      const int P = i / AO_W, k = w0 + i % AO_W;
      const double* __restrict__ Dp = Dc + (long long)(p0 + P) * nact;
      double x = 0.0;
      if (i % AO_W < nw) {
        const int q = q_idx[k % nq];
        if (Jq && k < nq) x = Dp[q];
        else
          for (int r = 0; r < nact; ++r) x += alpha[(long long)q * nact + r] * Dp[r];
      }
      w[P][i % AO_W] = x;
    }
    __syncthreads();
    const SB* __restrict__ src = Bc + (long long)p0 * n2 + e;
#pragma unroll 4
    for (int P = wave; P < pc; P += AO_NW) {
      SB v[2] = {};
      if (e + 1 < n2) __builtin_memcpy(v, src + P * n2, sizeof(v));
      else if (e < n2) v[0] = src[P * n2];
      double b0, b1;
      if constexpr (sizeof(SB) == 2) {
        b0 = (double)bf16_bits_to_f32(v[0]);
        b1 = (double)bf16_bits_to_f32(v[1]);
      } else {
        b0 = v[0];
        b1 = v[1];
      }
#pragma unroll
      for (int k = 0; k < AO_W; ++k) {
        acc[k][0] += w[P][k] * b0;
        acc[k][1] += w[P][k] * b1;
      }
    }
  }
  if (wave) {
#pragma unroll
    for (int k = 0; k < AO_W; ++k) {
      red[wave - 1][lane][2 * k] = acc[k][0];
      red[wave - 1][lane][2 * k + 1] = acc[k][1];
    }
  }
  __syncthreads();
  if (wave) return;
#pragma unroll
  for (int k = 0; k < AO_W; ++k) {
    if (k >= nw) break;
    const int c = w0 + k;
    double* __restrict__ out = (Jq && c < nq ? Jq : Fq) + (long long)(c % nq) * n2;
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (e + u < n2) {
        double s = acc[k][u];
#pragma unroll
        for (int v = 0; v < AO_NW - 1; ++v) s += red[v][lane][2 * k + u];
        out[e + u] = first ? s : out[e + u] + s;
      }
  }
}

// The products of x: C^k += sum over (P, r) of w_r x_Pr x_Pr^T, r = q and w = 1 (K), or every r with w = beta_qr (F).
// 64 x 64 tiles on and below the diagonal by v_mfma_f64_16x16x4, 32 terms (P, r) per slab, the next slab in
// registers; stored with its image.  K of 8 orbitals at 200 functions fills 80 blocks: bound by the length of one
// (400 rows: 16 terms per slab 42 us, 32 35 us).
constexpr int AT = 64, AK = 32, APITCH = AT + 8;
template <bool FOCK>
__global__ __launch_bounds__(NT) void ao_x_k(int nbf, int nact, int np, const int32_t* __restrict__ q_idx,
                                             const double* __restrict__ beta, Xt x, const uint32_t* __restrict__ bnd,
                                             int chunk, int ldx, long long xps, double* __restrict__ out, int first) {
  __shared__ double sa[2][AK * APITCH], sb[2][AK * APITCH];
  if (x.lo) x.invX = (double)chunk_scales(bnd, chunk, false).invX;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int tm = 0, tn = blockIdx.x;
  while (tn > tm) tn -= ++tm;   // tile (tm, tn <= tm) of the lower triangle
  const int m0 = tm * AT, n0 = tn * AT, wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int q = q_idx[blockIdx.y], per = FOCK ? nact : 1, total = np * per, slabs = (total + AK - 1) / AK;
  const int kr = t >> 4, c0 = 4 * (t & 15);   // this thread's terms (kr, kr + 16) and columns of a slab
  double va[2][4], vb[2][4];
  auto load = [&](int sl) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = sl * AK + kr + 16 * h, P = k / per, r = FOCK ? k - P * per : q;
      const bool in = k < total;
      const long long o = (long long)(in ? P : 0) * xps + (long long)(in ? r : 0) * ldx;
      x.at4(o + m0 + c0, in ? nbf - m0 - c0 : 0, va[h]);
      x.at4(o + n0 + c0, in ? nbf - n0 - c0 : 0, vb[h]);
      if (FOCK) {
        const double w = in ? beta[(long long)q * nact + r] : 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) va[h][u] *= w;
      }
    }
  };
  auto store = [&](int st) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        sa[st][(kr + 16 * h) * APITCH + c0 + u] = va[h][u];
        sb[st][(kr + 16 * h) * APITCH + c0 + u] = vb[h][u];
      }
  };
  f64x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  load(0);
  store(0);
  if (slabs > 1) load(1);
  __syncthreads();
  for (int sl = 0; sl < slabs; ++sl) {
    const int st = sl & 1;
    if (sl + 1 < slabs) {
      store(st ^ 1);
      if (sl + 2 < slabs) load(sl + 2);
    }
#pragma unroll
    for (int s = 0; s < AK / 4; ++s) {
      double a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = sa[st][(4 * s + (lane >> 4)) * APITCH + wm + 16 * i + (lane & 15)];
        b[i] = sb[st][(4 * s + (lane >> 4)) * APITCH + wn + 16 * i + (lane & 15)];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  double* __restrict__ o = out + (long long)blockIdx.y * nbf * nbf;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + wm + 16 * i + (lane >> 4) + 4 * e, n = n0 + wn + 16 * j + (lane & 15);
        if (m >= nbf || n > m) continue;
        const double v = acc[i][j][e];
        double* lo = o + (long long)m * nbf + n;
        double* up = o + (long long)n * nbf + m;
        const double y = first ? v : *lo + v;
        if (m != n) *up = first ? v : *up + v;
        *lo = y;
      }
}

}  // namespace

hipError_t eri_jk_ao(hipStream_t s, int nbf, int nact, const double* ERI, const double* C, double* Jr, double* Kr) {
  const dim3 grid(nbf, cdiv(nact, 2));
  if (nbf <= 32) hipLaunchKernelGGL(eri_jk_ao_k<32>, grid, dim3(NT), 0, s, nbf, nact, ERI, C, Jr, Kr);
  else if (nbf <= 64) hipLaunchKernelGGL(eri_jk_ao_k<64>, grid, dim3(NT), 0, s, nbf, nact, ERI, C, Jr, Kr);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t eri_no(hipStream_t s, int nbf, int nact, const double* C, const double* alpha, const double* beta,
                  const double* Jr, const double* Kr, double* J, double* K, double* Y2e) {
  if (nact > nbf) return hipErrorInvalidValue;
  const dim3 grid(nact + (Y2e ? nbf : 0));
  if (nbf <= 32) hipLaunchKernelGGL(eri_no_k<32>, grid, dim3(NT), 0, s, nbf, nact, C, alpha, beta, Jr, Kr, J, K, Y2e);
  else if (nbf <= 64) hipLaunchKernelGGL(eri_no_k<64>, grid, dim3(NT), 0, s, nbf, nact, C, alpha, beta, Jr, Kr, J, K, Y2e);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t df_ao_accum(hipStream_t s, int nbf, int nact, int np, int nq, const int32_t* q_idx, const void* Bchunk,
                       int b_is_bf16, const double* Dchunk, const double* alpha, const double* beta, const double* XT,
                       const float* XT32, const u16* XT_hi, const u16* XT_lo, int ldx, long long xps, double* Jq, double* Kq,
                       double* Fq, const uint32_t* bnd, int chunk, int first) {
  if (nq <= 0 || np <= 0) return hipSuccess;
  const dim3 blk(NT);
  // sums over B_P: columns 0 .. nq - 1 are J's, nq .. 2 nq - 1 F's
  const int c0 = Jq ? 0 : nq, c1 = Fq ? 2 * nq : nq;
  const dim3 gb((unsigned)cdiv((long long)nbf * nbf, 128));
  for (int w0 = c0; w0 < c1; w0 += AO_W) {
    const int nw = c1 - w0 < AO_W ? c1 - w0 : AO_W;
    if (b_is_bf16)
      hipLaunchKernelGGL(ao_b_k<u16>, gb, dim3(64 * AO_NW), 0, s, nbf, nact, np, nq, q_idx, w0, nw, static_cast<const u16*>(Bchunk), Dchunk,
                         alpha, Jq, Fq, first);
    else
      hipLaunchKernelGGL(ao_b_k<double>, gb, dim3(64 * AO_NW), 0, s, nbf, nact, np, nq, q_idx, w0, nw, static_cast<const double*>(Bchunk),
                         Dchunk, alpha, Jq, Fq, first);
  }
  const Xt x{XT, XT32, XT_hi, XT_lo, 1.0};
  const int tm = (int)cdiv(nbf, AT);
  for (int q0 = 0; q0 < nq; q0 += 65535) {
    const dim3 gx((unsigned)(tm * (tm + 1) / 2), (unsigned)(nq - q0 < 65535 ? nq - q0 : 65535));
    const long long oq = (long long)q0 * nbf * nbf;
    if (Kq) hipLaunchKernelGGL(ao_x_k<false>, gx, blk, 0, s, nbf, nact, np, q_idx + q0, beta, x, bnd, chunk, ldx, xps, Kq + oq, first);
    if (Fq) hipLaunchKernelGGL(ao_x_k<true>, gx, blk, 0, s, nbf, nact, np, q_idx + q0, beta, x, bnd, chunk, ldx, xps, Fq + oq, 0);
  }
  return hipGetLastError();
}

}  // namespace pnof
