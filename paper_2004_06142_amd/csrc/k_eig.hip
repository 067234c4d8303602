// Householder reduction of a symmetric float64 matrix to tridiagonal form: the last 1024 columns in one
// launch (trd_reduce_k, below), the columns before them one kernel each (trd_step_k, described here).
//
// The orbital step diagonalises an n x n symmetric matrix every iteration (n = 1200 at the largest
// workload).  The reduction is a chain of n dependent steps, so its cost is per-step latency, not
// bandwidth.  Each step here is a single launch: it applies the previous step's rank-2 update to
// the rows it owns and, in the same pass over each row, accumulates that row's product with the new
// Householder vector.  The update is never a separate kernel, and no step reads the matrix twice.
//
// Step k (0 <= k < n), with v_{k-1}, tau_{k-1} and p_{k-1} = tau_{k-1} A v_{k-1} from step k - 1:
//   w_{k-1} = p_{k-1} - (tau_{k-1} / 2) (p_{k-1} . v_{k-1}) v_{k-1};
//   c = row k of A with the pending update A -= v w^T + w v^T applied (A is symmetric, so row k is
//       column k); d_k = c_k;
//   Householder vector of c_{k+1..n-1}: v_k (v_k[k+1] = 1), tau_k, e_k = beta (LAPACK's dlarfg
//       convention: beta = -sign(alpha) |c_{k+1..}|, tau = (beta - alpha) / beta; tau = 0 when the
//       column below the subdiagonal is already zero);
//   rows i > k: apply the pending update, store, p_k[i] = tau_k (row i . v_k).
// Every block recomputes w_{k-1}, c and v_k identically (same data, same reduction order); block 0
// stores v_k as row k of Vh, which read column-major is the lower-storage reflector layout that
// LAPACK-style routines (ormtr) take: Q = H_0 H_1 ... H_{n-2}, H_k = I - tau_k v_k v_k^T, A = Q T Q^T.
#include <climits>
#include <type_traits>

#include "common.h"

namespace pnof {
namespace {

// Sums over the lanes of a wavefront with DPP lane moves, which stay in the vector unit (a shuffle
// goes through the LDS crossbar on every level).  Quad permutes (lane ^ 1, lane ^ 2) and the
// half-row and row mirrors (lane i <-> 7 - i, 15 - i) leave every lane of a row of 16 with the row's
// sum; two row broadcasts (lane 15 into rows 1 and 3, lane 31 into rows 2 and 3) then carry the row
// sums into lane 63, which is read back.  All 64 lanes must be active.
template <int CTRL, int ROWMASK = 0xf>
__device__ __forceinline__ double dpp_mov(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWMASK, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWMASK, 0xf, false);
  return __hiloint2double(hi, lo);
}
// sum over each group of 8 lanes (lanes 8g .. 8g + 7), in every lane of the group
__device__ __forceinline__ double group8_sum(double v) {
  v += dpp_mov<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += dpp_mov<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  v += dpp_mov<0x141>(v);   // row_half_mirror
  return v;
}
// sum over the 64 lanes, returned in every lane
__device__ __forceinline__ double wave_sum(double v) {
  v = group8_sum(v);
  v += dpp_mov<0x140>(v);        // row_mirror
  v += dpp_mov<0x142, 0xa>(v);   // row_bcast:15
  v += dpp_mov<0x143, 0xc>(v);   // row_bcast:31
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
  return __hiloint2double(hi, lo);
}

constexpr int TNT = 256;   // threads per block
constexpr int TROWS = 4;   // rows of the trailing matrix per block (one per wavefront)
constexpr int TPQ = 4;     // prologue elements per thread held in registers (loops cover the rest)
constexpr int TPRE = 24;   // row elements per lane loaded before the prologue (loops cover the rest)

__host__ __device__ inline int trd_group_base(int k) { return ((k + 1) / TROWS) & ~7; }

__device__ double tblock_sum(double v, double* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < TNT / 64; ++i) s += red[i];
  return s;
}

__global__ __launch_bounds__(TNT) void trd_step_k(int n, int k, double* __restrict__ A, double* __restrict__ Vh,
                                                  const double* __restrict__ pprev, double* __restrict__ pcur,
                                                  double* __restrict__ d, double* __restrict__ e,
                                                  double* __restrict__ tau) {
  extern __shared__ double sh[];
  const int m = n - k;          // active indices k .. n-1, stored from 0
  double* vp = sh;              // v_{k-1}
  double* wp = sh + m;          // p_{k-1}, then w_{k-1}
  double* vk = sh + 2 * m;      // c, then v_k
  __shared__ double red[TNT / 64];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  // this wavefront's row: its first TPRE * 64 elements are loaded before the prologue, so their
  // latency overlaps the prologue's
  // row group g = irow / TROWS goes to block g - gb, with gb a multiple of 8: workgroups are dealt to
  // the 8 XCDs round-robin, so each row stays on one XCD (and its L2) from step to step
  const int gb = trd_group_base(k);
  const int irow = (gb + (int)blockIdx.x) * TROWS + wv;
  const bool has_row = (irow > k) && (irow < n) && (m >= 2);
  double* __restrict__ row = A + (long long)(has_row ? irow : k) * n + k;
  double a[TPRE];
#pragma unroll
  for (int c = 0; c < TPRE; ++c) {
    const int jl = 1 + lane + 64 * c;
    a[c] = (has_row && jl < m) ? row[jl] : 0.0;
  }
  // prologue: v_{k-1}, p_{k-1} and row k loaded together
  const double* vprev = Vh + (long long)(k > 0 ? k - 1 : 0) * n + k;
  const double* pp = pprev + k;
  const double* rowk = A + (long long)k * n + k;
  double rv[TPQ], rp[TPQ], rc[TPQ];
#pragma unroll
  for (int q = 0; q < TPQ; ++q) {
    const int i = t + TNT * q;
    const bool ok = i < m;
    rv[q] = (ok && k > 0) ? vprev[i] : 0.0;
    rp[q] = (ok && k > 0) ? pp[i] : 0.0;
    rc[q] = ok ? rowk[i] : 0.0;
  }
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < TPQ; ++q) {
    const int i = t + TNT * q;
    if (i < m) {
      vp[i] = rv[q];
      s += rv[q] * rp[q];
    }
  }
  for (int i = t + TNT * TPQ; i < m; i += TNT) {
    const double v = k > 0 ? vprev[i] : 0.0, p = k > 0 ? pp[i] : 0.0;
    vp[i] = v;
    wp[i] = p;
    s += v * p;
  }
  s = tblock_sum(s, red);   // its syncs also publish vp and wp
  const double half = k > 0 ? 0.5 * tau[k - 1] * s : 0.0;
  const double v0 = vp[0], w0 = (k > 0 ? pp[0] : 0.0) - half * v0;
  double sig = 0.0;
#pragma unroll
  for (int q = 0; q < TPQ; ++q) {
    const int i = t + TNT * q;
    if (i < m) {
      const double w = rp[q] - half * rv[q];
      wp[i] = w;
      const double c = rc[q] - v0 * w - w0 * rv[q];
      rc[q] = c;
      vk[i] = c;
      if (i >= 2) sig += c * c;
    }
  }
  for (int i = t + TNT * TPQ; i < m; i += TNT) {
    const double w = wp[i] - half * vp[i];
    wp[i] = w;
    const double c = rowk[i] - v0 * w - w0 * vp[i];
    vk[i] = c;
    if (i >= 2) sig += c * c;
  }
  sig = tblock_sum(sig, red);   // also publishes wp and vk
  double tk = 0.0, beta = 0.0, scal = 0.0;
  if (m >= 2) {
    const double alpha = vk[1];
    if (sig == 0.0) {
      beta = alpha;
    } else {
      beta = -copysign(sqrt(alpha * alpha + sig), alpha);
      tk = (beta - alpha) / beta;
      scal = 1.0 / (alpha - beta);
    }
  }
  const double dk = vk[0];
  __syncthreads();   // every thread has read vk[0] and vk[1]
#pragma unroll
  for (int q = 0; q < TPQ; ++q) {
    const int i = t + TNT * q;
    if (i < m) vk[i] = (i == 0) ? 0.0 : (i == 1 ? 1.0 : rc[q] * scal);
  }
  for (int i = t + TNT * TPQ; i < m; i += TNT) vk[i] = (i == 0) ? 0.0 : (i == 1 ? 1.0 : vk[i] * scal);
  __syncthreads();
  if (blockIdx.x == 0) {
    double* vrow = Vh + (long long)k * n + k;
    for (int i = t; i < m; i += TNT) vrow[i] = vk[i];
    if (t == 0) {
      d[k] = dk;
      if (m >= 2) {
        e[k] = beta;
        tau[k] = tk;
      }
    }
  }
  if (!has_row) return;
  const int il = irow - k;
  const double vpi = vp[il], wpi = wp[il];
  double acc = 0.0;
#pragma unroll
  for (int c = 0; c < TPRE; ++c) {
    const int jl = 1 + lane + 64 * c;
    if (jl < m) {
      const double x = a[c] - vpi * wp[jl] - wpi * vp[jl];
      row[jl] = x;
      acc += x * vk[jl];
    }
  }
  constexpr int CH = 8;
  for (int j0 = 1 + 64 * TPRE; j0 < m; j0 += 64 * CH) {
    double b[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int jl = j0 + lane + 64 * c;
      b[c] = jl < m ? row[jl] : 0.0;
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int jl = j0 + lane + 64 * c;
      if (jl < m) {
        const double x = b[c] - vpi * wp[jl] - wpi * vp[jl];
        row[jl] = x;
        acc += x * vk[jl];
      }
    }
  }
  acc = wave_sum(acc);
  if (lane == 0) pcur[irow] = tk * acc;
}

// ---------------------------------------------------------------- the reduction in one launch
// The trailing m0 x m0 block (columns k0 .. n-1, m0 = n - k0) with its rows in registers for the whole
// reduction, so that a column costs one exchange of two vectors instead of a launch.  NW wavefronts per
// workgroup (in MULTI one per SIMD: what every wavefront computes alike would otherwise be issued several
// times on each), each holding up to NR rows; lane l holds columns l, l + 64, ... (NJ of them).  Indices below
// are relative to k0.  Column k, in every wavefront alike (the values and the order of the sums are the
// same everywhere, so all agree bit for bit):
//   w = p - (tau/2)(p . v) v from p_{k-1} and v_{k-1} (whose entry k is 1), c = row k - w - w_k v, the
//   Householder vector v_k, then for each own row i > k: row -= v_i w + w_i v, p_k[i] = tau_k (row . v_k);
//   the owner of row k + 1 publishes it with its p.
//
// MULTI (m0 > 32): the workgroups of one accelerator die exchange p and the row through that die's L2,
// every 8-byte value announcing itself: a slot holds TRD_EMPTY until its value arrives, and each reader
// polls the values that it needs (no store is waited for, no flag follows the data; loads bypass the
// compute unit's L1, nothing is written back or invalidated).  Four slots in turn: column k is published
// in slot (k + 1) & 3, read at column k + 1, and emptied by its writers at column k + 2, for column
// k + 4.  Every workgroup also publishes a word per column, after a barrier behind which its wavefronts'
// earlier stores have reached the L2; having read that word of all workgroups for column k, a workgroup
// knows that slot k's values were read by all, and the emptying at column k - 1 is done everywhere.
// Which workgroups take part is settled at run time: the first one to start claims its die, those of
// other dies leave at once, and the first one closes the list when `want` have registered or TRD_WINDOW
// ticks have passed.  A workgroup on the list is running, so nothing waits for one that is not; with
// fewer than are needed to hold the rows (a device busy with other work) the first one takes all rows of a block of
// at most 128 itself; otherwise it declines (info[1] = 1, d, e, tau zero), and the caller takes the launches per
// column, after the rest of the step has run on zeros.  A wait that outlasts TRD_STALL ticks ends the same way, so
// every wavefront ends.
// Beside products that fill the chip on another stream (4096^3 in float32, one after the other) the orbital step of 75
// functions takes 6.5 ms, of 140 16.6, of 300 13.5 (with launches per column and one workgroup for the last 128
// columns 6.5, 10.3 and 54.8); all 8 x 32 workgroups instead of 8 x `want`, and a decline for 75, took 10.4 there.
// One workgroup (m0 <= 32): p and the row go through LDS, one barrier per column.
//
// What bounds it: the chain of two wavefront sums, a square root and, in MULTI, one exchange per column.
// Measured, the whole reduction: n = 24 26 us (40 us as one workgroup with the block in LDS), 75 105 us
// (157 us), 200 310 us (348 us of launches per column and 370 us for the last 128), 500 1.11 ms
// (2.24 ms); from 1024 on per column 4.6 us in here against 7 us a launch (n = 1200: 6.0 against
// 6.7 ms).  A column at n = 500: 2.2 us, of it 0.5 waiting for the other workgroups' values.
constexpr int TRD_SOLO = 32;                 // at most: one workgroup
constexpr int TRD_SOLO2 = 128;               // and after launches per column
constexpr int TRD_MMAX = 1024;               // at most: the rows fit one die's registers
constexpr int TRD_PAD = 82 * 1024;           // LDS request that keeps a second workgroup off a compute unit (blocks over
                                             // 256: fewer workgroups spread by themselves, and wait less without it)
constexpr int TRD_WMAX = 64;                 // workgroups that take part at most
constexpr int TRD_CTL = 32;                  // words: die, registered, closed, abort
constexpr int TRD_SLOTS = 4;
constexpr int trd_slot(int m) { return 2 * m + TRD_WMAX; }   // p, the row, a word per workgroup
constexpr long long TRD_EMPTY = 0x7FF7A5A5C3C35A5ALL;        // a NaN that no operation makes
constexpr unsigned long long TRD_WINDOW = 5000, TRD_STALL = 500000000;   // 100 MHz ticks: 50 us, 5 s

__device__ __forceinline__ int trd_ld(const int* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double trd_ld(const double* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// To the die's L2, where trd_ld of the die's other workgroups finds it: stores at workgroup scope go through the L1 to
// the L2 that all workgroups of the list share (one die).  The language promises this of stores at agent scope only,
// which would go past the L2; readers on another die would not see these.
__device__ __forceinline__ void trd_st(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ bool trd_empty(double v) { return __double_as_longlong(v) == TRD_EMPTY; }
__device__ __forceinline__ double trd_value(double v) { return trd_empty(v) ? __longlong_as_double(0x7FF8000000000000LL) : v; }
__device__ __forceinline__ int trd_die() { return (int)__builtin_amdgcn_s_getreg((3 << 11) | 20); }   // XCC_ID[3:0]

// Clears the exchange state and the outputs that the solver after the reduction reads whatever happens.
__global__ __launch_bounds__(256) void trd_reset_k(int n, int k0, int slots, double* __restrict__ xch, int* __restrict__ ctl,
                                                   int* __restrict__ info, double* __restrict__ d, double* __restrict__ e,
                                                   double* __restrict__ tau) {
  const int g = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
  if (g < TRD_CTL) ctl[g] = 0;
  if (g == 0) info[1] = 0;
  for (int i = g; i < slots; i += step) xch[i] = __longlong_as_double(TRD_EMPTY);
  for (int i = k0 + g; i < n; i += step) {   // columns before k0 are done
    d[i] = 0.0;
    if (i + 1 < n) {
      e[i] = 0.0;
      tau[i] = 0.0;
    }
  }
}

// 1 / x from the hardware estimate and one third-order step.
__device__ __forceinline__ double rcp_f64(double x) {
  double y = __builtin_amdgcn_rcp(x);
  double r = fma(-x, y, 1.0);
  y = fma(y, fma(r, r, r), y);
  return y;
}

// Registers this workgroup (MULTI): its index among the W taking part, TRD_ALONE for the first one if there are too few
// and it is to go on without the others, or -1 to leave.
constexpr int TRD_ALONE = -2;
__device__ int trd_register(int* ctl, int want, int need, bool alone, int* info, int& W) {
  __shared__ int s_id, s_w;
  if (threadIdx.x == 0) {
    int id = -1, w = 0;
    const int die = trd_die() + 1;
    const int prev = atomicCAS(ctl, 0, die);
    if (prev == 0 || prev == die) {
      const int t = atomicAdd(ctl + 1, 1);
      if (t < want) {
        const unsigned long long t0 = wall_clock64();
        if (t == 0) {
          while (trd_ld(ctl + 1) < want && wall_clock64() - t0 < TRD_WINDOW) __builtin_amdgcn_s_sleep(2);
          const int cnt = atomicAdd(ctl + 1, 1 << 20);   // late ones see a count past any `want`
          w = cnt < want ? cnt : want;
          if (w < need) {
            if (alone) id = TRD_ALONE;
            else atomicExch(info + 1, 1);
            w = -1;
          }
          atomicExch(ctl + 2, w);
        } else {
          while ((w = trd_ld(ctl + 2)) == 0 && wall_clock64() - t0 < TRD_STALL) __builtin_amdgcn_s_sleep(2);
          if (w == 0) atomicExch(info + 1, 1);
        }
        if (w > 0) id = t < w ? t : -1;
      }
    }
    s_id = id;
    s_w = w;
  }
  __syncthreads();
  W = s_w;
  return s_id;
}

// Sums over the 64 lanes of NR values at once: the values are paired off while the lanes are folded (two
// values share one register after each of the first steps), so 8 sums take 10 additions instead of 48.
// Lane L ends with the sum of value sum_slot<NR>(L).
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// a = [a's lower 32 lanes, b's lower], b = [a's upper, b's upper]; with 16: the same within each half.
__device__ __forceinline__ double fold32(double a, double b) {
  const u32x2 lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const u32x2 hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi.x, lo.x) + __hiloint2double(hi.y, lo.y);
}
__device__ __forceinline__ double fold16(double a, double b) {
  const u32x2 lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const u32x2 hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi.x, lo.x) + __hiloint2double(hi.y, lo.y);
}
template <int NR>
__device__ __forceinline__ int sum_slot(int lane) {
  if constexpr (NR == 8) return ((lane >> 5) & 1) * 4 + ((lane >> 4) & 1) * 2 + ((lane >> 3) & 1);
  else if constexpr (NR == 4) return ((lane >> 5) & 1) * 2 + ((lane >> 4) & 1);
  else if constexpr (NR == 2) return (lane >> 5) & 1;
  return 0;
}
template <int NR>
__device__ __forceinline__ double sum_rows(const double* x) {
  static_assert(NR == 1 || NR == 2 || NR == 4 || NR == 8, "row counts");
  if constexpr (NR == 8) {
    const double y0 = fold32(x[0], x[4]), y1 = fold32(x[1], x[5]), y2 = fold32(x[2], x[6]), y3 = fold32(x[3], x[7]);
    const double z0 = fold16(y0, y2), z1 = fold16(y1, y3);
    // lanes with bit 3 clear keep z0, the others z1; each receives its value's half from lane ^ 8
    const bool up = (threadIdx.x & 8) != 0;
    const double keep = up ? z1 : z0, send = up ? z0 : z1;
    return group8_sum(keep + dpp_mov<0x128>(send));   // row_ror:8
  } else {
    double y;
    if constexpr (NR == 4) y = fold16(fold32(x[0], x[2]), fold32(x[1], x[3]));
    else if constexpr (NR == 2) y = fold32(x[0], x[1]);
    else y = x[0];
    y = group8_sum(y);
    y += dpp_mov<0x140>(y);   // row_mirror
    if constexpr (NR <= 2) y = fold16(y, y);
    if constexpr (NR == 1) y = fold32(y, y);
    return y;
  }
}

// f(std::integral_constant<int, r>) for the run-time r in [LO, HI) (registers take no run-time index).
template <int LO, int HI, typename F>
__device__ __forceinline__ void trd_pick(int r, F f) {
  if constexpr (HI - LO == 1) {
    f(std::integral_constant<int, LO>{});
  } else {
    constexpr int MID = (LO + HI) / 2;
    if (r < MID) trd_pick<LO, MID>(r, f);
    else trd_pick<MID, HI>(r, f);
  }
}

template <int NJ>
struct TrdLds {   // by parity of the column: a slow wavefront may still read one while a fast one fills the other
  double ps[2][64 * NJ], rs[2][64 * NJ], vs[2][64 * NJ];
  int stop;
};
// The columns, by workgroup id of W.
template <bool MULTI, int NW, int NR, int NJ>
__device__ __forceinline__ void trd_columns(TrdLds<NJ>& sm, int id, int W, int n, int k0, const double* __restrict__ A,
                                            double* __restrict__ Vh, const double* __restrict__ pprev,
                                            double* __restrict__ d, double* __restrict__ e, double* __restrict__ tau,
                                            int* ctl, double* xch, int* info) {
  constexpr int M = 64 * NJ;
  constexpr int NG = NR > 4 ? 8 : NR == 3 ? 4 : NR, NP = (NR + NG - 1) / NG * NG;   // rows summed together
  constexpr int NL = MULTI ? (NJ + NW - 1) / NW : 1;  // values of each kind that a thread reads
  auto &ps = sm.ps, &rs = sm.rs, &vs = sm.vs;
  int& s_stop = sm.stop;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int m0 = n - k0;
  double a[NR][NJ], v[NJ];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int i = id + W * (wave + NW * r);
#pragma unroll
    for (int c = 0; c < NJ; ++c) {
      const int j = 64 * c + lane;
      a[r][c] = (i < m0 && j < m0) ? A[(long long)(k0 + i) * n + k0 + j] : 0.0;
    }
  }
#pragma unroll
  for (int c = 0; c < NJ; ++c) {
    const int j = 64 * c + lane;
    v[c] = (k0 > 0 && j < m0) ? Vh[(long long)(k0 - 1) * n + k0 + j] : 0.0;
  }
  for (int j = t; j < M; j += 64 * NW) {
    const bool ok = j < m0;
    ps[0][j] = (ok && k0 > 0) ? pprev[k0 + j] : 0.0;
    rs[0][j] = ok ? A[(long long)k0 * n + k0 + j] : 0.0;
    vs[1][j] = (ok && k0 > 0) ? Vh[(long long)(k0 - 1) * n + k0 + j] : 0.0;
    ps[1][j] = 0.0;
    rs[1][j] = 0.0;
    vs[0][j] = 0.0;
  }
  if (t == 0) {
    s_stop = 0;
    if (!MULTI) info[1] = 0;
  }
  double tprev = k0 > 0 ? tau[k0 - 1] : 0.0;
  // the workgroup, wavefront and register row that hold row k + 1, and whether rows k, k - 1 were this
  // wavefront's
  int turn = 0, ow = 0, orow = 0;
  bool mine1 = id == 0 && wave == 0, mine2 = false;
  for (int k = 0; k < m0; ++k) {
    const int cur = k & 1, nxt = cur ^ 1;
    if constexpr (MULTI) {
      if (k > 0) {
        const double* px = xch + (k & (TRD_SLOTS - 1)) * trd_slot(M);
        double x[NL], y[NL], h;
        unsigned spin = 0;
        unsigned long long t0 = 0;
        for (;;) {
          bool ok = true;
#pragma unroll
          for (int q = 0; q < NL; ++q) {
            const int j = t + 64 * NW * q;
            x[q] = y[q] = 0.0;
            if (j >= k && j < m0) {
              x[q] = trd_ld(px + j);
              y[q] = trd_ld(px + M + j);
            }
          }
          h = t < W ? trd_ld(px + 2 * M + t) : 0.0;
#pragma unroll
          for (int q = 0; q < NL; ++q) ok = ok && !trd_empty(x[q]) && !trd_empty(y[q]);
          if (ok && !trd_empty(h)) break;
          if ((++spin & 1023u) == 0) {
            const unsigned long long now = wall_clock64();
            if (t0 == 0) t0 = now;
            if (trd_ld(ctl + 3) != 0 || now - t0 > TRD_STALL) {
              atomicExch(ctl + 3, 1);
              atomicExch(info + 1, 1);
              s_stop = 1;
              break;
            }
          }
        }
#pragma unroll
        for (int q = 0; q < NL; ++q) {
          const int j = t + 64 * NW * q;
          if (j >= k && j < m0) {
            ps[cur][j] = x[q];
            rs[cur][j] = y[q];
          }
        }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's earlier stores have reached the L2
    }
    __syncthreads();
    if constexpr (MULTI) {
      if (s_stop) return;
      if (t == 0 && k + 1 < m0) trd_st(xch + ((k + 1) & (TRD_SLOTS - 1)) * trd_slot(M) + 2 * M + id, 0.0);
    }
    // everything this column reads from LDS, at once
    double w[NJ], vn[NJ], vi[NR], wi[NR];
#pragma unroll
    for (int c = 0; c < NJ; ++c) {
      w[c] = ps[cur][64 * c + lane];
      vn[c] = rs[cur][64 * c + lane];
    }
    const int k1 = k + 1 < M ? k + 1 : k;
    const double pk = ps[cur][k], rk = rs[cur][k], pk1 = ps[cur][k1], rk1 = rs[cur][k1], vk1 = vs[nxt][k1];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int i = min(id + W * (wave + NW * r), M - 1);
      vi[r] = vs[nxt][i];
      wi[r] = ps[cur][i];
    }
    // (entries before k are stale but finite, and meet zeros of v and of the new vector)
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < NJ; ++c) s += w[c] * v[c];
    s = wave_sum(s);
    const double half = 0.5 * tprev * s;
    const double w0 = pk - half;
    double sig = 0.0;
#pragma unroll
    for (int c = 0; c < NJ; ++c) {
      w[c] -= half * v[c];
      const double x = vn[c] - w[c] - w0 * v[c];
      vn[c] = 64 * c + lane > k + 1 ? x : 0.0;
      sig += vn[c] * vn[c];
    }
    sig = wave_sum(sig);
    const double dk = rk - 2.0 * w0;
    const double alpha = rk1 - (pk1 - half * vk1) - w0 * vk1;
    double tk = 0.0, beta = alpha, scal = 0.0;
    if (k + 1 < m0 && sig != 0.0) {
      const double q = alpha * alpha + sig;
      if (__builtin_expect(q > 1e-280 && q < 1e280, 1)) {
        const double y = rsqrt_f64(q), nrm = q * y, aa = fabs(alpha);
        beta = -copysign(nrm, alpha);
        tk = fma(aa, y, 1.0);
        scal = copysign(rcp_f64(aa + nrm), alpha);
      } else {
        beta = -copysign(sqrt(q), alpha);
        tk = (beta - alpha) / beta;
        scal = 1.0 / (alpha - beta);
      }
    }
#pragma unroll
    for (int c = 0; c < NJ; ++c) {
      const int j = 64 * c + lane;
      vn[c] = j == k + 1 ? 1.0 : vn[c] * scal;
      if (wave == 0) vs[cur][j] = vn[c];
    }
    const int kc1 = (k + 1) >> 6;   // first chunk with an index > k
    double* const px = xch + ((k + 1) & (TRD_SLOTS - 1)) * trd_slot(M);   // published now
    double* const pe = xch + ((k + 3) & (TRD_SLOTS - 1)) * trd_slot(M);   // read by all: emptied
    // own rows; those already reduced (and those past the matrix) keep their values
    double acc[NP];
#pragma unroll
    for (int r = 0; r < NP; ++r) acc[r] = 0.0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int i = id + W * (wave + NW * r);
      wi[r] = i > k && i < m0 ? wi[r] - half * vi[r] : 0.0;
      vi[r] = i > k && i < m0 ? vi[r] : 0.0;
    }
#pragma unroll
    for (int c = 0; c < NJ; ++c)
      if (c >= kc1) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          const double x = a[r][c] - vi[r] * w[c] - wi[r] * v[c];
          a[r][c] = x;
          acc[r] += x * vn[c];
        }
      }
    if (++turn == W) {
      turn = 0;
      if (++ow == NW) {
        ow = 0;
        ++orow;
      }
    }
    const bool mine = turn == id && ow == wave;
    if (mine) {   // the next column's row
      trd_pick<0, NR>(orow, [&](auto rc) {
        constexpr int r = decltype(rc)::value;
#pragma unroll
        for (int c = 0; c < NJ; ++c) {
          const int j = 64 * c + lane;
          if constexpr (MULTI) {
            if (c >= kc1 && j < m0) trd_st(px + M + j, trd_value(a[r][c]));
          } else {
            rs[nxt][j] = a[r][c];
          }
        }
      });
    }
#pragma unroll
    for (int g = 0; g < NP; g += NG) {
      const double p = tk * sum_rows<NG>(acc + g);
      const int r = g + sum_slot<NG>(lane);
      const int i = id + W * (wave + NW * r);
      if ((lane & (64 / NG - 1)) == 0 && r < NR && i < m0) {
        if constexpr (MULTI) {
          if (i > k) trd_st(px + i, trd_value(p));
          trd_st(pe + i, __longlong_as_double(TRD_EMPTY));
        } else {
          if (i > k) ps[nxt][i] = p;
        }
      }
    }
    if constexpr (MULTI) {
      if (t == 0) trd_st(pe + 2 * M + id, __longlong_as_double(TRD_EMPTY));
      if (mine2) {   // row k - 1, published two columns ago
#pragma unroll
        for (int c = 0; c < NJ; ++c) trd_st(pe + M + 64 * c + lane, __longlong_as_double(TRD_EMPTY));
      }
    }
    mine2 = mine1;
    mine1 = mine;
    if (wave == NW - 1 && (!MULTI || id == turn)) {   // column k's results, by one wavefront
#pragma unroll
      for (int c = 0; c < NJ; ++c) {
        const int j = 64 * c + lane;
        if (j >= k && j < m0) Vh[(long long)(k0 + k) * n + k0 + j] = vn[c];
      }
      if (lane == 0) {
        d[k0 + k] = dk;
        if (k + 1 < m0) {
          e[k0 + k] = beta;
          tau[k0 + k] = tk;
        }
      }
    }
#pragma unroll
    for (int c = 0; c < NJ; ++c) v[c] = vn[c];
    tprev = tk;
  }
}

template <bool MULTI, int NW, int NR, int NJ>
__global__ __launch_bounds__(64 * NW, MULTI && NJ == 2 ? 2 : 1) void trd_reduce_k(int n, int k0, int want, int need, const double* __restrict__ A,
                                                    double* __restrict__ Vh, const double* __restrict__ pprev,
                                                    double* __restrict__ d, double* __restrict__ e,
                                                    double* __restrict__ tau, int* ctl, double* xch, int* info) {
  __shared__ TrdLds<NJ> sm;
  if constexpr (MULTI) {
    constexpr bool ALONE = 64 * NJ == TRD_SOLO2;   // one workgroup can hold the rows
    int W;
    const int id = __builtin_amdgcn_readfirstlane(trd_register(ctl, want, need, ALONE, info, W));
    if constexpr (ALONE)
      if (id == TRD_ALONE) trd_columns<false, NW, TRD_SOLO2 / NW, NJ>(sm, 0, 1, n, k0, A, Vh, pprev, d, e, tau, ctl, xch, info);
    if (id < 0) return;
    trd_columns<true, NW, NR, NJ>(sm, id, __builtin_amdgcn_readfirstlane(W), n, k0, A, Vh, pprev, d, e, tau, ctl, xch, info);
  } else {
    trd_columns<false, NW, NR, NJ>(sm, 0, 1, n, k0, A, Vh, pprev, d, e, tau, ctl, xch, info);
  }
}

// ---------------------------------------------------------------- back-transformation
// Q = H_0 ... H_{n-2} formed explicitly (column-major n x n); the eigenvectors are then Q times
// those of the tridiagonal matrix.  The reflectors are taken in blocks of QNB:
// Q_b = H_{k0} ... H_{k0+QNB-1} = I - V T V^T with V the block's vectors as columns and T upper
// triangular (the compact WY form of a product of reflectors, Schreiber and Van Loan 1989).  Q is
// built from the identity by applying Q_last, ..., Q_0 in turn, each as three float64 GEMMs on the
// trailing part [k0 + 1, n) x [k0 + 1, n) (columns at or before k0 are still unit columns there, and
// rows at or before k0 are untouched by the block).

// V as explicit columns (zero above the unit entry, zero past the last reflector), and Q = I.
__global__ __launch_bounds__(256) void formq_init_k(int n, int nref, int ncol, const double* __restrict__ Vh,
                                                    double* __restrict__ Vc, double* __restrict__ Q) {
  const long long tot = (long long)n * ncol, i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i < tot) {
    const int c = (int)(i / n), r = (int)(i % n);
    Vc[i] = (c < nref && r > c) ? (r == c + 1 ? 1.0 : Vh[(long long)c * n + r]) : 0.0;
  }
  if (i < (long long)n * n) Q[i] = (i / n == i % n) ? 1.0 : 0.0;
}

// T of every block (one workgroup each) from the block's Gram matrix G = V^T V (row-major QNB x QNB).
// Within a run of 16 reflectors, column j follows from the earlier ones: T[j][j] = tau_j,
// T[0:j][j] = -tau_j T[0:j][0:j] G[0:j][j] (row i in one lane's registers, the eight runs in parallel).
// Adjacent triangles then merge as T = [[T1, -T1 G12 T2], [0, T2]] (the product of two compact WY
// factors), 16 + 16 up to 64 + 64, on the float64 matrix cores; the scratch X = G12 T2 lives in T's lower
// triangle.  Zero past the block's last reflector.  A latency chain: 126 us with runs of 32 and the
// merges as loops over G in global memory, 18 us here.
constexpr int FQR = 16, FQW = 8;   // reflectors of a run, wavefronts
// acc = sum over 16-wide k-tiles kt in [k0, k1) of A(i, k) B(k, j); A(i, k) = a[i * lda + k], B(k, j) = b[k * ldb + j]
__device__ __forceinline__ f64x4 fq_tile(const double* __restrict__ a, int lda, const double* __restrict__ b, int ldb,
                                         int k0, int k1) {
  const int l = threadIdx.x & 63, r = l & 15, kq = l >> 4;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int kt = k0; kt < k1; ++kt)
#pragma unroll
    for (int kk = 0; kk < 16; kk += 4) {
      const int k = 16 * kt + kk + kq;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r * lda + k], b[k * ldb + r], acc, 0, 0, 0);
    }
  return acc;
}

__global__ __launch_bounds__(64 * FQW) void formq_t_k(int nref, const double* __restrict__ tau,
                                                      const double* __restrict__ Gall, double* __restrict__ Tall) {
  __shared__ double T[QNB][QNB + 1];
  __shared__ double Gd[QNB / FQR][FQR][FQR + 1];
  static_assert(QNB == FQR * FQW, "one run per wavefront");
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int k0 = blockIdx.x * QNB, nb = min(QNB, nref - k0);
  const double* G = Gall + (long long)blockIdx.x * QNB * QNB;
  const int c0 = FQR * wv;
  for (int x = lane; x < FQR * FQR; x += 64) Gd[wv][x / FQR][x % FQR] = G[(c0 + x / FQR) * QNB + c0 + x % FQR];
  const double tl = (lane < FQR && c0 + lane < nb) ? tau[k0 + c0 + lane] : 0.0;
  __syncthreads();
  if (lane < FQR) {
    double row[FQR];
#pragma unroll
    for (int j = 0; j < FQR; ++j) {
      const double tj = __shfl(tl, j, FQR);
      double a = 0.0;
#pragma unroll
      for (int l = 0; l < j; ++l) a += row[l] * Gd[wv][l][j];   // zero below the row's diagonal
      row[j] = lane < j ? -tj * a : (lane == j ? tj : 0.0);
    }
#pragma unroll
    for (int j = 0; j < FQR; ++j) T[c0 + lane][c0 + j] = row[j];
  }
  __syncthreads();
  const int r4 = lane >> 4, cl = lane & 15;
  for (int h = FQR; h < QNB; h *= 2) {
    const int ht = h / FQR, per = ht * ht, ntile = (QNB / (2 * h)) * per;
    // X = G12 T2 (T2 upper triangular: k-tiles up to the column's)
    for (int x = wv; x < ntile; x += FQW) {
      const int off = (x / per) * 2 * h, tm = (x % per) / ht, tn = x % ht;
      const f64x4 acc = fq_tile(G + (off + 16 * tm) * QNB + off + h, QNB, &T[off + h][off + h + 16 * tn], QNB + 1, 0, tn + 1);
#pragma unroll
      for (int q = 0; q < 4; ++q) T[off + h + 16 * tm + r4 + 4 * q][off + 16 * tn + cl] = acc[q];
    }
    __syncthreads();
    // T12 = -T1 X (k-tiles from the row's)
    for (int x = wv; x < ntile; x += FQW) {
      const int off = (x / per) * 2 * h, tm = (x % per) / ht, tn = x % ht;
      const f64x4 acc = fq_tile(&T[off + 16 * tm][off], QNB + 1, &T[off + h][off + 16 * tn], QNB + 1, tm, ht);
#pragma unroll
      for (int q = 0; q < 4; ++q) T[off + 16 * tm + r4 + 4 * q][off + h + 16 * tn + cl] = -acc[q];
    }
    __syncthreads();
  }
  double* Tb = Tall + (long long)blockIdx.x * QNB * QNB;
  for (int e = t; e < QNB * QNB; e += 64 * FQW) {
    const int i = e / QNB, c = e % QNB;
    Tb[e] = c >= i ? T[i][c] : 0.0;
  }
}

// W1 (QNB x mb, ld n) = the sum of the ks split-K slabs (each QNB x mb, dense).
__global__ __launch_bounds__(256) void formq_sum_k(int mb, int n, int ks, const double* __restrict__ part,
                                                   double* __restrict__ W1) {
  const long long tot = (long long)QNB * mb, e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= tot) return;
  double a = 0.0;
  for (int s = 0; s < ks; ++s) a += part[s * tot + e];
  W1[(e / mb) * n + e % mb] = a;
}

}  // namespace

long long form_q_ws_doubles(int n) {
  const long long nb = formq_blocks(n);
  return nb * QNB * n + 2 * nb * QNB * QNB + (2LL + FORMQ_KS) * QNB * n + 64;
}

hipError_t form_q_f64(hipStream_t s, int n, const double* Vh, const double* tau, double* ws, double* Q) {
  if (n < 3 || n > TRIDIAG_MAX_N) return hipErrorInvalidValue;
  const int nref = n - 1, nb = formq_blocks(n), ncol = nb * QNB;
  double* Vc = ws;                                  // n x ncol, column-major
  double* G = Vc + (long long)n * ncol;             // nb x QNB x QNB
  double* T = G + (long long)nb * QNB * QNB;        // nb x QNB x QNB
  double* W1 = T + (long long)nb * QNB * QNB;       // QNB x n, row-major (ld n)
  double* W2 = W1 + (long long)QNB * n;             // QNB x n
  double* part = W2 + (long long)QNB * n;           // FORMQ_KS slabs of QNB x mb
  const long long tot = (long long)n * std::max(ncol, n);
  hipLaunchKernelGGL(formq_init_k, dim3((unsigned)cdiv(tot, 256)), dim3(256), 0, s, n, nref, ncol, Vh, Vc, Q);
  // G_b = V_b^T V_b
  hipError_t e = gemm_f64(s, QNB, QNB, n, nb, 1.0, Vc, n, 1, (long long)QNB * n, Vc, 1, n, (long long)QNB * n, 0.0,
                          G, QNB, 1, (long long)QNB * QNB);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(formq_t_k, dim3(nb), dim3(64 * FQW), 0, s, nref, tau, G, T);
  for (int b = nb - 1; b >= 0; --b) {
    const int k0 = b * QNB, mb = n - k0 - 1;
    const double* Vb = Vc + (long long)k0 * n + k0 + 1;   // V_b(r, i) = Vb[i * n + r], rows k0 + 1 ..
    double* Zb = Q + (long long)(k0 + 1) * n + k0 + 1;    // Z(r, c) = Zb[c * n + r]
    // W1 = V_b^T Z, W2 = T_b W1, Z -= V_b W2
    // the first product has few output tiles (QNB x mb) and a long k: split over k, slabs summed
    const int ks = std::min(FORMQ_KS, std::max(1, mb / 128));
    if ((e = gemm_f64_splitk(s, QNB, mb, mb, ks, Vb, n, 1, Zb, 1, n, part)) != hipSuccess) return e;
    hipLaunchKernelGGL(formq_sum_k, dim3((unsigned)cdiv((long long)QNB * mb, 256)), dim3(256), 0, s, mb, n, ks, part, W1);
    if ((e = gemm_f64(s, QNB, mb, QNB, 1, 1.0, T + (long long)b * QNB * QNB, QNB, 1, 0, W1, n, 1, 0, 0.0, W2, n, 1, 0)) !=
        hipSuccess)
      return e;
    if ((e = gemm_f64(s, mb, mb, QNB, 1, -1.0, Vb, 1, n, 0, W2, n, 1, 0, 1.0, Zb, 1, n, 0)) != hipSuccess) return e;
  }
  return hipGetLastError();
}

bool tridiag_may_decline(int n) { return n > TRD_SOLO && n <= TRIDIAG_MAX_N; }
long long tridiag_ws_doubles(int n) { return 2LL * n + TRD_SLOTS * trd_slot(TRD_MMAX) + TRD_CTL; }

hipError_t tridiag_f64(hipStream_t s, int n, double* A, double* Vh, double* ws, double* d, double* e, double* tau,
                       int* info, int form) {
  if (n <= 0 || n > TRIDIAG_MAX_N) return hipErrorInvalidValue;
  double* p2 = ws;                  // two vectors of n by column parity
  double* xch = ws + 2LL * n;
  int* ctl = reinterpret_cast<int*>(xch + TRD_SLOTS * trd_slot(TRD_MMAX));
  const int kend = std::max(0, n - (form == REDUCE_LAUNCHES ? TRD_SOLO2 : TRD_MMAX));   // columns 0 .. kend-1: a launch each
  const size_t shm = 3 * (size_t)n * sizeof(double);
  for (int k = 0; k < kend; ++k) {
    const int blocks = std::max(1, (n - 1) / TROWS - trd_group_base(k) + 1);
    hipLaunchKernelGGL(trd_step_k, dim3(blocks), dim3(TNT), shm, s, n, k, A, Vh, p2 + ((k + 1) & 1) * (long long)n,
                       p2 + (k & 1) * (long long)n, d, e, tau);
  }
  const double* pp = p2 + ((kend + 1) & 1) * (long long)n;
  const int m = n - kend;
#define TRD_REDUCE(MULTI, NW, NR, NJ, grid, want, pad)                                                                 \
  hipLaunchKernelGGL((trd_reduce_k<MULTI, NW, NR, NJ>), dim3(grid), dim3(64 * NW), pad, s, n, kend, want,               \
                     form == REDUCE_DECLINE ? INT_MAX : (int)cdiv(m, NW * NR), A, Vh, pp, d, e, tau, ctl, xch, info)
  if (m <= TRD_SOLO) TRD_REDUCE(false, 8, 4, 1, 1, 1, 0);
  else if (form == REDUCE_LAUNCHES) TRD_REDUCE(false, 16, 8, 2, 1, 1, 0);
  else {
    const int M = m <= 128 ? 128 : m <= 256 ? 256 : m <= 512 ? 512 : m <= 768 ? 768 : 1024, slots = TRD_SLOTS * trd_slot(M);
    hipLaunchKernelGGL(trd_reset_k, dim3(cdiv(slots, 1024)), dim3(256), 0, s, n, kend, slots, xch, ctl, info, d, e, tau);
    // `want` workgroups on each of 8 dies
#define TRD_MULTI(NW, NR, NJ) TRD_REDUCE(true, NW, NR, NJ, 8 * cdiv(m, NW * NR), cdiv(m, NW * NR), NJ <= 4 ? 0 : TRD_PAD)
    if (M == 128) TRD_MULTI(4, 2, 2);
    else if (M == 256) TRD_MULTI(4, 2, 4);
    else if (M == 512) TRD_MULTI(4, 4, 8);
    else if (M == 768) TRD_MULTI(8, 3, 12);
    else TRD_MULTI(4, 8, 16);
#undef TRD_MULTI
  }
#undef TRD_REDUCE
  return hipGetLastError();
}

}  // namespace pnof
