// 16-bit matrix-core (v_mfma_f32_16x16x32_bf16 / _f16) contractions with float32 accumulation.
//
// Operands may be carried as a hi + lo pair of 16-bit values; the accumulator then receives
//   terms = 1: hi*hi                              (bf16, one pass)
//   terms = 2: Ahi*Bhi + Alo*Bhi                  (B exact in bf16: X from a bf16 B)
//   terms = 3: Ahi*Bhi + Ahi*Blo + Alo*Bhi        (the lo*lo product is below float32 rounding)
// In the split mode the pairs of the b and Y contractions (and of X when B is float64) are fp16
// pairs of the value times a power of two (11 + 11 significant bits; the scales are fixed per P-chunk
// from bounds, see chunk_scales), multiplied by the fp16 matrix-core instruction; X from a bf16 B
// multiplies the compact bf16 pair of C by B and writes fp16 pairs.
//
// Block tiles BM x BN x 32: 256 x 256 (8 waves) or 128 x 128 (4 waves, two blocks per compute unit) for X and Y,
// 128 x 128 for the symmetric b; in 16 x 16 MFMA blocks.  Operand k-tiles go global -> LDS directly through a ring
// of stages, one barrier per k-tile (where rows are not 16-byte aligned, through registers and two buffers).
// MFMA lane layout (16x16x32): lane l supplies row l%16 and the eight k values 8*(l/16)..+7 of each operand; result
// element (4*(l/16)+j, l%16) is component j.
//
// Operand storage in global memory:
//   "row" operand: row r (an output index) is contiguous in k  -> LDS [r][k] (16-byte chunks
//     XOR-swizzled within the row), 16-byte reads;
//   "col" operand: row k is contiguous in the output index    -> LDS [k][r], read with the
//     transposing LDS load (ds_read_b64_tr_b16), which within each 16-lane group hands lane i
//     element i%4 of the 8-byte chunks fetched by lanes 4j + i/4 (j = 0..3), i.e. four consecutive
//     k of one row when lane 4j+q fetched rows 4q..4q+3 of k-row j.
// Blocks are numbered so that the eight XCDs each receive one contiguous range of work items:
// items sharing an operand (same P, or same split of P) run on the same XCD and share its L2.
#include <type_traits>

#include "batch_dev.h"
#include "common.h"
#include "f64_tile.h"

namespace pnof {
namespace {

constexpr int BK = 32;
constexpr int RP = BK;              // row-layout LDS pitch (bf16 elements): 64 bytes, chunks swizzled
constexpr int NXCD = 8;
constexpr int T2 = 128;             // tile of the symmetric nact x nact products

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// One 16 x 16 x 32 product; fragments hold raw 16-bit patterns (bf16 or fp16 by F16).
template <bool F16>
__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

struct Opnd {
  const u16* hi;
  const u16* lo;
  long long ld;   // elements between consecutive rows
  int R, K;       // valid rows, valid k
};

// 8 consecutive elements src[0..7] of a storage row, zero beyond `valid` elements.
__device__ __forceinline__ u32x4 ld8(const u16* __restrict__ src, int valid) {
  uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (i < valid) w[i >> 1] |= ((uint32_t)src[i]) << (16 * (i & 1));
  return u32x4{w[0], w[1], w[2], w[3]};
}

// LDS bank model of gfx950 (measured with the bank-conflict counter): 64 banks of 4 bytes; a 16-byte
// read is served in four 16-lane groups, lane L in group (bit 5, bit 2 ^ bit 3 ^ bit 4) of L, and a
// group is conflict-free when its 16 addresses fall in distinct 16-byte slots of a 256-byte line;
// an 8-byte read is served in two groups of 32 consecutive lanes, each needing distinct 8-byte slots.
// Row layout swizzle: in a fragment read (lane L: row L % 16, chunk L / 16), the four lanes of one
// group that share row % 4 are rows r, r + 12 (chunk g) and r + 4, r + 8 (chunk g ^ 1); flipping
// bit 1 of the chunk on rows with bit 3 set spreads them over four distinct slots.
__device__ __forceinline__ int swz(int r) { return 2 * ((r >> 3) & 1); }

// Row of the operand that row r of an interleaved slice holds (a permutation within each 32 rows): the
// two 16 x 16 products of a row pair then leave each lane eight consecutive output elements (rows
// 4 g .. 4 g + 3 of the first are 8 g .. 8 g + 3, those of the second 8 g + 4 .. 8 g + 7).
__device__ __forceinline__ int ileave(int r) { return (r & ~31) | (((r >> 2) & 3) << 3) | (((r >> 4) & 1) << 2) | (r & 3); }

// Global -> registers -> LDS: one BK-deep k-tile of one operand slice (D x BK elements, 4 chunks of 8 along
// k per row), element by element.  IL: interleaved rows.
template <int D>
struct Chunks {
  u32x4 v[D * BK / 8 / 256];
};
template <int D, bool IL>
__device__ __forceinline__ void fetch(const u16* __restrict__ base, const Opnd& o, int r0, int k0, Chunks<D>& ch) {
#pragma unroll
  for (int c = 0; c < D * BK / 8 / 256; ++c) {
    const int idx = threadIdx.x + 256 * c;
    const int gr = r0 + (IL ? ileave(idx >> 2) : idx >> 2), gk = k0 + (idx & 3) * 8;
    ch.v[c] = gr < o.R && gk < o.K ? ld8(base + (long long)gr * o.ld + gk, o.K - gk) : u32x4{0u, 0u, 0u, 0u};
  }
}
// The four 16-byte chunks of row r are stored permuted, chunk c at c ^ swz(r), so that fragment reads (one
// chunk of 16 consecutive rows per lane group) are free of bank conflicts.
template <int D>
__device__ __forceinline__ void stash(u16* __restrict__ s, const Chunks<D>& ch) {
#pragma unroll
  for (int c = 0; c < D * BK / 8 / 256; ++c) {
    const int idx = threadIdx.x + 256 * c;
    *reinterpret_cast<u32x4*>(s + (idx >> 2) * RP + (((idx & 3) ^ swz(idx >> 2)) * 8)) = ch.v[c];
  }
}
// MFMA operand fragment for the 16 rows starting at r: lane l gets row r + l%16 and the eight k values
// 8*(l/16)..+7 of the current k-tile.
__device__ __forceinline__ bf16x8 frag(const u16* __restrict__ s, int r) {
  const int lane = threadIdx.x & 63, rr = r + (lane & 15);
  return *reinterpret_cast<const bf16x8*>(s + rr * RP + (((lane >> 4) ^ swz(rr)) * 8));
}

template <int BM, int BN, bool ALO, bool BLO>
struct Stage {
  u16 a[2][ALO ? 2 : 1][BM * RP];
  u16 b[2][BLO ? 2 : 1][BN * RP];
};

template <int MI, int NI>
__device__ __forceinline__ void zero(f32x4 (&acc)[MI][NI]) {
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// Main loop over k in [0, K) for a BM x BN block tile whose operands' rows need not be aligned; 4 waves in
// 2 x 2, each owning (BM/2) x (BN/2).  Transposed products of interleaved rows of B, as mainloop_dl with
// lay 2.
template <int BM, int BN, bool ALO, bool BLO, bool F16>
__device__ __forceinline__ void mainloop(Stage<BM, BN, ALO, BLO>& sm, int K, int m0, int n0, const Opnd& A, const Opnd& B,
                                         f32x4 (&acc)[BM / 32][BN / 32]) {
  constexpr int MI = BM / 32, NI = BN / 32;
  const int wave = threadIdx.x >> 6;
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
  Chunks<BM> ra[ALO ? 2 : 1];
  Chunks<BN> rb[BLO ? 2 : 1];
  auto load = [&](int k) {
    fetch<BM, false>(A.hi, A, m0, k, ra[0]);
    if (ALO) fetch<BM, false>(A.lo, A, m0, k, ra[ALO ? 1 : 0]);
    fetch<BN, true>(B.hi, B, n0, k, rb[0]);
    if (BLO) fetch<BN, true>(B.lo, B, n0, k, rb[BLO ? 1 : 0]);
  };
  auto store = [&](int buf) {
    stash<BM>(sm.a[buf][0], ra[0]);
    if (ALO) stash<BM>(sm.a[buf][ALO ? 1 : 0], ra[ALO ? 1 : 0]);
    stash<BN>(sm.b[buf][0], rb[0]);
    if (BLO) stash<BN>(sm.b[buf][BLO ? 1 : 0], rb[BLO ? 1 : 0]);
  };
  load(0);
  store(0);
  __syncthreads();
  zero(acc);
  for (int k = 0, buf = 0; k < K; k += BK, buf ^= 1) {
    const bool more = k + BK < K;
    if (more) load(k + BK);
    bf16x8 ah[MI], bh[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) ah[i] = frag(sm.a[buf][0], wm + 16 * i);
#pragma unroll
    for (int j = 0; j < NI; ++j) bh[j] = frag(sm.b[buf][0], wn + 16 * j);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = mma<F16>(bh[j], ah[i], acc[i][j]);
    if (BLO) {
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const bf16x8 bl = frag(sm.b[buf][BLO ? 1 : 0], wn + 16 * j);
#pragma unroll
        for (int i = 0; i < MI; ++i) acc[i][j] = mma<F16>(bl, ah[i], acc[i][j]);
      }
    }
    if (ALO) {
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const bf16x8 al = frag(sm.a[buf][ALO ? 1 : 0], wm + 16 * i);
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = mma<F16>(bh[j], al, acc[i][j]);
      }
    }
    if (more) store(buf ^ 1);
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------
// Direct-to-LDS pipeline (aligned operands).  Each k-tile slice is fetched by buffer loads that
// write LDS directly (16 bytes per lane, a wave filling one contiguous 1 KB block), S stages deep,
// so S-1 k-tiles are in flight while the matrix cores work on the oldest one; no registers are
// spent on staging.  Loads past the buffer's record limit return zeros.  Requirements: every
// storage row starts 16-byte aligned; rows of the workspace operands are zero-padded to a
// multiple of 32 in k, so the k-tail of the last tile contributes nothing.
// Slice layouts (no padding): row mode element (r, k) at r*BK + ((k/8) ^ swz(r))*8 + k%8;
// col mode element (kr, r) at kr*D + ((r/8) ^ cswz(kr))*8 + r%8.  A transposing fragment read
// serves lanes 0-31 together: k rows kr and kr + 8 land on one bank set unless bit 3 of kr also
// moves the chunk (possible when a row holds at least 16 chunks).
template <int D>
__device__ __forceinline__ int cswz(int kr) {
  return 2 * (kr & 3) ^ (D >= 128 ? 8 * ((kr >> 3) & 1) : 0);
}

constexpr int waitcnt_vm(int n) {
  // gfx9 s_waitcnt immediate: vmcnt[3:0] bits 3:0, vmcnt[5:4] bits 15:14; expcnt and lgkmcnt maxed
  return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8);
}

struct RowItself {
  __device__ int operator()(int r) const { return r; }
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, int limit) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, limit, 0x00020000);
}
__device__ __forceinline__ int record_limit(long long bytes) { return bytes > 0x7FFFFFFFLL ? 0x7FFFFFFF : (int)bytes; }

// Operand of one k-tile for the direct path: slice base, its record limit, storage layout.
struct DOpnd {
  const u16* hi;
  const u16* lo;
  long long ld;
  long long bytes;   // readable bytes from hi (and from lo) onwards
};

// Byte offsets of this lane's 16-byte chunks of one slice from the slice's k-tile (see dl_issue): row operand,
// chunk q % 4 of row row(q / 4); col operand, chunk q % (D / 8) of k-row q / (D / 8).
template <int D, int NW, bool COL, typename F>
__device__ __forceinline__ void dl_offsets(unsigned* ofs, int ld, int r0, F row) {
  static_assert(D % (16 * NW) == 0, "slice rows per wave");
#pragma unroll
  for (int i = 0; i < D / (16 * NW); ++i) {
    const int q = ((threadIdx.x >> 6) * (D / (16 * NW)) + i) * 64 + (threadIdx.x & 63);
    if constexpr (!COL) ofs[i] = 2u * (unsigned)(row(q >> 2) * ld + ((q & 3) ^ swz(q >> 2)) * 8);
    else ofs[i] = 2u * (unsigned)((q / (D / 8)) * ld + r0 + ((q % (D / 8)) ^ cswz<D>(q / (D / 8))) * 8);
  }
}
// One k-tile of a slice: every wave's share of its 1 KB blocks.  The k-tile's place is a scalar offset, so a load
// costs no address arithmetic.
template <int D, int NW>
__device__ __forceinline__ void dl_issue(u16* lds_slice, const u16* base, int limit, const unsigned* ofs,
                                         unsigned k_ofs, int wave) {
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(base, limit);
#pragma unroll
  for (int i = 0; i < D / (16 * NW); ++i)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rs, (__attribute__((address_space(3))) void*)(lds_slice + (wave * (D / (16 * NW)) + i) * 512), 16, ofs[i], k_ofs, 0, 0);
}

template <int D, bool COL>
__device__ __forceinline__ bf16x8 dl_frag(const u16* __restrict__ s, int r) {
  const int lane = threadIdx.x & 63;
  if constexpr (!COL) {
    const int rr = r + (lane & 15);
    return *reinterpret_cast<const bf16x8*>(s + rr * BK + (((lane >> 4) ^ swz(rr)) * 8));
  }
  const int g = lane >> 4, L = lane & 15, j = L >> 2, q = L & 3;
  typedef __attribute__((address_space(3))) v4s* lds_v4s;
  const int m = r + 4 * q;
  const int k0 = 8 * g + j, k1 = 8 * g + 4 + j;
  const u16* p0 = s + k0 * D + (((m >> 3) ^ cswz<D>(k0)) << 3) + (m & 7);
  const u16* p1 = s + k1 * D + (((m >> 3) ^ cswz<D>(k1)) << 3) + (m & 7);
  union { v4s h[2]; bf16x8 v; } u;
  u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p0));
  u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p1));
  return u.v;
}

// Pipeline depth that fits `budget` bytes of LDS (at most 5 stages: up to four k-tiles in flight
// while one is consumed, which is what covers the latency of operands streamed from HBM).
constexpr int ring_depth(int BM, int BN, bool ALO, bool BLO, int budget) {
  const int stage = 2 * BK * (BM * (ALO ? 2 : 1) + BN * (BLO ? 2 : 1));
  const int s = budget / stage;
  return s > 5 ? 5 : s;
}

template <int BM, int BN, bool ALO, bool BLO, int S>
struct Ring {
  u16 a[S][ALO ? 2 : 1][BM * BK];
  u16 b[S][BLO ? 2 : 1][BN * BK];
};

// The ring of a contraction body: the caller's (EXT: e.g. one union shared by the bodies of a
// persistent kernel, ext pointing into LDS) or the body's own static LDS.
template <typename RT, bool EXT>
__device__ __forceinline__ RT& ring_of(void* ext) {
  if constexpr (EXT) {
    return *reinterpret_cast<RT*>(ext);
  } else {
    __shared__ RT sm;
    return sm;
  }
}

// Contraction over segments seg = 0..nseg-1 and k in [0, ke) of each; ACOL / BCOL fix the storage
// order of the operands at compile time.
// ILV: the k-tile's products run row block by row block (i-major), with the A fragments of block
// i + 1 read while the products of block i issue, in an order pinned by scheduling groups: a wave
// then waits only for its B fragments and first A block after the barrier, instead of for most of
// the k-tile's fragment reads, and the LDS stays busy through the tile.
// WB > 0: the B operand is W as gemm2 writes it (the WB x WB blocks on and above the diagonal), read per
// part of the tile that lies in one block column: block (q-block, k-block) is read row-wise (W[q][k])
// when k-block >= q-block and column-wise (W[k][q], its transpose) otherwise; each part of the stage
// is laid out for its view.
// LAY: which output elements a lane holds, for the stores of the epilogue.  0: acc[i][j][e] is row
// 4 (lane / 16) + e, column lane % 16 of the 16 x 16 block; 1: A's slices are interleaved (ileave), so that
// acc[2 h][j] and acc[2 h + 1][j] are eight consecutive rows (row8_of); 2: the products are transposed and B's
// slices interleaved: acc[i][2 h] and acc[i][2 h + 1] are eight consecutive columns (col8_of) of row
// lane % 16.  Every element's sum runs in the same order in all of them.  brow (LAY 2): storage row of B for
// row r of the tile.
template <int BM, int BN, bool ALO, bool BLO, int S, bool ACOL, bool BCOL, bool RESET, bool F16, int WGM = 2,
          int WGN = 2, bool ILV = false, int WB = 0, int LAY = 0, typename FA, typename FB, typename EPI, typename BR = RowItself>
__device__ __forceinline__ void mainloop_dl(Ring<BM, BN, ALO, BLO, S>& sm, int nseg, int ke, int m0, int n0,
                                            FA A, FB B, f32x4 (&acc)[BM / (16 * WGM)][BN / (16 * WGN)], EPI epi,
                                            BR brow = BR{}) {
  constexpr bool BSYM = WB > 0;
  constexpr int SH = BSYM && WB < BN ? WB : BN;   // width of one part of the B tile (BSYM: within one block of W)
  static_assert(!BSYM || (BN % SH == 0 && WB % SH == 0 && !BCOL && (BN / WGN) <= SH), "BSYM: whole parts, one per wave");
  static_assert((LAY != 1 || !ACOL) && (LAY != 2 || (!BCOL && !BSYM)), "row operands are interleaved");
  constexpr int NW = WGM * WGN;   // waves in a WGM x WGN grid, each owning (BM / WGM) x (BN / WGN)
  auto mm = [](bf16x8 a, bf16x8 b, f32x4 c) { return LAY == 2 ? mma<F16>(b, a, c) : mma<F16>(a, b, c); };
  constexpr int MI = BM / (16 * WGM), NI = BN / (16 * WGN);
  constexpr int L = (ALO ? 2 : 1) * (BM / (16 * NW)) + (BLO ? 2 : 1) * (BN / (16 * NW));   // loads per wave per tile
  static_assert(L * (S - 2) < 64, "vmcnt range");
  const int wave = threadIdx.x >> 6, swave = __builtin_amdgcn_readfirstlane(wave);
  const int wm = (wave / WGN) * (BM / WGM), wn = (wave % WGN) * (BN / WGN);
  const int KT = (ke + BK - 1) / BK;
  const int total = nseg * KT;
  if (total <= 0) return;
  // the loads' addresses: a descriptor per operand and segment, lane offsets that stay, and the k-tile's offset
  constexpr int NP = BN / SH;   // BSYM: parts of the B tile
  unsigned ao[BM / (16 * NW)], bo[NP][SH / (16 * NW)], bc[NP][SH / (16 * NW)];
  const int lda = (int)A(0).ld, ldb = (int)B(0).ld;
  dl_offsets<BM, NW, ACOL>(ao, lda, m0, [&](int r) { return m0 + (LAY == 1 ? ileave(r) : r); });
#pragma unroll
  for (int h = 0; h < NP; ++h) {
    dl_offsets<SH, NW, BCOL>(bo[h], ldb, n0 + SH * h,
                             [&](int r) { return LAY == 2 ? brow(ileave(r)) : n0 + SH * h + r; });
    if constexpr (BSYM) dl_offsets<SH, NW, true>(bc[h], ldb, n0 + SH * h, [](int r) { return r; });
  }
  int lseg = 0, lk = 0;
  DOpnd a = A(0), b = B(0);
  int alim = record_limit(a.bytes), blim = record_limit(b.bytes);
  auto issue = [&](int stage) {
    const unsigned ka = 2u * (unsigned)(ACOL ? lk * lda : lk);
    dl_issue<BM, NW>(sm.a[stage][0], a.hi, alim, ao, ka, swave);
    if (ALO) dl_issue<BM, NW>(sm.a[stage][ALO ? 1 : 0], a.lo, alim, ao, ka, swave);
#pragma unroll
    for (int h = 0; h < NP; ++h) {
      if (BSYM && lk / WB < (n0 + SH * h) / WB) {
        const unsigned kb = 2u * (unsigned)(lk * ldb);
        dl_issue<SH, NW>(sm.b[stage][0] + h * SH * BK, b.hi, blim, bc[h], kb, swave);
        if (BLO) dl_issue<SH, NW>(sm.b[stage][BLO ? 1 : 0] + h * SH * BK, b.lo, blim, bc[h], kb, swave);
      } else {
        const unsigned kb = 2u * (unsigned)(BCOL ? lk * ldb : lk);
        dl_issue<SH, NW>(sm.b[stage][0] + h * SH * BK, b.hi, blim, bo[h], kb, swave);
        if (BLO) dl_issue<SH, NW>(sm.b[stage][BLO ? 1 : 0] + h * SH * BK, b.lo, blim, bo[h], kb, swave);
      }
    }
    lk += BK;
    if (lk >= ke) {
      lk = 0;
      ++lseg;
      a = A(lseg);
      b = B(lseg);
      alim = record_limit(a.bytes);
      blim = record_limit(b.bytes);
    }
  };
#pragma unroll
  for (int t = 0; t < S - 1; ++t)
    if (t < total) issue(t);
  if (RESET) zero(acc);
  // segments outside, k-tiles inside: the epilogue sits outside the inner loop, so the register
  // allocator keeps the accumulators in place through the k-loop (an epilogue inside the k-loop made
  // it shuttle them between AGPRs and VGPRs on every k-tile)
  // B fragment at wave column c (0 .. BN / WGN) of the stage; bv: the part is read column-wise
  // (BSYM; the wave's columns lie in one part)
  auto bfrag = [&](auto bv, const u16* base, int c) -> bf16x8 {
    if constexpr (BSYM) {
      return dl_frag<SH, decltype(bv)::value>(base + (wn / SH) * SH * BK, wn % SH + c);
    } else {
      return dl_frag<BN, BCOL>(base, wn + c);
    }
  };
  int stage = 0, it = 0;
  // one k-tile's products from stage `stage`; bv as for bfrag (a compile-time view, so that each
  // form is straight-line code with its own read counts in the scheduling groups)
  auto ktile = [&](auto bv) {
    constexpr bool BC = BSYM ? decltype(bv)::value : BCOL;   // B read with transposing reads
    if constexpr (ILV) {
      // reads of one A block: 1 (row layout) or 2 (transposing) instructions per hi / lo part
      constexpr int RA = (ACOL ? 2 : 1) * (ALO ? 2 : 1);
      constexpr int RB = (BC ? 2 : 1) * (BLO ? 2 : 1) * NI;
      constexpr int PR = NI * (1 + (BLO ? 1 : 0) + (ALO ? 1 : 0));   // products per A block
      bf16x8 bh[NI], bl[NI], ah[2], al[2];
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        bh[j] = bfrag(bv, sm.b[stage][0], 16 * j);
        if (BLO) bl[j] = bfrag(bv, sm.b[stage][BLO ? 1 : 0], 16 * j);
      }
      ah[0] = dl_frag<BM, ACOL>(sm.a[stage][0], wm);
      if (ALO) al[0] = dl_frag<BM, ACOL>(sm.a[stage][ALO ? 1 : 0], wm);
      __builtin_amdgcn_sched_group_barrier(0x100, RB + RA, 0);
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int c = i & 1, n = c ^ 1;
        if (i + 1 < MI) {
          ah[n] = dl_frag<BM, ACOL>(sm.a[stage][0], wm + 16 * (i + 1));
          if (ALO) al[n] = dl_frag<BM, ACOL>(sm.a[stage][ALO ? 1 : 0], wm + 16 * (i + 1));
          __builtin_amdgcn_sched_group_barrier(0x100, RA, 0);
        }
        // products in passes over j, so no two consecutive products share an accumulator
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = mm(ah[c], bh[j], acc[i][j]);
        if (BLO) {
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = mm(ah[c], bl[j], acc[i][j]);
        }
        if (ALO) {
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = mm(al[c], bh[j], acc[i][j]);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, PR, 0);
      }
    } else {
      bf16x8 ah[MI], bh[NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) ah[i] = dl_frag<BM, ACOL>(sm.a[stage][0], wm + 16 * i);
#pragma unroll
      for (int j = 0; j < NI; ++j) bh[j] = bfrag(bv, sm.b[stage][0], 16 * j);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
          acc[i][j] = mm(ah[i], bh[j], acc[i][j]);
      if (BLO) {
        bf16x8 bl[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) bl[j] = bfrag(bv, sm.b[stage][BLO ? 1 : 0], 16 * j);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[i][j] = mm(ah[i], bl[j], acc[i][j]);
      }
      if (ALO) {
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          const bf16x8 al = dl_frag<BM, ACOL>(sm.a[stage][ALO ? 1 : 0], wm + 16 * i);
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[i][j] = mm(al, bh[j], acc[i][j]);
        }
      }
    }
  };
  for (int seg = 0; seg < nseg; ++seg) {
    for (int kt = 0; kt < KT; ++kt, ++it) {
      if (it + S - 2 < total) __builtin_amdgcn_s_waitcnt(waitcnt_vm(L * (S - 2)));
      else __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      __builtin_amdgcn_s_barrier();
      if (it + S - 1 < total) issue((stage + S - 1) % S);
      if constexpr (BSYM) {
        // this wave's part is read column-wise when the k-tile's block lies before the part's
        if (kt * BK / WB < (n0 + wn) / WB) ktile(std::true_type{});
        else ktile(std::false_type{});
      } else {
        ktile(std::false_type{});
      }
      stage = (stage + 1 == S) ? 0 : stage + 1;
    }
    epi(seg, acc);
    if (RESET) zero(acc);
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  __builtin_amdgcn_s_barrier();
}

// Output row / column of component j of acc[i][jn] relative to the block tile origin.
template <int BM, int WGM = 2, int WGN = 2>
__device__ __forceinline__ int row_of(int i, int j) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  return (wave / WGN) * (BM / WGM) + i * 16 + 4 * (lane >> 4) + j;
}
template <int BN, int WGM = 2, int WGN = 2>
__device__ __forceinline__ int col_of(int jn) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  return (wave % WGN) * (BN / WGN) + jn * 16 + (lane & 15);
}

// LAY 1: first of the eight rows of acc[2 h], acc[2 h + 1]; LAY 2: first of the eight columns, and the row.
template <int BM, int WGM, int WGN>
__device__ __forceinline__ int row8_of(int h) {
  return ((threadIdx.x >> 6) / WGN) * (BM / WGM) + 32 * h + 8 * ((threadIdx.x & 63) >> 4);
}
template <int BN, int WGM, int WGN>
__device__ __forceinline__ int col8_of(int h) {
  return ((threadIdx.x >> 6) % WGN) * (BN / WGN) + 32 * h + 8 * ((threadIdx.x & 63) >> 4);
}
template <int BM, int WGM, int WGN>
__device__ __forceinline__ int row1_of(int i) {
  return ((threadIdx.x >> 6) / WGN) * (BM / WGM) + 16 * i + (threadIdx.x & 15);
}

// Lower-triangle tile t of a tt x tt tiling, ordered by column (tiles sharing tn are consecutive,
// so the blocks an XCD holds at once read few distinct column panels).
__device__ __forceinline__ void tri_tile(int t, int tt, int& tm, int& tn) {
  int r = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
  while ((r + 1) * (r + 2) / 2 <= t) ++r;
  while (r * (r + 1) / 2 > t) --r;
  tn = tt - 1 - r;
  tm = tt - 1 - (t - r * (r + 1) / 2);
}

// Tile t of a tm_n x tn_n grid in groups of G rows: consecutive tiles sweep G rows of one column,
// then the next column, so a run of consecutive tiles covers a compact G x (run / G) patch.
template <int G>
__device__ __forceinline__ void grouped_tile(int t, int tm_n, int tn_n, int& tm, int& tn) {
  const int per_group = G * tn_n;
  const int g = t / per_group, r = t % per_group;
  const int rows = min(G, tm_n - g * G);
  tm = g * G + r % rows;
  tn = r / rows;
}

// Shapes of the workspace operands (WsDims): Ct is nact32 x ldk, each XT_P is nact32 x ldx and each
// W_P is nact32 x ldw (nact32 = nact rounded up to 32), row-major, zero outside the valid block.

// Instance of a grouped launch that owns work item w: off[i] <= w < off[i+1].
__device__ __forceinline__ int find_instance(const int* __restrict__ off, int ninst, int w) {
  int lo = 0, hi = ninst - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= w) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// gemm1: XT_P[p][mu] = sum_nu Ct[p][nu] B_P[mu][nu], written as a hi/lo pair.  Tile G1M (p) x G1N in a
// WGM x WGN wave grid, one tile per work item (items covering several tiles measured slower: the
// epilogue's stores then stall the next tile's operand waits, as the vector-memory counter retires
// loads and stores in order).
// VEC: the n-tiles run over the stacked rows (P, mu) of all np B_P (bstride == nbf * ldb), each P counted as
// nbf rounded up to 8, so only the last tile of the launch is padding, where tiles of one P each pad
// every P's rows to a multiple of the tile (1200 rows on 256 tiles: 6 % of the products; 200 on 128: 22 %), and
// a lane's eight columns of XT are one aligned 16-byte store (2-byte stores of 32-byte runs: X of 1200 functions,
// 4800 rows 33.5 -> 31.7 ms; 16-byte stores at the rows' own alignment slowed 64 problems of 40 to 300
// functions from 2.55 to 3.65 ms).  The tile's first P is the base of its loads, so the 32-bit load offsets stay
// small however large the chunk is.
// Otherwise (rows that are not 16-byte aligned) one P per tile, staged through registers.
// EXT / ext: the ring is the caller's (see ring_of); BUDGET: LDS bytes for the ring (0: the whole
// unit's LDS shared by MINB blocks).
template <int TERMS, bool BLO, int G1M, int G1N, int WGM, int WGN, int MINB, bool VEC, bool BATCH = false, bool EXT = false,
          int BUDGET = 0>
__device__ __forceinline__ void gemm1_body(int w, const G1Args& g, void* ext = nullptr) {
  constexpr bool ALO = TERMS >= 2;
  constexpr int MI = G1M / (16 * WGM), NI = G1N / (16 * WGN);
  const int nbf = g.nbf, nact = g.nact, ldx = g.ldx, nbf8 = (nbf + 7) & ~7;
  const int tm_n = (nact + G1M - 1) / G1M;
  int P0, m0, r0;   // first P of the tile, and the tile's first row there
  if constexpr (VEC) {
    m0 = (w % tm_n) * G1M;
    const uint32_t n0 = (uint32_t)(w / tm_n) * G1N;
    P0 = (int)(n0 / (uint32_t)nbf8);
    r0 = (int)(n0 - (uint32_t)P0 * nbf8);
  } else {
    const int tn_n = (nbf + G1N - 1) / G1N;
    P0 = w / (tm_n * tn_n);
    const int tile = w % (tm_n * tn_n);
    m0 = (tile / tn_n) * G1M;
    r0 = (tile % tn_n) * G1N;
  }
  const long long pstride = (long long)g.ws.nact32 * ldx;
  u16* XTh = g.xt_hi + P0 * pstride;
  u16* XTl = g.xt_lo ? g.xt_lo + P0 * pstride : nullptr;
  // split mode: X is written as the fp16 pair of X sX
  const float xmul = TERMS >= 2 ? chunk_scales(g.bnd, g.chunk, TERMS == 3).xmul : 1.0f;
  f32x4 acc[MI][NI];
  // XT rows to nact32 and columns to ldx are written, those past nact (Ct's are zero) and nbf with zeros; a
  // batch clears this padding once, when its plan is made
  const int prows = BATCH ? nact : g.ws.nact32;
  auto epi = [&](int, f32x4(&a)[MI][NI]) {
    int mu[NI / 2];
    long long xo[NI / 2];
#pragma unroll
    for (int h = 0; h < NI / 2; ++h) {
      const int c = r0 + col8_of<G1N, WGM, WGN>(h), dP = VEC ? (int)((uint32_t)c / (uint32_t)nbf8) : 0;
      mu[h] = P0 + dP < g.np ? c - dP * nbf8 : nbf8;
      xo[h] = dP * pstride + mu[h];
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int p = m0 + row1_of<G1M, WGM, WGN>(i);
      if (p >= prows) continue;
#pragma unroll
      for (int h = 0; h < NI / 2; ++h) {
        if (mu[h] >= nbf8) continue;
        u32x4 hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f32x4 v = a[i][2 * h + (e >> 1)];
          const float v0 = mu[h] + 2 * e < nbf ? v[2 * (e & 1)] : 0.f, v1 = mu[h] + 2 * e + 1 < nbf ? v[2 * (e & 1) + 1] : 0.f;
          uint32_t x, y = 0;
          if (TERMS == 1) x = cvt2_bf16(v0, v1);
          else split2_f16(v0 * xmul, v1 * xmul, x, y);
          hi[e] = x;
          lo[e] = y;
        }
        const long long o = xo[h] + (long long)p * ldx;
        *reinterpret_cast<u32x4*>(XTh + o) = hi;
        if (XTl) *reinterpret_cast<u32x4*>(XTl + o) = lo;
      }
    }
    if (!BATCH && ldx > nbf8) {
#pragma unroll
      for (int h = 0; h < NI / 2; ++h)
        if (mu[h] + 8 == nbf8)
#pragma unroll
          for (int i = 0; i < MI; ++i) {
            const int p = m0 + row1_of<G1M, WGM, WGN>(i);
            if (p >= prows) continue;
            for (int k = 8; mu[h] + k < ldx; k += 8) {
              const long long o = xo[h] + (long long)p * ldx + k;
              *reinterpret_cast<u32x4*>(XTh + o) = u32x4{0u, 0u, 0u, 0u};
              if (XTl) *reinterpret_cast<u32x4*>(XTl + o) = u32x4{0u, 0u, 0u, 0u};
            }
          }
    }
  };
  const long long o = P0 * g.bstride;
  if constexpr (VEC) {
    // the LDS of one compute unit is shared by MINB blocks
    constexpr int S = ring_depth(G1M, G1N, ALO, BLO, BUDGET > 0 ? BUDGET : (MINB == 2 ? 81920 : 163840));
    auto& sm = ring_of<Ring<G1M, G1N, ALO, BLO, S>, EXT>(ext);
    auto A = [&](int) { return DOpnd{g.ct_hi, g.ct_lo, g.ldk, g.ws.ct_bytes}; };
    auto B = [&](int) { return DOpnd{g.b_hi + o, BLO ? g.b_lo + o : nullptr, g.ldb, g.b_bytes - 2 * o}; };
    auto brow = [&](int r) {   // row of the stored B of the tile's row r
      const int c = r0 + r, dP = min((int)((uint32_t)c / (uint32_t)nbf8), g.np - 1 - P0);
      return dP * nbf + min(c - dP * nbf8, nbf - 1);
    };
    mainloop_dl<G1M, G1N, ALO, BLO, S, false, false, true, (TERMS == 3), WGM, WGN, (WGM * WGN == 8), false, 2>(
        sm, 1, nbf, m0, 0, A, B, acc, epi, brow);
  } else {
    static_assert(VEC || (WGM == 2 && WGN == 2), "register-staged path: 2 x 2 waves");
    __shared__ Stage<G1M, G1N, ALO, BLO> sm;
    mainloop<G1M, G1N, ALO, BLO, (TERMS == 3)>(sm, nbf, m0, r0, Opnd{g.ct_hi, g.ct_lo, g.ldk, nact, nbf},
                                               Opnd{g.b_hi + o, BLO ? g.b_lo + o : nullptr, g.ldb, nbf, nbf}, acc);
    epi(0, acc);
  }
}

// gemm2: b_P = Ct XT_P^T on lower-triangle tiles; Kpart[s] += sum_{P in s} b^2 (lower triangle, summed
// over the successive P-chunks of one call, the first of which stores: kset), D[P][p] = b_pp, W_P = b o beta
// as a hi/lo pair, written only as the transposed image of each tile: the TT x TT blocks on and above the
// diagonal, which gemm3 reads.
// 2 x WGN waves.  128 tile, WGN 2: 4 waves of 64 x 64, two blocks per compute unit: such a wave reads 16 KB of LDS per
// k-tile for 48 products, a 64 x 32 one 12 KB for 24, which LDS bandwidth bounds, and while one block forms K and W
// the other keeps the matrix cores busy; against 8 waves and one block, b over the step: 1200 functions 42.7 ->
// 35.5 ms, 500 functions (300 active, 2000 rows) 1.40 -> 1.05, 413 functions 0.85 -> 0.66 (with the splits that the
// planner takes for it).  WGN 4: 8 waves of 64 x 32, for launches whose blocks wait rather than compute (G2_FEW).
// The sums of b^2 are float32 over at most krows rows (at most 8), then float64 in Kpart: each block adds to its own
// partial sums only, with atomics, which need no wait (as loads and stores, 1200 functions in 164 splits 53.0 ms, with
// atomics 40.0).
// TT: the square tile (128, or 64 for the short active spaces of batch instances, with 4 waves).
// BATCH: one launch covers every P of the problem (K is stored); the blocks on the diagonal hold W[p][q]
// itself, in place of its image (b_pq and b_qp differ in the last bits): their products are formed transposed, so that
// a lane holds eight consecutive q (by a transpose between lanes, 4 problems of 30 functions took 206 us, now 172; 64 of
// 50 functions 244 and 228; as 2-byte stores of W[p][q] and its image in every tile, b of 64 problems of 40 to 300
// functions took 1.98 ms).
template <int TERMS, int TT = T2, bool BATCH = false, int WGN = 2, bool EXT = false, int BUDGET = 0>
__device__ __forceinline__ void gemm2_body(int w, const G2Args& g, void* ext = nullptr) {
  constexpr bool LO = TERMS >= 3;
  constexpr int NI = TT / (16 * WGN), MI = TT / 32;
  const int nbf = g.nbf, nact = g.nact, np = g.np, nsplit = g.nsplit, ldw = g.ldw, ldx = g.ldx;
  const int tt = (nact + TT - 1) / TT;
  const int ntri = tt * (tt + 1) / 2;
  const int s = w / ntri;
  int tm, tn;
  tri_tile(w % ntri, tt, tm, tn);
  const int m0 = tm * TT, n0 = tn * TT;
  const int pb = (int)((long long)np * s / nsplit), pe = (int)((long long)np * (s + 1) / nsplit);
  // split mode: the accumulator holds b sC sX; W is written as the fp16 pair of W sW
  float invB = 1.0f, wmul = 1.0f;
  if constexpr (LO) {
    const Scales sc = chunk_scales(g.bnd, g.chunk, false);
    invB = sc.invB;
    wmul = sc.wmul;
  }
  const bool diag = (tm == tn);
  const int wrows = BATCH ? nact : g.ws.nact32;
  constexpr int S = ring_depth(TT, TT, LO, LO, BUDGET > 0 ? BUDGET : WGN == 2 ? 81920 : 163840);
  auto& sm = ring_of<Ring<TT, TT, LO, LO, S>, EXT>(ext);
  auto A = [&](int) { return DOpnd{g.ct_hi, g.ct_lo, g.ldk, g.ws.ct_bytes}; };
  auto B = [&](int seg) {
    const long long off = (long long)(pb + seg) * g.ws.nact32 * ldx;
    return DOpnd{g.xt_hi + off, LO ? g.xt_lo + off : nullptr, ldx, g.ws.xt_bytes - 2 * off};
  };
  // LAY as in mainloop_dl: runs (u, v) of eight elements along p (1) or q (2), from r0(u, v) on, at q or p c(u, v)
  auto run = [&](auto lay) {
    constexpr int LAY = decltype(lay)::value;
    constexpr int NU = LAY == 1 ? MI / 2 : MI, NV = LAY == 1 ? NI : NI / 2;
    auto r0 = [&](int u, int v) { return LAY == 1 ? m0 + row8_of<TT, 2, WGN>(u) : n0 + col8_of<TT, 2, WGN>(v); };
    auto c = [&](int u, int v) { return LAY == 1 ? n0 + col_of<TT, 2, WGN>(v) : m0 + row1_of<TT, 2, WGN>(u); };
    auto at = [&](f32x4(&a)[MI][NI], int u, int v, int e) -> f32x4& {
      return LAY == 1 ? a[2 * u + (e >> 2)][v] : a[u][2 * v + (e >> 2)];
    };
    // beta (symmetric, nact32 x nact32) of this lane's runs.  With 32 x 32 and 64 x 32 elements per wave it is kept in
    // registers for the whole P-range; with 64 x 64, whose sums of b^2 and accumulators fill them, each P reads it anew
    constexpr bool BREG = MI * NI <= 8;
    auto beta8 = [&](int u, int v, f32x4(&b)[2]) {
      const int p0 = r0(u, v), q = c(u, v);
      if (p0 < g.ws.nact32 && q < g.ws.nact32) {
        const f32x4* src = reinterpret_cast<const f32x4*>(g.beta32 + (long long)q * g.ws.nact32 + p0);
        b[0] = src[0] * wmul;
        b[1] = src[1] * wmul;
      } else b[0] = b[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    f32x4 bet[BREG ? NU : 1][BREG ? NV : 1][2];
    if constexpr (BREG)
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int v = 0; v < NV; ++v) beta8(u, v, bet[u][v]);
    f32x4 kacc[MI][NI], acc[MI][NI];
    zero(kacc);
    bool kset = BATCH || g.kset;
    auto add_k = [&]() {   // to the block's own partial sums
      double* Kp = g.Kpart + (long long)s * nact * nact;
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int x = r0(u, v) + e, y = c(u, v), p = LAY == 1 ? x : y, q = LAY == 1 ? y : x;
            if (p < nact && q <= p) {
              double* k = Kp + (long long)p * nact + q;
              const double sum = (double)at(kacc, u, v, e)[e & 3];
              if (kset) *k = sum;
              else unsafeAtomicAdd(k, sum);   // nobody else's: an add that needs no wait
            }
          }
    };
    int kleft = min(g.krows, pe - pb);   // rows of P left for the float32 sums
    auto epi = [&](int seg, f32x4(&a)[MI][NI]) {
      const int P = pb + seg;
      u16* Wh = g.w_hi + (long long)P * g.ws.nact32 * ldw;
      u16* Wl = LO ? g.w_lo + (long long)P * g.ws.nact32 * ldw : nullptr;
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const int r = r0(u, v), cc = c(u, v);
          float wv[8];
          f32x4 bv[2];
          if constexpr (BREG) {
            bv[0] = bet[u][v][0];
            bv[1] = bet[u][v][1];
          } else beta8(u, v, bv);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float x = at(a, u, v, e)[e & 3], b = x * invB;
            at(kacc, u, v, e)[e & 3] += b * b;
            wv[e] = x * bv[e >> 2][e & 3];
            if (diag && r + e == cc && cc < nact) g.Dc[(long long)P * nact + cc] = (double)b;
          }
          u32x4 hi, lo;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            uint32_t x, y = 0;
            if constexpr (LO) split2_f16(wv[2 * e], wv[2 * e + 1], x, y);
            else x = cvt2_bf16(wv[2 * e], wv[2 * e + 1]);
            hi[e] = x;
            lo[e] = y;
          }
          // rows and columns from nact to nact32 receive zeros; a batch clears them once, when its plan is made
          if (cc < wrows && r < wrows) {
            const long long o = (long long)cc * ldw + r;
            *reinterpret_cast<u32x4*>(Wh + o) = hi;
            if (LO) *reinterpret_cast<u32x4*>(Wl + o) = lo;
          }
        }
      if (!BATCH && --kleft <= 0) {
        add_k();
        zero(kacc);
        kset = false;
        kleft = min(g.krows, pe - 1 - P);
      }
    };
    mainloop_dl<TT, TT, LO, LO, S, false, false, true, LO, 2, WGN, false, 0, LAY>(sm, pe - pb, nbf, m0, n0, A, B, acc, epi,
                                                                               [&](int r) { return n0 + r; });
    if (BATCH) add_k();
  };
  if constexpr (BATCH)
    if (diag) {
      run(std::integral_constant<int, 2>{});
      return;
    }
  run(std::integral_constant<int, 1>{});
}

// gemm3: Ypart[s][mu][q] = sum_{P in s} sum_r XT_P[r][mu] W_P[q][r].  XT is read as a col operand,
// W as a row operand (each WB-wide block from the orientation gemm2 stored it in: rows on and above
// the diagonal, columns below); every block walks (P, r) in the same order, so blocks of one
// split that share an operand panel read it at about the same time.  Split mode: 3 fp16 products
// (2 products, dropping X_lo W_hi at about 2^-12 relative, left lambda 2.2e-5 from the exact values on
// a 77-function edge shape).
// Tile G3M (mu) x G3N (q), waves in a WGM x WGN grid.  Each wave's share of the tile sets how many
// matrix-core products one byte read from LDS feeds: a 64 x 64 wave reads 16 KB per k-tile for 48
// products, a 128 x 64 wave 24 KB for 96; LDS bandwidth (about 128 bytes per clock per compute unit)
// is what limits the 64 x 64 form.
// WB: the tile of the b contraction that wrote W.
template <int TERMS, int G3M, int G3N, int WGM, int WGN, int MINB, int WB, bool EXT = false, int BUDGET = 0>
__device__ __forceinline__ void gemm3_body(int w, const G3Args& g, void* ext = nullptr) {
  constexpr bool LO = TERMS >= 3;
  constexpr int MI = G3M / (16 * WGM), NI = G3N / (16 * WGN);
  const int nbf = g.nbf, nact = g.nact, np = g.np, nsplit = g.nsplit, ldx = g.ldx, ldw = g.ldw;
  const int tm_n = (nbf + G3M - 1) / G3M, tn_n = (nact + G3N - 1) / G3N;
  const int s = w / (tm_n * tn_n);
  int tm, tn;
  grouped_tile<4>(w % (tm_n * tn_n), tm_n, tn_n, tm, tn);
  const int m0 = tm * G3M, n0 = tn * G3N;
  const int pb = (int)((long long)np * s / nsplit), pe = (int)((long long)np * (s + 1) / nsplit);
  f32x4 acc[MI][NI];
  zero(acc);
  auto none = [&](int, f32x4(&)[MI][NI]) {};
  // the 128 x 128 tile runs two blocks per compute unit (two-stage ring each): while one block
  // waits on its fragment reads or barrier, the other keeps the matrix cores busy
  constexpr int S = ring_depth(G3M, G3N, LO, LO, BUDGET > 0 ? BUDGET : (MINB == 2 ? 81920 : 163840));
  auto& sm = ring_of<Ring<G3M, G3N, LO, LO, S>, EXT>(ext);
  auto A = [&](int seg) {
    const long long off = (long long)(pb + seg) * g.ws.nact32 * ldx;
    return DOpnd{g.xt_hi + off, LO ? g.xt_lo + off : nullptr, ldx, g.ws.xt_bytes - 2 * off};
  };
  auto B = [&](int seg) {
    const long long off = (long long)(pb + seg) * g.ws.nact32 * ldw;
    return DOpnd{g.w_hi + off, LO ? g.w_lo + off : nullptr, ldw, g.ws.w_bytes - 2 * off};
  };
  mainloop_dl<G3M, G3N, LO, LO, S, true, false, false, LO, WGM, WGN, (WGM * WGN == 8), WB>(sm, pe - pb, nact, m0, n0,
                                                                                           A, B, acc, none);
  float* Y = g.Ypart + (long long)s * nbf * nact;
  const float invY = LO ? chunk_scales(g.bnd, g.chunk, false).invY : 1.0f;   // acc = Y sX sW
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int jn = 0; jn < NI; ++jn)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int m = m0 + row_of<G3M, WGM, WGN>(i, j), n = n0 + col_of<G3N, WGM, WGN>(jn);
        if (m < nbf && n < nact) Y[(long long)m * nact + n] = acc[i][jn][j] * invY;
      }
}

template <int TERMS, bool BLO, int G1M, int G1N, int WGM, int WGN, int MINB, bool VEC>
__global__ __launch_bounds__(64 * WGM * WGN, MINB) void gemm1_kernel(G1Args g) {
  const int w = xcd_item(g1_items(g, G1M, G1N, VEC));
  if (w < 0) return;
  gemm1_body<TERMS, BLO, G1M, G1N, WGM, WGN, MINB, VEC>(w, g);
}
template <int TERMS, int WGN>
__global__ __launch_bounds__(128 * WGN, WGN == 2 ? 2 : 1) void gemm2_kernel(G2Args g) {
  const int w = xcd_item(g2_items(g, T2));
  if (w < 0) return;
  gemm2_body<TERMS, T2, false, WGN>(w, g);
}
template <int TERMS, int G3M, int G3N, int WGM, int WGN, int MINB>
__global__ __launch_bounds__(64 * WGM * WGN, MINB) void gemm3_kernel(G3Args g) {
  const int w = xcd_item(g3_items(g, G3M, G3N));
  if (w < 0) return;
  gemm3_body<TERMS, G3M, G3N, WGM, WGN, MINB, T2>(w, g);
}

// Grouped forms: one launch over the work items of every instance of a batch.  The tile width along
// the active orbitals is a template parameter (128, or 64 when the instances' active spaces are
// short); the 64-wide forms run 4 waves and two blocks per compute unit.
// (X at two blocks per compute unit, as the single-problem 128 x 128 form: 8.6 -> 7.7 ms per
// 64-instance PES batch)
template <int TERMS, int TM>
__global__ __launch_bounds__(256, 2) void gemm1_grouped(const G1Args* __restrict__ tab, const int* __restrict__ off,
                                                        int ninst, int total) {
  const int w = xcd_item(total);
  if (w < 0) return;
  const int i = find_instance(off, ninst, w);
  const G1Args g = tab[i];
  gemm1_body<TERMS, false, TM, 128, 2, 2, 2, true, true>(w - off[i], g);
}
template <int TERMS, int TT, int WGN>
__global__ __launch_bounds__(128 * WGN, WGN == 2 ? 2 : 1) void gemm2_grouped(
    const G2Args* __restrict__ tab, const int* __restrict__ off, int ninst, int total) {
  const int w = xcd_item(total);
  if (w < 0) return;
  const int i = find_instance(off, ninst, w);
  const G2Args g = tab[i];
  gemm2_body<TERMS, TT, true, WGN>(w - off[i], g);
}
template <int TERMS, int TN, int WB>
__global__ __launch_bounds__(256, 2) void gemm3_grouped(const G3Args* __restrict__ tab, const int* __restrict__ off,
                                                        int ninst, int total) {
  const int w = xcd_item(total);
  if (w < 0) return;
  const int i = find_instance(off, ninst, w);
  const G3Args g = tab[i];
  gemm3_body<TERMS, 128, TN, 2, 2, 2, WB>(w - off[i], g);
}

// ------------------------------------------------------------------------------------------
// Persistent batch kernel.  Every block loops: claim a work item of the first instance (in index
// order) whose current phase still has unclaimed items -- every item of the phases before it being
// complete, a claimed item never waits -- run it, publish it.  The block that completes a phase's
// last item moves the instance to the next phase; the instance's last phase stamps its completion
// time.  A block that finds nothing to claim polls; once stall_ticks of the device clock pass with
// no item completed anywhere it raises the stall flag and exits, and the others exit on seeing the
// flag, so every block ends whatever happens.
constexpr int PBUDGET = 79872;   // LDS of the largest ring; with the small arrays, two blocks per unit

template <int TX, int TY>
union PersistLds {
  Ring<TX, 128, true, false, ring_depth(TX, 128, true, false, PBUDGET)> x;
  Ring<64, 64, true, true, ring_depth(64, 64, true, true, PBUDGET)> b;
  Ring<128, TY, true, true, ring_depth(128, TY, true, true, PBUDGET)> y;
  f64t::F64Smem f;
};

__device__ __forceinline__ int ld_dev(const int* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// The call-level scale bounds (the grouped launches take two launches and a global array for them; the words
// are the same): a wave per orbital, its maxima raised in the instance's words.
__host__ __device__ inline int bnd_items(int nact) { return cdiv(nact, 4) < PERSIST_PARTS ? cdiv(nact, 4) : PERSIST_PARTS; }
__device__ inline void persist_bounds(const BInst& d, int part, int nparts, uint32_t* words) {
  const int lane = threadIdx.x & 63;
  for (int q = 4 * part + (threadIdx.x >> 6); q < d.nact; q += 4 * nparts) {
    double s1 = 0.0, cm = 0.0, sa = 0.0, bm = 0.0;
    for (int mu = lane; mu < d.nbf; mu += 64) {
      const double c = fabs(d.C[(long long)mu * d.nbf + q]);
      s1 += c;
      cm = fmax(cm, c);
    }
    for (int r = lane; r < d.nact; r += 64) {
      double a, b;
      pnof_coeff(q, r, d.n[q], d.n[r], d.npairs, d.ncwo, d.nsingle, d.functional, a, b);
      sa += fabs(a);
      bm = fmax(bm, fabs(b));
    }
    for (int off = 32; off > 0; off >>= 1) {
      s1 += __shfl_down(s1, off, 64);
      sa += __shfl_down(sa, off, 64);
      cm = fmax(cm, __shfl_down(cm, off, 64));
      bm = fmax(bm, __shfl_down(bm, off, 64));
    }
    if (lane == 0) {
      atomicMax(&words[0], __float_as_uint((float)s1));
      atomicMax(&words[1], __float_as_uint((float)cm));
      atomicMax(&words[2], __float_as_uint((float)sa));
      atomicMax(&words[3], __float_as_uint((float)bm));
    }
  }
}
__device__ inline void persist_prep(const BInst& d, int part, int nparts, const uint32_t* words) {
  const int* m = reinterpret_cast<const int*>(words);
  const uint32_t w0 = (uint32_t)ld_dev(m + 1), w1 = (uint32_t)ld_dev(m);
  if (part == 0 && threadIdx.x == 0) {
    d.bnd[0] = w0;
    d.bnd[1] = w1;
    d.bnd[2] = __float_as_uint(__int_as_float(ld_dev(m + 3)) + __int_as_float(ld_dev(m + 2)));
  }
  // sC exactly as chunk_scales forms it from bnd[0]
  bdev::prep(d, part, nparts, ldexpf(1.0f, 13 - bound_exp(__uint_as_float(w0) * 1.01f)));
}

template <int TX, int TY>
__device__ __forceinline__ void persist_item(const PArgs& a, int i, int ph, int idx, void* lds) {
  const BInst& d = a.inst[i];
  f64t::F64Smem& fs = *reinterpret_cast<f64t::F64Smem*>(lds);
  const int n = a.ninst;
  switch (ph) {
    case PH_BND:
      persist_bounds(d, idx, bnd_items(d.nact), reinterpret_cast<uint32_t*>(a.sc.claim + i * PH_ROW + PH_BND_WORDS));
      break;
    case PH_PREP:
      persist_prep(d, idx, PERSIST_PARTS, reinterpret_cast<const uint32_t*>(a.sc.claim + i * PH_ROW + PH_BND_WORDS));
      break;
    case PH_X: {
      const G1Args g = a.g1[i];
      const int nh = f64t::grouped_tiles(d.nbf, d.nact), nt = g1_items(g, TX, 128, true);
      if (idx < nh) {
        f64t::grouped_tile<false, true>(a.f64[i], idx, fs);                                // H C_A
      } else {
        const int t0 = (idx - nh) * PERSIST_XG, t1 = t0 + PERSIST_XG < nt ? t0 + PERSIST_XG : nt;
        for (int t = t0; t < t1; ++t) {
          if (t > t0) __syncthreads();   // the ring of the tile before is free again
          gemm1_body<2, false, TX, 128, 2, 2, 2, true, true, true, PBUDGET>(t, g, lds);
        }
      }
      break;
    }
    case PH_B: {
      const G2Args g = a.g2[i];
      if (idx == 0) bdev::hpp(d, 0, 1);
      else gemm2_body<3, 64, true, 2, true, PBUDGET>(idx - 1, g, lds);
      break;
    }
    case PH_DA:
      f64t::grouped_tile<false, true>(a.f64[n + i], idx, fs);                              // D alpha
      break;
    case PH_DIAG:
      bdev::add_diag(d, idx, PERSIST_PARTS);
      break;
    case PH_Y: {
      const G3Args g = a.g3[i];
      const int nj = f64t::grouped_tiles(d.nact, d.nact);
      if (idx < nj) f64t::grouped_tile<true, true>(a.f64[2 * n + i], idx, fs);             // J = D^T D
      else gemm3_body<3, 128, TY, 2, 2, 2, 64, true, PBUDGET>(idx - nj, g, lds);
      break;
    }
    case PH_RED:
      bdev::reduce(d, idx, PERSIST_PARTS);
      break;
    case PH_EY:
      if (idx < BATCH_EPARTS) bdev::energy_part(d, idx);
      else bdev::y_assemble(d, idx - BATCH_EPARTS, PERSIST_PARTS);
      break;
    case PH_LAM:
      f64t::grouped_tile<true, true>(a.f64[3 * n + i], idx, fs);                          // lambda = C^T Y
      break;
    case PH_FIN:
      bdev::finish(d, idx, PERSIST_PARTS);
      break;
    default:
      bdev::vjp(d, 0, 1);
      break;
  }
}

// Every instance runs on one die: a block reads the id of the die it runs on from the hardware and
// claims items of that die's group of instances only (group = id modulo the device's die count;
// the first block of a group records its die id, and a block of another die mapping to the same
// group stops the run with the error flag rather than share an L2-resident instance).  All of an instance's intermediate data then stays in
// one L2, so a block makes its item's stores visible by waiting for them to reach L2 (before the
// barrier that ends the item) and sees the other blocks' stores after invalidating its compute
// unit's L1 (after claiming); no L2 write-back or invalidation is needed.  The scheduling words are
// touched with device-scope atomics and coherent loads only.
// A block that ends an item claims the next one of the same phase in the round trip that publishes it, and looks
// further only when the phase has none left; each instance's counters and each die's progress word lie in a line of
// their own.  (With one progress word for the device, raised by every item, and the state read in seven round trips
// an item, halving the items' size cost 24 problems of 40 to 180 functions 1.33 -> 1.81 ms; now it costs nothing.
// With this, the bounds and prep in parts, J beside Y instead of before it, and 32 parts of the element-wise phases
// instead of 8: 1.33 -> 0.96 ms.)  What bounds the run is the die that holds the largest problem.
// The scheduling runs in wavefront 0 as a whole; the other wavefronts wait at the barrier.  Lane l
// of wavefront 0 looks at the die's instance base + l, a ballot picks the first one with unclaimed
// items of its open phase, and lane 0 alone performs the atomics (every value the lanes branch on
// is uniform).  Publishing an item and claiming the next form a single region of wavefront 0 at
// the top of the loop, so that no code path of the loop distinguishes lanes of one wavefront around
// a barrier: were the two separate lane-0 regions on either side of the loop's back edge, the
// compiler may join them into one and leave lanes 1..63 cycling through the barriers without lane 0.
__device__ __forceinline__ int die_id() { return (int)__builtin_amdgcn_s_getreg((3 << 11) | 20); }   // XCC_ID[3:0]
__device__ __forceinline__ void l1_invalidate() { asm volatile("buffer_inv sc0" ::: "memory"); }

template <int TX, int TY>
__global__ __launch_bounds__(256, 2) void batch_persist_k(PArgs a) {
  __shared__ PersistLds<TX, TY> u;
  __shared__ int s_it[3];
  const PSched& sc = a.sc;
  const int die = die_id(), grp = die % sc.ndie;
  if (threadIdx.x == 0) {
    const int prev = atomicCAS(sc.die_of + grp, -1, die);
    s_it[0] = (prev == -1 || prev == die) ? 0 : 1;
    if (s_it[0]) atomicExch(sc.prog + 2, 2);   // two dies in one group: stop every block
  }
  __syncthreads();
  if (s_it[0]) return;
  const int lo = __builtin_amdgcn_readfirstlane(sc.xoff[grp]), hi = __builtin_amdgcn_readfirstlane(sc.xoff[grp + 1]);
  const int lane = threadIdx.x;   // in wavefront 0
  const bool lead = threadIdx.x == 0;
  int last = -1;   // instance * PH_N + phase of the item this block completed last
  for (;;) {
    if (threadIdx.x < 64) {
      int inst = -1, ph = 0, idx = 0;
      if (last >= 0) {   // publish it, and claim the next item of its phase in the same round trip
        const int i = last / PH_N, p = last % PH_N, cc = sc.cnt[last];
        int* row = sc.claim + i * PH_ROW + p;
        int dn = 0, c = 0;
        if (lead) {
          c = atomicAdd(row, 1);
          dn = atomicAdd(row + PH_DONE, 1) + 1;
          __hip_atomic_store(sc.prog + PROG_ROW * (1 + grp), (int)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        c = __builtin_amdgcn_readlane(c, 0);
        dn = __builtin_amdgcn_readlane(dn, 0);
        if (dn == cc && lead) {
          if (p + 1 == PH_N) __hip_atomic_store(sc.t_end + i, wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          atomicExch(sc.phase + i, p + 1);
          if (p + 1 == PH_N) atomicAdd(sc.prog + 1, 1);
        }
        if (c < cc) {
          inst = i;
          ph = p;
          idx = c;
        }
      }
      // lanes: the groups' progress words, then instances completed and the stall flag
      const int* word = sc.prog + (lane < sc.ndie ? PROG_ROW * (1 + lane) : lane == sc.ndie ? 1 : 2);
      int seen = 0;
      unsigned long long t_seen = wall_clock64();
      for (bool first = true; inst < 0; first = false) {
        const int now = lane < sc.ndie + 2 ? ld_dev(word) : 0;
        if (__builtin_amdgcn_readlane(now, sc.ndie) >= a.ninst || __builtin_amdgcn_readlane(now, sc.ndie + 1) != 0) break;
        const unsigned long long t = wall_clock64();
        if (first || __ballot(lane < sc.ndie && now != seen) != 0) {
          seen = now;
          t_seen = t;
        } else if (t - t_seen > sc.stall_ticks) {
          if (lead) atomicExch(sc.prog + 2, 1);
          break;
        }
        for (int base = lo; base < hi && inst < 0; base += 64) {
          int i = -1, p = PH_N, k = 0, cnt = 0;
          bool open = false;
          if (base + lane < hi) {
            i = sc.order[base + lane];
            p = ld_dev(sc.phase + i);
            if (p < PH_N) {
              k = i * PH_ROW + p;
              cnt = sc.cnt[i * PH_N + p];
              open = ld_dev(sc.claim + k) < cnt;
            }
          }
          unsigned long long m = __ballot(open);
          while (m) {
            const int l = __ffsll((long long)m) - 1;
            const int kk = __builtin_amdgcn_readlane(k, l), cc = __builtin_amdgcn_readlane(cnt, l);
            int c = 0;
            if (lead) c = atomicAdd(sc.claim + kk, 1);
            c = __builtin_amdgcn_readlane(c, 0);
            if (c < cc) {
              inst = __builtin_amdgcn_readlane(i, l);
              ph = __builtin_amdgcn_readlane(p, l);
              idx = c;
              break;
            }
            m &= m - 1;   // that phase ran out meanwhile: the next instance
          }
        }
        if (inst < 0) __builtin_amdgcn_s_sleep(8);
      }
      if (inst >= 0) l1_invalidate();
      if (lead) {
        s_it[0] = inst;
        s_it[1] = ph;
        s_it[2] = idx;
      }
    }
    __syncthreads();
    const int inst = __builtin_amdgcn_readfirstlane(s_it[0]), ph = __builtin_amdgcn_readfirstlane(s_it[1]),
              idx = __builtin_amdgcn_readfirstlane(s_it[2]);
    if (inst < 0) return;
    persist_item<TX, TY>(a, inst, ph, idx, &u);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // this wavefront's stores have reached L2
    __syncthreads();
    last = inst * PH_N + ph;
  }
}

// Clears the scheduling state of a run and stamps its start.
__global__ void persist_reset_k(PSched sc, int ninst) {
  for (int i = threadIdx.x; i < ninst * PH_ROW; i += blockDim.x) sc.claim[i] = 0;
  for (int i = threadIdx.x; i < ninst; i += blockDim.x) sc.phase[i] = 0;
  for (int i = threadIdx.x; i < sc.ndie; i += blockDim.x) sc.die_of[i] = -1;
  for (int i = threadIdx.x; i < PROG_ROW * (1 + sc.ndie); i += blockDim.x) sc.prog[i] = 0;
  if (threadIdx.x == 0) *sc.t_start = wall_clock64();
}

// Rows (P, mu) of a stacked X launch are counted in 32 bits.
inline bool rows32(const G1Args& g) { return (long long)g.np * round_up(g.nbf, 8) < (1LL << 31); }

inline dim3 xcd_grid(long long items) { return dim3((unsigned)(cdiv(items, NXCD) * NXCD)); }

}  // namespace

inline bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
template <int TERMS, bool BLO, int G1M, int G1N, int WGM, int WGN, int MINB>
static void launch_g1(hipStream_t s, const G1Args& g) {
  const dim3 grid = xcd_grid(g1_items(g, G1M, G1N, true));
  // direct-to-LDS needs 16-byte aligned rows of B, densely stacked (the caller's own when nbf % 8 == 0,
  // otherwise the chunk's padded copy)
  const bool vec = rows32(g) && (g.ldb % 8 == 0) && (g.bstride == (long long)g.nbf * g.ldb) && al16(g.b_hi) &&
                   (!g.b_lo || al16(g.b_lo)) && al16(g.ct_hi) && (!g.ct_lo || al16(g.ct_lo)) && (g.ldk % 32 == 0) &&
                   (g.ldx % 32 == 0);
  // operands without aligned rows (a workspace with no room for the copy) take the register-staged
  // 128 x 128 form whatever the variant
  if (vec)
    hipLaunchKernelGGL((gemm1_kernel<TERMS, BLO, G1M, G1N, WGM, WGN, MINB, true>), grid, dim3(64 * WGM * WGN), 0, s, g);
  else
    hipLaunchKernelGGL((gemm1_kernel<TERMS, BLO, 128, 128, 2, 2, 2, false>), xcd_grid(g1_items(g, 128, 128, false)),
                       dim3(256), 0, s, g);
}

// variant (resolved by the planner): 1 = 128 x 128 (4 waves of 64 x 64, two blocks per CU),
// 2 = 128 x 256 (4 waves of 64 x 128), 3 = 256 x 256 (8 waves of 128 x 64)
template <int TERMS, bool BLO>
static void launch_g1v(hipStream_t s, const G1Args& g, int variant) {
  switch (variant) {
    case 2: launch_g1<TERMS, BLO, 128, 256, 2, 2, 1>(s, g); break;
    case 3: launch_g1<TERMS, BLO, 256, 256, 2, 4, 1>(s, g); break;
    default: launch_g1<TERMS, BLO, 128, 128, 2, 2, 2>(s, g); break;
  }
}

hipError_t df_bf16_gemm1(hipStream_t s, int nbf, int nact, int np, int terms, SplitPtr Ct, int ldk, SplitPtr Bp,
                         long long bstride, int ldb, long long b_bytes, u16* XT_hi, u16* XT_lo, int ldx, int variant,
                         const WsDims& d, const uint32_t* bnd, int chunk) {
  if (np <= 0) return hipSuccess;
  const G1Args g{nbf, nact, np, Ct.hi, Ct.lo, ldk, Bp.hi, Bp.lo, bstride, ldb, b_bytes, XT_hi, XT_lo, ldx, d, bnd, chunk};
  if (terms == 1) launch_g1v<1, false>(s, g, variant);
  else if (Bp.lo == nullptr) launch_g1v<2, false>(s, g, variant);
  else launch_g1v<3, true>(s, g, variant);
  return hipGetLastError();
}

// b's 128 tile: 8 waves and one block per compute unit up to this many blocks (at most one for each unit, bound by the
// length of a block: a batch of one problem of 40 functions 180 us, 220 with 4 waves) and with one product per term
// (LDS bounds neither: 500 functions, 300 active 2.67 ms, 2.83 with 4 waves); otherwise 4 waves and two blocks (500
// functions in the split mode 3.71 ms, 3.75 with 8 waves; 12 problems of 520 functions 11.61 and 11.89 ms).
constexpr int G2_FEW = 256;
hipError_t df_bf16_gemm2(hipStream_t s, int nbf, int nact, int np, int nsplit, int terms, SplitPtr Ct, int ldk,
                         SplitPtr XT, int ldx, const float* beta32, double* Kpart, int kset, int krows, double* Dchunk,
                         u16* W_hi, u16* W_lo, int ldw, const WsDims& d, const uint32_t* bnd, int chunk) {
  if (np <= 0) return hipSuccess;
  const G2Args g{nbf,   nact,  np,     nsplit, Ct.hi, Ct.lo, ldk, XT.hi, XT.lo, ldx, beta32,
                 Kpart, Dchunk, W_hi, W_lo,   ldw,   d,     bnd, chunk, kset, krows};
  if (ldk % 32 || ldx % 32 || ldw % 32 || !al16(Ct.hi) || !al16(Ct.lo) || !al16(XT.hi) || !al16(XT.lo) || !al16(W_hi) ||
      !al16(W_lo))
    return hipErrorInvalidValue;
  const int items = g2_items(g, T2);
  const dim3 grid = xcd_grid(items);
  if (terms == 1) hipLaunchKernelGGL((gemm2_kernel<1, 4>), grid, dim3(512), 0, s, g);
  else if (items <= G2_FEW) hipLaunchKernelGGL((gemm2_kernel<3, 4>), grid, dim3(512), 0, s, g);
  else hipLaunchKernelGGL((gemm2_kernel<3, 2>), grid, dim3(256), 0, s, g);
  return hipGetLastError();
}

template <int TERMS, int G3M, int G3N, int WGM, int WGN, int MINB>
static void launch_g3(hipStream_t s, const G3Args& g) {
  hipLaunchKernelGGL((gemm3_kernel<TERMS, G3M, G3N, WGM, WGN, MINB>), xcd_grid(g3_items(g, G3M, G3N)), dim3(64 * WGM * WGN),
                     0, s, g);
}

hipError_t df_bf16_gemm3(hipStream_t s, int nbf, int nact, int np, int nsplit, int terms, SplitPtr XT, int ldx,
                         SplitPtr W, int ldw, float* Ypart, int variant, const WsDims& d, const uint32_t* bnd,
                         int chunk) {
  if (np <= 0) return hipSuccess;
  const G3Args g{nbf, nact, np, nsplit, XT.hi, XT.lo, ldx, W.hi, W.lo, ldw, Ypart, d, bnd, chunk};
  if (ldx % 32 || ldw % 32 || !al16(XT.hi) || !al16(XT.lo) || !al16(W.hi) || !al16(W.lo)) return hipErrorInvalidValue;
  // variant (resolved by the planner): 1 = 128 x 128 (4 waves of 64 x 64, two blocks per CU),
  // 2 = 256 x 128 (4 waves of 128 x 64), 3 = 256 x 256 (8 waves of 128 x 64)
  if (terms == 1) {
    switch (variant) {
      case 2: launch_g3<1, 256, 128, 2, 2, 1>(s, g); break;
      case 3: launch_g3<1, 256, 256, 2, 4, 1>(s, g); break;
      default: launch_g3<1, 128, 128, 2, 2, 2>(s, g); break;
    }
  } else {
    switch (variant) {
      case 2: launch_g3<3, 256, 128, 2, 2, 1>(s, g); break;
      case 3: launch_g3<3, 256, 256, 2, 4, 1>(s, g); break;
      default: launch_g3<3, 128, 128, 2, 2, 2>(s, g); break;
    }
  }
  return hipGetLastError();
}

hipError_t df_bf16_gemm1_grouped(hipStream_t s, int ninst, int total, int terms, int tile, const G1Args* tab,
                                 const int* off) {
  if (total <= 0) return hipSuccess;
  const dim3 gr = xcd_grid(total);
  if (tile == 64) {
    if (terms == 1) hipLaunchKernelGGL((gemm1_grouped<1, 64>), gr, dim3(256), 0, s, tab, off, ninst, total);
    else hipLaunchKernelGGL((gemm1_grouped<2, 64>), gr, dim3(256), 0, s, tab, off, ninst, total);
  } else {
    if (terms == 1) hipLaunchKernelGGL((gemm1_grouped<1, 128>), gr, dim3(256), 0, s, tab, off, ninst, total);
    else hipLaunchKernelGGL((gemm1_grouped<2, 128>), gr, dim3(256), 0, s, tab, off, ninst, total);
  }
  return hipGetLastError();
}
hipError_t df_bf16_gemm2_grouped(hipStream_t s, int ninst, int total, int terms, int tile, const G2Args* tab,
                                 const int* off) {
  if (total <= 0) return hipSuccess;
  const dim3 gr = xcd_grid(total);
  if (tile == 64) {
    if (terms == 1) hipLaunchKernelGGL((gemm2_grouped<1, 64, 2>), gr, dim3(256), 0, s, tab, off, ninst, total);
    else hipLaunchKernelGGL((gemm2_grouped<3, 64, 2>), gr, dim3(256), 0, s, tab, off, ninst, total);
  } else {
    if (terms == 1) hipLaunchKernelGGL((gemm2_grouped<1, 128, 4>), gr, dim3(512), 0, s, tab, off, ninst, total);
    else if (total <= G2_FEW) hipLaunchKernelGGL((gemm2_grouped<3, 128, 4>), gr, dim3(512), 0, s, tab, off, ninst, total);
    else hipLaunchKernelGGL((gemm2_grouped<3, 128, 2>), gr, dim3(256), 0, s, tab, off, ninst, total);
  }
  return hipGetLastError();
}
template <int TERMS, int TN>
static void launch_g3_grouped(hipStream_t s, int ninst, int total, int btile, const G3Args* tab, const int* off) {
  if (btile == 64) hipLaunchKernelGGL((gemm3_grouped<TERMS, TN, 64>), xcd_grid(total), dim3(256), 0, s, tab, off, ninst, total);
  else hipLaunchKernelGGL((gemm3_grouped<TERMS, TN, 128>), xcd_grid(total), dim3(256), 0, s, tab, off, ninst, total);
}
hipError_t df_bf16_gemm3_grouped(hipStream_t s, int ninst, int total, int terms, int tile, int btile, const G3Args* tab,
                                 const int* off) {
  if (total <= 0) return hipSuccess;
  if (tile == 64) {
    if (terms == 1) launch_g3_grouped<1, 64>(s, ninst, total, btile, tab, off);
    else launch_g3_grouped<3, 64>(s, ninst, total, btile, tab, off);
  } else {
    if (terms == 1) launch_g3_grouped<1, 128>(s, ninst, total, btile, tab, off);
    else launch_g3_grouped<3, 128>(s, ninst, total, btile, tab, off);
  }
  return hipGetLastError();
}

}  // namespace pnof

namespace pnof {

void persist_counts(const BInst& d, const G1Args& g1, const G2Args& g2, const G3Args& g3, int tx, int ty, int* cnt) {
  cnt[PH_BND] = bnd_items(d.nact);
  cnt[PH_PREP] = PERSIST_PARTS;
  cnt[PH_X] = cdiv(g1_items(g1, tx, 128, true), PERSIST_XG) + f64t::grouped_tiles(d.nbf, d.nact);
  cnt[PH_B] = g2_items(g2, 64) + 1;
  cnt[PH_DA] = f64t::grouped_tiles(d.naux, d.nact);
  cnt[PH_DIAG] = PERSIST_PARTS;
  cnt[PH_Y] = f64t::grouped_tiles(d.nact, d.nact) + g3_items(g3, 128, ty);
  cnt[PH_RED] = PERSIST_PARTS;
  cnt[PH_EY] = BATCH_EPARTS + PERSIST_PARTS;
  cnt[PH_LAM] = f64t::grouped_tiles(d.nbf, d.nact);
  cnt[PH_FIN] = PERSIST_PARTS;
  cnt[PH_VJP] = 1;
}

hipError_t batch_persist(hipStream_t s, const PArgs& a, int tx, int ty, int blocks) {
  hipLaunchKernelGGL(persist_reset_k, dim3(1), dim3(256), 0, s, a.sc, a.ninst);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (tx == 64 && ty == 64) hipLaunchKernelGGL((batch_persist_k<64, 64>), dim3(blocks), dim3(256), 0, s, a);
  else if (tx == 64) hipLaunchKernelGGL((batch_persist_k<64, 128>), dim3(blocks), dim3(256), 0, s, a);
  else if (ty == 64) hipLaunchKernelGGL((batch_persist_k<128, 64>), dim3(blocks), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((batch_persist_k<128, 128>), dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace pnof
