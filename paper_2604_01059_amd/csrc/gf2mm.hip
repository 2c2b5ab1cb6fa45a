// Dense products over GF(2) on the matrix cores, and the phase-pair product.
//
// 1. C[i][j] = (sum_k A[i][k] B[j][k]) mod 2 for bit-packed rows A_i, B_j.
//    This is the batched parity contraction a_k = XOR_i u_ki f_i of the
//    paper's parameterized evaluation (appendix "Parameterized evaluation of
//    Clifford ZX diagrams", equation parities), with A = U and B = the
//    parameter settings, and it is the symplectic commutation table of Pauli
//    strings with A_i = [x_i | z_i], B_j = [z_j | x_j] (appendix "Pauli
//    channels" for the encoding).  The paper contracts in floating point on
//    BLAS; here the bits enter v_mfma_scale_f32_32x32x64_f8f6f4 as FP4
//    (E2M1) values: a set bit is the code 0b0001 (0.5), the block scale 2^1
//    makes it 1.0, so every product is 0 or 1 and the fp32 sums (of at most
//    2^22 bits: longer rows go in parts, a launch each) are exact counts; bit
//    0 of the count is the parity.  Bits are unpacked by bit plane: plane t of
//    four consecutive dwords (bits 4r + t) is an operand as it stands,
//    d & (0x11111111 << t).
//
//    One persistent kernel, 256 x 256 or 128 x 128 output tiles; a wavefront
//    owns 64 x 128 (64 x 64) of a tile: 2 x 4 blocks of 32 x 32, 128 fp32
//    accumulators per lane, two wavefronts per SIMD.  Rows go through LDS in
//    chunks of 512 bits, double buffered, the next chunk's loads in flight
//    during a chunk's products and across tiles.  B's rows are the
//    instruction's first operand, so that a lane's accumulators are
//    neighbouring columns of one row of C: one funnel shift each packs the
//    parities, and the mirrored half of the symmetric table is a transpose of
//    32 x 32 bit blocks across lanes.  (With A's rows first, 16 ballots a
//    block and as many LDS writes gathered the row words: as many VALU cycles
//    as the products took.)
//
//    Bound: the matrix cores.  65536-string table, 1024 qubits: 2.49 -> 1.50
//    ms (5.9 PFLOP/s; the instruction with this unpacking and nothing else
//    reaches 7.7 PFLOP/s at the clock the card holds); 4096 x 65536 x 1024
//    bits: 196 -> 112 us (4.9 PFLOP/s).  The rest is the parity write-out
//    (about 10 %) and the row loads (about 10 %).
//
// 2. Per setting l: omega^phase8 sqrt(2)^pow * prod_k h(alpha_k, beta_k;
//    a_kl, b_kl), h of equation phase_pair, phases multiples of pi/4.  Terms
//    whose values are all 2 i^s are counted bit-sliced; with any other term,
//    one lane per setting, fp32 complex products, renormalised to a power of
//    two every 8 factors.
#include <algorithm>

#include "zx_internal.h"

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int MM_W = 8;  // words of a row staged at a time (two 256-bit groups)
constexpr int MM_PART = 1 << 16;  // words of a row per launch: 2^22 bits

struct MmArgs {
  // Words of a row are staged in two groups of four: group g of chunk c holds
  // words cs c .. cs c + 3 from a[g] / b[g], of which those below kg[g] exist
  // (one part: a[1] = a[0] + 4, cs = 8; the two parts of a Pauli row: one
  // group each, cs = 4).
  const uint64_t* a[2];
  const uint64_t* b[2];
  int64_t lda, ldb;       // words per row
  int64_t m, n;           // rows of A, rows of B
  int32_t kg[2], cs, nch;  // words per group, words per chunk step, chunks
  uint64_t last;          // valid bits of the row's (or part's) last word
  int32_t last_w[2];      // that word in each group's count (-1: not in the group)
  uint64_t* C;
  int64_t ldc;
  int64_t cw;             // words of C written per row: ceil(n / 64)
  int32_t tm, tn;         // tiles along m and n
  int32_t sym;            // symmetric table: tiles on and above the diagonal, mirror written too
  int32_t bh;             // rows of tiles per band of the tile order
  int64_t n_tiles;
  int64_t per_xcd;        // tiles per XCD run
};

// Accumulators start at 2^23: a count below 2^23 added to it stays an exact
// fp32 integer in [2^23, 2^24), where one unit is the last mantissa bit, so
// bit 0 of the float's bits is the count's parity.
constexpr float ACC_BASE = 8388608.0f;

// Bit plane T (bits 4 r + T) of four dwords as an FP4 operand: planes 0, 1, 2
// are 0.5, 1, 2 as they stand (one AND a dword); plane 3 would be the sign
// bit and is shifted onto plane 2.  plane_scale: the E8M0 block scale that
// makes the set value 1.  Which bit meets which k does not matter as long as
// both operands agree.
template <int T>
__device__ __forceinline__ v8i plane_fp4(const uint4& d) {
  const uint32_t w[4] = {d.x, d.y, d.z, d.w};
  v8i o;
#pragma unroll
  for (int q = 0; q < 4; ++q) o[q] = (int)(T < 3 ? w[q] & (0x11111111u << (T & 3)) : (w[q] >> 1) & 0x44444444u);
  o[4] = o[5] = o[6] = o[7] = 0;
  return o;
}
constexpr int plane_scale(int t) { return t == 0 ? 128 : (t == 1 ? 127 : 126); }

// Parities of the 16 accumulators of a 32 x 32 block: this lane half's bits
// (register 4 q + s at bit 8 q + s + 4).  One funnel shift per accumulator
// brings its bit 0 in at the top.
__device__ __forceinline__ uint32_t parity_bits(const v16f& acc) {
  uint32_t d = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (r > 0 && (r & 3) == 0) d >>= 4;
    d = __builtin_amdgcn_alignbit(__float_as_uint(acc[r]), d, 1);
  }
  return d;
}

// a.lanes 32..63 <-> b.lanes 0..31
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}

// Transposes of two 32 x 32 bit matrices per lane half at once (lane = row,
// bit = column): five butterfly steps; the 16-lane step swaps register halves
// between the two, the others fetch the partner lane's word by DPP and merge
// under the lane's mask.
__device__ __forceinline__ void transpose32x2(uint32_t& a, uint32_t& b) {
  const int lane = threadIdx.x & 63;
  {  // 16: (a.lo, b.lo) and (a.hi, b.hi), odd rows of one against even rows of the other
    const uint32_t p = __builtin_amdgcn_perm(b, a, 0x05040100u), q = __builtin_amdgcn_perm(b, a, 0x07060302u);
    const auto r = __builtin_amdgcn_permlane16_swap(p, q, false, false);
    a = __builtin_amdgcn_perm(r[1], r[0], 0x05040100u);
    b = __builtin_amdgcn_perm(r[1], r[0], 0x07060302u);
  }
  const uint32_t sel8 = (lane & 8) ? 0x03070105u : 0x06020400u;
  const uint32_t m4 = (lane & 4) ? 0xF0F0F0F0u : 0x0F0F0F0Fu, r4 = (lane & 4) ? 4u : 28u;
  const uint32_t m2 = (lane & 2) ? 0xCCCCCCCCu : 0x33333333u, r2 = (lane & 2) ? 2u : 30u;
  const uint32_t m1 = (lane & 1) ? 0xAAAAAAAAu : 0x55555555u, r1 = (lane & 1) ? 1u : 31u;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    uint32_t x = k ? b : a, y;
    y = dpp<0x128>(x);                               // lane ^ 8
    x = __builtin_amdgcn_perm(y, x, sel8);
    y = dpp<0x1B>(dpp<0x141>(x));                    // lane ^ 4: within 8 reversed, then within 4
    x = (x & m4) | (__builtin_amdgcn_alignbit(y, y, r4) & ~m4);
    y = dpp<0x4E>(x);                                // lane ^ 2
    x = (x & m2) | (__builtin_amdgcn_alignbit(y, y, r2) & ~m2);
    y = dpp<0xB1>(x);                                // lane ^ 1
    x = (x & m1) | (__builtin_amdgcn_alignbit(y, y, r1) & ~m1);
    (k ? b : a) = x;
  }
}

// Tile order.  Bands of a.bh rows of tiles, each walked column by column, so
// that the tiles in flight on an XCD (32 workgroups: 4 rows by 8 columns) read
// few different rows of A and B (65536-string table under the profiler: 1.72
// -> 1.67 ms).  Band b
// of the symmetric table starts at its first row's diagonal; the few tiles of
// a band below the diagonal are computed like any other (without a mirror),
// which costs 1 % of the work at 256 rows of tiles.  (Both write the same
// words, so parts of long rows, which add to C, walk bands of one row.)
struct TileOrder {
  int64_t b, r;  // band, place within it

  static __device__ __forceinline__ int64_t first_col(const MmArgs& a, int64_t b) { return a.sym ? b * a.bh : 0; }
  static __device__ __forceinline__ int64_t height(const MmArgs& a, int64_t b) {
    const int64_t left = a.tm - b * a.bh;
    return left < a.bh ? left : a.bh;
  }
  // tiles of the bands before b (all of them full)
  static __device__ __forceinline__ int64_t start(const MmArgs& a, int64_t b) {
    return a.bh * (b * a.tn - (a.sym ? a.bh * (b * (b - 1) / 2) : 0));
  }
  __device__ __forceinline__ void seek(const MmArgs& a, int64_t t) {
    int64_t lo = 0, hi = (a.tm + a.bh - 1) / a.bh - 1;
    while (lo < hi) {
      const int64_t mid = (lo + hi + 1) >> 1;
      if (start(a, mid) <= t) lo = mid;
      else hi = mid - 1;
    }
    b = lo;
    r = t - start(a, lo);
  }
  // G tiles further.  Past the last tile the band reaches the row count; such
  // a tile is never multiplied (its loads read the first row).
  __device__ __forceinline__ void step(const MmArgs& a, int G) {
    r += G;
    while (b * a.bh < a.tm) {
      const int64_t len = height(a, b) * (a.tn - first_col(a, b));
      if (r < len) break;
      r -= len;
      ++b;
    }
  }
  __device__ __forceinline__ void tile(const MmArgs& a, int& ti, int& tj) const {
    const int h = (int)height(a, b), q = (int)r;
    if (h <= 0) {
      ti = a.tm;
      tj = 0;
      return;
    }
    const int col = h == 4 ? q >> 2 : q / h;
    ti = (int)(b * a.bh) + q - col * h;
    tj = (int)first_col(a, b) + col;
  }
};

// ADD: a later part of long rows, whose parities C takes by XOR.
template <bool ADD>
__device__ __forceinline__ void put_word(const MmArgs& a, int64_t row, int64_t word, uint64_t v) {
  uint64_t* const p = a.C + row * a.ldc + word;
  *p = ADD ? *p ^ v : v;
}

// Parities out of a wave's 64 x 32 BJ part at row r0, column c0.  The
// instruction's first operand holds B's rows, so a lane holds one row of C
// and its registers are columns: the row words are packed within the lane.
template <int BJ, bool ADD>
__device__ __forceinline__ void write_part(const MmArgs& a, const v16f (&acc)[2][BJ], int64_t r0, int64_t c0,
                                           bool mirror) {
  const int lane = threadIdx.x & 63, h = lane >> 5, l32 = lane & 31;
  uint32_t d[BJ];  // row r0 + lane, columns c0 + 32 j ..
#pragma unroll
  for (int j = 0; j < BJ; ++j) {
    uint32_t x = parity_bits(acc[0][j]), y = parity_bits(acc[1][j]);
    swap32(x, y);  // x: lane half 0 of rows 0..31, then of rows 32..63; y: lane half 1
    d[j] = (x >> 4) | y;
  }
  const int64_t gi = r0 + lane;
  if (gi < a.m) {
#pragma unroll
    for (int j = 0; j < BJ; j += 2) {
      const int64_t wcol = c0 / 64 + j / 2;
      if (wcol < a.cw) {
        // columns at or beyond n hold the parities of rows that do not exist
        const int64_t left = a.n - wcol * 64;
        const uint64_t v = (uint64_t)d[j] | ((uint64_t)d[j + 1] << 32);
        put_word<ADD>(a, gi, wcol, left >= 64 ? v : v & ((1ull << left) - 1));
      }
    }
  }
  if (!mirror) return;
  // row c0 + 32 (j + h) + l32, the word of rows r0 .. r0 + 63
  const int64_t wcol = r0 / 64;
  const int64_t left = a.m - r0;  // may be <= 0: rows beyond the table
  const uint64_t keep = left >= 64 ? ~0ull : (left <= 0 ? 0ull : (1ull << left) - 1);
#pragma unroll
  for (int j = 0; j < BJ; j += 2) {
    uint32_t x = d[j], y = d[j + 1];
    transpose32x2(x, y);
    swap32(x, y);
    const int64_t gj = c0 + 32 * (j + h) + l32;
    if (gj < a.n && wcol < a.cw) put_word<ADD>(a, gj, wcol, ((uint64_t)x | ((uint64_t)y << 32)) & keep);
  }
}

// Persistent: workgroup k of XCD x (blockIdx = 8 k + x) takes tiles
// x * per_xcd + k + j G (j = 0, 1, ...; G workgroups per XCD) of its XCD's
// run, so the tiles in flight on one XCD are a contiguous window of the
// tile order and share rows in its L2.  The chunks of all its tiles form one
// sequence: the next chunk waits in registers while a chunk is multiplied,
// goes to the other LDS buffer, and the loads of the one after start, so the
// next tile's first chunk is in flight during a tile's parity write-out.
//
// WR x WC wavefronts, each a 64 x 32 BJ part.  Eight lanes load one row's
// chunk (64 bytes), so a load instruction touches 8 rows; the chunk sits in
// LDS as two groups of 256 bits a row, and a fragment (32 rows, this lane
// half's 128 bits of the group) is one conflict-free 16-byte read for four
// products.
template <int WR, int WC, int BJ, bool ADD>
__global__ __launch_bounds__(64 * WR * WC, 2) void gf2mm_kernel(MmArgs a) {
  constexpr int BS = 64 * WR * WC;
  constexpr int TI = 64 * WR, TJ = 32 * BJ * WC;  // tile rows, columns
  constexpr int RS = BS / MM_W;                   // rows per load instruction of the workgroup
  constexpr int NL = (TI + TJ) / RS;              // loads per thread and chunk
  static_assert(TI % RS == 0 && TJ % RS == 0, "a load is all A or all B");
  __shared__ __attribute__((aligned(16))) uint64_t sbuf[2][2][TI + TJ][4];  // [buffer][group][row][word]
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int G = (int)(gridDim.x >> 3);
  const int64_t t_first = (int64_t)(blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
  int64_t t_last = (int64_t)((blockIdx.x & 7) + 1) * a.per_xcd;
  if (t_last > a.n_tiles) t_last = a.n_tiles;
  if (t_first >= t_last) return;
  const int nch = a.nch;
  const int n_my = (int)((t_last - t_first + G - 1) / G);

  // The loads of a chunk are straight-line code (no branch may separate them
  // from the stash that uses them, or the compiler waits for each at once):
  // its tile is one of the next three, whose first rows are kept in
  // rm[0..2] / rn[0..2].
  int64_t rm[3], rn[3];
  TileOrder order;
  order.seek(a, t_first);
  auto next_tile = [&](int64_t& r0, int64_t& c0) {
    int ti, tj;
    order.tile(a, ti, tj);
    r0 = (int64_t)ti * TI;
    c0 = (int64_t)tj * TJ;
    order.step(a, G);
  };
#pragma unroll
  for (int q = 0; q < 3; ++q) next_tile(rm[q], rn[q]);
  const int lw = tid & (MM_W - 1), lr = tid / MM_W;  // this thread's word of a chunk, and its first row
  const int lg = lw >> 2, l4 = lw & 3;               // its group, and word of the group
  const uint64_t* const pa = (lg ? a.a[1] : a.a[0]) + (int64_t)lr * a.lda;
  const uint64_t* const pb = (lg ? a.b[1] : a.b[0]) + (int64_t)lr * a.ldb;
  const int kg = lg ? a.kg[1] : a.kg[0], last_w = lg ? a.last_w[1] : a.last_w[0];
  uint64_t rr[NL], mask = 0;
  // Words of chunk c of the rows of the tile at (r0, c0).  Only A's words are
  // masked (bits at or beyond the row length, words past the last; by the
  // stash, so that nothing here waits for a load): a zero on one side makes
  // the product zero.  Rows and words that do not exist read
  // the first row or word; the parities of such rows are not written.
  auto fetch = [&](int64_t r0, int64_t c0, int c) {
    const int w = c * a.cs + l4;
    const bool in_k = w < kg;
    mask = !in_k ? 0 : (w == last_w ? a.last : ~0ull);
    const int ww = in_k ? w : 0;
    const uint64_t* qa = pa + ww;
    const uint64_t* qb = pb + ww;
    if (r0 + TI <= a.m && c0 + TJ <= a.n) {  // the same for the workgroup
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        const bool isb = k * RS >= TI;
        const int64_t off = isb ? (c0 + k * RS - TI) * a.ldb : (r0 + k * RS) * a.lda;
        rr[k] = (isb ? qb : qa)[off];
      }
    } else {
#pragma unroll
      for (int k = 0; k < NL; ++k) {
        const bool isb = k * RS >= TI;
        const int64_t row = isb ? c0 + k * RS - TI : r0 + k * RS;
        const bool ok = row + lr < (isb ? a.n : a.m);
        const int64_t off = row * (isb ? a.ldb : a.lda), first = -(int64_t)lr * (isb ? a.ldb : a.lda);
        rr[k] = (isb ? qb : qa)[ok ? off : first];
      }
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int k = 0; k < NL; ++k) sbuf[buf][lg][k * RS + lr][l4] = k * RS >= TI ? rr[k] : rr[k] & mask;
  };

  const int wr = (wv / WC) * 64, wc = (wv % WC) * 32 * BJ;  // this wave's part
  const int h = lane >> 5, l32 = lane & 31;
  v16f base;
#pragma unroll
  for (int r = 0; r < 16; ++r) base[r] = ACC_BASE;
  fetch(rm[0], rn[0], 0);
  stash(0);
  {
    const int q = nch > 1 ? 0 : 1;
    fetch(q ? rm[1] : rm[0], q ? rn[1] : rn[0], nch > 1 ? 1 : 0);
  }
  __syncthreads();
  int buf = 0;
  for (int j = 0; j < n_my; ++j) {
    v16f acc[2][BJ];
    for (int c = 0; c < nch; ++c) {
      // the next chunk into the other buffer (past the end: a buffer no one
      // reads), then the loads of the one after, in flight during this chunk's
      // products
      stash(buf ^ 1);
      const int c2 = c + 2;
      const int jo = c2 < nch ? 0 : (c2 < 2 * nch ? 1 : 2);
      fetch(jo == 0 ? rm[0] : (jo == 1 ? rm[1] : rm[2]), jo == 0 ? rn[0] : (jo == 1 ? rn[1] : rn[2]), c2 - jo * nch);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        uint4 fa[2], fb[BJ];
#pragma unroll
        for (int i = 0; i < 2; ++i) fa[i] = *(const uint4*)&sbuf[buf][g][wr + 32 * i + l32][2 * h];
#pragma unroll
        for (int i = 0; i < BJ; ++i) fb[i] = *(const uint4*)&sbuf[buf][g][TI + wc + 32 * i + l32][2 * h];
#define GF2MM_PLANE(T, C_IN)                                                                                    \
  do {                                                                                                          \
    v8i oa[2], ob[BJ];                                                                                          \
    _Pragma("unroll") for (int i = 0; i < 2; ++i) oa[i] = plane_fp4<T>(fa[i]);                                   \
    _Pragma("unroll") for (int i = 0; i < BJ; ++i) ob[i] = plane_fp4<T>(fb[i]);                                  \
    _Pragma("unroll") for (int i = 0; i < 2; ++i) _Pragma("unroll") for (int jj = 0; jj < BJ; ++jj) acc[i][jj] = \
        __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ob[jj], oa[i], C_IN, 4, 4, 0, plane_scale(T), 0,         \
                                                        plane_scale(T));                                        \
  } while (0)
        if (g == 0 && c == 0)
          GF2MM_PLANE(0, base);
        else
          GF2MM_PLANE(0, acc[i][jj]);
        GF2MM_PLANE(1, acc[i][jj]);
        GF2MM_PLANE(2, acc[i][jj]);
        GF2MM_PLANE(3, acc[i][jj]);
#undef GF2MM_PLANE
      }
      __syncthreads();
      buf ^= 1;
    }
    write_part<BJ, ADD>(a, acc, rm[0] + wr, rn[0] + wc, a.sym && rm[0] < rn[0]);
    rm[0] = rm[1];
    rn[0] = rn[1];
    rm[1] = rm[2];
    rn[1] = rn[2];
    next_tile(rm[2], rn[2]);
  }
}

// ------------------------------------------------------ phase-pair product --

constexpr int PP_BS = 256;      // settings per workgroup (four words of a row)
// Terms up to which a workgroup has 256 threads instead of 1024: one a setting,
// and no more slices than terms.  10^6 settings of 4 terms 9 against 22 us, of
// 64 terms 9 against 22; from 65536 settings down the two are the same.
constexpr int PP_FEW = 64;
constexpr int PP_CHUNK = 256;   // terms whose h tables sit in LDS at a time
constexpr float RH = 0.70710678118654752440f;

// cos(k pi/4): exact 0 and +-1 where they occur
__device__ __forceinline__ float cos_q(int k) {
  k &= 7;
  const float mag = (k & 1) ? RH : ((k & 2) ? 0.0f : 1.0f);
  return (k >= 3 && k <= 5) ? -mag : mag;
}

// e^{i k pi/4} = (cos(k pi/4), sin(k pi/4)), sin(x) = cos(x - pi/2)
__device__ __forceinline__ float2 omega_pow(int k) { return make_float2(cos_q(k), cos_q(k + 6)); }

__device__ __forceinline__ float2 cmul(float2 x, float2 y) {
  return make_float2(x.x * y.x - x.y * y.y, x.x * y.y + x.y * y.x);
}

// scale z by a power of two so that max(|re|, |im|) is in [0.5, 1)
__device__ __forceinline__ void renorm(float2& z, int& e) {
  const float mx = fmaxf(fabsf(z.x), fabsf(z.y));
  if (mx == 0.0f) return;
  const int ex = __builtin_amdgcn_frexp_expf(mx);
  z.x = ldexpf(z.x, -ex);
  z.y = ldexpf(z.y, -ex);
  e += ex;
}

// A term is a unit term when each of its four values h(k; a, b) is 2 i^s: both
// codes even and one of them 0 or 4 (the two kinds that the rewrite rules
// leave, (0 or 4, 2) and (0 or 4, 0 or 4), are).  With that code first, h = 2
// if its phase comes out 0 and 2 e^{i beta'} if it comes out pi.
__device__ __forceinline__ bool unit_term(int ka, int kb) { return ((ka | kb) & 1) == 0 && ((ka & 3) == 0 || (kb & 3) == 0); }

// One block: 256 settings (four words of every row of A and B).
//
// Unit terms only: the product is 2^m i^(sum of s), so the settings need one
// two-bit counter each, kept bit-sliced over a word's 64 settings.  Thread
// (slice, word) adds the terms slice, slice + T / 4, ...; the T / 4 partial
// counters are added by lane swaps and once through LDS.  Products by 2 i^s
// are exact in fp32, so mantissa and exponent are those of the factor-by-
// factor product.  Bound: reading A and B once; 16 wavefronts a CU keep the
// loads in flight (46 us with four).
//
// Any other term: the factor-by-factor product, one lane per setting, the
// term's words and h values from LDS (256 terms at a time), eight terms'
// reads in flight.  Bound: ten VALU operations per term and setting.
//
// 4096 terms x 65536 settings: 1190 us with one dependent scalar load chain
// per term -> 20 us (unit terms), 160 us (any codes).
template <int T>
__global__ __launch_bounds__(T) void phase_pair_kernel(const uint64_t* __restrict__ A,
                                                           const uint64_t* __restrict__ B, int64_t ld,
                                                           int32_t m, int64_t n_set,
                                                           const int8_t* __restrict__ ka,
                                                           const int8_t* __restrict__ kb, int32_t phase8,
                                                           int64_t pow_sqrt2, float2* __restrict__ mant,
                                                           int32_t* __restrict__ expo) {
  __shared__ float2 tab[PP_CHUNK][4];       // h(k; a, b) at index a + 2 b
  __shared__ uint2 bits[PP_CHUNK][PP_BS / 32];  // 32 settings' bits of A's row and of B's
  __shared__ uint64_t part[T / 64][4][2];    // the waves' counters
  __shared__ int odd_wave[T / 64];           // a wave saw a term that is no unit term
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // neighbouring blocks share cache lines of the rows: runs of them on one XCD
  const int64_t nb = (n_set + PP_BS - 1) / PP_BS, per = (nb + 7) / 8;
  const int64_t blk = (int64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int64_t)(blockIdx.x >> 3) >= per || blk >= nb) return;
  const int64_t l = blk * PP_BS + tid;
  const int64_t nw = (n_set + 63) / 64, w0 = blk * (PP_BS / 64);
  // c = omega^phase8 sqrt(2)^pow
  const bool odd = (pow_sqrt2 & 1) != 0;
  int e = (int)((pow_sqrt2 - (odd ? 1 : 0)) / 2);
  float2 z = omega_pow(phase8);
  if (odd) {
    z.x *= 1.41421356237309504880f;
    z.y *= 1.41421356237309504880f;
  }
  renorm(z, e);

  // bit-sliced sum of s over this thread's terms
  uint64_t c0 = 0, c1 = 0;
  bool other = false;
  {
    const int64_t w = w0 + (tid & 3) < nw ? w0 + (tid & 3) : nw - 1;
    const int slice = tid >> 2;
    const uint64_t* pa = A + w;
    const uint64_t* pb = B + w;
#pragma unroll 4
    for (int k = slice; k < m; k += T / 4) {
      const int ak = ka[k] & 7, bk = kb[k] & 7;
      const uint64_t aw = pa[(int64_t)k * ld], bw = pb[(int64_t)k * ld];
      other |= !unit_term(ak, bk);
      const bool swap = (ak & 3) != 0;  // B's code is the one in {0, 4}
      const int f = swap ? bk : ak, g = swap ? ak : bk;
      const uint64_t on = (swap ? bw : aw) ^ (uint64_t)(int64_t)(-(f >> 2));  // settings whose s is not 0
      const uint64_t hi = (swap ? aw : bw) ^ (uint64_t)(int64_t)(-(g >> 2));
      const uint64_t lo = on & (uint64_t)(int64_t)(-((g >> 1) & 1));
      c1 ^= (on & hi) ^ (c0 & lo);
      c0 ^= lo;
    }
  }
#pragma unroll
  for (int d = 4; d < 64; d <<= 1) {  // the 16 slices of the wave
    const uint64_t o0 = (uint64_t)__shfl_xor((long long)c0, d), o1 = (uint64_t)__shfl_xor((long long)c1, d);
    c1 ^= o1 ^ (c0 & o0);
    c0 ^= o0;
  }
  const uint64_t any_other = __ballot(other);
  if (lane < 4) {
    part[wv][lane][0] = c0;
    part[wv][lane][1] = c1;
  }
  if (lane == 0) odd_wave[wv] = any_other != 0;
  __syncthreads();
  int general = 0;
#pragma unroll
  for (int v = 0; v < T / 64; ++v) general |= odd_wave[v];

  if (!general) {
    // this thread's setting: bit lane of word wv
    if (tid >= PP_BS) return;
    uint32_t s = 0;
#pragma unroll
    for (int v = 0; v < T / 64; ++v)
      s += (uint32_t)((part[v][wv][0] >> lane) & 1) + 2u * (uint32_t)((part[v][wv][1] >> lane) & 1);
    if (s & 1) z = make_float2(-z.y, z.x);
    if (s & 2) z = make_float2(-z.x, -z.y);
    z = make_float2(z.x + 0.0f, z.y + 0.0f);  // a negative zero would turn the angle of -1 round
    e += m;
  } else {
    for (int k0 = 0; k0 < m; k0 += PP_CHUNK) {
      const int nk = m - k0 < PP_CHUNK ? m - k0 : PP_CHUNK;
      __syncthreads();
      for (int x = tid; x < nk * 4; x += T) {
        const int k = x >> 2, ab = x & 3, av = ab & 1, bv = ab >> 1;
        const int ak = ka[k0 + k], bk = kb[k0 + k];
        const float2 p = omega_pow(ak + 4 * av), q = omega_pow(bk + 4 * bv), r = omega_pow(ak + bk + 4 * av + 4 * bv);
        tab[k][ab] = make_float2(1.0f + p.x + q.x - r.x, p.y + q.y - r.y);
        const int64_t w = w0 + ab < nw ? w0 + ab : nw - 1;
        const uint64_t aw = A[(int64_t)(k0 + k) * ld + w], bw = B[(int64_t)(k0 + k) * ld + w];
        bits[k][2 * ab] = make_uint2((uint32_t)aw, (uint32_t)bw);
        bits[k][2 * ab + 1] = make_uint2((uint32_t)(aw >> 32), (uint32_t)(bw >> 32));
      }
      __syncthreads();
      if (tid >= PP_BS) continue;  // staging only
      const int col = tid >> 5, sh = tid & 31;
      int k = 0;
      for (; k + 8 <= nk; k += 8) {
        float2 hv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const uint2 ab = bits[k + u][col];
          hv[u] = tab[k + u][((ab.x >> sh) & 1) + 2 * ((ab.y >> sh) & 1)];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) z = cmul(z, hv[u]);
        renorm(z, e);
      }
      for (; k < nk; ++k) {
        const uint2 ab = bits[k][col];
        z = cmul(z, tab[k][((ab.x >> sh) & 1) + 2 * ((ab.y >> sh) & 1)]);
      }
      renorm(z, e);
    }
  }
  if (tid < PP_BS && l < n_set) {
    if (z.x == 0.0f && z.y == 0.0f) e = 0;
    mant[l] = z;
    expo[l] = e;
  }
}

// coeff[i] bit j = D[i][piv[j]] for j < rank (zero beyond), words < cwords
__global__ void basis_coeff_kernel(const uint64_t* __restrict__ D, int32_t m, int64_t ld,
                                   const int32_t* __restrict__ rank_dev, const int32_t* __restrict__ piv,
                                   uint64_t* __restrict__ coeff, int64_t ldc, int32_t cwords) {
  const int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (it >= (int64_t)m * cwords) return;
  const int i = (int)(it / cwords), jw = (int)(it - (int64_t)i * cwords);
  const int rank = *rank_dev;
  uint64_t w = 0;
  for (int b = 0; b < 64; ++b) {
    const int j = 64 * jw + b;
    if (j >= rank) break;
    const int c = piv[j];
    w |= ((D[(int64_t)i * ld + (c >> 6)] >> (c & 63)) & 1ull) << b;
  }
  coeff[(int64_t)i * ldc + jw] = w;
}

template <int WR, int WC, int BJ>
zx_status launch_tiles(MmArgs a, bool add, int per_cu, hipStream_t s) {
  constexpr int TI = 64 * WR, TJ = 32 * BJ * WC;
  a.tm = (int32_t)((a.m + TI - 1) / TI);
  a.tn = (int32_t)((a.n + TJ - 1) / TJ);
  static_assert(TI == TJ, "the symmetric table pairs tile (i, j) with (j, i)");
  const ZxDevice* d = zx_device();
  if (!d) return ZX_EDEVICE;
  // persistent workgroups, the same count on every XCD
  const int64_t per = (d->n_cu / 8 > 0 ? d->n_cu / 8 : 1) * per_cu;
  // Symmetric: with few rows of tiles, those under the diagonal cost more than
  // the reuse gives; added to C, they would count twice.  Else bands high
  // enough for an XCD's tiles in flight, or a workgroup's way to its next tile
  // leads through many (100000 x 1 x 64 bits: 20.6 us with four rows, 9.6 so).
  a.bh = a.sym ? (a.tm < 64 || add ? 1 : 4) : (int32_t)std::max<int64_t>(4, (per + a.tn - 1) / a.tn);
  a.n_tiles = 0;
  for (int64_t b = 0; b * a.bh < a.tm; ++b) {
    const int64_t h = a.tm - b * a.bh < a.bh ? a.tm - b * a.bh : a.bh;
    a.n_tiles += h * (a.tn - (a.sym ? b * a.bh : 0));
  }
  a.per_xcd = (a.n_tiles + 7) / 8;
  if (a.per_xcd > 0x7fffffff / 8) {
    zx_set_error("product of %lld x %lld rows has too many tiles", (long long)a.m, (long long)a.n);
    return ZX_ECAPACITY;
  }
  const int64_t g = per < a.per_xcd ? per : a.per_xcd;
  // (a kernel of its own for parts that add: asking in the write-out costs 1 %)
  if (add)
    hipLaunchKernelGGL((gf2mm_kernel<WR, WC, BJ, true>), dim3((unsigned)(8 * g)), dim3(64 * WR * WC), 0, s, a);
  else
    hipLaunchKernelGGL((gf2mm_kernel<WR, WC, BJ, false>), dim3((unsigned)(8 * g)), dim3(64 * WR * WC), 0, s, a);
  ZX_HIP(hipGetLastError());
  return ZX_OK;
}

// 256 x 256 tiles (one workgroup of eight waves a CU) or 128 x 128 (two of
// four waves).  The large ones read half the rows per product and are 1.2
// times as fast where both fill the chip (4096 x 65536 x 1024 bits: 112
// against 136 us; 65536-string table under the profiler: 1.67 against 2.1 ms);
// the small ones where the large ones leave CUs without a tile (300 x 5000 x 200 bits: 5.5
// against 6.7 us) or end on a nearly empty round (8000 strings of 300 qubits,
// 528 large tiles: 23 against 28 us).
zx_status launch_gf2mm(const MmArgs& a, bool add, hipStream_t s) {
  const ZxDevice* d = zx_device();
  if (!d) return ZX_EDEVICE;
  auto tiles = [&](int64_t e) {
    const int64_t u = (a.n + e - 1) / e;
    return a.sym ? u * (u + 1) / 2 : (a.m + e - 1) / e * u;
  };
  const int64_t cu = d->n_cu, big = tiles(256);
  const double t_big = 4.0 * (double)((big + cu - 1) / cu);                              // in 128 x 128 tiles
  const double t_small = 1.2 * 2.0 * (double)((tiles(128) + 2 * cu - 1) / (2 * cu));
  return big < cu || t_small < t_big ? launch_tiles<2, 2, 2>(a, add, 2, s) : launch_tiles<4, 2, 4>(a, add, 1, s);
}

}  // namespace

// Symmetric commutation table on the matrix cores (called by zx_pauli_commute).
zx_status zx_pauli_commute_mfma(const uint64_t* X, const uint64_t* Z, int64_t n, int32_t n_qubits, int64_t ldq,
                                uint64_t* C, int64_t ldc, hipStream_t s) {
  MmArgs a{};
  const int qw = (int)(((int64_t)n_qubits + 63) / 64);
  a.lda = a.ldb = ldq;
  a.m = a.n = n;
  a.cs = 4;
  a.C = C;
  a.ldc = ldc;
  a.cw = (n + 63) / 64;
  a.sym = 1;
  for (int w0 = 0; w0 < qw; w0 += MM_PART / 2) {
    const int w = qw - w0 < MM_PART / 2 ? qw - w0 : MM_PART / 2;
    a.a[0] = a.b[1] = X + w0;
    a.a[1] = a.b[0] = Z + w0;
    a.kg[0] = a.kg[1] = w;
    a.nch = (w + 3) / 4;
    a.last = w0 + w == qw && (n_qubits % 64) ? ((1ull << (n_qubits % 64)) - 1) : ~0ull;
    a.last_w[0] = a.last_w[1] = w - 1;
    const zx_status rc = launch_gf2mm(a, w0 > 0, s);
    if (rc != ZX_OK) return rc;
  }
  return ZX_OK;
}

extern "C" zx_status zx_gf2_matmul(const uint64_t* A, int64_t m, int64_t lda, const uint64_t* B, int64_t n,
                                   int64_t ldb, int32_t k_bits, uint64_t* C, int64_t ldc, uint32_t flags,
                                   hipStream_t s) {
  zx_clear_error();
  ZX_CHECK_ARG(A && B && C, "null argument");
  ZX_CHECK_ARG(m > 0 && n > 0 && k_bits > 0, "empty product: m=%lld n=%lld k_bits=%d", (long long)m,
               (long long)n, k_bits);
  const int kw = (int)(((int64_t)k_bits + 63) / 64);
  ZX_CHECK_ARG(lda >= kw && ldb >= kw, "lda/ldb below %d words", kw);
  ZX_CHECK_ARG(ldc >= (n + 63) / 64, "ldc below %lld words", (long long)((n + 63) / 64));
  MmArgs a{};
  a.lda = lda;
  a.ldb = ldb;
  a.m = m;
  a.n = n;
  a.cs = MM_W;
  a.C = C;
  a.ldc = ldc;
  a.cw = (n + 63) / 64;
  a.sym = 0;
  for (int w0 = 0; w0 < kw; w0 += MM_PART) {
    const int w = kw - w0 < MM_PART ? kw - w0 : MM_PART;
    a.a[0] = A + w0;
    a.a[1] = A + w0 + (w > 4 ? 4 : 0);
    a.b[0] = B + w0;
    a.b[1] = B + w0 + (w > 4 ? 4 : 0);
    a.kg[0] = w;
    a.kg[1] = w - 4;
    a.nch = (w + MM_W - 1) / MM_W;
    a.last = w0 + w == kw && (k_bits % 64) ? ((1ull << (k_bits % 64)) - 1) : ~0ull;
    a.last_w[0] = w - 1;
    a.last_w[1] = w - 5;
    const zx_status rc = launch_gf2mm(a, w0 > 0, s);
    if (rc != ZX_OK) return rc;
  }
  if (flags & ZX_SYNC) ZX_HIP(hipStreamSynchronize(s));
  return ZX_OK;
}

extern "C" zx_status zx_phase_pair_product(const uint64_t* A, const uint64_t* B, int64_t ld, int32_t n_terms,
                                           int64_t n_settings, const int8_t* k_alpha, const int8_t* k_beta,
                                           int32_t phase8, int64_t pow_sqrt2, float* mant, int32_t* expo,
                                           hipStream_t s) {
  zx_clear_error();
  ZX_CHECK_ARG(mant && expo, "null output");
  ZX_CHECK_ARG(n_terms >= 0 && n_settings > 0, "bad sizes: n_terms=%d n_settings=%lld", n_terms,
               (long long)n_settings);
  ZX_CHECK_ARG(n_terms == 0 || (A && B && k_alpha && k_beta), "null term input");
  ZX_CHECK_ARG(n_terms == 0 || ld >= (n_settings + 63) / 64, "ld below %lld words",
               (long long)((n_settings + 63) / 64));
  const int64_t blocks = ((n_settings + PP_BS - 1) / PP_BS + 7) / 8 * 8;  // whole runs per XCD
  ZX_CHECK_ARG(blocks <= 0x7fffffff, "too many settings");
  if (n_terms <= PP_FEW)
    hipLaunchKernelGGL(phase_pair_kernel<256>, dim3((unsigned)blocks), dim3(256), 0, s, A, B, ld, n_terms,
                       n_settings, k_alpha, k_beta, phase8 & 7, pow_sqrt2, (float2*)mant, expo);
  else
    hipLaunchKernelGGL(phase_pair_kernel<1024>, dim3((unsigned)blocks), dim3(1024), 0, s, A, B, ld, n_terms,
                       n_settings, k_alpha, k_beta, phase8 & 7, pow_sqrt2, (float2*)mant, expo);
  ZX_HIP(hipGetLastError());
  return ZX_OK;
}

extern "C" zx_status zx_gf2_basis(const uint64_t* D, int32_t m, int32_t n_cols, int64_t ld, uint64_t* R,
                                  int32_t* rank_dev, int32_t* pivot_cols_dev, uint64_t* coeff, int64_t ldc,
                                  void* ws, size_t ws_bytes, hipStream_t s) {
  zx_clear_error();
  ZX_CHECK_ARG(D && R && coeff && D != R, "null argument or D == R");
  ZX_CHECK_ARG(m > 0 && n_cols > 0, "empty matrix");
  const int cwords = ((m < n_cols ? m : n_cols) + 63) / 64;
  ZX_CHECK_ARG(ldc >= cwords, "ldc %lld < %d", (long long)ldc, cwords);
  zx_status rc = zx_gf2_eliminate(D, R, m, n_cols, ld, rank_dev, pivot_cols_dev, nullptr, 0, ws, ws_bytes, s);
  if (rc != ZX_OK) return rc;
  const int64_t total = (int64_t)m * cwords;
  hipLaunchKernelGGL(basis_coeff_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, D, m, ld,
                     rank_dev, pivot_cols_dev, coeff, ldc, cwords);
  ZX_HIP(hipGetLastError());
  return ZX_OK;
}
