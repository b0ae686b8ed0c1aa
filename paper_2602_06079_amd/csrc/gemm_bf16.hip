// Batched bf16 MFMA GEMMs of the Newton-Schulz iteration (step 4 of the operator):
//   C[b][i][j] = sum_k P[b][i][k] * Q[b][j][k]        fp32 accumulate
// Both operands are contiguous along k (see kernels.h for why both orientations of X are
// kept), which is the lane layout v_mfma_f32_32x32x16_bf16 wants: lane l supplies 8
// consecutive k of row (l % 32), k-group (l / 32).  Operands and bf16 results live in the
// panel layout of panel_layout.h.
//
// Tiling: one 256-thread block (4 wavefronts, 2 x 2) owns a 256 x 256 tile of C; each
// wavefront owns 128 x 128 = 4 x 4 MFMA tiles, i.e. 256 fp32 accumulators per lane (one
// wavefront per SIMD, 512 registers each).  K is walked in steps of 32.
//
// Operand staging: a 256 x 32 panel is 16 KiB of contiguous memory that already has the
// bank-conflict-free LDS arrangement, so it goes from global memory straight into LDS as
// a linear copy (global_load_lds_dwordx4: a wavefront moves 1 KiB per instruction), into
// one of four 32 KiB stages (P panel + Q panel).
//
// Pipeline: moving 32 KiB per k-step from L2 into LDS takes about as long as the 32 MFMAs
// of the step, and a fetch needs more than a microsecond to land, so the ring is four
// stages deep: while step t is multiplied, steps t+1 .. t+3 are resident or in flight and
// step t+4 is being requested.  The MFMA operand fragments are double-buffered in
// registers.  A wavefront issues in order and an MFMA keeps the matrix pipe busy for 32
// cycles, so every other instruction is placed in the shadow of one MFMA: one LDS operand
// load after each of the first 8 MFMAs of a half-step, one direct load after every
// fourth.  One barrier per k-step, between its two half-steps: before it each wavefront
// waits for its own share of step t+1 (s_waitcnt vmcnt(16): the 16 younger loads of steps
// t+2 and t+3 may stay in flight); after it stage t is free for step t+4.
//
// Epilogue: the accumulators are re-arranged through LDS (free after the last step) into
// panel-layout images, one per wavefront, and leave as linear 16-byte-per-lane stores; the
// last product of the chain instead stages fp32 rows and applies the parameter update
// with 16-byte accesses on the caller's row-major buffers.
//
// Blocks are persistent (one per CU) and loop over tiles, so the stores of one tile's
// epilogue drain while the next tile is multiplied.  In every round the 32 blocks of one XCD
// (blockIdx % 8 selects the XCD) form a 4 x 8 patch of tiles of one matrix and share panels
// in that XCD's L2.
// Symmetric products (Gram, polynomial) run only the tiles on or above the diagonal and
// write the mirror image as well.  Extents are multiples of 256 (zero padded by the
// producer), so only the final epilogue clips to the caller's shape.
#include <algorithm>
#include <type_traits>

#include "device_util.h"
#include "panel_layout.h"

namespace canz {
namespace {

constexpr int BM = 256, BN = 256, BK = 32;
constexpr int NTHREADS = 256;
constexpr int CHUNKS = BK / 8;   // 16-byte chunks per panel row
constexpr int GROUP_M = 4;       // tile rows per raster band
constexpr int N_XCD = 8;
static_assert(BM == PANEL_ROWS && BK == PANEL_K, "tile = panel");

enum { EPI_GRAM = 0, EPI_POLY = 1, EPI_UPDATE = 2, EPI_FINAL = 3, EPI_FINAL_SYM = 4, EPI_MUL = 5, EPI_MUL_Q = 6, EPI_MUL_Q2 = 7,
       EPI_POLY_APART = 8, EPI_GRAM_APART = 9, EPI_UPDATE_APART = 10, EPI_B3 = 11, EPI_B3_SYM = 12, EPI_OUT_TERMS = 13, EPI_GRAM_T = 14 };
// EPI_FINAL_SYM: the last-product epilogue (the caller's dense buffers) over the tiles on and above the diagonal of a
// symmetric result only; the caller mirrors them into the lower triangle afterwards.
// EPI_*_APART, EPI_MUL*: the diagonals of the symmetric matrices are kept apart and their images are fp16 (kernels.h: SymSpec).
// EPI_MUL: product of two symmetric matrices that commute (polynomials in one Gram matrix): symmetric as well.
// EPI_MUL_Q: its result leaves as bf16 image and diagonal, for the update (EPI_UPDATE_APART); EPI_MUL_Q2: as two bf16 terms, diagonal
// included, for the last product (EPI_OUT_TERMS).
constexpr bool epi_mul(int epi) { return epi == EPI_MUL || epi == EPI_MUL_Q || epi == EPI_MUL_Q2; }
constexpr bool epi_f16_in(int epi) { return epi == EPI_POLY_APART || epi_mul(epi); }
constexpr bool epi_f16_out(int epi) { return epi == EPI_GRAM_APART || epi == EPI_POLY_APART || epi == EPI_MUL; }
constexpr bool epi_apart(int epi) { return epi_f16_in(epi) || epi == EPI_UPDATE_APART; }   // reads diagonals
constexpr bool epi_mspace(int epi) { return epi == EPI_GRAM || epi == EPI_GRAM_T || epi == EPI_GRAM_APART || epi == EPI_POLY || epi == EPI_POLY_APART || epi_mul(epi); }
// EPI_B3, EPI_B3_SYM, EPI_OUT_TERMS: products of matrices of up to three bf16 terms (launch_split3*): the result as three
// terms, the same for symmetric matrices that commute, and the last-product epilogue.
constexpr bool epi_terms(int epi) { return epi == EPI_B3 || epi == EPI_B3_SYM || epi == EPI_OUT_TERMS; }
constexpr bool epi_symmetric(int epi) { return epi_mspace(epi) || epi == EPI_FINAL_SYM || epi == EPI_B3_SYM; }
// symmetric, but element (i, j) not bit for bit (j, i): of two different matrices, or (POLY_APART) with a term of such a product
constexpr bool epi_two_factors(int epi) { return epi_f16_in(epi) || epi == EPI_B3_SYM; }
// EPI_GRAM_T, EPI_GRAM_APART: the Gram product reads its operand X from X^T, in which k runs over the rows: 32 x 32 pieces (32 k of 32 rows of
// X, 2 KiB of a panel) go into LDS as they lie, and the transposing LDS reads turn them into operands (k_major).  X itself is then nobody's
// operand, and neither the momentum kernel nor the update writes it.  The same products in the same order: an element has the same bits.
constexpr bool epi_k_major(int epi) { return epi == EPI_GRAM_T || epi == EPI_GRAM_APART; }
constexpr bool epi_final(int epi) { return epi == EPI_FINAL || epi == EPI_FINAL_SYM || epi == EPI_OUT_TERMS; }

struct EpiArgs {
  void* c;                 // GRAM/POLY: [nb][M][N] panels; UPDATE: straight output [nb][M][N] panels
  void* ct;                // UPDATE: transposed output [nb][N][M] panels; B3_SYM: 5/4 I - 1/4 C, or nullptr
  SymSpec sym;             // GRAM/POLY/MUL/UPDATE_APART: how the symmetric matrices are represented (kernels.h)
  const float* scale;      // per-matrix factor applied to the accumulator, or nullptr
  float ca, cb, cc;        // POLY coefficients
  // schedule of the persistent blocks (see launch()): full rounds of whole tiles, then the
  // `left` remaining tiles, each cut into `splits` k-slices that different blocks compute
  int full_rounds, left, splits, main_grid;
  float* partial;          // [gridDim][256 regs][256 threads] fp32 accumulators of the k-slices
};

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

#define CANZ_LDS(p) ((__attribute__((address_space(3))) void*)(p))
#define CANZ_GLB(p) ((const __attribute__((address_space(1))) void*)(p))

__device__ __forceinline__ int swz(int row, int chunk) {
  return (row * CHUNKS + (chunk ^ ((row >> 2) & (CHUNKS - 1)))) * 8;  // element offset in the panel
}

// The MFMA operand of 32 rows of X and 16 k from a piece of X^T in LDS, 32 k x 32 rows (from its k 0 or 16 on).  ds_read_b64_tr_b16: the 16
// lanes of a group supply the addresses of 4 k x 16 rows, 4 rows each, and lane j receives the 4 k of row j.  Groups 0 and 1 take
// rows 0 and 16 of k 0 .. 7, groups 2 and 3 those of k 8 .. 15, in two reads of 4 k (`half`): a half-wave reads 256 bytes of four consecutive k.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int k_major_lane(int lane, int half) {
  const int hi = lane >> 5, l = lane & 15, k = 8 * hi + 4 * half + (l >> 2);
  const int chunk = 2 * ((lane >> 4) & 1) + ((l >> 1) & 1);
  return k * 32 + ((chunk ^ ((k >> 2) & 3)) << 3) + 4 * (l & 1);
}
__device__ __forceinline__ bf16x8 k_major(const __bf16* piece, int lane0, int lane1) {
  typedef __attribute__((address_space(3))) s16x4 lds_vec;
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_vec*)CANZ_LDS(piece + lane0));
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_vec*)CANZ_LDS(piece + lane1));
  const s16x4 v[2] = {a, b};
  return __builtin_bit_cast(bf16x8, v);
}

// value of the neighbouring lane (lane ^ 1), through the DPP quad permute [1, 0, 3, 2]
__device__ __forceinline__ unsigned lane_xor1(unsigned v) {
  return static_cast<unsigned>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0xB1, 0xF, 0xF, false));
}

// logical tile index -> (matrix b, tile row tm, tile column tn)
template <int EPI>
__device__ __forceinline__ void decode_tile(int logical, int tiles_m, int tiles_n, int per_batch, int& b, int& tm,
                                            int& tn) {
  b = logical / per_batch;
  const int tix = logical - b * per_batch;
  if (epi_symmetric(EPI)) {
    // symmetric output: only tiles with tn >= tm exist (per_batch = nt (nt + 1) / 2); the
    // epilogue writes each off-diagonal tile twice, straight and mirrored.  Raster: bands of
    // 4 tile rows; inside the band starting at r0 the columns r0, r0+1, ... are walked one
    // after the other, column c holding the rows r0 .. min(r0 + 3, c).
    int rem = tix, band = 0;
    for (;;) {
      const int rows = min(GROUP_M, tiles_m - band * GROUP_M), cols = tiles_m - band * GROUP_M;
      const int cnt = rows * cols - rows * (rows - 1) / 2;
      if (rem < cnt) break;
      rem -= cnt;
      ++band;
    }
    const int r0 = band * GROUP_M;
    const int rows = min(GROUP_M, tiles_m - r0);
    const int tri = rows * (rows + 1) / 2;
    if (rem < tri) {
      int c = 0;
      while (rem >= c + 1) rem -= c + 1, ++c;
      tn = r0 + c;
      tm = r0 + rem;
    } else {
      rem -= tri;
      tn = r0 + rows + rem / rows;
      tm = r0 + rem % rows;
    }
  } else {
    // bands of 4 tile rows, walked column by column
    const int band = tix / (GROUP_M * tiles_n);
    const int in_band = tix - band * GROUP_M * tiles_n;
    const int rows_here = min(GROUP_M, tiles_m - band * GROUP_M);
    tn = in_band / rows_here;
    tm = band * GROUP_M + (in_band - tn * rows_here);
  }

}

// Matrices with their diagonal apart (kernels.h: SymSpec).  An image holds UNIT_A or UNIT_B times the off-diagonal elements;
// a product of two images is scaled to the unit of its result, and what a diagonal multiplies is added in the epilogue.
// Written once with the roundings pinned, so that both kernels produce the same bits.
//   factor of the accumulator
template <int EPI>
__device__ __forceinline__ float apart_factor(const EpiArgs& e) {
  return EPI == EPI_POLY_APART ? e.cc * (UNIT_B / (UNIT_A * UNIT_A)) : EPI == EPI_GRAM_APART ? UNIT_A : 1.f / UNIT_B;
}
//   weights of the elements of the first (row) and second (column) image: POLY has one image with both diagonals
template <int EPI>
__device__ __forceinline__ float apart_weight(const EpiArgs& e, float x, float y, bool second) {
  if (EPI == EPI_POLY_APART) return __builtin_fmaf(e.cc, x + y, e.cb) * (UNIT_B / UNIT_A);
  if (epi_mul(EPI) && second) return y * (e.sym.unit * (1.f / UNIT_B));
  return x;
}
//   the diagonal element itself, from what the accumulator holds after all of the above
template <int EPI>
__device__ __forceinline__ float apart_diagonal(float acc, float dx, float dy, const EpiArgs& e) {
  if (EPI == EPI_GRAM_APART) return acc * (1.f / UNIT_A);
  if (EPI == EPI_POLY_APART) return __builtin_fmaf(acc, 1.f / UNIT_B, __builtin_fmaf(__builtin_fmaf(e.cc, dx, e.cb), dx, e.ca));
  return __builtin_fmaf(acc, 1.f / e.sym.unit, dx * dy);
}

// two values of a 16-bit image, packed, and four of them
template <int EPI>
__device__ __forceinline__ unsigned image_pair(float a, float b) {
  if constexpr (epi_f16_out(EPI)) {
    const f16x2 t = {static_cast<_Float16>(a), static_cast<_Float16>(b)};
    return __builtin_bit_cast(unsigned, t);
  } else {
    bf16x2 t;
    t[0] = static_cast<__bf16>(a), t[1] = static_cast<__bf16>(b);
    return __builtin_bit_cast(unsigned, t);
  }
}
template <int EPI>
struct ImageIn {   // four consecutive elements of the images the epilogue reads
  typedef bf16x4 vec4;
};
template <>
struct ImageIn<EPI_POLY_APART> {
  typedef f16x4 vec4;
};
template <>
struct ImageIn<EPI_MUL> {
  typedef f16x4 vec4;
};
template <>
struct ImageIn<EPI_MUL_Q> {
  typedef f16x4 vec4;
};
template <>
struct ImageIn<EPI_MUL_Q2> {
  typedef f16x4 vec4;
};

// two bf16 values, packed, times -1/4
__device__ __forceinline__ unsigned minus_quarter(unsigned pair) {
  bf16x2 t;
  t[0] = static_cast<__bf16>(-0.25f * __builtin_bit_cast(float, pair << 16));
  t[1] = static_cast<__bf16>(-0.25f * __builtin_bit_cast(float, pair & 0xffff0000u));
  return __builtin_bit_cast(unsigned, t);
}
// the three bf16 terms of one element, `step` apart
__device__ __forceinline__ void put_three_terms(__bf16* to, int64_t step, float v) {
#pragma unroll
  for (int term = 0; term < 3; ++term) {
    to[term * step] = static_cast<__bf16>(v);
    v -= static_cast<float>(static_cast<__bf16>(v));
  }
}

// Epilogue of one 256 x 256 tile held in the accumulators of the block's four wavefronts
// (shared by the GEMM kernel and by the kernel that finishes k-split tiles).
// `stage`: this wavefront's private 32 KiB of LDS; `vec`: 128 floats of its own (epi_apart).
template <int EPI>
__device__ __forceinline__ void tile_epilogue(f32x16 (&acc)[4][4], __bf16* stage, int lane, int wm, int wn, int b,
                                              int tm, int tn, const GemmDims& d, const EpiArgs& e, const Shape& s,
                                              const OutSpec& o, float* vec) {
  // ---- epilogue.  Accumulator register r of lane l in MFMA tile (it, jt) is element
  //      row = 32 it + 8 (r / 4) + 4 (l / 32) + (r % 4),  col = 32 jt + (l % 32)
  //      of the wavefront's 128 x 128 part.  Each wavefront stages through its own 32 KiB.
  const int lj = lane & 31, lh = lane >> 5;

  // scale (first iteration: folded normalisation), or the polynomial in A for EPI_POLY
  if constexpr (EPI == EPI_POLY) {
    // A is symmetric bit for bit (the Gram epilogue writes both halves from the same
    // accumulators), so element (i, j) is read as (j, i): the wavefront's part of the mirrored
    // tile is copied linearly into its staging area (global -> LDS, 16 bytes per lane) and is
    // then the transposed image, in which a lane's four consecutive rows are four consecutive k.
    const __bf16* A = static_cast<const __bf16*>(e.sym.aux) + static_cast<int64_t>(b) * d.M * d.N;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      const __bf16* src = A + (static_cast<int64_t>(tn) * (d.M >> 5) + 8 * tm + 4 * wm + kb) * PANEL_ELEMS +
                          wn * 128 * PANEL_K + lane * 8;
#pragma unroll
      for (int x = 0; x < 8; ++x)
        __builtin_amdgcn_global_load_lds(CANZ_GLB(src + x * 512), CANZ_LDS(stage + kb * 4096 + x * 512), 16, 0, 0);
    }
    int a_base[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) a_base[g] = lj * 32 + ((g ^ ((lj >> 2) & 3)) << 3) + 4 * lh;
    __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0): the copy has landed
#pragma unroll
    for (int it = 0; it < 4; ++it)
#pragma unroll
      for (int jt = 0; jt < 4; ++jt) {
        const int col = tn * BN + wn * 128 + jt * 32 + lj;
        const int row0 = tm * BM + wm * 128 + it * 32 + 4 * lh;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const bf16x4 av = *reinterpret_cast<const bf16x4*>(stage + it * 4096 + jt * 32 * 32 + a_base[g]);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            acc[it][jt][4 * g + q] =
                poly_value(static_cast<float>(av[q]), acc[it][jt][4 * g + q], e.ca, e.cb, e.cc, row0 + 8 * g + q == col);
          }
        }
      }
    // every read of the staging area is done before the images below overwrite it
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  } else if constexpr (epi_apart(EPI) || EPI == EPI_GRAM_APART) {
    // The terms that carry a diagonal (SymSpec), and the element-wise term of the polynomial.  The images are
    // symmetric (off-diagonal tiles bit for bit: both halves are written from the same accumulators) or, for UPDATE,
    // there as X^T, so element (i, j) is read as (j, i), as above.
    constexpr bool UPD = EPI == EPI_UPDATE_APART;
    const int row_w = tm * BM + wm * 128 + 4 * lh, col_w = tn * BN + wn * 128 + lj;
    const float* const xv = epi_apart(EPI) ? e.sym.x + static_cast<int64_t>(b) * d.M : nullptr;
    const float* const yv = epi_f16_in(EPI) ? e.sym.y + static_cast<int64_t>(b) * d.M : nullptr;
    if constexpr (!UPD) {
      const float f = EPI == EPI_GRAM_APART && e.scale ? e.scale[b] * UNIT_A : apart_factor<EPI>(e);
#pragma unroll
      for (int it = 0; it < 4; ++it)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[it][jt][r] *= f;
    }
    if constexpr (epi_apart(EPI)) {
      int a_base[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) a_base[g] = lj * 32 + ((g ^ ((lj >> 2) & 3)) << 3) + 4 * lh;
      // the diagonal elements of the part's 128 rows, once per tile (a load per group of rows would cost a memory latency each)
      vec[lane] = xv[tm * BM + wm * 128 + lane], vec[64 + lane] = xv[tm * BM + wm * 128 + 64 + lane];
      // acc(i, j) += weight(i, j) image(i, j)
      auto fold = [&](const void* matrix, auto second) {
        constexpr bool SECOND = decltype(second)::value;
        const __bf16* A = static_cast<const __bf16*>(matrix) + static_cast<int64_t>(b) * d.M * d.N;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
          const __bf16* src = A + (static_cast<int64_t>(tn) * (d.M >> 5) + 8 * tm + 4 * wm + kb) * PANEL_ELEMS +
                              wn * 128 * PANEL_K + lane * 8;
#pragma unroll
          for (int x = 0; x < 8; ++x)
            __builtin_amdgcn_global_load_lds(CANZ_GLB(src + x * 512), CANZ_LDS(stage + kb * 4096 + x * 512), 16, 0, 0);
        }
        float cw[4];
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) cw[jt] = EPI == EPI_POLY_APART || SECOND ? yv[col_w + jt * 32] : 0.f;
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0): the copy has landed
#pragma unroll
        for (int it = 0; it < 4; ++it)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            f32x4 rw = {0.f, 0.f, 0.f, 0.f};
            if (!SECOND) rw = *reinterpret_cast<const f32x4*>(vec + it * 32 + 8 * g + 4 * lh);
#pragma unroll
            for (int jt = 0; jt < 4; ++jt) {
              const auto av = *reinterpret_cast<const typename ImageIn<EPI>::vec4*>(stage + it * 4096 + jt * 32 * 32 + a_base[g]);
#pragma unroll
              for (int q = 0; q < 4; ++q)
                acc[it][jt][4 * g + q] = __builtin_fmaf(apart_weight<EPI>(e, rw[q], cw[jt], SECOND), static_cast<float>(av[q]), acc[it][jt][4 * g + q]);
            }
            __builtin_amdgcn_sched_barrier(0);   // one group's reads at a time: the accumulators leave few registers
          }
        // every read of the staging area is done before it is written again
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      };
      // always, but a branch: as straight-line code behind the k loop the fold is spilled by the hundred
      if (e.sym.aux) fold(e.sym.aux, std::false_type{});
      if constexpr (epi_mul(EPI))
        if (e.sym.aux2) fold(e.sym.aux2, std::true_type{});
    }
    if constexpr (UPD) {
      const float sc = e.scale ? e.scale[b] : 1.f;
#pragma unroll
      for (int it = 0; it < 4; ++it)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[it][jt][r] *= sc;
    } else if (tm == tn && wm == wn) {   // the diagonal goes to its own fp32 vector, the image holds zeros there (Q2: all in the image)
      float* dv = EPI == EPI_MUL_Q2 ? nullptr : e.sym.diag + static_cast<int64_t>(b) * d.M;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int col = col_w + it * 32;
        const float dx = xv ? xv[col] : 0.f, dy = yv ? yv[col] : 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (row_w + it * 32 + 8 * (r >> 2) + (r & 3) == col) {
            const float v = apart_diagonal<EPI>(acc[it][it][r], dx, dy, e);
            if (EPI != EPI_MUL_Q2) dv[col] = v;
            acc[it][it][r] = EPI == EPI_MUL_Q2 ? v * e.sym.unit : 0.f;
          }
      }
    }
    if constexpr (EPI == EPI_MUL_Q || EPI == EPI_MUL_Q2) {
      const float inv = 1.f / e.sym.unit;   // a power of two
#pragma unroll
      for (int it = 0; it < 4; ++it)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[it][jt][r] *= inv;
    }
    if constexpr (epi_f16_out(EPI)) {
      // one fp32 value for both images: no operation is fused into one of the two conversions and not into the other
#pragma unroll
      for (int it = 0; it < 4; ++it)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) asm volatile("" : "+a"(acc[it][jt]));
    }
  } else if (e.scale) {
    const float sc = e.scale[b];
#pragma unroll
    for (int it = 0; it < 4; ++it)
#pragma unroll
      for (int jt = 0; jt < 4; ++jt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[it][jt][r] *= sc;
  }

  // the wavefront's part of an output tile in panel layout: four pieces of 8 KiB (the four
  // 32-wide k-blocks it covers), 128 rows each; LDS image == memory image
  auto flush_stage = [&](__bf16* out, int64_t row_block, int64_t kc, int64_t kblock0, int half_rows) {
    // out: matrix base; the wavefront's rows start at row_block * 256 + half_rows * 128
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      __bf16* dst = out + (row_block * (kc >> 5) + kblock0 + kb) * PANEL_ELEMS + half_rows * 128 * PANEL_K;
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(stage + kb * 4096 + (x * 64 + lane) * 8);
        *reinterpret_cast<u32x4*>(dst + (x * 64 + lane) * 8) = v;
      }
    }
  };

  if constexpr (EPI == EPI_B3 || EPI == EPI_B3_SYM || EPI == EPI_MUL_Q2) {
    // Three terms per element (Q2: two), through the staging area as the bf16 images below (whose offsets these are): each pass rounds
    // what is left to bf16, writes it (for a symmetric result also mirrored) and takes it away.  5/4 I - 1/4 C, where it is
    // asked for, has -1/4 of the terms of C off the diagonal, exactly; its diagonal is put in place at the end.
    constexpr bool SYM = EPI != EPI_B3;
    constexpr int NT = EPI == EPI_MUL_Q2 ? 2 : 3;
    if (e.c == nullptr) return;   // never: a branch that parts the epilogue from the k loop's block, see the folds above
    int s_base[2], t_base[4];
#pragma unroll
    for (int g1 = 0; g1 < 2; ++g1)
      s_base[g1] = (4 * lh + (lane & 1)) * 32 + ((((lj >> 3) ^ (2 * g1 + lh)) & 3) << 3) + (lj & 6);
#pragma unroll
    for (int g = 0; g < 4; ++g) t_base[g] = lj * 32 + ((g ^ ((lj >> 2) & 3)) << 3) + 4 * lh;
    const unsigned pair_sel = (lane & 1) ? 0x03020706u : 0x05040100u;
    const int64_t nkb = d.N >> 5, elems = NT * d.M * d.N;
    __bf16* const C = static_cast<__bf16*>(e.c) + static_cast<int64_t>(b) * elems;
    __bf16* const T = EPI == EPI_B3_SYM && e.ct ? static_cast<__bf16*>(e.ct) + static_cast<int64_t>(b) * elems : nullptr;
    const bool diagonal = SYM && tm == tn && wm == wn;
    float dv[4];
    if (T && diagonal) {
#pragma unroll
      for (int it = 0; it < 4; ++it)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (8 * (r >> 2) + (r & 3) + 4 * lh == lj) dv[it] = acc[it][it][r];
    }
#pragma unroll 1
    for (int term = 0; term < NT; ++term) {
      auto flush = [&](int64_t row_block, int64_t kblock0, int half_rows) {
        const int64_t at = (row_block * NT * nkb + term * nkb + kblock0) * PANEL_ELEMS + half_rows * 128 * PANEL_K + lane * 8;
#pragma unroll
        for (int k4 = 0; k4 < 4; ++k4)
#pragma unroll
          for (int x = 0; x < 8; ++x)
            *reinterpret_cast<u32x4*>(C + at + k4 * PANEL_ELEMS + x * 512) = *reinterpret_cast<const u32x4*>(stage + k4 * 4096 + (x * 64 + lane) * 8);
        if (T) {
#pragma unroll
          for (int k4 = 0; k4 < 4; ++k4)
#pragma unroll
            for (int x = 0; x < 8; ++x) {
              u32x4 v = *reinterpret_cast<const u32x4*>(stage + k4 * 4096 + (x * 64 + lane) * 8);
#pragma unroll
              for (int q = 0; q < 4; ++q) v[q] = minus_quarter(v[q]);
              *reinterpret_cast<u32x4*>(T + at + k4 * PANEL_ELEMS + x * 512) = v;
            }
        }
      };
      auto pair = [&](int it, int jt, int r) {
        bf16x2 own;
        own[0] = static_cast<__bf16>(acc[it][jt][r]);
        own[1] = static_cast<__bf16>(acc[it][jt][r + 1]);
        return own;
      };
      if (SYM) {
        if (tm != tn || wm < wn) {
#pragma unroll
          for (int it = 0; it < 4; ++it)
#pragma unroll
            for (int jt = 0; jt < 4; ++jt)
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                const u32x2 w = {__builtin_bit_cast(unsigned, pair(it, jt, 4 * g)), __builtin_bit_cast(unsigned, pair(it, jt, 4 * g + 2))};
                *reinterpret_cast<u32x2*>(stage + it * 4096 + jt * 32 * 32 + t_base[g]) = w;
              }
          flush(tn, 8 * tm + 4 * wm, wn);
        }
        // the straight image rounds anew: kept from the mirrored one, the pairs would be spilled by the hundred
#pragma unroll
        for (int it = 0; it < 4; ++it)
#pragma unroll
          for (int jt = 0; jt < 4; ++jt) asm volatile("" : "+a"(acc[it][jt]));
      }
#pragma unroll
      for (int it = 0; it < 4; ++it)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
#pragma unroll
          for (int rp = 0; rp < 8; ++rp) {
            const bf16x2 own = pair(it, jt, 2 * rp);
            acc[it][jt][2 * rp] -= static_cast<float>(own[0]);
            acc[it][jt][2 * rp + 1] -= static_cast<float>(own[1]);
            const unsigned mine = __builtin_bit_cast(unsigned, own);
            const int g = rp >> 1, p = rp & 1;
            *reinterpret_cast<unsigned*>(stage + jt * 4096 + (it * 32 + 8 * g + 2 * p) * 32 + s_base[g & 1]) =
                __builtin_amdgcn_perm(lane_xor1(mine), mine, pair_sel);
          }
      if (!SYM || tm != tn || wm <= wn) flush(tm, 8 * tn + 4 * wn, wm);
    }
    if (T && diagonal && ((lj >> 2) & 1) == lh) {
      __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0): the images are written, these elements go over theirs
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int64_t i = tm * BM + wm * 128 + 32 * it + lj;
        put_three_terms(T + panel_chunk_off(i, i & ~7, 3 * d.N) + (i & 7), nkb * PANEL_ELEMS, 1.25f - 0.25f * dv[it]);
      }
    }
    return;
  }
  if (!epi_final(EPI)) {
    // ---- straight image: element (i, j) of C is (row i, k = j) of the result's panels.
    // A 16-byte chunk is 8 consecutive j of one row, i.e. one value from each of 8 lanes:
    // neighbouring lanes exchange their packed pairs so that every lane writes two bf16 of
    // one row.
    const int64_t image = static_cast<int64_t>(b) * d.M * d.N;
    // Staging offset = (lane-only base) + (compile-time part), so that the compiler keeps two
    // address registers instead of one per store.  Element (row_l, col_l) of the wavefront's
    // part, row_l = 32 it + 8 g + 2 p + 4 lh + odd (rp = 2 g + p), col_l = 32 jt + lj, lies in
    // k-block jt at row_l * 32 + ((chunk ^ swizzle) << 3) with chunk = lj >> 3 and
    // swizzle = (row_l >> 2) & 3 = 2 (g & 1) + lh: lane bits except for g & 1.
    // byte selector of v_perm_b32 over {theirs (bytes 4..7), mine (bytes 0..3)}
    const unsigned pair_sel = (lane & 1) ? 0x03020706u : 0x05040100u;
    const bool diagonal_tile = epi_mspace(EPI) && tm == tn;
    if (epi_mspace(EPI) || e.c != nullptr) {   // (an update may be asked for the transposed image alone)
    int s_base[2];
#pragma unroll
    for (int g1 = 0; g1 < 2; ++g1)
      s_base[g1] = (4 * lh + (lane & 1)) * 32 + ((((lj >> 3) ^ (2 * g1 + lh)) & 3) << 3) + (lj & 6);
#pragma unroll
    for (int it = 0; it < 4; ++it)
#pragma unroll
      for (int jt = 0; jt < 4; ++jt)
#pragma unroll
        for (int rp = 0; rp < 8; ++rp) {  // register pairs (2 rp, 2 rp + 1): rows differ by one
          // both rows of this lane's column, packed; the even lane keeps the low halves of
          // the pair of lanes (row 2 rp), the odd lane the high halves (row 2 rp + 1)
          const unsigned mine = image_pair<EPI>(acc[it][jt][2 * rp], acc[it][jt][2 * rp + 1]);
          const unsigned theirs = lane_xor1(mine);
          const unsigned pk = __builtin_amdgcn_perm(theirs, mine, pair_sel);
          const int g = rp >> 1, p = rp & 1;
          const int fixed = jt * 4096 + (it * 32 + 8 * g + 2 * p) * 32;
          *reinterpret_cast<unsigned*>(stage + fixed + s_base[g & 1]) = pk;
        }
    // In a diagonal tile the lower left quarter is the mirror image of the upper right one, as in the small kernel: the
    // two are equal bit for bit when both factors are the same matrix, but only to rounding in a product of two.
    if (!diagonal_tile || wm <= wn) flush_stage(static_cast<__bf16*>(e.c) + image, tm, d.N, 8 * tn + 4 * wn, wm);
    }

    // ---- transposed image: element (i, j) is (row j, k = i) of CT (UPDATE) or of the mirror
    // tile of C (symmetric products).  A lane's 4 consecutive rows are half a chunk.
    const bool mirror = epi_mspace(EPI);
    if (!diagonal_tile || wm < wn) {
      __bf16* const CT = static_cast<__bf16*>(mirror ? e.c : e.ct) + image;
      // element (i_l, j_l) goes to row j_l = 32 jt + lj, k = i_l = 32 it + 8 g + 4 lh + q:
      // k-block it, chunk g, swizzle (lj >> 2) & 3: one lane base per g, the rest immediate
      int t_base[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) t_base[g] = lj * 32 + ((g ^ ((lj >> 2) & 3)) << 3) + 4 * lh;
#pragma unroll
      for (int it = 0; it < 4; ++it)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const u32x2 pk = {image_pair<EPI>(acc[it][jt][4 * g], acc[it][jt][4 * g + 1]), image_pair<EPI>(acc[it][jt][4 * g + 2], acc[it][jt][4 * g + 3])};
            *reinterpret_cast<u32x2*>(stage + it * 4096 + jt * 32 * 32 + t_base[g]) = pk;
          }
      flush_stage(CT, tn, d.M, 8 * tm + 4 * wm, wn);
    }
  } else {
    // ---- last product: O in the caller's orientation (the host orders the operands so).
    const int ld = static_cast<int>(o.out_mode == CANZ_OUT_DELTA ? s.wfrag : s.cols);
    // whole 128 x 128 part inside the matrix (uniform over the wavefront): no predicates
    const bool inside = tm * BM + wm * 128 + 128 <= s.rows && tn * BN + wn * 128 + 128 <= s.cols;
    // fp32 rows through LDS, 64 rows x 128 columns at a time; the column index is XOR-ed
    // with 32 on rows whose bit 2 is set so that the two half-waves hit different banks.
    // A lane handles 4 columns, in rows of any length: aligned to an element only where that is no multiple of 4.
    // One instantiation per (output mode, output dtype): the branches stay outside the
    // unrolled code.
    auto run = [&](auto mode_tag, auto dtype_tag) {
      constexpr int MODE = decltype(mode_tag)::value, DTYPE = decltype(dtype_tag)::value;
      float* sf = reinterpret_cast<float*>(stage);
      int f_base[2], r_base[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        f_base[p] = 4 * lh * 128 + lj + 32 * (p ^ lh);
        r_base[p] = lh * 128 + ((lj * 4) ^ (p << 5));
      }
      // per-lane element offset of (row 0 of the wavefront's part, its 4 columns) in the
      // caller's buffer, and the buffer itself (TP: the fragment that holds these columns)
      const int col = tn * BN + wn * 128 + lj * 4;
      const bool col_ok = col + 4 <= s.cols;
      const int n_tail = col_ok ? 0 : max(static_cast<int>(s.cols) - col, 0);   // columns before the edge that cuts the four
      int c_in = col, tab = b;
      if (MODE == CANZ_OUT_DELTA) {
        const int f = col < s.cols ? col / ld : 0;
        c_in = col - f * ld;
        tab = b * s.tp + f;
      }
      char* base = static_cast<char*>(o.out.p[tab]);
      constexpr int ESZ = DTYPE == CANZ_DT_F32 ? 4 : 2;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int row_base = tm * BM + wm * 128 + half * 64 + lh;
        auto stage_half = [&]() {
#pragma unroll
          for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
            for (int jt = 0; jt < 4; ++jt)
#pragma unroll
              for (int r = 0; r < 16; ++r) {
                // (32 jt + lj) ^ (32 lh) = lj + 32 (jt ^ lh): lane base per parity of jt
                const int fixed = (i2 * 32 + 8 * (r >> 2) + (r & 3)) * 128 + (jt & ~1) * 32;
                sf[fixed + f_base[jt & 1]] = acc[half * 2 + i2][jt][r];
              }
        };
        if (inside) {
          // The lane handles 4 columns of the 32 rows row_base + 2 i.  All old values of the
          // half are requested at once and every one of them is consumed before the first
          // store is issued: the half then costs one memory latency (with loads and stores
          // interleaved, each group of rows would wait for the stores of the one before).
          char* const ptr0 = base + (static_cast<int64_t>(row_base) * ld + c_in) * ESZ;
          const int64_t pitch2 = static_cast<int64_t>(2) * ld * ESZ;
          f32x4 val[32];
          if (MODE == CANZ_OUT_PARAM) {
#pragma unroll
            for (int i = 0; i < 32; ++i) {
              if (DTYPE == CANZ_DT_F32) {
                val[i] = *reinterpret_cast<const f32x4_any*>(ptr0 + i * pitch2);
              } else {
                const bf16x4 ob = *reinterpret_cast<const bf16x4_any*>(ptr0 + i * pitch2);
#pragma unroll
                for (int q = 0; q < 4; ++q) val[i][q] = static_cast<float>(ob[q]);
              }
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          stage_half();
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < 32; ++i) {
            // row 2 i + lh of the staged half; bit 2 of that row is bit 1 of i
            const f32x4 v = *reinterpret_cast<const f32x4*>(sf + 2 * i * 128 + r_base[(i >> 1) & 1]);
#pragma unroll
            for (int q = 0; q < 4; ++q)
              val[i][q] = MODE == CANZ_OUT_PARAM ? apply_update(val[i][q], o.decay, o.neg_lr_scale, v[q])
                                                 : o.neg_lr_scale * v[q];
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < 32; ++i) {
            if (DTYPE == CANZ_DT_F32) {
              *reinterpret_cast<f32x4_any*>(ptr0 + i * pitch2) = val[i];
            } else {
              bf16x4 rb;
#pragma unroll
              for (int q = 0; q < 4; ++q) rb[q] = static_cast<__bf16>(val[i][q]);
              *reinterpret_cast<bf16x4_any*>(ptr0 + i * pitch2) = rb;
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          continue;
        }
        // ragged edge of the matrix: rows and columns checked one by one, 4 rows at a time
        stage_half();
#pragma unroll
        for (int x4 = 0; x4 < 8; ++x4) {  // loads of old values first
          f32x4 v[4], old[4];
          char* ptr[4];
          bool live[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            // lane reads 4 columns of row 2 (4 x4 + u) + lh; bit 2 of that row is bit 1 of u
            v[u] = *reinterpret_cast<const f32x4*>(sf + 2 * (x4 * 4 + u) * 128 + r_base[(u >> 1) & 1]);
            const int row = row_base + 2 * (x4 * 4 + u);
            live[u] = col_ok && row < s.rows;
            ptr[u] = base + (static_cast<int64_t>(row) * ld + c_in) * ESZ;
          }
          if (MODE == CANZ_OUT_PARAM) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (!live[u]) continue;
              if (DTYPE == CANZ_DT_F32) {
                old[u] = *reinterpret_cast<const f32x4_any*>(ptr[u]);
              } else {
                const bf16x4 ob = *reinterpret_cast<const bf16x4_any*>(ptr[u]);
#pragma unroll
                for (int q = 0; q < 4; ++q) old[u][q] = static_cast<float>(ob[q]);
              }
            }
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (!live[u]) continue;
            f32x4 res;
#pragma unroll
            for (int q = 0; q < 4; ++q)
              res[q] = MODE == CANZ_OUT_PARAM ? apply_update(old[u][q], o.decay, o.neg_lr_scale, v[u][q])
                                              : o.neg_lr_scale * v[u][q];
            if (DTYPE == CANZ_DT_F32) {
              *reinterpret_cast<f32x4_any*>(ptr[u]) = res;
            } else {
              bf16x4 rb;
#pragma unroll
              for (int q = 0; q < 4; ++q) rb[q] = static_cast<__bf16>(res[q]);
              *reinterpret_cast<bf16x4_any*>(ptr[u]) = rb;
            }
          }
        }
        if (n_tail > 0) {
          typedef typename std::conditional<DTYPE == CANZ_DT_F32, float, __bf16>::type elem;
#pragma unroll 1
          for (int i = 0; i < 32; ++i) {
            const int row = row_base + 2 * i;
            if (row >= s.rows) break;
#pragma unroll 1
            for (int q = 0; q < n_tail; ++q) {
              elem* const at = reinterpret_cast<elem*>(base) + static_cast<int64_t>(row) * ld + c_in + q;
              const float v = sf[2 * i * 128 + ((i & 2) ? r_base[1] : r_base[0]) + q];
              *at = static_cast<elem>(MODE == CANZ_OUT_PARAM ? apply_update(static_cast<float>(*at), o.decay, o.neg_lr_scale, v)
                                                             : o.neg_lr_scale * v);
            }
          }
        }
      }
    };
    using P_ = std::integral_constant<int, CANZ_OUT_PARAM>;
    using D_ = std::integral_constant<int, CANZ_OUT_DELTA>;
    using F_ = std::integral_constant<int, CANZ_DT_F32>;
    using B_ = std::integral_constant<int, CANZ_DT_BF16>;
    if (o.out_mode == CANZ_OUT_PARAM) {
      if (o.out_dtype == CANZ_DT_F32) run(P_{}, F_{}); else run(P_{}, B_{});
    } else {
      if (o.out_dtype == CANZ_DT_F32) run(D_{}, F_{}); else run(D_{}, B_{});
    }
  }
}

template <int EPI>
__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  if constexpr (epi_f16_in(EPI))
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Element offset of the next panel of an operand of several terms: nk panels of the first segment's term, then of the
// second's, ...  No branches: one in the k loop would cost the compiler its count of the loads in flight.  Behind the
// last segment the code reads 0: a harmless re-read of term 0.
struct TermWalk {
  int64_t off, nk;
  unsigned code;
  int left;
  __device__ __forceinline__ TermWalk(unsigned c, int64_t n) : off((c & 15) * n * PANEL_ELEMS), nk(n), code(c), left(static_cast<int>(n)) {}
  __device__ __forceinline__ void next() {
    const bool end = --left == 0;
    code = end ? code >> 4 : code;
    off = end ? (code & 15) * nk * PANEL_ELEMS : off + PANEL_ELEMS;
    left = end ? static_cast<int>(nk) : left;
  }
};

// Element offset of k-step k of an operand that is read from X^T (epi_k_major): 32 rows further, 256 of which lie in a row of `panels` panels.
__device__ __forceinline__ int64_t k_major_off(int k, int64_t panels) { return (k >> 3) * panels * PANEL_ELEMS + (k & 7) * 1024; }

// Operands of a launch: one product (the usual case), or several of different shapes.
struct OneProblem {
  static constexpr bool multi = false, finals = false;
  GemmDims d;
  const __bf16* P;
  const __bf16* Q;
};
template <int MAX>
struct ManyProblemsOf {
  static constexpr bool multi = true, finals = false;
  static constexpr int max = MAX;
  int n;
  int begin[MAX + 1];  // first logical tile of each problem, then the total
  GemmProblem pr[MAX];
};
// Last products of several parts of a call.
struct FinalParts {
  static constexpr bool multi = true, finals = true;
  int n;
  int begin[MAX_PARTS + 1];
  FinalPart pr[MAX_PARTS];
};
// Room for two problems of each shape class only where a launch holds two: every block reads the descriptor first.
template <int EPI>
using ManyProblems = ManyProblemsOf<EPI == EPI_MUL || EPI == EPI_B3_SYM ? MAX_PROBLEMS : MAX_KINDS>;

template <int EPI, bool SPLIT, typename Args>
__global__ __launch_bounds__(NTHREADS) void k_gemm_nt_bf16(Args args, EpiArgs e_launch, Shape s, OutSpec o) {
  // one array per stage (not one carved buffer): the compiler then knows that a fetch into
  // one stage does not alias the operand reads of another and keeps them overlapped.
  // Elements [0, 8192) hold the P panel, [8192, 16384) the Q panel.
  constexpr int QOFF = BM * BK;
  __shared__ __attribute__((aligned(1024))) __bf16 st0[(BM + BN) * BK];
  __shared__ __attribute__((aligned(1024))) __bf16 st1[(BM + BN) * BK];
  __shared__ __attribute__((aligned(1024))) __bf16 st2[(BM + BN) * BK];
  __shared__ __attribute__((aligned(1024))) __bf16 st3[(BM + BN) * BK];

  // ---- persistent blocks: the grid is one block per CU (or fewer); block `bid` works on the
  //      logical tiles round * gridDim + slot(bid).  slot() makes the 32 blocks of one XCD
  //      (blockIdx % 8 selects the XCD) neighbours, so that in every round they form a 4 x 8
  //      patch of tiles of one matrix and share panels in that XCD's L2.
  GemmDims d{};
  const __bf16 *P = nullptr, *Q = nullptr;
  EpiArgs e = e_launch;
  if constexpr (!Args::multi) d = args.d, P = args.P, Q = args.Q;
  int tiles_n = static_cast<int>(d.N / BN);
  int tiles_m = static_cast<int>(d.M / BM);
  int per_batch = epi_symmetric(EPI) ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  int slot;
  {
    const int nblocks = gridDim.x, bid = blockIdx.x;
    const int per = nblocks / N_XCD, rem = nblocks % N_XCD;
    const int xcd = bid % N_XCD, q = bid / N_XCD;
    slot = xcd < rem ? xcd * (per + 1) + q : rem * (per + 1) + (xcd - rem) * per + q;
  }

  const int t = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  int nk_all = static_cast<int>(d.K / BK);  // multiple of 8: K is a multiple of 256
  __shared__ __attribute__((aligned(16))) float vec[epi_apart(EPI) ? 4 * 128 : 4];

  for (int work = 0;; ++work) {
  // ---- what to do in this round: a whole tile, or one k-slice of a left-over tile.  When
  //      the tiles do not fill the last round, each left-over tile is cut along k so that the
  //      whole chip shares them (second launch); the slices' accumulators are parked in global
  //      memory and k_split_finish adds them up and runs the epilogue.
  // SPLIT = false: persistent blocks over whole tiles (the full rounds, plus the left-over
  // tiles if they are not split).  SPLIT = true: a second launch in which every block
  // computes one k-slice of one left-over tile and parks its accumulators.
  int logical, k_begin = 0, nk = nk_all;
  if (!SPLIT) {
    const int rounds = e.full_rounds + (e.splits == 1 && slot < e.left ? 1 : 0);
    if (work >= rounds) break;
    logical = work * e.main_grid + slot;
  } else {
    if (work > 0) break;
    const int l = slot / e.splits, sl = slot - l * e.splits;
    logical = e.full_rounds * e.main_grid + l;
    const int groups = nk_all / 4, base = groups / e.splits, extra = groups % e.splits;
    k_begin = 4 * (sl * base + min(sl, extra));
    nk = 4 * (base + (sl < extra ? 1 : 0));
  }
  // The lane id is made opaque once per tile: otherwise every lane-dependent address of the
  // loop body (hundreds of them) is hoisted out of the tile loop and kept alive in scratch.
  int lane = t & 63;
  asm volatile("" : "+v"(lane));
  if constexpr (Args::multi) {
    // which product this tile belongs to; its extents, operands and outputs
    int j = 0;
    while (j + 1 < args.n && logical >= args.begin[j + 1]) ++j;
    const GemmProblem& pr = args.pr[j];
    d = pr.d;
    P = static_cast<const __bf16*>(pr.p), Q = static_cast<const __bf16*>(pr.q);
    e.c = pr.c, e.ct = pr.ct, e.sym = pr.sym, e.scale = pr.scale;
    logical -= args.begin[j];
    tiles_n = static_cast<int>(d.N / BN), tiles_m = static_cast<int>(d.M / BM);
    per_batch = epi_symmetric(EPI) ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
    nk_all = static_cast<int>(d.K / BK);
    nk = nk_all;
  }
  if constexpr (epi_terms(EPI)) nk = nk_all * d.nseg;
  int b, tm, tn;
  decode_tile<EPI>(logical, tiles_m, tiles_n, per_batch, b, tm, tn);

  // ---- global -> LDS: panel (tile row, k-step) is 16 KiB contiguous; wavefront w copies the
  //      1 KiB pieces w, w+4, w+8, w+12 of both panels, lane l the 16 bytes at l * 16.
  const int64_t nkb = d.K / BK;
  // panels per row block (operands that are a part of longer rows: only of the last products and those of several terms)
  const int64_t nkp = epi_terms(EPI) || epi_final(EPI) ? d.ldp / BK : nkb, nkq = epi_terms(EPI) || epi_final(EPI) ? d.ldq / BK : nkb;
  constexpr bool KM = epi_k_major(EPI);
  constexpr int G_STEP = KM ? 2 * PANEL_ELEMS : 2048;   // from one of a wavefront's 1 KiB pieces of a panel to the next
  const int64_t km_lane = (wave >> 1) * PANEL_ELEMS + (wave & 1) * 512 + lane * 8;
  const __bf16* pl = P + static_cast<int64_t>(b) * d.sp + (KM ? 8 * tm * PANEL_ELEMS + km_lane : (static_cast<int64_t>(tm) * nkp + k_begin) * PANEL_ELEMS + wave * 512 + lane * 8);
  const __bf16* ql = Q + static_cast<int64_t>(b) * d.sq + (KM ? 8 * tn * PANEL_ELEMS + km_lane : (static_cast<int64_t>(tn) * nkq + k_begin) * PANEL_ELEMS + wave * 512 + lane * 8);
  // operands of several terms: where the next panel of each is (the panels are requested in order)
  TermWalk wp(d.pseg, nkb), wq(d.qseg, nkb);
  // one of the 8 direct loads of a stage: idx 0..3 -> P pieces, 4..7 -> Q pieces
  auto fetch_one = [&](__bf16* st, int64_t kt, int idx) {
    const int g = idx & 3;
    if (idx < 4) {
      const int64_t off = epi_terms(EPI) ? wp.off : KM ? k_major_off(static_cast<int>(kt) + k_begin, d.M >> 5) : kt * PANEL_ELEMS;
      __builtin_amdgcn_global_load_lds(CANZ_GLB(pl + off + g * G_STEP), CANZ_LDS(st + wave * 512 + g * 2048), 16, 0, 0);
      if (epi_terms(EPI) && g == 3) wp.next();
    } else {
      const int64_t off = epi_terms(EPI) ? wq.off : KM ? k_major_off(static_cast<int>(kt) + k_begin, d.M >> 5) : kt * PANEL_ELEMS;
      __builtin_amdgcn_global_load_lds(CANZ_GLB(ql + off + g * G_STEP), CANZ_LDS(st + QOFF + wave * 512 + g * 2048), 16, 0, 0);
      if (epi_terms(EPI) && g == 3) wq.next();
    }
  };
  auto fetch = [&](__bf16* st, int64_t kt) {
#pragma unroll
    for (int idx = 0; idx < 8; ++idx) fetch_one(st, kt, idx);
  };

  // not cleared: the first 16 MFMAs of a tile take the constant 0 as their addend
  f32x16 acc[4][4];

  // MFMA operand fragments, double-buffered in registers: idx 0..3 -> rows of P, 4..7 -> rows of Q
  const int frag_row = lane & 31, frag_kg = lane >> 5;
  bf16x8 fa[2][4], fb[2][4];
  const int km0 = k_major_lane(lane, 0), km1 = k_major_lane(lane, 1);
  auto frag_one = [&](const __bf16* st, int kk, int set, int idx) {
    if (KM && idx < 4)
      fa[set][idx] = k_major(st + (wm * 4 + idx) * 1024 + kk * 512, km0, km1);
    else if (KM)
      fb[set][idx - 4] = k_major(st + QOFF + (wn * 4 + idx - 4) * 1024 + kk * 512, km0, km1);
    else if (idx < 4)
      fa[set][idx] = *reinterpret_cast<const bf16x8*>(st + swz(wm * 128 + idx * 32 + frag_row, kk * 2 + frag_kg));
    else
      fb[set][idx - 4] =
          *reinterpret_cast<const bf16x8*>(st + QOFF + swz(wn * 128 + (idx - 4) * 32 + frag_row, kk * 2 + frag_kg));
  };
  auto mma_one = [&](auto first, int set, int idx) {
    const int i = idx >> 2, j = idx & 3;
    if (decltype(first)::value) {
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      acc[i][j] = mfma<EPI>(fa[set][i], fb[set][j], zero);
    } else {
      acc[i][j] = mfma<EPI>(fa[set][i], fb[set][j], acc[i][j]);
    }
  };

  // The issue order below is pinned with scheduling fences (left to itself the compiler
  // clusters the loads and the matrix pipe drains meanwhile).
#define CANZ_FENCE() __builtin_amdgcn_sched_barrier(0)
  // One k-step on stage `cur`; `nxt` holds step kt+1, `prv` (free since the barrier of the
  // previous step) receives the Q panel of step kt+3, `cur` after this step's barrier the P
  // panel of step kt+4.  The loads of the whole tile are issued in the order P0 Q0 P1 Q1 ...;
  // in the middle of step kt the youngest is Q(kt+3), so "all but the 16 youngest have
  // landed" means that step kt+1 is complete.  The last four steps of a tile have nothing
  // left to request: they are separate instances (compile-time flags, no branch in the
  // body - a branch would cost the compiler its count of the loads in flight) with the
  // wait counts that follow from the shorter queue.
  using Yes = std::true_type;
  using No = std::false_type;
  auto k_step = [&](auto first, auto fetch_q, auto fetch_p, auto read_next, auto wait_code, __bf16* cur,
                    const __bf16* nxt, __bf16* prv, int kt) {
#pragma unroll
    for (int idx = 0; idx < 16; ++idx) {
      mma_one(first, 0, idx);
      CANZ_FENCE();
      if (idx < 8) {
        frag_one(cur, 1, 1, idx);  // second half-step's operands, land under the next 8 MFMAs
        CANZ_FENCE();
      }
      if (decltype(fetch_q)::value && (idx & 3) == 2) {
        fetch_one(prv, kt + 3, 4 + (idx >> 2));  // Q panel of step kt+3
        CANZ_FENCE();
      }
    }
    // own share of step kt+1 has landed; this wavefront's reads of `cur` are complete.
    // simm16 = vmcnt[3:0] | expcnt 7 << 4 | lgkmcnt << 8 | vmcnt[5:4] << 14
    __builtin_amdgcn_s_waitcnt(decltype(wait_code)::value);
    __builtin_amdgcn_s_barrier();
    CANZ_FENCE();
#pragma unroll
    for (int idx = 0; idx < 16; ++idx) {
      mma_one(No{}, 1, idx);
      CANZ_FENCE();
      if (decltype(read_next)::value && idx < 8) {
        frag_one(nxt, 0, 0, idx);  // first operands of step kt+1
        CANZ_FENCE();
      }
      if (decltype(fetch_p)::value && (idx & 3) == 2) {
        fetch_one(cur, kt + 4, idx >> 2);  // P panel of step kt+4
        CANZ_FENCE();
      }
    }
  };
  using Vm16 = std::integral_constant<int, 0x4070>;  // vmcnt(16) lgkmcnt(0)
  using Vm8 = std::integral_constant<int, 0x0078>;   // vmcnt(8)  lgkmcnt(0)
  using Vm0 = std::integral_constant<int, 0x0070>;   // vmcnt(0)  lgkmcnt(0)

  // steps 0..2 whole and the P panel of step 3; its Q panel is the first request of step 0
  fetch(st0, 0);
  fetch(st1, 1);
  fetch(st2, 2);
#pragma unroll
  for (int idx = 0; idx < 4; ++idx) fetch_one(st3, 3, idx);
  __syncthreads();
#pragma unroll
  for (int idx = 0; idx < 8; ++idx) frag_one(st0, 0, 0, idx);
  // first four steps (the very first one starts the accumulators), whole groups of four,
  // last four steps; nk is a multiple of 4 and at least 8
  k_step(Yes{}, Yes{}, Yes{}, Yes{}, Vm16{}, st0, st1, st3, 0);
  k_step(No{}, Yes{}, Yes{}, Yes{}, Vm16{}, st1, st2, st0, 1);
  k_step(No{}, Yes{}, Yes{}, Yes{}, Vm16{}, st2, st3, st1, 2);
  k_step(No{}, Yes{}, Yes{}, Yes{}, Vm16{}, st3, st0, st2, 3);
  for (int kt = 4; kt < nk - 4; kt += 4) {
    k_step(No{}, Yes{}, Yes{}, Yes{}, Vm16{}, st0, st1, st3, kt);
    k_step(No{}, Yes{}, Yes{}, Yes{}, Vm16{}, st1, st2, st0, kt + 1);
    k_step(No{}, Yes{}, Yes{}, Yes{}, Vm16{}, st2, st3, st1, kt + 2);
    k_step(No{}, Yes{}, Yes{}, Yes{}, Vm16{}, st3, st0, st2, kt + 3);
  }
  {
    // the tail: Q(nk-1) is the last request; then the queue drains: 16, 8, 0 younger loads
    const int kt = nk - 4;
    k_step(No{}, Yes{}, No{}, Yes{}, Vm16{}, st0, st1, st3, kt);
    k_step(No{}, No{}, No{}, Yes{}, Vm8{}, st1, st2, st0, kt + 1);
    k_step(No{}, No{}, No{}, Yes{}, Vm0{}, st2, st3, st1, kt + 2);
    k_step(No{}, No{}, No{}, No{}, Vm0{}, st3, st0, st2, kt + 3);
  }
  __syncthreads();  // every wavefront is done with the stages; LDS is free for the epilogue
#undef CANZ_FENCE

  if (SPLIT) {
    // k-slice: park the accumulators (register r of thread t at [r][t]: coalesced stores);
    // k_split_finish adds the slices of each tile up and runs its epilogue.
    float* mine = e.partial + static_cast<int64_t>(slot) * (256 * NTHREADS) + t;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[((i * 4 + j) * 16 + r) * NTHREADS] = acc[i][j][r];
        __builtin_amdgcn_sched_barrier(0);
      }
    break;
  }

  {
    __bf16* stage = wave == 0 ? st0 : wave == 1 ? st1 : wave == 2 ? st2 : st3;
    tile_epilogue<EPI>(acc, stage, lane, wm, wn, b, tm, tn, d, e, s, o, epi_apart(EPI) ? vec + 128 * wave : vec);
  }

  // the next tile's loads overwrite every wavefront's staging area: wait for all of them.
  // The global stores issued above keep draining while the next tile is multiplied.
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) only
  __builtin_amdgcn_s_barrier();
  }  // persistent work loop
}

// Finishes the tiles whose k range was split: one block per tile adds the parked slices
// (always in slice order, so the sum does not depend on timing) and runs the epilogue.
template <int EPI>
__global__ __launch_bounds__(NTHREADS) void k_split_finish(GemmDims d, EpiArgs e, Shape s, OutSpec o) {
  __shared__ __attribute__((aligned(1024))) __bf16 stg[4][(BM + BN) * BK];
  __shared__ __attribute__((aligned(16))) float vec[4][128];
  const int tiles_n = static_cast<int>(d.N / BN);
  const int tiles_m = static_cast<int>(d.M / BM);
  const int per_batch = epi_symmetric(EPI) ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  const int l = blockIdx.x;
  int b, tm, tn;
  decode_tile<EPI>(e.full_rounds * e.main_grid + l, tiles_m, tiles_n, per_batch, b, tm, tn);
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const float* first = e.partial + static_cast<int64_t>(l) * e.splits * (256 * NTHREADS) + t;
  f32x16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f32x16 sum;
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[r] = 0.f;
      for (int sl = 0; sl < e.splits; ++sl) {
        const float* p = first + static_cast<int64_t>(sl) * (256 * NTHREADS) + (i * 4 + j) * 16 * NTHREADS;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[r] += p[r * NTHREADS];
      }
      acc[i][j] = sum;
    }
  tile_epilogue<EPI>(acc, stg[wave], lane, wave >> 1, wave & 1, b, tm, tn, d, e, s, o, vec[wave]);
}

// ---------------------------------------------------------------------------------------
// Small-product variant: 128 x 128, 64 x 64 or 256 x 128 tiles, one block per tile, up to three resident blocks per CU.
//
// The persistent 256 x 256 kernel above is built for products with many rounds of long tiles.
// A launch with few tiles (the 0.6B-shaped shares: 260 Gram tiles for 256 CUs) leaves most
// of its last round idle and pays the un-overlapped prologue and epilogue of a tile on every
// short k range.  Here a tile is a quarter of that: four times as many blocks balance over
// the chip, 48 KiB of LDS and 64 accumulator registers per lane let three blocks share a CU, so
// that one block's loads and epilogue run under the others' MFMAs.  The price is twice the
// L2 -> LDS traffic per FLOP, which is why long products stay with the large tile.
// It therefore takes what the large kernel handles badly: launches with few tiles, and the
// left-over tiles behind the last full round of a launch with a short k range (each left-over
// 256 x 256 tile becomes four blocks here).
//
// Same operands (panel layout: the 128 rows of a tile are one contiguous 8 KiB half of a
// panel), same MFMA, same order of accumulation over k, same epilogue arithmetic: an element
// comes out with the same bits from either kernel.  Epilogues store straight from the
// accumulators (4 bytes per lane for the straight image after the lane-pair exchange, 8 bytes
// per lane for the transposed one): there is no LDS to spare for staging with three blocks
// per CU, and the stores of one block drain under the work of the others.  Only the last
// product, whose rows go to the caller's row-major buffers, stages them through the stages
// the k loop has left free.
// Three variants, by how many blocks a launch has (launch_small).  What bounds a block that has its CU to itself is the wait for
// its panels: a k-step of 128 x 128 takes 0.12 us on the matrix cores, 0.15 us from L2 into LDS (110 to 140 KB/us per CU) and
// 0.44 us with two k-steps of loads in flight.  So where there are no three blocks for every CU, the ring is eight stages deep and the
// operands are double-buffered in registers (0.19 us), and where there are fewer than two tiles for every CU, tiles are
// 64 x 64: four times as many blocks, two on a CU.  us a launch, 128 x 128 with three stages -> the variant that now runs:
//   64 x 64, 8 stages     8 x 256^2, k 512: 7.9 -> 5.0;  2 x 512^2, k 4096: 38 -> 22;  a 1024 x 2048 update: 12.8 -> 9.3
//   128 x 128, 8 stages   2048^2, k 4096: 38 -> 29.5;  seven 1024^2 with k 1024 to 3072: 38 -> 33
// Left-over tiles for half of the CUs, and launches of no more, are 256 x 128 where k is long: one per CU, with six stages and three
// quarters of the bytes per FLOP: 128 tiles of 3072 x 1024 with k 18432 385 -> 325, 96 of the Shampoo roots 310 -> 276.
// blocks that share a CU:
constexpr int small_blocks(int sm, int nst) { return nst == 3 ? 3 : sm == 64 ? 2 : 1; }

template <int EPI, int SM, int NST, typename Args>
__global__ __launch_bounds__(NTHREADS, small_blocks(SM, NST)) void k_gemm_nt_bf16_small(Args args, EpiArgs e_launch, Shape s, OutSpec o) {
  static_assert((SM == 128 && NST == 3) || (SM == 256 && NST == 6) || (SM <= 128 && NST == 8), "variants");
  constexpr int SN = SM == 256 ? 128 : SM;
  constexpr int S_STAGE = (SM + SN) * BK;        // elements per stage: the P and the Q part of a panel
  constexpr int RM = BM / SM, RN = BN / SN;      // tiles per 256 rows, columns
  constexpr int TI = SM / 64, TJ = SN / 64;      // 32 x 32 MFMA tiles of a wavefront
  constexpr int LPK = TI + TJ;                   // direct loads of a wavefront per stage
  // one array per stage, as in the large kernel
  __shared__ __attribute__((aligned(1024))) __bf16 sa[S_STAGE];
  __shared__ __attribute__((aligned(1024))) __bf16 sb[S_STAGE];
  __shared__ __attribute__((aligned(1024))) __bf16 sc[S_STAGE];
  __shared__ __attribute__((aligned(1024))) __bf16 sd[NST > 3 ? S_STAGE : 8], se[NST > 3 ? S_STAGE : 8], sf_[NST > 3 ? S_STAGE : 8],
      sg[NST > 6 ? S_STAGE : 8], sh[NST > 6 ? S_STAGE : 8];

  GemmDims d{};
  const __bf16 *P = nullptr, *Q = nullptr;
  EpiArgs e = e_launch;
  // neighbouring tiles on one XCD (blockIdx % 8 selects the XCD): they share panels in its L2
  int logical;
  {
    const int nblocks = gridDim.x, bid = blockIdx.x;
    const int per = nblocks / N_XCD, rem = nblocks % N_XCD;
    const int xcd = bid % N_XCD, q = bid / N_XCD;
    logical = xcd < rem ? xcd * (per + 1) + q : rem * (per + 1) + (xcd - rem) * per + q;
  }
  // A launch of small tiles alone (e.main_grid = 0) numbers those that there are, one block each.  Behind a launch of the
  // large kernel consecutive blocks are the parts of one 256 x 256 tile of its numbering, from tile e.main_grid on; 256 x 128 tiles
  // always are.
  // A product of two symmetric matrices is symmetric only to rounding, and within 128 x 128 elements on the diagonal all of it is
  // computed, here as in the large kernel: 64 x 64 tiles are then numbered as the quarters of 128 x 128 ones.
  const bool behind = e.main_grid > 0;
  constexpr bool QUARTERS = epi_two_factors(EPI) && SM == 64;
  const int parts_m = behind ? RM : QUARTERS ? 2 : 1, parts_n = behind || SM == 256 ? RN : QUARTERS ? 2 : 1;
  const int part = logical % (parts_m * parts_n);
  logical = e.main_grid + logical / (parts_m * parts_n);
  float neg_lr_scale = o.neg_lr_scale;
  int out_dtype = o.out_dtype, first_out = 0;
  if constexpr (Args::multi) {
    int j = 0;
    while (j + 1 < args.n && logical >= args.begin[j + 1]) ++j;
    const auto& pr = args.pr[j];
    d = pr.d;
    P = static_cast<const __bf16*>(pr.p), Q = static_cast<const __bf16*>(pr.q);
    if constexpr (Args::finals) {
      s = pr.s, neg_lr_scale = pr.neg_lr_scale, out_dtype = pr.out_dtype, first_out = pr.first_out;
    } else {
      e.c = pr.c, e.ct = pr.ct, e.sym = pr.sym;
    }
    e.scale = pr.scale;
    logical -= args.begin[j];
  } else {
    d = args.d, P = args.P, Q = args.Q;
  }
  const int tile = parts_m * SM;
  const int tiles_m = static_cast<int>(d.M) / tile, tiles_n = static_cast<int>(d.N) / tile;
  const bool symmetric = epi_symmetric(EPI);
  const int per_batch = symmetric ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  int b, tm, tn;
  decode_tile<EPI>(logical, tiles_m, tiles_n, per_batch, b, tm, tn);
  // in a diagonal tile of a symmetric product what is below the diagonal is the mirror of what is above
  constexpr int LEVEL = QUARTERS ? 1 : 0;   // what lies on the diagonal is counted in tiles of SM << LEVEL
  tm = parts_m * tm + part / parts_n, tn = parts_n * tn + part % parts_n;
  if (SM < 256 && symmetric && tm >> LEVEL > tn >> LEVEL) return;

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  // (of a 256 x 128 tile, which may hold both, in 128 x 128 elements: the rows of a wavefront and the columns of the tile)
  const bool mirrored = symmetric && (SM == 256 ? 2 * tm + wm != tn : tm >> LEVEL != tn >> LEVEL);
  const bool below = SM == 256 && symmetric && 2 * tm + wm > tn;
  const int64_t nkb = d.K / BK;
  const int nk = static_cast<int>(nkb) * (epi_terms(EPI) ? d.nseg : 1);
  // panels per row block (operands that are a part of longer rows: only of the last products and those of several terms)
  const int64_t nkp = epi_terms(EPI) || epi_final(EPI) ? d.ldp / BK : nkb, nkq = epi_terms(EPI) || epi_final(EPI) ? d.ldq / BK : nkb;

  // global -> LDS: the part of a panel is SM / 16 (SN / 16) pieces of 1 KiB; wavefront w copies the pieces w, w + 4, ..
  // lane l the 16 bytes at l * 16
  const __bf16* pl = P + static_cast<int64_t>(b) * d.sp + (static_cast<int64_t>(tm / RM) * nkp) * PANEL_ELEMS +
                     (tm % RM) * (SM * BK) + wave * 512 + lane * 8;
  const __bf16* ql = Q + static_cast<int64_t>(b) * d.sq + (static_cast<int64_t>(tn / RN) * nkq) * PANEL_ELEMS +
                     (tn % RN) * (SN * BK) + wave * 512 + lane * 8;
  TermWalk wp(d.pseg, nkb), wq(d.qseg, nkb);
  constexpr bool KM = epi_k_major(EPI);
  constexpr int G_STEP = KM ? 2 * PANEL_ELEMS : 2048;
  if (KM) {   // as in the large kernel
    const int64_t km_lane = (wave >> 1) * PANEL_ELEMS + (wave & 1) * 512 + lane * 8;
    pl = P + static_cast<int64_t>(b) * d.sp + tm * (SM / 32) * PANEL_ELEMS + km_lane;
    ql = Q + static_cast<int64_t>(b) * d.sq + tn * (SN / 32) * PANEL_ELEMS + km_lane;
  }
  auto fetch_one = [&](__bf16* st, int kt, int idx) {   // idx 0 .. TI - 1: pieces of P, then those of Q
    const int kc = kt < nk ? kt : nk - 1;   // past the end: a harmless re-read
    const int64_t off = KM ? k_major_off(kc, d.M >> 5) : static_cast<int64_t>(kc) * PANEL_ELEMS;
    if (idx < TI) {
      const int64_t po = epi_terms(EPI) ? wp.off : off;
      __builtin_amdgcn_global_load_lds(CANZ_GLB(pl + po + idx * G_STEP), CANZ_LDS(st + wave * 512 + idx * 2048), 16, 0, 0);
      if (epi_terms(EPI) && idx == TI - 1) wp.next();
    } else {
      const int64_t qo = epi_terms(EPI) ? wq.off : off;
      __builtin_amdgcn_global_load_lds(CANZ_GLB(ql + qo + (idx - TI) * G_STEP), CANZ_LDS(st + SM * BK + wave * 512 + (idx - TI) * 2048), 16, 0, 0);
      if (epi_terms(EPI) && idx == LPK - 1) wq.next();
    }
  };
  auto fetch = [&](__bf16* st, int kt) {
#pragma unroll
    for (int idx = 0; idx < LPK; ++idx) fetch_one(st, kt, idx);
  };

  f32x16 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int frag_row = lane & 31, frag_kg = lane >> 5;
  constexpr int SETS = NST == 3 ? 1 : 2;
  bf16x8 fa[2 * SETS][TI], fb[2 * SETS][TJ];   // operands of the two half-steps, of this step and of the next
  const int km0 = k_major_lane(lane, 0), km1 = k_major_lane(lane, 1);
  auto frag = [&](const __bf16* st, int kk, int set, int idx) {   // idx 0 .. TI - 1: rows of P, then those of Q
    const int chunk = kk * 2 + frag_kg, to = 2 * set + kk;
    if (KM && idx < TI)
      fa[to][idx] = k_major(st + (wm * TI + idx) * 1024 + kk * 512, km0, km1);
    else if (KM)
      fb[to][idx - TI] = k_major(st + SM * BK + (wn * TJ + idx - TI) * 1024 + kk * 512, km0, km1);
    else if (idx < TI)
      fa[to][idx] = *reinterpret_cast<const bf16x8*>(st + swz((wm * TI + idx) * 32 + frag_row, chunk));
    else
      fb[to][idx - TI] = *reinterpret_cast<const bf16x8*>(st + SM * BK + swz((wn * TJ + idx - TI) * 32 + frag_row, chunk));
  };
  auto mma = [&](int kk, int set, int idx) {
    const int i = idx / TJ, j = idx % TJ;
    acc[i][j] = mfma<EPI>(fa[2 * set + kk][i], fb[2 * set + kk][j], acc[i][j]);
  };
  if constexpr (NST == 3) {
    auto multiply = [&](const __bf16* st) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int idx = 0; idx < LPK; ++idx) frag(st, kk, 0, idx);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int idx = 0; idx < TI * TJ; ++idx) mma(kk, 0, idx);
    };
    // One k-step on stage `cur`: the 4 loads of the following step may stay in flight; after the
    // barrier every wavefront has finished the step before, whose stage `nxt2` then receives step kt + 2.
    auto k_step = [&](const __bf16* cur, __bf16* nxt2, int kt) {
      __builtin_amdgcn_s_waitcnt(0x0074);  // vmcnt(4) lgkmcnt(0)
      __builtin_amdgcn_s_barrier();
      fetch(nxt2, kt + 2);
      multiply(cur);
    };
    fetch(sa, 0);
    fetch(sb, 1);
    int kt = 0;
    for (; kt + 3 <= nk; kt += 3) {
      k_step(sa, sc, kt);
      k_step(sb, sa, kt + 1);
      k_step(sc, sb, kt + 2);
    }
    if (kt < nk) k_step(sa, sc, kt), ++kt;
    if (kt < nk) k_step(sb, sa, kt), ++kt;
    __builtin_amdgcn_s_waitcnt(0x0070);  // the re-reads past the end have landed before the block leaves
  } else {
    // The operands are double-buffered in registers, those of a step read under the MFMAs of the one before.  At the start of
    // step kt every wavefront has read all of `cur`, which then receives step kt + NST, and
    // step kt + 1 has landed in `nxt`, `younger` later ones still in flight.
    using Yes = std::true_type;
    using No = std::false_type;
    constexpr int NM = 2 * TI * TJ, NF = 2 * (TI + TJ);   // MFMAs and operands of a step
#define CANZ_FENCE() __builtin_amdgcn_sched_barrier(0)
    auto k_step = [&](auto fetches, auto younger, auto parity, __bf16* cur, const __bf16* nxt, int kt) {
      constexpr int left = decltype(younger)::value, set = decltype(parity)::value;   // left -1: the last step
      constexpr int vm = left < 0 ? 0 : left * LPK;
      __builtin_amdgcn_s_waitcnt((vm & 15) | 0x70 | (vm >> 4) << 14);  // vmcnt(vm) lgkmcnt(0)
      if (left >= 0) __builtin_amdgcn_s_barrier();
      CANZ_FENCE();
#pragma unroll
      for (int idx = 0; idx < NM; ++idx) {
        mma(idx / (NM / 2), set, idx % (NM / 2));
        CANZ_FENCE();
        if (left >= 0)
#pragma unroll
          for (int x = idx * NF / NM; x < (idx + 1) * NF / NM; ++x) frag(nxt, x / (NF / 2), set ^ 1, x % (NF / 2));
        CANZ_FENCE();
        if (decltype(fetches)::value)
#pragma unroll
          for (int x = idx * LPK / NM; x < (idx + 1) * LPK / NM; ++x) fetch_one(cur, kt + NST, x);
        CANZ_FENCE();
      }
    };
#undef CANZ_FENCE
#define CANZ_INT(n) std::integral_constant<int, n> {}
    fetch(sa, 0), fetch(sb, 1), fetch(sc, 2), fetch(sd, 3), fetch(se, 4), fetch(sf_, 5);
    if constexpr (NST == 8) fetch(sg, 6), fetch(sh, 7);
    constexpr int vm0 = (NST - 1) * LPK;
    __builtin_amdgcn_s_waitcnt((vm0 & 15) | 0x70 | (vm0 >> 4) << 14);
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int x = 0; x < NF; ++x) frag(sa, x / (NF / 2), 0, x % (NF / 2));
    int kt = 0;
    if constexpr (NST == 8) {   // nk is a multiple of 8; the last eight steps request nothing and the queue drains
      for (; kt + 8 < nk; kt += 8) {
        k_step(Yes{}, CANZ_INT(6), CANZ_INT(0), sa, sb, kt);
        k_step(Yes{}, CANZ_INT(6), CANZ_INT(1), sb, sc, kt + 1);
        k_step(Yes{}, CANZ_INT(6), CANZ_INT(0), sc, sd, kt + 2);
        k_step(Yes{}, CANZ_INT(6), CANZ_INT(1), sd, se, kt + 3);
        k_step(Yes{}, CANZ_INT(6), CANZ_INT(0), se, sf_, kt + 4);
        k_step(Yes{}, CANZ_INT(6), CANZ_INT(1), sf_, sg, kt + 5);
        k_step(Yes{}, CANZ_INT(6), CANZ_INT(0), sg, sh, kt + 6);
        k_step(Yes{}, CANZ_INT(6), CANZ_INT(1), sh, sa, kt + 7);
      }
      k_step(No{}, CANZ_INT(6), CANZ_INT(0), sa, sb, kt);
      k_step(No{}, CANZ_INT(5), CANZ_INT(1), sb, sc, kt);
      k_step(No{}, CANZ_INT(4), CANZ_INT(0), sc, sd, kt);
      k_step(No{}, CANZ_INT(3), CANZ_INT(1), sd, se, kt);
      k_step(No{}, CANZ_INT(2), CANZ_INT(0), se, sf_, kt);
      k_step(No{}, CANZ_INT(1), CANZ_INT(1), sf_, sg, kt);
      k_step(No{}, CANZ_INT(0), CANZ_INT(0), sg, sh, kt);
      k_step(No{}, CANZ_INT(-1), CANZ_INT(1), sh, sa, kt);
    } else {
      for (; kt + 6 <= nk; kt += 6) {
        k_step(Yes{}, CANZ_INT(4), CANZ_INT(0), sa, sb, kt);
        k_step(Yes{}, CANZ_INT(4), CANZ_INT(1), sb, sc, kt + 1);
        k_step(Yes{}, CANZ_INT(4), CANZ_INT(0), sc, sd, kt + 2);
        k_step(Yes{}, CANZ_INT(4), CANZ_INT(1), sd, se, kt + 3);
        k_step(Yes{}, CANZ_INT(4), CANZ_INT(0), se, sf_, kt + 4);
        k_step(Yes{}, CANZ_INT(4), CANZ_INT(1), sf_, sa, kt + 5);
      }
      if (kt < nk) k_step(Yes{}, CANZ_INT(4), CANZ_INT(0), sa, sb, kt), ++kt;
      if (kt < nk) k_step(Yes{}, CANZ_INT(4), CANZ_INT(1), sb, sc, kt), ++kt;
      if (kt < nk) k_step(Yes{}, CANZ_INT(4), CANZ_INT(0), sc, sd, kt), ++kt;
      if (kt < nk) k_step(Yes{}, CANZ_INT(4), CANZ_INT(1), sd, se, kt), ++kt;
      if (kt < nk) k_step(Yes{}, CANZ_INT(4), CANZ_INT(0), se, sf_, kt), ++kt;
      __builtin_amdgcn_s_waitcnt(0x0070);  // the re-reads past the end have landed
    }
#undef CANZ_INT
  }

  // ---- epilogue.  Accumulator register r of lane l in MFMA tile (i, j): row 32 i + 8 (r / 4) + 4 (l / 32) + (r % 4),
  //      column 32 j + (l % 32) of the wavefront's part, a quarter of the tile.
  const int lj = lane & 31, lh = lane >> 5;
  const int row_w = tm * SM + wm * 32 * TI, col_w = tn * SN + wn * 32 * TJ;
  // Where the elements of 32 x 32 tile (i, j) of the wavefront's part lie in a panel image: a part that is the same for
  // all lanes, a lane's own offset (two for the straight image, by the parity of the group of 8 rows; four for the
  // transposed one, by group) and a constant.
  auto transposed_at = [&](int i, int j) {
    return (static_cast<int64_t>(col_w >> 8) * (d.M >> 5) + ((row_w + 32 * i) >> 5)) * PANEL_ELEMS + ((col_w & 255) + 32 * j) * PANEL_K;
  };
  int s_lane[2], t_lane[4];
#pragma unroll
  for (int g1 = 0; g1 < 2; ++g1)
    s_lane[g1] = (4 * lh + (lane & 1)) * PANEL_K + ((((lj >> 3) ^ (2 * g1 + lh)) & 3) << 3) + (lj & 6);
#pragma unroll
  for (int g = 0; g < 4; ++g) t_lane[g] = lj * PANEL_K + ((g ^ ((lj >> 2) & 3)) << 3) + 4 * lh;
  if constexpr (EPI == EPI_POLY) {
    // A(i, j) is read as A(j, i) (symmetric bit for bit): the lane's four consecutive rows are
    // four consecutive k of row j, one 8-byte load
    const __bf16* A = static_cast<const __bf16*>(e.sym.aux) + static_cast<int64_t>(b) * d.M * d.N;
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const int col = col_w + 32 * j + lj;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int row0 = row_w + 32 * i + 8 * g + 4 * lh;
          const bf16x4 av = *reinterpret_cast<const bf16x4*>(A + panel_chunk_off(col, row0 & ~7, d.M) + (row0 & 7));
#pragma unroll
          for (int q = 0; q < 4; ++q)
            acc[i][j][4 * g + q] = poly_value(static_cast<float>(av[q]), acc[i][j][4 * g + q], e.ca, e.cb, e.cc, row0 + q == col);
        }
      }
  } else if constexpr (epi_apart(EPI) || EPI == EPI_GRAM_APART) {
    // as in the large kernel
    constexpr bool UPD = EPI == EPI_UPDATE_APART;
    typedef typename ImageIn<EPI>::vec4 vec4;
    const float* const xv = epi_apart(EPI) ? e.sym.x + static_cast<int64_t>(b) * d.M : nullptr;
    const float* const yv = epi_f16_in(EPI) ? e.sym.y + static_cast<int64_t>(b) * d.M : nullptr;
    const float f = UPD ? 1.f : EPI == EPI_GRAM_APART && e.scale ? e.scale[b] * UNIT_A : apart_factor<EPI>(e);
    if constexpr (!epi_apart(EPI)) {
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] *= f;
    } else if (const __bf16* const m1 = static_cast<const __bf16*>(e.sym.aux) + static_cast<int64_t>(b) * d.M * d.N; m1 != nullptr) {
      // always: keeps this apart from the k loop's block, see the large kernel
      const __bf16* const m3 = static_cast<const __bf16*>(e.sym.aux2) + static_cast<int64_t>(b) * d.M * d.N;
      const float sc1 = UPD && e.scale ? e.scale[b] : 1.f;
      // all loads of a 32 x 32 tile at once: a few memory latencies for the whole epilogue, within the registers that
      // three blocks per CU leave
#pragma unroll
      for (int i = 0; i < TI; ++i) {
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          asm volatile("" ::: "memory");   // or the compiler brings the loads of all four tiles together and spills
          vec4 v1[4], v3[4];
          f32x4 rw[4];
          const float cw = epi_f16_in(EPI) ? yv[col_w + 32 * j + lj] : 0.f;
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int64_t at = transposed_at(i, j) + t_lane[g];
            rw[g] = *reinterpret_cast<const f32x4*>(xv + row_w + 32 * i + 8 * g + 4 * lh);
            v1[g] = *reinterpret_cast<const vec4*>(m1 + at);
            if constexpr (epi_mul(EPI)) v3[g] = *reinterpret_cast<const vec4*>(m3 + at);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              float v = UPD ? acc[i][j][4 * g + q] : acc[i][j][4 * g + q] * f;
              v = __builtin_fmaf(apart_weight<EPI>(e, rw[g][q], cw, false), static_cast<float>(v1[g][q]), v);
              if constexpr (epi_mul(EPI)) v = __builtin_fmaf(apart_weight<EPI>(e, 0.f, cw, true), static_cast<float>(v3[g][q]), v);
              acc[i][j][4 * g + q] = UPD ? v * sc1 : v;
            }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if (!UPD && tm == tn && wm == wn) {
      float* dv = EPI == EPI_MUL_Q2 ? nullptr : e.sym.diag + static_cast<int64_t>(b) * d.M;
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        const int col = col_w + 32 * i + lj;
        const float dx = xv ? xv[col] : 0.f, dy = yv ? yv[col] : 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (row_w + 32 * i + 4 * lh + 8 * (r >> 2) + (r & 3) == col) {
            const float v = apart_diagonal<EPI>(acc[i][i][r], dx, dy, e);
            if (EPI != EPI_MUL_Q2) dv[col] = v;
            acc[i][i][r] = EPI == EPI_MUL_Q2 ? v * e.sym.unit : 0.f;
          }
      }
    }
    if constexpr (EPI == EPI_MUL_Q || EPI == EPI_MUL_Q2) {
      const float inv = 1.f / e.sym.unit;
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] *= inv;
    }
    if constexpr (epi_f16_out(EPI)) {
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) asm volatile("" : "+v"(acc[i][j]));
    }
  } else if (e.scale) {
    const float sc1 = e.scale[b];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] *= sc1;
  }
  if constexpr (EPI == EPI_B3 || EPI == EPI_B3_SYM || EPI == EPI_MUL_Q2) {
    // as in the large kernel, straight from the accumulators
    constexpr bool SYM = EPI != EPI_B3;
    constexpr int NT = EPI == EPI_MUL_Q2 ? 2 : 3;
    const unsigned pair_sel = (lane & 1) ? 0x03020706u : 0x05040100u;
    const int64_t nkb = d.N >> 5, elems = NT * d.M * d.N;
    __bf16* const C = static_cast<__bf16*>(e.c) + static_cast<int64_t>(b) * elems;
    __bf16* const T = EPI == EPI_B3_SYM && e.ct ? static_cast<__bf16*>(e.ct) + static_cast<int64_t>(b) * elems : nullptr;
    if (below) return;
    const bool diagonal = SYM && col_w >= row_w && col_w < row_w + 32 * TI;   // the part holds the diagonal elements of its columns
    float dv[TJ];
    if (T && diagonal) {
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int i = 0; i < TI; ++i)
          if (row_w + 32 * i == col_w + 32 * j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (8 * (r >> 2) + (r & 3) + 4 * lh == lj) dv[j] = acc[i][j][r];
    }
#pragma unroll 1
    for (int term = 0; term < NT; ++term)
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          const int64_t at = ((row_w >> 8) * NT * nkb + term * nkb + ((col_w + 32 * j) >> 5)) * PANEL_ELEMS + ((row_w & 255) + 32 * i) * PANEL_K;
          const int64_t tt = ((col_w >> 8) * NT * nkb + term * nkb + ((row_w + 32 * i) >> 5)) * PANEL_ELEMS + ((col_w & 255) + 32 * j) * PANEL_K;
          unsigned mine[8];
#pragma unroll
          for (int rp = 0; rp < 8; ++rp) {
            bf16x2 own;
            own[0] = static_cast<__bf16>(acc[i][j][2 * rp]);
            own[1] = static_cast<__bf16>(acc[i][j][2 * rp + 1]);
            acc[i][j][2 * rp] -= static_cast<float>(own[0]);
            acc[i][j][2 * rp + 1] -= static_cast<float>(own[1]);
            mine[rp] = __builtin_bit_cast(unsigned, own);
          }
          auto put = [&](__bf16* to) {
#pragma unroll
            for (int rp = 0; rp < 8; ++rp)
              *reinterpret_cast<unsigned*>(to + at + s_lane[(rp >> 1) & 1] + (8 * (rp >> 1) + 2 * (rp & 1)) * PANEL_K) =
                  __builtin_amdgcn_perm(lane_xor1(mine[rp]), mine[rp], pair_sel);
            if (mirrored)
#pragma unroll
              for (int g = 0; g < 4; ++g) *reinterpret_cast<u32x2*>(to + tt + t_lane[g]) = u32x2{mine[2 * g], mine[2 * g + 1]};
          };
          put(C);
          if (T) {
#pragma unroll
            for (int rp = 0; rp < 8; ++rp) mine[rp] = minus_quarter(mine[rp]);
            put(T);
          }
        }
    if (T && diagonal && ((lj >> 2) & 1) == lh) {
      __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0): the images are written, these elements go over theirs
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const int64_t at = col_w + 32 * j + lj;
        put_three_terms(T + panel_chunk_off(at, at & ~7, 3 * d.N) + (at & 7), nkb * PANEL_ELEMS, 1.25f - 0.25f * dv[j]);
      }
    }
    return;
  }

  if (epi_final(EPI)) {
    // The stages are free once every wavefront has left the k loop: each wavefront turns its part
    // through half a stage of LDS, 32 rows at a time, into rows of fp32 and updates the
    // caller's buffer with 16-byte accesses (4 columns per lane, LPR lanes per row; at rows whose length is no multiple of 4
    // they are aligned to an element only, and the last columns go one by one).  All old values of 32 rows are requested
    // at once, from clamped addresses: a predicate or a switch of the type at each load would wait for it there and make the
    // epilogue a chain of 16 memory latencies.
    constexpr int W = 32 * TJ, LPR = W / 4, RPP = 64 / LPR, NX = 32 / RPP;
    const int ld = static_cast<int>(o.out_mode == CANZ_OUT_DELTA ? s.wfrag : s.cols);
    __syncthreads();
    float* sf = reinterpret_cast<float*>((wave < 2 ? sa : sb) + (wave & 1) * (S_STAGE / 2));
    const int rows = static_cast<int>(s.rows), cols = static_cast<int>(s.cols);
    const int col = col_w + (lane % LPR) * 4;
    if (row_w >= rows || col_w >= cols || below) return;
    const bool col_ok = col + 4 <= cols;             // all four columns
    const int n_tail = col_ok ? 0 : max(cols - col, 0);
    const bool all_rows = row_w + 32 * TI <= rows;   // uniform
    auto run = [&](auto mode_tag, auto dtype_tag) {
      constexpr bool PARAM = decltype(mode_tag)::value == CANZ_OUT_PARAM, F32 = decltype(dtype_tag)::value == CANZ_DT_F32;
      constexpr int ESZ = F32 ? 4 : 2;
      typedef typename std::conditional<F32, f32x4_any, bf16x4_any>::type vec;
      int c_in = col < cols ? col : 0;
      char* base = static_cast<char*>(o.out.p[first_out + (PARAM ? b : b * s.tp)]);
      if (!PARAM && s.tp > 1) {
        const int f = c_in / ld;
        c_in -= f * ld;
        base = static_cast<char*>(o.out.p[first_out + b * s.tp + f]);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the pointer is there, or every store below would wait for the one before
      }
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        const int row0 = row_w + 32 * i + lane / LPR;
        vec res[NX];   // first the old values
        if (PARAM && col_ok)
#pragma unroll
          for (int x = 0; x < NX; ++x)
            res[x] = *reinterpret_cast<const vec*>(base + (static_cast<int64_t>(min(row0 + RPP * x, rows - 1)) * ld + c_in) * ESZ);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) sf[(8 * (r >> 2) + 4 * lh + (r & 3)) * W + 32 * j + lj] = acc[i][j][r];
        __builtin_amdgcn_sched_barrier(0);
        if (col_ok) {
#pragma unroll
          for (int x = 0; x < NX; ++x) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(sf + (RPP * x + lane / LPR) * W + (lane % LPR) * 4);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float val = PARAM ? apply_update(static_cast<float>(res[x][q]), o.decay, neg_lr_scale, v[q]) : neg_lr_scale * v[q];
              if constexpr (F32) res[x][q] = val; else res[x][q] = static_cast<__bf16>(val);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
          char* const to = base + (static_cast<int64_t>(row0) * ld + c_in) * ESZ;
          const int64_t pitch = static_cast<int64_t>(RPP) * ld * ESZ;
          if (all_rows) {
#pragma unroll
            for (int x = 0; x < NX; ++x) *reinterpret_cast<vec*>(to + x * pitch) = res[x];
          } else {
#pragma unroll
            for (int x = 0; x < NX; ++x)
              if (row0 + RPP * x < rows) *reinterpret_cast<vec*>(to + x * pitch) = res[x];
          }
        } else {
          for (int q = 0; q < n_tail; ++q)
#pragma unroll 1
            for (int x = 0; x < NX; ++x) {
              const int row = row0 + RPP * x;
              if (row >= rows) break;
              typedef typename std::conditional<F32, float, __bf16>::type elem;
              elem* const at = reinterpret_cast<elem*>(base) + static_cast<int64_t>(row) * ld + c_in + q;
              const float v = sf[(RPP * x + lane / LPR) * W + (lane % LPR) * 4 + q];
              *at = static_cast<elem>(PARAM ? apply_update(static_cast<float>(*at), o.decay, neg_lr_scale, v) : neg_lr_scale * v);
            }
        }
        // the second half is staged in the same area (this wavefront's own: no barrier needed)
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      }
    };
    using P_ = std::integral_constant<int, CANZ_OUT_PARAM>;
    using D_ = std::integral_constant<int, CANZ_OUT_DELTA>;
    using F_ = std::integral_constant<int, CANZ_DT_F32>;
    using B_ = std::integral_constant<int, CANZ_DT_BF16>;
    if (o.out_mode == CANZ_OUT_PARAM) {
      if (out_dtype == CANZ_DT_F32) run(P_{}, F_{}); else run(P_{}, B_{});
    } else {
      if (out_dtype == CANZ_DT_F32) run(D_{}, F_{}); else run(D_{}, B_{});
    }
    return;
  }

  const int64_t image = static_cast<int64_t>(b) * d.M * d.N;
  // straight image: (row i, k = j).  Neighbouring lanes exchange their packed pairs so that each
  // lane holds two consecutive columns of one row: the even lane of row 2 rp, the odd lane of row 2 rp + 1.
  const unsigned pair_sel = (lane & 1) ? 0x03020706u : 0x05040100u;
  if (symmetric || e.c != nullptr) {   // (an update may be asked for the transposed image alone)
    __bf16* const C = static_cast<__bf16*>(e.c) + image;
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int col = col_w + 32 * j + (lj & ~1);
#pragma unroll
      for (int rp = 0; rp < 8; ++rp) {
        const unsigned mine = image_pair<EPI>(acc[i][j][2 * rp], acc[i][j][2 * rp + 1]);
        const unsigned theirs = lane_xor1(mine);
        const unsigned pk = __builtin_amdgcn_perm(theirs, mine, pair_sel);
        const int row = row_w + 32 * i + 8 * (rp >> 1) + 4 * lh + 2 * (rp & 1) + (lane & 1);
        *reinterpret_cast<unsigned*>(C + panel_chunk_off(row, col & ~7, d.N) + (col & 7)) = pk;
      }
    }
  }
  // transposed image: (row j, k = i) of CT (UPDATE) or of the mirror tile of C (symmetric products)
  if (!symmetric || mirrored) {
    __bf16* const CT = static_cast<__bf16*>(symmetric ? e.c : e.ct) + image;
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const int col = col_w + 32 * j + lj;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int row0 = row_w + 32 * i + 8 * g + 4 * lh;
          const u32x2 pk = {image_pair<EPI>(acc[i][j][4 * g], acc[i][j][4 * g + 1]), image_pair<EPI>(acc[i][j][4 * g + 2], acc[i][j][4 * g + 3])};
          *reinterpret_cast<u32x2*>(CT + panel_chunk_off(col, row0 & ~7, d.M) + (row0 & 7)) = pk;
        }
      }
  }
}

// Compute units of the current device.  The answer is cached per device in a plain array: the
// first calls from several threads may each query the attribute and store the same value
// (a benign race on an int that only ever takes one non-zero value).
int cu_count() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// How a launch is divided between the two kernels.  Launches of at most half a round run on small tiles, unless a k-split pays
// (split_pays).  Of the others long products (k above SMALL_MAX_K; the small tile moves twice the bytes per FLOP) stay with the large
// kernel and its k-split.  Otherwise the large kernel runs the full rounds of one tile per CU, and the left-over tiles go to the
// small kernel when they would leave at least half of the chip idle for a whole tile time.
constexpr int64_t SMALL_MAX_K = 4096;
// ... except the products of m x m matrices of merged steps, whose left-over tiles gain up to here (4 x 5120^2, 840 tiles on 256
// CUs)
constexpr int64_t SMALL_MAX_K_MSPACE = 8192;
constexpr int64_t SMALL_ALL_MAX_K = 2048;   // polynomial products up to this k and under two rounds: small tiles only

template <int EPI>
int64_t tile_count(const GemmDims& d, int tile = BM) {
  const int64_t tm = d.M / tile, tn = d.N / tile;
  return (epi_symmetric(EPI) ? tm * (tm + 1) / 2 : tm * tn) * d.nb;
}

// the length of k that a tile walks: of all segments, where there are several
template <int EPI>
int64_t k_length(const GemmDims& d) {
  return epi_terms(EPI) ? d.K * d.nseg : d.K;
}

// number of tiles [0, whole) for the large kernel; the rest, if any, for the small one
template <int EPI>
int64_t large_share(int64_t tiles, int64_t cus, int64_t longest_k, int out_mode = CANZ_OUT_DELTA) {
  const int64_t left = tiles % cus;
  if (2 * tiles <= cus) return 0;   // no round to fill
  constexpr bool msquare = EPI == EPI_POLY || epi_f16_in(EPI);
  if (!epi_terms(EPI) && longest_k > (epi_f16_in(EPI) ? SMALL_MAX_K_MSPACE : SMALL_MAX_K)) return tiles;
  // a polynomial product (k = m, the shortest k range of the step) of less than two rounds runs faster on small
  // tiles throughout: 59.6 -> 52.4 us on 26 matrices of 1024 x 1024; the same rule costs the Gram product 7 %
  if (msquare && tiles < 2 * cus && longest_k <= SMALL_ALL_MAX_K) return 0;
  // A last product with a short k waits for memory, which the blocks of small tiles that share a CU hide from each other, up to a
  // few rounds; longer for parameters, whose old values are waited for, than for Delta W.  us a step of n x 2048x1024 (32 n tiles, k 1024) and of
  // n x 2047x1023, large tiles for the full rounds -> small ones:
  //   fp32 parameters   512 tiles 877 -> 866, 704 1156 -> 1141, 832 1383 -> 1363, 896 1492 -> 1474, 960 1572 -> 1558, 992 1597 -> 1593, 1024 1621 -> 1621,
  //                     1536 2417 -> 2427;  bf16 ones   640 1047 -> 1032, 832 1346 -> 1333, 992 1504 -> 1499, 1024 1527 -> 1528, 1280 1935 -> 1940;
  //                     odd rows   640 1194 -> 1104, 960 1785 -> 1632
  //   fp32 Delta W      512 867 -> 858, 704 1138 -> 1127, 768 and 832 within 0.8 % either way (two machines), 864 1357 -> 1366, 992 1526 -> 1550;
  //                     odd rows   640 1150 -> 1126, 832 1442 -> 1408
  if (EPI == EPI_FINAL && longest_k <= 1024 && (out_mode == CANZ_OUT_PARAM ? tiles < 4 * cus : 4 * tiles <= 13 * cus)) return 0;
  if (left == 0 || 2 * left > cus) return tiles;
  return tiles - left;
}

// The numbers of a launch of SM x SM tiles alone: how many, and where each problem's begin.
template <int EPI, int SM>
int64_t small_tiles(const GemmDims& d) {
  return epi_two_factors(EPI) && SM == 64 ? 4 * tile_count<EPI>(d, 128) : tile_count<EPI>(d, SM);
}
// Left-over tiles cut into k-slices (each at least 8 k-steps long) so that they occupy as many blocks as fit: how many slices a tile, or 1.
// Splitting costs two more launches plus parking and re-reading the accumulators, about 0.2 ms all told; a k-step takes about 0.65 us.
// Split only where the part of a tile time it saves, (1 - 1/sp) * k-steps, is clearly longer than that.
template <int EPI>
int64_t k_slices(int64_t left, int64_t steps, int64_t cus, const SplitWs& w) {
  if (left == 0 || !w.partial || epi_terms(EPI)) return 1;
  const int64_t sp = std::max<int64_t>(1, std::min<int64_t>({std::min<int64_t>(cus, w.max_blocks) / left, steps / 8, 8}));
  return sp > 1 && steps * (sp - 1) / sp >= 400 ? sp : 1;
}
// Whether a launch of at most half a round, whose tiles can be split, is faster so than on small tiles (launch_small): from a length of k on
// that depends on how many of those share a CU.  us of a Gram product, small tiles / split:
//   64 x 64, a CU each (0.08 to 0.11 us a k-step)     1 x 256, k 131072: 313 / 366, 196352: 474 / 482, 262144: 652 / 617;  1 x 1024, k 196608: 586 / 551
//   64 x 64, or 128 x 128 with eight stages (0.17 to 0.21)   1536, k 32768: 181 / 216, 45056: 251 / 234;  2048, k 32768: 197 / 231, 45056: 272 / 261,
//                                                            65536: 386 / 324;  2560, k 45056: 297 / 303, 65536: 432 / 410
//   128 x 128 with three stages (0.40 to 0.48)        3072, k 16384: 205 / 266, 24576: 308 / 235;  3840, k 16384: 237 / 268, 25600: 376 / 321
// The last ones cross where k_slices begins to split them.
template <int EPI>
bool split_pays(const GemmDims& d, int64_t steps, int64_t cus) {
  if (small_tiles<EPI, 64>(d) <= cus) return steps >= 6144;
  const bool three_stages = small_tiles<EPI, 64>(d) > 2 * cus && small_tiles<EPI, 128>(d) > cus;
  return three_stages || steps >= 1408;
}

template <int EPI, int SM>
int64_t renumber(OneProblem& args) {
  return small_tiles<EPI, SM>(args.d);
}
template <int EPI, int SM, typename Args>
int64_t renumber(Args& args) {
  int64_t tiles = 0;
  // in the numbers that the kernel compares: of 128 x 128 tiles where 64 x 64 ones are their quarters
  constexpr int per = epi_two_factors(EPI) && SM == 64 ? 4 : 1;
  for (int j = 0; j < args.n; ++j) args.begin[j] = static_cast<int>(tiles / per), tiles += small_tiles<EPI, SM>(args.pr[j].d);
  for (int j = args.n; j < static_cast<int>(sizeof(args.begin) / sizeof(args.begin[0])); ++j) args.begin[j] = static_cast<int>(tiles / per);
  return tiles;
}
template <int EPI, int SM, int NST, typename Args>
void launch_small_as(Args args, EpiArgs e, int64_t first, int64_t tiles, const Shape& s, const OutSpec& o, hipStream_t st) {
  constexpr int R = BM / SM;
  const int64_t blocks = SM == 256 ? 2 * (tiles - first) : first > 0 ? R * R * (tiles - first) : renumber<EPI, SM>(args);
  e.main_grid = static_cast<int>(first);
  hipLaunchKernelGGL((k_gemm_nt_bf16_small<EPI, SM, NST, Args>), dim3(static_cast<unsigned>(blocks)), dim3(NTHREADS), 0, st, args, e, s, o);
}
// (the epilogues of matrices with their diagonal apart are written for square parts)
constexpr bool epi_256x128(int epi) { return epi_terms(epi) || epi == EPI_UPDATE || epi_final(epi); }
// Tiles [first, tiles) of the large kernel's numbering on the small one (k_gemm_nt_bf16_small says what the variants are for).  64 x 64
// up to two blocks per CU: behind that they move twice the bytes for nothing (544 against 144 blocks of 128 x 128 at k = 4096: 33
// us against 30; 1088 against 288: 52 and 50).  Eight stages up to one block per CU (288 blocks on 256 CUs: 1.1 times the three-stage
// time) and from k = 1024 on, below which there is nothing to run ahead of (160 blocks, k 512: 9.9 us, three stages 9.4).  256 x 128 from 2048 on
// (k = 1024, 88 tiles: 24 us against 22) and only where every one has a CU.  k is that of all segments together, whether a launch holds one
// product or several (Shampoo roots of both sides in one launch, k of one segment / of all six, ms a step: 4 x 1024x1024 7.58 / 7.17,
// 2 x 1537x1025 12.05 / 11.1, 8 x 512x512 3.13 / 2.85).
template <int EPI, typename Args>
void launch_small(const Args& args, const EpiArgs& e, int64_t first, int64_t tiles, int64_t longest_k, int64_t cus, const Shape& s,
                  const OutSpec& o, hipStream_t st) {
  Args numbered = args;
  const int64_t n128 = first > 0 ? 4 * (tiles - first) : renumber<EPI, 128>(numbered);
  const int64_t n64 = first > 0 ? 16 * (tiles - first) : renumber<EPI, 64>(numbered);
  constexpr bool can_be_wide = epi_256x128(EPI) && !Args::finals;
  const bool wide = can_be_wide && 2 * (tiles - first) <= cus && longest_k >= 2048;
  if (n64 <= 2 * cus)
    launch_small_as<EPI, 64, 8>(args, e, first, tiles, s, o, st);
  else if (n128 <= cus && longest_k >= 1024)
    launch_small_as<EPI, 128, 8>(args, e, first, tiles, s, o, st);
  else if (wide)
    launch_small_as<EPI, can_be_wide ? 256 : 128, can_be_wide ? 6 : 3>(args, e, first, tiles, s, o, st);
  else
    launch_small_as<EPI, 128, 3>(args, e, first, tiles, s, o, st);
}

template <int EPI>
hipError_t launch(const GemmDims& d, const void* P, const void* Q, EpiArgs e, const SplitWs& w, const Shape& s,
                  const OutSpec& o, hipStream_t st) {
  // the k loop of both kernels takes whole panels in groups of four with a tail of four: K is a
  // multiple of 256 (the producers pad to PAD), hence at least 8 k-steps
  if (d.K < 8 * BK || d.K % (8 * BK) || d.M % BM || d.N % BN) return hipErrorInvalidValue;
  const int64_t tiles = tile_count<EPI>(d);
  const int64_t cus = cu_count();
  const OneProblem one{d, static_cast<const __bf16*>(P), static_cast<const __bf16*>(Q)};
  const int64_t left = tiles % cus, splits = k_slices<EPI>(left, d.K / BK, cus, w);
  const bool split_all = 2 * tiles <= cus && splits > 1 && split_pays<EPI>(d, d.K / BK, cus);
  const int64_t whole_large = split_all ? tiles : large_share<EPI>(tiles, cus, d.K, o.out_mode);
  if (whole_large < tiles) {
    if (whole_large > 0) {
      e.full_rounds = static_cast<int>(whole_large / cus), e.left = 0, e.splits = 1, e.partial = nullptr;
      e.main_grid = static_cast<int>(cus);
      hipLaunchKernelGGL((k_gemm_nt_bf16<EPI, false, OneProblem>), dim3(static_cast<unsigned>(cus)), dim3(NTHREADS), 0, st,
                         one, e, s, o);
    }
    launch_small<EPI>(one, e, whole_large, tiles, k_length<EPI>(d), cus, s, o, st);
    return hipGetLastError();
  }
  // full rounds of one tile per block, then the left-over tiles cut into k-slices
  e.full_rounds = static_cast<int>(tiles / cus);
  e.left = static_cast<int>(left);
  e.splits = static_cast<int>(splits);
  e.partial = w.partial;
  // whole tiles: one persistent block per CU (fewer if there are fewer tiles)
  const int64_t whole = e.splits > 1 ? e.full_rounds * cus : tiles;
  e.main_grid = static_cast<int>(std::min<int64_t>(cus, std::max<int64_t>(whole, 1)));
  if (whole > 0)
    hipLaunchKernelGGL((k_gemm_nt_bf16<EPI, false, OneProblem>), dim3(static_cast<unsigned>(e.main_grid)), dim3(NTHREADS),
                       0, st, one, e, s, o);
  if constexpr (!epi_terms(EPI)) if (e.splits > 1) {
    hipLaunchKernelGGL((k_gemm_nt_bf16<EPI, true, OneProblem>), dim3(static_cast<unsigned>(e.left * e.splits)),
                       dim3(NTHREADS), 0, st, one, e, s, o);
    hipLaunchKernelGGL((k_split_finish<EPI>), dim3(static_cast<unsigned>(e.left)), dim3(NTHREADS), 0, st, d, e, s, o);
  }
  return hipGetLastError();
}

// Several products in one launch: whole tiles only (no k-split), one persistent block per CU.
template <int EPI>
hipError_t launch_multi(const GemmBatch& g, EpiArgs e, hipStream_t st) {
  const int64_t cus = cu_count();
  ManyProblems<EPI> many{};
  if (g.n > many.max) return hipErrorInvalidValue;
  many.n = g.n;
  int64_t tiles = 0, longest_k = 0;
  for (int j = 0; j < g.n; ++j) {
    many.begin[j] = static_cast<int>(tiles);
    many.pr[j] = g.pr[j];
    const GemmDims& d = g.pr[j].d;
    if (d.K < 8 * BK || d.K % (8 * BK) || d.M % BM || d.N % BN) return hipErrorInvalidValue;
    tiles += tile_count<EPI>(d);
    longest_k = std::max(longest_k, k_length<EPI>(d));
  }
  for (int j = g.n; j <= many.max; ++j) many.begin[j] = static_cast<int>(tiles);
  if (tiles == 0) return hipSuccess;
  const int64_t whole_large = large_share<EPI>(tiles, cus, longest_k);
  e.splits = 1;
  e.partial = nullptr;
  if (whole_large > 0) {
    e.full_rounds = static_cast<int>(whole_large / cus);
    e.left = static_cast<int>(whole_large % cus);
    e.main_grid = static_cast<int>(std::min<int64_t>(cus, whole_large));
    hipLaunchKernelGGL((k_gemm_nt_bf16<EPI, false, ManyProblems<EPI>>), dim3(static_cast<unsigned>(e.main_grid)), dim3(NTHREADS),
                       0, st, many, e, Shape{}, OutSpec{});
  }
  if (whole_large < tiles) launch_small<EPI>(many, e, whole_large, tiles, longest_k, cus, Shape{}, OutSpec{}, st);
  return hipGetLastError();
}

}  // namespace

namespace {
template <int EPI>
hipError_t launch_problems(const GemmBatch& g, EpiArgs e, const SplitWs& w, hipStream_t st) {
  if (g.n != 1) return launch_multi<EPI>(g, e, st);
  const GemmProblem& pr = g.pr[0];
  e.c = pr.c, e.ct = pr.ct, e.sym = pr.sym, e.scale = pr.scale;
  return launch<EPI>(pr.d, pr.p, pr.q, e, w, Shape{}, OutSpec{}, st);
}
}  // namespace

hipError_t launch_gram_bf16(const GemmBatch& g, bool from_xt, const SplitWs& w, hipStream_t st) {
  if (g.n > 0 && g.pr[0].sym.diag) return from_xt ? launch_problems<EPI_GRAM_APART>(g, EpiArgs{}, w, st) : hipErrorInvalidValue;
  return from_xt ? launch_problems<EPI_GRAM_T>(g, EpiArgs{}, w, st) : launch_problems<EPI_GRAM>(g, EpiArgs{}, w, st);
}

hipError_t launch_poly_bf16(const GemmBatch& g, float ca, float cb, float cc, const SplitWs& w, hipStream_t st) {
  EpiArgs e{};
  e.ca = ca, e.cb = cb, e.cc = cc;
  return g.n > 0 && g.pr[0].sym.x ? launch_problems<EPI_POLY_APART>(g, e, w, st) : launch_problems<EPI_POLY>(g, e, w, st);
}

hipError_t launch_mul_f16(const GemmBatch& g, MulResult result, const SplitWs& w, hipStream_t st) {
  switch (result) {
    case MulResult::Q: return launch_problems<EPI_MUL_Q>(g, EpiArgs{}, w, st);
    case MulResult::Q2: return launch_problems<EPI_MUL_Q2>(g, EpiArgs{}, w, st);
    default: return launch_problems<EPI_MUL>(g, EpiArgs{}, w, st);
  }
}

hipError_t launch_split3_sym(const GemmBatch& g, hipStream_t st) {
  return launch_problems<EPI_B3_SYM>(g, EpiArgs{}, SplitWs{nullptr, 0}, st);
}

hipError_t launch_update_bf16(const GemmBatch& g, const SplitWs& w, hipStream_t st) {
  return g.n > 0 && g.pr[0].sym.x ? launch_problems<EPI_UPDATE_APART>(g, EpiArgs{}, w, st)
                                  : launch_problems<EPI_UPDATE>(g, EpiArgs{}, w, st);
}

hipError_t launch_update_bf16(const GemmDims& d, const void* b_in, const void* xt_in, void* xw_out, void* xt_out,
                              const float* scale, const SplitWs& w, hipStream_t st) {
  EpiArgs e{};
  e.c = xw_out;
  e.ct = xt_out;
  e.scale = scale;
  return launch<EPI_UPDATE>(d, b_in, xt_in, e, w, Shape{}, OutSpec{}, st);
}

hipError_t launch_split3(const GemmDims& d, const void* p, const void* q, void* c, hipStream_t st) {
  EpiArgs e{};
  e.c = c;
  return launch<EPI_B3>(d, p, q, e, SplitWs{nullptr, 0}, Shape{}, OutSpec{}, st);
}

hipError_t launch_terms_final(const GemmDims& d, const void* p, const void* q, const Shape& s, const OutSpec& o, hipStream_t st) {
  return launch<EPI_OUT_TERMS>(d, p, q, EpiArgs{}, SplitWs{nullptr, 0}, s, o, st);
}

hipError_t launch_final_bf16(const GemmDims& d, const void* p, const void* q, const float* scale, const SplitWs& w,
                             const Shape& s, const OutSpec& o, hipStream_t st) {
  EpiArgs e{};
  e.scale = scale;
  return launch<EPI_FINAL>(d, p, q, e, w, s, o, st);
}

// Small tiles throughout: up to two rounds of 256 x 256 ones, and no k that the large tile is for.  Seven matrices of four shape classes
// (208 tiles, k 1024): four launches 73 us, one 50.  us a step, a launch each -> one, by tiles: 40 (k 1024) 181 -> 176; 112 303 -> 290;
// 128 (k 2048) 469 -> 460; 176 (k 512) 337 -> 342; 224 (k 2048) 765 -> 747; 240 501 -> 466; 288 636 -> 629; 396 (k 1536) 1107 -> 1122; 448
// (k 2048) 1398 -> 1385; 480 900 -> 892: of 29 calls the two with 176 and 396 lose, 1.5 %.
bool final_parts_fit(int n, const FinalPart* parts) {
  int64_t tiles = 0, longest_k = 0;
  for (int i = 0; i < n; ++i) tiles += tile_count<EPI_FINAL>(parts[i].d), longest_k = std::max(longest_k, parts[i].d.K);
  return n <= MAX_PARTS && tiles <= 2 * cu_count() && longest_k <= 2048;
}
hipError_t launch_final_parts_bf16(int n, const FinalPart* parts, const OutSpec& o, hipStream_t st) {
  if (n < 1 || n > MAX_PARTS) return hipErrorInvalidValue;
  FinalParts many{};
  many.n = n;
  int64_t tiles = 0, longest_k = 0;
  for (int i = 0; i < n; ++i) {
    const GemmDims& d = parts[i].d;
    if (d.K < 8 * BK || d.K % (8 * BK) || d.M % BM || d.N % BN) return hipErrorInvalidValue;
    many.pr[i] = parts[i];
    tiles += tile_count<EPI_FINAL>(d), longest_k = std::max(longest_k, d.K);
  }
  EpiArgs e{};
  e.splits = 1;
  launch_small<EPI_FINAL>(many, e, 0, tiles, longest_k, cu_count(), Shape{}, o, st);
  return hipGetLastError();
}

hipError_t launch_final_sym_bf16(const GemmDims& d, const void* x, const SplitWs& w, const Shape& s, const OutSpec& o,
                                 hipStream_t st) {
  if (d.M != d.N) return hipErrorInvalidValue;
  return launch<EPI_FINAL_SYM>(d, x, x, EpiArgs{}, w, s, o, st);
}

}  // namespace canz
