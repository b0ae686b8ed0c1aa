// Launchers of the device kernels behind canz_muon_step (internal, not part of the ABI).
//
// Working layout of one sub-batch of nb same-shape matrices (m = min(rows, cols),
// n = max(rows, cols), mp / np = m / n rounded up to PAD):
//   XT  [nb][np][mp]  the iterate X, transposed from its wide orientation (two buffers, ping-pong)
//   XW  [nb][mp][np]  the same values in the wide orientation, where they are wanted (muon_step.hip: wants_x)
//   A,B [nb][mp][mp]  Gram matrix and the polynomial aI + bA + cAA
// Padding rows / columns hold zeros; zeros stay zero under the iteration, so the GEMM
// kernels run on the padded extents without bounds checks.  Every product but one contracts over a contiguous index of both operands
// (C[i][j] = sum_k P[i][k] Q[j][k]), which is the operand form of the bf16 MFMA; the Gram product can also contract over the rows of
// X^T, through transposing LDS reads, so that X need not be written in both orientations.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "canz_internal.h"

namespace canz {

constexpr int PAD = 256;           // working extents are multiples of this
constexpr int MAX_TP = 8;
constexpr int MAX_PTRS = 128;      // buffers per pointer table: a launch takes up to MAX_PTRS / tp matrices
// ... and no more than this many padded elements, which bounds the workspace of a launch
constexpr int64_t MAX_BATCH_ELEMS = int64_t(1) << 30;
constexpr int EW_TILE = 64;        // elementwise kernels work on 64 x 64 tiles

// Pointer tables travel as kernel arguments, so nothing is copied to the device.
struct PtrTable {
  void* p[MAX_PTRS];
};

struct Shape {
  int64_t rows, cols;   // caller's matrix
  int64_t m, n;         // min / max extent
  int64_t mp, np;       // padded
  int tall;             // rows > cols: the wide orientation is the transpose
  int tp;               // column fragments of grad / delta
  int64_t wfrag;        // cols / tp
};

// ---- per-kernel timing (canz_profile_*) --------------------------------------------
// Records an event on `st` before (begin) or after a launch of the given CANZ_KERNEL_* kind;
// does nothing while profiling is off.
void prof_mark(hipStream_t st, int kind, bool begin);

#define CANZ_HIP(kind, expr, what)                                                      \
  do {                                                                                  \
    ::canz::prof_mark(st, kind, true);                                                  \
    hipError_t err__ = (expr);                                                          \
    ::canz::prof_mark(st, kind, false);                                                 \
    if (err__ != hipSuccess) return ::canz::fail(CANZ_EHIP, "%s: %s", what, hipGetErrorString(err__)); \
  } while (0)

// ---- elementwise -----------------------------------------------------------------
// M <- beta M + G; U = M or G + beta M; U written (type T = bf16 or float) to XW (unless null) and XT
// (padding zero-filled); per-tile sums of U^2 to partial[b][tile].
template <typename T>
hipError_t launch_momentum(const Shape& s, int nb, const PtrTable& grad, int grad_dtype,
                           const PtrTable& mom, float beta, int nesterov, T* xw, T* xt,
                           float* partial, hipStream_t st);
int momentum_tiles(const Shape& s);  // partial sums per matrix

// The same for several parts of one call (matrices of one shape and orientation each) in one launch: the buffers of part i are
// number first_grad (first_mom) and on of the tables.
constexpr int MAX_PARTS = 8;   // two orientations of MAX_KINDS shape classes
template <typename T>
struct MomentumPart {
  Shape s;
  int nb, grad_dtype, first_grad, first_mom;
  T *xw, *xt;
  float* partial;
};
hipError_t launch_momentum_parts(int n, const MomentumPart<__bf16>* parts, const PtrTable& grad, const PtrTable& mom, float beta,
                                 int nesterov, hipStream_t st);

// scale[b] = 1 / (sqrt(sum partial[b][*]) + eps), scale2[b] = scale[b]^2
hipError_t launch_norm_scale(int nb, int n_partial, const float* partial, float eps, float* scale,
                             float* scale2, hipStream_t st);
// the same for up to MAX_KINDS batches in one launch
constexpr int MAX_KINDS = 4;                  // shape classes that run side by side
struct NormBatch {
  int nb, n_partial;
  const float* partial;
  float *scale, *scale2;
};
hipError_t launch_norm_scale_batches(int n, const NormBatch* batches, float eps, hipStream_t st);

struct OutSpec {
  PtrTable out;
  int out_dtype;      // CANZ_DT_*
  int out_mode;       // CANZ_OUT_*
  float decay;        // 1 - lr * weight_decay
  float neg_lr_scale; // -lr * scale
};

// ns_steps == 0: O = scale[b] * U taken from the orientation that matches the caller's.
template <typename T>
hipError_t launch_apply(const Shape& s, int nb, const T* x_straight, int64_t ld, int64_t batch_stride,
                        const float* scale, const OutSpec& o, hipStream_t st);

// ---- bf16 MFMA GEMMs -------------------------------------------------------------
struct GemmDims {
  int64_t M, N, K;          // multiples of PAD
  int64_t ldp, ldq;         // row lengths of P and Q (K, or more where the product runs over a part of their columns)
  int64_t sp, sq;           // batch strides
  int nb;
  // Operands of several terms (launch_split3*): an operand of t terms is a panel matrix of t * K columns, term i in the
  // columns i K .. ; the product runs over nseg segments of K, segment s multiplying term (pseg >> 4 s) & 15 of P
  // with term (qseg >> 4 s) & 15 of Q, all into one accumulator.
  int nseg;
  unsigned pseg, qseg;
};
// Scratch for the k-split of left-over tiles: fp32 accumulators of up to max_blocks blocks
// (256 KiB each), written by the split launch and read by the kernel that finishes the tiles.
struct SplitWs {
  float* partial;
  int max_blocks;
};
constexpr int SPLIT_MAX_BLOCKS = 256;                       // CU count of MI355X; fewer blocks split on a smaller part
constexpr size_t SPLIT_BLOCK_BYTES = 256 * 256 * sizeof(float);
// How the products of the symmetric m x m matrices (all of them polynomials in one Gram matrix) take their factors
// and leave their result.  In single steps a matrix is a bf16 image in the panel layout.  In merged steps, where several of them
// follow each other without X in between, its diagonal is kept apart as an fp32 vector (the image holds zeros there), and the
// image is fp16.  The MFMA products use the images; everything that multiplies a diagonal, and the element-wise terms, are
// added in the epilogue in fp32:
//   (D_P + H_P)(D_Y + H_Y) = D_P D_Y + D_P H_Y + H_P D_Y + H_P H_Y.
// The diagonals are what all these matrices consist of once X is close to orthogonal, and their nearly equal elements
// round alike.  fp16 has 11 bits where bf16 has 8; its exponents suffice, since these matrices have known magnitude (the caller
// sees to it): the images hold UNIT_A times the elements of A, B A (eigenvalues up to 1.69) and UNIT_B times those of B and
// of products of B (up to 3.5^3).  A and B A have elements down to 1 / (m sqrt(n)), far above 2^-14 / UNIT_A, where fp16 begins to lose bits.
constexpr float UNIT_A = 16384.f, UNIT_B = 1024.f;
struct SymSpec {
  const void* aux;      // POLY: A;  MUL: the second factor Y;  UPDATE: X^T
  const void* aux2;     // MUL: the first factor P (always a B)
  const float* x;       // POLY: the diagonal of A, or nullptr (a bf16 image that holds it);  MUL: the diagonal of P;  UPDATE: of Q   [nb][M]
  const float* y;       // POLY: as x;  MUL: the diagonal of Y
  float* diag;          // result: diagonal, or nullptr (a bf16 image that holds it)
  float unit;           // MUL: the unit of Y and of the result, UNIT_A or UNIT_B
};
// Several products of one kind in one launch: matrices of different shapes, or independent products of one chain.
// The persistent blocks walk the tiles of problem 0, then of problem 1, ...
constexpr int MAX_PROBLEMS = 2 * MAX_KINDS;   // two independent products of each
struct GemmProblem {
  GemmDims d;
  const void* p;       // first operand  [nb][M][K] panels
  const void* q;       // second operand [nb][N][K] panels
  void* c;             // output (UPDATE: the straight image)
  void* ct;            // UPDATE: the transposed image
  SymSpec sym;         // GRAM, POLY, MUL, UPDATE
  const float* scale;  // per-matrix factor or nullptr
};
struct GemmBatch {
  int n;
  GemmProblem pr[MAX_PROBLEMS];
};
// A = scale2[b] * X X^T, from XW or from XT  (P = Q = XW [nb][M][K] or XT [nb][K][M]); all problems with sym.diag (from XT), or none
hipError_t launch_gram_bf16(const GemmBatch& g, bool from_xt, const SplitWs& w, hipStream_t st);
// B = ca I + cb A + cc A A                   (P = Q = A, symmetric); all problems with sym.x and sym.y, or none
hipError_t launch_poly_bf16(const GemmBatch& g, float ca, float cb, float cc, const SplitWs& w, hipStream_t st);
// C = P Y, P and Y symmetric and commuting   (Q = Y).  The result leaves as fp16 image and diagonal (CHAIN), as bf16 image and
// diagonal for the update (Q), or as two bf16 terms [nb][M][2 M] for the last product (Q2)
enum class MulResult { CHAIN, Q, Q2 };
hipError_t launch_mul_f16(const GemmBatch& g, MulResult result, const SplitWs& w, hipStream_t st);
// as launch_update_bf16 below, for several problems (c null: the transposed image alone); with sym.x: Q's diagonal apart (and
// sym.aux = X^T)
hipError_t launch_update_bf16(const GemmBatch& g, const SplitWs& w, hipStream_t st);

// X' = scale[b] * B X: XW' [mp][np] straight and XT' [np][mp] transposed  (P = B, Q = XT)
hipError_t launch_update_bf16(const GemmDims& d, const void* b_in, const void* xt_in, void* xw_out, void* xt_out,
                              const float* scale, const SplitWs& w, hipStream_t st);
// last step: O = scale[b] * P Q^T goes straight into the caller's buffers; the caller of
// this launcher orders the operands so that C is in the matrix's own orientation:
// wide matrix: P = B, Q = XT (C = B X);  tall matrix: P = XT, Q = B (C = X^T B = (B X)^T)
hipError_t launch_final_bf16(const GemmDims& d, const void* p, const void* q, const float* scale, const SplitWs& w,
                             const Shape& s, const OutSpec& o, hipStream_t st);
// several of them in one launch, on small tiles: part i writes the buffers number first_out and on of o.out with its own type and factor
// (out_mode and decay are those of o)
struct FinalPart {
  GemmDims d;
  const void *p, *q;
  const float* scale;
  Shape s;
  int out_dtype, first_out;
  float neg_lr_scale;
};
// whether that is the faster way: launches that leave most of the chip idle or end in a round that does
bool final_parts_fit(int n, const FinalPart* parts);
hipError_t launch_final_parts_bf16(int n, const FinalPart* parts, const OutSpec& o, hipStream_t st);
// the same for a symmetric result O = X X^T (M = N): only the tiles on and above the diagonal are computed and
// written; the elements below the diagonal tiles are left as they were (the caller mirrors them)
hipError_t launch_final_sym_bf16(const GemmDims& d, const void* x, const SplitWs& w, const Shape& s, const OutSpec& o,
                                 hipStream_t st);

// ---- fp32 products on the 16-bit matrix cores ---------------------------------------
// A value of 24 bits is the sum of three bf16 values (8 bits each), which have fp32's exponents: matrices of any magnitude and
// of elements of any ratio keep the accuracy they have in fp32.  The products of the terms are exact in fp32 and are
// added up in fp32, the small ones first, K / 16 roundings per product where the fp32 MFMA rounds K / 2 times.  Six products
// (those left out are at most 2^-26 of the result), three if one operand is a matrix of bf16 values, i.e. of one term.
// An infinity in an operand (or a value above 3.39e38, which bf16 rounds to one) gives NaN where the fp32 product would
// give an infinity or NaN: it is inf - inf in the terms, and inf * 0 against terms that are zero.
// C = P Q^T, P [nb][M][3 K], Q [nb][N][qterms K]:
//   c [nb][M][3 N], the result as three terms
hipError_t launch_split3(const GemmDims& d, const void* p, const void* q, void* c, hipStream_t st);
//   the same for symmetric P and Q that commute: the tiles on and above the diagonal, mirrored.  ct of a problem, or
//   nullptr: 5/4 I - 1/4 c as three terms
hipError_t launch_split3_sym(const GemmBatch& g, hipStream_t st);
//   the result as the last product of launch_final_bf16 (o: the caller's buffers); operands of one, two or three terms
hipError_t launch_terms_final(const GemmDims& d, const void* p, const void* q, const Shape& s, const OutSpec& o, hipStream_t st);
inline GemmDims split3_dims(int64_t M, int64_t N, int64_t K, int qterms, int nb, int pterms = 3) {
  // terms 2 0, 0 2, 1 1, 1 0, 0 1, 0 0 of P and Q, or 2, 1, 0 of P: the small products first
  if (pterms == 1) return GemmDims{M, N, K, K, 3 * K, M * K, 3 * N * K, nb, 3, 0u, 0x012u};
  if (qterms == 1) return GemmDims{M, N, K, 3 * K, K, 3 * M * K, N * K, nb, 3, 0x012u, 0u};
  return GemmDims{M, N, K, 3 * K, 3 * K, 3 * M * K, 3 * N * K, nb, 6, 0x001102u, 0x010120u};
}

// ---- fp32 verification GEMMs (same contracts, float storage) ----------------------
hipError_t launch_gram_f32(const GemmDims& d, const void* xw, void* a_out, const float* scale2, hipStream_t st);
hipError_t launch_poly_f32(const GemmDims& d, const void* a_in, void* b_out, float ca, float cb, float cc,
                           hipStream_t st);
hipError_t launch_update_f32(const GemmDims& d, const void* b_in, const void* xt_in, void* xw_out, void* xt_out,
                             const float* scale, hipStream_t st);
hipError_t launch_final_f32(const GemmDims& d, const void* p, const void* q, const float* scale,
                            const Shape& s, const OutSpec& o, hipStream_t st);

}  // namespace canz
