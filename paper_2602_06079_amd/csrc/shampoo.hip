// canz_shampoo_step / canz_shampoo_workspace_bytes: the Shampoo step the paper runs through
// the same planner as Muon ("Generalization to Other Optimizers (Shampoo & SOAP)", App. C;
// App. B.3), per matrix:
//   L <- beta L + G G^T,  R <- beta R + G^T G,
//   O = (L + eps I)^(-1/4) G (R + eps I)^(-1/4),  P <- P (1 - lr wd) - lr O  (or Delta W = -lr O).
// State and results are fp32 (the statistics span many orders of magnitude; bf16 would lose the small
// eigenvalues the inverse root amplifies).
//
// All products have the form C[i][j] = sum_k P[i][k] Q[j][k] with both operands contiguous
// along k: the statistics are Gram products of G in its two orientations (both are written by
// the load kernel), and every matrix of the root iteration is a polynomial in the symmetric
// A = S + eps I, hence symmetric itself, so "times Q" and "times Q^T" coincide.  Symmetric
// products compute only the tiles on or above the diagonal and write the mirror tile from the
// same accumulators, which halves their work and keeps the iterates symmetric (bit for bit across
// tiles; inside a diagonal tile the two halves are rounded separately and agree to an ulp or two).
//
// Inverse fourth root (coupled Newton iteration for the inverse p-th root, p = 4): from
// M = z A, X = z^(1/4) I with z = 5 / (2 b), b an upper bound of the largest eigenvalue (see k_sh_init),
// repeat T = (5 I - M) / 4, X <- X T,
// M <- T^4 M; M -> I and X -> A^(-1/4).  Four products per round: X T, T T, T^2 T^2, T^4 M (the
// last one also writes the next T).  The round count is fixed by the caller: no test of
// convergence is read back, so the step never synchronises and can be captured in a graph.
//
// These products, nearly all of the step's work, run on the bf16 matrix cores: every matrix of the iteration is held as
// three bf16 terms per element (fp32's 24 bits and its exponents) and a product is the sum of six products of terms with fp32
// sums (launch_split3_sym), 6 / 16 of the fp32 MFMA's time at full rate.  The exponents matter: rows without signal, or
// scales that differ from row to row, give elements many orders of magnitude below ||A|| that the root is made of, and a
// representation with an absolute resolution loses them (two fp16 terms took half the products; half the rows empty at eps =
// 1e-8 lambda_max gave a root error of 6e-5 where fp32 has 1e-7).  Against fp32 matrices on the fp32 MFMA, whose 32 x 32 x 2
// steps round a sum k / 2 times, the roots are closer to 64 bits: 1.4e-5 instead of 1.6e-4 on 3072 x 3072 statistics at
// eps = 1e-4 lambda_max.  4 x 3072 x 1024, 22 rounds: 92.3 ms on the fp32 MFMA, 65.8 ms on three terms.
// Both sides run their rounds side by side (the tiles of one alone leave the last round of the chip half empty), and
// X T shares a launch with T T.
//
// Statistics of bf16 gradients run on the bf16 matrix cores (statistic_bf16), those of fp32 gradients on
// v_mfma_f32_32x32x2_f32; the two preconditioning products on the bf16 cores with three terms per fp32 element
// (launch_split3).  Working extents are multiples of 128 for the fp32 MFMA and of 256 elsewhere (zero padding: the padded part
// of every iterate is a separate diagonal block that never mixes with the matrix and is multiplied by zeros at the end).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "canz.h"
#include "canz_internal.h"
#include "device_util.h"
#include "f32_mfma_gemm.h"
#include "kernels.h"
#include "panel_layout.h"

namespace canz {
namespace {

using namespace f32mfma;

constexpr int NPART = 64;        // partial sums per matrix of the Frobenius norm
constexpr int64_t MAX_EXTENT = 32768;
constexpr size_t BATCH_BYTES = size_t(8) << 30;

// sum over the block's threads -> *to
__device__ __forceinline__ void block_sum_to(float ss, float* to) {
  __shared__ float wsum[NTH / 64];
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = ss;
  __syncthreads();
  if (threadIdx.x == 0) *to = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}
// partial[b][p] = sum of squares of the elements p, p + NPART * NTH, ... (in blocks of NTH) of A[b] = S + eps I
__global__ __launch_bounds__(NTH) void k_sh_sumsq(PtrTable stat, int64_t d, float eps, float* __restrict__ partial) {
  const int b = blockIdx.y, p = blockIdx.x;
  const float* s = static_cast<const float*>(stat.p[b]);
  float ss = 0.f;
  for (int64_t i = static_cast<int64_t>(p) * NTH + threadIdx.x; i < d * d; i += static_cast<int64_t>(NPART) * NTH) ss += s[i] * s[i];
  for (int64_t i = static_cast<int64_t>(p) * NTH + threadIdx.x; i < d; i += static_cast<int64_t>(NPART) * NTH)
    ss += eps * (2.f * s[i * d + i] + eps);   // (S_ii + eps)^2 - S_ii^2
  block_sum_to(ss, partial + b * NPART + p);
}

// Eight consecutive elements of a matrix of three bf16 terms: chunk `i` of the first term's panels, in memory order.
// [dp][3 dp] columns: panel (row block, k block) of term t is number row_block * 3 nkb + t nkb + k_block.
struct Chunk {
  int64_t at, step, row, col;   // the first term's place, from one term to the next; the elements
  __device__ __forceinline__ Chunk(int64_t i, int64_t dp) {
    const int64_t nkb = dp / PANEL_K, panel = i / (PANEL_ELEMS / 8), w = i - panel * (PANEL_ELEMS / 8);
    const int64_t rb = panel / nkb, kb = panel - rb * nkb;
    at = ((rb * 3 * nkb) + kb) * PANEL_ELEMS + w * 8;
    step = nkb * PANEL_ELEMS;
    row = rb * PANEL_ROWS + w / 4;
    col = kb * PANEL_K + (((w & 3) ^ ((row >> 2) & 3)) << 3);
  }
};
__device__ __forceinline__ void put_terms(__bf16* m, const Chunk& c, float (&v)[8]) {
#pragma unroll
  for (int term = 0; term < 3; ++term) {
    bf16x8 t;
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] = static_cast<__bf16>(v[e]), v[e] -= static_cast<float>(t[e]);
    *reinterpret_cast<bf16x8*>(m + c.at + term * c.step) = t;
  }
}
__device__ __forceinline__ void get_terms(const __bf16* m, const Chunk& c, float (&v)[8]) {
  bf16x8 t[3];
#pragma unroll
  for (int term = 0; term < 3; ++term) t[term] = *reinterpret_cast<const bf16x8*>(m + c.at + term * c.step);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (static_cast<float>(t[0][e]) + static_cast<float>(t[1][e])) + static_cast<float>(t[2][e]);
}

// partial sums as above of a matrix of three terms
__global__ __launch_bounds__(NTH) void k_sh_sumsq_terms(const __bf16* __restrict__ a, int64_t dp, float* __restrict__ partial) {
  const int b = blockIdx.y, p = blockIdx.x;
  const __bf16* ab = a + static_cast<int64_t>(b) * 3 * dp * dp;
  float ss = 0.f;
  for (int64_t i = static_cast<int64_t>(p) * NTH + threadIdx.x; i < dp * dp / 8; i += static_cast<int64_t>(NPART) * NTH) {
    float v[8];
    get_terms(ab, Chunk(i, dp), v);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
  }
  block_sum_to(ss, partial + b * NPART + p);
}

// the caller's dense d x d matrices <- matrices of three terms [dp][3 dp] (the sum of the terms is the fp32 value, exactly)
__global__ __launch_bounds__(NTH) void k_sh_store_terms(const __bf16* __restrict__ a, PtrTable to, int64_t d, int64_t dp) {
  const int b = blockIdx.y;
  const __bf16* ab = a + static_cast<int64_t>(b) * 3 * dp * dp;
  float* m = static_cast<float*>(to.p[b]);
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * NTH + threadIdx.x; i < dp * dp / 8; i += static_cast<int64_t>(gridDim.x) * NTH) {
    const Chunk c(i, dp);
    if (c.row >= d || c.col >= d) continue;
    float v[8];
    get_terms(ab, c, v);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (c.col + e < d) m[c.row * d + c.col + e] = v[e];
  }
}

// Start of the root iteration.  The iteration needs M = z A with eigenvalues in (0, 5); the closer the largest
// comes to 5/2 the fewer rounds the smallest needs to grow to 1.  ||A||_F bounds the largest eigenvalue of A,
// but loosely (by sqrt(d) for a flat spectrum: three and a half rounds at d = 3072); ||A'^4||_F^(1/4) with
// A' = A / ||A||_F is a bound too, at most d^(1/8) above it, for two products.
//   k_sh_prescale:  A' = A / ||A||_F
//   k_sh_init:      z' = 5 / (2 ||A'^4||_F^(1/4));  M = z' A';  T = 5/4 I - 1/4 M;  X = (z' / ||A||_F)^(1/4) I
__device__ __forceinline__ double sum_partials(const float* partial, int b) {
  double sum = 0.0;
  for (int i = 0; i < NPART; ++i) sum += static_cast<double>(partial[b * NPART + i]);
  return sum;
}

__global__ __launch_bounds__(NTH) void k_sh_prescale(PtrTable stat, int64_t d, int64_t dp, float eps,
                                                      const float* __restrict__ partial, __bf16* __restrict__ m) {
  const int b = blockIdx.y;
  const float* s = static_cast<const float*>(stat.p[b]);
  const float nrm = static_cast<float>(sqrt(sum_partials(partial, b)));
  const float inv = nrm > 0.f ? 1.f / nrm : 0.f;
  __bf16* mb = m + static_cast<int64_t>(b) * 3 * dp * dp;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * NTH + threadIdx.x; i < dp * dp / 8; i += static_cast<int64_t>(gridDim.x) * NTH) {
    const Chunk c(i, dp);
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[e] = 0.f;
      if (c.row < d && c.col + e < d) v[e] = inv * (s[c.row * d + c.col + e] + (c.row == c.col + e ? eps : 0.f));
    }
    put_terms(mb, c, v);
  }
}

__global__ __launch_bounds__(NTH) void k_sh_init(const float* __restrict__ partial, const float* __restrict__ partial4,
                                                  int64_t d, int64_t dp, __bf16* __restrict__ x, __bf16* __restrict__ m,
                                                  __bf16* __restrict__ tt) {
  const int b = blockIdx.y;
  const float nrm = static_cast<float>(sqrt(sum_partials(partial, b)));
  const float bound = static_cast<float>(pow(sum_partials(partial4, b), 0.125));   // ||A'^4||_F^(1/4) >= lambda_max(A')
  const float z = bound > 0.f ? 2.5f / bound : 1.f;
  const float x0 = nrm > 0.f ? sqrtf(sqrtf(z / nrm)) : 1.f;
  const int64_t off = static_cast<int64_t>(b) * 3 * dp * dp;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * NTH + threadIdx.x; i < dp * dp / 8; i += static_cast<int64_t>(gridDim.x) * NTH) {
    const Chunk c(i, dp);
    float mv[8], tv[8], xv[8];
    get_terms(m + off, c, mv);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool diag = c.row == c.col + e, pad = diag && c.row >= d;
      mv[e] = pad ? 1.f : z * mv[e];   // the padding stands at the fixed point M = T = X = I
      tv[e] = (diag ? 1.25f : 0.f) - 0.25f * mv[e];
      xv[e] = pad ? 1.f : diag ? x0 : 0.f;
    }
    put_terms(m + off, c, mv);
    put_terms(tt + off, c, tv);
    put_terms(x + off, c, xv);
  }
}

// The same for fp32 matrices on the fp32 MFMA (see Path).
// partial[b][p] = sum of squares of the elements p, p + NPART * NTH, ... (in blocks of NTH) of A[b]
__global__ __launch_bounds__(NTH) void k_sh_sumsq_f32(const float* __restrict__ a, int64_t elems, float* __restrict__ partial) {
  const int b = blockIdx.y, p = blockIdx.x;
  const float* ab = a + static_cast<int64_t>(b) * elems;
  float ss = 0.f;
  for (int64_t i = static_cast<int64_t>(p) * NTH + threadIdx.x; i < elems; i += static_cast<int64_t>(NPART) * NTH) ss += ab[i] * ab[i];
  block_sum_to(ss, partial + b * NPART + p);
}

__global__ __launch_bounds__(NTH) void k_sh_prescale_f32(const float* __restrict__ a, const float* __restrict__ partial,
                                                      int64_t elems, float* __restrict__ m) {
  const int b = blockIdx.y;
  const float nrm = static_cast<float>(sqrt(sum_partials(partial, b)));
  const float inv = nrm > 0.f ? 1.f / nrm : 0.f;
  const int64_t off = static_cast<int64_t>(b) * elems;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * NTH + threadIdx.x; i < elems; i += static_cast<int64_t>(gridDim.x) * NTH)
    m[off + i] = inv * a[off + i];
}

__global__ __launch_bounds__(NTH) void k_sh_init_f32(const float* __restrict__ partial, const float* __restrict__ partial4,
                                                  int64_t dp, float* __restrict__ x, float* __restrict__ m,
                                                  float* __restrict__ tt) {
  const int b = blockIdx.y;
  const float nrm = static_cast<float>(sqrt(sum_partials(partial, b)));
  const float bound = static_cast<float>(pow(sum_partials(partial4, b), 0.125));   // ||A'^4||_F^(1/4) >= lambda_max(A')
  const float z = bound > 0.f ? 2.5f / bound : 1.f;
  const float x0 = nrm > 0.f ? sqrtf(sqrtf(z / nrm)) : 1.f;
  const int64_t elems = dp * dp, off = static_cast<int64_t>(b) * elems;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * NTH + threadIdx.x; i < elems; i += static_cast<int64_t>(gridDim.x) * NTH) {
    const bool diag = (i / dp) == (i % dp);
    const float mv = z * m[off + i];
    m[off + i] = mv;
    tt[off + i] = (diag ? 1.25f : 0.f) - 0.25f * mv;
    x[off + i] = diag ? x0 : 0.f;
  }
}

// G (bf16 or fp32, whole or tp column fragments) -> what its readers want.  bf16: panels padded to 256 in both
// orientations, for the statistics and the preconditioning product.  fp32: copies padded to 128 in both orientations for
// the statistics, and the transposed one as three bf16 terms for the product.  One block per 64 x 64 tile of the larger padding.
__global__ __launch_bounds__(NTH) void k_sh_load_grad(Shape s, PtrTable grad, int grad_dtype, int64_t rp, int64_t cp,
                                                       float* __restrict__ gs, float* __restrict__ gt, int64_t rp2, int64_t cp2,
                                                       __bf16* __restrict__ gp, __bf16* __restrict__ gpt,
                                                       __bf16* __restrict__ g3t) {
  __shared__ float tile[64][65];
  const int b = blockIdx.z, r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
  const int wf = static_cast<int>(s.wfrag);
  float val[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, row = r0 + (idx >> 6), col = c0 + (idx & 63);
    val[e] = 0.f;
    if (row < s.rows && col < s.cols) {
      const int f = col / wf;
      const int64_t at = static_cast<int64_t>(row) * wf + (col - f * wf);
      val[e] = grad_dtype == CANZ_DT_BF16 ? static_cast<float>(static_cast<const __bf16*>(grad.p[b * s.tp + f])[at])
                                          : static_cast<const float*>(grad.p[b * s.tp + f])[at];
    }
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;
    if (gs && r0 + r < rp && c0 + c < cp) gs[(b * rp + r0 + r) * cp + c0 + c] = val[e];
    tile[r][c] = val[e];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;  // r: column of G, c: row of G
    if (gt && c0 + r < cp && r0 + c < rp) gt[(b * cp + c0 + r) * rp + r0 + c] = tile[c][r];
  }
  if (g3t) tile_to_terms3(tile, g3t + b * 3 * rp2 * cp2, r0, c0, rp2, true, t);
  if (gp) tile_to_panels(tile, gp + b * rp2 * cp2, r0, c0, cp2, false, t);
  if (gpt) tile_to_panels(tile, gpt + b * rp2 * cp2, r0, c0, rp2, true, t);
}

bool bf16_statistics(const canz_shampoo_group& g) { return g.grad_dtype == CANZ_DT_BF16; }

struct Carve32 {   // float offsets into the workspace of one launch batch: the fp32 layout
  size_t gs, gt, tmp, lroot, rroot, a, x[2], m[2], t, t2, t4, partial, partial4, total_bytes;
};

Carve32 carve32(int64_t rows, int64_t cols, int nb) {
  const size_t rp = pad128(rows), cp = pad128(cols), dm = std::max(rp, cp);
  Carve32 c{};
  size_t off = 0;
  auto take = [&](size_t floats) {
    const size_t at = off;
    off += align_up(floats * sizeof(float)) / sizeof(float);
    return at;
  };
  c.gs = take(nb * rp * cp), c.gt = take(nb * rp * cp), c.tmp = take(nb * rp * cp);
  c.lroot = take(nb * rp * rp), c.rroot = take(nb * cp * cp);
  c.a = take(nb * dm * dm);
  c.x[0] = take(nb * dm * dm), c.x[1] = take(nb * dm * dm);
  c.m[0] = take(nb * dm * dm), c.m[1] = take(nb * dm * dm);
  c.t = take(nb * dm * dm), c.t2 = take(nb * dm * dm), c.t4 = take(nb * dm * dm);
  c.partial = take(static_cast<size_t>(nb) * NPART);
  c.partial4 = take(static_cast<size_t>(nb) * NPART);
  c.total_bytes = off * sizeof(float);
  return c;
}

// The three-term layout.  slot, left3, g3t: three bf16 terms per element, 1.5 floats.
struct Carve3 {
  size_t gs, gt, g3t, gp, gpt;         // G as its readers want it; gs, gt, gp are done with when the iteration begins
  size_t slot[2][5];                   // root iteration of each side; one set if the sides take turns
  size_t partial[2], partial4[2];
  size_t left3;                        // the sides take turns: the left root, kept over the right side's iteration
  size_t total_bytes;
};

Carve3 carve3(int64_t rows, int64_t cols, int nb, bool stat16, bool side_by_side) {
  const size_t rp2 = pad256(rows), cp2 = pad256(cols), plane = pad128(rows) * pad128(cols), p2 = nb * rp2 * cp2;
  Carve3 c{};
  size_t off = 0;
  auto take = [&](size_t floats) {
    const size_t at = off;
    off += align_up(floats * sizeof(float)) / sizeof(float);
    return at;
  };
  c.g3t = take(stat16 ? 0 : p2 * 3 / 2), c.gpt = take(stat16 ? p2 / 2 : 0);
  c.left3 = take(side_by_side ? 0 : nb * rp2 * rp2 * 3 / 2);
  const size_t begin = off;
  for (int side = 0; side < 2; ++side) {
    if (side == 1 && !side_by_side) {
      for (int k = 0; k < 5; ++k) c.slot[1][k] = c.slot[0][k];
      c.partial[1] = c.partial[0], c.partial4[1] = c.partial4[0];
      break;
    }
    const size_t d = side_by_side ? (side == 0 ? rp2 : cp2) : std::max(rp2, cp2), dd = nb * d * d;
    for (int k = 0; k < 5; ++k) c.slot[side][k] = take(dd * 3 / 2);
    c.partial[side] = take(static_cast<size_t>(nb) * NPART), c.partial4[side] = take(static_cast<size_t>(nb) * NPART);
  }
  const size_t end = off;
  off = begin;   // the statistics' operands, where the iteration will be
  c.gs = take(stat16 ? 0 : nb * plane), c.gt = take(stat16 ? 0 : nb * plane), c.gp = take(stat16 ? p2 / 2 : 0);
  c.total_bytes = std::max(off, end) * sizeof(float);
  return c;
}

// How a launch batch is computed.  With both sides' rounds side by side (TOGETHER) it is fastest: 4 x 1024 x 1024, 22 rounds
// 7.4 ms against 9.9 with the sides in turns (TURNS) and 13.8 in fp32 matrices on the fp32 MFMA (FP32), 4 x 384 x 384 2.7
// against 5.8 ms.  But three-term matrices padded to 256 can need more scratch than fp32 matrices padded to 128: square
// ones of one size 16 or 17 matrices instead of 13, up to 128 x 128 four times as much.  canz_shampoo_workspace_bytes asks for
// enough for the fastest; whatever suffices for the fp32 layout is accepted, and then the fastest that fits is taken, in
// smaller batches before in another way.
enum class Path { TOGETHER, TURNS, FP32 };
size_t batch_bytes(const canz_shampoo_group& g, int nb, Path p) {
  return p == Path::FP32 ? carve32(g.rows, g.cols, nb).total_bytes
                         : carve3(g.rows, g.cols, nb, bf16_statistics(g), p == Path::TOGETHER).total_bytes;
}
// matrices per batch: what the pointer tables and about 8 GB hold, at least one
int batch_cap(const canz_shampoo_group& g, Path p) {
  const int64_t by_bytes = std::max<int64_t>(1, static_cast<int64_t>(BATCH_BYTES / batch_bytes(g, 1, p)));
  return static_cast<int>(std::min<int64_t>({MAX_PTRS / g.tp, by_bytes, std::max<int64_t>(1, g.n_mats)}));
}
struct Plan {
  Path path;
  int nb;
};
Plan plan_of(const canz_shampoo_group& g, size_t have) {
  for (Path p : {Path::TOGETHER, Path::TURNS}) {   // one matrix of more than the batch memory: the sides in turns
    const int nb = batch_cap(g, p);
    if (batch_bytes(g, nb, p) <= (p == Path::TOGETHER ? std::min(have, BATCH_BYTES) : have)) return {p, nb};
  }
  for (Path p : {Path::TOGETHER, Path::TURNS})
    if (batch_bytes(g, 1, p) <= (p == Path::TOGETHER ? std::min(have, BATCH_BYTES) : have))
      return {p, std::min(batch_cap(g, p), static_cast<int>(std::min<size_t>(have, BATCH_BYTES) / batch_bytes(g, 1, p)))};
  return {Path::FP32, batch_cap(g, Path::FP32)};
}
size_t least_bytes(const canz_shampoo_group& g) { return batch_bytes(g, batch_cap(g, Path::FP32), Path::FP32); }

int check_hparams(const canz_shampoo_hparams* hp) {
  if (!hp) return fail(CANZ_EINVAL, "null hparams");
  if (hp->root_iters < 1) return fail(CANZ_EINVAL, "root_iters must be >= 1");
  if (!(hp->eps >= 0.f)) return fail(CANZ_EINVAL, "eps must be >= 0");
  if (hp->out_mode != CANZ_OUT_PARAM && hp->out_mode != CANZ_OUT_DELTA)
    return fail(CANZ_EUNSUPPORTED, "unknown out_mode %d", hp->out_mode);
  return CANZ_OK;
}

int check_group(const canz_shampoo_group& g, int idx, bool need_ptrs, int out_mode, bool keep_roots) {
  if (g.n_mats < 0) return fail(CANZ_EINVAL, "group %d: n_mats < 0", idx);
  if (g.rows < 1 || g.cols < 1) return fail(CANZ_EINVAL, "group %d: empty shape", idx);
  if (g.rows > MAX_EXTENT || g.cols > MAX_EXTENT)
    return fail(CANZ_ESHAPE, "group %d: extent above %lld", idx, static_cast<long long>(MAX_EXTENT));
  if (g.tp < 1 || g.tp > MAX_TP) return fail(CANZ_EINVAL, "group %d: tp must be in 1..%d", idx, MAX_TP);
  if (g.cols % g.tp) return fail(CANZ_ESHAPE, "group %d: cols not divisible by tp", idx);
  if (g.tp > 1 && (g.cols / g.tp) % 8) return fail(CANZ_ESHAPE, "group %d: fragment width not a multiple of 8", idx);
  if (g.grad_dtype != CANZ_DT_F32 && g.grad_dtype != CANZ_DT_BF16)
    return fail(CANZ_EUNSUPPORTED, "group %d: unknown grad_dtype", idx);
  if (g.out_dtype != CANZ_DT_F32 && g.out_dtype != CANZ_DT_BF16)
    return fail(CANZ_EUNSUPPORTED, "group %d: unknown out_dtype", idx);
  if (!need_ptrs || g.n_mats == 0) return CANZ_OK;
  if (!g.grad || !g.left || !g.right || !g.out) return fail(CANZ_EINVAL, "group %d: null pointer table", idx);
  if ((g.lroot == nullptr) != (g.rroot == nullptr)) return fail(CANZ_EINVAL, "group %d: one root table without the other", idx);
  if (keep_roots && !g.lroot) return fail(CANZ_EINVAL, "group %d: keep_roots needs the root tables", idx);
  const int n_out = out_mode == CANZ_OUT_DELTA ? g.n_mats * g.tp : g.n_mats;
  auto bad = [](const void* p) { return p == nullptr || (reinterpret_cast<uintptr_t>(p) & 15u) != 0; };
  for (int i = 0; i < g.n_mats * g.tp; ++i)
    if (bad(g.grad[i])) return fail(CANZ_EINVAL, "group %d: grad[%d] null or not 16-byte aligned", idx, i);
  for (int i = 0; i < g.n_mats; ++i)
    if (bad(g.left[i]) || bad(g.right[i]) || (g.lroot && (bad(g.lroot[i]) || bad(g.rroot[i]))))
      return fail(CANZ_EINVAL, "group %d: statistic or root %d null or not 16-byte aligned", idx, i);
  for (int i = 0; i < n_out; ++i)
    if (bad(g.out[i])) return fail(CANZ_EINVAL, "group %d: out[%d] null or not 16-byte aligned", idx, i);
  return CANZ_OK;
}

// what the kernels of one launch batch are told about it
struct BatchArgs {
  Shape s{};
  PtrTable grad{};
  OutSpec o{};
};
BatchArgs batch_args(const canz_shampoo_group& g, int first, int nb, const canz_shampoo_hparams& hp) {
  const int64_t rp = pad128(g.rows), cp = pad128(g.cols);
  BatchArgs a;
  Shape& s = a.s;
  s.rows = g.rows, s.cols = g.cols;
  s.m = std::min(g.rows, g.cols), s.n = std::max(g.rows, g.cols);
  s.mp = rp, s.np = cp;
  s.tall = g.rows > g.cols;
  s.tp = g.tp;
  s.wfrag = g.cols / g.tp;
  PtrTable& grad = a.grad;
  for (int i = 0; i < nb * g.tp; ++i) grad.p[i] = const_cast<void*>(g.grad[first * g.tp + i]);
  OutSpec& o = a.o;
  const int per_out = hp.out_mode == CANZ_OUT_DELTA ? g.tp : 1;
  for (int i = 0; i < nb * per_out; ++i) o.out.p[i] = g.out[first * per_out + i];
  o.out_dtype = g.out_dtype;
  o.out_mode = hp.out_mode;
  o.decay = static_cast<float>(1.0 - static_cast<double>(hp.lr) * static_cast<double>(hp.weight_decay));
  o.neg_lr_scale = -hp.lr;
  return a;
}

// One launch batch: matrices first .. first + nb - 1 of group g, everything on the fp32 MFMA.
int run_batch_f32(const canz_shampoo_group& g, int first, int nb, const canz_shampoo_hparams& hp, float* ws, hipStream_t st) {
  const int64_t rp = pad128(g.rows), cp = pad128(g.cols);
  const Carve32 c = carve32(g.rows, g.cols, nb);
  const BatchArgs args = batch_args(g, first, nb, hp);
  const Shape& s = args.s;
  const PtrTable& grad = args.grad;
  const OutSpec& o = args.o;
  const PtrTable none{};

  float *gs = ws + c.gs, *gt = ws + c.gt, *tmp = ws + c.tmp;
  {
    const dim3 grid(static_cast<unsigned>(cp / 64), static_cast<unsigned>(rp / 64), static_cast<unsigned>(nb));
    prof_mark(st, CANZ_KERNEL_SH_LOAD, true);
    hipLaunchKernelGGL(k_sh_load, grid, dim3(NTH), 0, st, s, grad, g.grad_dtype, rp, cp, gs, gt);
    prof_mark(st, CANZ_KERNEL_SH_LOAD, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "load kernel: %s", hipGetErrorString(e));
  }

  // one side: statistic (d x d, in the caller's buffers) from the operand `side` [dp][kp], then
  // its inverse fourth root into `root`
  auto one_side = [&](void* const* stat_tab, void* const* root_tab, int64_t d, int64_t dp, int64_t kp, const float* side,
                      float* root) -> int {
    PtrTable stat{}, kept{};
    for (int i = 0; i < nb; ++i) stat.p[i] = stat_tab[first + i];
    if (root_tab)
      for (int i = 0; i < nb; ++i) kept.p[i] = root_tab[first + i];
    Shape sq{};   // the d x d matrices of this side, for the padded load and the dense store of a kept root
    sq.rows = d, sq.cols = d, sq.tp = 1, sq.wfrag = d;
    const dim3 sq_tiles(static_cast<unsigned>(dp / 64), static_cast<unsigned>(dp / 64), static_cast<unsigned>(nb));
    const int64_t dd = dp * dp;
    float *a = ws + c.a, *x[2] = {ws + c.x[0], ws + c.x[1]}, *m[2] = {ws + c.m[0], ws + c.m[1]};
    float *tt = ws + c.t, *t2 = ws + c.t2, *t4 = ws + c.t4, *partial = ws + c.partial, *partial4 = ws + c.partial4;
    ShGemm q{};
    q.M = dp, q.N = dp, q.K = kp, q.ldp = kp, q.ldq = kp, q.sp = dp * kp, q.sq = dp * kp;
    q.P = side, q.Q = side, q.c = hp.keep_roots ? nullptr : a, q.d = d, q.beta = hp.beta, q.gscale = 1.f, q.eps = hp.eps;
    CANZ_HIP(CANZ_KERNEL_SH_STAT, (launch_gemm<SE_STAT, true>(q, nb, stat, s, o, st)), "statistics kernel");
    if (hp.keep_roots) {   // the caller's root, padded (its transposed image, which equals it, goes to a free buffer)
      prof_mark(st, CANZ_KERNEL_SH_LOAD, true);
      hipLaunchKernelGGL(k_sh_load, sq_tiles, dim3(NTH), 0, st, sq, kept, static_cast<int>(CANZ_DT_F32), dp, dp, root, x[0]);
      prof_mark(st, CANZ_KERNEL_SH_LOAD, false);
      if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "root load: %s", hipGetErrorString(e));
      return CANZ_OK;
    }
    auto prod = [&](const float* P, const float* Q, float* C) {
      ShGemm r{};
      r.M = dp, r.N = dp, r.K = dp, r.ldp = dp, r.ldq = dp, r.sp = dd, r.sq = dd;
      r.P = P, r.Q = Q, r.c = C;
      return r;
    };
    const unsigned init_blocks = static_cast<unsigned>(std::min<int64_t>(4096, (dd + NTH - 1) / NTH));
    prof_mark(st, CANZ_KERNEL_SH_INIT, true);
    hipLaunchKernelGGL(k_sh_sumsq_f32, dim3(NPART, nb), dim3(NTH), 0, st, a, dd, partial);
    hipLaunchKernelGGL(k_sh_prescale_f32, dim3(init_blocks, nb), dim3(NTH), 0, st, a, partial, dd, m[0]);
    prof_mark(st, CANZ_KERNEL_SH_INIT, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "root start: %s", hipGetErrorString(e));
    CANZ_HIP(CANZ_KERNEL_SH_ROOT, (launch_gemm<SE_PLAIN, true>(prod(m[0], m[0], t2), nb, none, s, o, st)), "root start (A A)");
    CANZ_HIP(CANZ_KERNEL_SH_ROOT, (launch_gemm<SE_PLAIN, true>(prod(t2, t2, t4), nb, none, s, o, st)), "root start (A2 A2)");
    prof_mark(st, CANZ_KERNEL_SH_INIT, true);
    hipLaunchKernelGGL(k_sh_sumsq_f32, dim3(NPART, nb), dim3(NTH), 0, st, t4, dd, partial4);
    hipLaunchKernelGGL(k_sh_init_f32, dim3(init_blocks, nb), dim3(NTH), 0, st, partial, partial4, dp, x[0], m[0], tt);
    prof_mark(st, CANZ_KERNEL_SH_INIT, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "root start: %s", hipGetErrorString(e));
    int cur = 0;
    for (int it = 0; it < hp.root_iters; ++it) {
      const bool last = it + 1 == hp.root_iters;
      CANZ_HIP(CANZ_KERNEL_SH_ROOT, (launch_gemm<SE_PLAIN, true>(prod(x[cur], tt, last ? root : x[cur ^ 1]), nb, none, s, o, st)),
               "root kernel (X T)");
      if (last) break;
      CANZ_HIP(CANZ_KERNEL_SH_ROOT, (launch_gemm<SE_PLAIN, true>(prod(tt, tt, t2), nb, none, s, o, st)), "root kernel (T T)");
      CANZ_HIP(CANZ_KERNEL_SH_ROOT, (launch_gemm<SE_PLAIN, true>(prod(t2, t2, t4), nb, none, s, o, st)), "root kernel (T2 T2)");
      ShGemm r = prod(t4, m[cur], m[cur ^ 1]);
      r.c2 = tt;
      CANZ_HIP(CANZ_KERNEL_SH_ROOT, (launch_gemm<SE_MT, true>(r, nb, none, s, o, st)), "root kernel (T4 M)");
      cur ^= 1;
    }
    if (root_tab) {
      prof_mark(st, CANZ_KERNEL_SH_LOAD, true);
      hipLaunchKernelGGL(k_unpad, sq_tiles, dim3(NTH), 0, st, sq, kept, root, dd, dp);
      prof_mark(st, CANZ_KERNEL_SH_LOAD, false);
      if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "root store: %s", hipGetErrorString(e));
    }
    return CANZ_OK;
  };
  float *lroot = ws + c.lroot, *rroot = ws + c.rroot;
  if (int rc = one_side(g.left, g.lroot, g.rows, rp, cp, gs, lroot)) return rc;
  if (int rc = one_side(g.right, g.rroot, g.cols, cp, rp, gt, rroot)) return rc;

  // O = (L^(-1/4) G) R^(-1/4): P = L root, Q = G^T gives rows x cols; then P = that, Q = R root
  ShGemm a1{};
  a1.M = rp, a1.N = cp, a1.K = rp, a1.ldp = rp, a1.ldq = rp, a1.sp = rp * rp, a1.sq = rp * cp;
  a1.P = lroot, a1.Q = gt, a1.c = tmp;
  CANZ_HIP(CANZ_KERNEL_SH_APPLY, (launch_gemm<SE_PLAIN, false>(a1, nb, none, s, o, st)), "preconditioning kernel (left)");
  ShGemm a2{};
  a2.M = rp, a2.N = cp, a2.K = cp, a2.ldp = cp, a2.ldq = cp, a2.sp = rp * cp, a2.sq = cp * cp;
  a2.P = tmp, a2.Q = rroot;
  CANZ_HIP(CANZ_KERNEL_SH_APPLY, (launch_gemm<SE_OUT, false>(a2, nb, none, s, o, st)), "preconditioning kernel (right)");
  return CANZ_OK;
}

// One launch batch: matrices first .. first + nb - 1 of group g, three bf16 terms per element.
int run_batch_terms(const canz_shampoo_group& g, int first, int nb, bool together, const canz_shampoo_hparams& hp, float* ws, hipStream_t st) {
  const int64_t rp = pad128(g.rows), cp = pad128(g.cols);
  const bool stat16 = bf16_statistics(g);
  const Carve3 c = carve3(g.rows, g.cols, nb, stat16, together);
  const BatchArgs args = batch_args(g, first, nb, hp);
  const Shape& s = args.s;
  const PtrTable& grad = args.grad;
  const OutSpec& o = args.o;

  float *gs = stat16 ? nullptr : ws + c.gs, *gt = stat16 ? nullptr : ws + c.gt;
  const int64_t rp2 = pad256(g.rows), cp2 = pad256(g.cols);
  __bf16 *gp = stat16 ? reinterpret_cast<__bf16*>(ws + c.gp) : nullptr, *gpt = stat16 ? reinterpret_cast<__bf16*>(ws + c.gpt) : nullptr;
  auto terms = [&](size_t at) { return reinterpret_cast<__bf16*>(ws + at); };
  {
    const dim3 grid(static_cast<unsigned>(cp2 / 64), static_cast<unsigned>(rp2 / 64), static_cast<unsigned>(nb));
    prof_mark(st, CANZ_KERNEL_SH_LOAD, true);
    hipLaunchKernelGGL(k_sh_load_grad, grid, dim3(NTH), 0, st, s, grad, g.grad_dtype, rp, cp, gs, gt, rp2, cp2, gp, gpt,
                       stat16 ? nullptr : terms(c.g3t));
    prof_mark(st, CANZ_KERNEL_SH_LOAD, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "load kernel: %s", hipGetErrorString(e));
  }

  // The two sides: statistic (d x d, in the caller's buffers) from the operand X, then its inverse fourth root.
  struct Side {
    PtrTable stat, kept;
    int64_t d, dp2;
    float *partial, *partial4;
    __bf16* slot[5];
    __bf16* root3;       // the root as three terms: where the iteration left it, or loaded from the caller
    bool keep;
  } side[2];
  for (int k = 0; k < 2; ++k) {
    Side& z = side[k];
    void* const* stat_tab = k == 0 ? g.left : g.right;
    void* const* root_tab = k == 0 ? g.lroot : g.rroot;
    z.keep = root_tab != nullptr;
    z.stat = PtrTable{}, z.kept = PtrTable{};
    for (int i = 0; i < nb; ++i) z.stat.p[i] = stat_tab[first + i], z.kept.p[i] = root_tab ? root_tab[first + i] : nullptr;
    z.d = k == 0 ? g.rows : g.cols, z.dp2 = k == 0 ? rp2 : cp2;
    z.partial = ws + c.partial[k], z.partial4 = ws + c.partial4[k];
    for (int q = 0; q < 5; ++q) z.slot[q] = terms(c.slot[k][q]);
    z.root3 = k == 0 && !together ? terms(c.left3) : nullptr;
    if (stat16) {
      if (int rc = statistic_bf16(CANZ_KERNEL_SH_STAT, z.stat, z.d, z.dp2, k == 0 ? cp2 : rp2, 1024, nb, hp.beta, 1.f, k == 0 ? gp : gpt, st))
        return rc;
    } else {
      const int64_t dp = k == 0 ? rp : cp, kp = k == 0 ? cp : rp;
      ShGemm q{};
      q.M = dp, q.N = dp, q.K = kp, q.ldp = kp, q.ldq = kp, q.sp = dp * kp, q.sq = dp * kp;
      q.P = k == 0 ? gs : gt, q.Q = q.P, q.c = nullptr, q.d = z.d, q.beta = hp.beta, q.gscale = 1.f, q.eps = 0.f;
      CANZ_HIP(CANZ_KERNEL_SH_STAT, (launch_gemm<SE_STAT, true>(q, nb, z.stat, s, o, st)), "statistics kernel");
    }
  }
  // The roots of the given sides, their rounds side by side.  Five matrices per side take turns: X, M and T, and two that
  // are free when a round begins.  X' and T^2 go there; T^4 takes X's place, M' that of T^2, the next T that of T.
  auto roots = [&](Side* const* z, int n) -> int {
    auto each = [&](int kind, const char* what, auto&& run) -> int {
      prof_mark(st, kind, true);
      for (int k = 0; k < n; ++k) run(*z[k]);
      prof_mark(st, kind, false);
      if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "%s: %s", what, hipGetErrorString(e));
      return CANZ_OK;
    };
    auto blocks = [](const Side& z_) { return static_cast<unsigned>(std::min<int64_t>(4096, z_.dp2 * z_.dp2 / 8 / NTH)); };
    GemmBatch gb{};
    auto add = [&](const Side& z_, const __bf16* P, const __bf16* Q, __bf16* C, __bf16* next_t) {
      GemmProblem& pr = gb.pr[gb.n++] = GemmProblem{};
      pr.d = split3_dims(z_.dp2, z_.dp2, z_.dp2, 3, nb), pr.p = P, pr.q = Q, pr.c = C, pr.ct = next_t;
    };
    auto launch = [&](const char* what) -> int {
      CANZ_HIP(CANZ_KERNEL_SH_ROOT, launch_split3_sym(gb, st), what);
      gb.n = 0;
      return CANZ_OK;
    };
    int x = 0, m = 1, f = 3, e = 4;
    const int t = 2;
    if (int rc = each(CANZ_KERNEL_SH_INIT, "root start", [&](Side& q) {
          hipLaunchKernelGGL(k_sh_sumsq, dim3(NPART, nb), dim3(NTH), 0, st, q.stat, q.d, hp.eps, q.partial);
          hipLaunchKernelGGL(k_sh_prescale, dim3(blocks(q), nb), dim3(NTH), 0, st, q.stat, q.d, q.dp2, hp.eps, q.partial, q.slot[m]);
        }))
      return rc;
    for (int k = 0; k < n; ++k) add(*z[k], z[k]->slot[m], z[k]->slot[m], z[k]->slot[f], nullptr);
    if (int rc = launch("root start (A A)")) return rc;
    for (int k = 0; k < n; ++k) add(*z[k], z[k]->slot[f], z[k]->slot[f], z[k]->slot[e], nullptr);
    if (int rc = launch("root start (A2 A2)")) return rc;
    if (int rc = each(CANZ_KERNEL_SH_INIT, "root start", [&](Side& q) {
          hipLaunchKernelGGL(k_sh_sumsq_terms, dim3(NPART, nb), dim3(NTH), 0, st, q.slot[e], q.dp2, q.partial4);
          hipLaunchKernelGGL(k_sh_init, dim3(blocks(q), nb), dim3(NTH), 0, st, q.partial, q.partial4, q.d, q.dp2, q.slot[x], q.slot[m],
                             q.slot[t]);
        }))
      return rc;
    for (int it = 0; it + 1 < hp.root_iters; ++it) {
      for (int k = 0; k < n; ++k) {
        __bf16* const* w = z[k]->slot;
        add(*z[k], w[x], w[t], w[f], nullptr), add(*z[k], w[t], w[t], w[e], nullptr);
      }
      if (int rc = launch("root kernel (X T, T T)")) return rc;
      for (int k = 0; k < n; ++k) add(*z[k], z[k]->slot[e], z[k]->slot[e], z[k]->slot[x], nullptr);
      if (int rc = launch("root kernel (T2 T2)")) return rc;
      for (int k = 0; k < n; ++k) add(*z[k], z[k]->slot[x], z[k]->slot[m], z[k]->slot[e], z[k]->slot[t]);
      if (int rc = launch("root kernel (T4 M)")) return rc;
      const int was_x = x, was_m = m;
      x = f, m = e, f = was_x, e = was_m;
    }
    for (int k = 0; k < n; ++k) {
      if (z[k]->root3 == nullptr) z[k]->root3 = z[k]->slot[f];
      add(*z[k], z[k]->slot[x], z[k]->slot[t], z[k]->root3, nullptr);
    }
    if (int rc = launch("root kernel (last X T)")) return rc;
    for (int k = 0; k < n; ++k) {
      if (!z[k]->keep) continue;
      const Side& q = *z[k];
      prof_mark(st, CANZ_KERNEL_SH_LOAD, true);
      hipLaunchKernelGGL(k_sh_store_terms, dim3(blocks(q), nb), dim3(NTH), 0, st, q.root3, q.kept, q.d, q.dp2);
      prof_mark(st, CANZ_KERNEL_SH_LOAD, false);
      if (hipError_t err = hipGetLastError(); err != hipSuccess) return fail(CANZ_EHIP, "root store: %s", hipGetErrorString(err));
    }
    return CANZ_OK;
  };
  if (hp.keep_roots) {   // the caller's roots as three terms
    for (int k = 0; k < 2; ++k) {
      Side& z = side[k];
      if (z.root3 == nullptr) z.root3 = z.slot[0];
      prof_mark(st, CANZ_KERNEL_SH_LOAD, true);
      const unsigned t64 = static_cast<unsigned>(z.dp2 / 64);
      hipLaunchKernelGGL(k_terms3, dim3(t64, t64, static_cast<unsigned>(nb)), dim3(NTH), 0, st, z.kept, z.d, z.d, z.dp2, z.root3);
      prof_mark(st, CANZ_KERNEL_SH_LOAD, false);
      if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "root load: %s", hipGetErrorString(e));
    }
  } else if (together) {
    Side* both[2] = {&side[0], &side[1]};
    if (int rc = roots(both, 2)) return rc;
  } else {
    for (Side& z : side) {
      Side* one = &z;
      if (int rc = roots(&one, 1)) return rc;
    }
  }
  // O = (L^(-1/4) G) R^(-1/4) on the bf16 cores, the roots and L^(-1/4) G as three terms per element (six products of
  // terms, three where G is bf16 itself): a step of 14 x 3072 x 1024 on kept roots 4.34 -> 2.26 ms against the fp32 MFMA.
  // L^(-1/4) G takes the place of the larger side's T (the roots lie in the free places, 0 or 3).
  __bf16* const tmp = side[rp2 >= cp2 ? 0 : 1].slot[2];
  // P = L root, Q = G^T gives rows x cols; then P = that, Q = R root
  const __bf16* gt_terms = stat16 ? gpt : terms(c.g3t);
  CANZ_HIP(CANZ_KERNEL_SH_APPLY, launch_split3(split3_dims(rp2, cp2, rp2, stat16 ? 1 : 3, nb), side[0].root3, gt_terms, tmp, st),
           "preconditioning kernel (left)");
  CANZ_HIP(CANZ_KERNEL_SH_APPLY, launch_terms_final(split3_dims(rp2, cp2, cp2, 3, nb), tmp, side[1].root3, s, o, st),
           "preconditioning kernel (right)");
  return CANZ_OK;
}

// Consecutive groups of a call that agree in shape, tp, dtypes and in which tables they pass run as one group: every
// matrix is computed on its own whatever shares its launch, and the products of small matrices fill the chip only
// when many of them share one.
struct MergedGroup {
  canz_shampoo_group g{};
  std::vector<const void*> grad;
  std::vector<void*> tab[5];   // left, right, out, lroot, rroot
};

void tables_of(const canz_shampoo_group& g, void* const* (&out)[5]) {
  out[0] = g.left, out[1] = g.right, out[2] = g.out, out[3] = g.lroot, out[4] = g.rroot;
}

bool mergeable(const canz_shampoo_group& a, const canz_shampoo_group& b) {
  if (a.rows != b.rows || a.cols != b.cols || a.tp != b.tp || a.grad_dtype != b.grad_dtype || a.out_dtype != b.out_dtype) return false;
  if ((a.grad == nullptr) != (b.grad == nullptr)) return false;
  void* const* ta[5];
  void* const* tb[5];
  tables_of(a, ta), tables_of(b, tb);
  for (int k = 0; k < 5; ++k)
    if ((ta[k] == nullptr) != (tb[k] == nullptr)) return false;
  return true;
}

std::vector<MergedGroup> merge_groups(const canz_shampoo_group* g, int n_groups, int out_mode) {
  std::vector<MergedGroup> all;
  for (int i = 0; i < n_groups; ++i) {
    const canz_shampoo_group& x = g[i];
    if (x.n_mats == 0) continue;
    if (all.empty() || !mergeable(all.back().g, x)) {
      all.emplace_back();
      all.back().g = x;
      all.back().g.n_mats = 0;
    }
    MergedGroup& m = all.back();
    void* const* t[5];
    tables_of(x, t);
    const int per_out = out_mode == CANZ_OUT_DELTA ? x.tp : 1;
    if (x.grad) m.grad.insert(m.grad.end(), x.grad, x.grad + static_cast<size_t>(x.n_mats) * x.tp);
    for (int k = 0; k < 5; ++k)
      if (t[k]) m.tab[k].insert(m.tab[k].end(), t[k], t[k] + static_cast<size_t>(x.n_mats) * (k == 2 ? per_out : 1));
    m.g.n_mats += x.n_mats;
  }
  for (MergedGroup& m : all) {   // the tables now stand still: point the group at them
    canz_shampoo_group& x = m.g;
    if (x.grad) x.grad = m.grad.data();
    if (x.left) x.left = m.tab[0].data();
    if (x.right) x.right = m.tab[1].data();
    if (x.out) x.out = m.tab[2].data();
    if (x.lroot) x.lroot = m.tab[3].data();
    if (x.rroot) x.rroot = m.tab[4].data();
  }
  return all;
}

}  // namespace
}  // namespace canz

extern "C" int canz_shampoo_workspace_bytes(const canz_shampoo_group* g, int32_t n_groups, const canz_shampoo_hparams* hp,
                                            size_t* bytes_out) {
  using namespace canz;
  if (!bytes_out) return fail(CANZ_EINVAL, "null bytes_out");
  if (n_groups < 0 || (n_groups > 0 && !g)) return fail(CANZ_EINVAL, "bad group array");
  if (int rc = check_hparams(hp)) return rc;
  size_t need = ALIGN;
  for (int i = 0; i < n_groups; ++i)
    if (int rc = check_group(g[i], i, false, hp->out_mode, hp->keep_roots != 0)) return rc;
  for (const MergedGroup& m : merge_groups(g, n_groups, hp->out_mode))
    if (const Plan p = plan_of(m.g, SIZE_MAX); m.g.n_mats > 0)
      need = std::max({need, batch_bytes(m.g, p.nb, p.path), least_bytes(m.g)});
  *bytes_out = need;
  return CANZ_OK;
}

extern "C" int canz_shampoo_step(const canz_shampoo_group* g, int32_t n_groups, const canz_shampoo_hparams* hp,
                                 void* workspace, size_t workspace_bytes, void* hip_stream) {
  using namespace canz;
  size_t need = 0;   // of the fastest way; checks the arguments
  if (int rc = canz_shampoo_workspace_bytes(g, n_groups, hp, &need)) return rc;
  bool any = false;
  for (int i = 0; i < n_groups; ++i) {
    if (int rc = check_group(g[i], i, true, hp->out_mode, hp->keep_roots != 0)) return rc;
    any = any || g[i].n_mats > 0;
  }
  if (!any) return CANZ_OK;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (ALIGN - 1)))
    return fail(CANZ_EWORKSPACE, "workspace null or not 256-byte aligned");
  const std::vector<MergedGroup> merged = merge_groups(g, n_groups, hp->out_mode);
  for (const MergedGroup& m : merged)
    if (workspace_bytes < least_bytes(m.g))
      return fail(CANZ_EWORKSPACE, "workspace too small: %zu bytes given, %zu needed", workspace_bytes, need);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  float* ws = static_cast<float*>(workspace);
  for (const MergedGroup& m : merged) {
    const Plan p = plan_of(m.g, workspace_bytes);
    for (int first = 0; first < m.g.n_mats; first += p.nb) {
      const int nb = std::min(p.nb, m.g.n_mats - first);
      const int rc = p.path == Path::FP32 ? run_batch_f32(m.g, first, nb, *hp, ws, st)
                                          : run_batch_terms(m.g, first, nb, p.path == Path::TOGETHER, *hp, ws, st);
      if (rc) return rc;
    }
  }
  return CANZ_OK;
}
