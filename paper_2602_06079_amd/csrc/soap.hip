// canz_soap_step / canz_soap_workspace_bytes: the SOAP step the paper runs through the same
// planner as Muon and Shampoo ("Generalization to Other Optimizers (Shampoo & SOAP)", App. C;
// App. B.3), per matrix (Adam in the eigenbasis of Shampoo's statistics):
//   M <- beta1 M + (1 - beta1) G;   G' = Q_L^T G Q_R,  M' = Q_L^T M Q_R;
//   V <- beta2 V + (1 - beta2) G'^2;   N' = m / (sqrt(v) + eps);   N = Q_L N' Q_R^T;
//   P <- P (1 - lr wd) - lr N  (or Delta W = -lr N);
//   L <- beta2 L + (1 - beta2) G G^T,  R <- beta2 R + (1 - beta2) G^T G;
//   on a refresh step  Q_L <- orthogonal factor of QR(L Q_L),  Q_R likewise.
// State and sums are fp32.  On the bf16 matrix cores (the kernels of the Muon step, operands in its panel layout) run
// the rotations, on fp32 values held as three bf16 terms (or, if the caller asks for it with bf16_rotations, with the
// bases, M and N' rounded to bf16), and the statistics of gradients that arrive as bf16 (their own values are the
// operands, every product is exact in fp32).  The statistics of fp32 gradients and the refresh run on
// v_mfma_f32_32x32x2_f32, but for the refresh's product S Q, which runs on three bf16 terms where the rotations do (an infinity in a
// statistic gives NaN there).
//
// The products all take the form C[i][j] = sum_k P[i][k] Q[j][k].  The rotation into the basis
// runs right side first with its result written transposed, (G Q_R)^T = Q_R^T-rows times G-rows,
// so that the left side finds its second operand contiguous along k; the rotation back runs
// the same way round.  G is rotated first, then M; with a rotated momentum kept by the caller (mom_rot) only G is rotated
// and M' follows M' <- beta1 M' + (1 - beta1) G' in the Adam kernel.
//
// QR refresh: blocked Householder factorisation with panels of 32 columns in blocks of 128, on the transposed
// matrix (a column of S = L Q is a contiguous row of the working copy), both sides of a batch in the same launches.  One workgroup
// per matrix finds the 32 reflectors of a panel (each wavefront owns whole columns); the products with them, and with the 128 of a
// block (compact WY form H = I - V T V^T), run on the whole chip.  Afterwards the orthogonal factor is accumulated from the last block
// to the first with the same two products (and T^T).  Tile boundaries of these products are rounded down to multiples of 128;
// the extra rows and columns they touch either hold zeros in V (no effect) or are columns the
// factorisation has finished with (R is never needed: only Q is).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>
#include <vector>

#include "canz.h"
#include "canz_internal.h"
#include "device_util.h"
#include "f32_mfma_gemm.h"
#include "kernels.h"

namespace canz {
namespace {

using namespace f32mfma;

constexpr int64_t MAX_EXTENT = 32768;
constexpr size_t BATCH_BYTES = size_t(32) << 30;   // working matrices of one launch batch: the more matrices share
                                                     // a batch, the more workgroups the panel kernel of a refresh has
constexpr int QB = 32;            // panel width of the QR factorisation
constexpr int QTH = 1024;         // threads of the panel kernel: 16 wavefronts
constexpr int QWAVES = QTH / 64;

// Where k_soap_load leaves its results: fp32 working copies and / or bf16 images in the panel layout
// (panel_layout.h; padded to multiples of 256, operands of the bf16 MFMA kernels), each in both orientations.
struct LoadOut {
  float *gm, *gmt, *mm, *mmt;    // fp32 G [rp][cp] and G^T [cp][rp] of each matrix, `stride` floats apart, and M; nullptr: not wanted
  int64_t stride;
  __bf16 *g3, *g3t, *m3, *m3t;   // three bf16 terms: G [nb][rp2][3 cp2], G^T [nb][cp2][3 rp2], M, M^T; nullptr: not wanted
  __bf16 *gp, *gpt, *mp, *mpt;   // bf16 panels: G [nb][rp2][cp2], G^T [nb][cp2][rp2], M, M^T; nullptr: not wanted
  int64_t rp2, cp2;
};

// G (bf16 or fp32, whole or tp column fragments) and the momentum M <- beta1 M + (1 - beta1) G
// (fp32, dense, in the caller's buffer) -> working copies of both as `w` asks, zero outside rows x cols.
// One block per 64 x 64 tile of the matrix padded to multiples of 256.
// VEC: cols and cols / tp are multiples of 8, so a lane's 8 consecutive elements lie in one fragment and every
// access of the caller's arrays is a 16-byte vector.
template <bool VEC>
__global__ __launch_bounds__(NTH) void k_soap_load(Shape s, PtrTable grad, int grad_dtype, PtrTable mom, float beta1,
                                                    int64_t rp, int64_t cp, LoadOut w) {
  __shared__ float tg[64][65], tm[64][65];
  const int b = blockIdx.z, r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
  const int wf = static_cast<int>(s.wfrag);
  float* gs = w.gm ? w.gm + b * w.stride : nullptr;
  float* gt = w.gm ? w.gmt + b * w.stride : nullptr;
  float* ms = w.mm ? w.mm + b * w.stride : nullptr;
  float* mt = w.mm ? w.mmt + b * w.stride : nullptr;
  float* m = static_cast<float*>(mom.p[b]);
  if (VEC) {
    const int cv = (t & 7) * 8;
    f32x4 gv[2][2], mv[2][2];
    bool live[2];
#pragma unroll
    for (int half = 0; half < 2; ++half) {   // all loads first: the tables may alias as far as the compiler knows
      const int row = r0 + (t >> 3) + half * 32, col = c0 + cv;
      live[half] = row < s.rows && col < s.cols;
      gv[half][0] = gv[half][1] = mv[half][0] = mv[half][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (!live[half]) continue;
      const int f = col / wf;
      const int64_t at = static_cast<int64_t>(row) * wf + (col - f * wf);
      if (grad_dtype == CANZ_DT_BF16) {
        const bf16x8 g8 = *reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(grad.p[b * s.tp + f]) + at);
#pragma unroll
        for (int e = 0; e < 4; ++e) gv[half][0][e] = static_cast<float>(g8[e]), gv[half][1][e] = static_cast<float>(g8[4 + e]);
      } else {
        const f32x4* g4 = reinterpret_cast<const f32x4*>(static_cast<const float*>(grad.p[b * s.tp + f]) + at);
        gv[half][0] = g4[0], gv[half][1] = g4[1];
      }
      const f32x4* m4 = reinterpret_cast<const f32x4*>(m + static_cast<int64_t>(row) * s.cols + col);
      mv[half][0] = m4[0], mv[half][1] = m4[1];
    }
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int rl = (t >> 3) + half * 32, row = r0 + rl, col = c0 + cv;
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          mv[half][q][e] = live[half] ? __builtin_fmaf(beta1, mv[half][q][e], (1.f - beta1) * gv[half][q][e]) : 0.f;
          tg[rl][cv + 4 * q + e] = gv[half][q][e];
          tm[rl][cv + 4 * q + e] = mv[half][q][e];
        }
      if (live[half]) {
        f32x4* m4 = reinterpret_cast<f32x4*>(m + static_cast<int64_t>(row) * s.cols + col);
        m4[0] = mv[half][0], m4[1] = mv[half][1];
      }
      if (row < rp && col < cp) {
        if (gs) {
          f32x4* o = reinterpret_cast<f32x4*>(gs + static_cast<int64_t>(row) * cp + col);
          o[0] = gv[half][0], o[1] = gv[half][1];
        }
        if (ms) {
          f32x4* o = reinterpret_cast<f32x4*>(ms + static_cast<int64_t>(row) * cp + col);
          o[0] = mv[half][0], o[1] = mv[half][1];
        }
      }
    }
  } else {
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;
    const int row = r0 + r, col = c0 + c;
    float g = 0.f, mv = 0.f;
    if (row < s.rows && col < s.cols) {
      const int f = col / wf;
      const int64_t at = static_cast<int64_t>(row) * wf + (col - f * wf);
      g = grad_dtype == CANZ_DT_BF16 ? static_cast<float>(static_cast<const __bf16*>(grad.p[b * s.tp + f])[at])
                                     : static_cast<const float*>(grad.p[b * s.tp + f])[at];
      const int64_t am = static_cast<int64_t>(row) * s.cols + col;
      mv = __builtin_fmaf(beta1, m[am], (1.f - beta1) * g);
      m[am] = mv;
    }
    if (row < rp && col < cp) {
      if (gs) gs[static_cast<int64_t>(row) * cp + col] = g;
      if (ms) ms[static_cast<int64_t>(row) * cp + col] = mv;
    }
    tg[r][c] = g;
    tm[r][c] = mv;
  }
  }
  __syncthreads();
  if (gs || ms) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;  // r: column of G, c: row of G
      if (c0 + r < cp && r0 + c < rp) {
        if (gs) gt[static_cast<int64_t>(c0 + r) * rp + r0 + c] = tg[c][r];
        if (ms) mt[static_cast<int64_t>(c0 + r) * rp + r0 + c] = tm[c][r];
      }
    }
  }
  const int64_t p2 = static_cast<int64_t>(b) * w.rp2 * w.cp2;
  if (w.gp) tile_to_panels(tg, w.gp + p2, r0, c0, w.cp2, false, t);
  if (w.gpt) tile_to_panels(tg, w.gpt + p2, r0, c0, w.rp2, true, t);
  if (w.mp) tile_to_panels(tm, w.mp + p2, r0, c0, w.cp2, false, t);
  if (w.mpt) tile_to_panels(tm, w.mpt + p2, r0, c0, w.rp2, true, t);
  if (w.g3) tile_to_terms3(tg, w.g3 + 3 * p2, r0, c0, w.cp2, false, t);
  if (w.g3t) tile_to_terms3(tg, w.g3t + 3 * p2, r0, c0, w.rp2, true, t);
  if (w.m3) tile_to_terms3(tm, w.m3 + 3 * p2, r0, c0, w.cp2, false, t);
  if (w.m3t) tile_to_terms3(tm, w.m3t + 3 * p2, r0, c0, w.rp2, true, t);
}

// Adam in the rotated space.  G' and (unless `incremental`) M' are fp32 of row length `ld`, `stride` floats apart; V (dense, caller's)
// is updated in place; N' = (c1 M') / (sqrt(c2 V) + eps) leaves as three bf16 terms per element, [rp2][3 cp2] panels or
// transposed [cp2][3 rp2] (np), or in fp32, [rp][cp] or transposed [cp][rp] (n32), zero outside rows x cols.  If the caller
// keeps the rotated momentum (`keep`, dense, mrot): incremental: M' = beta1 mrot + (1 - beta1) G'; either way mrot <- M'.
__global__ __launch_bounds__(NTH) void k_soap_adam(Shape s, PtrTable var, PtrTable mrot, bool keep, bool incremental,
                                                    const float* __restrict__ grot, const float* __restrict__ m_rot, int64_t ld, int64_t stride,
                                                    int64_t rp2, int64_t cp2, float beta1, float beta2, float c1, float c2, float eps,
                                                    int transposed, __bf16* __restrict__ np, float* __restrict__ n32) {
  __shared__ float tile[64][65];
  const int b = blockIdx.z, r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
  const int64_t at = b * stride;
  const float* gr = grot + at;
  float* v = static_cast<float*>(var.p[b]);
  float* mr = static_cast<float*>(mrot.p[b]);
  float go[16], vo[16], mo[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {   // all old values first: one memory latency for the tile
    const int idx = e * NTH + t, row = r0 + (idx >> 6), col = c0 + (idx & 63);
    const bool in = row < s.rows && col < s.cols;
    const int64_t av = static_cast<int64_t>(row) * s.cols + col, ar = row * ld + col;
    go[e] = in ? gr[ar] : 0.f;
    vo[e] = in ? v[av] : 0.f;
    mo[e] = !in ? 0.f : incremental ? mr[av] : m_rot[at + ar];
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63, row = r0 + r, col = c0 + c;
    float n = 0.f;
    if (row < s.rows && col < s.cols) {
      const int64_t av = static_cast<int64_t>(row) * s.cols + col;
      const float g = go[e];
      const float m = incremental ? __builtin_fmaf(beta1, mo[e], (1.f - beta1) * g) : mo[e];
      if (keep) mr[av] = m;
      const float vn = __builtin_fmaf(beta2, vo[e], (1.f - beta2) * (g * g));
      v[av] = vn;
      n = (c1 * m) / (sqrtf(c2 * vn) + eps);
    }
    tile[r][c] = n;
  }
  __syncthreads();
  if (n32) {
    const int64_t rp = s.mp, cp = s.np;   // the fp32 padding
    float* out = n32 + b * rp * cp;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;
      if (transposed) {
        if (c0 + r < cp && r0 + c < rp) out[(c0 + r) * rp + r0 + c] = tile[c][r];
      } else if (r0 + r < rp && c0 + c < cp) {
        out[(r0 + r) * cp + c0 + c] = tile[r][c];
      }
    }
    return;
  }
  tile_to_terms3(tile, np + static_cast<int64_t>(b) * 3 * rp2 * cp2, r0, c0, transposed ? rp2 : cp2, transposed != 0, t);
}

// The caller's basis Q (d x d, dense fp32) -> what its readers want, zero outside d x d, in both orientations: fp32 [dp][dp]
// (transposed also for the refresh), bf16 panels [dp2][dp2] or three bf16 terms [dp2][3 dp2]; nullptr: not
// wanted.  One block per 64 x 64 tile of the larger padding.
struct BasisOut {
  float *s32, *t32;
  __bf16 *sp, *tp, *s3, *t3;
};
__global__ __launch_bounds__(NTH) void k_soap_load_basis(PtrTable q, int64_t d, int64_t dp, int64_t dp2, BasisOut w) {
  __shared__ float tile[64][65];
  const int b = blockIdx.z, r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
  const float* src = static_cast<const float*>(q.p[b]);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;
    const int64_t row = r0 + r, col = c0 + c;
    const float val = row < d && col < d ? src[row * d + col] : 0.f;
    if (w.s32 && row < dp && col < dp) w.s32[(b * dp + row) * dp + col] = val;
    tile[r][c] = val;
  }
  __syncthreads();
  if (w.t32) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;  // r: column of Q, c: row of Q
      if (c0 + r < dp && r0 + c < dp) w.t32[(b * dp + c0 + r) * dp + r0 + c] = tile[c][r];
    }
  }
  const int64_t p2 = b * dp2 * dp2;
  if (w.sp) tile_to_panels(tile, w.sp + p2, r0, c0, dp2, false, t);
  if (w.tp) tile_to_panels(tile, w.tp + p2, r0, c0, dp2, true, t);
  if (w.s3) tile_to_terms3(tile, w.s3 + 3 * p2, r0, c0, dp2, false, t);
  if (w.t3) tile_to_terms3(tile, w.t3 + 3 * p2, r0, c0, dp2, true, t);
}

// Adam in the rotated space on bf16 panels: G' (and, unless `incremental`, M') [rp2][cp2] panels in, N' panels
// out, straight [rp2][cp2] and / or transposed [cp2][rp2], zero outside rows x cols; V and the kept rotated
// momentum are the caller's dense fp32 arrays as in k_soap_adam.  One block per 64 x 64 tile: the panel chunks
// (8 consecutive elements of a row) go through LDS so that the dense fp32 arrays are read and written with one
// row of 64 elements per wavefront, whatever the row length of the caller's matrix.
__global__ __launch_bounds__(NTH) void k_soap_adam_bf16(Shape s, PtrTable var, PtrTable mrot, bool keep, bool incremental,
                                                         const __bf16* __restrict__ grot, const __bf16* __restrict__ mrot_p,
                                                         int64_t rp2, int64_t cp2, float beta1, float beta2, float c1,
                                                         float c2, float eps, __bf16* __restrict__ n_straight,
                                                         __bf16* __restrict__ n_transposed) {
  __shared__ float tg[64][65], tm[64][65];
  const int b = blockIdx.z, r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
  const int64_t plane = rp2 * cp2;
  const __bf16* gp = grot + static_cast<int64_t>(b) * plane;
  float* v = static_cast<float*>(var.p[b]);
  float* mr = static_cast<float*>(mrot.p[b]);
  const int cv = (t & 7) * 8;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int rl = (t >> 3) + half * 32;
    const int64_t at = panel_chunk_off(r0 + rl, c0 + cv, cp2);
    const bf16x8 g8 = *reinterpret_cast<const bf16x8*>(gp + at);
#pragma unroll
    for (int e = 0; e < 8; ++e) tg[rl][cv + e] = static_cast<float>(g8[e]);
    if (!incremental) {
      const bf16x8 m8 = *reinterpret_cast<const bf16x8*>(mrot_p + static_cast<int64_t>(b) * plane + at);
#pragma unroll
      for (int e = 0; e < 8; ++e) tm[rl][cv + e] = static_cast<float>(m8[e]);
    }
  }
  __syncthreads();
  float vo[16], mo[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {   // all old values first: one memory latency for the tile
    const int idx = e * NTH + t, row = r0 + (idx >> 6), col = c0 + (idx & 63);
    const bool in = row < s.rows && col < s.cols;
    const int64_t av = static_cast<int64_t>(row) * s.cols + col;
    vo[e] = in ? v[av] : 0.f;
    mo[e] = in && incremental ? mr[av] : 0.f;
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63, row = r0 + r, col = c0 + c;
    float n = 0.f;
    if (row < s.rows && col < s.cols) {
      const int64_t av = static_cast<int64_t>(row) * s.cols + col;
      const float g = tg[r][c];
      const float m = incremental ? __builtin_fmaf(beta1, mo[e], (1.f - beta1) * g) : tm[r][c];
      if (keep) mr[av] = m;
      const float vn = __builtin_fmaf(beta2, vo[e], (1.f - beta2) * (g * g));
      v[av] = vn;
      n = (c1 * m) / (sqrtf(c2 * vn) + eps);
    }
    tg[r][c] = n;   // the element this thread read
  }
  __syncthreads();
  if (n_straight) tile_to_panels(tg, n_straight + static_cast<int64_t>(b) * plane, r0, c0, cp2, false, t);
  if (n_transposed) tile_to_panels(tg, n_transposed + static_cast<int64_t>(b) * plane, r0, c0, rp2, true, t);
}

// a[b][i] = (identity ? (row == col) : 0) for the [rows][ld] matrices of a batch
__global__ __launch_bounds__(NTH) void k_soap_fill(float* __restrict__ a, int64_t elems, int64_t ld, int identity) {
  float* ab = a + static_cast<int64_t>(blockIdx.y) * elems;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * NTH + threadIdx.x; i < elems; i += static_cast<int64_t>(gridDim.x) * NTH)
    ab[i] = identity && (i / ld) == (i % ld) ? 1.f : 0.f;
}

// Caller's basis Q (d x d, dense, columns are the vectors) <- the transposed working copy qt [dp][dp].
__global__ __launch_bounds__(NTH) void k_soap_store_q(PtrTable q, const float* __restrict__ qt, int64_t d, int64_t dp) {
  __shared__ float tile[64][65];
  const int b = blockIdx.z, r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
  const float* src = qt + static_cast<int64_t>(b) * dp * dp;
  float* dst = static_cast<float*>(q.p[b]);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;
    tile[r][c] = src[static_cast<int64_t>(r0 + r) * dp + c0 + c];   // qt[col of Q][row of Q]
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;
    const int row = c0 + r, col = r0 + c;                          // row / column of Q
    if (row < d && col < d) dst[static_cast<int64_t>(row) * d + col] = tile[c][r];
  }
}

// The QR refresh: blocked Householder factorisation of S Q_old, on the transposed matrix (column c is row c of wk, row length
// dp), and the accumulation of its orthogonal factor.  Blocks of 128 columns, four panels of 32 each:
//   k_qr_panel_*   one workgroup per matrix finds the 32 reflectors of a panel,  vall row j0 + c <- v_c,  tau
//   k_qr_gram      V_a^T V for the panels a of the block so far and W = (later columns of the block)^T V, in pieces of k
//   k_qr_panel_sub sums the pieces and applies the panel to the block's later columns:  X -= W' V^T
//   k_qr_block_t   (after the fourth panel) T of the whole block from the V_a^T V:  H_0 ... H_127 = I - V T V^T
//   k_qr_block_w   W' = (X V) T of the rows X beyond the block, k_qr_sub  X -= W' V^T: the trailing matrix goes through memory once per block
// and, from the last block to the first, the latter two again on Q^T with T^T.  For a row x of X, x H_0 H_1 ... = x - w' V^T, where w' = (x V) T
// solves w'_c = tau_c (w_c - sum_{l < c} w'_l v_l^T v_c), w = x V: 32 steps by a thread per row inside the block.
// Both sides of a batch run in the same launches: the chain of panels is a chain of latencies, with a workgroup per matrix busy.
// 4 x 2048x1024, both sides: 17.9 ms with the sides one after the other, T, Y = V T^T and V T formed by one workgroup per matrix and panel
// (33 us each, the panel itself 47), and the products W on one workgroup per 128 rows (60 of 256 CUs in the longest: 129 us).
constexpr int QBLK = 128;   // columns of a block: four panels
constexpr int QCHUNKS = 16; // pieces of k in the products with one panel: at most this many, of 128 or more
struct QrSide {
  float* wk;       // [nb][dp][dp]
  float* vall;     // [nb][dp][dp]
  float* qt;       // [nb][dp][dp]  Q^T
  float* tau;      // [nb][128] of the block under way
  float* strip;    // [nb][dp][128]: pieces of the products with one panel, W' of a block
  float* gram;     // [nb][128][128]: V_a^T V_b of the block under way (a <= b), then its T
  float* tt;       // [nb][dp / 128][128][128]: T^T of every block
  int dp, d;
};
struct QrArgs {
  QrSide side[2];
  int nb;          // matrices of a side; matrix m of a launch is number m % nb of side m / nb
  int jb;          // first column of the block
  int pos;         // panel of the block
};
struct QrMatrix {  // one matrix of a launch
  float *wk, *vall, *qt, *tau, *strip, *gram, *tt;
  int dp, d;
};
__device__ __forceinline__ QrMatrix qr_matrix(const QrArgs& a, int m) {
  const QrSide& s = a.side[m >= a.nb ? 1 : 0];
  const int64_t b = m >= a.nb ? m - a.nb : m, dd = static_cast<int64_t>(s.dp) * s.dp;
  return QrMatrix{s.wk + b * dd, s.vall + b * dd, s.qt + b * dd, s.tau + b * QBLK, s.strip + b * s.dp * QBLK,
                  s.gram + b * QBLK * QBLK, s.tt + b * s.dp * QBLK, s.dp, s.d};
}
// the pieces of k that the products with one panel of the block are cut into
__device__ __forceinline__ void qr_chunks(int dp, int jb, int& count, int& len) {
  const int units = (dp - jb) / 128, per = (units + QCHUNKS - 1) / QCHUNKS;
  count = (units + per - 1) / per, len = per * 128;
}

constexpr int VMAX = 12288;   // rows of a reflector kept in LDS: the largest extent a side with a basis may have

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// tau and the scale of v for a column with diagonal element al and sum of squares ss below it.  The root and the quotients are on the
// chain of every column: from the chip's estimates with a step of Newton's method each (and the quotient's remainder), which leaves what rounding
// leaves, in a third of the time of the library's, except where the squares are close to the smallest numbers there are.  Not in the
// kernels for long columns (REFINED = false), which have no registers for it.
__device__ __forceinline__ float refined_rcp(float x, float r) { return __builtin_fmaf(__builtin_fmaf(-x, r, 1.f), r, r); }
template <bool REFINED = true>
__device__ __forceinline__ void reflector_of(bool live, float ss, float al, float& tau, float& scale) {
  tau = 0.f, scale = 0.f;
  if (live && ss > 0.f) {
    const float x2 = __builtin_fmaf(al, al, ss);
    if (REFINED && x2 > 1e-30f) {
      const float y = __builtin_amdgcn_rsqf(x2);
      float nrm = x2 * y;
      nrm = __builtin_fmaf(__builtin_fmaf(-nrm, nrm, x2), 0.5f * y, nrm);
      const float inv = refined_rcp(nrm, y);
      const float sum = nrm + fabsf(al);   // |al - beta|, beta = -sign(al) nrm
      const float q = sum * inv;
      tau = __builtin_fmaf(__builtin_fmaf(-nrm, q, sum), inv, q);
      const float r = refined_rcp(sum, __builtin_amdgcn_rcpf(sum));
      scale = al >= 0.f ? r : -r;
    } else {
      const float nrm = sqrtf(x2);
      const float beta = al >= 0.f ? -nrm : nrm;
      tau = (beta - al) / beta;
      scale = 1.f / (al - beta);
    }
  }
}
// the element at row c < 32 of a column whose lane l holds rows 4 l .. 4 l + 3 in k
__device__ __forceinline__ float element_of(const f32x4& k, int c) {
  const float v = (c & 2) ? ((c & 1) ? k[3] : k[2]) : ((c & 1) ? k[1] : k[0]);
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), c >> 2));
}
// sum of squares of a lane's elements below row c; the rows up to c < 32 lie in the first slot
template <int XS>
__device__ __forceinline__ float squares_below(const f32x4 (&k)[XS], int lane, int c) {
  float ss = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x = 4 * lane + e > c ? k[0][e] : 0.f;
    ss = __builtin_fmaf(x, x, ss);
  }
#pragma unroll
  for (int sl = 1; sl < XS; ++sl)
#pragma unroll
    for (int e = 0; e < 4; ++e) ss = __builtin_fmaf(k[sl][e], k[sl][e], ss);
  return ss;
}
// elements 4 q .. 4 q + 3 of v_c from those of the column
__device__ __forceinline__ f32x4 v_of(const f32x4& x, int q, int c, float scale) {
  f32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = 4 * q + e;
    o[e] = r < c ? 0.f : (r == c ? 1.f : x[e] * scale);
  }
  return o;
}

// Sum over the 64 lanes through the data-parallel-primitive lanes of the vector ALU (no LDS crossbar
// round trips, which dominate a step of the register-resident panel kernel otherwise): an inclusive scan
// inside each row of 16 lanes (shifts by 1, 2, 4, 8, out-of-row sources read as 0), then the row totals
// are carried into the following rows (row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3);
// lane 63 holds the total, which every lane receives.
template <int CTRL, int ROW_MASK, bool BOUND>
__device__ __forceinline__ float dpp_mov(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, BOUND));
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
  v += dpp_mov<0x111, 0xf, true>(v);    // row_shr:1
  v += dpp_mov<0x112, 0xf, true>(v);    // row_shr:2
  v += dpp_mov<0x114, 0xf, true>(v);    // row_shr:4
  v += dpp_mov<0x118, 0xf, true>(v);    // row_shr:8
  v += dpp_mov<0x142, 0xa, false>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp_mov<0x143, 0xc, false>(v);   // row_bcast:31 into rows 2 and 3
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// Columns ka and / or kb (registers) <- H_c applied to them, v_c in LDS.  v_c stays in registers between the dot products and the updates
// where there is room beside the columns.  Long columns leave 32 registers: a test before every slot keeps the reads of v apart.
template <int XS, bool DO_A, bool DO_B>
__device__ __forceinline__ void apply_reflector(f32x4 (&ka)[XS], f32x4 (&kb)[XS], const f32x4* s_v4, int nvec, int lane, float tau) {
  constexpr bool HOLD_V = XS <= 4, LONG = XS > 8;
  f32x4 v[HOLD_V ? XS : 1];
  float da = 0.f, db = 0.f;
#pragma unroll
  for (int sl = 0; sl < XS; ++sl) {
    if (LONG && lane + 64 * sl >= nvec) continue;
    const f32x4 y = s_v4[lane + 64 * sl];
    if (HOLD_V) v[sl] = y;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (DO_A) da = __builtin_fmaf(ka[sl][e], y[e], da);
      if (DO_B) db = __builtin_fmaf(kb[sl][e], y[e], db);
    }
    if (!HOLD_V && !LONG && (sl & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // few reads of v at a time: more would be spilled
  }
  const float fa = DO_A ? tau * wave_sum_dpp(da) : 0.f;
  const float fb = DO_B ? tau * wave_sum_dpp(db) : 0.f;
#pragma unroll
  for (int sl = 0; sl < XS; ++sl) {
    if (LONG && lane + 64 * sl >= nvec) continue;
    const f32x4 y = HOLD_V ? v[sl] : s_v4[lane + 64 * sl];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (DO_A) ka[sl][e] = __builtin_fmaf(-fa, y[e], ka[sl][e]);
      if (DO_B) kb[sl][e] = __builtin_fmaf(-fb, y[e], kb[sl][e]);
    }
    if (!HOLD_V && !LONG && (sl & 3) == 3) __builtin_amdgcn_sched_barrier(0);
  }
}

// The products of the block run over the rows of the reflectors from the block's first column on: zero before the panel.
__device__ __forceinline__ void zero_before_panel(const QrMatrix& a, const QrArgs& args, int t) {
  const int before = QB * args.pos;
  for (int e = t; e < QB * before; e += QTH) {
    const int r = e / before, q = e - r * before;
    a.vall[static_cast<int64_t>(args.jb + before + r) * a.dp + args.jb + q] = 0.f;
  }
}

// The panel kernels.  Column c2 of the panel belongs to wavefront (c2 - 1) mod 16 for the whole kernel: it alone reads and
// writes that column, so the columns need no synchronisation between wavefronts.  What the others
// need of step c is the reflector v_c, which its owner leaves in LDS together with tau_c.  Two copies of v in turn: while all
// apply H_c to their later columns, the owner of column c + 1 does that one first, turns it into v_(c+1) and leaves that in the other
// copy; one barrier per step, and the chain of a step is that one column, whose wavefront goes before the three others of its SIMD
// meanwhile.  With v in LDS the barriers only have to order LDS traffic, so they do not wait for the stores in flight.
// Columns at or beyond d (padding) and columns that are already zero below the diagonal get tau = 0 (H = I).
// Bound by that chain (LDS round trips, two wave sums, a root and two quotients): us a panel of 512, 1024, 2048 rows 27, 36, 58 with two
// divisions and a root of the library and every wavefront alike, 20, 25, 41 now.  Fewer wavefronts of more columns are slower (8 of 4 columns:
// 27, 35, 53): a wavefront on its own does not fill its SIMD.
//
// At most 256 XS remaining rows (XS = 2, 4, 8: 512 .. 2048): every
// wavefront loads its two columns (wave + 1 and wave + 17) into registers once and keeps them there.  The
// columns are never written back: what the factorisation leaves in them is R, which nothing uses.
template <int XS>
__global__ __launch_bounds__(QTH) void k_qr_panel_regs(QrArgs args) {
  __shared__ f32x4 s_v4[2][64 * XS];
  __shared__ float s_tau[QB];
  const QrMatrix a = qr_matrix(args, blockIdx.x);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t dp = a.dp;
  const int j0 = args.jb + args.pos * QB;
  const int nvec = (a.dp - j0) / 4;                   // <= 64 XS
  const int ca = wave + 1, cb = wave + 1 + QWAVES;    // this wavefront's columns (cb only if < 32)
  f32x4 ka[XS], kb[XS];

  auto load_col = [&](f32x4 (&k)[XS], int c) {
    const f32x4* x = reinterpret_cast<const f32x4*>(a.wk + static_cast<int64_t>(j0 + c) * dp + j0);
#pragma unroll
    for (int sl = 0; sl < XS; ++sl) {   // zero beyond the column: stays zero, and so do the reflectors in LDS
      const int q = lane + 64 * sl;
      k[sl] = q < nvec ? x[q] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  // column c (in k) becomes the reflector v_c: to LDS, to the reflector array, tau to LDS
  auto make_v = [&](const f32x4 (&k)[XS], int c) {
    const float al = element_of(k[0], c), ss = wave_sum_dpp(squares_below(k, lane, c));
    float tau, scale;
    reflector_of(j0 + c < a.d, ss, al, tau, scale);
    f32x4* vg = reinterpret_cast<f32x4*>(a.vall + static_cast<int64_t>(j0 + c) * dp + j0);
    if (lane == 0) s_tau[c] = tau;
#pragma unroll
    for (int sl = 0; sl < XS; ++sl) {
      f32x4 o;
      if (sl == 0)
        o = v_of(k[0], lane, c, scale);
      else
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = k[sl][e] * scale;
      s_v4[c & 1][lane + 64 * sl] = o;
      if (lane + 64 * sl < nvec) vg[lane + 64 * sl] = o;
    }
  };

  if (wave == 0) {
    load_col(ka, 0);
    make_v(ka, 0);
  }
  load_col(ka, ca);
  if (cb < QB) load_col(kb, cb);
  zero_before_panel(a, args, t);

  for (int c = 0; c + 1 < QB; ++c) {
    lds_barrier();   // v_c and tau_c are in place, and every wavefront has finished with v_(c-1)
    const float tau = s_tau[c];
    const f32x4* v = s_v4[c & 1];
    const bool live = tau != 0.f;
    if (c + 1 == ca) {
      __builtin_amdgcn_s_setprio(3);
      if (live) apply_reflector<XS, true, false>(ka, kb, v, nvec, lane, tau);
      make_v(ka, c + 1);
      __builtin_amdgcn_s_setprio(0);
      if (live && cb < QB) apply_reflector<XS, false, true>(ka, kb, v, nvec, lane, tau);
    } else if (c + 1 == cb) {
      __builtin_amdgcn_s_setprio(3);
      if (live) apply_reflector<XS, false, true>(ka, kb, v, nvec, lane, tau);
      make_v(kb, c + 1);
      __builtin_amdgcn_s_setprio(0);
    } else if (live) {   // columns that have become reflectors are left alone
      const bool do_a = ca > c, do_b = cb < QB && cb > c;
      if (do_a && do_b)
        apply_reflector<XS, true, true>(ka, kb, v, nvec, lane, tau);
      else if (do_b)
        apply_reflector<XS, false, true>(ka, kb, v, nvec, lane, tau);
      else if (do_a)
        apply_reflector<XS, true, false>(ka, kb, v, nvec, lane, tau);
    }
  }
  lds_barrier();
  if (t < QB) a.tau[args.pos * QB + t] = s_tau[t];
}

// Longer columns.  A second copy of v_c and the pipelined chain of k_qr_panel_regs cost these more in spilled registers than they save
// (us a panel, pipelined / with two barriers a step, one copy and the library's root and quotients: 2049 to 3072 rows 100 / 70, 3073 to 8192
// on average 420 / 380), so: every wavefront applies H_c to its later columns and the owner of column c + 1 takes that one's head; barrier;
// the owner writes v_(c+1); barrier.
//
// Up to 3072 remaining rows (XS = 12) the columns stay in registers.
template <int XS>
__global__ __launch_bounds__(QTH) void k_qr_panel_long(QrArgs args) {
  __shared__ f32x4 s_v4[64 * XS];
  __shared__ float s_tau[QB];
  const QrMatrix a = qr_matrix(args, blockIdx.x);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t dp = a.dp;
  const int j0 = args.jb + args.pos * QB;
  const int nvec = (a.dp - j0) / 4;                   // <= 64 XS
  const int ca = wave + 1, cb = wave + 1 + QWAVES;    // this wavefront's columns (cb only if < 32)
  f32x4 ka[XS], kb[XS];

  auto load_col = [&](f32x4 (&k)[XS], int c) {
    const f32x4* x = reinterpret_cast<const f32x4*>(a.wk + static_cast<int64_t>(j0 + c) * dp + j0);
#pragma unroll
    for (int sl = 0; sl < XS; ++sl) {   // beyond the column nothing is read, here and below
      const int q = lane + 64 * sl;
      if (q < nvec) k[sl] = x[q];
    }
  };
  // sum of squares below row c and the element at row c, over the wavefront
  auto head = [&](const f32x4 (&k)[XS], int c, float& ss, float& al) {
    ss = 0.f, al = 0.f;
#pragma unroll
    for (int sl = 0; sl < XS; ++sl) {
      const int q = lane + 64 * sl;
      if (q < nvec) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * q + e;
          if (r > c) ss += k[sl][e] * k[sl][e];
          if (r == c) al = k[sl][e];
        }
      }
    }
    ss = wave_sum_dpp(ss), al = wave_sum_dpp(al);
  };
  // column c (in k), whose head is (ss, al), becomes the reflector v_c: to LDS, to the reflector array, tau to LDS
  auto make_v = [&](const f32x4 (&k)[XS], int c, float ss, float al) {
    float tau, scale;
    reflector_of<false>(j0 + c < a.d, ss, al, tau, scale);
    f32x4* vg = reinterpret_cast<f32x4*>(a.vall + static_cast<int64_t>(j0 + c) * dp + j0);
#pragma unroll
    for (int sl = 0; sl < XS; ++sl) {
      const int q = lane + 64 * sl;
      if (q < nvec) {
        const f32x4 o = v_of(k[sl], q, c, scale);
        s_v4[q] = o;
        vg[q] = o;
      }
    }
    if (lane == 0) s_tau[c] = tau;
  };

  if (wave == 0) {
    float ss, al;
    load_col(ka, 0);
    head(ka, 0, ss, al);
    make_v(ka, 0, ss, al);
  }
  load_col(ka, ca);
  if (cb < QB) load_col(kb, cb);
  lds_barrier();

  for (int c = 0; c < QB; ++c) {
    const float tau = s_tau[c];
    const bool do_a = ca > c, do_b = cb < QB && cb > c;
    if (tau != 0.f) {   // columns that have become reflectors are left alone
      if (do_a && do_b)
        apply_reflector<XS, true, true>(ka, kb, s_v4, nvec, lane, tau);
      else if (do_a)
        apply_reflector<XS, true, false>(ka, kb, s_v4, nvec, lane, tau);
      else if (do_b)
        apply_reflector<XS, false, true>(ka, kb, s_v4, nvec, lane, tau);
    }
    // the owner of column c + 1 takes its head while the others are still busy with their columns
    const bool owner = c + 1 < QB && wave == c % QWAVES;
    float ss = 0.f, al = 0.f;
    if (owner) {
      if (c + 1 == ca)
        head(ka, c + 1, ss, al);
      else
        head(kb, c + 1, ss, al);
    }
    lds_barrier();   // every wavefront has finished with v_c
    if (owner) {
      if (c + 1 == ca)
        make_v(ka, c + 1, ss, al);
      else
        make_v(kb, c + 1, ss, al);
    }
    lds_barrier();   // v_(c+1) and tau_(c+1) are in place
  }
  zero_before_panel(a, args, t);
  if (t < QB) a.tau[args.pos * QB + t] = s_tau[t];
}

// Beyond 3072 remaining rows every wavefront
// keeps the first 256 XS rows of its two columns in registers for the whole kernel; the rows beyond are streamed
// from the working copy on every step (read for the dot product, read and written for the update: the wavefront's
// own stores, which it reads back itself).  v_c is in LDS at full length.
template <int XS>
__global__ __launch_bounds__(QTH) void k_qr_panel_hybrid(QrArgs args) {
  __shared__ f32x4 s_v4[VMAX / 4];
  __shared__ float s_tau[QB];
  constexpr int NR = 64 * XS;   // float4 of a column kept in registers
  constexpr int TU = 2;         // loads in flight per lane in the streaming loops
  const QrMatrix a = qr_matrix(args, blockIdx.x);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t dp = a.dp;
  const int j0 = args.jb + args.pos * QB;
  const int nvec = (a.dp - j0) / 4;   // > NR
  auto col = [&](int c) { return reinterpret_cast<f32x4*>(a.wk + static_cast<int64_t>(j0 + c) * dp + j0); };
  const int ca = wave + 1, cb = wave + 1 + QWAVES;    // this wavefront's columns (cb only if < 32)
  f32x4 ka[XS], kb[XS];

  auto load_col = [&](f32x4 (&k)[XS], int c) {
    const f32x4* x = col(c);
#pragma unroll
    for (int sl = 0; sl < XS; ++sl) k[sl] = x[lane + 64 * sl];
  };
  // sum of squares below row c and the element at row c (c < 32: it lies in the registers), over the wavefront
  auto head = [&](const f32x4 (&k)[XS], int c, float& ss, float& al) {
    ss = 0.f, al = 0.f;
#pragma unroll
    for (int sl = 0; sl < XS; ++sl) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * (lane + 64 * sl) + e;
        if (r > c) ss += k[sl][e] * k[sl][e];
        if (r == c) al = k[sl][e];
      }
    }
    const f32x4* x = col(c);
    for (int q0 = NR + lane; q0 < nvec; q0 += 64 * TU) {
      f32x4 xv[TU];
#pragma unroll
      for (int u = 0; u < TU; ++u) xv[u] = x[min(q0 + 64 * u, nvec - 1)];   // in bounds; surplus loads unused
#pragma unroll
      for (int u = 0; u < TU; ++u)
        if (q0 + 64 * u < nvec)
#pragma unroll
          for (int e = 0; e < 4; ++e) ss += xv[u][e] * xv[u][e];
    }
    ss = wave_sum_dpp(ss), al = wave_sum_dpp(al);
  };
  // column c, whose head is (ss, al), becomes the reflector v_c: to LDS, to the reflector array, tau to LDS
  auto make_v = [&](const f32x4 (&k)[XS], int c, float ss, float al) {
    float tau, scale;
    reflector_of<false>(j0 + c < a.d, ss, al, tau, scale);
    f32x4* vg = reinterpret_cast<f32x4*>(a.vall + static_cast<int64_t>(j0 + c) * dp + j0);
#pragma unroll
    for (int sl = 0; sl < XS; ++sl) {
      const int q = lane + 64 * sl;
      const f32x4 o = v_of(k[sl], q, c, scale);
      s_v4[q] = o;
      vg[q] = o;
    }
    const f32x4* x = col(c);
    for (int q = NR + lane; q < nvec; q += 64) {
      f32x4 o = x[q];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] *= scale;
      s_v4[q] = o;
      vg[q] = o;
    }
    if (lane == 0) s_tau[c] = tau;
  };
  // H_c applied to column c2, held in k and, beyond the registers, in memory
  auto apply = [&](f32x4 (&k)[XS], int c2, float tau) {
    f32x4* x = col(c2);
    float dot = 0.f;
#pragma unroll
    for (int sl = 0; sl < XS; ++sl) {
      const f32x4 y = s_v4[lane + 64 * sl];
#pragma unroll
      for (int e = 0; e < 4; ++e) dot = __builtin_fmaf(k[sl][e], y[e], dot);
    }
    for (int q0 = NR + lane; q0 < nvec; q0 += 64 * TU) {
      f32x4 xv[TU];
#pragma unroll
      for (int u = 0; u < TU; ++u) xv[u] = x[min(q0 + 64 * u, nvec - 1)];
#pragma unroll
      for (int u = 0; u < TU; ++u) {
        const int q = q0 + 64 * u;
        if (q < nvec) {
          const f32x4 y = s_v4[q];
#pragma unroll
          for (int e = 0; e < 4; ++e) dot = __builtin_fmaf(xv[u][e], y[e], dot);
        }
      }
    }
    const float f = tau * wave_sum_dpp(dot);
#pragma unroll
    for (int sl = 0; sl < XS; ++sl) {
      const f32x4 y = s_v4[lane + 64 * sl];
#pragma unroll
      for (int e = 0; e < 4; ++e) k[sl][e] = __builtin_fmaf(-f, y[e], k[sl][e]);
    }
    for (int q0 = NR + lane; q0 < nvec; q0 += 64 * TU) {
      f32x4 xv[TU];
#pragma unroll
      for (int u = 0; u < TU; ++u) xv[u] = x[min(q0 + 64 * u, nvec - 1)];
#pragma unroll
      for (int u = 0; u < TU; ++u) {
        const int q = q0 + 64 * u;
        if (q < nvec) {
          const f32x4 y = s_v4[q];
#pragma unroll
          for (int e = 0; e < 4; ++e) xv[u][e] = __builtin_fmaf(-f, y[e], xv[u][e]);
          x[q] = xv[u];
        }
      }
    }
  };

  if (wave == 0) {
    float ss, al;
    load_col(ka, 0);
    head(ka, 0, ss, al);
    make_v(ka, 0, ss, al);
  }
  load_col(ka, ca);
  if (cb < QB) load_col(kb, cb);
  lds_barrier();

  for (int c = 0; c < QB; ++c) {
    const float tau = s_tau[c];
    if (tau != 0.f) {   // columns that have become reflectors are left alone
      if (ca > c) apply(ka, ca, tau);
      if (cb < QB && cb > c) apply(kb, cb, tau);
    }
    // the owner of column c + 1 takes its head while the others are still busy with their columns
    const bool owner = c + 1 < QB && wave == c % QWAVES;
    float ss = 0.f, al = 0.f;
    if (owner) {
      if (c + 1 == ca)
        head(ka, c + 1, ss, al);
      else
        head(kb, c + 1, ss, al);
    }
    lds_barrier();   // every wavefront has finished with v_c
    if (owner) {
      if (c + 1 == ca)
        make_v(ka, c + 1, ss, al);
      else
        make_v(kb, c + 1, ss, al);
    }
    lds_barrier();   // v_(c+1) and tau_(c+1) are in place
  }
  zero_before_panel(a, args, t);
  if (t < QB) a.tau[args.pos * QB + t] = s_tau[t];
}

// Piece blockIdx.x of k of the products with panel `pos` of the block, V its reflectors: 32 x 32 blocks
//   a <= pos:  V_a^T V  (V_a: panel a of the block),      a > pos:  W = (columns of panel a)^T V.
// One wavefront per block; the pieces lie in the strip, [piece][128][32].  Rows through LDS k-major, all loads of 128 k at once.
constexpr int GLD = 32 + 1, GRD = 128 + 5;   // row lengths in LDS: the stores of a stage spread over the banks
__global__ __launch_bounds__(NTH) void k_qr_gram(QrArgs args) {
  __shared__ float s_r[32][GRD], s_v[32][GLD];
  const QrMatrix a = qr_matrix(args, blockIdx.y);
  int chunks, len;
  qr_chunks(a.dp, args.jb, chunks, len);
  if (static_cast<int>(blockIdx.x) >= chunks) return;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, pos = args.pos;
  const int64_t dp = a.dp;
  const int j0 = args.jb + pos * QB;
  const int k_end = min(args.jb + (static_cast<int>(blockIdx.x) + 1) * len, a.dp);
  const int k_begin = args.jb + static_cast<int>(blockIdx.x) * len;
  // thread t loads rows t / 8 + 32 x of the four blocks and row t / 8 of V, 4 k at 4 (t % 8)
  const int row = t >> 3, kq = (t & 7) * 4;
  const float* src[5];
#pragma unroll
  for (int x = 0; x < 4; ++x) src[x] = (x <= pos ? a.vall : a.wk) + static_cast<int64_t>(args.jb + 32 * x + row) * dp + kq;
  src[4] = a.vall + static_cast<int64_t>(j0 + row) * dp + kq;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  for (int k0 = k_begin; k0 < k_end; k0 += 128) {
    f32x4 v[4][5];
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
      for (int x = 0; x < 5; ++x) v[st][x] = *reinterpret_cast<const f32x4*>(src[x] + k0 + 32 * st);
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      const bool live = k0 + 32 * st >= j0;   // before the panel's first row V is zero
      __syncthreads();
#pragma unroll
      for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int x = 0; x < 4; ++x) s_r[kq + c][row + 32 * x] = v[st][x][c];
        s_v[kq + c][row] = v[st][4][c];
      }
      __syncthreads();
      if (live)
#pragma unroll
        for (int kk = 0; kk < 32; kk += 2)
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(s_r[kk + (lane >> 5)][32 * wave + (lane & 31)], s_v[kk + (lane >> 5)][lane & 31], acc, 0, 0, 0);
    }
  }
  float* out = a.strip + static_cast<int64_t>(blockIdx.x) * (QBLK * QB) + (32 * wave + 4 * (lane >> 5)) * QB + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) out[(8 * (r >> 2) + (r & 3)) * QB] = acc[r];
}

// The sum of the pieces of four consecutive elements, in order.
__device__ __forceinline__ f32x4 sum_pieces(const float* p, int chunks) {
  f32x4 v = *reinterpret_cast<const f32x4*>(p);
#pragma unroll 5
  for (int i = 1; i < chunks; ++i) v += *reinterpret_cast<const f32x4*>(p + i * (QBLK * QB));
  return v;
}

// Panel `pos` (< 3) applied to the later columns of its block: X -= W' V^T in 128 columns (k of the rows of wk) per workgroup, each of
// which solves for W' itself (see above); the first also leaves the V_a^T V of this panel in `gram`.
__global__ __launch_bounds__(NTH) void k_qr_panel_sub(QrArgs args) {
  __shared__ __attribute__((aligned(16))) float s_g[QB][QB + 4];   // s_g[c][l] = v_l^T v_c
  __shared__ float s_w[3 * QB][QB + 1];
  __shared__ float s_tau[QB];
  const QrMatrix a = qr_matrix(args, blockIdx.y);
  const int pos = args.pos, later = 3 - pos;
  const int64_t dp = a.dp;
  const int n0 = args.jb + static_cast<int>(blockIdx.x) * 128, j0 = args.jb + pos * QB;
  if (n0 >= a.dp) return;
  int chunks, len;
  qr_chunks(a.dp, args.jb, chunks, len);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  // this wavefront's 32 columns of V, asked for first: lane l holds rows 2 kk + l / 32
  const int n = n0 + 32 * wave;
  float vb[QB / 2];
#pragma unroll
  for (int kk = 0; kk < QB / 2; ++kk) vb[kk] = a.vall[static_cast<int64_t>(j0 + 2 * kk + (lane >> 5)) * dp + n + (lane & 31)];
  if (t < QB) s_tau[t] = a.tau[pos * QB + t];
  const int i4 = t >> 3, c4 = (t & 7) * 4;   // row of a 32 x 32 block, 4 columns
  if (blockIdx.x == 0)
    for (int x = 0; x < pos; ++x)
      *reinterpret_cast<f32x4*>(a.gram + (32 * x + i4) * QBLK + 32 * pos + c4) = sum_pieces(a.strip + (32 * x + i4) * QB + c4, chunks);
  {
    const f32x4 v = sum_pieces(a.strip + (32 * pos + i4) * QB + c4, chunks);
    if (blockIdx.x == 0) *reinterpret_cast<f32x4*>(a.gram + (32 * pos + i4) * QBLK + 32 * pos + c4) = v;
#pragma unroll
    for (int c = 0; c < 4; ++c) s_g[c4 + c][i4] = v[c];
  }
  for (int x = 0; x < later; ++x) {
    const f32x4 v = sum_pieces(a.strip + (32 * (pos + 1 + x) + i4) * QB + c4, chunks);
#pragma unroll
    for (int c = 0; c < 4; ++c) s_w[32 * x + i4][c4 + c] = v[c];
  }
  __syncthreads();
  if (t < 32 * later) {
    float w[QB];
#pragma unroll
    for (int c = 0; c < QB; ++c) w[c] = s_w[t][c];
#pragma unroll
    for (int c = 0; c < QB; ++c) {
      float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int l4 = 0; l4 < c; l4 += 4) {
        const f32x4 g = *reinterpret_cast<const f32x4*>(&s_g[c][l4]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (l4 + e < c) part[e] = __builtin_fmaf(w[l4 + e], g[e], part[e]);
      }
      const float tau = s_tau[c];
      w[c] = tau == 0.f ? 0.f : tau * (w[c] - ((part[0] + part[1]) + (part[2] + part[3])));
      s_w[t][c] = w[c];
    }
  }
  __syncthreads();
  for (int x = 0; x < later; ++x) {
    float* C = a.wk + static_cast<int64_t>(args.jb + 32 * (pos + 1 + x) + 4 * (lane >> 5)) * dp + n + (lane & 31);
    float old[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) old[r] = C[static_cast<int64_t>(8 * (r >> 2) + (r & 3)) * dp];
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < QB / 2; ++kk)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(s_w[32 * x + (lane & 31)][2 * kk + (lane >> 5)], vb[kk], acc, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 16; ++r) C[static_cast<int64_t>(8 * (r >> 2) + (r & 3)) * dp] = old[r] - acc[r];
  }
}

// T of a block of 128 reflectors, T = (diag(1 / tau) + strictly upper part of V^T V)^(-1) with zero rows and columns where tau = 0: its 32 x 32
// blocks on the diagonal row by row, T[i][c] = tau_c ((i == c) - sum_{i <= l < c} T[i][l] v_l^T v_c), then those at distance 1, 2, 3,
// T_ab = -(sum_{a <= c < b} T_ac G_cb) T_bb.  T goes where V^T V was, T^T to `tt`.  One workgroup per matrix.
__global__ __launch_bounds__(QTH) void k_qr_block_t(QrArgs args) {
  constexpr int GTLD = QBLK + 4;
  __shared__ __attribute__((aligned(16))) float s_gt[QBLK][GTLD];   // s_gt[c][l] = v_l^T v_c
  __shared__ float s_t[QBLK][QBLK + 1];
  __shared__ float s_x[3][QB][QB + 1];
  __shared__ float s_tau[QBLK];
  const QrMatrix a = qr_matrix(args, blockIdx.x);
  int chunks, len;
  qr_chunks(a.dp, args.jb, chunks, len);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (t < QBLK) s_tau[t] = a.tau[t];
  {   // the last panel's column of blocks is still in pieces
    const int i = t >> 3, c4 = (t & 7) * 4;
    const f32x4 v = sum_pieces(a.strip + i * QB + c4, chunks);
#pragma unroll
    for (int c = 0; c < 4; ++c) s_gt[3 * QB + c4 + c][i] = v[c];
  }
  for (int e = t; e < QBLK * QBLK; e += QTH) {
    const int r = e >> 7, q = e & 127;
    if (q < 3 * QB) s_gt[q][r] = (r >> 5) <= (q >> 5) ? a.gram[e] : 0.f;
    s_t[r][q] = 0.f;
  }
  __syncthreads();
  if (t < QBLK) {
    const int base = t & ~31, i = t & 31;
    float row[QB];
#pragma unroll
    for (int c = 0; c < QB; ++c) {
      float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int l4 = 0; l4 < c; l4 += 4) {
        const f32x4 g = *reinterpret_cast<const f32x4*>(&s_gt[base + c][base + l4]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (l4 + e < c) part[e] = __builtin_fmaf(row[l4 + e], g[e], part[e]);
      }
      const float tau = s_tau[base + c], sum = (part[0] + part[1]) + (part[2] + part[3]);
      row[c] = i == c ? tau : (i < c && tau != 0.f ? -tau * sum : 0.f);   // left of the diagonal the row is zero, and so is the sum
      s_t[t][base + c] = row[c];
    }
  }
  __syncthreads();
  // a wavefront per block at distance k, on the matrix cores
  const int lj = lane & 31, lh = lane >> 5;
  for (int k = 1; k < 4; ++k) {
    if (wave + k < 4) {
      const int lo = wave, hi = wave + k;
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
      for (int c = lo; c < hi; ++c)
#pragma unroll
        for (int kk = 0; kk < QB; kk += 2)
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(s_t[lo * QB + lj][c * QB + kk + lh], s_gt[hi * QB + lj][c * QB + kk + lh], acc, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) s_x[lo][8 * (r >> 2) + (r & 3) + 4 * lh][lj] = acc[r], acc[r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < QB; kk += 2)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(s_x[lo][lj][kk + lh], s_t[hi * QB + kk + lh][hi * QB + lj], acc, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r) s_t[lo * QB + 8 * (r >> 2) + (r & 3) + 4 * lh][hi * QB + lj] = -acc[r];
    }
    __syncthreads();
  }
  float* tt = a.tt + static_cast<int64_t>(args.jb / QBLK) * QBLK * QBLK;
  for (int e = t; e < QBLK * QBLK; e += QTH) {
    a.gram[e] = s_t[e >> 7][e & 127];
    tt[e] = s_t[e & 127][e >> 7];
  }
}

// W' = (X V) T of a block (BACK: (X V) T^T), X the rows lo.. of wk (BACK: of Q^T) from column jb on, V the block's 128 reflectors: 32 rows
// per workgroup, a wavefront per panel, and the second product from LDS.  Bound by the fp32 matrix cores (32 rows and not more, so that
// the 2048-long sums of 4 x 1920 rows have 240 workgroups: 129 -> 35 us).
template <bool BACK>
__global__ __launch_bounds__(NTH) void k_qr_block_w(QrArgs args, int lo) {
  __shared__ float s_x[2][32][GLD], s_v[2][32][GRD];
  __shared__ float s_w[32][QBLK + 1];
  const QrMatrix a = qr_matrix(args, blockIdx.y);
  const int r0 = lo + static_cast<int>(blockIdx.x) * 32;
  if (r0 >= a.dp) return;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t dp = a.dp;
  const int row = t >> 3, kq = (t & 7) * 4;
  const float* xs = (BACK ? a.qt : a.wk) + static_cast<int64_t>(r0 + row) * dp + args.jb + kq;
  const float* vs = a.vall + static_cast<int64_t>(args.jb + row) * dp + args.jb + kq;
  // this wavefront's 32 columns of T; what is zero in it (below or above the diagonal blocks) is left out
  const float* tm = BACK ? a.tt + static_cast<int64_t>(args.jb / QBLK) * QBLK * QBLK : a.gram;
  const int c_lo = BACK ? wave : 0, c_hi = BACK ? 4 : wave + 1;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  const int nk = (a.dp - args.jb) / 32;   // a multiple of 4
  f32x4 pv[2][5];
  auto fetch = [&](int kt, int set) {
    pv[set][4] = *reinterpret_cast<const f32x4*>(xs + 32 * kt);
#pragma unroll
    for (int x = 0; x < 4; ++x) pv[set][x] = *reinterpret_cast<const f32x4*>(vs + 32 * x * dp + 32 * kt);
  };
  auto stash = [&](int buf, int set) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      s_x[buf][kq + c][row] = pv[set][4][c];
#pragma unroll
      for (int x = 0; x < 4; ++x) s_v[buf][kq + c][row + 32 * x] = pv[set][x][c];
    }
  };
  auto stage = [&](int kt, int buf, int mine, int other) {
    if (kt + 2 < nk) fetch(kt + 2, mine);
#pragma unroll
    for (int k = 0; k < 32; k += 2)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(s_x[buf][k + (lane >> 5)][lane & 31], s_v[buf][k + (lane >> 5)][32 * wave + (lane & 31)], acc, 0, 0, 0);
    if (kt + 1 < nk) stash(buf ^ 1, other);
    __syncthreads();
  };
  fetch(0, 0);
  fetch(1, 1);
  stash(0, 0);
  __syncthreads();
  for (int kt = 0; kt < nk; kt += 2) {
    stage(kt, 0, 0, 1);
    stage(kt + 1, 1, 1, 0);
  }
  float tb[QBLK / 2];   // the whole column block of T: its loads are out before the barrier below
#pragma unroll
  for (int kk = 0; kk < QBLK / 2; ++kk) {
    const int k = 2 * kk + (lane >> 5);
    if (kk / 16 >= c_lo && kk / 16 < c_hi) tb[kk] = tm[k * QBLK + 32 * wave + (lane & 31)];
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) s_w[8 * (r >> 2) + (r & 3) + 4 * (lane >> 5)][32 * wave + (lane & 31)] = acc[r];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (c >= c_lo && c < c_hi)
#pragma unroll
      for (int kk = 16 * c; kk < 16 * c + 16; ++kk)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(s_w[lane & 31][2 * kk + (lane >> 5)], tb[kk], acc, 0, 0, 0);
  float* out = a.strip + static_cast<int64_t>(r0 + 4 * (lane >> 5)) * QBLK + 32 * wave + (lane & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) out[(8 * (r >> 2) + (r & 3)) * QBLK] = acc[r];
}

// Products of the refresh on both sides of a batch in one launch: the blocks of side 0 first.
template <int EPI, bool QT>
__global__ __launch_bounds__(NTH) void k_qr_gemm(ShGemm g0, ShGemm g1, int first1, PtrTable none, Shape s, OutSpec o) {
  const int block = blockIdx.x;
  sh_gemm_body<EPI, false, false, QT>(block < first1 ? g0 : g1, block < first1 ? block : block - first1, none, s, o);
}

// How the rotations of a launch batch are computed (plan_of): on fp32 matrices, on three bf16 terms per element, or on bf16
// operands.
enum class Rot { F32, TERMS, BF16 };

struct Carve {   // float offsets into the workspace of one launch batch
  size_t gm, gmt, t1, rot, np, yt, ql, qlt, qr, qrt, pool, total_bytes;
  // rotations on three bf16 terms: G', M' dense; three bf16 terms per element, padded to 256 (offsets in floats as well): G (if it is not
  // bf16 itself) and M in the orientations wanted, X Q_R transposed, N', its half-rotated image, the bases
  size_t rotg, rotm, g3, g3t, m3, m3t, t3, n3, y3, ql3, ql3t, qr3, qr3t;
  // bf16 rotations (offsets in floats as well; each array holds bf16 panels padded to 256)
  size_t gp, gpt, mp, mpt, as_g, at_g, as_m, at_m, rg, rgt, rm, rmt, npn, npt, ys, yst, qlp, qltp, qrp, qrtp;
};

struct Sides {
  bool left, right;
};
Sides sides(const canz_soap_group& g, const canz_soap_hparams& hp) {
  return {g.rows <= hp.max_precond_dim, g.cols <= hp.max_precond_dim};
}
// Gradients that arrive as bf16 are exact operands of the bf16 matrix cores: the products of G G^T and G^T G are
// exact in fp32 and are accumulated in fp32, so the statistics lose nothing against the fp32 kernel and take
// a fraction of its time.
bool bf16_statistics(const canz_soap_group& g) { return g.grad_dtype == CANZ_DT_BF16; }

// floats from one dense rows x cols working matrix to the next: each starts aligned, as the callers' own buffers do
inline int64_t dense_stride(int64_t rows, int64_t cols) { return (rows * cols + 63) / 64 * 64; }

Carve carve(int64_t rows, int64_t cols, int nb, Sides u, bool refresh, Rot rot, bool stat16) {
  const size_t rp = pad128(rows), cp = pad128(cols);
  const size_t dm = std::max(u.left ? rp : 0, u.right ? cp : 0);
  const bool both = u.left && u.right, bf16 = rot == Rot::BF16;
  Carve c{};
  size_t off = 0;
  auto take = [&](size_t floats) {
    const size_t at = off;
    off += align_up(floats * sizeof(float)) / sizeof(float);
    return at;
  };
  const size_t plane = rp * cp;
  if (rot == Rot::TERMS) {
    c.gm = take(stat16 ? 0 : nb * plane), c.gmt = take(stat16 ? 0 : nb * plane);
  } else {   // the bf16 rotations use G, G^T and the statistic of these only
    c.gm = take(2 * nb * plane), c.gmt = take(2 * nb * plane);
    c.t1 = take(both ? 2 * nb * plane : 0);
    c.rot = take(2 * nb * plane);
    c.np = take(nb * plane);
    c.yt = take(both ? nb * plane : 0);
    c.ql = take(u.left ? nb * rp * rp : 0), c.qlt = take(u.left ? nb * rp * rp : 0);
    c.qr = take(u.right ? nb * cp * cp : 0), c.qrt = take(u.right ? nb * cp * cp : 0);
    take(nb * dm * dm);   // not used (once a padded statistic): with less a matrix, batches would hold more of them and could need more in all
                          // than a workspace that was measured by this sum
  }
  if (refresh) {
    // The refresh of both sides (one_side lays them out): two square matrices and a strip of 256 columns a side and 128 x 129 floats.  Four
    // squares of the larger side, 544 columns and the rest hold them, whatever the other side is.
    c.pool = take(nb * (4 * dm * dm + 544 * dm + 3 * QBLK * QBLK));
    take(nb * QB);   // not used, as above
  }
  const size_t rp2 = pad256(rows), cp2 = pad256(cols), p2 = nb * rp2 * cp2 / 2;   // floats that hold a batch of panels
  const bool all_of_g = bf16 || rot == Rot::TERMS;   // G is an operand of the rotations, too
  if (bf16 || stat16) c.gp = take(all_of_g || u.left ? p2 : 0), c.gpt = take(all_of_g || u.right ? p2 : 0);
  if (rot == Rot::TERMS) {
    const size_t p3 = nb * rp2 * cp2 * 3 / 2, l3 = nb * rp2 * rp2 * 3 / 2, r3 = nb * cp2 * cp2 * 3 / 2;
    c.rotg = take(nb * dense_stride(rows, cols)), c.rotm = take(nb * dense_stride(rows, cols));
    c.g3 = take(!stat16 && u.right ? p3 : 0), c.g3t = take(!stat16 && !u.right ? p3 : 0);
    c.m3 = take(u.right ? p3 : 0), c.m3t = take(u.right ? 0 : p3);
    c.t3 = c.y3 = take(both ? p3 : 0);   // t3 is done with before y3 is written, and G's terms before those of N'
    c.n3 = stat16 ? take(p3) : u.right ? c.g3 : c.g3t;
    c.ql3 = take(u.left ? l3 : 0), c.qr3 = take(u.right ? r3 : 0);
    c.ql3t = take(u.left ? l3 : 0), c.qr3t = take(u.right ? r3 : 0);
  }
  if (bf16) {
    c.mp = take(p2), c.mpt = take(p2);
    c.as_g = take(u.right ? p2 : 0), c.at_g = take(u.right ? p2 : 0), c.as_m = take(u.right ? p2 : 0), c.at_m = take(u.right ? p2 : 0);
    c.rg = take(u.left ? p2 : 0), c.rgt = take(u.left ? p2 : 0), c.rm = take(u.left ? p2 : 0), c.rmt = take(u.left ? p2 : 0);
    c.npn = take(p2), c.npt = take(p2);
    c.ys = take(both ? p2 : 0), c.yst = take(both ? p2 : 0);
    c.qlp = take(u.left ? nb * rp2 * rp2 / 2 : 0), c.qltp = take(u.left ? nb * rp2 * rp2 / 2 : 0);
    c.qrp = take(u.right ? nb * cp2 * cp2 / 2 : 0), c.qrtp = take(u.right ? nb * cp2 * cp2 / 2 : 0);
  }
  c.total_bytes = off * sizeof(float);
  return c;
}

size_t batch_bytes(const canz_soap_group& g, const canz_soap_hparams& hp, int nb, Rot rot) {
  return carve(g.rows, g.cols, nb, sides(g, hp), hp.refresh != 0, rot, bf16_statistics(g)).total_bytes;
}
// matrices per batch: what the pointer tables and the batch memory hold, at least one
int batch_cap(const canz_soap_group& g, const canz_soap_hparams& hp, Rot rot) {
  const int64_t by_bytes = std::max<int64_t>(1, static_cast<int64_t>(BATCH_BYTES / batch_bytes(g, hp, 1, rot)));
  return static_cast<int>(std::min<int64_t>({MAX_PTRS / g.tp, by_bytes, std::max<int64_t>(1, g.n_mats)}));
}
// The rotations in fp32 accuracy run on three bf16 terms, except up to 128 x 128, where fp32 matrices padded to 128 are
// faster than terms padded to 256 (8 x 128 x 128: 111 us against 122 with bf16 gradients, 133 against 160 with fp32 ones; from
// 129 rows or columns on terms win, 4 x 300 x 384 with fp32 gradients 268 us against 286).
// Terms can need more scratch than fp32 matrices do (where 256 is a poor padding): canz_soap_workspace_bytes asks for enough;
// whatever suffices for fp32 matrices is accepted, and then the batches are smaller, or if not even one matrix fits, the
// rotations run on fp32 matrices.
struct Plan {
  Rot rot;
  int nb;
};
Plan plan_of(const canz_soap_group& g, const canz_soap_hparams& hp, size_t have) {
  if (hp.bf16_rotations) return {Rot::BF16, batch_cap(g, hp, Rot::BF16)};
  if (g.rows <= SB && g.cols <= SB) return {Rot::F32, batch_cap(g, hp, Rot::F32)};
  const int nb = batch_cap(g, hp, Rot::TERMS);
  if (batch_bytes(g, hp, nb, Rot::TERMS) <= have) return {Rot::TERMS, nb};
  if (const size_t one = batch_bytes(g, hp, 1, Rot::TERMS); one <= have) return {Rot::TERMS, std::min(nb, static_cast<int>(have / one))};
  return {Rot::F32, batch_cap(g, hp, Rot::F32)};
}
size_t least_bytes(const canz_soap_group& g, const canz_soap_hparams& hp) {
  const Rot rot = hp.bf16_rotations ? Rot::BF16 : Rot::F32;
  return batch_bytes(g, hp, batch_cap(g, hp, rot), rot);
}

int check_hparams(const canz_soap_hparams* hp) {
  if (!hp) return fail(CANZ_EINVAL, "null hparams");
  if (!(hp->beta1 >= 0.f && hp->beta1 < 1.f) || !(hp->beta2 >= 0.f && hp->beta2 < 1.f))
    return fail(CANZ_EINVAL, "beta1 and beta2 must be in [0, 1)");
  if (!(hp->eps >= 0.f)) return fail(CANZ_EINVAL, "eps must be >= 0");
  if (hp->step < 1) return fail(CANZ_EINVAL, "step must be >= 1");
  if (hp->max_precond_dim < 1) return fail(CANZ_EINVAL, "max_precond_dim must be >= 1");
  if (hp->out_mode != CANZ_OUT_PARAM && hp->out_mode != CANZ_OUT_DELTA)
    return fail(CANZ_EUNSUPPORTED, "unknown out_mode %d", hp->out_mode);
  return CANZ_OK;
}

int check_group(const canz_soap_group& g, int idx, bool need_ptrs, const canz_soap_hparams& hp) {
  if (g.n_mats < 0) return fail(CANZ_EINVAL, "group %d: n_mats < 0", idx);
  if (g.rows < 1 || g.cols < 1) return fail(CANZ_EINVAL, "group %d: empty shape", idx);
  if (g.rows > MAX_EXTENT || g.cols > MAX_EXTENT)
    return fail(CANZ_ESHAPE, "group %d: extent above %lld", idx, static_cast<long long>(MAX_EXTENT));
  const Sides u = sides(g, hp);
  if ((u.left && g.rows > VMAX) || (u.right && g.cols > VMAX))
    return fail(CANZ_ESHAPE, "group %d: a side with a basis may have at most %d rows or columns (lower max_precond_dim)", idx, VMAX);
  if (!u.left && !u.right)
    return fail(CANZ_EUNSUPPORTED, "group %d: both extents exceed max_precond_dim (plain Adam is not part of this library)", idx);
  if (g.tp < 1 || g.tp > MAX_TP) return fail(CANZ_EINVAL, "group %d: tp must be in 1..%d", idx, MAX_TP);
  if (g.cols % g.tp) return fail(CANZ_ESHAPE, "group %d: cols not divisible by tp", idx);
  if (g.tp > 1 && (g.cols / g.tp) % 8) return fail(CANZ_ESHAPE, "group %d: fragment width not a multiple of 8", idx);
  if (g.grad_dtype != CANZ_DT_F32 && g.grad_dtype != CANZ_DT_BF16)
    return fail(CANZ_EUNSUPPORTED, "group %d: unknown grad_dtype", idx);
  if (g.out_dtype != CANZ_DT_F32 && g.out_dtype != CANZ_DT_BF16)
    return fail(CANZ_EUNSUPPORTED, "group %d: unknown out_dtype", idx);
  if (!need_ptrs || g.n_mats == 0) return CANZ_OK;
  if (!g.grad || !g.mom || !g.var || !g.out || (u.left && (!g.left || !g.qleft)) || (u.right && (!g.right || !g.qright)))
    return fail(CANZ_EINVAL, "group %d: null pointer table", idx);
  const int n_out = hp.out_mode == CANZ_OUT_DELTA ? g.n_mats * g.tp : g.n_mats;
  auto bad = [](const void* p) { return p == nullptr || (reinterpret_cast<uintptr_t>(p) & 15u) != 0; };
  for (int i = 0; i < g.n_mats * g.tp; ++i)
    if (bad(g.grad[i])) return fail(CANZ_EINVAL, "group %d: grad[%d] null or not 16-byte aligned", idx, i);
  for (int i = 0; i < g.n_mats; ++i) {
    if (bad(g.mom[i]) || bad(g.var[i]) || (g.mom_rot && bad(g.mom_rot[i])))
      return fail(CANZ_EINVAL, "group %d: moment %d null or not 16-byte aligned", idx, i);
    if (u.left && (bad(g.left[i]) || bad(g.qleft[i])))
      return fail(CANZ_EINVAL, "group %d: left state %d null or not 16-byte aligned", idx, i);
    if (u.right && (bad(g.right[i]) || bad(g.qright[i])))
      return fail(CANZ_EINVAL, "group %d: right state %d null or not 16-byte aligned", idx, i);
  }
  for (int i = 0; i < n_out; ++i)
    if (bad(g.out[i])) return fail(CANZ_EINVAL, "group %d: out[%d] null or not 16-byte aligned", idx, i);
  return CANZ_OK;
}

// Basis refresh of the sides of a batch (one or two, the longer first): q (caller's, d x d) <- Q factor of QR(S q), S the padded
// statistic in `qt` [nb][dp][dp] (later Q^T), the transposed padded copy of the current basis in `vall` (later the reflectors).
// `product`: S q is in `wk` already.
int refresh(const QrSide* side, int n_sides, bool product, void* const* const* q_tab, int first, int nb, const Shape& s, const OutSpec& o,
            hipStream_t st) {
  const PtrTable none{};
  QrArgs a{};
  a.nb = nb;
  for (int i = 0; i < n_sides; ++i) a.side[i] = side[i];
  auto dd = [&](int i) { return static_cast<int64_t>(side[i].dp) * side[i].dp; };
  auto check = [&](const char* what) -> int {
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "refresh, %s: %s", what, hipGetErrorString(e));
    return CANZ_OK;
  };
  // one product per side (`make` gives it, M = 0: nothing to do) in one launch
  auto products = [&](auto epi, auto transposed, int sides, auto&& make, const char* what) -> int {
    ShGemm g[2]{};
    int64_t blocks[2] = {0, 0};
    for (int i = 0; i < sides; ++i) {
      g[i] = make(i);
      blocks[i] = g[i].M / SB * (g[i].N / SB) * nb;
    }
    if (blocks[0] + blocks[1] == 0) return CANZ_OK;
    prof_mark(st, CANZ_KERNEL_SOAP_QR, true);
    hipLaunchKernelGGL((k_qr_gemm<decltype(epi)::value, decltype(transposed)::value>), dim3(static_cast<unsigned>(blocks[0] + blocks[1])),
                       dim3(NTH), 0, st, g[0], g[1], static_cast<int>(blocks[0]), none, s, o);
    prof_mark(st, CANZ_KERNEL_SOAP_QR, false);
    return check(what);
  };
  using Plain = std::integral_constant<int, SE_PLAIN>;
  using Sub = std::integral_constant<int, SE_SUB>;

  // working copy, transposed: wk[c][r] = (S q)[r][c] = sum_k qt_old[c][k] S[r][k]
  if (int rc = product ? CANZ_OK : products(Plain{}, std::false_type{}, n_sides, [&](int i) {
        ShGemm g{};
        g.M = g.N = g.K = g.ldp = g.ldq = g.ldc = side[i].dp, g.sp = g.sq = g.sc = dd(i);
        g.P = side[i].vall, g.Q = side[i].qt, g.c = side[i].wk;
        return g;
      }, "product with the statistic")) return rc;
  prof_mark(st, CANZ_KERNEL_SOAP_PANEL, true);
  for (int i = 0; i < n_sides; ++i) {   // nothing else has to start from a known state: what is read is written first
    const unsigned blocks = static_cast<unsigned>(std::min<int64_t>(2048, (dd(i) + NTH - 1) / NTH));
    hipLaunchKernelGGL(k_soap_fill, dim3(blocks, nb), dim3(NTH), 0, st, side[i].qt, dd(i), static_cast<int64_t>(side[i].dp), 1);
  }
  prof_mark(st, CANZ_KERNEL_SOAP_PANEL, false);
  if (int rc = check("fill")) return rc;

  // X -= W' V^T in the rows lo.. and the columns jb.. of the sides' matrices
  auto block_sub = [&](int sides, bool back, int jb, int lo, const char* what) -> int {
    return products(Sub{}, std::true_type{}, sides, [&](int i) {
      ShGemm g{};
      const int64_t dp = side[i].dp;
      if (lo >= dp) return g;
      g.M = dp - lo, g.N = dp - jb, g.K = QBLK, g.ldp = QBLK, g.ldq = dp, g.sp = dp * QBLK, g.sq = dd(i);
      g.P = side[i].strip + static_cast<int64_t>(lo) * QBLK, g.Q = side[i].vall + jb * dp + jb;
      g.c = (back ? side[i].qt : side[i].wk) + lo * dp + jb, g.ldc = dp, g.sc = dd(i);
      return g;
    }, what);
  };
  auto panel = [&](const QrArgs& p, int rows, int mats) {
    const dim3 grid(static_cast<unsigned>(mats)), block(QTH);
    if (rows <= 64 * 4 * 2)
      hipLaunchKernelGGL(k_qr_panel_regs<2>, grid, block, 0, st, p);
    else if (rows <= 64 * 4 * 4)
      hipLaunchKernelGGL(k_qr_panel_regs<4>, grid, block, 0, st, p);
    else if (rows <= 64 * 4 * 8)
      hipLaunchKernelGGL(k_qr_panel_regs<8>, grid, block, 0, st, p);
    else if (rows <= 64 * 4 * 12)
      hipLaunchKernelGGL(k_qr_panel_long<12>, grid, block, 0, st, p);
    else
      hipLaunchKernelGGL(k_qr_panel_hybrid<8>, grid, block, 0, st, p);
  };
  const int dp0 = side[0].dp;
  for (int jb = 0; jb < dp0; jb += QBLK) {              // factorisation, block by block
    const int sides = n_sides == 2 && jb < side[1].dp ? 2 : 1;
    const unsigned mats = static_cast<unsigned>(nb * sides);
    a.jb = jb;
    int units = (dp0 - jb) / QBLK;
    const unsigned chunks = static_cast<unsigned>(std::min(units, QCHUNKS));
    for (a.pos = 0; a.pos < 4; ++a.pos) {
      prof_mark(st, CANZ_KERNEL_SOAP_PANEL, true);
      const int rows0 = dp0 - jb - QB * a.pos, rows1 = sides == 2 ? side[1].dp - jb - QB * a.pos : rows0;
      if (rows0 > 64 * 4 * 12 && rows1 <= 64 * 4 * 8) {   // the kernel for long columns has no place for such short ones
        QrArgs one = a;
        one.side[0] = side[1];
        panel(a, rows0, nb);
        panel(one, rows1, nb);
      } else {
        panel(a, rows0, static_cast<int>(mats));
      }
      hipLaunchKernelGGL(k_qr_gram, dim3(chunks, mats), dim3(NTH), 0, st, a);
      if (a.pos < 3)
        hipLaunchKernelGGL(k_qr_panel_sub, dim3(static_cast<unsigned>(units), mats), dim3(NTH), 0, st, a);
      else
        hipLaunchKernelGGL(k_qr_block_t, dim3(mats), dim3(QTH), 0, st, a);
      prof_mark(st, CANZ_KERNEL_SOAP_PANEL, false);
      if (int rc = check("panel kernels")) return rc;
    }
    if (jb + QBLK >= dp0) break;   // no columns after this block
    prof_mark(st, CANZ_KERNEL_SOAP_QR, true);
    hipLaunchKernelGGL(k_qr_block_w<false>, dim3(static_cast<unsigned>((dp0 - jb - QBLK) / 32), mats), dim3(NTH), 0, st, a, jb + QBLK);
    prof_mark(st, CANZ_KERNEL_SOAP_QR, false);
    if (int rc = check("block of reflectors")) return rc;
    if (int rc = block_sub(sides, false, jb, jb + QBLK, "QR (block update)")) return rc;
  }
  // Q = H(0) H(1) ... applied to the identity from the last block to the first
  for (int jb = dp0 - QBLK; jb >= 0; jb -= QBLK) {
    const int sides = n_sides == 2 && jb < side[1].dp ? 2 : 1;
    a.jb = jb;
    prof_mark(st, CANZ_KERNEL_SOAP_QR, true);
    hipLaunchKernelGGL(k_qr_block_w<true>, dim3(static_cast<unsigned>((dp0 - jb) / 32), static_cast<unsigned>(nb * sides)), dim3(NTH), 0, st, a, jb);
    prof_mark(st, CANZ_KERNEL_SOAP_QR, false);
    if (int rc = check("block of reflectors (Q)")) return rc;
    if (int rc = block_sub(sides, true, jb, jb, "Q (block update)")) return rc;
  }
  prof_mark(st, CANZ_KERNEL_SOAP_PANEL, true);
  for (int i = 0; i < n_sides; ++i) {
    PtrTable q{};
    for (int k = 0; k < nb; ++k) q.p[k] = q_tab[i][first + k];
    const unsigned t64 = static_cast<unsigned>(side[i].dp / 64);
    hipLaunchKernelGGL(k_soap_store_q, dim3(t64, t64, static_cast<unsigned>(nb)), dim3(NTH), 0, st, q, side[i].qt,
                       static_cast<int64_t>(side[i].d), static_cast<int64_t>(side[i].dp));
  }
  prof_mark(st, CANZ_KERNEL_SOAP_PANEL, false);
  return check("basis store");
}

// One launch batch: matrices first .. first + nb - 1 of group g.
int run_batch(const canz_soap_group& g, int first, int nb, Rot rot, const canz_soap_hparams& hp, float* ws, hipStream_t st) {
  const int64_t rp = pad128(g.rows), cp = pad128(g.cols), plane = rp * cp;
  const Sides u = sides(g, hp);
  const bool bf16 = rot == Rot::BF16, terms3 = rot == Rot::TERMS, f32 = rot == Rot::F32;
  const bool stat16 = bf16_statistics(g);
  const Carve c = carve(g.rows, g.cols, nb, u, hp.refresh != 0, rot, stat16);
  Shape s{};
  s.rows = g.rows, s.cols = g.cols;
  s.m = std::min(g.rows, g.cols), s.n = std::max(g.rows, g.cols);
  s.mp = rp, s.np = cp;
  s.tall = g.rows > g.cols;
  s.tp = g.tp;
  s.wfrag = g.cols / g.tp;
  PtrTable grad{}, mom{}, var{}, none{};
  for (int i = 0; i < nb * g.tp; ++i) grad.p[i] = const_cast<void*>(g.grad[first * g.tp + i]);
  for (int i = 0; i < nb; ++i) mom.p[i] = g.mom[first + i], var.p[i] = g.var[first + i];
  OutSpec o{};
  const int per_out = hp.out_mode == CANZ_OUT_DELTA ? g.tp : 1;
  for (int i = 0; i < nb * per_out; ++i) o.out.p[i] = g.out[first * per_out + i];
  o.out_dtype = g.out_dtype;
  o.out_mode = hp.out_mode;
  o.decay = static_cast<float>(1.0 - static_cast<double>(hp.lr) * static_cast<double>(hp.weight_decay));
  o.neg_lr_scale = -hp.lr;

  float *gm = ws + c.gm, *gmt = ws + c.gmt;

  // With a valid rotated momentum from the caller only G is rotated (M' follows its own recurrence in the rotated
  // space, which is the same linear map as long as the bases stand still); otherwise G and M.
  const bool incremental = g.mom_rot != nullptr && hp.mom_rot_valid != 0;
  // bf16 images in the panel layout (padded to 256): operands of the bf16 rotations and of the statistics
  const int64_t rp2 = pad256(g.rows), cp2 = pad256(g.cols), p2 = rp2 * cp2;
  const SplitWs no_split{nullptr, 0};
  auto pan = [&](size_t at) { return reinterpret_cast<__bf16*>(ws + at); };
  const int64_t g_stride = f32 ? 2 * plane : plane;   // from one matrix's fp32 copy of G to the next

  prof_mark(st, CANZ_KERNEL_SOAP_LOAD, true);
  {
    // fp32 copies: G for the fp32 statistics, G and M side by side for rotations on fp32 matrices; bf16 images: G for the bf16 statistics and for either kind of rotation if it
    // arrives as bf16, M for the bf16 rotations of a step that rotates it (also the re-rotation of a kept M' after a
    // refresh); three terms: G that is fp32 and M for the fp32 rotations, in the orientation of the first product
    LoadOut w{};
    if (f32 || !stat16) w.gm = gm, w.gmt = gmt;
    if (f32) w.mm = gm + plane, w.mmt = gmt + plane;
    w.stride = g_stride;
    const bool rotate_m = !incremental || (hp.refresh && g.mom_rot != nullptr);
    if (terms3 && !stat16) (u.right ? w.g3 : w.g3t) = pan(u.right ? c.g3 : c.g3t);
    if (terms3 && rotate_m) (u.right ? w.m3 : w.m3t) = pan(u.right ? c.m3 : c.m3t);
    w.rp2 = rp2, w.cp2 = cp2;
    if (bf16 || (stat16 && (terms3 || u.left))) w.gp = pan(c.gp);
    if (bf16 || (stat16 && (terms3 || u.right))) w.gpt = pan(c.gpt);
    if (bf16 && rotate_m) w.mp = pan(c.mp), w.mpt = pan(c.mpt);
    const dim3 grid(static_cast<unsigned>(cp2 / 64), static_cast<unsigned>(rp2 / 64), static_cast<unsigned>(nb));
    if (g.cols % 8 == 0 && s.wfrag % 8 == 0)
      hipLaunchKernelGGL(k_soap_load<true>, grid, dim3(NTH), 0, st, s, grad, g.grad_dtype, mom, hp.beta1, rp, cp, w);
    else
      hipLaunchKernelGGL(k_soap_load<false>, grid, dim3(NTH), 0, st, s, grad, g.grad_dtype, mom, hp.beta1, rp, cp, w);
  }
  // the bases, zero outside d x d: three terms, fp32 copies or bf16 images for the three kinds of rotations, in both
  // orientations; later, fp32 and transposed, for the refresh (which multiplies the new statistic with the old basis)
  auto load_basis = [&](void* const* tab, int64_t d, int64_t dp, int64_t dp2, BasisOut w) {
    PtrTable q{};
    for (int i = 0; i < nb; ++i) q.p[i] = tab[first + i];
    const unsigned side = static_cast<unsigned>(dp2 / 64);
    hipLaunchKernelGGL(k_soap_load_basis, dim3(side, side, static_cast<unsigned>(nb)), dim3(NTH), 0, st, q, d, dp, dp2, w);
  };
  auto basis_out = [&](size_t s32, size_t t32, size_t sp, size_t tp, size_t s3, size_t t3) {
    BasisOut w{};
    if (f32) w.s32 = ws + s32, w.t32 = ws + t32;
    if (bf16) w.sp = pan(sp), w.tp = pan(tp);
    if (terms3) w.s3 = pan(s3), w.t3 = pan(t3);
    return w;
  };
  if (u.left) load_basis(g.qleft, g.rows, rp, f32 ? rp : rp2, basis_out(c.ql, c.qlt, c.qlp, c.qltp, c.ql3, c.ql3t));
  if (u.right) load_basis(g.qright, g.cols, cp, f32 ? cp : cp2, basis_out(c.qr, c.qrt, c.qrp, c.qrtp, c.qr3, c.qr3t));
  prof_mark(st, CANZ_KERNEL_SOAP_LOAD, false);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "load kernels: %s", hipGetErrorString(e));

  // The fp32 rotations run on the bf16 cores as well: the bases, M, N' and the intermediates are three bf16 terms per
  // element (G too, if it is not bf16 itself), a product is six products of terms (three with a bf16 G) with fp32 sums
  // (launch_split3).  At the rates the two kinds of core reach here (1.3 PFLOP/s against 150 TFLOP/s) that is 0.7 (0.35) of
  // the fp32 MFMA's time, and closer to 64 bits, since that core rounds its sum every two k.  A plain step of
  // 8 x 3072 x 1024 with bf16 gradients takes 2.78 ms against 4.00 ms with fp32 MFMA products; error of the update
  // 0.9e-7 against 2.7e-7.
  // X' = Q_L^T X Q_R for X [rp2][cp2] (two-sided or right side only) or X^T (left side only) of `terms` terms, dense
  // rows x cols to the buffers of `to`
  auto rotate_in = [&](const __bf16* x, int terms, const PtrTable& to) -> int {
    Shape whole = s;
    whole.tp = 1, whole.wfrag = g.cols;
    OutSpec ro{};
    ro.out = to, ro.out_dtype = CANZ_DT_F32, ro.out_mode = CANZ_OUT_DELTA, ro.decay = 1.f, ro.neg_lr_scale = 1.f;
    if (!u.left) {   // X Q_R
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_terms_final(split3_dims(rp2, cp2, cp2, 3, nb, terms), x, pan(c.qr3t), whole, ro, st),
               "rotation (right)");
      return CANZ_OK;
    }
    if (u.right) {   // (X Q_R)^T [cp2][3 rp2]
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_split3(split3_dims(cp2, rp2, cp2, terms, nb), pan(c.qr3t), x, pan(c.t3), st),
               "rotation (right)");
      x = pan(c.t3), terms = 3;
    }
    CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_terms_final(split3_dims(rp2, cp2, rp2, terms, nb), pan(c.ql3t), x, whole, ro, st),
             "rotation (left)");
    return CANZ_OK;
  };
  // On fp32 matrices (plan_of): rotation into the bases of `per` planes of each matrix's (G, M) pair, from plane `p0` on: problem p is
  // plane p0 + p % per of matrix p / per; consecutive problems of a matrix share the basis operand
  float *t1 = ws + c.t1, *rot32 = ws + c.rot, *ql = ws + c.ql, *qlt = ws + c.qlt, *qr = ws + c.qr, *qrt = ws + c.qrt;
  auto rotate_in32 = [&](int p0, int per) -> int {
    const int64_t step_ = per == 2 ? plane : 2 * plane, at = p0 * plane;
    const int count = per * nb;
    if (u.left && u.right) {
      ShGemm a{};   // t1 = (X Q_R)^T: [cp][rp]
      a.M = cp, a.N = rp, a.K = cp, a.ldp = cp, a.ldq = cp, a.sp = cp * cp, a.pshare = per - 1, a.sq = step_;
      a.P = qrt, a.Q = gm + at, a.c = t1 + at, a.ldc = rp, a.sc = step_;
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, (launch_gemm<SE_PLAIN, false, true>(a, count, none, s, o, st)), "rotation (right)");
      ShGemm bq{};  // rot32 = Q_L^T (X Q_R): [rp][cp]
      bq.M = rp, bq.N = cp, bq.K = rp, bq.ldp = rp, bq.ldq = rp, bq.sp = rp * rp, bq.pshare = per - 1, bq.sq = step_;
      bq.P = qlt, bq.Q = t1 + at, bq.c = rot32 + at, bq.ldc = cp, bq.sc = step_;
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, (launch_gemm<SE_PLAIN, false, true>(bq, count, none, s, o, st)), "rotation (left)");
    } else if (u.left) {
      ShGemm bq{};  // rot32 = Q_L^T X with X^T as the second operand
      bq.M = rp, bq.N = cp, bq.K = rp, bq.ldp = rp, bq.ldq = rp, bq.sp = rp * rp, bq.pshare = per - 1, bq.sq = step_;
      bq.P = qlt, bq.Q = gmt + at, bq.c = rot32 + at, bq.ldc = cp, bq.sc = step_;
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, (launch_gemm<SE_PLAIN, false, true>(bq, count, none, s, o, st)), "rotation (left)");
    } else {
      ShGemm a{};   // rot32 = X Q_R
      a.M = rp, a.N = cp, a.K = cp, a.ldp = cp, a.ldq = cp, a.sp = step_, a.sq = cp * cp, a.qshare = per - 1;
      a.P = gm + at, a.Q = qrt, a.c = rot32 + at, a.ldc = cp, a.sc = step_;
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, (launch_gemm<SE_PLAIN, false, true>(a, count, none, s, o, st)), "rotation (right)");
    }
    return CANZ_OK;
  };
  PtrTable mrot{};
  if (g.mom_rot)
    for (int i = 0; i < nb; ++i) mrot.p[i] = g.mom_rot[first + i];
  const double c1 = hp.bias_correction ? 1.0 / (1.0 - std::pow(static_cast<double>(hp.beta1), hp.step)) : 1.0;
  const double c2 = hp.bias_correction ? 1.0 / (1.0 - std::pow(static_cast<double>(hp.beta2), hp.step)) : 1.0;

  const int want_transposed = u.left && !u.right;   // the left side alone takes N'^T as its second operand
  const dim3 tiles2(static_cast<unsigned>(cp2 / 64), static_cast<unsigned>(rp2 / 64), static_cast<unsigned>(nb));
  auto adam = [&](const float* g_rot, const float* m_rot, int64_t ld, int64_t stride, __bf16* n3, float* n32) -> int {
    prof_mark(st, CANZ_KERNEL_SOAP_ADAM, true);
    hipLaunchKernelGGL(k_soap_adam, tiles2, dim3(NTH), 0, st, s, var, mrot, g.mom_rot != nullptr, incremental, g_rot, m_rot, ld, stride, rp2,
                       cp2, hp.beta1, hp.beta2, static_cast<float>(c1), static_cast<float>(c2), hp.eps, want_transposed, n3, n32);
    prof_mark(st, CANZ_KERNEL_SOAP_ADAM, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "adam kernel: %s", hipGetErrorString(e));
    return CANZ_OK;
  };

  // shapes of the bf16 rotation products (first operand: a basis)
  const GemmDims right_dims{cp2, rp2, cp2, cp2, cp2, cp2 * cp2, p2, nb};   // (basis rows) x (matrix rows), k over columns
  const GemmDims left_dims{rp2, cp2, rp2, rp2, rp2, rp2 * rp2, p2, nb};    // (basis rows) x (matrix columns), k over rows
  if (bf16) {
    // The rotations on the bf16 matrix cores (fp32 accumulation): the bases, G (and M on a step that rotates it) and
    // N' are rounded to bf16 once each, the intermediate of a two-sided rotation once more; momentum, second
    // moment, the statistics' accumulation and the refresh stay in fp32.  The products reuse the update kernel of the
    // Muon step (it writes its result in both orientations, which is what the next product wants as its second
    // operand) and its last product (which writes the parameter update).
    // X' = Q_L^T X Q_R for X given as straight and transposed panels; the result as straight panels
    auto rotate_in16 = [&](const __bf16* xs, const __bf16* xt, size_t as_, size_t at_, size_t r_, size_t rt_,
                           const __bf16** result) -> int {
      if (u.right)   // as = (X Q_R)^T [cp2][rp2], at = X Q_R [rp2][cp2]
        CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_update_bf16(right_dims, pan(c.qrtp), xs, pan(as_), pan(at_), nullptr, no_split, st),
                 "rotation (right, bf16)");
      if (u.left)    // r = Q_L^T (.) [rp2][cp2] from the transposed image of what the right side left (or of X)
        CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE,
                 launch_update_bf16(left_dims, pan(c.qltp), u.right ? pan(as_) : xt, pan(r_), pan(rt_), nullptr, no_split, st),
                 "rotation (left, bf16)");
      *result = u.left ? pan(r_) : pan(at_);
      return CANZ_OK;
    };
    const __bf16 *g_rot = nullptr, *m_rot = nullptr;
    if (int rc = rotate_in16(pan(c.gp), pan(c.gpt), c.as_g, c.at_g, c.rg, c.rgt, &g_rot)) return rc;
    if (!incremental)
      if (int rc = rotate_in16(pan(c.mp), pan(c.mpt), c.as_m, c.at_m, c.rm, c.rmt, &m_rot)) return rc;
    prof_mark(st, CANZ_KERNEL_SOAP_ADAM, true);
    hipLaunchKernelGGL(k_soap_adam_bf16, tiles2, dim3(NTH), 0, st, s, var, mrot, g.mom_rot != nullptr, incremental, g_rot, m_rot,
                       rp2, cp2, hp.beta1, hp.beta2, static_cast<float>(c1), static_cast<float>(c2), hp.eps,
                       want_transposed ? nullptr : pan(c.npn), want_transposed ? pan(c.npt) : nullptr);
    prof_mark(st, CANZ_KERNEL_SOAP_ADAM, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "adam kernel: %s", hipGetErrorString(e));
    if (u.left && u.right) {
      // ys = (N' Q_R^T)^T [cp2][rp2]; then Q_L times it, into the caller's buffers
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_update_bf16(right_dims, pan(c.qrp), pan(c.npn), pan(c.ys), pan(c.yst), nullptr, no_split, st),
               "back rotation (right, bf16)");
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_final_bf16(left_dims, pan(c.qlp), pan(c.ys), nullptr, no_split, s, o, st),
               "back rotation (left, bf16)");
    } else if (u.left) {
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_final_bf16(left_dims, pan(c.qlp), pan(c.npt), nullptr, no_split, s, o, st),
               "back rotation (left, bf16)");
    } else {
      const GemmDims d{rp2, cp2, cp2, cp2, cp2, p2, cp2 * cp2, nb};   // N' [rp2][cp2] times Q_R^T
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_final_bf16(d, pan(c.npn), pan(c.qrp), nullptr, no_split, s, o, st),
               "back rotation (right, bf16)");
    }
  } else if (f32) {
    float *np = ws + c.np, *yt = ws + c.yt;
    if (int rc = rotate_in32(0, incremental ? 1 : 2)) return rc;
    if (int rc = adam(rot32, rot32 + plane, cp, 2 * plane, nullptr, np)) return rc;
    // rotation back, the last product writes the update
    if (u.left && u.right) {
      ShGemm cq{};  // yt = (N' Q_R^T)^T: [cp][rp]
      cq.M = cp, cq.N = rp, cq.K = cp, cq.ldp = cp, cq.ldq = cp, cq.sp = cp * cp, cq.sq = plane;
      cq.P = qr, cq.Q = np, cq.c = yt;
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, (launch_gemm<SE_PLAIN, false>(cq, nb, none, s, o, st)), "back rotation (right)");
      ShGemm dq{};
      dq.M = rp, dq.N = cp, dq.K = rp, dq.ldp = rp, dq.ldq = rp, dq.sp = rp * rp, dq.sq = plane;
      dq.P = ql, dq.Q = yt;
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, (launch_gemm<SE_OUT, false>(dq, nb, none, s, o, st)), "back rotation (left)");
    } else if (u.left) {
      ShGemm dq{};  // np holds N'^T
      dq.M = rp, dq.N = cp, dq.K = rp, dq.ldp = rp, dq.ldq = rp, dq.sp = rp * rp, dq.sq = plane;
      dq.P = ql, dq.Q = np;
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, (launch_gemm<SE_OUT, false>(dq, nb, none, s, o, st)), "back rotation (left)");
    } else {
      ShGemm cq{};
      cq.M = rp, cq.N = cp, cq.K = cp, cq.ldp = cp, cq.ldq = cp, cq.sp = plane, cq.sq = cp * cp;
      cq.P = np, cq.Q = qr;
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, (launch_gemm<SE_OUT, false>(cq, nb, none, s, o, st)), "back rotation (right)");
    }
  } else {
    auto dense = [&](size_t at) {   // the batch's dense rows x cols matrices in the workspace
      PtrTable t{};
      for (int i = 0; i < nb; ++i) t.p[i] = ws + at + i * dense_stride(g.rows, g.cols);
      return t;
    };
    const __bf16* gx = stat16 ? pan(u.right ? c.gp : c.gpt) : pan(u.right ? c.g3 : c.g3t);
    if (int rc = rotate_in(gx, stat16 ? 1 : 3, dense(c.rotg))) return rc;
    if (!incremental)
      if (int rc = rotate_in(pan(u.right ? c.m3 : c.m3t), 3, dense(c.rotm))) return rc;
    if (int rc = adam(ws + c.rotg, ws + c.rotm, g.cols, dense_stride(g.rows, g.cols), pan(c.n3), nullptr)) return rc;

    // rotation back, the last product writes the update
    if (!u.left) {
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_terms_final(split3_dims(rp2, cp2, cp2, 3, nb), pan(c.n3), pan(c.qr3), s, o, st),
               "back rotation (right)");
    } else {
      const __bf16* n = pan(c.n3);
      if (u.right) {   // (N' Q_R^T)^T [cp2][3 rp2]
        CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_split3(split3_dims(cp2, rp2, cp2, 3, nb), pan(c.qr3), n, pan(c.y3), st),
                 "back rotation (right)");
        n = pan(c.y3);
      }
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_terms_final(split3_dims(rp2, cp2, rp2, 3, nb), pan(c.ql3), n, s, o, st),
               "back rotation (left)");
    }
  }

  // Statistics; on a refresh step also the padded copies of the new statistic and of the transposed old basis.  What the refresh of a side works
  // on lies in the pool, one side behind the other, but for the statistic and Q^T, which take the place of the side's basis: the update is
  // out, and its images are not needed again (three terms: 1.5 d^2 an orientation; bf16: half that, both; fp32: d^2).
  QrSide side[2]{};
  void* const* side_q[2]{};
  int n_sides = 0;
  float* pool = ws + c.pool;
  auto one_side = [&](void* const* stat_tab, void* const* q_tab, int64_t d, int64_t dp, int64_t kp, const float* grad32, const __bf16* grad16,
                      int64_t d2, int64_t k2, size_t stat_at, size_t basis_t3) -> int {
    PtrTable tab{};
    for (int i = 0; i < nb; ++i) tab.p[i] = stat_tab[first + i];
    QrSide qs{};
    if (hp.refresh) {
      const int64_t dd = dp * dp;
      qs.wk = pool, qs.vall = qs.wk + nb * dd, qs.strip = qs.vall + nb * dd, qs.tt = qs.strip + nb * dp * QBLK;
      qs.gram = qs.tt + nb * dp * QBLK, qs.tau = qs.gram + nb * QBLK * QBLK;
      pool = qs.tau + nb * QBLK;
      qs.qt = ws + stat_at;
      qs.dp = static_cast<int>(dp), qs.d = static_cast<int>(d);
    }
    if (stat16) {
      Shape sq{};   // the caller's dense d x d matrix
      sq.rows = d, sq.cols = d, sq.m = d, sq.n = d, sq.tp = 1, sq.wfrag = d;
      if (int rc = statistic_bf16(CANZ_KERNEL_SOAP_STAT, tab, d, d2, k2, k2, nb, hp.beta2, 1.f - hp.beta2, grad16, st)) return rc;
      if (hp.refresh && !terms3) {   // (the transposed image lands in wk, unused)
        prof_mark(st, CANZ_KERNEL_SOAP_STAT, true);
        hipLaunchKernelGGL(k_sh_load, dim3(static_cast<unsigned>(dp / 64), static_cast<unsigned>(dp / 64), static_cast<unsigned>(nb)),
                           dim3(NTH), 0, st, sq, tab, static_cast<int>(CANZ_DT_F32), dp, dp, qs.qt, qs.wk);
        prof_mark(st, CANZ_KERNEL_SOAP_STAT, false);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "statistic copy: %s", hipGetErrorString(e));
      }
    } else {
      ShGemm q{};
      q.M = dp, q.N = dp, q.K = kp, q.ldp = kp, q.ldq = kp, q.sp = g_stride, q.sq = g_stride;
      q.P = grad32, q.Q = grad32, q.c = terms3 ? nullptr : qs.qt, q.d = d, q.beta = hp.beta2, q.gscale = 1.f - hp.beta2, q.eps = 0.f;
      CANZ_HIP(CANZ_KERNEL_SOAP_STAT, (launch_gemm<SE_STAT, true>(q, nb, tab, s, o, st)), "statistics kernel");
    }
    if (!hp.refresh) return CANZ_OK;
    prof_mark(st, CANZ_KERNEL_SOAP_LOAD, true);
    if (terms3)
      hipLaunchKernelGGL(k_terms3, dim3(static_cast<unsigned>(d2 / 64), static_cast<unsigned>(d2 / 64), static_cast<unsigned>(nb)), dim3(NTH), 0, st,
                         tab, d, d, d2, reinterpret_cast<__bf16*>(qs.qt));
    else
      load_basis(q_tab, d, dp, dp, BasisOut{nullptr, qs.vall, nullptr, nullptr, nullptr, nullptr});
    prof_mark(st, CANZ_KERNEL_SOAP_LOAD, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "basis load: %s", hipGetErrorString(e));
    if (terms3) {
      // S q, transposed, on three terms as the rotations (4 x 2048^2 and 1024^2: 708 us on the fp32 cores, 440 so): the transposed old
      // basis is there from the rotation into it, the statistic takes the place of the straight one
      Shape sq{};
      sq.rows = sq.cols = sq.m = sq.n = dp, sq.mp = sq.np = d2, sq.tp = 1, sq.wfrag = dp;
      OutSpec wo{};
      for (int i = 0; i < nb; ++i) wo.out.p[i] = qs.wk + i * dp * dp;
      wo.out_dtype = CANZ_DT_F32, wo.out_mode = CANZ_OUT_DELTA, wo.decay = 1.f, wo.neg_lr_scale = 1.f;
      CANZ_HIP(CANZ_KERNEL_SOAP_QR, launch_terms_final(split3_dims(d2, d2, d2, 3, nb), pan(basis_t3), reinterpret_cast<const __bf16*>(qs.qt), sq, wo, st),
               "refresh product");
    }
    const int at = n_sides == 1 && qs.dp > side[0].dp ? 0 : n_sides;   // the longer side first
    if (at == 0) side[1] = side[0], side_q[1] = side_q[0];
    side[at] = qs, side_q[at] = q_tab;
    ++n_sides;
    return CANZ_OK;
  };
  auto basis_at = [&](size_t terms_at, size_t bf16_at, size_t f32_at) { return terms3 ? terms_at : bf16 ? bf16_at : f32_at; };
  if (u.left)
    if (int rc = one_side(g.left, g.qleft, g.rows, rp, cp, gm, pan(c.gp), rp2, cp2, basis_at(c.ql3, c.qlp, c.ql), c.ql3t)) return rc;
  if (u.right)
    if (int rc = one_side(g.right, g.qright, g.cols, cp, rp, gmt, pan(c.gpt), cp2, rp2, basis_at(c.qr3, c.qrp, c.qr), c.qr3t)) return rc;
  if (hp.refresh)
    if (int rc = refresh(side, n_sides, terms3, side_q, first, nb, s, o, st)) return rc;
  if (hp.refresh && g.mom_rot && bf16) {
    // the caller's rotated momentum follows the new bases, M' = Q_L^T M Q_R once more with the M of this step: bf16
    // operands as for every rotation of this mode; the last product leaves its fp32 sums in the caller's array
    prof_mark(st, CANZ_KERNEL_SOAP_LOAD, true);
    if (u.left) load_basis(g.qleft, g.rows, rp, rp2, BasisOut{nullptr, nullptr, nullptr, pan(c.qltp), nullptr, nullptr});
    if (u.right) load_basis(g.qright, g.cols, cp, cp2, BasisOut{nullptr, nullptr, nullptr, pan(c.qrtp), nullptr, nullptr});
    prof_mark(st, CANZ_KERNEL_SOAP_LOAD, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "basis load: %s", hipGetErrorString(e));
    Shape whole = s;
    whole.tp = 1, whole.wfrag = g.cols;
    OutSpec mo{};
    mo.out = mrot, mo.out_dtype = CANZ_DT_F32, mo.out_mode = CANZ_OUT_DELTA, mo.decay = 1.f, mo.neg_lr_scale = 1.f;
    if (u.left && u.right) {
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE,
               launch_update_bf16(right_dims, pan(c.qrtp), pan(c.mp), pan(c.as_m), pan(c.at_m), nullptr, no_split, st),
               "momentum re-rotation (right, bf16)");
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_final_bf16(left_dims, pan(c.qltp), pan(c.as_m), nullptr, no_split, whole, mo, st),
               "momentum re-rotation (left, bf16)");
    } else if (u.left) {
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_final_bf16(left_dims, pan(c.qltp), pan(c.mpt), nullptr, no_split, whole, mo, st),
               "momentum re-rotation (left, bf16)");
    } else {
      const GemmDims d{rp2, cp2, cp2, cp2, cp2, p2, cp2 * cp2, nb};   // M [rp2][cp2] times (Q_R^T)^T
      CANZ_HIP(CANZ_KERNEL_SOAP_ROTATE, launch_final_bf16(d, pan(c.mp), pan(c.qrtp), nullptr, no_split, whole, mo, st),
               "momentum re-rotation (right, bf16)");
    }
  } else if (hp.refresh && g.mom_rot && f32) {
    // the same on fp32 matrices
    prof_mark(st, CANZ_KERNEL_SOAP_LOAD, true);
    if (u.left) load_basis(g.qleft, g.rows, rp, rp, BasisOut{nullptr, qlt, nullptr, nullptr, nullptr, nullptr});
    if (u.right) load_basis(g.qright, g.cols, cp, cp, BasisOut{nullptr, qrt, nullptr, nullptr, nullptr, nullptr});
    prof_mark(st, CANZ_KERNEL_SOAP_LOAD, false);
    if (int rc = rotate_in32(1, 1)) return rc;
    prof_mark(st, CANZ_KERNEL_SOAP_ADAM, true);
    hipLaunchKernelGGL(k_unpad, dim3(static_cast<unsigned>(cp / 64), static_cast<unsigned>(rp / 64), static_cast<unsigned>(nb)), dim3(NTH), 0, st,
                       s, mrot, rot32 + plane, 2 * plane, cp);
    prof_mark(st, CANZ_KERNEL_SOAP_ADAM, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "momentum re-rotation: %s", hipGetErrorString(e));
  } else if (hp.refresh && g.mom_rot) {
    // the same on three terms
    prof_mark(st, CANZ_KERNEL_SOAP_LOAD, true);
    if (u.left) load_basis(g.qleft, g.rows, rp, rp2, BasisOut{nullptr, nullptr, nullptr, nullptr, nullptr, pan(c.ql3t)});
    if (u.right) load_basis(g.qright, g.cols, cp, cp2, BasisOut{nullptr, nullptr, nullptr, nullptr, nullptr, pan(c.qr3t)});
    prof_mark(st, CANZ_KERNEL_SOAP_LOAD, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "basis load: %s", hipGetErrorString(e));
    if (int rc = rotate_in(pan(u.right ? c.m3 : c.m3t), 3, mrot)) return rc;
  }
  return CANZ_OK;
}

// Consecutive groups of a call that agree in shape, tp, dtypes and in which tables they pass run as one group: every
// matrix is computed on its own whatever shares its launch, a refresh keeps only one workgroup per matrix busy in
// its panel kernel, and its products are small - the more matrices share a launch, the better the chip is filled.
struct MergedGroup {
  canz_soap_group g{};
  std::vector<const void*> grad;
  std::vector<void*> tab[8];   // mom, var, left, right, qleft, qright, out, mom_rot
};

void* const* const* tables_of(const canz_soap_group& g, void* const* (&out)[8]) {
  out[0] = g.mom, out[1] = g.var, out[2] = g.left, out[3] = g.right, out[4] = g.qleft, out[5] = g.qright, out[6] = g.out,
  out[7] = g.mom_rot;
  return out;
}

bool mergeable(const canz_soap_group& a, const canz_soap_group& b) {
  if (a.rows != b.rows || a.cols != b.cols || a.tp != b.tp || a.grad_dtype != b.grad_dtype || a.out_dtype != b.out_dtype) return false;
  if ((a.grad == nullptr) != (b.grad == nullptr)) return false;
  void* const* ta[8];
  void* const* tb[8];
  tables_of(a, ta), tables_of(b, tb);
  for (int k = 0; k < 8; ++k)
    if ((ta[k] == nullptr) != (tb[k] == nullptr)) return false;
  return true;
}

std::vector<MergedGroup> merge_groups(const canz_soap_group* g, int n_groups, const canz_soap_hparams& hp) {
  std::vector<MergedGroup> all;
  const auto append = [&](MergedGroup& m, const canz_soap_group& x) {
    void* const* t[8];
    tables_of(x, t);
    const int per_out = hp.out_mode == CANZ_OUT_DELTA ? x.tp : 1;
    if (x.grad) m.grad.insert(m.grad.end(), x.grad, x.grad + static_cast<size_t>(x.n_mats) * x.tp);
    for (int k = 0; k < 8; ++k)
      if (t[k]) m.tab[k].insert(m.tab[k].end(), t[k], t[k] + static_cast<size_t>(x.n_mats) * (k == 6 ? per_out : 1));
    m.g.n_mats += x.n_mats;
  };
  for (int i = 0; i < n_groups; ++i) {
    if (g[i].n_mats == 0) continue;
    if (all.empty() || !mergeable(all.back().g, g[i])) {
      all.emplace_back();
      all.back().g = g[i];
      all.back().g.n_mats = 0;
    }
    append(all.back(), g[i]);
  }
  for (MergedGroup& m : all) {   // the tables now stand still: point the group at them
    canz_soap_group& x = m.g;
    if (x.grad) x.grad = m.grad.data();
    if (x.mom) x.mom = m.tab[0].data();
    if (x.var) x.var = m.tab[1].data();
    if (x.left) x.left = m.tab[2].data();
    if (x.right) x.right = m.tab[3].data();
    if (x.qleft) x.qleft = m.tab[4].data();
    if (x.qright) x.qright = m.tab[5].data();
    if (x.out) x.out = m.tab[6].data();
    if (x.mom_rot) x.mom_rot = m.tab[7].data();
  }
  return all;
}

}  // namespace
}  // namespace canz

extern "C" int canz_soap_workspace_bytes(const canz_soap_group* g, int32_t n_groups, const canz_soap_hparams* hp,
                                         size_t* bytes_out) {
  using namespace canz;
  if (!bytes_out) return fail(CANZ_EINVAL, "null bytes_out");
  if (n_groups < 0 || (n_groups > 0 && !g)) return fail(CANZ_EINVAL, "bad group array");
  if (int rc = check_hparams(hp)) return rc;
  size_t need = ALIGN;
  for (int i = 0; i < n_groups; ++i)
    if (int rc = check_group(g[i], i, false, *hp)) return rc;
  for (const MergedGroup& m : merge_groups(g, n_groups, *hp)) {
    const Plan p = plan_of(m.g, *hp, SIZE_MAX);
    need = std::max({need, batch_bytes(m.g, *hp, p.nb, p.rot), least_bytes(m.g, *hp)});
  }
  *bytes_out = need;
  return CANZ_OK;
}

extern "C" int canz_soap_step(const canz_soap_group* g, int32_t n_groups, const canz_soap_hparams* hp, void* workspace,
                              size_t workspace_bytes, void* hip_stream) {
  using namespace canz;
  size_t need = 0;   // of the fastest way; checks the arguments
  if (int rc = canz_soap_workspace_bytes(g, n_groups, hp, &need)) return rc;
  bool any = false;
  for (int i = 0; i < n_groups; ++i) {
    if (int rc = check_group(g[i], i, true, *hp)) return rc;
    any = any || g[i].n_mats > 0;
  }
  if (!any) return CANZ_OK;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (ALIGN - 1)))
    return fail(CANZ_EWORKSPACE, "workspace null or not 256-byte aligned");
  const std::vector<MergedGroup> merged = merge_groups(g, n_groups, *hp);
  for (const MergedGroup& m : merged)
    if (workspace_bytes < least_bytes(m.g, *hp))
      return fail(CANZ_EWORKSPACE, "workspace too small: %zu bytes given, %zu needed", workspace_bytes, need);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  for (const MergedGroup& m : merged) {
    const Plan p = plan_of(m.g, *hp, workspace_bytes);
    for (int first = 0; first < m.g.n_mats; first += p.nb)
      if (int rc = run_batch(m.g, first, std::min(p.nb, m.g.n_mats - first), p.rot, *hp, static_cast<float*>(workspace), st)) return rc;
  }
  return CANZ_OK;
}
