// fp32 products on v_mfma_f32_32x32x2_f32, shared by the Shampoo and SOAP steps (internal).
//
// All products have the form C[i][j] = sum_k P[i][k] Q[j][k] with both operands contiguous
// along k.  A product whose natural form is different is brought to this one by choosing
// which factor is P and which is Q (which decides whether C or its transpose is written) and
// by keeping the operands in the orientation their consumer needs.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "canz.h"
#include "canz_internal.h"
#include "device_util.h"
#include "kernels.h"
#include "panel_layout.h"

namespace canz {
namespace f32mfma {

constexpr int SB = 128;          // block tile (rows and columns)
constexpr int SK = 32;           // k extent of one LDS stage: long enough that the next stage's global loads land under it
constexpr int NTH = 256;
constexpr int LDS_LD = SB + 5;   // odd row length: the k-major stores of a stage spread over all banks
constexpr int FLUSH = 16;        // stages (512 k) between folds of the running accumulator
constexpr size_t ALIGN = 256;

inline int64_t pad128(int64_t x) { return (x + SB - 1) / SB * SB; }
inline size_t align_up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }

// Epilogues: SE_STAT  S <- beta S + gscale C into the caller's dense statistic, S + eps I to c;
//            SE_PLAIN c = C;   SE_MT  c = C and c2 = 5/4 I - 1/4 C;   SE_OUT  the optimizer update
//            into the caller's parameters or Delta W fragments;   SE_SUB  c <- c - C.
enum { SE_STAT = 0, SE_PLAIN = 1, SE_MT = 2, SE_OUT = 3, SE_SUB = 4 };

struct ShGemm {
  int64_t M, N, K;      // multiples of 128
  int64_t ldp, ldq;     // row strides of P [M][K] and Q [N][K]
  int64_t sp, sq;       // batch strides: matrix b reads P + b sp and Q + b sq
  const float* P;
  const float* Q;
  float* c;             // output
  int64_t ldc, sc;      // its row and batch strides; 0, 0 means dense: N and M * N
  // SE_STAT: the caller's statistic (d x d, dense) is updated in place and A = S + eps I is written to c
  int64_t d;
  float beta, gscale, eps;
  float* c2;            // SE_MT: the next T = 5/4 I - 1/4 C (strides as c)
  int pshare, qshare;   // SHARE: 1 lets two consecutive problems read the same P (or Q): matrix (b >> pshare)
};

// Straight and (for off-diagonal tiles of a symmetric product) mirrored store of the 16 values
// a lane holds of a 32 x 32 accumulator tile: rows row0 + 8 (r / 4) + (r % 4), column col.
__device__ __forceinline__ void put16(float* C, int64_t ld, int row0, int col, const float (&v)[16], bool mirror) {
#pragma unroll
  for (int r = 0; r < 16; ++r) C[static_cast<int64_t>(row0 + 8 * (r >> 2) + (r & 3)) * ld + col] = v[r];
  if (mirror) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 q;
#pragma unroll
      for (int e = 0; e < 4; ++e) q[e] = v[4 * g + e];
      *reinterpret_cast<f32x4*>(C + static_cast<int64_t>(col) * ld + row0 + 8 * g) = q;
    }
  }
}

// 128 x 128 tiles, each wavefront a 64 x 64 quarter.
// SHARE is a variant of its own (the SOAP rotations of G and M): with the division of the problem number in every launch
// the refresh, some 300 launches of 4 to 50 us, took 18.00 ms on 4 x 2048x1024, with a shift 17.93, without either 17.83.
// QT: the second operand as [K][N] (the reflectors of the refresh), which goes into LDS as it is.
template <int EPI, bool SYM, bool SHARE, bool QT>
__device__ __forceinline__ void sh_gemm_body(const ShGemm& g, int block, const PtrTable& stat, const Shape& s, const OutSpec& o) {
  constexpr int NI = 2;                // 32 x 32 MFMA tiles per wavefront, along M and along N
  constexpr int LQ = QT ? SB + 4 : LDS_LD;
  __shared__ float sP[2][SK][LDS_LD];  // k-major: the lanes of one MFMA operand read consecutive rows
  __shared__ __attribute__((aligned(16))) float sQ[2][SK][LQ];

  const int tiles_m = static_cast<int>(g.M / SB), tiles_n = static_cast<int>(g.N / SB);
  const int per = SYM ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  const int b = block / per;
  int tix = block - b * per;
  int tm, tn;
  if (SYM) {
    // upper triangle row by row: row tm holds the columns tm .. tiles_m - 1
    tm = 0;
    for (int len = tiles_m; tix >= len; --len) tix -= len, ++tm;
    tn = tm + tix;
  } else {
    tm = tix / tiles_n;
    tn = tix - tm * tiles_n;
  }

  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const float* Pg = g.P + static_cast<int64_t>(SHARE ? b >> g.pshare : b) * g.sp + static_cast<int64_t>(tm) * SB * g.ldp;
  const float* Qg = g.Q + static_cast<int64_t>(SHARE ? b >> g.qshare : b) * g.sq + static_cast<int64_t>(tn) * SB * (QT ? 1 : g.ldq);

  const int ld_row = t >> 3, ld_k = (t & 7) * 4;  // rows ld_row + 32 x (x = 0..3), 4 consecutive k
  const int qt_k = t >> 5, qt_n = (t & 31) * 4;   // QT: k qt_k + 8 x, 4 consecutive columns
  // Long sums of the statistics (k up to the other extent of the matrix, terms of one sign on the
  // diagonal) are folded into a second accumulator every FLUSH stages; the products of the root
  // iteration and the preconditioning accumulate in one go (their rounding, about 1e-5 relative,
  // is corrected by the following rounds and is far below the tolerance of the update).
  constexpr bool FOLD = EPI == SE_STAT;
  f32x16 acc[NI][NI], tot[NI][NI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f, tot[i][j][r] = 0.f;

  // Two register sets: stage kt + 2 is requested while stage kt is multiplied and stage kt + 1
  // waits in the other set, so a request has two stage times (about 3.5 us) to land.
  f32x4 pv[2][4], qv[2][4];
  auto fetch = [&](int kt, int set) {
    const int64_t k0 = static_cast<int64_t>(kt) * SK + ld_k;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      pv[set][x] = *reinterpret_cast<const f32x4*>(Pg + static_cast<int64_t>(ld_row + 32 * x) * g.ldp + k0);
      qv[set][x] = *reinterpret_cast<const f32x4*>(QT ? Qg + (static_cast<int64_t>(kt) * SK + qt_k + 8 * x) * g.ldq + qt_n
                                                      : Qg + static_cast<int64_t>(ld_row + 32 * x) * g.ldq + k0);
    }
  };
  auto stash = [&](int buf, int set) {
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      if (QT) *reinterpret_cast<f32x4*>(&sQ[buf][qt_k + 8 * x][qt_n]) = qv[set][x];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        sP[buf][ld_k + c][ld_row + 32 * x] = pv[set][x][c];
        if (!QT) sQ[buf][ld_k + c][ld_row + 32 * x] = qv[set][x][c];
      }
    }
  };
  // one stage: LDS buffer `buf` holds stage kt, register set `other` stage kt + 1, set `mine` is free
  const int nk = static_cast<int>(g.K / SK);   // a multiple of 4
  auto stage = [&](int kt, int buf, int mine, int other) {
    if (kt + 2 < nk) fetch(kt + 2, mine);
#pragma unroll
    for (int k = 0; k < SK; k += 2) {
      float fa[NI], fb[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) fa[i] = sP[buf][k + (lane >> 5)][wm * 32 * NI + i * 32 + (lane & 31)];
#pragma unroll
      for (int j = 0; j < NI; ++j) fb[j] = sQ[buf][k + (lane >> 5)][wn * 64 + j * 32 + (lane & 31)];
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
    if (FOLD && ((kt + 1) % FLUSH == 0 || kt + 1 == nk)) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) tot[i][j][r] += acc[i][j][r], acc[i][j][r] = 0.f;
    }
    if (kt + 1 < nk) stash(buf ^ 1, other);
    __syncthreads();  // stage kt + 1 is complete in LDS; every wavefront is done reading stage kt
  };
  fetch(0, 0);
  fetch(1, 1);
  stash(0, 0);
  __syncthreads();
  for (int kt = 0; kt < nk; kt += 2) {   // pairs of stages without a test between them: the two halves schedule as one body
    stage(kt, 0, 0, 1);
    stage(kt + 1, 1, 1, 0);
  }
  if (!FOLD) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) tot[i][j] = acc[i][j];
  }

  const int row_base = tm * SB + wm * 32 * NI + 4 * (lane >> 5);
  const int col_base = tn * SB + wn * 64 + (lane & 31);
  const bool mirror = SYM && tm != tn;
  const int64_t cb = static_cast<int64_t>(b) * g.sc;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int row0 = row_base + i * 32, col = col_base + j * 32;
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = tot[i][j][r];
      if (EPI == SE_OUT) {
        store_out_tile(o, s, b, row0, col, v);
      } else if (EPI == SE_PLAIN) {
        put16(g.c + cb, g.ldc, row0, col, v, mirror);
      } else if (EPI == SE_SUB) {
        float* C = g.c + cb;
        float old[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) old[r] = C[static_cast<int64_t>(row0 + 8 * (r >> 2) + (r & 3)) * g.ldc + col];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = old[r] - v[r];
        put16(C, g.ldc, row0, col, v, false);
      } else if (EPI == SE_MT) {
        put16(g.c + cb, g.ldc, row0, col, v, mirror);
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = (row0 + 8 * (r >> 2) + (r & 3) == col ? 1.25f : 0.f) - 0.25f * v[r];
        put16(g.c2 + cb, g.ldc, row0, col, v, mirror);
      } else {  // SE_STAT
        float* S = static_cast<float*>(stat.p[b]);
        const int d = static_cast<int>(g.d);
        // all old values are requested before the first store, so that the 16 read-modify-writes overlap
        // instead of running as a chain of dependent memory round trips
        float old[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row0 + 8 * (r >> 2) + (r & 3);
          old[r] = g.beta != 0.f && row < d && col < d ? S[static_cast<int64_t>(row) * d + col] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row0 + 8 * (r >> 2) + (r & 3);
          float val = 0.f;
          if (row < d && col < d) {
            const int64_t at = static_cast<int64_t>(row) * d + col;
            val = g.gscale * v[r];
            if (g.beta != 0.f) val += g.beta * old[r];
            S[at] = val;
            if (mirror) S[static_cast<int64_t>(col) * d + row] = val;
            if (row == col) val += g.eps;
          }
          v[r] = val;
        }
        if (g.c == nullptr) continue;   // the padded copy is only wanted when something reads it
        put16(g.c + cb, g.ldc, row0, col, v, mirror);
      }
    }
  }
}

template <int EPI, bool SYM, bool SHARE = false>
__global__ __launch_bounds__(NTH) void k_sh_gemm(ShGemm g, PtrTable stat, Shape s, OutSpec o) {
  sh_gemm_body<EPI, SYM, SHARE, false>(g, static_cast<int>(blockIdx.x), stat, s, o);
}
// The statistics variant carries a second set of accumulators; left to itself the register allocator takes
// more than half of a SIMD's registers for it, which leaves one block per CU and nothing to cover its
// barriers and epilogue with (MFMA pipe 40 % busy).  Held to two wavefronts per SIMD it fits without spills.
// The other variants are left alone: under the same limit they lose their AGPR accumulators and 5 % of their rate.
template <int EPI, bool SYM, bool SHARE = false>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_sh_gemm_2w(ShGemm g, PtrTable stat, Shape s,
                                                                                             OutSpec o) {
  sh_gemm_body<EPI, SYM, SHARE, false>(g, static_cast<int>(blockIdx.x), stat, s, o);
}

template <int EPI, bool SYM, bool SHARE = false>
hipError_t launch_gemm(ShGemm g, int nb, const PtrTable& stat, const Shape& s, const OutSpec& o, hipStream_t st) {
  if (g.M < SB || g.N < SB || g.K < SB || g.M % SB || g.N % SB || g.K % SB || (SYM && g.M != g.N) ||
      (g.pshare | g.qshare) >> (SHARE ? 1 : 0)) return hipErrorInvalidValue;
  if (g.ldc == 0) g.ldc = g.N, g.sc = g.M * g.N;
  const int64_t tm = g.M / SB, tn = g.N / SB;
  const int64_t blocks = (SYM ? tm * (tm + 1) / 2 : tm * tn) * nb;
  if constexpr (EPI == SE_STAT)
    hipLaunchKernelGGL((k_sh_gemm_2w<EPI, SYM, SHARE>), dim3(static_cast<unsigned>(blocks)), dim3(NTH), 0, st, g, stat, s, o);
  else
    hipLaunchKernelGGL((k_sh_gemm<EPI, SYM, SHARE>), dim3(static_cast<unsigned>(blocks)), dim3(NTH), 0, st, g, stat, s, o);
  return hipGetLastError();
}

// G (bf16 or fp32, whole or tp column fragments) -> fp32 working copies in both orientations,
// zero outside rows x cols.  One block per 64 x 64 tile; the transposed copy goes through LDS.
static __global__ __launch_bounds__(NTH) void k_sh_load(Shape s, PtrTable grad, int grad_dtype, int64_t rp, int64_t cp,
                                                  float* __restrict__ gs, float* __restrict__ gt) {
  __shared__ float tile[64][65];
  const int b = blockIdx.z, r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
  const int wf = static_cast<int>(s.wfrag);
  float* gsb = gs + static_cast<int64_t>(b) * rp * cp;
  float* gtb = gt + static_cast<int64_t>(b) * rp * cp;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;
    const int row = r0 + r, col = c0 + c;
    float val = 0.f;
    if (row < s.rows && col < s.cols) {
      const int f = col / wf;
      const int64_t at = static_cast<int64_t>(row) * wf + (col - f * wf);
      val = grad_dtype == CANZ_DT_BF16 ? static_cast<float>(static_cast<const __bf16*>(grad.p[b * s.tp + f])[at])
                                       : static_cast<const float*>(grad.p[b * s.tp + f])[at];
    }
    gsb[static_cast<int64_t>(row) * cp + col] = val;
    tile[r][c] = val;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;  // r: column of G, c: row of G
    gtb[static_cast<int64_t>(c0 + r) * rp + r0 + c] = tile[c][r];
  }
}

// dense rows x cols matrices of the caller <- the padded working copies src[b * stride] (row length cp)
static __global__ __launch_bounds__(NTH) void k_unpad(Shape s, PtrTable dst, const float* __restrict__ src, int64_t stride,
                                                     int64_t cp) {
  const int b = blockIdx.z, r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
  const float* from = src + static_cast<int64_t>(b) * stride;
  float* to = static_cast<float*>(dst.p[b]);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, row = r0 + (idx >> 6), col = c0 + (idx & 63);
    if (row < s.rows && col < s.cols) to[static_cast<int64_t>(row) * s.cols + col] = from[static_cast<int64_t>(row) * cp + col];
  }
}

// one 64 x 64 fp32 tile in LDS -> the 8-element chunks of its bf16 panel image, straight (dst rows = tile rows) or
// transposed (dst rows = tile columns); (r0, c0): the tile's place in the matrix, kc: row length of the image
static __device__ __forceinline__ void tile_to_panels(const float (*tile)[65], __bf16* __restrict__ dst, int64_t r0, int64_t c0,
                                               int64_t kc, bool transposed, int t) {
  const int cv = (t & 7) * 8;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int rl = (t >> 3) + half * 32;
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = static_cast<__bf16>(transposed ? tile[cv + e][rl] : tile[rl][cv + e]);
    *reinterpret_cast<bf16x8*>(dst + (transposed ? panel_chunk_off(c0 + rl, r0 + cv, kc) : panel_chunk_off(r0 + rl, c0 + cv, kc))) = o;
  }
}

// The same tile as three bf16 terms per element (kernels.h: launch_split3): term i of a matrix of kc columns lies in the
// columns i kc .. of a panel matrix of 3 kc columns.
static __device__ __forceinline__ void tile_to_terms3(const float (*tile)[65], __bf16* __restrict__ dst, int64_t r0, int64_t c0,
                                                      int64_t kc, bool transposed, int t) {
  const int cv = (t & 7) * 8;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int rl = (t >> 3) + half * 32;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = transposed ? tile[cv + e][rl] : tile[rl][cv + e];
    const int64_t row = (transposed ? c0 : r0) + rl, col = (transposed ? r0 : c0) + cv;
#pragma unroll
    for (int term = 0; term < 3; ++term) {
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = static_cast<__bf16>(v[e]), v[e] -= static_cast<float>(o[e]);
      *reinterpret_cast<bf16x8*>(dst + panel_chunk_off(row, term * kc + col, 3 * kc)) = o;
    }
  }
}

// fp32 matrices of d x d elements (row length ld) -> three bf16 terms per element, [dp2][3 dp2] panels, zero outside d x d.
// One block per 64 x 64 tile.
static __global__ __launch_bounds__(NTH) void k_terms3(PtrTable src, int64_t d, int64_t ld, int64_t dp2, __bf16* __restrict__ to) {
  __shared__ float tile[64][65];
  const int b = blockIdx.z, r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
  const float* m = static_cast<const float*>(src.p[b]);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;
    tile[r][c] = r0 + r < d && c0 + c < d ? m[static_cast<int64_t>(r0 + r) * ld + c0 + c] : 0.f;
  }
  __syncthreads();
  tile_to_terms3(tile, to + static_cast<int64_t>(b) * 3 * dp2 * dp2, r0, c0, dp2, false, t);
}

// S[row][col] <- S[col][row] for row > col of the caller's dense d x d matrices: the symmetric statistic is computed
// on and above the diagonal tiles only.  One block per 64 x 64 tile on or below the diagonal (blockIdx.y >= blockIdx.x).
static __global__ __launch_bounds__(NTH) void k_mirror(PtrTable stat, int64_t d) {
  __shared__ float tile[64][65];
  if (blockIdx.y < blockIdx.x) return;
  const int b = blockIdx.z, r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
  float* m = static_cast<float*>(stat.p[b]);
#pragma unroll
  for (int e = 0; e < 16; ++e) {   // the tile above the diagonal that mirrors this one: rows c0.., columns r0..
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;
    const int64_t row = c0 + r, col = r0 + c;
    tile[r][c] = row < d && col < d ? m[row * d + col] : 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int idx = e * NTH + t, r = idx >> 6, c = idx & 63;
    const int64_t row = r0 + r, col = c0 + c;
    if (row < d && col < row) m[row * d + col] = tile[c][r];
  }
}

inline int64_t pad256(int64_t x) { return (x + PAD - 1) / PAD * PAD; }

// S <- beta S + gscale X X^T of the caller's dense fp32 d x d matrices on the bf16 matrix cores, X [nb][d2][k2] bf16 panels:
// the operands are bf16 values themselves, every product is exact in fp32 and the sums are fp32, so nothing is lost
// against the fp32 kernel, at a fraction of its time.  The product is the "last product" of the Muon step's kernels:
// old * decay + factor * product in place (beta = 0: factor * product, whatever S held).
// k_piece: k per launch (a multiple of 256; k2 for all at once).  A sum accumulated in one go loses with its length what the
// fp32 kernel's folds keep: at k = 3072 the error against 64 bits is 2.9e-7 in one piece and 1.7e-7 in pieces of 1024
// (fp32 kernel: 1.6e-7), at the cost of a pass over the statistic per piece.
inline int statistic_bf16(int kind, const PtrTable& tab, int64_t d, int64_t d2, int64_t k2, int64_t k_piece, int nb, float beta,
                          float gscale, const __bf16* x, hipStream_t st) {
  Shape sq{};
  sq.rows = d, sq.cols = d, sq.m = d, sq.n = d, sq.mp = d2, sq.np = d2, sq.tp = 1, sq.wfrag = d;
  OutSpec so{};
  so.out = tab, so.out_dtype = CANZ_DT_F32, so.neg_lr_scale = gscale;
  const SplitWs no_split{nullptr, 0};
  // Only the tiles on and above the diagonal, mirrored afterwards, where that pays: the products it saves (about
  // 0.65 us per 32-long k-step of a tile, a round of tiles on 256 CUs at a time) against one more pass over the
  // statistic at some 4 TB/s that does not overlap with anything.  Long sums win (25600 x 5120: 3.9 -> 1.3 ms),
  // short ones do not (3072 x 1024: the mirror pass costs what the products save).
  const int64_t t256 = d2 / 256;
  const double saved_us = static_cast<double>(t256 * (t256 - 1) / 2 * nb) / 256.0 * static_cast<double>(k2 / 32) * 0.65;
  const double mirror_us = 15.0 + static_cast<double>(d) * static_cast<double>(d) * nb * 4.0 / 4.0e6;
  const bool upper = saved_us > 1.5 * mirror_us;
  for (int64_t k0 = 0; k0 < k2; k0 += k_piece) {
    so.decay = k0 == 0 ? beta : 1.f;
    so.out_mode = so.decay == 0.f ? CANZ_OUT_DELTA : CANZ_OUT_PARAM;
    const GemmDims sd{d2, d2, k2 - k0 < k_piece ? k2 - k0 : k_piece, k2, k2, d2 * k2, d2 * k2, nb};
    const __bf16* xk = x + k0 / PANEL_K * PANEL_ELEMS;
    if (upper)
      CANZ_HIP(kind, launch_final_sym_bf16(sd, xk, no_split, sq, so, st), "statistics kernel (bf16 operands)");
    else
      CANZ_HIP(kind, launch_final_bf16(sd, xk, xk, nullptr, no_split, sq, so, st), "statistics kernel (bf16 operands)");
  }
  if (upper) {
    prof_mark(st, kind, true);
    const unsigned t64 = static_cast<unsigned>((d + 63) / 64);
    hipLaunchKernelGGL(k_mirror, dim3(t64, t64, static_cast<unsigned>(nb)), dim3(NTH), 0, st, tab, d);
    prof_mark(st, kind, false);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return fail(CANZ_EHIP, "statistic mirror: %s", hipGetErrorString(e));
  }
  return CANZ_OK;
}

}  // namespace f32mfma
}  // namespace canz
