// Streaming kernels of the Muon step: momentum update fused with the (TP) gather, the
// cast into both working orientations and the Frobenius-norm partial sums; the norm
// scale; and the direct update used when no Newton-Schulz step is requested.
// These passes are HBM-bound: every global access is a 16-byte vector per lane on
// contiguous rows, the transpose goes through LDS, the reduction through wave shuffles.
#include <type_traits>

#include "device_util.h"
#include "panel_layout.h"

namespace canz {
namespace {

constexpr int TILE = EW_TILE;     // 64 x 64 elements per block
constexpr int NTHREADS = 256;

template <typename T>
struct Vec8;
template <>
struct alignas(16) Vec8<float> {
  float v[8];
};
template <>
struct alignas(16) Vec8<__bf16> {
  __bf16 v[8];
};

// VEC: rows and fragments of a multiple of 8 elements.  Otherwise the same accesses, aligned to an element only, and element by element
// where the edge of the matrix cuts the eight.  Either way eight columns lie in one fragment: those of several fragments are multiples
// of 8, whatever shares the launch (its parts may differ in tp, and one ragged part sends all of them here without VEC).
// One block = one 64 x 64 tile of one matrix in the caller's orientation, extended over
// the padded extents (elements outside rows x cols are zeros and touch no caller memory).
// Step 2 of the operator: M <- beta M + G, U = M (or G + beta M); step 1 (TP gather) is
// the fragment lookup on the load.
template <typename T, bool VEC>
__device__ __forceinline__ void momentum_tile(const Shape& s, const void* const* grad, int grad_dtype, void* const* mom, float beta,
                                              int nesterov, T* __restrict__ xw, T* __restrict__ xt, float* __restrict__ partial,
                                              int bx, int by, int b, int tiles_x, int tiles_y) {
  typedef typename std::conditional<VEC, f32x4, f32x4_any>::type f32x4v;
  typedef typename std::conditional<VEC, bf16x8, bf16x8_any>::type bf16x8v;
  __shared__ float tile[TILE][TILE + 1];
  __shared__ float wsum[NTHREADS / 64];

  const int r0 = by * TILE, c0 = bx * TILE;
  const int rows = static_cast<int>(s.rows), cols = static_cast<int>(s.cols);
  const int wf = static_cast<int>(s.wfrag);
  // straight = same orientation as the caller's matrix; transposed = the other one
  const int64_t pr = s.tall ? s.np : s.mp, pc = s.tall ? s.mp : s.np;
  T* straight = s.tall ? xt : xw;
  T* transposed = s.tall ? xw : xt;
  const bool put_straight = straight != nullptr, put_transposed = transposed != nullptr;   // xw is not always asked for
  const int64_t at = static_cast<int64_t>(b) * pr * pc;
  if (put_straight) straight += at;
  if (put_transposed) transposed += at;
  float* mptr = static_cast<float*>(mom[b]);

  const int t = threadIdx.x;
  const int cv = (t & 7) * 8;
  float ss = 0.f;
  // Phase 1: every load of both half-tiles is issued before the first store (the momentum
  // store of one half must not hold back the loads of the other: the buffers come from
  // pointer tables and may alias as far as the compiler knows).
  float g[2][8], mo[2][8];
  bool live[2];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int row = r0 + (t >> 3) + half * 32, col = c0 + cv;
    live[half] = row < rows && col < cols;
#pragma unroll
    for (int e = 0; e < 8; ++e) g[half][e] = 0.f, mo[half][e] = 0.f;
    if (!live[half]) continue;
    const int f = s.tp > 1 ? col / wf : 0;
    const int64_t gi = static_cast<int64_t>(row) * wf + (col - f * wf);
    if (VEC || col + 8 <= cols) {
      if (grad_dtype == CANZ_DT_BF16) {
        const bf16x8 gv = *reinterpret_cast<const bf16x8v*>(static_cast<const __bf16*>(grad[b * s.tp + f]) + gi);
#pragma unroll
        for (int e = 0; e < 8; ++e) g[half][e] = static_cast<float>(gv[e]);
      } else {
        const f32x4v* gp = reinterpret_cast<const f32x4v*>(static_cast<const float*>(grad[b * s.tp + f]) + gi);
        const f32x4 g0 = gp[0], g1 = gp[1];
#pragma unroll
        for (int e = 0; e < 4; ++e) g[half][e] = g0[e], g[half][4 + e] = g1[e];
      }
      const f32x4v* mp4 = reinterpret_cast<const f32x4v*>(mptr + static_cast<int64_t>(row) * cols + col);
      const f32x4 m0 = mp4[0], m1 = mp4[1];
#pragma unroll
      for (int e = 0; e < 4; ++e) mo[half][e] = m0[e], mo[half][4 + e] = m1[e];
    } else {
#pragma unroll
      for (int e = 0; e < 7; ++e) {
        if (col + e >= cols) break;
        g[half][e] = grad_dtype == CANZ_DT_BF16 ? static_cast<float>(static_cast<const __bf16*>(grad[b * s.tp + f])[gi + e])
                                                : static_cast<const float*>(grad[b * s.tp + f])[gi + e];
        mo[half][e] = mptr[static_cast<int64_t>(row) * cols + col + e];
      }
    }
  }
  // Phase 2: momentum, stores, working copies
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int rl = (t >> 3) + half * 32;
    const int row = r0 + rl, col = c0 + cv;
    float u[8], mn[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // roundings pinned: a matrix has the same bits from either kernel
      mn[e] = __builtin_fmaf(beta, mo[half][e], g[half][e]);
      u[e] = nesterov ? __builtin_fmaf(beta, mn[e], g[half][e]) : mn[e];
    }
    if (live[half]) {
      if (VEC || col + 8 <= cols) {
        f32x4 n0, n1;
#pragma unroll
        for (int e = 0; e < 4; ++e) n0[e] = mn[e], n1[e] = mn[4 + e];
        f32x4v* mp4 = reinterpret_cast<f32x4v*>(mptr + static_cast<int64_t>(row) * cols + col);
        mp4[0] = n0;
        mp4[1] = n1;
      } else {
#pragma unroll
        for (int e = 0; e < 7; ++e)
          if (col + e < cols) mptr[static_cast<int64_t>(row) * cols + col + e] = mn[e];
      }
    }
    Vec8<T> o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // (the first two squares as one product and one fused multiply-add)
      if (half == 0 && e < 2)
        ss = e == 0 ? u[1] * u[1] : __builtin_fmaf(u[0], u[0], ss);
      else
        ss = __builtin_fmaf(u[e], u[e], ss);
      o.v[e] = from_f32<T>(u[e]);
      if (put_transposed) tile[rl][cv + e] = u[e];
    }
    if (put_straight) *reinterpret_cast<Vec8<T>*>(straight + WorkLayout<T>::chunk_off(row, col, pc)) = o;
  }
  if (put_transposed) __syncthreads();
  if (put_transposed)
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int cl = (t >> 3) + half * 32;  // column of the tile = row of the transposed tile
    Vec8<T> o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o.v[e] = from_f32<T>(tile[cv + e][cl]);
    *reinterpret_cast<Vec8<T>*>(transposed + WorkLayout<T>::chunk_off(c0 + cl, r0 + cv, pr)) = o;
  }
  // sum of squares of this tile, fixed order: lanes -> waves -> thread 0
  ss = wave_sum(ss);
  if ((t & 63) == 0) wsum[t >> 6] = ss;
  __syncthreads();
  if (t == 0) {
    partial[static_cast<int64_t>(b) * tiles_x * tiles_y + by * tiles_x + bx] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
  }
}
template <typename T, bool VEC>
__global__ __launch_bounds__(NTHREADS) void k_momentum(Shape s, PtrTable grad, int grad_dtype, PtrTable mom,
                                                        float beta, int nesterov, T* __restrict__ xw,
                                                        T* __restrict__ xt, float* __restrict__ partial) {
  momentum_tile<T, VEC>(s, grad.p, grad_dtype, mom.p, beta, nesterov, xw, xt, partial, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.x,
                        gridDim.y);
}
// Several parts in one launch: the tiles of part 0, then of part 1, ...
struct MomentumParts {
  int n;
  int begin[MAX_PARTS + 1];
  MomentumPart<__bf16> part[MAX_PARTS];
};
template <bool VEC>
__global__ __launch_bounds__(NTHREADS) void k_momentum_parts(MomentumParts a, PtrTable grad, PtrTable mom, float beta, int nesterov) {
  int j = 0, tile = blockIdx.x;
  while (j + 1 < a.n && tile >= a.begin[j + 1]) ++j;
  const MomentumPart<__bf16>& p = a.part[j];
  const Shape s = p.s;
  tile -= a.begin[j];
  const int tiles_x = static_cast<int>((s.tall ? s.mp : s.np) / TILE), tiles_y = static_cast<int>((s.tall ? s.np : s.mp) / TILE);
  const int by = tile / tiles_x, bx = tile - by * tiles_x, b = by / tiles_y;
  momentum_tile<__bf16, VEC>(s, grad.p + p.first_grad, p.grad_dtype, mom.p + p.first_mom, beta, nesterov, p.xw, p.xt, p.partial, bx,
                             by - b * tiles_y, b, tiles_x, tiles_y);
}

// Step 3 of the operator, as a scalar: 1 / (||U||_F + eps).  One block per matrix; the
// tile sums are added in fp64 in a fixed order, so the result does not depend on timing.
struct NormBatches {
  int n;
  NormBatch b[MAX_KINDS];
};
__global__ __launch_bounds__(NTHREADS) void k_norm_scale(NormBatches batches, float eps) {
  __shared__ double red[NTHREADS];
  int b = blockIdx.x, j = 0;
  while (j + 1 < batches.n && b >= batches.b[j].nb) b -= batches.b[j].nb, ++j;
  const int n_partial = batches.b[j].n_partial, t = threadIdx.x;
  const float* __restrict__ partial = batches.b[j].partial;
  double acc = 0.0;
  for (int i = t; i < n_partial; i += NTHREADS) acc += static_cast<double>(partial[static_cast<int64_t>(b) * n_partial + i]);
  red[t] = acc;
  __syncthreads();
  for (int w = NTHREADS / 2; w > 0; w >>= 1) {
    if (t < w) red[t] += red[t + w];
    __syncthreads();
  }
  if (t == 0) {
    const float sc = static_cast<float>(1.0 / (sqrt(red[0]) + static_cast<double>(eps)));
    batches.b[j].scale[b] = sc;
    batches.b[j].scale2[b] = sc * sc;
  }
}

// ns_steps == 0: O = scale * U, read back from the working copy in the caller's orientation.
template <typename T>
__global__ __launch_bounds__(NTHREADS) void k_apply(Shape s, const T* __restrict__ x, int64_t ld, int64_t batch_stride,
                                                     const float* __restrict__ scale, OutSpec o) {
  const int b = blockIdx.z;
  const float sc = scale[b];
  const T* xb = x + static_cast<int64_t>(b) * batch_stride;
  for (int row = blockIdx.y; row < s.rows; row += gridDim.y)
    for (int col = blockIdx.x * NTHREADS + threadIdx.x; col < s.cols; col += gridDim.x * NTHREADS)
      store_out(o, s, b, row, col, sc * static_cast<float>(xb[WorkLayout<T>::chunk_off(row, col & ~7, ld) + (col & 7)]));
}

}  // namespace

int momentum_tiles(const Shape& s) {
  return static_cast<int>((s.mp / TILE) * (s.np / TILE));
}

template <typename T>
hipError_t launch_momentum(const Shape& s, int nb, const PtrTable& grad, int grad_dtype, const PtrTable& mom,
                           float beta, int nesterov, T* xw, T* xt, float* partial, hipStream_t st) {
  const int64_t pr = s.tall ? s.np : s.mp, pc = s.tall ? s.mp : s.np;
  const dim3 grid(static_cast<unsigned>(pc / TILE), static_cast<unsigned>(pr / TILE), static_cast<unsigned>(nb));
  const bool vec = (s.cols % 8 == 0) && (s.wfrag % 8 == 0);
  if (vec)
    hipLaunchKernelGGL((k_momentum<T, true>), grid, dim3(NTHREADS), 0, st, s, grad, grad_dtype, mom, beta, nesterov,
                       xw, xt, partial);
  else
    hipLaunchKernelGGL((k_momentum<T, false>), grid, dim3(NTHREADS), 0, st, s, grad, grad_dtype, mom, beta, nesterov,
                       xw, xt, partial);
  return hipGetLastError();
}

template hipError_t launch_momentum<__bf16>(const Shape&, int, const PtrTable&, int, const PtrTable&, float, int,
                                            __bf16*, __bf16*, float*, hipStream_t);
template hipError_t launch_momentum<float>(const Shape&, int, const PtrTable&, int, const PtrTable&, float, int,
                                           float*, float*, float*, hipStream_t);

hipError_t launch_norm_scale(int nb, int n_partial, const float* partial, float eps, float* scale, float* scale2,
                             hipStream_t st) {
  const NormBatch one{nb, n_partial, partial, scale, scale2};
  return launch_norm_scale_batches(1, &one, eps, st);
}

hipError_t launch_norm_scale_batches(int n, const NormBatch* batches, float eps, hipStream_t st) {
  if (n < 1 || n > MAX_KINDS) return hipErrorInvalidValue;
  NormBatches a{};
  a.n = n;
  int blocks = 0;
  for (int i = 0; i < n; ++i) a.b[i] = batches[i], blocks += batches[i].nb;
  hipLaunchKernelGGL(k_norm_scale, dim3(static_cast<unsigned>(blocks)), dim3(NTHREADS), 0, st, a, eps);
  return hipGetLastError();
}

hipError_t launch_momentum_parts(int n, const MomentumPart<__bf16>* parts, const PtrTable& grad, const PtrTable& mom, float beta,
                                 int nesterov, hipStream_t st) {
  if (n < 1 || n > MAX_PARTS) return hipErrorInvalidValue;
  MomentumParts a{};
  a.n = n;
  int64_t tiles = 0;
  bool vec = true;
  for (int i = 0; i < n; ++i) {
    a.part[i] = parts[i];
    a.begin[i] = static_cast<int>(tiles);
    tiles += static_cast<int64_t>(momentum_tiles(parts[i].s)) * parts[i].nb;
    vec = vec && parts[i].s.cols % 8 == 0 && parts[i].s.wfrag % 8 == 0;
  }
  for (int i = n; i <= MAX_PARTS; ++i) a.begin[i] = static_cast<int>(tiles);
  if (vec)
    hipLaunchKernelGGL(k_momentum_parts<true>, dim3(static_cast<unsigned>(tiles)), dim3(NTHREADS), 0, st, a, grad, mom, beta, nesterov);
  else
    hipLaunchKernelGGL(k_momentum_parts<false>, dim3(static_cast<unsigned>(tiles)), dim3(NTHREADS), 0, st, a, grad, mom, beta, nesterov);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_apply(const Shape& s, int nb, const T* x_straight, int64_t ld, int64_t batch_stride,
                        const float* scale, const OutSpec& o, hipStream_t st) {
  const unsigned gx = static_cast<unsigned>((s.cols + NTHREADS - 1) / NTHREADS);
  const dim3 grid(gx > 64 ? 64 : gx, static_cast<unsigned>(s.rows > 32768 ? 32768 : s.rows), static_cast<unsigned>(nb));
  hipLaunchKernelGGL((k_apply<T>), grid, dim3(NTHREADS), 0, st, s, x_straight, ld, batch_stride, scale, o);
  return hipGetLastError();
}
template hipError_t launch_apply<__bf16>(const Shape&, int, const __bf16*, int64_t, int64_t, const float*,
                                         const OutSpec&, hipStream_t);
template hipError_t launch_apply<float>(const Shape&, int, const float*, int64_t, int64_t, const float*,
                                        const OutSpec&, hipStream_t);

}  // namespace canz
