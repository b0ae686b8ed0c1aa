// canz_muon_step / canz_muon_workspace_bytes: host side of the per-rank Muon step
// (Delta W = Muon_step(G, States), Sec. 4.1 stage (2); zero-communication owner update,
// Sec. 3.3 stage (2)).  Validates the groups, carves the caller's workspace and enqueues
// the kernels of each micro-group on the caller's stream:
//   momentum (+ TP gather, cast, norm partials) -> norm scale ->
//   ns_steps x { Gram, polynomial, update }, or several steps at a time (stage_plan), with the
//   last update writing the caller's buffers (+ TP scatter).  Nothing here allocates, copies to the device or synchronises.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <vector>

#include "canz.h"
#include "canz_internal.h"
#include "kernels.h"

namespace canz {

// ---- optional per-kernel timing (canz_profile_*): a pool of event pairs recorded around
// each launch on the step's own stream.  Process-wide state behind a mutex; while profiling is
// off a launch only reads one atomic flag.  Steps recorded from several threads at once would
// interleave their launches in one pool: the timing is meant for one benchmark thread.
namespace {
struct Profiler {
  std::atomic<bool> on{false};
  std::mutex lock;
  std::vector<hipEvent_t> ev;   // 2 per launch
  std::vector<int> kind;        // kind of each recorded launch
  size_t used = 0;              // launches recorded
};
Profiler g_prof;
}  // namespace

void prof_mark(hipStream_t st, int kind, bool begin) {
  if (!g_prof.on.load(std::memory_order_relaxed)) return;
  std::lock_guard<std::mutex> hold(g_prof.lock);
  if (g_prof.used * 2 + 1 >= g_prof.ev.size()) return;
  if (begin) {
    (void)hipEventRecord(g_prof.ev[g_prof.used * 2], st);
  } else {
    (void)hipEventRecord(g_prof.ev[g_prof.used * 2 + 1], st);
    g_prof.kind[g_prof.used] = kind;
    ++g_prof.used;
  }
}

}  // namespace canz

namespace canz {
namespace {

constexpr size_t ALIGN = 256;
inline size_t align_up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }
inline int64_t pad_up(int64_t x) { return (x + PAD - 1) / PAD * PAD; }

struct Carve {   // byte offsets of one launch batch's arrays, relative to its own base
  size_t xw, xt0, xt1, a, b, partial, scale, scale2, total;
};

Shape make_shape(const canz_group& g) {
  Shape s{};
  s.rows = g.rows, s.cols = g.cols;
  s.m = std::min(g.rows, g.cols), s.n = std::max(g.rows, g.cols);
  s.mp = pad_up(s.m), s.np = pad_up(s.n);
  s.tall = g.rows > g.cols;
  s.tp = g.tp;
  s.wfrag = g.cols / g.tp;
  return s;
}

Carve carve(const Shape& s, int nb, int precision) {
  const size_t esz = precision == CANZ_PREC_BF16 ? 2 : 4;
  const size_t x_bytes = align_up(static_cast<size_t>(nb) * s.mp * s.np * esz);
  const size_t a_bytes = align_up(static_cast<size_t>(nb) * s.mp * s.mp * esz);
  Carve c{};
  size_t off = 0;
  c.xt0 = off, off += x_bytes;   // X lies between the two X^T: with the unused one it is one free piece (see Spare)
  c.xw = off, off += x_bytes;
  c.xt1 = off, off += x_bytes;
  c.a = off, off += a_bytes;
  c.b = off, off += a_bytes;
  c.partial = off, off += align_up(static_cast<size_t>(nb) * momentum_tiles(s) * sizeof(float));
  c.scale = off, off += align_up(nb * sizeof(float));
  c.scale2 = off, off += align_up(nb * sizeof(float));
  c.total = off;
  return c;
}

// scratch of the k-split, shared by all launches of a call (bf16 mode only)
size_t split_bytes(int precision) {
  return precision == CANZ_PREC_BF16 ? align_up(SPLIT_MAX_BLOCKS * SPLIT_BLOCK_BYTES) : 0;
}

int check_hparams(const canz_muon_hparams* hp) {
  if (!hp) return fail(CANZ_EINVAL, "null hparams");
  if (hp->ns_steps < 0) return fail(CANZ_EINVAL, "ns_steps must be >= 0");
  if (hp->scale_mode < CANZ_SCALE_NONE || hp->scale_mode > CANZ_SCALE_RMS)
    return fail(CANZ_EUNSUPPORTED, "unknown scale_mode %d", hp->scale_mode);
  if (hp->precision != CANZ_PREC_BF16 && hp->precision != CANZ_PREC_F32)
    return fail(CANZ_EUNSUPPORTED, "unknown precision %d", hp->precision);
  if (hp->out_mode != CANZ_OUT_PARAM && hp->out_mode != CANZ_OUT_DELTA)
    return fail(CANZ_EUNSUPPORTED, "unknown out_mode %d", hp->out_mode);
  return CANZ_OK;
}

int check_group(const canz_group& g, int idx, bool need_ptrs, int out_mode) {
  if (g.n_mats < 0) return fail(CANZ_EINVAL, "group %d: n_mats < 0", idx);
  if (g.rows < 1 || g.cols < 1) return fail(CANZ_EINVAL, "group %d: empty shape", idx);
  // 65535 grid rows of 64-row tiles in the element-wise kernels
  constexpr int64_t MAX_EXTENT = 65535 * 64;
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
  if (!g.grad || !g.mom || !g.out) return fail(CANZ_EINVAL, "group %d: null pointer table", idx);
  const int n_out = out_mode == CANZ_OUT_DELTA ? g.n_mats * g.tp : g.n_mats;
  auto bad = [](const void* p) { return p == nullptr || (reinterpret_cast<uintptr_t>(p) & 15u) != 0; };
  for (int i = 0; i < g.n_mats * g.tp; ++i)
    if (bad(g.grad[i])) return fail(CANZ_EINVAL, "group %d: grad[%d] null or not 16-byte aligned", idx, i);
  for (int i = 0; i < g.n_mats; ++i)
    if (bad(g.mom[i])) return fail(CANZ_EINVAL, "group %d: mom[%d] null or not 16-byte aligned", idx, i);
  for (int i = 0; i < n_out; ++i)
    if (bad(g.out[i])) return fail(CANZ_EINVAL, "group %d: out[%d] null or not 16-byte aligned", idx, i);
  return CANZ_OK;
}

double update_scale(const canz_group& g, int mode) {
  if (mode == CANZ_SCALE_ASPECT) return std::sqrt(std::max(1.0, static_cast<double>(g.rows) / static_cast<double>(g.cols)));
  if (mode == CANZ_SCALE_RMS) return 0.2 * std::sqrt(static_cast<double>(std::max(g.rows, g.cols)));
  return 1.0;
}

// Launch batches: consecutive matrices of the call that share dtypes and shape - up to a
// transpose, since the iteration runs on the wide orientation of either - are batched
// together, up to batch_cap() per launch, across micro-group boundaries (a matrix's result
// does not depend on its batch, and small matrices need the larger batch to fill the chip).
bool same_kind(const canz_group& a, const canz_group& b) {
  return std::min(a.rows, a.cols) == std::min(b.rows, b.cols) && std::max(a.rows, a.cols) == std::max(b.rows, b.cols) &&
         a.tp == b.tp && a.grad_dtype == b.grad_dtype && a.out_dtype == b.out_dtype;
}

// matrices of this kind per launch: bounded by the pointer tables (kernel arguments) and by
// the workspace a launch needs.  Small matrices go many to a launch, so that the persistent
// GEMM grids have whole rounds of tiles and the launch count stays low.
int batch_cap(const canz_group& g) {
  const Shape s = make_shape(g);
  const int64_t by_ptrs = MAX_PTRS / g.tp;
  const int64_t by_elems = std::max<int64_t>(1, MAX_BATCH_ELEMS / (s.mp * s.np));
  return static_cast<int>(std::min(by_ptrs, by_elems));
}

// calls fn(proto group, first group index, first matrix in it, count) for every launch batch
template <typename F>
int for_each_batch(const canz_group* g, int n_groups, F&& fn) {
  int proto = -1, count = 0, start_group = 0, start_mat = 0;
  for (int i = 0; i < n_groups; ++i) {
    for (int m = 0; m < g[i].n_mats; ++m) {
      if (count > 0 && (count == batch_cap(g[proto]) || !same_kind(g[proto], g[i]))) {
        if (int rc = fn(g[proto], start_group, start_mat, count)) return rc;
        count = 0;
      }
      if (count == 0) proto = i, start_group = i, start_mat = m;
      ++count;
    }
  }
  if (count > 0) return fn(g[proto], start_group, start_mat, count);
  return CANZ_OK;
}

// The matrices of one orientation inside a launch batch.
struct Part {
  const canz_group* proto = nullptr;
  std::vector<const void*> grad;
  std::vector<void*> mom, out;
  int n() const { return static_cast<int>(mom.size()); }
};

// One launch batch: part[0] holds its wide (rows <= cols) matrices, part[1] the tall ones of
// the transposed shape.  They occupy consecutive slots of the batch's workspace arrays, the
// wide ones first; the kernels that touch the caller's buffers (momentum, last product,
// apply) run once per part.
struct Batch {
  Part part[2];
  Shape s0{};     // shape of any member: the padded extents are those of the whole batch
  int nb = 0;
  int64_t update_tiles() const { return (s0.mp / PAD) * (s0.np / PAD) * nb; }
};

// Collects the launch batches of a call (pointers only when `with_ptrs`).
int collect_batches(const canz_group* g, int n_groups, int out_mode, bool with_ptrs, std::vector<Batch>& out) {
  return for_each_batch(g, n_groups, [&](const canz_group& proto, int gi, int mi, int count) {
    out.emplace_back();
    Batch& bt = out.back();
    bt.s0 = make_shape(proto);
    bt.nb = count;
    for (int left = count; left > 0; ++gi, mi = 0) {
      const canz_group& src = g[gi];
      const int take = std::min(left, src.n_mats - mi);
      if (take <= 0) continue;
      Part& p = bt.part[src.rows > src.cols ? 1 : 0];
      if (!p.proto) p.proto = &src;
      const int per_out = out_mode == CANZ_OUT_DELTA ? src.tp : 1;
      for (int m = mi; m < mi + take; ++m) {
        if (with_ptrs) {
          for (int f = 0; f < src.tp; ++f) p.grad.push_back(src.grad[m * src.tp + f]);
          for (int f = 0; f < per_out; ++f) p.out.push_back(src.out[m * per_out + f]);
        }
        p.mom.push_back(with_ptrs ? src.mom[m] : nullptr);
      }
      left -= take;
    }
    return CANZ_OK;
  });
}

// Merged steps keep their m x m matrices in fp16 (kernels.h: SymSpec), scaled to the magnitudes of an iteration that stays
// bounded: f(s) = a s + b s^3 + c s^5 has to keep the singular values in [0, S], S <= 1.3 the largest value they reach from [0, 1] (with 5 % to
// spare for rounding), and |a + b t + c t^2| <= 3.5 on [0, S^2].  The quintic (3.4445, -4.775, 2.0315) reaches S = 1.202.
bool bounded_map(const canz_muon_hparams& hp) {
  auto p = [&](float t) { return hp.a + t * (hp.b + t * hp.c); };
  constexpr int N = 256;
  float top = 1.f;
  for (int i = 0; i <= N; ++i) {
    const float s = static_cast<float>(i) / N;
    top = std::max(top, std::fabs(s * p(s * s)));
  }
  top *= 1.05f;
  bool ok = top <= 1.3f;
  for (int i = 0; i <= N; ++i) {
    const float s = top * static_cast<float>(i) / N, v = p(s * s);
    ok = ok && std::fabs(s * v) <= top && std::fabs(v) <= 3.5f;   // NaN: false
  }
  return ok;
}

// Stages of the iteration.  One Newton-Schulz step needs A = X X^T (m^2 n products, upper half), B = aI + bA + cAA (m^3)
// and X <- B X (2 m^2 n).  The next Gram matrix is A' = B A B, so several steps can stay among the m x m matrices,
//   B_1 = p(A_1),  A_2 = B_1 (B_1 A_1),  B_2 = p(A_2),  Q = B_2 B_1, ...        (3 m^3 per step after the first)
// and X be touched once, X <- Q X: with r = m / n and in units of m^2 n, five steps cost 15 + 5 r one by one and
// 8 + 14 r merged as 3 + 2 (the two terms of the last Q among them).
// Precision decides how.  An error in A_k is not seen by X and grows with a^2 per step in the small singular values, and Q = B_3 B_2 B_1
// spans a range of a^3.  So the m x m matrices are fp16 images and fp32 diagonals (kernels.h: SymSpec), Q is a bf16 image and
// an fp32 diagonal where a later step corrects what its rounding did, and two bf16 terms in the last product, where nothing
// does.  The first three steps are merged and the last two, with single ones between.  The update's error against 64 bits is then
// 0.3 to 0.5 of that of single steps for inputs of many comparable directions (Gaussian, plus a low-rank part, outliers,
// row and column scales, one-sided), and below it, 0.97 at most, for all that were tried (also duplicated rows, rows in groups of eight
// alike, a constant plus noise, low rank), at 1536 x 3072, 2560 x 3900, 2048 x 8192, 4096 x 12288 and 5120 x 25600, for 3 to
// 8 steps.  With bf16 images it is up to 2 times that of single steps (columns falling like 1 / j); with a last Q of one term up to 1.7
// times (groups of alike rows), in bf16 throughout 2.9 times; merging four steps 2 times (constant plus noise).
// Of the 25.9 ms of 4 x 25600 x 5120 the diagonal of Q costs the update 0.2 and the second term the last product 4.2.
// Speed (us, single steps -> merged): 4 x 25600 x 5120 34900 -> 25900, 5 x 4096 x 12288 14400 -> 12600, 1 x 5120 x 13824 5180 -> 4460, 2 x
// 2048 x 4800 1070 -> 970, 1 x 5120 x 10240 4020 -> 3840; but 2 x 4096 x 6400 4090 -> 4210, 1 x 4096 x 8192 2230 ->
// 2290, 4 x 2048 x 4096 1430 -> 1470: hence m <= 0.45 n, from 5120 rows on m <= n / 2.  Merged classes do not share launches with
// single-step ones (group_runs): a matrix of fewer than 256 update tiles, which would have shared them, loses more by
// that than it gains (1 x 2048 x 6144 with three smaller classes 1300 -> 1380, 1 x 4096 x 1536 550 -> 760; 1 x 9728 x 2560 1960 -> 1850): hence m n >=
// 2^24.  The rule looks at the shape and the coefficients alone, so that a matrix's result does not depend on what
// shares its launch.  The spare arrays (Spare) fit wherever it holds.
struct StagePlan {
  int steps, first, last;   // steps in all, in the first stage (if it is merged) and in the last one (if that is), 0 otherwise
  int count() const { return steps - (first ? first - 1 : 0) - (last ? last - 1 : 0); }
  int len(int i) const { return i == 0 && first ? first : i + 1 == count() && last ? last : 1; }
  bool operator==(const StagePlan& o) const { return steps == o.steps && first == o.first && last == o.last; }
};
StagePlan stage_plan(const Shape& s, const canz_muon_hparams& hp) {
  const bool wide = s.m >= 1536 && s.m * s.n >= (int64_t(1) << 24) && (s.m >= 5120 ? 2 * s.m <= s.n : 20 * s.m <= 9 * s.n);
  if (!(hp.precision == CANZ_PREC_BF16 && hp.ns_steps >= 3 && hp.c != 0.f && wide && bounded_map(hp))) return {hp.ns_steps, 0, 0};
  return {hp.ns_steps, hp.ns_steps >= 4 ? 3 : 2, hp.ns_steps >= 5 ? 2 : 0};
}

// Launch batches that are too small to fill the chip on their own for long (fewer than 8
// rounds of update tiles on 256 CUs) are run together, up to MAX_KINDS consecutive ones of them: their Gram,
// polynomial and update products then share launches.  Batches that share launches must agree in their stages (which
// depend on the shape alone: a matrix's result does not depend on what shares its launch), so merged and single-step batches of
// such a window are two runs; they are put in that order.  first[i] .. first[i + 1] are the batches of run i.  Only in bf16
// mode; the fp32 verification path keeps one batch per run.
constexpr int64_t SMALL_BATCH_TILES = 8 * 256;
std::vector<int> group_runs(std::vector<Batch>& batches, const canz_muon_hparams& hp) {
  std::vector<int> first;
  const int n = static_cast<int>(batches.size());
  for (int i = 0; i < n;) {
    int j = i + 1;
    if (hp.precision == CANZ_PREC_BF16 && batches[i].update_tiles() < SMALL_BATCH_TILES) {
      int64_t elems = batches[i].s0.mp * batches[i].s0.np * batches[i].nb;
      while (j < n && j - i < MAX_KINDS && batches[j].update_tiles() < SMALL_BATCH_TILES) {
        const int64_t more = batches[j].s0.mp * batches[j].s0.np * batches[j].nb;
        if (elems + more > MAX_BATCH_ELEMS) break;
        elems += more;
        ++j;
      }
    }
    first.push_back(i);
    if (j > i + 1) {
      const StagePlan plan = stage_plan(batches[i].s0, hp);
      const auto rest = std::stable_partition(batches.begin() + i, batches.begin() + j,
                                              [&](const Batch& b) { return stage_plan(b.s0, hp) == plan; });
      if (const int k = static_cast<int>(rest - batches.begin()); k < j) first.push_back(k);   // there are two plans at most
    }
    i = j;
  }
  first.push_back(n);
  return first;
}

// Where the further m x m arrays of a batch whose steps are merged lie: B A, two more images for the polynomials and their
// products, five diagonals.  Between a Gram product and the next update (or last product) neither X nor the X^T that is not in use
// (xt[cur ^ 1]) is read, and they lie side by side: 2 m n elements of two bytes, of which 3 m m images leave at least 512 m bytes
// (3 m < 2 n, both multiples of 256).  The diagonals are at the end that belongs to X^T, since the Gram product leaves that
// of A while it reads X.  What X is multiplied with must not lie there: its image takes the place of A and its diagonal that of B,
// two terms take both.
struct Spare {
  size_t t, b1, b2, diag;   // byte offsets from the start of the free piece
};
Spare spare(const Shape& s, int nb, int cur) {
  const size_t img = align_up(static_cast<size_t>(nb) * s.mp * s.mp * 2);
  const size_t diag = align_up(static_cast<size_t>(5) * nb * s.mp * sizeof(float));
  const size_t all = 2 * align_up(static_cast<size_t>(nb) * s.mp * s.np * 2);
  const size_t at = cur == 0 ? 0 : diag;   // X, X^T  or  X^T, X
  return Spare{at, at + img, at + 2 * img, cur == 0 ? all - diag : 0};
}

size_t run_bytes(const std::vector<Batch>& batches, int lo, int hi, const canz_muon_hparams& hp) {
  size_t total = split_bytes(hp.precision);
  for (int k = lo; k < hi; ++k) total += carve(batches[k].s0, batches[k].nb, hp.precision).total;
  return total;
}

// One run: the batches lo .. hi-1 side by side in the workspace, then the split scratch.
template <typename T>
int run_batches(const std::vector<Batch>& batches, int lo, int hi, const canz_muon_hparams& hp, char* ws,
                hipStream_t st) {
  constexpr bool is_bf16 = sizeof(T) == 2;
  const int nk = hi - lo;
  const StagePlan stages = stage_plan(batches[lo].s0, hp);   // the same for all batches of a run
  struct Kind {
    T *xw, *xt[2], *a, *bm;
    void *t, *b[3];            // merged steps: B A, three images for polynomials and their products
    float *da, *dt, *db[3];    // ... and the diagonals
    float *partial, *scale, *scale2;
    int64_t x_elems, a_elems;
    int tiles, nb;
    Shape s0, shape[2];
    OutSpec out[2];
    int first[2];
    GemmDims gram, poly, upd;
  };
  Kind kind[MAX_KINDS];
  size_t base = 0;
  for (int k = 0; k < nk; ++k) {
    const Batch& bt = batches[lo + k];
    Kind& kd = kind[k];
    const Carve c = carve(bt.s0, bt.nb, hp.precision);
    char* w = ws + base;
    kd.xw = reinterpret_cast<T*>(w + c.xw);
    kd.xt[0] = reinterpret_cast<T*>(w + c.xt0), kd.xt[1] = reinterpret_cast<T*>(w + c.xt1);
    kd.a = reinterpret_cast<T*>(w + c.a), kd.bm = reinterpret_cast<T*>(w + c.b);
    kd.partial = reinterpret_cast<float*>(w + c.partial);
    kd.scale = reinterpret_cast<float*>(w + c.scale), kd.scale2 = reinterpret_cast<float*>(w + c.scale2);
    base += c.total;
    const Shape& s = kd.s0 = bt.s0;
    kd.nb = bt.nb;
    kd.x_elems = s.mp * s.np, kd.a_elems = s.mp * s.mp;
    kd.tiles = momentum_tiles(s);
    kd.first[0] = 0, kd.first[1] = bt.part[0].n();
    kd.gram = GemmDims{s.mp, s.mp, s.np, s.np, s.np, kd.x_elems, kd.x_elems, bt.nb};
    kd.poly = GemmDims{s.mp, s.mp, s.mp, s.mp, s.mp, kd.a_elems, kd.a_elems, bt.nb};
    kd.upd = GemmDims{s.mp, s.np, s.mp, s.mp, s.mp, kd.a_elems, kd.x_elems, bt.nb};
  }
  const SplitWs split{reinterpret_cast<float*>(ws + base), SPLIT_MAX_BLOCKS};
  // X itself, beside X^T: in fp32 mode, for the update without a Newton-Schulz step, and for Gram products of few tiles.  From X^T those take
  // longer (the transposing LDS reads run at half the rate: 1 x 25600x128 65 us -> 80, 26 x 2048x1024 76 -> 85), which a second image of
  // few rows in all, written by the momentum kernel and every update, does not outweigh.  us a step, with X -> without, by rows in all and length:
  //    256   x 4096 127 -> 134, x 25600 421 -> 451                    512   2 x 256x4096 143 -> 143, x 16384 326 -> 344; 1 x 512x4096 157 -> 152
  //   1024   4 x 256x2048 110 -> 112, x 8192 225 -> 235; 2 x 512x2048 131 -> 127, x 8192 253 -> 256; 1 x 1024x2048 144 -> 142, x 12288 383 -> 388
  //   1536   3 x 512x1024 119 -> 113, x 25600 844 -> 812; 1 x 1536x2048 225 -> 219, x 8192 529 -> 510
  //   1792   7 x 256x1024 99 -> 97, x 8192 274 -> 269, x 16384 539 -> 513
  // and beyond: 8 x 512x1024 153 -> 143, 1 x 2048x8192 677 -> 667, 8 x 512x8192 628 -> 598, 26 x 2048x1024 1460 -> 1363, 4 x 25600x5120
  // 26500 -> 26100.  Up to 1024 rows either may win, from 1536 on it never pays.
  int64_t all_rows = 0;
  for (int k = 0; k < nk; ++k) all_rows += kind[k].s0.mp * kind[k].nb;
  const bool wants_x = !is_bf16 || hp.ns_steps == 0 || (all_rows < 1536 && !stages.first && !stages.last);

  // momentum (+ gather, cast, both orientations, tile sums of U^2) per part, norm per batch; several parts whose buffers fit one
  // table go in one launch each (four classes of a 0.6B-shaped layer: 55 -> 33 us and 12 -> 4)
  int n_parts = 0, n_grads = 0, n_outs = 0;
  for (int k = 0; k < nk; ++k)
    for (const Part& part : batches[lo + k].part)
      if (part.n() > 0) ++n_parts, n_grads += static_cast<int>(part.grad.size()), n_outs += static_cast<int>(part.out.size());
  const bool shared = is_bf16 && n_parts > 1 && n_parts <= MAX_PARTS && n_grads <= MAX_PTRS && n_outs <= MAX_PTRS;
  PtrTable all_grad{}, all_mom{};
  OutSpec all_out{};
  MomentumPart<__bf16> mparts[MAX_PARTS];
  FinalPart fparts[MAX_PARTS];
  int first_out[MAX_KINDS][2] = {};
  n_parts = n_grads = n_outs = 0;
  int n_moms = 0;
  for (int k = 0; k < nk; ++k) {
    const Batch& bt = batches[lo + k];
    Kind& kd = kind[k];
    for (int h = 0; h < 2; ++h) {
      const Part& part = bt.part[h];
      const int n = part.n();
      if (n == 0) continue;
      const canz_group& g = *part.proto;
      kd.shape[h] = make_shape(g);
      PtrTable grad{}, mom{};
      OutSpec& o = kd.out[h];
      o = OutSpec{};
      const int n_out = hp.out_mode == CANZ_OUT_DELTA ? n * g.tp : n;
      for (int i = 0; i < n * g.tp; ++i) grad.p[i] = const_cast<void*>(part.grad[i]);
      for (int i = 0; i < n; ++i) mom.p[i] = part.mom[i];
      for (int i = 0; i < n_out; ++i) o.out.p[i] = part.out[i];
      o.out_dtype = g.out_dtype;
      o.out_mode = hp.out_mode;
      o.decay = static_cast<float>(1.0 - static_cast<double>(hp.lr) * static_cast<double>(hp.weight_decay));
      o.neg_lr_scale = static_cast<float>(-static_cast<double>(hp.lr) * update_scale(g, hp.scale_mode));
      const int f = kd.first[h];
      if constexpr (is_bf16) if (shared) {
        mparts[n_parts++] = MomentumPart<__bf16>{kd.shape[h], n, g.grad_dtype, n_grads, n_moms, wants_x ? reinterpret_cast<__bf16*>(kd.xw) + f * kd.x_elems : nullptr,
                                                 kd.xt[0] + f * kd.x_elems, kd.partial + static_cast<int64_t>(f) * kd.tiles};
        first_out[k][h] = n_outs;
        for (int i = 0; i < n * g.tp; ++i) all_grad.p[n_grads++] = grad.p[i];
        for (int i = 0; i < n; ++i) all_mom.p[n_moms++] = mom.p[i];
        for (int i = 0; i < n_out; ++i) all_out.out.p[n_outs++] = o.out.p[i];
        all_out.out_mode = o.out_mode, all_out.decay = o.decay;
        continue;
      }
      CANZ_HIP(CANZ_KERNEL_MOMENTUM,
               launch_momentum<T>(kd.shape[h], n, grad, g.grad_dtype, mom, hp.beta, hp.nesterov, wants_x ? kd.xw + f * kd.x_elems : nullptr,
                                  kd.xt[0] + f * kd.x_elems, kd.partial + static_cast<int64_t>(f) * kd.tiles, st),
               "momentum kernel");
    }
    if (!shared)
      CANZ_HIP(CANZ_KERNEL_NORM, launch_norm_scale(kd.nb, kd.tiles, kd.partial, hp.eps, kd.scale, kd.scale2, st),
               "norm kernel");
  }
  if (shared) {
    NormBatch nb[MAX_KINDS];
    for (int k = 0; k < nk; ++k) nb[k] = NormBatch{kind[k].nb, kind[k].tiles, kind[k].partial, kind[k].scale, kind[k].scale2};
    CANZ_HIP(CANZ_KERNEL_MOMENTUM, launch_momentum_parts(n_parts, mparts, all_grad, all_mom, hp.beta, hp.nesterov, st), "momentum kernel");
    CANZ_HIP(CANZ_KERNEL_NORM, launch_norm_scale_batches(nk, nb, hp.eps, st), "norm kernel");
  }

  if (hp.ns_steps == 0) {
    for (int k = 0; k < nk; ++k)
      for (int h = 0; h < 2; ++h) {
        const int n = batches[lo + k].part[h].n();
        if (n == 0) continue;
        const Kind& kd = kind[k];
        const Shape& s = kd.shape[h];
        const T* straight = (s.tall ? kd.xt[0] : kd.xw) + kd.first[h] * kd.x_elems;
        const int64_t ld = s.tall ? s.mp : s.np;
        CANZ_HIP(CANZ_KERNEL_APPLY,
                 launch_apply<T>(s, n, straight, ld, kd.x_elems, kd.scale + kd.first[h], kd.out[h], st), "apply kernel");
      }
    return CANZ_OK;
  }

  // The products of one stage (see stage_plan) among the m x m matrices, every shape class of the run side by side;
  // q[k]: the image that X is multiplied with (or its two terms, in a last stage of merged steps), dq[k]: its diagonal, if it
  // is apart.  `cur`: which X^T buffer is in use.
  const void* q[MAX_KINDS] = {};
  const float* dq[MAX_KINDS] = {};
  auto stage_bf16 = [&](int len, bool first, bool last_stage, int cur) -> int {
    GemmBatch gb;
    const bool apart = len > 1;
    for (int k = 0; apart && k < nk; ++k) {
      Kind& kd = kind[k];
      const Spare x = spare(kd.s0, kd.nb, cur);
      char* w = reinterpret_cast<char*>(cur == 0 ? kd.xw : kd.xt[0]);
      kd.t = w + x.t, kd.b[0] = kd.bm, kd.b[1] = w + x.b1, kd.b[2] = w + x.b2;
      float* dv = reinterpret_cast<float*>(w + x.diag);
      const int64_t len_d = static_cast<int64_t>(kd.nb) * kd.s0.mp;
      kd.da = dv, kd.dt = dv + len_d, kd.db[0] = dv + 2 * len_d, kd.db[1] = dv + 3 * len_d, kd.db[2] = dv + 4 * len_d;
    }
    gb.n = nk;
    for (int k = 0; k < nk; ++k) {
      const Kind& kd = kind[k];
      GemmProblem& pr = gb.pr[k] = GemmProblem{};
      pr.d = kd.gram, pr.p = pr.q = wants_x ? kd.xw : kd.xt[cur], pr.c = kd.a, pr.scale = first ? kd.scale2 : nullptr;
      pr.sym.diag = apart ? kd.da : nullptr;
    }
    CANZ_HIP(CANZ_KERNEL_GRAM, launch_gram_bf16(gb, !wants_x, split, st), "gram kernel");
    // the product of the symmetric images P (index ip of b, unit B) and Y with their diagonals
    auto mul = [&](const Kind& kd, int ip, const void* y, const float* dy, float unit, void* c, float* dc) {
      GemmProblem pr{};
      pr.d = kd.poly, pr.p = kd.b[ip], pr.q = y, pr.c = c;
      pr.sym.aux = y, pr.sym.aux2 = kd.b[ip], pr.sym.x = kd.db[ip], pr.sym.y = dy, pr.sym.diag = dc, pr.sym.unit = unit;
      return pr;
    };
    // B_1 -> b[0] (or, of two steps, b[2]), the later ones -> b[1], the product of the first two -> b[2]: the last product
    // reads b[1] and b[2], so that b[0], behind A, is free for its diagonal or second term
    int iq = -1;   // where the product of the polynomials so far lies
    for (int i = 0; i < len; ++i) {
      const bool last = i + 1 == len;
      const int ib = i > 0 ? 1 : len == 2 ? 2 : 0;
      for (int k = 0; k < nk; ++k) {
        const Kind& kd = kind[k];
        GemmProblem& pr = gb.pr[k] = GemmProblem{};
        pr.d = kd.poly, pr.p = kd.a, pr.q = kd.a, pr.c = apart ? kd.b[ib] : static_cast<void*>(kd.bm);
        pr.sym.aux = kd.a;
        if (apart) pr.sym.x = kd.da, pr.sym.y = kd.da, pr.sym.diag = kd.db[ib];
      }
      gb.n = nk;
      CANZ_HIP(CANZ_KERNEL_POLY, launch_poly_bf16(gb, hp.a, hp.b, hp.c, split, st), "poly kernel");
      if (!apart) break;
      gb.n = 0;
      if (last) {
        for (int k = 0; k < nk; ++k) {
          const Kind& kd = kind[k];
          float* dlast = reinterpret_cast<float*>(kd.bm);
          gb.pr[gb.n++] = mul(kd, ib, kd.b[iq], kd.db[iq], UNIT_B, kd.a, dlast);
        }
        CANZ_HIP(CANZ_KERNEL_POLY, launch_mul_f16(gb, last_stage ? MulResult::Q2 : MulResult::Q, split, st), "product kernel (Q)");
        break;
      }
      for (int k = 0; k < nk; ++k) gb.pr[gb.n++] = mul(kind[k], ib, kind[k].a, kind[k].da, UNIT_A, kind[k].t, kind[k].dt);
      if (iq >= 0)
        for (int k = 0; k < nk; ++k) gb.pr[gb.n++] = mul(kind[k], ib, kind[k].b[iq], kind[k].db[iq], UNIT_B, kind[k].b[2], kind[k].db[2]);
      CANZ_HIP(CANZ_KERNEL_POLY, launch_mul_f16(gb, MulResult::CHAIN, split, st), "product kernel (B A, Q)");
      iq = iq < 0 ? ib : 2;
      gb.n = nk;
      for (int k = 0; k < nk; ++k) gb.pr[k] = mul(kind[k], ib, kind[k].t, kind[k].dt, UNIT_A, kind[k].a, kind[k].da);
      CANZ_HIP(CANZ_KERNEL_POLY, launch_mul_f16(gb, MulResult::CHAIN, split, st), "product kernel (B A B)");
    }
    for (int k = 0; k < nk; ++k) {
      q[k] = apart ? kind[k].a : kind[k].bm;
      dq[k] = apart ? reinterpret_cast<const float*>(kind[k].bm) : nullptr;
    }
    return CANZ_OK;
  };

  int cur = 0;
  for (int sg = 0; sg < stages.count(); ++sg) {
    const bool first_it = sg == 0, last = sg + 1 == stages.count();
    if (is_bf16) {
      if (int rc = stage_bf16(stages.len(sg), first_it, last, cur)) return rc;
      if (!last) {
        GemmBatch gb;
        gb.n = nk;
        for (int k = 0; k < nk; ++k) {
          const Kind& kd = kind[k];
          GemmProblem& pr = gb.pr[k] = GemmProblem{};
          pr.d = kd.upd, pr.p = q[k], pr.q = kd.xt[cur], pr.c = wants_x ? kd.xw : nullptr, pr.ct = kd.xt[cur ^ 1];
          pr.scale = first_it ? kd.scale : nullptr;
          pr.sym.x = dq[k], pr.sym.aux = kd.xt[cur];
        }
        CANZ_HIP(CANZ_KERNEL_UPDATE, launch_update_bf16(gb, split, st), "update kernel");
      }
    }
    n_parts = 0;
    for (int k = 0; k < nk; ++k) {
      const Kind& kd = kind[k];
      const float* sc1 = first_it ? kd.scale : nullptr;
      const float* sc2 = first_it ? kd.scale2 : nullptr;
      if (!is_bf16) {
        CANZ_HIP(CANZ_KERNEL_GRAM, launch_gram_f32(kd.gram, kd.xw, kd.a, sc2, st), "gram kernel");
        CANZ_HIP(CANZ_KERNEL_POLY, launch_poly_f32(kd.poly, kd.a, kd.bm, hp.a, hp.b, hp.c, st), "poly kernel");
        if (!last)
          CANZ_HIP(CANZ_KERNEL_UPDATE, launch_update_f32(kd.upd, kd.bm, kd.xt[cur], kd.xw, kd.xt[cur ^ 1], sc1, st),
                   "update kernel");
        q[k] = kd.bm;
      }
      if (!last) continue;
      // last product, written in the caller's orientation: for the tall part the roles of
      // the polynomial and of X swap, so that C comes out as rows x cols
      for (int h = 0; h < 2; ++h) {
        const int n = batches[lo + k].part[h].n();
        if (n == 0) continue;
        const Shape& s = kd.s0;
        const int terms = is_bf16 && stages.len(sg) > 1 ? 2 : 1;
        const T* bk = static_cast<const T*>(q[k]) + kd.first[h] * kd.a_elems * terms;
        const T* xk = kd.xt[cur] + kd.first[h] * kd.x_elems;
        const float* sk = sc1 ? sc1 + kd.first[h] : nullptr;
        const bool tall = kd.shape[h].tall;
        GemmDims fin = tall ? GemmDims{s.np, s.mp, s.mp, s.mp, s.mp, kd.x_elems, kd.a_elems, n} : kd.upd;
        fin.nb = n;
        const void* P = tall ? static_cast<const void*>(xk) : static_cast<const void*>(bk);
        const void* Q = tall ? static_cast<const void*>(bk) : static_cast<const void*>(xk);
        if (terms == 2) {   // the second term first
          (tall ? fin.ldq : fin.ldp) = 2 * s.mp, (tall ? fin.sq : fin.sp) = 2 * kd.a_elems;
          fin.nseg = 2, (tall ? fin.qseg : fin.pseg) = 0x01u;
          CANZ_HIP(CANZ_KERNEL_FINAL, launch_terms_final(fin, P, Q, kd.shape[h], kd.out[h], st), "final kernel");
        } else if (is_bf16 && shared)   // below, all parts together if that pays
          fparts[n_parts++] = FinalPart{fin, P, Q, sk, kd.shape[h], kd.out[h].out_dtype, first_out[k][h], kd.out[h].neg_lr_scale};
        else if (is_bf16)
          CANZ_HIP(CANZ_KERNEL_FINAL, launch_final_bf16(fin, P, Q, sk, split, kd.shape[h], kd.out[h], st), "final kernel");
        else
          CANZ_HIP(CANZ_KERNEL_FINAL, launch_final_f32(fin, P, Q, sk, kd.shape[h], kd.out[h], st), "final kernel");
      }
    }
    if (n_parts > 0 && final_parts_fit(n_parts, fparts)) {
      CANZ_HIP(CANZ_KERNEL_FINAL, launch_final_parts_bf16(n_parts, fparts, all_out, st), "final kernel");
    } else {
      for (int i = 0; i < n_parts; ++i) {
        const FinalPart& f = fparts[i];
        OutSpec o = all_out;
        o.out_dtype = f.out_dtype, o.neg_lr_scale = f.neg_lr_scale;
        std::copy(all_out.out.p + f.first_out, all_out.out.p + MAX_PTRS, o.out.p);
        CANZ_HIP(CANZ_KERNEL_FINAL, launch_final_bf16(f.d, f.p, f.q, f.scale, split, f.s, o, st), "final kernel");
      }
    }
    cur ^= 1;
  }
  return CANZ_OK;
}

}  // namespace
}  // namespace canz

extern "C" int canz_muon_workspace_bytes(const canz_group* g, int32_t n_groups, const canz_muon_hparams* hp,
                                         size_t* bytes_out) {
  using namespace canz;
  if (!bytes_out) return fail(CANZ_EINVAL, "null bytes_out");
  if (n_groups < 0 || (n_groups > 0 && !g)) return fail(CANZ_EINVAL, "bad group array");
  if (int rc = check_hparams(hp)) return rc;
  size_t need = ALIGN;
  for (int i = 0; i < n_groups; ++i)
    if (int rc = check_group(g[i], i, false, hp->out_mode)) return rc;
  std::vector<Batch> batches;
  if (int rc = collect_batches(g, n_groups, hp->out_mode, false, batches)) return rc;
  const std::vector<int> first = group_runs(batches, *hp);
  for (size_t r = 0; r + 1 < first.size(); ++r)
    need = std::max(need, run_bytes(batches, first[r], first[r + 1], *hp));
  *bytes_out = need;
  return CANZ_OK;
}

namespace canz {
namespace {

// Validates the call and enqueues every run of launch batches on `st`, using `workspace`.
int muon_step_on(const canz_group* g, int32_t n_groups, const canz_muon_hparams* hp, void* workspace,
                 size_t workspace_bytes, hipStream_t st) {
  if (n_groups < 0 || (n_groups > 0 && !g)) return fail(CANZ_EINVAL, "bad group array");
  if (int rc = check_hparams(hp)) return rc;
  size_t need = 0;
  if (int rc = canz_muon_workspace_bytes(g, n_groups, hp, &need)) return rc;
  for (int i = 0; i < n_groups; ++i)
    if (int rc = check_group(g[i], i, true, hp->out_mode)) return rc;
  bool any = false;
  for (int i = 0; i < n_groups; ++i) any = any || g[i].n_mats > 0;
  if (!any) return CANZ_OK;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (ALIGN - 1)))
    return fail(CANZ_EWORKSPACE, "workspace null or not 256-byte aligned");
  if (workspace_bytes < need)
    return fail(CANZ_EWORKSPACE, "workspace too small: %zu bytes given, %zu needed", workspace_bytes, need);

  char* ws = static_cast<char*>(workspace);
  std::vector<Batch> batches;
  if (int rc = collect_batches(g, n_groups, hp->out_mode, true, batches)) return rc;
  const std::vector<int> first = group_runs(batches, *hp);
  for (size_t r = 0; r + 1 < first.size(); ++r) {
    const int rc = hp->precision == CANZ_PREC_BF16 ? run_batches<__bf16>(batches, first[r], first[r + 1], *hp, ws, st)
                                                   : run_batches<float>(batches, first[r], first[r + 1], *hp, ws, st);
    if (rc) return rc;
  }
  return CANZ_OK;
}

// ---- workspace that lives in the library (canz_muon_step_static).  The array sits in the
// code object of this file; every device that loads the library holds its own copy at its own
// address until the process ends.  Host code never uses the array's name as an address: the
// device address is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[CANZ_STATIC_WORKSPACE_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_lock;
void* g_scratch_ptr[MAX_DEVICES] = {nullptr};

// Device address of `scratch` on the current device (nullptr + error message on failure).
void* scratch_address() {
  int dev = -1;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
    fail(CANZ_EHIP, "hipGetDevice: %s (device %d)", hipGetErrorString(err), dev);
    return nullptr;
  }
  std::lock_guard<std::mutex> hold(g_scratch_lock);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (err != hipSuccess || !ptr) {
      fail(CANZ_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(err));
      return nullptr;
    }
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}

}  // namespace
}  // namespace canz

extern "C" int canz_muon_step(const canz_group* g, int32_t n_groups, const canz_muon_hparams* hp, void* workspace,
                              size_t workspace_bytes, void* hip_stream) {
  return canz::muon_step_on(g, n_groups, hp, workspace, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

extern "C" int canz_muon_step_static(const canz_group* g, int32_t n_groups, const canz_muon_hparams* hp,
                                     void* hip_stream) {
  using namespace canz;
  if (n_groups < 0 || (n_groups > 0 && !g)) return fail(CANZ_EINVAL, "bad group array");
  size_t need = 0;
  if (int rc = canz_muon_workspace_bytes(g, n_groups, hp, &need)) return rc;
  if (need > CANZ_STATIC_WORKSPACE_BYTES)
    return fail(CANZ_EWORKSPACE, "step needs %zu bytes of scratch, the built-in workspace holds %zu", need,
                static_cast<size_t>(CANZ_STATIC_WORKSPACE_BYTES));
  void* ptr = scratch_address();
  if (!ptr) return CANZ_EHIP;
  return muon_step_on(g, n_groups, hp, ptr, CANZ_STATIC_WORKSPACE_BYTES, static_cast<hipStream_t>(hip_stream));
}

extern "C" int canz_profile_enable(int32_t max_launches) {
  using namespace canz;
  if (max_launches < 1) return fail(CANZ_EINVAL, "max_launches must be >= 1");
  std::lock_guard<std::mutex> hold(g_prof.lock);
  while (g_prof.ev.size() < static_cast<size_t>(max_launches) * 2) {
    hipEvent_t e;
    hipError_t err = hipEventCreate(&e);
    if (err != hipSuccess) return fail(CANZ_EHIP, "hipEventCreate: %s", hipGetErrorString(err));
    g_prof.ev.push_back(e);
  }
  g_prof.kind.assign(g_prof.ev.size() / 2, 0);
  g_prof.used = 0;
  g_prof.on.store(true);
  return CANZ_OK;
}

extern "C" int canz_profile_collect(double* ms_out, int64_t* launches_out) {
  using namespace canz;
  if (!ms_out || !launches_out) return fail(CANZ_EINVAL, "null output pointer");
  for (int k = 0; k < CANZ_KERNEL_KINDS; ++k) ms_out[k] = 0.0, launches_out[k] = 0;
  std::lock_guard<std::mutex> hold(g_prof.lock);
  for (size_t i = 0; i < g_prof.used; ++i) {
    hipError_t err = hipEventSynchronize(g_prof.ev[2 * i + 1]);
    float ms = 0.f;
    if (err == hipSuccess) err = hipEventElapsedTime(&ms, g_prof.ev[2 * i], g_prof.ev[2 * i + 1]);
    if (err != hipSuccess) return fail(CANZ_EHIP, "profile event: %s", hipGetErrorString(err));
    ms_out[g_prof.kind[i]] += ms;
    launches_out[g_prof.kind[i]] += 1;
  }
  g_prof.used = 0;
  return CANZ_OK;
}

extern "C" int canz_profile_disable(void) {
  std::lock_guard<std::mutex> hold(canz::g_prof.lock);
  canz::g_prof.on.store(false);
  canz::g_prof.used = 0;
  return CANZ_OK;
}
