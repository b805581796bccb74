// Spectral projected gradient (SPG) on the l1-constrained least-squares
// problem of Section 5.2 (basis pursuit):
//     min 1/2 ||A x - b||^2   s.t.  ||x||_1 <= radius,
// with every projection onto the l1 ball done by the library's projection
// (Section 3.2, Algorithm 4 with Algorithm 2 as the start), warm-started from
// the current iterate as Section 3.1 suggests.  The SPG steps are those of
// Birgin, Martinez and Raydan's SPG2: x_0 = 0, the spectral step
// lam_{k+1} = s's / s'y clipped to [1e-30, 1e30] (the first one
// 1/||P(x_0 - g_0) - x_0||_inf), the direction d = P(x - lam g) - x, and a
// non-monotone line search over the last `memory` objective values with
// safeguarded quadratic interpolation; stop when ||P(x - g) - x||_inf <= tol.
//
// For this f the line search needs no extra product: with r = A x - b and
// Ad = A d,  f(x + t d) = f(x) + t g'd + t^2/2 ||Ad||^2  (g'd = r'Ad), and
// s'y = t^2 ||Ad||^2, s's = t^2 ||d||^2, so each iteration costs two
// products with A (A d, then A^T r at the new point) and two projections
// (the direction and the stopping test).
//
// A is dense, row-major m x n, FP64.  Kernels:
//   spg_gemv_n_kernel   y = A v (- b): one block per row, 16-byte loads;
//   spg_gemv_t_kernel   partial column sums of A^T v over row chunks,
//   spg_cols_kernel     the chunks summed in order (deterministic);
//   spg_vec_kernel      fused vector updates with their reductions;
//   spg_reduce_kernel   one block: the partial records to a result array.
// The host runs the scalar part and reads a few reduced values per step; it
// waits four times (two projections, the line search's values, the projected
// gradient's).  Eight steps on 2048 x 65536: 4.6 ms, 3.5 of them in the
// products (5.3-5.7 TB/s); with a copy and a wait for each reduction 4.9 ms.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>

#include "cqk_device.h"
#include "cqk_internal.h"

namespace cqk {
namespace {

constexpr int kBlock = 256;
constexpr int kRBlock = 1024;
constexpr int kRowsPerChunk = 128;  // rows per block of the transposed product
constexpr int kColsPerBlock = 2 * kBlock;
constexpr double kLMin = 1e-30, kLMax = 1e30, kGamma = 1e-4, kSigma1 = 0.1, kSigma2 = 0.9;

// y_i = sum_j A_ij v_j (minus b_i when b is given); one block per row.
template <bool VEC>
__global__ __launch_bounds__(kBlock) void spg_gemv_n_kernel(const double* A, const double* v,
                                                           const double* b, int64_t n,
                                                           double* y) {
  const int64_t i = blockIdx.x;
  const double* row = A + i * n;
  double acc = 0.0;
  if (VEC) {
    // row and v 16-byte aligned (n even): pairs, four in flight per thread
    const int64_t np = n / 2;
    const double2* r2 = reinterpret_cast<const double2*>(row);
    const double2* v2 = reinterpret_cast<const double2*>(v);
    int64_t j = threadIdx.x;
    for (; j + 3 * kBlock < np; j += 4 * kBlock) {
      double2 a[4], w[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        a[k] = r2[j + k * kBlock];
        w[k] = v2[j + k * kBlock];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) acc += a[k].x * w[k].x + a[k].y * w[k].y;
    }
    for (; j < np; j += kBlock) {
      const double2 a = r2[j], w = v2[j];
      acc += a.x * w.x + a.y * w.y;
    }
  } else {
    for (int64_t j = threadIdx.x; j < n; j += kBlock) acc += row[j] * v[j];
  }
  __shared__ double lds[kBlock / kWave];
  __shared__ double tot[1];
  block_reduce<1, 0, 0, kBlock>(&acc, nullptr, nullptr, lds, tot);
  if (threadIdx.x == 0) y[i] = b ? tot[0] - b[i] : tot[0];
}

// part[c][j] = sum over the rows of chunk c of v_i A_ij; block (x: column
// tile of kColsPerBlock, y: chunk c), two adjacent columns per thread.
template <bool VEC>
__global__ __launch_bounds__(kBlock) void spg_gemv_t_kernel(const double* A, const double* v,
                                                           int64_t m, int64_t n, double* part) {
  const int64_t j = (int64_t)blockIdx.x * kColsPerBlock + 2 * (int64_t)threadIdx.x;
  const int64_t i0 = (int64_t)blockIdx.y * kRowsPerChunk;
  const int64_t i1 = min(i0 + (int64_t)kRowsPerChunk, m);
  double s0 = 0.0, s1 = 0.0;
  if (j < n) {
    if (VEC && j + 1 < n) {
      for (int64_t i = i0; i < i1; ++i) {
        const double2 a = *reinterpret_cast<const double2*>(A + i * n + j);
        const double w = v[i];
        s0 += w * a.x;
        s1 += w * a.y;
      }
    } else {
      const bool two = j + 1 < n;
      for (int64_t i = i0; i < i1; ++i) {
        const double w = v[i];
        s0 += w * A[i * n + j];
        if (two) s1 += w * A[i * n + j + 1];
      }
    }
    double* out = part + (int64_t)blockIdx.y * n;
    out[j] = s0;
    if (j + 1 < n) out[j + 1] = s1;
  }
}

// g_j = sum over chunks c (in order) of part[c][j].
__global__ __launch_bounds__(kBlock) void spg_cols_kernel(const double* part, int nchunk,
                                                          int64_t n, double* g) {
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (j >= n) return;
  double s = 0.0;
  for (int c = 0; c < nchunk; ++c) s += part[(int64_t)c * n + j];
  g[j] = s;
}

// Fused vector steps over n (or m) values, each block writing one partial
// record of kVS sums (then one max):
//   OP_STEP:  out = x - lam g                                   (no sums)
//   OP_DIR:   d = p - x;  sums g'd, d'd;  max |d|
//   OP_DOT:   sums u'w, w'w, u'u  over m                        (no writes)
enum SpgOp { OP_STEP = 0, OP_DIR = 1, OP_DOT = 2 };
constexpr int kVS = 3;

template <int OP>
__global__ __launch_bounds__(kBlock) void spg_vec_kernel(int64_t n, double c, const double* x,
                                                        const double* u, double* out,
                                                        double* partials, uint64_t* clock) {
  // the projection's time: from the end of OP_STEP to the start of OP_DIR
  if (OP == OP_DIR && blockIdx.x == 0 && threadIdx.x == 0)
    clock[1] = __builtin_amdgcn_s_memrealtime();
  double acc[kVS] = {0.0, 0.0, 0.0};
  double mx = 0.0;
  for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * kBlock) {
    if (OP == OP_STEP) {
      out[j] = x[j] - c * u[j];
    } else if (OP == OP_DIR) {
      // x: the iterate, u: the gradient, out: in the projection p, out d
      const double dj = out[j] - x[j];
      out[j] = dj;
      acc[0] += u[j] * dj;
      acc[1] += dj * dj;
      mx = fmax(mx, fabs(dj));
    } else {
      const double a = x[j], w = u[j];
      acc[0] += a * w;
      acc[1] += w * w;
      acc[2] += a * a;
    }
  }
  if (OP == OP_STEP && blockIdx.x == 0 && threadIdx.x == 0)
    clock[0] = __builtin_amdgcn_s_memrealtime();
  if (OP == OP_DIR || OP == OP_DOT) {
    __shared__ double lds[(kVS + 1) * (kBlock / kWave)];
    __shared__ double tot[kVS + 1];
    block_reduce<kVS, 0, 1, kBlock>(acc, nullptr, &mx, lds, tot);
    if (threadIdx.x == 0) write_partial(partials, tot, kVS + 1);
  }
}

// The accepted step: x += t d over n, r += t Ad over m with the sum r'r of the
// new r (its blocks' records as OP_DOT of r writes them).
__global__ __launch_bounds__(kBlock) void spg_move_kernel(int64_t n, int64_t m, double t,
                                                          const double* d, double* x,
                                                          const double* Ad, double* r,
                                                          double* partials) {
  const int64_t j0 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * kBlock;
  for (int64_t j = j0; j < n; j += step) x[j] += t * d[j];
  double acc[kVS] = {0.0, 0.0, 0.0};
  for (int64_t j = j0; j < m; j += step) {
    const double a = r[j] + t * Ad[j];
    r[j] = a;
    acc[0] += a * a;
  }
  acc[1] = acc[2] = acc[0];
  const double mx = 0.0;
  __shared__ double lds[(kVS + 1) * (kBlock / kWave)];
  __shared__ double tot[kVS + 1];
  block_reduce<kVS, 0, 1, kBlock>(acc, nullptr, &mx, lds, tot);
  if (threadIdx.x == 0) write_partial(partials, tot, kVS + 1);
}

// One block: G partial records of kVS sums and one max -> res[0..kVS], in the
// context's pinned host memory: the host reads them after the next wait on
// the stream, which it has to do anyway (a copy and a wait of their own took
// about 30 us per reduction).
__global__ __launch_bounds__(kRBlock) void spg_reduce_kernel(const double* partials, int G,
                                                             double* res) {
  __shared__ double lds[(kVS + 1) * (kRBlock / kWave)];
  __shared__ double tot[kVS + 1];
  reduce_partials<kVS, 0, 1, kRBlock>(partials, G, lds, tot);
  if (threadIdx.x <= kVS) res[threadIdx.x] = tot[threadIdx.x];
}

struct SpgWs {
  double *r, *Ad, *g, *z, *p, *d, *part, *partials;
  int nchunk, gvec;
};

}  // namespace

void fill_default_spg_opts(cqk_spg_opts* o) {
  std::memset(o, 0, sizeof(*o));
  o->tol = 1e-4;
  o->max_iter = 10000;
  o->memory = 10;
  o->warm = 1;
}

cqk_status run_spg_l1_lasso_f64(cqk_ctx* ctx, int64_t m, int64_t n, const double* A,
                                const double* b, double radius, double* x,
                                const cqk_spg_opts& so, cqk_spg_info* info) {
  using clock = std::chrono::steady_clock;
  const auto t_start = clock::now();
  double proj_ms = 0.0;
  hipStream_t s = ctx->stream;
  SpgWs W;
  W.nchunk = (int)((m + kRowsPerChunk - 1) / kRowsPerChunk);
  W.gvec = (int)std::max<int64_t>(1, std::min<int64_t>((std::max(m, n) + kBlock - 1) / kBlock,
                                                       (int64_t)ctx->num_cus * 4));
  auto al = [](size_t bytes) { return (bytes + 255) / 256 * 256; };
  const size_t bm = al((size_t)m * 8), bn = al((size_t)n * 8);
  const size_t bpart = al((size_t)W.nchunk * n * 8);
  const size_t bpar = al((size_t)(kVS + 1) * W.gvec * 8);
  const size_t total = 2 * bm + 4 * bn + bpart + bpar;
  cqk_status st = ensure_buffer(ctx, ctx->spg, total);
  if (st != CQK_OK) return st;
  char* w = (char*)ctx->spg.ptr;
  W.r = (double*)w;
  W.Ad = (double*)(w + bm);
  W.g = (double*)(w + 2 * bm);
  W.z = (double*)(w + 2 * bm + bn);
  W.p = (double*)(w + 2 * bm + 2 * bn);
  W.d = (double*)(w + 2 * bm + 3 * bn);
  W.part = (double*)(w + 2 * bm + 4 * bn);
  W.partials = (double*)(w + 2 * bm + 4 * bn + bpart);
  // scalars come back through the upper half of the context's pinned buffer
  // (its start mirrors the projection's state)
  // (three results of kVS + 1 values: of d or the projected gradient, of Ad,
  // of r)
  double* const hdir = (double*)((char*)ctx->host_pinned + ctx->host_pinned_bytes / 2);
  double* const had = hdir + 8;
  double* const hr = hdir + 16;
  uint64_t* const clock100 = (uint64_t*)(hdir + 24);  // 100 MHz ticks around a projection
  auto projected = [&]() { proj_ms += 1e-5 * (double)(clock100[1] - clock100[0]); };

  const bool vec = (n % 2 == 0) && ((uintptr_t)A % 16 == 0);
  auto gemv_n = [&](const double* v, const double* bb, double* y) {
    if (vec && ((uintptr_t)v % 16 == 0))
      hipLaunchKernelGGL(spg_gemv_n_kernel<true>, dim3((unsigned)m), dim3(kBlock), 0, s, A, v, bb, n, y);
    else
      hipLaunchKernelGGL(spg_gemv_n_kernel<false>, dim3((unsigned)m), dim3(kBlock), 0, s, A, v, bb, n, y);
  };
  auto gemv_t = [&](const double* v, double* out) {
    const dim3 grid((unsigned)((n + kColsPerBlock - 1) / kColsPerBlock), (unsigned)W.nchunk);
    if (vec)
      hipLaunchKernelGGL(spg_gemv_t_kernel<true>, grid, dim3(kBlock), 0, s, A, v, m, n, W.part);
    else
      hipLaunchKernelGGL(spg_gemv_t_kernel<false>, grid, dim3(kBlock), 0, s, A, v, m, n, W.part);
    hipLaunchKernelGGL(spg_cols_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock),
                       0, s, W.part, W.nchunk, n, out);
  };
  // queue a reduction; its results are there after the next wait
  auto reduce = [&](double* dst) {
    hipLaunchKernelGGL(spg_reduce_kernel, dim3(1), dim3(kRBlock), 0, s, W.partials, W.gvec, dst);
  };
  auto wait = [&]() -> cqk_status {
    if (hip_ok(hipGetLastError()) != CQK_OK) return CQK_DEVICE_ERROR;
    return hip_ok(hipStreamSynchronize(s));
  };
  cqk_opts po;
  fill_default_opts(&po);
  po.lambda0_mode = CQK_LAMBDA0_CONDAT;
  int64_t nproj = 0, newton = 0;
  // p = P(z), warm-started from x when asked; returns the projection status
  auto project = [&](const double* z, double* p) -> cqk_status {
    cqk_info pi;
    cqk_status e = run_simplex_f64(ctx, n, z, so.warm ? x : nullptr, nullptr, radius, p, true,
                                   po, &pi);
    nproj += 1;
    newton += pi.iterations;
    if (e != CQK_OK) return e;
    return (pi.status == CQK_OK) ? CQK_OK : (cqk_status)pi.status;
  };

  // x_0 = 0 = P(0); r = A x_0 - b; g = A^T r
  if (hip_ok(hipMemsetAsync(x, 0, (size_t)n * 8, s)) != CQK_OK) return CQK_DEVICE_ERROR;
  gemv_n(x, b, W.r);
  double fx = 0.0;
  std::vector<double> hist;
  double lam = 1.0;
  int it = 0;
  int status = CQK_OK;
  double pg = 0.0;
  // the projected gradient at x: pg = ||P(x - g) - x||_inf
  auto proj_grad = [&]() -> cqk_status {
    hipLaunchKernelGGL(spg_vec_kernel<OP_STEP>, dim3(W.gvec), dim3(kBlock), 0, s, n, 1.0, x, W.g,
                       W.z, W.partials, clock100);
    cqk_status e = project(W.z, W.p);
    if (e != CQK_OK) return e;
    hipLaunchKernelGGL(spg_vec_kernel<OP_DIR>, dim3(W.gvec), dim3(kBlock), 0, s, n, 0.0, x, W.g,
                       W.p, W.partials, clock100);
    reduce(hdir);
    e = wait();
    projected();
    pg = hdir[kVS];
    fx = 0.5 * hr[2];  // reduced before the projection
    return e;
  };
  gemv_t(W.r, W.g);
  hipLaunchKernelGGL(spg_vec_kernel<OP_DOT>, dim3(W.gvec), dim3(kBlock), 0, s, m, 0.0, W.r, W.r,
                     nullptr, W.partials, nullptr);
  reduce(hr);
  cqk_status e = proj_grad();
  if (e != CQK_OK) return e;
  hist.push_back(fx);
  lam = (pg > 0.0) ? std::min(kLMax, std::max(kLMin, 1.0 / pg)) : 1.0;
  const int M = std::max(1, so.memory);
  while (pg > so.tol) {
    if (it >= so.max_iter) {
      status = CQK_NOT_CONVERGED;
      break;
    }
    // d = P(x - lam g) - x, with g'd and d'd
    hipLaunchKernelGGL(spg_vec_kernel<OP_STEP>, dim3(W.gvec), dim3(kBlock), 0, s, n, lam, x, W.g,
                       W.z, W.partials, clock100);
    e = project(W.z, W.d);
    if (e != CQK_OK) return e;
    hipLaunchKernelGGL(spg_vec_kernel<OP_DIR>, dim3(W.gvec), dim3(kBlock), 0, s, n, 0.0, x, W.g,
                       W.d, W.partials, clock100);
    reduce(hdir);
    // Ad and ||Ad||^2
    gemv_n(W.d, nullptr, W.Ad);
    hipLaunchKernelGGL(spg_vec_kernel<OP_DOT>, dim3(W.gvec), dim3(kBlock), 0, s, m, 0.0, W.Ad,
                       W.Ad, nullptr, W.partials, nullptr);
    reduce(had);
    if ((e = wait()) != CQK_OK) return e;
    projected();
    const double gtd = hdir[0], dd = hdir[1], c2 = had[1];
    // non-monotone line search on f(x + t d) = f + t gtd + t^2/2 c2
    const size_t h0 = (hist.size() > (size_t)M) ? hist.size() - M : 0;
    const double fmax = *std::max_element(hist.begin() + h0, hist.end());
    double t = 1.0, fn = 0.0;
    for (int ls = 0; ls < 200; ++ls) {
      fn = fx + t * gtd + 0.5 * t * t * c2;
      if (fn <= fmax + kGamma * t * gtd) break;
      const double tq = -0.5 * t * t * gtd / (fn - fx - t * gtd);
      t = (tq >= kSigma1 && tq <= kSigma2 * t) ? tq : 0.5 * t;
    }
    // x += t d, r += t Ad, f = 1/2 ||r||^2, g = A^T r
    hipLaunchKernelGGL(spg_move_kernel, dim3(W.gvec), dim3(kBlock), 0, s, n, m, t, W.d, x, W.Ad,
                       W.r, W.partials);
    reduce(hr);
    gemv_t(W.r, W.g);
    // spectral step: s's / s'y = d'd / ||Ad||^2
    lam = (c2 <= 0.0) ? kLMax : std::min(kLMax, std::max(kLMin, dd / c2));
    it += 1;
    if ((e = proj_grad()) != CQK_OK) return e;
    hist.push_back(fx);
  }
  if (info) {
    std::memset(info, 0, sizeof(*info));
    info->status = status;
    info->iterations = it;
    info->projections = nproj;
    info->newton_iterations = newton;
    info->objective = fx;
    info->pg = pg;
    info->proj_ms = proj_ms;
    info->total_ms = std::chrono::duration<double, std::milli>(clock::now() - t_start).count();
  }
  return CQK_OK;
}

}  // namespace cqk
