// Exact pairwise sums at chosen targets: the direct summation of Eq. (1)
// with the kernels of Eq. (2) that the FMM approximates, for checking an FMM
// result against it at a sample of particles.
//
//   phi_k = sum_{j: r > 0} q_j / r^p,   F_k = q_i sum_{j: r > 0} q_j p (x_i - x_j) / r^(p+2)
//
// with i = targets[k], r = |x_i - x_j| and p = 1 (1/r) or 2 (1/r^2).
//
// Layout of the work: the sources are cut into S equal chunks; workgroup
// (g, c) takes targets 64 g .. 64 g + 63 (one per lane) against chunk c, each
// of its four wavefronts a quarter of the chunk's sources, and writes the
// chunk's four partial sums per target to a scratch buffer [S][nt64][4].  A
// second kernel adds the S partials of each target, one wavefront per
// target.  The split depends only on (n, nt), so the summation order and the
// bits are the same on every call.
//
// The FP64 vector units bound it: 18 instructions and one v_rsq_f64 a pair.
// A source is the same for a whole wavefront, so it is read through the
// scalar cache into scalar registers, with no LDS staging and no barriers;
// 1/r and 1/r^2 come from the hardware's approximation and one third-order
// step instead of a divide and a square root (1M sources, 1024 targets:
// 2253 -> 710 us; the loads not
// pipelined and half the workgroups: 908 us).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>

#include "device_util.h"
#include "fmm_internal.h"

namespace fmm {
namespace {

constexpr int kDirTargets = 64;    // targets per workgroup, one per lane
constexpr int kDirThreads = 256;   // four wavefronts share a chunk
constexpr int kDirBlock = 64;      // sources between two checks of the sums
constexpr int kDirGroup = 4;       // sources loaded at once
constexpr int64_t kDirMinChunk = 1024;  // sources per chunk at least
constexpr int64_t kDirGroups = 2048;    // workgroups wanted: eight wavefronts a SIMD
constexpr int kDirMaxChunks = 1024;

__host__ __device__ inline int64_t pad64(int64_t nt) {
  return (nt + kDirTargets - 1) / kDirTargets * kDirTargets;
}

struct Sums {
  double ph, fx, fy, fz;
};

// One pair, x - x_j = (dx, dy, dz) at squared distance r2 > 0.
// v_rsq_f64 and v_rcp_f64 are good to about 2^-24; one third-order step
// (Halley's iteration for the root, the cubic Neumann sum for the
// reciprocal) leaves an error below 2^-70 before rounding.  Where r2 or 1/r2
// overflows the sums are not finite, and SAFE takes division and root instead
// (an infinite 1/r^2 of a very close pair, zeros at an infinite distance, NaN in
// the direction of an infinite difference).
template <int P, bool SAFE>
__device__ __forceinline__ void add_pair(double dx, double dy, double dz, double r2, double q,
                                         Sums& a) {
  double pot, g;
  if (SAFE) {
    const double ir2 = 1.0 / r2;
    pot = P == 2 ? q * ir2 : q * (1.0 / sqrt(r2));
    g = (P == 2 ? 2.0 * pot : pot) * ir2;
  } else if (P == 2) {
    const double y = __builtin_amdgcn_rcp(r2);
    const double e = fma(-r2, y, 1.0);
    const double ir2 = fma(y, fma(e, e, e), y);
    pot = q * ir2;
    g = 2.0 * pot * ir2;
  } else {
    const double y = __builtin_amdgcn_rsq(r2);
    const double e = fma(-(r2 * y), y, 1.0);
    const double ir = fma(y * e, fma(e, 0.375, 0.5), y);
    pot = q * ir;
    g = pot * (ir * ir);
  }
  a.ph += pot;
  a.fx = fma(g, dx, a.fx);
  a.fy = fma(g, dy, a.fy);
  a.fz = fma(g, dz, a.fz);
}

// kDirGroup sources, the same in every lane (scalar registers).
struct Sources {
  double p[3 * kDirGroup], q[kDirGroup];
};

__device__ __forceinline__ Sources load_sources(const double* __restrict__ pos,
                                                const double* __restrict__ q, int64_t j) {
  Sources s;
#pragma unroll
  for (int e = 0; e < 3 * kDirGroup; ++e) s.p[e] = pos[3 * j + e];
#pragma unroll
  for (int e = 0; e < kDirGroup; ++e) s.q[e] = q[j + e];
  return s;
}

// Whether a lane's sums hold a NaN or an infinity (the same in every lane).
__device__ __forceinline__ bool not_finite(const Sums& a) {
  const double v = (a.ph + a.fx) + (a.fy + a.fz);
  return __any(!(fabs(v) < INFINITY));
}

__device__ __forceinline__ void add_sums(Sums& a, const Sums& b) {
  a.ph += b.ph;
  a.fx += b.fx;
  a.fy += b.fy;
  a.fz += b.fz;
}

// Sums over sources j0 .. j0 + cnt - 1 but for pairs at zero or NaN distance.
template <int P, bool SAFE>
__device__ __forceinline__ Sums sum_pairs(const double* __restrict__ pos,
                                          const double* __restrict__ q, int64_t j0, int cnt,
                                          double xi, double yi, double zi) {
  Sums a = {0.0, 0.0, 0.0, 0.0};
  for (int e = 0; e < cnt; ++e) {
    const int64_t j = j0 + e;
    const double dx = xi - pos[3 * j], dy = yi - pos[3 * j + 1], dz = zi - pos[3 * j + 2];
    const double r2 = (dx * dx + dy * dy) + dz * dz;
    if (r2 > 0.0) add_pair<P, SAFE>(dx, dy, dz, r2, q[j], a);
  }
  return a;
}

template <int P>
__device__ __forceinline__ Sums sum_checked(const double* __restrict__ pos,
                                            const double* __restrict__ q, int64_t j0, int cnt,
                                            double xi, double yi, double zi) {
  Sums a = sum_pairs<P, false>(pos, q, j0, cnt, xi, yi, zi);
  if (not_finite(a)) a = sum_pairs<P, true>(pos, q, j0, cnt, xi, yi, zi);
  return a;
}

template <int P>
__device__ __forceinline__ Sums sum_range(const double* __restrict__ pos,
                                          const double* __restrict__ q, int64_t j0, int64_t j1,
                                          double xi, double yi, double zi) {
  Sums a = {0.0, 0.0, 0.0, 0.0};
  int64_t b = j0;
  if (j1 - j0 >= kDirBlock) {
    Sources cur = load_sources(pos, q, j0);
    for (; b + kDirBlock <= j1; b += kDirBlock) {
      // a block's sums start from zero: one that is not finite tells of this
      // block's pairs alone
      Sums s = {0.0, 0.0, 0.0, 0.0};
      for (int e = 0; e < kDirBlock; e += kDirGroup) {
        // the next group's loads are in flight while this one is computed
        // (past the range's end: its last group again, not used).  Scalar
        // loads complete out of order, so a wait is for all of them: the
        // current group's has to come before the next one's loads
        const int64_t jn = b + e + kDirGroup;
#pragma unroll
        for (int u = 0; u < kDirGroup; ++u) asm volatile("" ::"s"(cur.p[3 * u]), "s"(cur.q[u]));
        __builtin_amdgcn_sched_barrier(0);
        const Sources next = load_sources(pos, q, jn < j1 - kDirGroup ? jn : j1 - kDirGroup);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kDirGroup; ++u) {
          const double dx = xi - cur.p[3 * u], dy = yi - cur.p[3 * u + 1],
                       dz = zi - cur.p[3 * u + 2];
          add_pair<P, false>(dx, dy, dz, (dx * dx + dy * dy) + dz * dz, cur.q[u], s);
        }
        cur = next;
      }
      // a pair at zero, NaN, infinite or vanishing distance left a NaN or an
      // infinity (the target itself does, once): that block again, with the
      // checks
      if (not_finite(s)) s = sum_checked<P>(pos, q, b, kDirBlock, xi, yi, zi);
      add_sums(a, s);
    }
  }
  add_sums(a, sum_checked<P>(pos, q, b, int(j1 - b), xi, yi, zi));
  return a;
}

__global__ __launch_bounds__(kDirThreads) void direct_partial_kernel(
    const double* __restrict__ pos, const double* __restrict__ q, int64_t n,
    const int64_t* __restrict__ targets, int64_t nt, int p, int chunks,
    double* __restrict__ part) {
  __shared__ double red[4][kDirTargets][4];
  const int lane = threadIdx.x & 63, w = wuni(int(threadIdx.x >> 6));
  const int64_t k = int64_t(blockIdx.x) * kDirTargets + lane;
  const int c = blockIdx.y;
  int64_t i = k < nt ? targets[k] : 0;
  const bool valid = k < nt && i >= 0 && i < n;
  if (!valid) i = 0;
  const double xi = pos[3 * i], yi = pos[3 * i + 1], zi = pos[3 * i + 2];
  // quarter w of the chunk
  const int64_t c0 = n * c / chunks, c1 = n * (c + 1) / chunks;
  const int64_t j0 = c0 + (c1 - c0) * w / 4, j1 = c0 + (c1 - c0) * (w + 1) / 4;
  const Sums a = p == 2 ? sum_range<2>(pos, q, j0, j1, xi, yi, zi)
                        : sum_range<1>(pos, q, j0, j1, xi, yi, zi);
  // the four wavefronts' sums, added in wavefront order
  red[w][lane][0] = a.ph;
  red[w][lane][1] = a.fx;
  red[w][lane][2] = a.fy;
  red[w][lane][3] = a.fz;
  __syncthreads();
  if (w == 0) {
    double acc[4];
    for (int v = 0; v < 4; ++v) acc[v] = red[0][lane][v];
    for (int u = 1; u < 4; ++u)
      for (int v = 0; v < 4; ++v) acc[v] += red[u][lane][v];
    double* out = part + ((int64_t(c) * pad64(nt)) + k) * 4;
    for (int v = 0; v < 4; ++v) out[v] = valid ? acc[v] : NAN;
  }
}

// One wavefront per target: lane l adds the partial sums of chunks l, l + 64,
// ..., then a butterfly over the lanes.
__global__ __launch_bounds__(256) void direct_sum_kernel(
    const double* __restrict__ q, int64_t n, const int64_t* __restrict__ targets, int64_t nt,
    int chunks, const double* __restrict__ part, double* __restrict__ phi,
    double* __restrict__ f) {
  const int lane = threadIdx.x & 63;
  const int64_t k = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (k >= nt) return;
  const int64_t stride = pad64(nt) * 4;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int c = lane; c < chunks; c += 64)
    for (int v = 0; v < 4; ++v) acc[v] += part[c * stride + 4 * k + v];
  for (int o = 32; o > 0; o >>= 1)
    for (int v = 0; v < 4; ++v) acc[v] += __shfl_xor(acc[v], o, 64);
  if (lane > 0) return;
  const int64_t i = targets[k];
  const double qi = (i >= 0 && i < n) ? q[i] : NAN;
  phi[k] = acc[0];
  f[3 * k] = qi * acc[1];
  f[3 * k + 1] = qi * acc[2];
  f[3 * k + 2] = qi * acc[3];
}

int fail(int code, const std::string& msg) {
  set_error(msg);
  return code;
}

template <typename F>
int guarded(F&& fn) {
  try {
    return fn();
  } catch (const FmmError& e) {
    return fail(e.code, e.msg);
  } catch (const std::exception& e) {
    return fail(FMM_ERR_HIP, e.what());
  }
}

}  // namespace

// Source chunks for n sources and nt targets: enough workgroups for eight
// wavefronts on every SIMD, chunks of at least 1024 sources (256 to a
// wavefront), and few enough that the partial sums stay within
// kDirectPartialMax values.
int direct_chunks(int64_t n, int64_t nt) {
  const int64_t groups = pad64(nt) / kDirTargets;
  int64_t s = (kDirGroups + groups - 1) / groups;
  s = std::min<int64_t>(s, (n + kDirMinChunk - 1) / kDirMinChunk);
  s = std::min<int64_t>(s, kDirMaxChunks);
  s = std::min<int64_t>(s, kDirectPartialMax / (4 * pad64(nt)));
  return int(std::max<int64_t>(s, 1));
}

size_t direct_partial_doubles(int64_t nt, int chunks) { return size_t(4) * chunks * pad64(nt); }

void launch_direct(const double* pos, const double* q, int64_t n, const int64_t* targets,
                   int64_t nt, int p, double* phi, double* f, double* part, int chunks,
                   hipStream_t s) {
  const dim3 grid(unsigned(pad64(nt) / kDirTargets), unsigned(chunks));
  direct_partial_kernel<<<grid, kDirThreads, 0, s>>>(pos, q, n, targets, nt, p, chunks, part);
  FMM_HIP_CHECK(hipGetLastError());
  direct_sum_kernel<<<unsigned((nt + 3) / 4), 256, 0, s>>>(q, n, targets, nt, chunks, part,
                                                              phi, f);
  FMM_HIP_CHECK(hipGetLastError());
}

int direct_check_args(const double* pos, const double* q, int64_t n, const int64_t* targets,
                      int64_t nt, int kernel, const double* phi, const double* f) {
  if (!pos || !q || !targets || !phi || !f) return fail(FMM_ERR_ARG, "NULL pointer argument");
  if (n < 1 || n > int64_t(2147483646)) return fail(FMM_ERR_ARG, "n outside 1 .. 2^31-2");
  if (nt < 1 || nt > int64_t(1) << 30) return fail(FMM_ERR_ARG, "nt outside 1 .. 2^30");
  if (kernel != FMM_KERNEL_INV_R && kernel != FMM_KERNEL_INV_R2)
    return fail(FMM_ERR_ARG, "unknown kernel " + std::to_string(kernel));
  return FMM_OK;
}

}  // namespace fmm

extern "C" int fmm_direct_sampled(const double* positions, const double* charges, int64_t n,
                                  const int64_t* targets, int64_t nt, int kernel,
                                  double* potential, double* forces, hipStream_t stream) {
  using namespace fmm;
  const int rc = direct_check_args(positions, charges, n, targets, nt, kernel, potential, forces);
  if (rc != FMM_OK) return rc;
  return guarded([&]() -> int {
    const int chunks = direct_chunks(n, nt);
    const size_t bytes = sizeof(double) * direct_partial_doubles(nt, chunks);
    double* part = static_cast<double*>(dev_alloc(bytes));
    try {
      launch_direct(positions, charges, n, targets, nt, kernel, potential, forces, part, chunks,
                    stream);
      FMM_HIP_CHECK(hipStreamSynchronize(stream));
    } catch (...) {
      (void)hipStreamSynchronize(stream);
      dev_free(part);
      throw;
    }
    dev_free(part);
    return FMM_OK;
  });
}
