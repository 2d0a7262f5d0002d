// Operator tables and the M2L kernel.
//
// M2L (Sec. 2.1.2, Eq. 3): for a target cell C and a far source cell B at
// level l, with centres differing by w_l t (t in [-3,3]^3, |t|_inf >= 2), the
// local expansion gains K_{l,t} W_B where
//     K_{l,t}[m][n] = 1 / |x_m - y_n| = 1 / |a_l (xb_m - xb_n - 2t)|,
// a_l = L / 2^(l+1) the half-width.  1/r is homogeneous, so every level uses
// the unit operators Kh_t[m][n] = 1 / |xb_m - xb_n - 2t| and one scalar
// 1/a_l per level (Sec. 2.1.2: the 316 operators are computed once).
// The 316 unit operators are signed permutations of 16 canonical ones
// (Sec. 2.1.2): with t = G tc, (G v)_d = s_d v_{pi(d)},
//     Kh_t[m][n] = Kh_tc[g(m)][g(n)],  g(m)_{pi(d)} = s_d > 0 ? m_d : l-1-m_d,
// because the mirrored Chebyshev nodes satisfy xb_{l-1-k} = -xb_k.
//
// FP32 operators (mixed modes) have their rows in the Chebyshev-coefficient
// basis instead of node values: Kh'_t = T3 Kh_t with T3 = T1 (x) T1 (x) T1,
// T1[n][m] = C[m][n] = (n == 0 ? 1 : 2 T_n(xb_m)) / l, which maps the values
// of a degree < l polynomial at the nodes to its Chebyshev coefficients
// (Eq. 5).  A local expansion then accumulates in FP32 as coefficients,
// whose magnitudes fall with the degree like those of the smooth far field
// they describe, so each rounding error is relative to its own coefficient;
// summed as node values, the rounding errors are alike at every node and the
// force, the gradient of the interpolant (L2P), multiplies their
// high-degree part by up to l^2.  The downward pass keeps the coefficients.
// Mirroring a dimension maps T_n to (-1)^n T_n, so the signed permutations
// act on coefficient rows as permutations with the sign (-1)^(sum of the
// mirrored dimensions' degrees).
//
// The contraction is organised target-stationary: a work tile holds 64
// target cells of one level and one child parity, which share the same 189
// offsets; for each offset the tile computes Y(l^3 x 64) += Kh_t (l^3 x l^3)
// X(l^3 x 64) on MFMA, X the gathered source multipoles, and writes its local
// expansions once (no atomics, deterministic).
#include <hip/hip_runtime.h>
#include <rocsolver/rocsolver.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <map>
#include <memory>
#include <mutex>
#include <tuple>
#include <vector>

#include "device_util.h"
#include "fmm_internal.h"
#include "jobs.h"
#include "m2l_dev.h"

namespace fmm {

thread_local hipEvent_t g_time_ev[kTimedSteps][2] = {{nullptr, nullptr}};

// ------------------------------------------------------------ tables
namespace {

struct OffsetInfo {
  int t[3];
  int canon;   // index into the 16 canonical offsets
  int pi[3];   // t_d = s_d * tc[pi[d]]
  int sg[3];
};

struct StaticTables {
  std::vector<OffsetInfo> offs;        // the 316 far offsets (packed order)
  std::vector<std::array<int, 3>> canon;  // 16 canonical offsets, tc0 >= tc1 >= tc2 >= 0
  int id_to_kid[343];
  std::vector<int> slot_kid;           // [8][189]
  std::vector<signed char> slot_t;     // [8][189][3]
};

const StaticTables& tables() {
  static StaticTables T = [] {
    StaticTables S;
    for (int i = 0; i < 343; ++i) S.id_to_kid[i] = -1;
    std::map<std::array<int, 3>, int> cidx;
    for (int tx = -3; tx <= 3; ++tx)
      for (int ty = -3; ty <= 3; ++ty)
        for (int tz = -3; tz <= 3; ++tz) {
          const int t[3] = {tx, ty, tz};
          int mx = 0;
          for (int d = 0; d < 3; ++d) mx = std::max(mx, std::abs(t[d]));
          if (mx < 2) continue;
          OffsetInfo o;
          int ord[3] = {0, 1, 2};
          std::stable_sort(ord, ord + 3, [&](int a, int b) { return std::abs(t[a]) > std::abs(t[b]); });
          std::array<int, 3> tc;
          for (int j = 0; j < 3; ++j) {
            tc[j] = std::abs(t[ord[j]]);
            o.pi[ord[j]] = j;
          }
          for (int d = 0; d < 3; ++d) {
            o.t[d] = t[d];
            o.sg[d] = t[d] < 0 ? -1 : 1;
          }
          auto it = cidx.find(tc);
          if (it == cidx.end()) {
            it = cidx.emplace(tc, int(S.canon.size())).first;
            S.canon.push_back(tc);
          }
          o.canon = it->second;
          S.id_to_kid[(tx + 3) * 49 + (ty + 3) * 7 + (tz + 3)] = int(S.offs.size());
          S.offs.push_back(o);
        }
    // per child parity p (bit d = parity of the cell coordinate along d):
    // offsets with t_d in [-2-p_d, 3-p_d], in the order the M2L kernels take
    // them: z outermost, x innermost, each axis in steps of two cells (-3,
    // -1, 1, 3, 2, 0, -2) and rows in alternate directions.  The targets of
    // a work item are same-parity cells two apart (4 x 4 x 2 of them), so an
    // offset two cells from the last one reads mostly the same source
    // multipoles, which are then still in L2 (30M-particle order-10 cube:
    // M2L 4327 -> 4222 ms against the lexicographic order)
    static const int zig[7] = {-3, -1, 1, 3, 2, 0, -2};
    for (int p = 0; p < 8; ++p) {
      int cnt = 0;
      for (int i0 = 0; i0 < 7; ++i0)
        for (int i1 = 0; i1 < 7; ++i1)
          for (int i2 = 0; i2 < 7; ++i2) {
            const int tz = zig[i0], ty = zig[i0 % 2 ? 6 - i1 : i1];
            const int tx = zig[(i0 * 7 + i1) % 2 ? 6 - i2 : i2];
            const int t[3] = {tx, ty, tz};
            bool ok = std::max({std::abs(tx), std::abs(ty), std::abs(tz)}) >= 2;
            for (int d = 0; d < 3; ++d) {
              const int pd = (p >> d) & 1;
              ok = ok && t[d] >= -2 - pd && t[d] <= 3 - pd;
            }
            if (!ok) continue;
            S.slot_kid.push_back(S.id_to_kid[(tx + 3) * 49 + (ty + 3) * 7 + (tz + 3)]);
            for (int d = 0; d < 3; ++d) S.slot_t.push_back((signed char)t[d]);
            ++cnt;
          }
      if (cnt != kSlots) throw FmmError{FMM_ERR_HIP, "internal: parity offset count"};
    }
    if (int(S.offs.size()) != kOffsets || S.canon.size() != 16)
      throw FmmError{FMM_ERR_HIP, "internal: offset tables"};
    return S;
  }();
  return T;
}

// Chebyshev roots of T_l, mirrored exactly (xb_{l-1-k} = -xb_k, 0 in the
// middle for odd l).
void cheb_nodes(int l, double* xi) {
  for (int m = 0; m < l; ++m) xi[m] = std::cos((2.0 * m + 1.0) * M_PI / (2.0 * l));
  for (int m = 0; m < l / 2; ++m) xi[l - 1 - m] = -xi[m];
  if (l & 1) xi[l / 2] = 0.0;
}

void cheb_T(int l, double x, double* T) {
  T[0] = 1.0;
  if (l > 1) T[1] = x;
  for (int n = 2; n < l; ++n) T[n] = 2.0 * x * T[n - 1] - T[n - 2];
}

// Canonical unit operators: Kc[c][m][n] = |xb_m - xb_n - 2 tc|^-p for the
// kernel |x - y|^-p (p = 1 or 2)
__global__ void canon_kernel(const double* __restrict__ xi, const int* __restrict__ tc,
                             int l, int ncanon, int p, double* __restrict__ Kc) {
  const int l3 = l * l * l;
  const int64_t total = int64_t(ncanon) * l3 * l3;
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int c = int(e / (int64_t(l3) * l3));
    const int r = int(e % (int64_t(l3) * l3));
    const int m = r / l3, n = r % l3;
    const int m1 = m / (l * l), m2 = (m / l) % l, m3 = m % l;
    const int n1 = n / (l * l), n2 = (n / l) % l, n3 = n % l;
    const double dx = xi[m1] - xi[n1] - 2.0 * tc[3 * c];
    const double dy = xi[m2] - xi[n2] - 2.0 * tc[3 * c + 1];
    const double dz = xi[m3] - xi[n3] - 2.0 * tc[3 * c + 2];
    const double r2 = dx * dx + dy * dy + dz * dz;
    Kc[e] = p == 2 ? 1.0 / r2 : 1.0 / sqrt(r2);
  }
}

// Rows to Chebyshev coefficients:
//   out[c][u][col] = sum_a T3[u][a] in[c][a][col],  T3[u][a] = prod_d C[a_d][u_d]
// for nmat row-major l^3 x ncol matrices (a and u are node and degree triples).
__global__ void modal_rows_kernel(const double* __restrict__ in, const double* __restrict__ cheb,
                                  int l, int ncol, int nmat, double* __restrict__ out) {
  const int l3 = l * l * l;
  const int64_t total = int64_t(nmat) * l3 * ncol;
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int col = int(e % ncol);
    const int64_t r = e / ncol;
    const int u = int(r % l3), c = int(r / l3);
    const int u1 = u / (l * l), u2 = (u / l) % l, u3 = u % l;
    const double* src = in + int64_t(c) * l3 * ncol + col;
    double v = 0.0;
    for (int a1 = 0; a1 < l; ++a1) {
      const double c1 = cheb[a1 * l + u1];
      for (int a2 = 0; a2 < l; ++a2) {
        const double c12 = c1 * cheb[a2 * l + u2];
        const double* s3 = src + int64_t((a1 * l + a2) * l) * ncol;
        for (int a3 = 0; a3 < l; ++a3) v += c12 * cheb[a3 * l + u3] * s3[int64_t(a3) * ncol];
      }
    }
    out[e] = v;
  }
}

// Row index and sign of a coefficient row u of offset kid in its canonical
// class's coefficient rows: the dimension permutation without the mirroring,
// which flips the sign of odd degrees.
__device__ inline int modal_row(const int* in, int l, int u, double& sgn) {
  const int uu[3] = {u / (l * l), (u / l) % l, u % l};
  int gu[3];
  sgn = 1.0;
  for (int d = 0; d < 3; ++d) {
    gu[in[1 + d]] = uu[d];
    if (in[4 + d] < 0 && (uu[d] & 1)) sgn = -sgn;
  }
  return (gu[0] * l + gu[1]) * l + gu[2];
}

// Pack the 316 operators in MFMA fragment order:
//   kp[((kid*mt + i)*kc + c)*256 + lane*4 + s] = Kh_t[16 i + lane%16][16 c + 4 (lane/16) + s]
// (zero outside l^3), gathering from the canonical operator through g; the
// FP32 pack from the coefficient rows KcM = T3 Kc through modal_row.
__global__ void pack_kernel(const double* __restrict__ Kc, const double* __restrict__ KcM,
                            const int* __restrict__ info, int l, int mt, int kc,
                            double* __restrict__ kp64, float* __restrict__ kp32) {
  const int l3 = l * l * l;
  const int64_t total = int64_t(kOffsets) * mt * kc * 256;
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int s = int(e & 3), lane = int((e >> 2) & 63);
    int64_t r = e >> 8;
    const int c = int(r % kc);
    r /= kc;
    const int i = int(r % mt);
    const int kid = int(r / mt);
    const int row = 16 * i + (lane & 15);
    const int col = 16 * c + 4 * (lane >> 4) + s;
    double v = 0.0, vm = 0.0;
    if (row < l3 && col < l3) {
      const int* in = info + 7 * kid;  // canon, pi[3], sg[3]
      int mm[3] = {row / (l * l), (row / l) % l, row % l};
      int nn[3] = {col / (l * l), (col / l) % l, col % l};
      int gm[3], gn[3];
      for (int d = 0; d < 3; ++d) {
        gm[in[1 + d]] = in[4 + d] > 0 ? mm[d] : l - 1 - mm[d];
        gn[in[1 + d]] = in[4 + d] > 0 ? nn[d] : l - 1 - nn[d];
      }
      const int gmi = (gm[0] * l + gm[1]) * l + gm[2];
      const int gni = (gn[0] * l + gn[1]) * l + gn[2];
      v = Kc[(int64_t(in[0]) * l3 + gmi) * l3 + gni];
      double sgn;
      const int gu = modal_row(in, l, row, sgn);
      vm = sgn * KcM[(int64_t(in[0]) * l3 + gu) * l3 + gni];
    }
    kp64[e] = v;
    kp32[e] = float(vm);
  }
}

std::mutex g_ops_mu;
// (device, order, kernel exponent)
std::map<std::tuple<int, int, int>, std::unique_ptr<OpSet>> g_ops;

}  // namespace

const OpSet* get_opset(int l, int kernel, hipStream_t s) {
  int dev = 0;
  FMM_HIP_CHECK(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_ops_mu);
  auto it = g_ops.find(std::make_tuple(dev, l, kernel));
  if (it != g_ops.end()) return it->second.get();
  const StaticTables& T = tables();
  auto op = std::make_unique<OpSet>();
  op->order = l;
  op->l3 = l * l * l;
  op->mt = (op->l3 + 15) / 16;
  op->kc = op->mt;
  op->ld = 16 * op->mt;

  double xi[kMaxOrder], Tm[kMaxOrder];
  cheb_nodes(l, xi);
  std::vector<double> cheb(l * l), child(2 * l * l), child_modal(2 * l * l, 0.0);
  for (int m = 0; m < l; ++m) {
    cheb_T(l, xi[m], Tm);
    for (int n = 0; n < l; ++n) {
      cheb[m * l + n] = (n == 0 ? 1.0 : 2.0 * Tm[n]) / l;
    }
  }
  // child-to-parent interpolation S(xb_m; (sigma + xb_m')/2), sigma = -1, +1
  for (int sg = 0; sg < 2; ++sg)
    for (int mp = 0; mp < l; ++mp) {
      double Tu[kMaxOrder];
      cheb_T(l, ((sg ? 1.0 : -1.0) + xi[mp]) / 2.0, Tu);
      for (int m = 0; m < l; ++m) {
        double v = 0.0;
        for (int n = 0; n < l; ++n) v += cheb[m * l + n] * Tu[n];
        child[(sg * l + m) * l + mp] = v;
      }
    }
  // the same re-expansion on Chebyshev coefficients: T_k((sigma + x)/2) is a
  // polynomial of degree k < l, so its coefficients are its values at the l
  // nodes transformed with C (exact): R[n][k] = sum_m C[m][n] T_k((sigma + xb_m)/2)
  for (int sg = 0; sg < 2; ++sg)
    for (int m = 0; m < l; ++m) {
      double Tu[kMaxOrder];
      cheb_T(l, ((sg ? 1.0 : -1.0) + xi[m]) / 2.0, Tu);
      for (int n = 0; n < l; ++n)
        for (int k = 0; k < l; ++k) child_modal[(sg * l + n) * l + k] += cheb[m * l + n] * Tu[k];
    }

  std::vector<int> tc(3 * 16), info(7 * kOffsets);
  for (int c = 0; c < 16; ++c)
    for (int d = 0; d < 3; ++d) tc[3 * c + d] = T.canon[c][d];
  for (int k = 0; k < kOffsets; ++k) {
    const OffsetInfo& o = T.offs[k];
    info[7 * k] = o.canon;
    for (int d = 0; d < 3; ++d) {
      info[7 * k + 1 + d] = o.pi[d];
      info[7 * k + 4 + d] = o.sg[d];
    }
  }

  std::vector<void*> tmp;
  auto up = [&](const void* h, size_t b, bool keep) {
    void* d = dev_alloc(b);
    if (!keep) tmp.push_back(d);
    FMM_HIP_CHECK(hipMemcpyAsync(d, h, b, hipMemcpyHostToDevice, s));
    return d;
  };
  try {
    op->cheb = static_cast<double*>(up(cheb.data(), sizeof(double) * cheb.size(), true));
    op->child_modal =
        static_cast<double*>(up(child_modal.data(), sizeof(double) * child_modal.size(), true));
    op->child = static_cast<double*>(up(child.data(), sizeof(double) * child.size(), true));
    op->slot_kid = static_cast<int*>(up(T.slot_kid.data(), sizeof(int) * T.slot_kid.size(), true));
    op->slot_t = static_cast<signed char*>(up(T.slot_t.data(), T.slot_t.size(), true));
    double* xi_d = static_cast<double*>(up(xi, sizeof(double) * l, false));
    int* tc_d = static_cast<int*>(up(tc.data(), sizeof(int) * tc.size(), false));
    int* info_d = static_cast<int*>(up(info.data(), sizeof(int) * info.size(), false));
    double* kc_d = static_cast<double*>(dev_alloc(sizeof(double) * 16 * size_t(op->l3) * op->l3));
    tmp.push_back(kc_d);
    double* kcm_d = static_cast<double*>(dev_alloc(sizeof(double) * 16 * size_t(op->l3) * op->l3));
    tmp.push_back(kcm_d);
    const size_t npack = size_t(kOffsets) * op->mt * op->kc * 256;
    op->kpack64 = static_cast<double*>(dev_alloc(sizeof(double) * npack));
    op->kpack32 = static_cast<float*>(dev_alloc(sizeof(float) * npack));
    canon_kernel<<<1024, 256, 0, s>>>(xi_d, tc_d, l, 16, kernel, kc_d);
    FMM_HIP_CHECK(hipGetLastError());
    modal_rows_kernel<<<4096, 256, 0, s>>>(kc_d, op->cheb, l, op->l3, 16, kcm_d);
    FMM_HIP_CHECK(hipGetLastError());
    pack_kernel<<<4096, 256, 0, s>>>(kc_d, kcm_d, info_d, l, op->mt, op->kc, op->kpack64,
                                     op->kpack32);
    FMM_HIP_CHECK(hipGetLastError());
    FMM_HIP_CHECK(hipStreamSynchronize(s));
  } catch (...) {
    (void)hipStreamSynchronize(s);
    for (void* q : tmp) dev_free(q);
    throw;
  }
  for (void* q : tmp) dev_free(q);
  const OpSet* r = op.get();
  g_ops[std::make_tuple(dev, l, kernel)] = std::move(op);
  return r;
}

// ------------------------------------------------------------- M2L kernel
// One workgroup = 4 wavefronts = one (tile, M-block) item.  Wavefront w owns
// the M-tiles [mt0, mt0 + MTW) of the output rows and all 64 target columns
// (four 16-column N-tiles).  K-chunks of 16 coefficients = 4 MFMA k-steps;
// lane group g = lane/16 holds k = 16c + 4g + s at step s, so both operands
// are fetched as 4 consecutive values per lane.  FOLD: FP32 partial sums are
// added into FP64 accumulators after every far offset.
// The matrix cores bound it (70% of their FP64 peak at 1M particles, order
// 7), so what a small plan lacks is items: the job's m2l_parts cuts each
// tile's offsets into ranges, one item each (4,000 particles, height 4,
// order 5: evaluation 2250 -> 210 us; the 1M cube, last round: 38.2 -> 34.3
// ms).  GS: 16-target groups without a source at an offset are skipped (the
// last tiles of a parity, the coarse levels, points on surfaces), for plans
// with many (dense_gskip); otherwise a K-step takes all accumulators in turn.
// Only the form for items of several ranges loops over them: the loop costs
// small items 2% (60,000 particles, height 5, order 4 mixed: 224 and 228 us).
// Build-time tuning of the dense kernel: wavefronts per SIMD the register
// allocation must allow, and whether FP64 double-buffers the B fragments.
#ifndef FMM_M2L_WAVES_PER_SIMD
#define FMM_M2L_WAVES_PER_SIMD 2
#endif
#ifndef FMM_M2L_F64_PREFETCH_B
#define FMM_M2L_F64_PREFETCH_B 1
#endif

// A product rounded before it is added: a range's sum adds up to the same bits
// from LocX (loc_sum_kernel) and from the accumulators.
__device__ __forceinline__ double scaled(double sc, double v) {
#pragma clang fp contract(off)
  return sc * v;
}

template <typename T, int MTW, bool FOLD, int FORM>
__global__ __launch_bounds__(256, FMM_M2L_WAVES_PER_SIMD) void m2l_kernel(
    const JobDev* __restrict__ jobs, const StepTab* __restrict__ tab) {
  typedef typename Vec4<T>::type T4;
  constexpr bool GS = FORM != kM2LFull;
  const int total = step_total(*tab);
  const int wave = wuni(int(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int g = lane >> 4, c16 = lane & 15;
  for (int it = blockIdx.x; it < total; it += gridDim.x) {
    // Items of a job: the leaf level's tiles, then the coarser ones (fewer
    // targets a tile, hence shorter); within each, offset ranges (parts)
    // outermost, so that consecutive items take the same operators.  With one
    // block per item, blocks are dealt round-robin to the 8 XCDs: each XCD
    // gets a contiguous run of either kind, whose tiles share operators and
    // source multipoles in its L2, and every CU starts on a long item
    // (4,000 particles, height 4, order 5: evaluation 209 -> 170 us)
    int b = it;
    if (int(gridDim.x) == total && tab->njobs == 1) {
      const JobDev& J0 = jobs[tab->job[0]];
      const int lo = min(max(J0.leaf_tiles * J0.nmb * J0.m2l_parts - tab->first[0], 0), total);
      b = b < lo ? xcd_run(b, lo) : lo + xcd_run(b - lo, total - lo);
    }
    const int k = step_find(*tab, b);
    const JobDev& J = jobs[tab->job[k]];
    const int parts = J.m2l_parts;
    int rel = b - tab->start[k] + tab->first[k], tile0 = 0, ntile = J.leaf_tiles;
    if (rel >= J.leaf_tiles * J.nmb * parts) {
      rel -= J.leaf_tiles * J.nmb * parts;
      tile0 = J.leaf_tiles;
      ntile = J.ntiles - J.leaf_tiles;
    }
    const int part = rel / (ntile * J.nmb);
    const int local = rel % (ntile * J.nmb);
    const int tile = tile0 + local / J.nmb, mb = local % J.nmb;
    const int MT = J.mt, KC = J.kc, ld = J.ld;
    const int mt0 = (mb * 4 + wave) * MTW;
    if (mt0 >= MT) continue;
    const int nmt = min(MTW, MT - mt0);
    const M2LTile tl = J.tiles[tile];
    const T* __restrict__ Wp = FOLD ? reinterpret_cast<const T*>(J.W32)
                                    : reinterpret_cast<const T*>(J.W);
    const T* __restrict__ Kp = FOLD ? reinterpret_cast<const T*>(J.kp32)
                                    : reinterpret_cast<const T*>(J.kp64);

    const int nact = wuni(gld(J.tile_nact + tile));
    const unsigned char* act = J.tile_act + int64_t(tile) * kSlots;
    const unsigned char* gmask = J.tile_gmask + int64_t(tile) * kSlots;
    const int* srcb = J.tile_src + int64_t(tile) * kSlots * kTileN;
    const int* kidp = J.slot_kid + tl.parity * kSlots;
    // the item's ranges: one, or every range of the tile in turn
    const int ranges = J.m2l_ranges;
    const int rg1 = FORM == kM2LRanges && parts == 1 ? ranges : part + 1;
    for (int rg = part; rg < rg1; ++rg) {
      const int ia0 = rg * nact / ranges, ia1 = (rg + 1) * nact / ranges;
      const bool first = FORM != kM2LRanges || rg == part;
      T4 acc[MTW][4];
      d4 acc64[FOLD ? MTW : 1][4];
      for (int i = 0; i < MTW; ++i)
        for (int j = 0; j < 4; ++j) {
          acc[i][j] = T4{0, 0, 0, 0};
          if (FOLD) acc64[FOLD ? i : 0][j] = d4{0, 0, 0, 0};
        }
      for (int ia = ia0; ia < ia1; ++ia) {
        const int s = wuni(int(gld(act + ia)));
        const int kid = wuni(gld(kidp + s));
        // GS: the 16-target groups with a source at this offset; the others'
        // products are zero (a wavefront-uniform branch per group and chunk)
        const int gm = GS ? wuni(int(gld(gmask + ia))) : 0xf;
        const T* bptr[4];
        for (int j = 0; j < 4; ++j)
          bptr[j] = Wp + int64_t(gld(srcb + s * kTileN + 16 * j + c16)) * ld + 4 * g;
        const T* aptr = Kp + (int64_t(kid) * MT + mt0) * KC * 256 + lane * 4;

        // The A and B fragments are double-buffered one chunk ahead.  In FP64
        // the B buffer costs a few spilled registers at MTW = 3 and still wins
        // (36.8 vs 42.7 ms for the 1M-particle order-7 M2L on gfx950).
        constexpr bool kPrefetchB = sizeof(T) == 4 || FMM_M2L_F64_PREFETCH_B;
        T4 bv[4], av[MTW];
        for (int j = 0; j < 4; ++j) bv[j] = gld(reinterpret_cast<const T4*>(bptr[j]));
        for (int i = 0; i < MTW; ++i)
          av[i] = i < nmt ? gld(reinterpret_cast<const T4*>(aptr + int64_t(i) * KC * 256))
                          : T4{0, 0, 0, 0};
        for (int c = 0; c < KC; ++c) {
          T4 bn[kPrefetchB ? 4 : 1], an[MTW];
          const bool more = c + 1 < KC;
          if (!kPrefetchB && c > 0)
            for (int j = 0; j < 4; ++j) bv[j] = gld(reinterpret_cast<const T4*>(bptr[j] + 16 * c));
          if (more) {
            if (kPrefetchB)
              for (int j = 0; j < 4; ++j)
                bn[kPrefetchB ? j : 0] = gld(reinterpret_cast<const T4*>(bptr[j] + 16 * (c + 1)));
            for (int i = 0; i < MTW; ++i)
              an[i] = i < nmt ? gld(reinterpret_cast<const T4*>(aptr + (int64_t(i) * KC + c + 1) * 256))
                              : T4{0, 0, 0, 0};
          }
          if constexpr (GS) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              if (!((gm >> j) & 1)) continue;
#pragma unroll
              for (int st = 0; st < 4; ++st)
#pragma unroll
                for (int i = 0; i < MTW; ++i)
                  acc[i][j] = mfma16x16x4(av[i][st], bv[j][st], acc[i][j]);
            }
          } else {
#pragma unroll
            for (int st = 0; st < 4; ++st)
#pragma unroll
              for (int i = 0; i < MTW; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                  acc[i][j] = mfma16x16x4(av[i][st], bv[j][st], acc[i][j]);
          }
          if (more) {
            if (kPrefetchB)
              for (int j = 0; j < 4; ++j) bv[j] = bn[kPrefetchB ? j : 0];
            for (int i = 0; i < MTW; ++i) av[i] = an[i];
          }
        }
        if (FOLD) {
          for (int i = 0; i < MTW; ++i)
            for (int j = 0; j < 4; ++j) {
              for (int r = 0; r < 4; ++r) acc64[FOLD ? i : 0][j][r] += double(acc[i][j][r]);
              acc[i][j] = T4{0, 0, 0, 0};
            }
        }
      }

      // D layout of the 16x16 outputs, column c16 in every lane group g: the
      // FP32 instruction holds rows 4g+r in item r, the FP64 one rows 4r+g
      // (both measured on gfx950).
      const double sc = J.scale[tl.level];
      const bool f64 = sizeof(T) == 8;
      for (int j = 0; j < 4; ++j) {
        const int col = 16 * j + c16;
        if (col >= tl.count) continue;
        double* out = m2l_out_row(J, part, gld(J.tgt + tl.first + col));
#pragma unroll
        for (int i = 0; i < MTW; ++i) {
          if (i >= nmt) continue;  // constant trip count keeps acc[] in registers
          const int base = 16 * (mt0 + i);
          if (f64) {
            for (int r = 0; r < 4; ++r) {
              double* const o = out + base + 4 * r + g;
              const double v = scaled(sc, FOLD ? acc64[FOLD ? i : 0][j][r] : double(acc[i][j][r]));
              gst(o, first ? v : gld(o) + v);
            }
          } else {
            d4* const o = reinterpret_cast<d4*>(out + base + 4 * g);
            d4 v;
            for (int r = 0; r < 4; ++r)
              v[r] = scaled(sc, FOLD ? acc64[FOLD ? i : 0][j][r] : double(acc[i][j][r]));
            gst(o, first ? v : gld(o) + v);
          }
        }
      }
    }
  }
}

template <typename T, bool FOLD, int FORM>
static void launch_mtw(int mtw, const JobDev* jobs, const StepTab* tab, int grid, hipStream_t s) {
  switch (mtw) {
    case 1: {
      // up to order 4 the skip costs full tiles nothing (200,000, height 6, mixed:
      // order 3 550 us, and 577 without, order 4 1138 and 1131)
      constexpr int F = FORM == kM2LFull ? kM2LSkip : FORM;
      m2l_kernel<T, 1, FOLD, F><<<grid, 256, 0, s>>>(jobs, tab);
      break;
    }
    case 2: m2l_kernel<T, 2, FOLD, FORM><<<grid, 256, 0, s>>>(jobs, tab); break;
    default: m2l_kernel<T, 3, FOLD, FORM><<<grid, 256, 0, s>>>(jobs, tab); break;
  }
}

// M-tiles per wavefront: fewest idle M-tile slots, then the largest count
// (fewest M-blocks, so the gathered source columns are read fewest times);
// at most 3, which keeps two wavefronts per SIMD without spills.
int m2l_mtw(int mt) {
  int best = 1, best_waste = 1 << 30;
  for (int w = 1; w <= 3; ++w) {
    const int per_block = 4 * w;
    const int nmb = (mt + per_block - 1) / per_block;
    const int waste = nmb * per_block - mt;
    if (waste < best_waste || (waste == best_waste && w > best)) {
      best = w;
      best_waste = waste;
    }
  }
  return best;
}

int m2l_nmb(int mt) {
  const int w = m2l_mtw(mt);
  return (mt + 4 * w - 1) / (4 * w);
}

double m2l_item_flops(int mt) { return 2.0 * kTileN * (64.0 * m2l_mtw(mt)) * (16.0 * mt); }

// Every job in `tab` must have the same order (same packed operator shape).
void launch_m2l_step(int order, bool fp32, const JobDev* jobs, const StepTab* tab, int grid,
                     hipStream_t s, int form) {
  const int l3 = order * order * order;
  const int mtw = m2l_mtw((l3 + 15) / 16);
#define M2L_CALL(F)                                              \
  if (fp32) launch_mtw<float, true, F>(mtw, jobs, tab, grid, s); \
  else launch_mtw<double, false, F>(mtw, jobs, tab, grid, s)
  switch (form) {
    case kM2LFull: M2L_CALL(kM2LFull); break;
    case kM2LSkip: M2L_CALL(kM2LSkip); break;
    default: M2L_CALL(kM2LRanges); break;
  }
#undef M2L_CALL
  FMM_HIP_CHECK(hipGetLastError());
}

// ============================================================ compressed M2L
// Sec. 2.1.2: instead of one large SVD of all 316 operators, each of the 16
// canonical operators Kc gets its own SVD Kc = Uc Sc Vc^T, truncated at
// s_k >= eps s_1.  An offset t = G tc reuses it through the same signed
// permutation g as the dense operators:
//     Kh_t[m][n] ~ sum_k Uc[g(m)][k] s_k Vc[g(n)][k],
// so per far offset the tile computes X = (S Vc^T)_g W (rank x 64) and then
// Loc += (Uc)_g X: 4 l^3 r flops per (target, source) pair instead of 2 l^6.
namespace {

// Factors in MFMA fragment order, per packed operator kid (rank padded to
// rp = 16 ceil(r/16)), both blocks rp * ld elements at off[kid]:
//   p1[((i*kc + c)*64 + lane)*4 + s] = s_k Vc[g(n)][k],  k = 16i + lane%16,
//                                                        n = 16c + 4(lane/16) + s
//   p2[((i*nr + c)*64 + lane)*4 + s] = Uc[g(m)][k],      m = 16i + lane%16,
//                                                        k = 16c + 4(lane/16) + s
// rocSOLVER works column-major: it factorises M = Kc^T (the row-major buffer
// read column-major) as M = U_M S V_M^T and returns U_M and V_M^T, so
// Uc[a][k] = Vt[a*n + k] and Vc[b][k] = U[k*n + b].
// Rank held by position p of the packed factors: inside each block of 16
// the 4 x 4 transpose, so that K-step st of a phase-2 MFMA chunk (positions
// 4g + st over the four lane groups g) takes the four consecutive ranks
// 4 st .. 4 st + 3, and the steps past the kept rank hold only zeros.  The
// order of the ranks in a sum over them is free; both factors use the same.
__host__ __device__ inline int rank_slot(int p) {
  return (p & ~15) | ((p & 3) << 2) | ((p >> 2) & 3);
}

__global__ void svd_pack_kernel(const double* __restrict__ U, const double* __restrict__ Vt,
                                const double* __restrict__ VtM,
                                const double* __restrict__ S, const int* __restrict__ info,
                                const int* __restrict__ rank, const int* __restrict__ rpad,
                                const int64_t* __restrict__ off, int l, int mt, int kc,
                                double* __restrict__ p1_64, float* __restrict__ p1_32,
                                double* __restrict__ p2_64, float* __restrict__ p2_32) {
  const int kid = blockIdx.y;
  const int l3 = l * l * l;
  const int* in = info + 7 * kid;  // canon, pi[3], sg[3]
  const int c = in[0];
  const int r = rank[c], rp = rpad[kid], nr = rp / 16;
  const int64_t nblk = int64_t(rp) * kc * 16;  // elements per factor block
  const double* Uc = U + int64_t(c) * l3 * l3;
  const double* Vc = Vt + int64_t(c) * l3 * l3;
  const double* VcM = VtM + int64_t(c) * l3 * l3;  // the same in coefficient rows
  const double* Sc = S + int64_t(c) * l3;
  auto gmap = [&](int m) {
    int mm[3] = {m / (l * l), (m / l) % l, m % l}, gm[3];
    for (int d = 0; d < 3; ++d) gm[in[1 + d]] = in[4 + d] > 0 ? mm[d] : l - 1 - mm[d];
    return (gm[0] * l + gm[1]) * l + gm[2];
  };
  for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < nblk;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int s = int(e & 3), lane = int((e >> 2) & 63);
    const int64_t q = e >> 8;
    {  // phase-1 factor: rows k (rp, in rank_slot order), columns n (ld)
      const int cc = int(q % kc), i = int(q / kc);
      const int k = rank_slot(16 * i + (lane & 15)), n = 16 * cc + 4 * (lane >> 4) + s;
      double v = 0.0;
      if (k < r && n < l3) v = Sc[k] * Uc[int64_t(k) * l3 + gmap(n)];
      p1_64[off[kid] + e] = v;
      p1_32[off[kid] + e] = float(v);
    }
    {  // phase-2 factor: rows m (ld), columns k (rp, in rank_slot order); the
       // FP32 factor's rows are Chebyshev coefficients
      const int cc = int(q % nr), i = int(q / nr);
      const int m = 16 * i + (lane & 15), k = rank_slot(16 * cc + 4 * (lane >> 4) + s);
      double v = 0.0, vm = 0.0;
      if (m < l3 && k < r) {
        v = Vc[int64_t(gmap(m)) * l3 + k];
        double sgn;
        const int gu = modal_row(in, l, m, sgn);
        vm = sgn * VcM[int64_t(gu) * l3 + k];
      }
      p2_64[off[kid] + e] = v;
      p2_32[off[kid] + e] = float(vm);
    }
  }
}

std::mutex g_svd_mu;
// (device, order, tolerance, kernel exponent)
std::map<std::tuple<int, int, double, int>, std::unique_ptr<SvdOps>> g_svd;
rocblas_handle g_blas[64] = {nullptr};

}  // namespace

int kid_canon(int kid) { return tables().offs[kid].canon; }

const SvdOps* get_svd_ops(int l, double eps, int kernel, hipStream_t s) {
  int dev = 0;
  FMM_HIP_CHECK(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_svd_mu);
  auto key = std::make_tuple(dev, l, eps, kernel);
  auto it = g_svd.find(key);
  if (it != g_svd.end()) return it->second.get();
  const OpSet* op = get_opset(l, kernel, s);
  const StaticTables& T = tables();
  const int l3 = l * l * l;
  auto sv = std::make_unique<SvdOps>();
  sv->order = l;
  sv->eps = eps;

  std::vector<void*> tmp;
  auto talloc = [&](size_t b) {
    void* q = dev_alloc(b);
    tmp.push_back(q);
    return q;
  };
  try {
    // the 16 canonical operators, then their SVDs (batched)
    double xi[kMaxOrder];
    cheb_nodes(l, xi);
    std::vector<int> tc(48), info(7 * kOffsets);
    for (int c = 0; c < 16; ++c)
      for (int d = 0; d < 3; ++d) tc[3 * c + d] = T.canon[c][d];
    for (int k = 0; k < kOffsets; ++k) {
      info[7 * k] = T.offs[k].canon;
      for (int d = 0; d < 3; ++d) {
        info[7 * k + 1 + d] = T.offs[k].pi[d];
        info[7 * k + 4 + d] = T.offs[k].sg[d];
      }
    }
    double* xi_d = static_cast<double*>(talloc(sizeof(double) * l));
    int* tc_d = static_cast<int*>(talloc(sizeof(int) * 48));
    int* info_d = static_cast<int*>(talloc(sizeof(int) * info.size()));
    FMM_HIP_CHECK(hipMemcpyAsync(xi_d, xi, sizeof(double) * l, hipMemcpyHostToDevice, s));
    FMM_HIP_CHECK(hipMemcpyAsync(tc_d, tc.data(), sizeof(int) * 48, hipMemcpyHostToDevice, s));
    FMM_HIP_CHECK(hipMemcpyAsync(info_d, info.data(), sizeof(int) * info.size(),
                                 hipMemcpyHostToDevice, s));
    const size_t nn = size_t(l3) * l3;
    double* A = static_cast<double*>(talloc(sizeof(double) * 16 * nn));
    double* U = static_cast<double*>(talloc(sizeof(double) * 16 * nn));
    double* Vt = static_cast<double*>(talloc(sizeof(double) * 16 * nn));
    double* S = static_cast<double*>(talloc(sizeof(double) * 16 * l3));
    double* E = static_cast<double*>(talloc(sizeof(double) * 16 * l3));
    int* dinfo = static_cast<int*>(talloc(sizeof(int) * 16));
    canon_kernel<<<1024, 256, 0, s>>>(xi_d, tc_d, l, 16, kernel, A);
    FMM_HIP_CHECK(hipGetLastError());
    if (dev < 0 || dev >= 64) throw FmmError{FMM_ERR_HIP, "device index out of range"};
    if (!g_blas[dev] && rocblas_create_handle(&g_blas[dev]) != rocblas_status_success)
      throw FmmError{FMM_ERR_HIP, "rocblas_create_handle failed"};
    if (rocblas_set_stream(g_blas[dev], s) != rocblas_status_success)
      throw FmmError{FMM_ERR_HIP, "rocblas_set_stream failed"};
    const rocblas_status st = rocsolver_dgesvd_strided_batched(
        g_blas[dev], rocblas_svect_all, rocblas_svect_all, l3, l3, A, l3, rocblas_stride(nn), S,
        rocblas_stride(l3), U, l3, rocblas_stride(nn), Vt, l3, rocblas_stride(nn), E,
        rocblas_stride(l3), rocblas_outofplace, dinfo, 16);
    if (st != rocblas_status_success) throw FmmError{FMM_ERR_HIP, "rocsolver gesvd failed"};
    std::vector<double> Sh(16 * size_t(l3));
    int hinfo[16];
    FMM_HIP_CHECK(hipMemcpyAsync(Sh.data(), S, sizeof(double) * Sh.size(), hipMemcpyDeviceToHost, s));
    FMM_HIP_CHECK(hipMemcpyAsync(hinfo, dinfo, sizeof(hinfo), hipMemcpyDeviceToHost, s));
    FMM_HIP_CHECK(hipStreamSynchronize(s));
    for (int c = 0; c < 16; ++c)
      if (hinfo[c] != 0) throw FmmError{FMM_ERR_HIP, "rocsolver gesvd did not converge"};

    // ranks: singular values come sorted, largest first
    int rank_h[16];
    for (int c = 0; c < 16; ++c) {
      const double* sc = &Sh[size_t(c) * l3];
      int r = 0;
      while (r < l3 && sc[r] >= eps * sc[0]) ++r;
      rank_h[c] = std::max(r, 1);
      sv->rank[c] = rank_h[c];
    }
    sv->rpad_h.resize(kOffsets);
    std::vector<int> rk_h(kOffsets);
    std::vector<int64_t> off(kOffsets);
    int64_t tot = 0;
    double wr = 0.0, wf = 0.0;
    for (int k = 0; k < kOffsets; ++k) {
      const int r = rank_h[T.offs[k].canon];
      const int rp = 16 * ((r + 15) / 16);
      sv->rpad_h[k] = rp;
      rk_h[k] = r;
      sv->rmax_pad = std::max(sv->rmax_pad, rp);
      off[k] = tot;
      tot += int64_t(rp) * op->ld;
      wr += r;
      wf += 4.0 * l3 * r;
    }
    sv->weighted_rank = wr / kOffsets;
    sv->flops_per_pair_weighted = int64_t(wf / kOffsets + 0.5);
    int* rank_d = static_cast<int*>(talloc(sizeof(int) * 16));
    FMM_HIP_CHECK(hipMemcpyAsync(rank_d, rank_h, sizeof(rank_h), hipMemcpyHostToDevice, s));
    sv->rpad = static_cast<int*>(dev_alloc(sizeof(int) * kOffsets));
    sv->off = static_cast<int64_t*>(dev_alloc(sizeof(int64_t) * kOffsets));
    FMM_HIP_CHECK(hipMemcpyAsync(sv->rpad, sv->rpad_h.data(), sizeof(int) * kOffsets,
                                 hipMemcpyHostToDevice, s));
    FMM_HIP_CHECK(hipMemcpyAsync(sv->off, off.data(), sizeof(int64_t) * kOffsets,
                                 hipMemcpyHostToDevice, s));
    sv->rk = static_cast<int*>(dev_alloc(sizeof(int) * kOffsets));
    FMM_HIP_CHECK(hipMemcpyAsync(sv->rk, rk_h.data(), sizeof(int) * kOffsets,
                                 hipMemcpyHostToDevice, s));
    const int64_t pad = int64_t(kSvdPadChunks) * 256;
    sv->p1_64 = static_cast<double*>(dev_alloc(sizeof(double) * (tot + pad)));
    sv->p2_64 = static_cast<double*>(dev_alloc(sizeof(double) * tot));
    sv->p1_32 = static_cast<float*>(dev_alloc(sizeof(float) * (tot + pad)));
    sv->p2_32 = static_cast<float*>(dev_alloc(sizeof(float) * tot));
    // Uc[a][k] = Vt[a * l3 + k]: its rows as Chebyshev coefficients, for FP32
    double* VtM = static_cast<double*>(talloc(sizeof(double) * 16 * nn));
    modal_rows_kernel<<<4096, 256, 0, s>>>(Vt, op->cheb, l, l3, 16, VtM);
    FMM_HIP_CHECK(hipGetLastError());
    svd_pack_kernel<<<dim3(64, kOffsets), 256, 0, s>>>(U, Vt, VtM, S, info_d, rank_d, sv->rpad,
                                                        sv->off, l, op->mt, op->kc, sv->p1_64,
                                                        sv->p1_32, sv->p2_64, sv->p2_32);
    FMM_HIP_CHECK(hipGetLastError());
    FMM_HIP_CHECK(hipStreamSynchronize(s));
  } catch (...) {
    (void)hipStreamSynchronize(s);
    for (void* q : tmp) dev_free(q);
    for (void* q : {(void*)sv->rpad, (void*)sv->rk, (void*)sv->off, (void*)sv->p1_64,
                    (void*)sv->p1_32, (void*)sv->p2_64, (void*)sv->p2_32})
      if (q) dev_free(q);
    throw;
  }
  for (void* q : tmp) dev_free(q);
  const SvdOps* r = sv.get();
  g_svd[key] = std::move(sv);
  return r;
}

}  // namespace fmm
