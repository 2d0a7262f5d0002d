// Plan construction on the GPU: root box, Morton keys, stable LSD radix sort,
// leaves and cells of every level, near lists and the M2L work tiles.
//
// The octree follows Sec. 3.2 (levels 0..h-1, leaf level h-1) with cells in
// Morton order (Sec. 4.2); near and far lists follow Sec. 2.1.2 (27 near
// cells, at most 189 far cells: children of the parent's near cells that are
// not adjacent).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "device_util.h"
#include "fmm_internal.h"

namespace fmm {

// ------------------------------------------------------------------ scan
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

template <typename T>
__device__ T block_exclusive_scan(T v, T* lds_wave, T* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  T x = v;
  for (int o = 1; o < 64; o <<= 1) {
    T y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) lds_wave[wave] = x;
  __syncthreads();
  T base = 0, all = 0;
  for (int w = 0; w < kScanThreads / 64; ++w) {
    if (w < wave) base += lds_wave[w];
    all += lds_wave[w];
  }
  __syncthreads();
  *total = all;
  return base + x - v;
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void scan_tiles_kernel(
    const T* __restrict__ in, T* __restrict__ out, T* __restrict__ sums,
    int64_t n) {
  __shared__ T lds[kScanThreads / 64];
  const int64_t base = int64_t(blockIdx.x) * kScanTile + int64_t(threadIdx.x) * kScanItems;
  T v[kScanItems];
  T s = 0;
  for (int k = 0; k < kScanItems; ++k) {
    int64_t i = base + k;
    v[k] = i < n ? in[i] : T(0);
    s += v[k];
  }
  T total;
  T run = block_exclusive_scan<T>(s, lds, &total);
  for (int k = 0; k < kScanItems; ++k) {
    int64_t i = base + k;
    if (i < n) out[i] = run;
    run += v[k];
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

template <typename T>
__global__ void scan_add_kernel(T* __restrict__ out, const T* __restrict__ offs,
                                int64_t n) {
  int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) out[i] += offs[i / kScanTile];
}

// n <= kScanSmall values in one workgroup (one launch instead of three).
constexpr int64_t kScanSmall = 16384;
constexpr int kScanSmallThreads = 1024, kScanSmallItems = 8;

template <typename T>
__global__ __launch_bounds__(kScanSmallThreads) void scan_small_kernel(const T* __restrict__ in,
                                                                       T* __restrict__ out,
                                                                       int n) {
  __shared__ T wave_sum[kScanSmallThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  T carry = 0;
  for (int base = 0; base < n; base += kScanSmallThreads * kScanSmallItems) {
    const int i0 = base + threadIdx.x * kScanSmallItems;
    T v[kScanSmallItems], sum = 0;
    for (int k = 0; k < kScanSmallItems; ++k) {
      v[k] = i0 + k < n ? in[i0 + k] : T(0);
      sum += v[k];
    }
    T x = sum;
    for (int o = 1; o < 64; o <<= 1) {
      const T y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) wave_sum[wave] = x;
    __syncthreads();
    T run = carry + x - sum, all = 0;
    for (int w = 0; w < kScanSmallThreads / 64; ++w) {
      if (w < wave) run += wave_sum[w];
      all += wave_sum[w];
    }
    carry += all;
    for (int k = 0; k < kScanSmallItems; ++k) {
      if (i0 + k < n) out[i0 + k] = run;
      run += v[k];
    }
    __syncthreads();
  }
}

// Exclusive scan of n values (in may equal out).  Temporary blocks are kept
// in `tmp` and released by the caller after the stream has drained.
template <typename T>
void exclusive_scan(const T* in, T* out, int64_t n, hipStream_t s,
                    std::vector<void*>& tmp) {
  if (n <= 0) return;
  if (n <= kScanSmall) {
    scan_small_kernel<T><<<1, kScanSmallThreads, 0, s>>>(in, out, int(n));
    FMM_HIP_CHECK(hipGetLastError());
    return;
  }
  const int64_t tiles = (n + kScanTile - 1) / kScanTile;
  T* sums = static_cast<T*>(dev_alloc(sizeof(T) * tiles));
  tmp.push_back(sums);
  scan_tiles_kernel<T><<<dim3(unsigned(tiles)), kScanThreads, 0, s>>>(in, out, sums, n);
  FMM_HIP_CHECK(hipGetLastError());
  exclusive_scan<T>(sums, sums, tiles, s, tmp);
  scan_add_kernel<T><<<dim3(unsigned((n + 255) / 256)), 256, 0, s>>>(out, sums, n);
  FMM_HIP_CHECK(hipGetLastError());
}

// ------------------------------------------------------------- bounding box
// Statistics gathered while a plan is built: far pairs per level, near pairs,
// active M2L slots, far pairs per operator, 16-target groups and empty ones.
constexpr int kStats = kMaxHeight + 4 + kOffsets;

// What the host needs to size the plan, read back once.
struct PlanHead {
  double box[6];  // per-axis minima, then maxima
  int bad;        // a position is NaN or infinite
  int pad;
  int cells[8 * kMaxHeight];  // cells of level l and child parity c at 8 l + c
};

constexpr int kBoxBlocks = 512;

// Per block: minima, maxima and whether a position is not finite.
__global__ __launch_bounds__(256) void bbox_partial_kernel(
    const double* __restrict__ pos, int64_t n, double* __restrict__ part,
    int* __restrict__ bad) {
  __shared__ double smin[3][256], smax[3][256];
  double mn[3] = {INFINITY, INFINITY, INFINITY};
  double mx[3] = {-INFINITY, -INFINITY, -INFINITY};
  int nonfinite = 0;
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * 256) {
    for (int d = 0; d < 3; ++d) {
      double v = pos[3 * i + d];
      if (!isfinite(v)) nonfinite = 1;
      mn[d] = fmin(mn[d], v);
      mx[d] = fmax(mx[d], v);
    }
  }
  nonfinite = __syncthreads_or(nonfinite);
  for (int d = 0; d < 3; ++d) {
    smin[d][threadIdx.x] = mn[d];
    smax[d][threadIdx.x] = mx[d];
  }
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o)
      for (int d = 0; d < 3; ++d) {
        smin[d][threadIdx.x] = fmin(smin[d][threadIdx.x], smin[d][threadIdx.x + o]);
        smax[d][threadIdx.x] = fmax(smax[d][threadIdx.x], smax[d][threadIdx.x + o]);
      }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    for (int d = 0; d < 3; ++d) {
      part[6 * blockIdx.x + d] = smin[d][0];
      part[6 * blockIdx.x + 3 + d] = smax[d][0];
    }
    bad[blockIdx.x] = nonfinite;
  }
}

// -------------------------------------------------------------- Morton keys
// k_d = min(floor((x_d - lo_d) / L * 2^(h-1)), 2^(h-1) - 1): IEEE divide, an
// exact scaling by a power of two and floor -- no contraction is possible.
// The root box comes from the device (per-axis min in box[0..2], max in
// box[3..5]); the cube side L = max extent (1 if zero) is formed here in the
// same FP64 operations as on the host.
__device__ __host__ inline double root_side(const double* box) {
  double L = 0.0;
  for (int d = 0; d < 3; ++d) L = fmax(L, box[3 + d] - box[d]);
  return L == 0.0 ? 1.0 : L;
}

// ITEMS particles a workgroup.  Every workgroup reduces the nb partial boxes
// itself (at most 24 KiB, from L2), which saves a launch; the first also
// writes the result to the head and clears the statistics.  All of them set
// the tslots entries of the lookup tables to -1.  D > 0: a workgroup is a tile
// of the sort and also counts its first digit, of D values.
template <int ITEMS, int D>
__global__ __launch_bounds__(256) void keys_kernel(
    const double* __restrict__ pos, int64_t n, const double* __restrict__ part,
    const int* __restrict__ bad, int nb, int bits, uint64_t* __restrict__ keys,
    int* __restrict__ idx, PlanHead* __restrict__ head,
    unsigned long long* __restrict__ stats, int* __restrict__ tables, int64_t tslots, int mask,
    int* __restrict__ hist) {
  __shared__ double red[6][4];
  __shared__ int digit[D > 0 ? D : 1];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  for (int d = t; d < D; d += 256) digit[d] = 0;
  for (int64_t i = int64_t(blockIdx.x) * 256 + t; i < tslots; i += int64_t(gridDim.x) * 256)
    tables[i] = -1;
  double v[6];
  for (int d = 0; d < 6; ++d) v[d] = d < 3 ? INFINITY : -INFINITY;
  int nonfinite = 0;
  for (int b = t; b < nb; b += 256) {
    for (int d = 0; d < 6; ++d) {
      const double x = part[6 * b + d];
      v[d] = d < 3 ? fmin(v[d], x) : fmax(v[d], x);
    }
    nonfinite |= bad[b];
  }
  for (int o = 32; o > 0; o >>= 1)
    for (int d = 0; d < 6; ++d) {
      const double x = __shfl_xor(v[d], o, 64);
      v[d] = d < 3 ? fmin(v[d], x) : fmax(v[d], x);
    }
  if (lane == 0)
    for (int d = 0; d < 6; ++d) red[d][wave] = v[d];
  nonfinite = __syncthreads_or(nonfinite);
  double box[6];
  for (int d = 0; d < 6; ++d) {
    box[d] = red[d][0];
    for (int w = 1; w < 4; ++w) box[d] = d < 3 ? fmin(box[d], red[d][w]) : fmax(box[d], red[d][w]);
  }
  if (blockIdx.x == 0) {
    if (t == 0) {
      for (int d = 0; d < 6; ++d) head->box[d] = box[d];
      head->bad = nonfinite;
    }
    for (int e = t; e < kStats; e += 256) stats[e] = 0;
  }
  const double side = double(int64_t(1) << bits);
  const int64_t kmax = (int64_t(1) << bits) - 1;
  const double L = root_side(box);
  const int64_t base = int64_t(blockIdx.x) * ITEMS;
  for (int e = t; e < ITEMS; e += 256) {
    const int64_t i = base + e;
    if (i >= n) break;
    uint32_t k3[3];
    for (int d = 0; d < 3; ++d) {
      double u = (pos[3 * i + d] - box[d]) / L;
      int64_t k = int64_t(floor(u * side));
      k = k > kmax ? kmax : (k < 0 ? 0 : k);
      k3[d] = uint32_t(k);
    }
    const uint64_t key = morton3(k3[0], k3[1], k3[2], bits);
    keys[i] = key;
    idx[i] = int(i);
    if (D > 0) atomicAdd(&digit[int(key) & mask], 1);
  }
  if (D > 0) {
    __syncthreads();
    for (int d = t; d < D; d += 256) hist[int64_t(blockIdx.x) * D + d] = digit[d];
  }
}

// ------------------------------------------------------- stable radix sort
// LSD radix sort of (key, value) pairs.  Stability (equal keys
// keep input order) is what makes the permutation unique: ties are ordered by
// input index.  Per pass: tile histograms, one exclusive scan over the
// digit-major histogram, then a scatter that ranks equal digits in input
// order with wavefront ballots.
// A tile is 256 IT particles, IT = 4 up to kRsSmall of them (a tile is a
// chain of IT ranked steps: 1,000 particles 11 -> 4.6 us a scatter) and 16 above.
// Up to kRsSmall, where launches and latency are what a pass takes, the
// histograms are tile-major, every scatter workgroup adds up the tiles'
// counts itself (at most 512 KiB, from L2; 60,000 particles: 4 us, a scan by
// one workgroup 16), and the first pass's counts come with the keys (steps of
// 1,000, 20,000, 60,000 particles 245 -> 222, 380 -> 363, 1323 -> 1288 us).
// There the digits have 9 bits where that saves a pass, i.e. in trees of height
// 4 (plan of 20,000 particles 125 -> 109 us) and 7 (60,000: 189 -> 180), and 8
// elsewhere (height 5, 60,000 particles: 135 us, and 139 in 9).
constexpr int kRsThreads = 256;
constexpr int64_t kRsSmall = 262144;

template <int IT, int D>
__global__ __launch_bounds__(kRsThreads) void radix_hist_kernel(
    const uint64_t* __restrict__ keys, int64_t n, int shift, int mask,
    int ntiles, int* __restrict__ hist) {
  __shared__ int h[D];
  for (int d = threadIdx.x; d < D; d += kRsThreads) h[d] = 0;
  __syncthreads();
  const int64_t base = int64_t(blockIdx.x) * (kRsThreads * IT);
  for (int it = 0; it < IT; ++it) {
    int64_t i = base + int64_t(it) * kRsThreads + threadIdx.x;
    if (i < n) atomicAdd(&h[int((keys[i] >> shift) & uint64_t(mask))], 1);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < D; d += kRsThreads)
    hist[IT == 4 ? int64_t(blockIdx.x) * D + d : int64_t(d) * ntiles + blockIdx.x] = h[d];
}

template <int IT, int D>
__global__ __launch_bounds__(kRsThreads) void radix_scatter_kernel(
    const uint64_t* __restrict__ kin, const int* __restrict__ vin,
    uint64_t* __restrict__ kout, int* __restrict__ vout, int64_t n, int shift,
    int mask, int ntiles, const int* __restrict__ offs) {
  __shared__ int base_d[D];
  __shared__ int wcnt[kRsThreads / 64][D];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  if (IT == 4) {
    // smaller digits of all tiles, and this digit of the earlier ones; E
    // adjacent digits a thread
    constexpr int E = D / kRsThreads;
    __shared__ int wave_sum[kRsThreads / 64];
    int before[E], total[E], incl = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) before[e] = total[e] = 0;
#pragma unroll 16
    for (int b = 0; b < ntiles; ++b)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int c = offs[int64_t(b) * D + E * tid + e];
        total[e] += c;
        before[e] += b < int(blockIdx.x) ? c : 0;
      }
#pragma unroll
    for (int e = 0; e < E; ++e) incl += total[e];
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += wave_sum[w];
#pragma unroll
    for (int e = E - 1; e >= 0; --e) {
      incl -= total[e];
      base_d[E * tid + e] = incl + before[e];
    }
    __syncthreads();
  } else {
    base_d[tid] = offs[int64_t(tid) * ntiles + blockIdx.x];
  }
  const int64_t tbase = int64_t(blockIdx.x) * (kRsThreads * IT);
  for (int it = 0; it < IT; ++it) {
    for (int k = lane; k < D; k += 64) wcnt[wave][k] = 0;
    const int64_t i = tbase + int64_t(it) * kRsThreads + tid;
    const bool valid = i < n;
    uint64_t key = valid ? kin[i] : 0;
    int val = valid ? vin[i] : 0;
    const int d = valid ? int((key >> shift) & uint64_t(mask)) : 0;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < (D == 512 ? 9 : 8); ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const int rank = __popcll(peers & lt);
    __syncthreads();
    if (valid && rank == 0) wcnt[wave][d] = __popcll(peers);
    __syncthreads();
    for (int e = tid; e < D; e += kRsThreads) {
      int run = base_d[e];
      for (int w = 0; w < kRsThreads / 64; ++w) {
        int c = wcnt[w][e];
        wcnt[w][e] = run;
        run += c;
      }
      base_d[e] = run;
    }
    __syncthreads();
    if (valid) {
      const int p = wcnt[wave][d] + rank;
      kout[p] = key;
      vout[p] = val;
    }
    __syncthreads();
  }
}

// Bits of a pass's digit, and passes, of a sort by `bits` key bits.
static int radix_digit(int64_t n, int bits) {
  return n <= kRsSmall && (bits + 8) / 9 < (bits + 7) / 8 ? 9 : 8;
}
static int radix_passes(int64_t n, int bits) {
  return n <= 1 ? 0 : ceil_div(bits, radix_digit(n, bits));
}

// Sorts n pairs by the low `bits` bits of the key, from (k, v) through
// (k2, v2) and back: after an odd number of passes the result is in the
// second pair of buffers.  hist: D counts a tile (IT == 4: the first
// pass's).
template <int IT, int D>
static void radix_sort(uint64_t* k, int* v, uint64_t* k2, int* v2, int64_t n, int bits,
                       hipStream_t s, std::vector<void*>& tmp, int* hist) {
  const int ntiles = ceil_div(n, kRsThreads * IT);
  for (int p = 0; p < radix_passes(n, bits); ++p) {
    constexpr int digit = D == 512 ? 9 : 8;
    const int shift = digit * p, db = std::min(digit, bits - shift);
    const int mask = (1 << db) - 1;
    if (IT != 4 || p > 0) {
      radix_hist_kernel<IT, D><<<ntiles, kRsThreads, 0, s>>>(k, n, shift, mask, ntiles, hist);
      FMM_HIP_CHECK(hipGetLastError());
    }
    if (IT != 4) exclusive_scan<int>(hist, hist, int64_t(256) * ntiles, s, tmp);
    radix_scatter_kernel<IT, D><<<ntiles, kRsThreads, 0, s>>>(k, v, k2, v2, n, shift, mask,
                                                              ntiles, hist);
    FMM_HIP_CHECK(hipGetLastError());
    std::swap(k, k2);
    std::swap(v, v2);
  }
}

// ------------------------------------------------- the cells of every level
// Particle i of the sorted keys k starts a new cell at level l exactly when
// (k[i] >> 3(h-1-l)) != (k[i-1] >> 3(h-1-l)), i.e. at every level from
// first(i) = h-1-floor(t/3) on, t the highest bit in which k[i] and k[i-1]
// differ (level 0 for i = 0, none if the keys are equal).  Two passes over the
// particles build every level at once: cells_count_kernel counts, per
// workgroup, the cells starting at each level and child parity,
// cells_scan_kernel scans those counts over the workgroups (and totals them
// for the host), and cells_emit_kernel ranks the starting particles with
// wavefront ballots and writes the cells' keys, first particles, children,
// parents, lookup entries and places among the M2L targets.  All of it is
// bound by launches and memory latency; level by level from the leaves it
// took three times the launches and a second read-back (whole step: 1,000
// particles 427 -> 236 us, 20,000 612 -> 446 us, 1M 5.17 -> 4.92 ms).
constexpr int kCellThreads = 256, kCellWaves = kCellThreads / 64;

// 64-particle rounds a wavefront takes in a row
static int cell_rounds(int64_t n) {
  return n <= (int64_t(1) << 18) ? 4 : n <= (int64_t(1) << 24) ? 16 : 64;
}

__device__ inline int first_level(const uint64_t* __restrict__ keys, int64_t i, uint64_t key,
                                  int h) {
  if (i == 0) return 0;
  const uint64_t x = key ^ keys[i - 1];
  return x ? h - 1 - (63 - __clzll(x)) / 3 : h;
}

// count[c * nblocks + b]: cells of level c / 8 and child parity c % 8 that
// start in workgroup b.  Also gathers the sorted positions.
__global__ __launch_bounds__(kCellThreads) void cells_count_kernel(
    const uint64_t* __restrict__ keys, const int* __restrict__ perm,
    const double* __restrict__ pos, int64_t n, int h, int rounds, double* __restrict__ px,
    double* __restrict__ py, double* __restrict__ pz, int* __restrict__ count) {
  __shared__ int cnt[8 * kMaxHeight];
  for (int e = threadIdx.x; e < 8 * h; e += kCellThreads) cnt[e] = 0;
  __syncthreads();
  const int64_t base = int64_t(blockIdx.x) * kCellThreads * rounds;
  for (int r = 0; r < rounds; ++r) {
    const int64_t i = base + int64_t(r) * kCellThreads + threadIdx.x;
    if (i >= n) break;
    const uint64_t key = keys[i];
    const int64_t j = perm[i];
    const double x = pos[3 * j], y = pos[3 * j + 1], z = pos[3 * j + 2];
    for (int l = first_level(keys, i, key, h); l < h; ++l)
      atomicAdd(&cnt[8 * l + int((key >> (3 * (h - 1 - l))) & 7u)], 1);
    px[i] = x;
    py[i] = y;
    pz[i] = z;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 8 * h; e += kCellThreads)
    count[int64_t(e) * gridDim.x + blockIdx.x] = cnt[e];
}

// Workgroup c: exclusive scan of count[c * nb ...], the total to the head.
__global__ __launch_bounds__(kScanThreads) void cells_scan_kernel(int* __restrict__ count,
                                                                  int nb,
                                                                  PlanHead* __restrict__ head) {
  __shared__ int lds[kScanThreads / 64];
  int* col = count + int64_t(blockIdx.x) * nb;
  int carry = 0;
  for (int b0 = 0; b0 < nb; b0 += kScanThreads) {
    const int b = b0 + int(threadIdx.x);
    const int v = b < nb ? col[b] : 0;
    int total;
    const int before = block_exclusive_scan<int>(v, lds, &total);
    if (b < nb) col[b] = carry + before;
    carry += total;
  }
  if (threadIdx.x == 0) head->cells[blockIdx.x] = carry;
}

struct CellsOut {
  uint64_t* keys[kMaxHeight];
  int* child_start[kMaxHeight];  // [ncell_l + 1] first child at level l+1
  int* parent[kMaxHeight];       // [ncell_l] cell of level l-1 containing it
  int* table[kMaxHeight];        // dense key -> index, or null
  int ncell[kMaxHeight];
  int off[kMaxHeight];           // global id of the level's first cell
  int tstart[8 * kMaxHeight];    // first target of (level, parity) in tgt
  int* leaf_start;
  int* tgt;                      // null below height 3
};

__global__ __launch_bounds__(kCellThreads) void cells_emit_kernel(
    const uint64_t* __restrict__ keys, int64_t n, int h, int rounds,
    const int* __restrict__ count, CellsOut out) {
  // cells of (level, parity), and of the level, that start before the
  // wavefront's next round
  __shared__ int pbase[kCellWaves][8 * kMaxHeight];
  __shared__ int lbase[kCellWaves][kMaxHeight];
  const int lane = threadIdx.x & 63, wave = wuni(int(threadIdx.x >> 6));
  for (int e = threadIdx.x; e < kCellWaves * 8 * kMaxHeight; e += kCellThreads)
    pbase[e / (8 * kMaxHeight)][e % (8 * kMaxHeight)] = 0;
  __syncthreads();
  const int64_t base = (int64_t(blockIdx.x) * kCellWaves + wave) * 64 * rounds;
  for (int r = 0; r < rounds; ++r) {
    const int64_t i = base + 64 * r + lane;
    if (i >= n) break;
    const uint64_t key = keys[i];
    for (int l = first_level(keys, i, key, h); l < h; ++l)
      atomicAdd(&pbase[wave][8 * l + int((key >> (3 * (h - 1 - l))) & 7u)], 1);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 8 * h; e += kCellThreads) {
    int run = count[int64_t(e) * gridDim.x + blockIdx.x];
    for (int w = 0; w < kCellWaves; ++w) {
      const int c = pbase[w][e];
      pbase[w][e] = run;
      run += c;
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kCellWaves * h; e += kCellThreads) {
    int v = 0;
    for (int c = 0; c < 8; ++c) v += pbase[e / h][8 * (e % h) + c];
    lbase[e / h][e % h] = v;
  }
  __syncthreads();
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  for (int r = 0; r < rounds; ++r) {
    if (base + 64 * r >= n) break;  // the same for the whole wavefront
    const int64_t i = base + 64 * r + lane;
    const uint64_t key = i < n ? keys[i] : 0;
    const int first = i < n ? first_level(keys, i, key, h) : h;
    uint64_t above = 0;      // lanes that start a cell of the level above
    int above_base = 0;      // its lbase before this round
    int above_cell = 0;      // the cell of the level above this lane starts
    for (int l = 0; l < h; ++l) {
      const int lb = lbase[wave][l];
      const uint64_t mask = __ballot(first <= l);
      if (mask) {
        const uint64_t ck = key >> (3 * (h - 1 - l));
        const int par = int(ck & 7u);
        uint64_t peers = mask;
        for (int b = 0; b < 3; ++b) {
          const uint64_t m = __ballot((par >> b) & 1);
          peers &= (par >> b) & 1 ? m : ~m;
        }
        const int c = lb + __popcll(mask & lt);
        if (first <= l) {
          const int pb = pbase[wave][8 * l + par];
          out.keys[l][c] = ck;
          if (out.table[l]) out.table[l][ck] = c;
          if (l > 0) out.parent[l][c] = above_base + __popcll(above & (lt | (lt + 1))) - 1;
          if (first < l) out.child_start[l - 1][above_cell] = c;
          if (l == h - 1) out.leaf_start[c] = int(i);
          if (l >= 2 && out.tgt)
            out.tgt[out.tstart[8 * l + par] + pb + __popcll(peers & lt)] = out.off[l] + c;
          above_cell = c;
          if ((peers & lt) == 0) pbase[wave][8 * l + par] = pb + __popcll(peers);
        }
        if (lane == 0) lbase[wave][l] = lb + __popcll(mask);
        wave_lds_sync();
      }
      above = mask;
      above_base = lb;
    }
  }
  if (blockIdx.x == 0)
    for (int l = threadIdx.x; l < h; l += kCellThreads) {
      if (l < h - 1) out.child_start[l][out.ncell[l]] = out.ncell[l + 1];
      else out.leaf_start[out.ncell[l]] = int(n);
    }
}

// ------------------------------------------------------------ near lists
// near[a][s], s = (dx+1)*9 + (dy+1)*3 + (dz+1): the leaf at offset (dx,dy,dz)
// or -1.  Also counts directed particle pairs n_a * sum_b n_b.  A workgroup
// takes 64 leaves, its threads their 27 slots side by side (one thread per
// leaf ran 27 lookups in a row: 1,000 particles 14 -> 5.4 us).
constexpr int kNearLeaves = 64;

__global__ __launch_bounds__(256) void near_kernel(LevelDev leaves,
                                                   const int* __restrict__ leaf_start,
                                                   int* __restrict__ near,
                                                   unsigned long long* __restrict__ pairs) {
  __shared__ int cell[kNearLeaves][4];  // coordinates, particles
  __shared__ unsigned long long sum[4];
  const int a0 = blockIdx.x * kNearLeaves, t = threadIdx.x;
  if (t < kNearLeaves && a0 + t < leaves.ncell) {
    const int a = a0 + t;
    demorton3(leaves.keys[a], leaves.bits, cell[t]);
    cell[t][3] = leaf_start[a + 1] - leaf_start[a];
  }
  __syncthreads();
  unsigned long long cnt = 0;
  const int na = min(kNearLeaves, leaves.ncell - a0);
  for (int e = t; e < 27 * na; e += 256) {
    const int k = e / 27, s = e % 27;
    const int b = level_find_xyz(leaves, cell[k][0] + s / 9 - 1, cell[k][1] + (s / 3) % 3 - 1,
                                 cell[k][2] + s % 3 - 1);
    near[27 * int64_t(a0) + e] = b;
    if (b >= 0)
      cnt += (unsigned long long)cell[k][3] * (unsigned long long)(leaf_start[b + 1] - leaf_start[b]);
  }
  for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
  if ((t & 63) == 0) sum[t >> 6] = cnt;
  __syncthreads();
  if (t == 0) atomicAdd(pairs, sum[0] + sum[1] + sum[2] + sum[3]);
}

// ------------------------------------------------------------ M2L tiles
// One workgroup of sixteen wavefronts per tile.  Lane j of every wavefront owns
// target j; wavefront w looks up the source cells of the slots w, w+16, ...
// (zero row if absent) and marks the slots with at least one source; then
// the marked slots are listed in slot order, each with the mask of its
// 16-target groups that have a source (bit g: targets 16g .. 16g+15), and
// the tile's groups of targets without a source at an active slot are
// counted.
constexpr int kTileThreads = 1024;

__global__ __launch_bounds__(kTileThreads) void tile_src_kernel(
    const M2LTile* __restrict__ tiles, const int* __restrict__ tgt,
    const LevelDev* __restrict__ levels, const int64_t* __restrict__ lev_off,
    const signed char* __restrict__ slot_t,  // [8][189][3]
    int zero_row, int* __restrict__ tile_src, unsigned char* __restrict__ act,
    unsigned char* __restrict__ gmask, int* __restrict__ nact, unsigned long long* __restrict__ pairs_level,
    const int* __restrict__ slot_kid, unsigned long long* __restrict__ pairs_kid,
    unsigned long long* __restrict__ active_total,
    unsigned long long* __restrict__ groups) {  // [0] groups at active slots, [1] empty ones
  __shared__ int npair[kSlots];
  __shared__ unsigned char smask[kSlots];
  const int tile = blockIdx.x, j = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const M2LTile T = tiles[tile];
  const LevelDev L = levels[T.level];
  const int first = int(lev_off[T.level]);
  constexpr int kStride = kTileThreads / 64, kBatch = (kSlots + kStride - 1) / kStride;
  // a wavefront's offsets are read beside its targets' keys, and all its
  // lookups are issued before any is used: a chain of five reads in all, which
  // bounds small plans (18 -> 12 us; eight wavefronts had three batches)
  int off[kBatch][3];
#pragma unroll
  for (int u = 0; u < kBatch; ++u) {
    const signed char* t = slot_t + (T.parity * kSlots + min(wave + u * kStride, kSlots - 1)) * 3;
#pragma unroll
    for (int d = 0; d < 3; ++d) off[u][d] = t[d];
  }
  int c[3] = {0, 0, 0};
  const bool have = j < T.count;
  if (have) {
    const int local = tgt[T.first + j] - first;
    demorton3(L.keys[local], L.bits, c);
  }
  int* out = tile_src + int64_t(tile) * kSlots * kTileN;
  {
    const int s0 = wave;
    int bs[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      bs[u] = -1;
      if (have && s0 + u * kStride < kSlots)
        bs[u] = level_find_xyz(L, c[0] + off[u][0], c[1] + off[u][1], c[2] + off[u][2]);
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int s = s0 + u * kStride;
      if (s >= kSlots) continue;  // the same for the whole wavefront
      out[s * kTileN + j] = bs[u] >= 0 ? bs[u] + first : zero_row;
      const uint64_t m = __ballot(bs[u] >= 0);
      if (j == 0) {
        npair[s] = __popcll(m);
        int g = 0;
        for (int q = 0; q < 4; ++q) g |= ((m >> (16 * q)) & 0xffffu) != 0 ? 1 << q : 0;
        smask[s] = (unsigned char)g;
      }
    }
  }
  __syncthreads();
  // active slots in ascending order: wavefront w compacts slots 64w .. 64w+63
  // (a ballot prefix within it, the earlier wavefronts' counts before it)
  __shared__ int wave_active[(kSlots + 63) / 64];
  constexpr int kSlotWaves = (kSlots + 63) / 64;
  static_assert(kSlotWaves * 64 <= kTileThreads, "one thread per slot");
  const int s = threadIdx.x;
  const int k = s < kSlots ? npair[s] : 0;
  const uint64_t m = __ballot(k > 0);
  if (wave < kSlotWaves && j == 0) wave_active[wave] = __popcll(m);
  __syncthreads();
  if (wave < kSlotWaves) {
    int base = 0;
    for (int w = 0; w < wave; ++w) base += wave_active[w];
    if (k > 0) {
      const int pos = base + __popcll(m & ((uint64_t(1) << j) - 1));
      act[int64_t(tile) * kSlots + pos] = (unsigned char)s;
      gmask[int64_t(tile) * kSlots + pos] = smask[s];
      atomicAdd(&pairs_kid[slot_kid[T.parity * kSlots + s]], (unsigned long long)k);
    }
    // pairs of this wavefront's slots, summed across its lanes
    unsigned long long np = (unsigned long long)k;
    for (int o = 32; o > 0; o >>= 1) np += __shfl_xor(np, o, 64);
    if (j == 0 && np) atomicAdd(&pairs_level[T.level], np);
    // groups of targets at the active slots, and those without a source
    const int ngr = (T.count + 15) / 16;
    unsigned long long gt = 0, ge = 0;
    if (k > 0) {
      gt = (unsigned long long)ngr;
      for (int q = 0; q < ngr; ++q) ge += (smask[s] >> q) & 1 ? 0 : 1;
    }
    for (int o = 32; o > 0; o >>= 1) {
      gt += __shfl_xor(gt, o, 64);
      ge += __shfl_xor(ge, o, 64);
    }
    if (j == 0 && gt) {
      atomicAdd(&groups[0], gt);
      if (ge) atomicAdd(&groups[1], ge);
    }
    if (threadIdx.x == 0) {
      int na = 0;
      for (int w = 0; w < kSlotWaves; ++w) na += wave_active[w];
      nact[tile] = na;
      atomicAdd(active_total, (unsigned long long)na);
    }
  }
}

// --------------------------------------------------------------- driver
static inline unsigned grid_for(int64_t n, int b) { return unsigned((n + b - 1) / b); }

void build_plan(fmm_plan_s* p, const double* pos, hipStream_t s) {
  std::vector<void*> tmp;
  struct TmpGuard {
    std::vector<void*>& v;
    hipStream_t s;
    ~TmpGuard() {
      (void)hipStreamSynchronize(s);  // returns at once where s has drained
      for (void* q : v) dev_free(q);
    }
  } guard{tmp, s};
  auto talloc = [&](size_t b) {
    void* q = dev_alloc(b);
    tmp.push_back(q);
    return q;
  };

  const int64_t n = p->n;
  const int h = p->height;
  const int bits = h - 1;

  // --- root box and keys (non-finite positions give clamped keys, and the
  // plan is rejected at the read-back) ---
  const int nb = int(std::min<int64_t>(kBoxBlocks, (n + 255) / 256));
  double* part = static_cast<double*>(talloc(sizeof(double) * 6 * nb));
  int* bad = static_cast<int*>(talloc(sizeof(int) * nb));
  PlanHead* head = static_cast<PlanHead*>(talloc(sizeof(PlanHead)));
  unsigned long long* stats =
      static_cast<unsigned long long*>(talloc(sizeof(unsigned long long) * kStats));
  bbox_partial_kernel<<<nb, 256, 0, s>>>(pos, n, part, bad);
  FMM_HIP_CHECK(hipGetLastError());

  // --- the stable sort, which ends in the plan's own buffers ---
  p->keys = static_cast<uint64_t*>(p->alloc(sizeof(uint64_t) * n));
  p->perm = static_cast<int*>(p->alloc(sizeof(int) * n));
  uint64_t* kt = static_cast<uint64_t*>(talloc(sizeof(uint64_t) * n));
  int* vt = static_cast<int*>(talloc(sizeof(int) * n));
  const bool odd = radix_passes(n, 3 * bits) % 2 != 0;
  uint64_t *k1 = odd ? kt : p->keys, *k2 = odd ? p->keys : kt;
  int *v1 = odd ? vt : p->perm, *v2 = odd ? p->perm : vt;
  // dense lookup tables for levels with at most 2^24 key slots, one block,
  // all -1
  int64_t tslots = 0;
  for (int l = 0; l < h && 3 * l <= 24; ++l) tslots += int64_t(1) << (3 * l);
  int* tables = static_cast<int*>(p->alloc(sizeof(int) * tslots));
  const bool small = n <= kRsSmall;
  const int items = small ? 4 * kRsThreads : 2048;
  const unsigned kb = grid_for(n, items);
  int64_t fill = tslots;  // by the keys' workgroups where they are enough
  if (tslots > int64_t(64) * 256 * kb) {
    FMM_HIP_CHECK(hipMemsetAsync(tables, 0xff, sizeof(int) * tslots, s));
    fill = 0;
  }
  const int digit = radix_digit(n, 3 * bits);
  int* hist = static_cast<int*>(
      talloc((sizeof(int) << digit) * size_t(ceil_div(n, kRsThreads * (small ? 4 : 16)))));
  if (small) {
    const int mask = (1 << std::min(digit, 3 * bits)) - 1;
    auto keys_and_sort = [&](auto d) {
      constexpr int D = decltype(d)::value;
      keys_kernel<4 * kRsThreads, D><<<kb, 256, 0, s>>>(pos, n, part, bad, nb, bits, k1, v1, head,
                                                        stats, tables, fill, mask, hist);
      FMM_HIP_CHECK(hipGetLastError());
      radix_sort<4, D>(k1, v1, k2, v2, n, 3 * bits, s, tmp, hist);
    };
    if (digit == 9) keys_and_sort(std::integral_constant<int, 512>{});
    else keys_and_sort(std::integral_constant<int, 256>{});
  } else {
    keys_kernel<2048, 0><<<kb, 256, 0, s>>>(pos, n, part, bad, nb, bits, k1, v1, head,
                                                stats, tables, fill, 0, nullptr);
    FMM_HIP_CHECK(hipGetLastError());
    radix_sort<16, 256>(k1, v1, k2, v2, n, 3 * bits, s, tmp, hist);
  }

  // --- sorted positions, cell counts of every level and child parity ---
  p->px = static_cast<double*>(p->alloc(sizeof(double) * n));
  p->py = static_cast<double*>(p->alloc(sizeof(double) * n));
  p->pz = static_cast<double*>(p->alloc(sizeof(double) * n));
  const int rounds = cell_rounds(n);
  const int cb = int(grid_for(n, kCellThreads * rounds));
  int* count = static_cast<int*>(talloc(sizeof(int) * 8 * size_t(h) * cb));
  cells_count_kernel<<<cb, kCellThreads, 0, s>>>(p->keys, p->perm, pos, n, h, rounds, p->px,
                                                 p->py, p->pz, count);
  FMM_HIP_CHECK(hipGetLastError());
  cells_scan_kernel<<<8 * h, kScanThreads, 0, s>>>(count, cb, head);
  FMM_HIP_CHECK(hipGetLastError());

  // --- the read-back that sizes the plan ---
  // pinned staging of the calling thread: the head, later the statistics
  static_assert(sizeof(PlanHead) <= 4096 && sizeof(unsigned long long) * kStats <= 4096, "staging");
  char* stage = static_cast<char*>(pinned_staging(4096));
  const PlanHead* hd = reinterpret_cast<const PlanHead*>(stage);
  FMM_HIP_CHECK(hipMemcpyAsync(stage, head, sizeof(PlanHead), hipMemcpyDeviceToHost, s));
  FMM_HIP_CHECK(hipStreamSynchronize(s));
  if (hd->bad) throw FmmError{FMM_ERR_ARG, "positions contain NaN or Inf"};
  for (int d = 0; d < 3; ++d) p->lo[d] = hd->box[d];
  p->L = root_side(hd->box);
  LevelView* lev = p->lev;
  CellsOut out{};
  int64_t off = 0;
  tslots = 0;
  // A tree has one root and at least as many cells per level down to the
  // leaves, at most n; anything else would make the kernels below write out
  // of bounds.
  for (int l = 0; l < h; ++l) {
    int64_t c = 0;
    for (int q = 0; q < 8; ++q) c += hd->cells[8 * l + q];
    if (c < 1 || c > n || (l == 0 ? c != 1 : c < lev[l - 1].ncell))
      throw FmmError{FMM_ERR_HIP, "inconsistent octree level counts"};
    lev[l].ncell = c;
    lev[l].off = off;
    off += c;
  }
  p->ncell_total = off;
  p->nleaf = lev[h - 1].ncell;
  const int64_t nl = p->nleaf;
  if (off >= (int64_t(1) << 31) - 1) throw FmmError{FMM_ERR_ARG, "too many cells"};

  // --- cells of every level, lookup tables, M2L targets ---
  LevelDev ldev[kMaxHeight];
  for (int l = 0; l < h; ++l) {
    lev[l].keys = static_cast<uint64_t*>(p->alloc(sizeof(uint64_t) * lev[l].ncell));
    if (l < h - 1)
      lev[l].child_start = static_cast<int*>(p->alloc(sizeof(int) * (lev[l].ncell + 1)));
    if (l > 0) lev[l].parent = static_cast<int*>(p->alloc(sizeof(int) * lev[l].ncell));
    if (3 * l <= 24) {
      lev[l].lookup = tables + tslots;
      tslots += int64_t(1) << (3 * l);
    }
    ldev[l] = {lev[l].keys, lev[l].lookup, int(lev[l].ncell), l};
    out.keys[l] = lev[l].keys;
    out.child_start[l] = lev[l].child_start;
    out.parent[l] = lev[l].parent;
    out.table[l] = lev[l].lookup;
    out.ncell[l] = int(lev[l].ncell);
    out.off[l] = int(lev[l].off);
  }
  p->leaf_start = static_cast<int*>(p->alloc(sizeof(int) * (nl + 1)));
  out.leaf_start = p->leaf_start;
  if (h >= 3) {
    // targets grouped by (level, child parity), in Morton order within
    p->tgt = static_cast<int*>(p->alloc(sizeof(int) * (p->ncell_total - lev[2].off)));
    out.tgt = p->tgt;
    int at = 0;
    for (int l = 2; l < h; ++l)
      for (int q = 0; q < 8; ++q) {
        out.tstart[8 * l + q] = at;
        at += hd->cells[8 * l + q];
      }
  }
  cells_emit_kernel<<<cb, kCellThreads, 0, s>>>(p->keys, n, h, rounds, count, out);
  FMM_HIP_CHECK(hipGetLastError());

  // --- near lists ---
  p->near = static_cast<int*>(p->alloc(sizeof(int) * 27 * nl));
  near_kernel<<<grid_for(nl, kNearLeaves), 256, 0, s>>>(ldev[h - 1], p->leaf_start, p->near,
                                                        stats + kMaxHeight);
  FMM_HIP_CHECK(hipGetLastError());
  p->q32 = static_cast<float*>(p->alloc(sizeof(float) * n));

  // --- M2L tiles: targets of each level >= 2 grouped by child parity ---
  if (h >= 3) {
    // finest level first: the largest tiles' work is scheduled before the
    // coarse levels fill in the tail.  Within a level the parities take
    // turns: the k-th tile of every parity covers about the same region of
    // space, so the eight run side by side (on one XCD, whose L2 then serves
    // the source multipoles they share) instead of one parity sweeping the
    // whole level after another.
    std::vector<M2LTile> tiles;
    for (int l = h - 1; l >= 2; --l) {
      int kmax = 0;
      for (int q = 0; q < 8; ++q) kmax = std::max(kmax, hd->cells[8 * l + q]);
      for (int k = 0; k < kmax; k += kTileN)
        for (int q = 0; q < 8; ++q) {
          const int c = hd->cells[8 * l + q];
          if (k < c) tiles.push_back({l, q, out.tstart[8 * l + q] + k, std::min(kTileN, c - k)});
        }
    }
    p->ntiles = int64_t(tiles.size());
    p->tiles_host = tiles;
    if (p->ntiles > 0) {
      // one transfer: the level tables, the level offsets, then the tiles
      // (the head has been read: the staging may grow)
      constexpr size_t kOffAt = 1024, kTilesAt = 2048;
      static_assert(sizeof(LevelDev) * kMaxHeight <= kOffAt &&
                        sizeof(int64_t) * kMaxHeight <= kTilesAt - kOffAt,
                    "staging layout");
      const size_t bytes = kTilesAt + sizeof(M2LTile) * tiles.size();
      stage = static_cast<char*>(pinned_staging(4096 + bytes));
      char* hs = stage + 4096;
      std::memset(hs, 0, kTilesAt);
      std::memcpy(hs, ldev, sizeof(LevelDev) * h);
      for (int l = 0; l < h; ++l) reinterpret_cast<int64_t*>(hs + kOffAt)[l] = lev[l].off;
      std::memcpy(hs + kTilesAt, tiles.data(), sizeof(M2LTile) * tiles.size());
      char* dev = static_cast<char*>(p->alloc(bytes));
      FMM_HIP_CHECK(hipMemcpyAsync(dev, hs, bytes, hipMemcpyHostToDevice, s));
      p->tiles = reinterpret_cast<M2LTile*>(dev + kTilesAt);
      p->tile_src = static_cast<int*>(p->alloc(sizeof(int) * size_t(p->ntiles) * kSlots * kTileN));
      p->tile_act = static_cast<unsigned char*>(p->alloc(size_t(p->ntiles) * kSlots));
      p->tile_gmask = static_cast<unsigned char*>(p->alloc(size_t(p->ntiles) * kSlots));
      p->tile_nact = static_cast<int*>(p->alloc(sizeof(int) * p->ntiles));
      tile_src_kernel<<<unsigned(p->ntiles), kTileThreads, 0, s>>>(
          p->tiles, p->tgt, reinterpret_cast<const LevelDev*>(dev),
          reinterpret_cast<const int64_t*>(dev + kOffAt), p->ops->slot_t, int(p->ncell_total),
          p->tile_src, p->tile_act, p->tile_gmask, p->tile_nact, stats, p->ops->slot_kid,
          stats + kMaxHeight + 2, stats + kMaxHeight + 1, stats + kMaxHeight + 2 + kOffsets);
      FMM_HIP_CHECK(hipGetLastError());
    }
  }

  // --- statistics ---
  FMM_HIP_CHECK(hipMemcpyAsync(stage, stats, sizeof(unsigned long long) * kStats,
                               hipMemcpyDeviceToHost, s));
  FMM_HIP_CHECK(hipStreamSynchronize(s));
  const unsigned long long* hc = reinterpret_cast<const unsigned long long*>(stage);
  for (int k = 0; k < kOffsets; ++k) p->pairs_by_kid[k] = int64_t(hc[kMaxHeight + 2 + k]);
  p->near_pairs = int64_t(hc[kMaxHeight]);
  p->far_pairs = 0;
  for (int l = 0; l < kMaxHeight; ++l) {
    p->far_pairs_level[l] = int64_t(hc[l]);
    p->far_pairs += int64_t(hc[l]);
  }
  p->active_slots = int64_t(hc[kMaxHeight + 1]);
  p->m2l_groups = int64_t(hc[kMaxHeight + 2 + kOffsets]);
  p->m2l_groups_empty = int64_t(hc[kMaxHeight + 3 + kOffsets]);
  // plans whose tiles leave many 16-target groups without a source at an
  // offset (points on surfaces) take the compressed M2L that skips them
  p->m2l_gskip = p->m2l_groups > 0 && 10 * p->m2l_groups_empty >= p->m2l_groups;
  // The dense M2L skips a group by a branch between its MFMAs, which costs full
  // tiles up to 5% (200,000 particles, height 6, 1% of the tiles' groups
  // without a source, ms skipping and not: order 10 mixed 155.6 and 149.1, fp64
  // 284.8 and 273.2, order 8 mixed 42.2 and 40.2) and pays where they are more:
  // 8% (60,000, height 5) fp64 order 8 8.95 and 9.39, order 9 17.7 and 18.8,
  // order 10 37.3 and 36.4; 28% (200,000 on a sphere, height 7) order 6 6.8 and
  // 8.1.  Of all four groups of a tile, those past its targets included.
  p->dense_gskip = 20 * (4 * p->active_slots - (p->m2l_groups - p->m2l_groups_empty)) >=
                   4 * p->active_slots;
}

// ------------------------------------------------------ mutual pair lists
// The mutual near field (Sec. 5, P2Preduce) visits every pair of distinct
// neighbour leaves once, as (a, near[a][s]) for the forward slots
// s = 14..26 (the offsets after the leaf itself in slot order; slot 26 - s
// is the opposite offset).  Launch (s, c) takes the leaves a of colour c:
// the parity of a's grid coordinate along the first non-zero axis of the
// offset.  Along that axis a and its neighbour differ by one, so their
// parities differ, and no leaf is a's side of one pair and the neighbour's
// side of another in the same launch: the launch's pairs touch disjoint
// leaves.  Flag (2k + c) * nl + a marks leaf a in list (14 + k, c).
__global__ void mutual_flags_kernel(const uint64_t* __restrict__ leaf_keys, int bits,
                                    const int* __restrict__ near, int64_t nl,
                                    int* __restrict__ flags) {
  const int64_t a = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (a >= nl) return;
  int c[3];
  demorton3(leaf_keys[a], bits, c);
  for (int k = 0; k < kMutualSlots; ++k) {
    const int s = kMutualFirstSlot + k;
    const int dx = s / 9 - 1, dy = (s / 3) % 3 - 1;
    const int colour = c[dx != 0 ? 0 : dy != 0 ? 1 : 2] & 1;
    const bool has = near[27 * a + s] >= 0;
    flags[(2 * k) * nl + a] = has && colour == 0;
    flags[(2 * k + 1) * nl + a] = has && colour == 1;
  }
}

// list[scan[i]] = leaf of flag i, for the set flags; then the list bounds
__global__ void mutual_emit_kernel(const int* __restrict__ flags, const int64_t* __restrict__ scan,
                                   int64_t nl, int* __restrict__ list) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= 2 * kMutualSlots * nl) return;
  if (flags[i]) list[scan[i]] = int(i % nl);
}

__global__ void mutual_bounds_kernel(const int* __restrict__ flags,
                                     const int64_t* __restrict__ scan, int64_t nl,
                                     int64_t* __restrict__ off) {
  const int k = threadIdx.x;
  const int64_t m = 2 * kMutualSlots * nl;
  if (k < 2 * kMutualSlots) off[k] = scan[k * nl];
  if (k == 2 * kMutualSlots) off[k] = scan[m - 1] + flags[m - 1];
}

__global__ void int_to_i64_kernel(const int* __restrict__ in, int64_t* __restrict__ out,
                                  int64_t n) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) out[i] = in[i];
}

void build_mutual_lists(fmm_plan_s* p, hipStream_t s) {
  const int64_t nl = p->nleaf, m = 2 * kMutualSlots * nl;
  std::vector<void*> tmp;
  struct TmpGuard {
    std::vector<void*>& v;
    hipStream_t s;
    ~TmpGuard() {
      (void)hipStreamSynchronize(s);
      for (void* q : v) dev_free(q);
    }
  } guard{tmp, s};
  auto talloc = [&](size_t b) {
    void* q = dev_alloc(b);
    tmp.push_back(q);
    return q;
  };
  int* flags = static_cast<int*>(talloc(sizeof(int) * m));
  int64_t* scan = static_cast<int64_t*>(talloc(sizeof(int64_t) * m));
  int64_t* off_d = static_cast<int64_t*>(talloc(sizeof(int64_t) * (2 * kMutualSlots + 1)));
  mutual_flags_kernel<<<grid_for(nl, 256), 256, 0, s>>>(p->lev[p->height - 1].keys,
                                                        p->height - 1, p->near, nl, flags);
  FMM_HIP_CHECK(hipGetLastError());
  int_to_i64_kernel<<<grid_for(m, 256), 256, 0, s>>>(flags, scan, m);
  FMM_HIP_CHECK(hipGetLastError());
  exclusive_scan<int64_t>(scan, scan, m, s, tmp);
  mutual_bounds_kernel<<<1, 64, 0, s>>>(flags, scan, nl, off_d);
  FMM_HIP_CHECK(hipGetLastError());
  int64_t off[2 * kMutualSlots + 1];
  FMM_HIP_CHECK(hipMemcpyAsync(off, off_d, sizeof(off), hipMemcpyDeviceToHost, s));
  FMM_HIP_CHECK(hipStreamSynchronize(s));
  const int64_t total = off[2 * kMutualSlots];
  int* list = static_cast<int*>(p->alloc(sizeof(int) * std::max<int64_t>(total, 1)));
  mutual_emit_kernel<<<grid_for(m, 256), 256, 0, s>>>(flags, scan, nl, list);
  FMM_HIP_CHECK(hipGetLastError());
  p->mutual_list = list;
  for (int k = 0; k <= 2 * kMutualSlots; ++k) p->mutual_off[k] = off[k];
}

}  // namespace fmm
