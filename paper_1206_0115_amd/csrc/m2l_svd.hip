// The compressed M2L kernel (Sec. 2.1.2; operators: get_svd_ops in m2l.hip).
//
// Per far offset t of a tile of 64 targets: X = (S V^T)_t W (rank x columns),
// then Y += U_t X (l^3 x columns), 4 l^3 r flops per (target, source) pair.
//
// One workgroup takes one item: a tile's offsets [ia0, ia1) (a range of them
// where the job splits its tiles), 16 NT of its 64 columns, an M-block of the
// output rows.  Wavefronts 0-3 are producers of X, the others consumers,
// each owning MTW 16-row M-tiles of Y.  In iteration ia the producers write
// X of offset ia to slab buffer ia % 2 while the consumers apply X of offset
// ia - 1 from the other; one barrier ends the iteration.
//
// A producer owns NJ of the item's 16-column N-tiles and, of the 16-row chunks
// of the l^3 contraction, KG of the four K-groups (chunk % 4).  A K-group's
// sum runs over its chunks in order, and X = ((P0 + P1) + P2) + P3 in FP32 and
// (P0 + P2) + (P1 + P3) in FP64: where a wavefront has several groups it adds
// in registers what that order allows, the rest are partial slabs added by
// the consumers, so every split and width gives the same bits (a serving
// batch takes one width for all its plans).  Pairs in FP64 leave two slabs
// where a wavefront has two groups; a third would not fit the LDS at the
// ranks that shape is for.  They are two chunks apart, so that a contraction
// of two chunks (order 3) still feeds both wavefronts.
//
// What bounds it is latency and the order in which wavefronts get at the
// matrix cores, not a memory rate: without reading ahead across offsets the
// matrix cores were busy half of the time and wavefronts waited 40-55% of
// theirs (order 7).  So both roles read ahead through a ring of fragments that is never drained,
// D chunks (producers) or RD fragments (consumers), across passes, offsets
// and the barrier; every load is unconditional (past the last chunk it reads
// on into padding, past the last offset it repeats it), so that a wait is for
// exactly the fragment needed; and a turn of the ring has its addresses
// formed once, so that little else is issued between the MFMAs.  Source rows
// and per-offset data come from LDS tables filled once an item.  M2L before and
// after: 1M cube order 7 3.70 -> 3.43 ms, 469k cube order 10 64.4 -> 54.2,
// 300,000 particles order 8 FP64 1.97 -> 1.56, 10M sphere order 7 8.4 -> 7.1;
// eight producers, and wavefronts that take both roles in turn, were slower
// (order 7: 3.6 and 4.0; order 10: 73 the latter).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "m2l_dev.h"

// register arrays stay in registers only where the lambda is inlined
#define FMM_INLINE __attribute__((always_inline))

namespace fmm {
namespace {

// f(0), f(1), ... f(N - 1) with the index a compile-time constant.
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// Per active offset of an item: the factors' place, the rank chunks, the
// K-steps of the last one, the 16-target groups with a source.
struct SvdMeta {
  int64_t off;
  int s;       // slot
  int nr_nst;  // nr | nst << 16 | gmask << 24
};
constexpr size_t kSvdMetaBytes = sizeof(SvdMeta) * kSlots;
static_assert(kSvdMetaBytes % 16 == 0, "tables stay 16-byte aligned");

struct SvdItem {
  const JobDev* J;
  M2LTile tl;
  int tile, mb, col0, part;
  int ia0, ia1;  // the item's range of the tile's active offsets
};

// How NPW producers split X: NJ of the item's NT N-tiles and KG of the four
// K-groups each, D chunks in flight, RP rank tiles a pass.
template <int NPW_, int NT_, int NJ_, int KG_, int D_, int RP_>
struct Producers {
  static constexpr int NPW = NPW_, NT = NT_, NJ = NJ_, KG = KG_, D = D_, RP = RP_;
  static_assert(NPW * NJ * KG == 4 * NT, "every N-tile and K-group once");
  static_assert(RP <= 5, "the rest of a rank's passes");
};
// Slabs of X per buffer: partial sums the producers cannot add in registers
// in the order X is defined in.
constexpr int svd_slabs(bool fp32, int kg) { return kg == 4 ? 1 : kg == 2 ? (fp32 ? 3 : 2) : 4; }

// Item `it` of the launch; false when its columns hold no target (the same
// for the whole workgroup).
template <int NT>
__device__ inline bool svd_item(const JobDev* __restrict__ jobs, const StepTab* __restrict__ tab,
                                int it, int total, SvdItem& I) {
  constexpr int NC = 16 * NT, NG = 4 / NT;
  const int b = int(gridDim.x) == total ? xcd_run(it, total) : it;
  const int k = step_find(*tab, b);
  const JobDev& J = jobs[tab->job[k]];
  const int local = b - tab->start[k] + tab->first[k];
  I.J = &J;
  const int per_tile = J.nmb * J.m2l_parts;
  I.tile = local / per_tile;
  const int rem = local % per_tile;
  I.part = rem / J.nmb;
  I.mb = rem % J.nmb / NG;
  I.col0 = NC * (rem % J.nmb % NG);
  I.tl = J.tiles[I.tile];
  const int nact = wuni(gld(J.tile_nact + I.tile));
  I.ia0 = int(int64_t(I.part) * nact / J.m2l_parts);
  I.ia1 = int(int64_t(I.part + 1) * nact / J.m2l_parts);
  return I.col0 < I.tl.count;
}

// The item's LDS tables, by all threads (both roles call it).
template <int NT, bool GS>
__device__ inline void svd_fill(const SvdItem& I, SvdMeta* meta, int* src) {
  const JobDev& J = *I.J;
  const unsigned char* act = J.tile_act + int64_t(I.tile) * kSlots + I.ia0;
  const int* kidp = J.slot_kid + I.tl.parity * kSlots;
  const int na = I.ia1 - I.ia0;
  for (int t = threadIdx.x; t < na; t += blockDim.x) {
    const int sl = gld(act + t);
    const int kid = gld(kidp + sl);
    const int nr = gld(J.svd_rpad + kid) >> 4;
    const int nst = (gld(J.svd_rank + kid) - 16 * (nr - 1) + 3) >> 2;
    const int gm = GS ? gld(J.tile_gmask + int64_t(I.tile) * kSlots + I.ia0 + t) : 0xf;
    meta[t] = SvdMeta{gld(J.svd_off + kid), sl, nr | (nst << 16) | (gm << 24)};
  }
  if (src) {
    const int* srcb = J.tile_src + int64_t(I.tile) * kSlots * kTileN + I.col0;
    for (int e = threadIdx.x; e < na * 16 * NT; e += blockDim.x)
      src[e] = gld(srcb + gld(act + e / (16 * NT)) * kTileN + e % (16 * NT));
  }
  __syncthreads();
}

// One fragment (four values a lane) at a uniform address: a scalar base and the
// lane's byte offset.
template <typename T>
__device__ __forceinline__ typename Vec4<T>::type frag(const T* base, unsigned lane_off) {
  typedef typename Vec4<T>::type T4;
  return *(const FMM_GLOBAL T4*)((const FMM_GLOBAL char*)base + lane_off);
}

template <typename T, typename PC, bool GS>
__device__ __forceinline__ void svd_produce(const JobDev* __restrict__ jobs,
                                            const StepTab* __restrict__ tab, SvdMeta* const meta,
                                            int* const srct, T* const slabs, int w) {
  typedef typename Vec4<T>::type T4;
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int NT = PC::NT, NJ = PC::NJ, D = PC::D, RP = PC::RP;
  constexpr int NC = 16 * NT, KG = PC::KG, KS = 4 / KG, NS = svd_slabs(F32, KG);
  static_assert(D % KG == 0, "a ring stage belongs to one K-group");
  static_assert(F32 || KG <= 2, "four FP64 groups in registers are added in pairs");
  const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
  const unsigned lo = lane * unsigned(sizeof(T4));
  const int j0 = w % (NT / NJ) * NJ, s = w / (NT / NJ);
  const int total = step_total(*tab);
  int buf = 0;
  for (int it = blockIdx.x; it < total; it += gridDim.x) {
    SvdItem I;
    if (!svd_item<NT>(jobs, tab, it, total, I)) continue;
    const JobDev& J = *I.J;
    const int KC = J.kc, XS = J.xs, na = I.ia1 - I.ia0;
    const int64_t ld = J.ld;
    const T* __restrict__ Wp = (F32 ? reinterpret_cast<const T*>(J.W32)
                                    : reinterpret_cast<const T*>(J.W)) + 4 * g;
    const T* __restrict__ P1 = (F32 ? reinterpret_cast<const T*>(J.p1_32)
                                    : reinterpret_cast<const T*>(J.p1_64));
    const int* srcg = J.tile_src + int64_t(I.tile) * kSlots * kTileN + I.col0 + 16 * j0 + c16;
    svd_fill<NT, GS>(I, meta, srct);
    // the wavefront's chunks: positions u0 .. u0 + D - 1 of a ring turn are the
    // chunks turn(u0) + step(u); positions from nck on are read (the buffers
    // are padded by kSvdPadChunks) and not used
    auto turn = [&](int u0) FMM_INLINE { return F32 ? u0 / KG * 4 + s * KG : u0 * KS + s; };
    auto step = [](int u) FMM_INLINE { return F32 ? u / KG * 4 + u % KG : u * KS; };
    static_assert(D + 4 * (D / KG) <= kSvdPadChunks, "padding");
    const int nck = F32 ? KC / 4 * KG + min(max(KC % 4 - s * KG, 0), KG)
                        : max(KC - s + KS - 1, 0) / KS;
    const int nckp = (max(nck, 1) + D - 1) / D * D;  // whole ring turns
    T4 rb[D][NJ], ra[D][RP];  // the ring
    // one stage of the turn that starts at b[] and a[]
    auto load = [&](auto u, const T* const* b, const T* const* a) FMM_INLINE {
      static_for<NJ>([&](auto jj) FMM_INLINE {
        rb[u][jj] = gld(reinterpret_cast<const T4*>(b[jj] + 16 * step(u)));
      });
      static_for<RP>([&](auto i) FMM_INLINE { ra[u][i] = frag(a[i] + 256 * step(u), lo); });
    };
    // the wavefront's N-tiles with a source at offset a; the next offset from
    // a on at which there is one
    const int bit = 24 + I.col0 / 16 + j0;
    auto groups = [&](int a) FMM_INLINE {
      return GS ? (wuni(meta[a].nr_nst) >> bit) & ((1 << NJ) - 1) : (1 << NJ) - 1;
    };
    auto next_on = [&](int a) FMM_INLINE {
      if (GS)
        while (a < na && !groups(a)) ++a;
      return a;
    };
    auto row = [&](int a, int jj) FMM_INLINE {
      return Wp + int64_t(srct ? srct[a * NC + 16 * (j0 + jj) + c16]
                               : gld(srcg + wuni(meta[a].s) * kTileN + 16 * jj)) * ld;
    };
    int cur = next_on(0);
    const T* bp[NJ];
    static_for<NJ>([&](auto jj) FMM_INLINE { bp[jj] = Wp; });
    if (cur < na) {
      const int nr = wuni(meta[cur].nr_nst) & 0xffff;
      const T* b0[NJ];
      const T* a0[RP];
      static_for<NJ>([&](auto jj) FMM_INLINE {
        bp[jj] = row(cur, jj);
        b0[jj] = bp[jj] + 16 * turn(0);
      });
      static_for<RP>([&](auto i) FMM_INLINE {
        a0[i] = P1 + wuni(meta[cur].off) + (int64_t(min(int(i), nr - 1)) * KC + turn(0)) * 256;
      });
      static_for<D>([&](auto u) FMM_INLINE { load(u, b0, a0); });
    }
    for (int ia = 0; ia <= na; ++ia) {
      if (ia < na && ia == cur) {
        const int nr = wuni(meta[cur].nr_nst) & 0xffff;
        const T* const a_cur = P1 + wuni(meta[cur].off);
        const int on = groups(cur);
        const int nxt = next_on(cur + 1);
        const int nx = nxt < na ? nxt : cur;  // past the last offset: itself again
        T* const X0 = slabs + (buf * NS * NC + 16 * j0 + c16) * XS;
        const T* bnx[NJ];
        static_for<NJ>([&](auto jj) FMM_INLINE { bnx[jj] = row(nx, jj); });
        for (int i0 = 0; i0 < nr; i0 += RP) {
          const int np = min(RP, nr - i0);
          const bool last = i0 + RP >= nr;
          T4 x[KG][NJ][RP];
          static_for<KG>([&](auto k) FMM_INLINE {
            static_for<NJ>([&](auto jj) FMM_INLINE {
              static_for<RP>([&](auto i) FMM_INLINE { x[k][jj][i] = T4{0, 0, 0, 0}; });
            });
          });
          const T* const a0 = a_cur + int64_t(i0) * KC * 256;
          // the first NP rank tiles' products with stage u, the accumulators
          // taken in turn (a step onto the one just written waits for it)
          auto mul_n = [&](auto u, auto np_c) FMM_INLINE {
            static_for<4>([&](auto st) FMM_INLINE {
              static_for<NJ>([&](auto jj) FMM_INLINE {
                if (!GS || NJ == 1 || ((on >> jj) & 1))
                  static_for<decltype(np_c)::value>([&](auto i) FMM_INLINE {
                    x[u % KG][jj][i] =
                        mfma16x16x4(ra[u][i][int(st)], rb[u][jj][int(st)], x[u % KG][jj][i]);
                  });
              });
            });
          };
          auto mul = [&](auto u) FMM_INLINE {
            if (np == RP) mul_n(u, std::integral_constant<int, RP>{});
            else if (RP == 2 || np == 1) mul_n(u, std::integral_constant<int, 1>{});
            else if (RP > 3 && np == 2) mul_n(u, std::integral_constant<int, 2>{});
            else if (RP > 4 && np == 3) mul_n(u, std::integral_constant<int, 3>{});
            else mul_n(u, std::integral_constant<int, RP - 1>{});
          };
          int u0 = 0;
          const T* bt[NJ];
          const T* at[RP];
          for (; u0 + D < nckp; u0 += D) {
            const int c = turn(u0 + D);
            static_for<NJ>([&](auto jj) FMM_INLINE { bt[jj] = bp[jj] + 16 * c; });
            static_for<RP>([&](auto i) FMM_INLINE {
              at[i] = a0 + (int64_t(min(int(i), np - 1)) * KC + c) * 256;
            });
            static_for<D>([&](auto u) FMM_INLINE {
              mul(u);
              __builtin_amdgcn_sched_barrier(0);  // a stage is free once used
              load(u, bt, at);
            });
          }
          // the last turn reads the next pass's or offset's first chunks
          const int left = (last ? wuni(meta[nx].nr_nst) & 0xffff : nr - i0 - RP) - 1;
          const T* const an = last ? P1 + wuni(meta[nx].off) : a0 + int64_t(RP) * KC * 256;
          static_for<NJ>([&](auto jj) FMM_INLINE {
            bt[jj] = (last ? bnx[jj] : bp[jj]) + 16 * turn(0);
          });
          static_for<RP>([&](auto i) FMM_INLINE {
            at[i] = an + (int64_t(min(int(i), left)) * KC + turn(0)) * 256;
          });
          static_for<D>([&](auto u) FMM_INLINE {
            if (u0 + u < nck) mul(u);
            __builtin_amdgcn_sched_barrier(0);
            load(u, bt, at);
          });
          // D rows: FP32 item r -> row 4g + r, FP64 item r -> row 4r + g
          static_for<RP>([&](auto i) FMM_INLINE {
            if (i >= np) return;
            static_for<NJ>([&](auto jj) FMM_INLINE {
              auto put = [&](int slab, const T4& v) FMM_INLINE {
                T* const xr = X0 + (slab * NC + 16 * jj) * XS + 16 * (i0 + i);
                if (F32) {
                  *reinterpret_cast<T4*>(xr + 4 * g) = v;
                } else {
#pragma unroll
                  for (int r = 0; r < 4; ++r) xr[4 * r + g] = v[r];
                }
              };
              if constexpr (KG == 4) {
                put(0, ((x[0][jj][i] + x[1][jj][i]) + x[2][jj][i]) + x[3][jj][i]);
              } else if constexpr (KG == 2) {
                if (!F32 || s == 0) {
                  put(s, x[0][jj][i] + x[1][jj][i]);
                } else {
                  put(1, x[0][jj][i]);
                  put(2, x[1][jj][i]);
                }
              } else {
                put(s, x[0][jj][i]);
              }
            });
          });
        }
        static_for<NJ>([&](auto jj) FMM_INLINE { bp[jj] = bnx[jj]; });
        cur = nxt;
      }
      buf ^= 1;
      __syncthreads();
    }
  }
}

template <typename T, int MTW, int NCW, typename PC, bool GS>
__device__ __forceinline__ void svd_consume(const JobDev* __restrict__ jobs,
                                            const StepTab* __restrict__ tab, SvdMeta* const meta,
                                            int* const srct, const T* const slabs, int wg) {
  typedef typename Vec4<T>::type T4;
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int NT = PC::NT, NC = 16 * NT, NS = svd_slabs(F32, PC::KG);
  // U fragments in flight; a divisor of MTW, so that a ring stage is an M-tile
  // (two where eight M-tiles' accumulators leave no registers for more)
  constexpr int RD = MTW % 4 == 0 ? (MTW == 8 && (F32 ? NT == 4 : PC::RP > 3) ? 2 : 4) : MTW % 3 == 0 ? 3 : MTW;
  static_assert(MTW % RD == 0, "ring");
  const int lane = threadIdx.x & 63, g = lane >> 4, c16 = lane & 15;
  const unsigned lo = lane * unsigned(sizeof(T4));
  const int total = step_total(*tab);
  int buf = 0;
  for (int it = blockIdx.x; it < total; it += gridDim.x) {
    SvdItem I;
    if (!svd_item<NT>(jobs, tab, it, total, I)) continue;
    const JobDev& J = *I.J;
    const int MT = wuni(J.mt), XS = wuni(J.xs), na = I.ia1 - I.ia0;
    const int64_t ld = J.ld;
    const int mt0 = (I.mb * NCW + wg) * MTW;
    const int nmt = mt0 < MT ? min(MTW, MT - mt0) : 0;
    const T* __restrict__ P2 = (F32 ? reinterpret_cast<const T*>(J.p2_32)
                                    : reinterpret_cast<const T*>(J.p2_64));
    T4 acc[MTW][NT];
    auto clear = [&]() FMM_INLINE {
      static_for<MTW>([&](auto i) FMM_INLINE {
        static_for<NT>([&](auto j) FMM_INLINE { acc[i][j] = T4{0, 0, 0, 0}; });
      });
    };
    clear();
    bool folded = false;
    svd_fill<NT, GS>(I, meta, srct);
    const int fold_every = wuni(J.fold_every);
    // GS, order 10 in FP64: the next offset from a on at which an N-tile of the
    // item has a source, so that the ring does not read the fragments of those
    // without (100,000 on a sphere, height 7: M2L 24.8 -> 23.6 ms; at low orders
    // the chain of table reads costs more: order 3 212 -> 230 us)
    constexpr bool SKIP = GS && !F32 && MTW == 8;
    auto next_on = [&](int a) FMM_INLINE {
      if (SKIP)
        while (a < na && !((wuni(meta[a].nr_nst) >> (24 + I.col0 / 16)) & ((1 << NT) - 1))) ++a;
      return a;
    };
    int cur = next_on(0);
    T4 ring[RD];
    if (nmt > 0 && cur < na) {
      const int nr = wuni(meta[cur].nr_nst) & 0xffff;
      const T* const a2 = P2 + wuni(meta[cur].off) + int64_t(mt0) * nr * 256;
      static_for<RD>([&](auto i) FMM_INLINE {
        ring[i] = frag(a2 + int64_t(min(int(i), nmt - 1)) * nr * 256, lo);
      });
    }
    for (int ia = 0; ia <= na; ++ia) {
      const int ic = ia - 1;
      if (ia > 0 && nmt > 0 && (!SKIP || ic == cur)) {
        // phase 2 of offset ia - 1 from the buffer the producers filled
        cur = next_on(ia);
        const int inx = cur < na ? cur : ic;  // past the last offset: itself again
        const int nrs = wuni(meta[ic].nr_nst);
        const int nr = nrs & 0xffff, nst = (nrs >> 16) & 0xff;  // rank chunks; K-steps of the last
        const int gon = nrs >> (24 + I.col0 / 16);
        const T* const X = slabs + ((buf ^ 1) * NS * NC + c16) * XS + 4 * g;
        const T* const a2 = P2 + wuni(meta[ic].off) + int64_t(mt0) * nr * 256;
        const int nrn = wuni(meta[inx].nr_nst) & 0xffff;
        const T* const a2n = P2 + wuni(meta[inx].off) + int64_t(mt0) * nrn * 256;
        for (int c = 0; c < nr; ++c) {
          T4 bv[NT];
          static_for<NT>([&](auto j) FMM_INLINE {
            bv[j] = T4{0, 0, 0, 0};
            if (GS && !((gon >> j) & 1)) return;
            auto part = [&](int k) FMM_INLINE {
              return *reinterpret_cast<const T4*>(X + (k * NC + 16 * j) * XS + 16 * c);
            };
            T4 v = part(0);
            if constexpr (!F32 && NS == 4) {
              v = (v + part(2)) + (part(1) + part(3));
            } else {
              static_for<NS - 1>([&](auto k) FMM_INLINE { v += part(k + 1); });
            }
            bv[j] = v;
          });
          const bool more = c + 1 < nr;
          // where the ring reads on past this chunk's last M-tile
          const T* const an = more ? a2 + int64_t(c + 1) * 256 : a2n;
          const int64_t sn = int64_t(more ? nr : nrn) * 256;
          // each accumulator takes the K-steps in order; the steps past the
          // kept rank (zeros in both operands) are skipped
          const int ns = more ? 4 : nst;
#pragma unroll
          for (int i = 0; i < MTW; ++i) {
            const T4 av = ring[i % RD];
            if (i < nmt) {
#pragma unroll
              for (int st = 0; st < 4; ++st) {
                if (st >= ns) continue;
#pragma unroll
                for (int j = 0; j < NT; ++j)
                  if (!GS || ((gon >> j) & 1)) acc[i][j] = mfma16x16x4(av[st], bv[j][st], acc[i][j]);
              }
            }
            __builtin_amdgcn_sched_barrier(0);  // a stage is free once used
            ring[i % RD] = frag(
                i + RD < MTW ? a2 + (int64_t(min(i + RD, nmt - 1)) * nr + c) * 256
                             : an + min(i + RD - MTW, nmt - 1) * sn, lo);
          }
        }
      }
      if (ia > 0 && nmt > 0) {
        if (F32 && ((ic + 1) % fold_every == 0 || ic == na - 1)) {
          // fold into this item's rows of Loc (scaled; the first fold
          // stores, later ones add): no other workgroup touches these rows
          const double sc = J.scale[I.tl.level];
          static_for<NT>([&](auto j) FMM_INLINE {
            const int col = I.col0 + 16 * j + c16;
            if (col < I.tl.count) {
              double* out = m2l_out_row(J, I.part, gld(J.tgt + I.tl.first + col));
              static_for<MTW>([&](auto i) FMM_INLINE {
                if (i >= nmt) return;
                d4* o = reinterpret_cast<d4*>(out + 16 * (mt0 + i) + 4 * g);  // rows 4g..4g+3
                d4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = sc * double(acc[i][j][r]);
                if (folded) v += gld(o);
                gst(o, v);
              });
            }
          });
          clear();
          folded = true;
        }
      }
      buf ^= 1;
      __syncthreads();
    }
    if (nmt == 0 || (F32 && folded)) continue;
    const double sc = J.scale[I.tl.level];
    static_for<NT>([&](auto j) FMM_INLINE {
      const int col = I.col0 + 16 * j + c16;
      if (col >= I.tl.count) return;
      double* out = m2l_out_row(J, I.part, gld(J.tgt + I.tl.first + col));
      static_for<MTW>([&](auto i) FMM_INLINE {
        if (i >= nmt) return;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          gst(out + 16 * (mt0 + i) + (F32 ? 4 * g + r : 4 * r + g), sc * double(acc[i][j][r]));
      });
    });
  }
}

// GS (plans with many empty 16-target groups): the N-tiles whose columns have
// no source at an offset, all products zero, are skipped by both roles.
template <typename T, int MTW, int NCW, typename PC, bool GS>
__global__ __launch_bounds__(64 * (PC::NPW + NCW), NCW == 4 && MTW < 6 ? 4 : (PC::NPW + NCW) / 4) void m2l_svd_kernel(
    const JobDev* __restrict__ jobs, const StepTab* __restrict__ tab, int staged) {
  // the offset table, the source rows (where they fit) and two sets of slabs
  extern __shared__ __align__(16) unsigned char lds_raw[];
  SvdMeta* const meta = reinterpret_cast<SvdMeta*>(lds_raw);
  int* const src = reinterpret_cast<int*>(lds_raw + kSvdMetaBytes);
  T* const slabs = reinterpret_cast<T*>(lds_raw + kSvdMetaBytes +
                                        (staged ? sizeof(int) * kSlots * 16 * PC::NT : 0));
  // the role is uniform per wavefront: a scalar branch, no lane masking
  const int wave = wuni(int(threadIdx.x >> 6));
  if (wave < PC::NPW) {
    // producers issue ahead of the consumers on their SIMD (30M-particle
    // order-10 cube: M2L 4255 -> 4223 ms; raising the consumers instead costs
    // 1.6%)
    __builtin_amdgcn_s_setprio(1);
    svd_produce<T, PC, GS>(jobs, tab, meta, staged ? src : nullptr, slabs, wave);
  } else {
    svd_consume<T, MTW, NCW, PC, GS>(jobs, tab, meta, staged ? src : nullptr, slabs,
                                     wave - PC::NPW);
  }
}

constexpr size_t kSvdLdsMax = 160 * 1024;  // LDS per workgroup on gfx950

// One kernel: consumers, M-tiles each, and its producers' split.
struct SvdShape {
  int ncw, mtw, npw, nt, kg;
  const void* fn[2];  // without and with the group skip
};

template <typename T, int MTW, int NCW, typename PC>
SvdShape svd_make() {
  return {NCW, MTW, PC::NPW, PC::NT, PC::KG,
          {reinterpret_cast<const void*>(&m2l_svd_kernel<T, MTW, NCW, PC, false>),
           reinterpret_cast<const void*>(&m2l_svd_kernel<T, MTW, NCW, PC, true>)}};
}

int svd_kc(int order) { return (order * order * order + 15) / 16; }

// The shape of an order at a slab stride of xs and nt N-tiles an item: four
// producers and, up to 16 M-tiles (order 6), four consumers, two such
// workgroups to a CU; eight above, in as many M-blocks of up to 8 M-tiles a
// consumer as the rows need (each M-block repeats phase 1).  The producers'
// split is the fastest measured (order 7 and 8: 1M and 250,000 particles,
// order 10: the 469k cube; M2L in ms):
//   FP32, 64 columns    KG = 1, D = 2   KG = 2, D = 4   KG = 4, D = 4
//     order 7                3.43            3.45            3.68
//     order 8                6.18            5.73            5.97
//     order 10               71.2            67.8            54.2
// At orders 11 and 12, whose rows take two M-blocks, 32-column items with
// KG = 1 are ahead of 64-column ones (60,000 particles, order 12: 6.3 against
// 7.7).  FP64 with KG = 1 needs four slabs of 32 columns: where they do not
// fit the LDS, KG = 2.
SvdShape svd_shape(int mt, bool fp32, int xs, int nt, bool gskip) {
  const int mb = (mt + 63) / 64;
  const int w = (mt + 8 * mb - 1) / (8 * mb);
  // whether four partial slabs of 64 FP32 or 32 FP64 columns fit the LDS
  const bool four = size_t(2048) * xs + kSvdMetaBytes <= kSvdLdsMax;
  if (fp32) {
    if (mt <= 4)
      return nt == 2 ? svd_make<float, 1, 4, Producers<4, 2, 1, 2, 2, 1>>()
                     : svd_make<float, 1, 4, Producers<4, 1, 1, 1, 1, 1>>();
    if (mt <= 8)
      return nt == 2 ? svd_make<float, 2, 4, Producers<4, 2, 1, 2, 2, 2>>()
                     : svd_make<float, 2, 4, Producers<4, 1, 1, 1, 2, 2>>();
    // four partial slabs (and the tables) of two workgroups in a CU's LDS, or
    // two slabs each: at ranks past that one workgroup a CU would be left
    // (1/r^2, order 6: 300,000 in a cube 2807 -> 2336 us, on a sphere 1714 -> 1330)
    if (mt <= 16 && nt == 2 && 1024 * size_t(xs) + 27 * 1024 > kSvdLdsMax / 2)
      return svd_make<float, 4, 4, Producers<4, 2, 1, 2, 2, 2>>();
    if (mt <= 16)
      return nt == 2 ? svd_make<float, 4, 4, Producers<4, 2, 2, 1, 2, 2>>()
                     : svd_make<float, 4, 4, Producers<4, 1, 1, 1, 2, 2>>();
    if (nt == 4) {
      if (w <= 3 && four) return svd_make<float, 3, 8, Producers<4, 4, 4, 1, 2, 2>>();
      if (w <= 4 && four) return svd_make<float, 4, 8, Producers<4, 4, 2, 2, 4, 2>>();
      if (w <= 4) return svd_make<float, 4, 8, Producers<4, 4, 1, 4, 4, 2>>();
      // order 9: at ranks up to 48 full tiles are faster with two groups a
      // wavefront (300,000, height 6, tolerance 1e-7: M2L 7.07 -> 6.72 ms),
      // surfaces not (300,000, height 7: 3.84 -> 4.00), nor higher ranks
      if (w <= 6 && !gskip && xs <= m2l_svd_xs(48, true))
        return svd_make<float, 6, 8, Producers<4, 4, 2, 2, 4, 2>>();
      if (w <= 6) return svd_make<float, 6, 8, Producers<4, 4, 1, 4, 4, 2>>();
      return svd_make<float, 8, 8, Producers<4, 4, 1, 4, 4, 2>>();
    }
    if (nt == 2) {
      if (w <= 4) return svd_make<float, 4, 8, Producers<4, 2, 2, 1, 2, 2>>();
      if (w <= 6) return svd_make<float, 6, 8, Producers<4, 2, 2, 1, 3, 2>>();
      if (w == 7) return svd_make<float, 7, 8, Producers<4, 2, 2, 1, 3, 2>>();
      return svd_make<float, 8, 8, Producers<4, 2, 2, 1, 3, 2>>();
    }
    if (w <= 4) return svd_make<float, 4, 8, Producers<4, 1, 1, 1, 4, 2>>();
    if (w <= 6) return svd_make<float, 6, 8, Producers<4, 1, 1, 1, 4, 2>>();
    if (w == 7) return svd_make<float, 7, 8, Producers<4, 1, 1, 1, 4, 2>>();
    return svd_make<float, 8, 8, Producers<4, 1, 1, 1, 4, 2>>();
  }
  if (mt <= 4)
    return nt == 2 ? svd_make<double, 1, 4, Producers<4, 2, 1, 2, 2, 1>>()
                   : svd_make<double, 1, 4, Producers<4, 1, 1, 1, 1, 1>>();
  if (nt == 2) {
    if (mt <= 8) return svd_make<double, 2, 4, Producers<4, 2, 1, 2, 2, 2>>();
    if (mt <= 16)
      return four ? svd_make<double, 2, 8, Producers<4, 2, 2, 1, 2, 2>>()
                  : svd_make<double, 2, 8, Producers<4, 2, 1, 2, 2, 2>>();
    if (w <= 3 && four) return svd_make<double, 3, 8, Producers<4, 2, 2, 1, 2, 2>>();
    if (w <= 4 && four) return svd_make<double, 4, 8, Producers<4, 2, 2, 1, 2, 2>>();
    if (w <= 4) return svd_make<double, 4, 8, Producers<4, 2, 1, 2, 2, 2>>();
    return svd_make<double, 6, 8, Producers<4, 2, 1, 2, 2, 2>>();
  }
  if (mt <= 8) return svd_make<double, 2, 4, Producers<4, 1, 1, 1, 2, 2>>();
  if (mt <= 16) return svd_make<double, 2, 8, Producers<4, 1, 1, 1, 2, 2>>();
  if (w <= 4) return svd_make<double, 4, 8, Producers<4, 1, 1, 1, 2, 2>>();
  if (w <= 6) return svd_make<double, 6, 8, Producers<4, 1, 1, 1, 2, 2>>();
  if (w == 7) return svd_make<double, 7, 8, Producers<4, 1, 1, 1, 2, 3>>();
  // order 10: with 16 columns a pass over the contraction gathers them again,
  // so five rank tiles a pass and one chunk ahead where the ranks fill them
  // (100,000 particles, height 6, M2L ms at ranks up to 112: 36.7, and 42.6 with
  // three tiles and two chunks ahead; up to 80 30.2 and 33.7, up to 64 26.2 and
  // 28.6), three at ranks up to 48 (20.9, and 21.9 with five; up to 32 15.6 and
  // 18.5)
  if (xs <= m2l_svd_xs(48, false)) return svd_make<double, 8, 8, Producers<4, 1, 1, 1, 2, 3>>();
  return svd_make<double, 8, 8, Producers<4, 1, 1, 1, 1, 5>>();
}

size_t svd_lds(const SvdShape& sh, int xs, bool fp32, bool staged) {
  return kSvdMetaBytes + (staged ? sizeof(int) * kSlots * 16 * sh.nt : 0) +
         size_t(2) * svd_slabs(fp32, sh.kg) * 16 * sh.nt * xs *
             (fp32 ? sizeof(float) : sizeof(double));
}

}  // namespace

// N-tiles per item of the widest shape of an order: 64 columns (FP32) or 32,
// 32 or 16 where the rows take two M-blocks or 8 M-tiles a consumer do not
// leave the registers.
static int svd_widest(int mt, bool fp32) {
  if (fp32) return mt <= 16 || mt > 64 ? 2 : 4;
  return (mt + 63) / 64 * 48 >= mt ? 2 : 1;
}

// N-tiles per item: the widest shape reads each operator fragment for the most
// columns, but a plan of few tiles then leaves CUs idle or ends on a partly
// empty round.  Half the columns take 0.62 of an item's time (order 7 to 10;
// 0.8 below, where an item's fixed work weighs more: points on spheres, order
// 3, 30,000 at height 6 117 -> 107 us, 100,000 at height 7 317 -> 220), so the
// fewest rounds in those units win (20,000 particles, height 4, order
// 7: 64, 32, 16 columns 379, 238, 157 us; 60,000, height 5: 515, 608, 743).
// Every column's sums are the same in each shape, in both precisions.
int64_t m2l_svd_slots(int mt, bool fp32, int cus) {
  return int64_t(mt <= (fp32 ? 16 : 8) ? 2 : 1) * std::max(1, cus);
}

int m2l_svd_nt(int order, bool fp32, int64_t tile_parts, int cus) {
  const int mt = svd_kc(order);
  const int widest = svd_widest(mt, fp32);
  const int64_t slots = m2l_svd_slots(mt, fp32, cus);
  int best = widest;
  double best_cost = 0.0, item = 1.0;
  for (int nt = widest; nt >= 1; nt /= 2, item *= mt <= 16 ? 0.8 : 0.62) {
    const int64_t items = tile_parts * m2l_svd_nmb(mt, fp32, nt);
    const double cost = double((items + slots - 1) / slots) * item;
    if (nt == widest || cost < 0.95 * best_cost) {
      best = nt;
      best_cost = cost;
    }
  }
  return best;
}

int m2l_svd_nmb(int mt, bool fp32, int nt) {
  const SvdShape sh = svd_shape(mt, fp32, 0, nt, false);
  return (mt + sh.ncw * sh.mtw - 1) / (sh.ncw * sh.mtw) * (4 / nt);
}

// Slab row stride: the padded rank plus 16 bytes, so that consecutive target
// columns start 16 bytes apart modulo the LDS banks.
int m2l_svd_xs(int rmax_pad, bool fp32) { return rmax_pad + (fp32 ? 4 : 2); }

// The rule of the offset ranges, and of the ranks that are refused.  Both
// follow the item shape they were set with (32 FP32 or 16 FP64 columns, whole
// FP32 tiles or 32 FP64 columns at orders 7 to 9 where four partial slabs fit
// the LDS), whatever shape runs: a rank's refusal is part of the interface,
// and ranges that stay where they are keep the order of the FP32 sums.  The
// latter is a choice; ranges by the shape that runs are not tried yet.
static int range_nt(int mt, bool fp32, int xs) {
  const int base = fp32 ? 2 : 1, full = 2 * base;
  const size_t need = size_t(2) * 4 * 16 * full * xs * (fp32 ? 4 : 8) + kSvdMetaBytes;
  return mt > 16 && mt <= 48 && need <= kSvdLdsMax ? full : base;
}

size_t m2l_svd_lds_need(int order, bool fp32, int xs) {
  return size_t(2) * 4 * 16 * range_nt(svd_kc(order), fp32, xs) * xs * (fp32 ? 4 : 8) +
         kSvdMetaBytes;
}

void m2l_svd_ranges(int order, bool fp32, int xs, int cus, int* items, int* slots) {
  const int mt = svd_kc(order);
  const int rows = mt <= 24 ? 4 * 6 : mt <= 64 ? mt : 64;  // M-tiles of an item
  *items = (mt + rows - 1) / rows * (4 / range_nt(mt, fp32, xs));
  const bool small = mt <= 24 && range_nt(mt, fp32, xs) == (fp32 ? 2 : 1);
  const int fit = int(kSvdLdsMax / m2l_svd_lds_need(order, fp32, xs));
  *slots = std::max(1, std::min(small ? 2 : 1, fit)) * std::max(1, cus);
}

void launch_m2l_svd_step(int order, bool fp32, const JobDev* jobs, const StepTab* tab, int grid,
                         int xs, int nt, hipStream_t s, bool gskip) {
  const SvdShape sh = svd_shape(svd_kc(order), fp32, xs, nt, gskip);
  // the source rows in LDS where they fit, and not at the cost of a CU's second
  // workgroup (FP64 order 5 at ranks up to 64: 60,000 on a sphere, height 6, M2L
  // 787 us staged, 600 not; at ranks that leave room for both staged is ahead)
  const bool two = sh.ncw == 4 && svd_lds(sh, xs, fp32, false) <= kSvdLdsMax / 2;
  int staged = svd_lds(sh, xs, fp32, true) <= kSvdLdsMax / (two ? 2 : 1) ? 1 : 0;
  const size_t lds = svd_lds(sh, xs, fp32, staged != 0);
  void* args[] = {&jobs, &tab, &staged};
  FMM_HIP_CHECK(hipLaunchKernel(sh.fn[gskip ? 1 : 0], dim3(grid), dim3(64 * (sh.npw + sh.ncw)),
                                args, lds, s));
  FMM_HIP_CHECK(hipGetLastError());
}

}  // namespace fmm
