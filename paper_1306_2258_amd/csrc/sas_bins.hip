// The binned form of the type-sorted sums: see sas_bins.hpp for the method.
//
//   plan     (after the pack's type sort) per structure the number of bins
//            from the bounding box's diagonal, its place in the pool, and per
//            type pair the work items: 64 lane-side atoms by up to 64 swept ones;
//   bins     one work-group of 16 waves per CU takes a contiguous range of
//            the items, keeps the bins of the type pairs in its range in LDS
//            and adds every pair to them by LDS atomics;
//   sums     bins to weights at six nodes each, sinc at the nodes in FP64, the
//            form factors and the sum over bins and type pairs.
#include "sas_bins.hpp"

#include <hip/hip_runtime.h>

#include <algorithm>

#include "sas_bins_device.hpp"
#include "sas_device.hpp"
#include "sas_reduce.hpp"
#include "sas_schedule.hpp"

namespace sas {

__global__ __launch_bounds__(256) void k_bins_plan(BinArgs b, DescView sd, const int32_t* __restrict__ toff) {
  bins_plan(b, sd, toff);
}

hipError_t launch_bins_plan(const BinArgs& b, const DescView& sd, const int32_t* toff, hipStream_t st) {
  hipLaunchKernelGGL(k_bins_plan, dim3(1), dim3(256), 0, st, b, sd, toff);
  return hipGetLastError();
}

// One (structure, type pair, window) of a work-group's current range.
struct BinSeg {
  int64_t item0;     // its first item in this pass
  int64_t pool;      // first bin of the window in the pool
  int32_t k0;        // item0's index inside the window
  int32_t a0, na, b0, nb, diag;
  int32_t lds, bins; // first bin in LDS, bins of the window
  int32_t win0;      // first bin of the window (0 when there is one window)
  int32_t windowed;
};

// The words of one LDS bin, decoded to the six integer sums.
struct BinSums {
  long long m[kBinMoments];
};

__device__ __forceinline__ BinSums decode_bin(unsigned long long wa, unsigned long long wb, unsigned long long wc) {
  constexpr unsigned long long kA = (1ull << (32 + kBinCountShift)) + kBinMagicBits;
  constexpr unsigned long long kB = (static_cast<unsigned long long>(kBinMagicBits << kBinShift5) << 32) + kBinMagicBits;
  constexpr unsigned long long kC = (static_cast<unsigned long long>(kBinMagicBits << kBinShift4) << 32) + kBinMagicBits;
  BinSums r;
  // (the remaining field is below 2^41 in magnitude, half a count's worth)
  const unsigned long long cnt = static_cast<unsigned long long>(static_cast<double>(wa) / static_cast<double>(kA) + 0.5);
  r.m[0] = static_cast<long long>(cnt);
  r.m[1] = static_cast<long long>(wa - cnt * kA);
  const unsigned long long tb = wb - cnt * kB, tc = wc - cnt * kC;
  constexpr int kLowB = 32 + kBinShift5, kLowC = 32 + kBinShift4;
  r.m[2] = static_cast<long long>(tb << (64 - kLowB)) >> (64 - kLowB);
  r.m[5] = static_cast<long long>(tb - static_cast<unsigned long long>(r.m[2])) >> kLowB;
  r.m[3] = static_cast<long long>(tc << (64 - kLowC)) >> (64 - kLowC);
  r.m[4] = static_cast<long long>(tc - static_cast<unsigned long long>(r.m[3])) >> kLowC;
  return r;
}

// Adds the LDS bins with at least `least` pairs to the pool and clears them.
// A group of R consecutive lanes holds the R copies of one bin.
__device__ __forceinline__ void empty_bins(unsigned long long* h, const BinSeg* seg, int nseg, int nbins, int logR,
                                           unsigned long long least, unsigned long long* __restrict__ pool) {
  const int total = nbins << logR;
  const unsigned long long below = least << (32 + kBinCountShift);
  for (int k0 = 0; k0 < total; k0 += kBinThreads) {
    const int k = k0 + threadIdx.x;
    const unsigned long long wa = k < total ? h[3 * k] : 0;
    const bool full = wa >= below && wa != 0;
    if (!__any(full)) continue;
    BinSums v{};
    if (full) {
      v = decode_bin(wa, h[3 * k + 1], h[3 * k + 2]);
      h[3 * k] = h[3 * k + 1] = h[3 * k + 2] = 0;
    }
    for (int off = 1; off < (1 << logR); off <<= 1) {
#pragma unroll
      for (int c = 0; c < kBinMoments; ++c) v.m[c] += __shfl_xor(v.m[c], off, kWave);
    }
    const int bin = k >> logR, copy = k & ((1 << logR) - 1);
    if (k < total && v.m[0] != 0) {
      int lo = 0, hi = nseg - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (seg[mid].lds <= bin)
          lo = mid;
        else
          hi = mid - 1;
      }
      unsigned long long* to = pool + (seg[lo].pool + (bin - seg[lo].lds)) * kBinMoments;
#pragma unroll
      for (int c = 0; c < kBinMoments; ++c)
        if ((c & ((1 << logR) - 1)) == copy)
          __hip_atomic_fetch_add(to + c, static_cast<unsigned long long>(v.m[c]), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// One item: the lane's atom against the swept atoms [j0, j1).
// What bounds it: per pair ten FP64 instructions, two transcendental and about
// twenty FP32 or integer ones, and three 64-bit LDS atomics, which random
// bins serve at about six lanes per cycle and CU (nine from 16 copies of
// each bin): the vector pipes and LDS take about the same time.
// Each pair's atomics are issued right after its arithmetic: with a batch's
// twelve together at its end the waves fell into step, LDS and vector pipes in
// turn idle (rod, 1.25e9 pairs: 2.44 ms).
// The swept atoms come through the scalar cache, four at a time.  Scalar loads
// and LDS operations share one wait counter, so a batch's loads are issued as
// soon as the last one's coordinates are used up, and waited for before the
// last pair's atomics.
constexpr int kBinBatch = 4;

struct PairWords {
  uint32_t at, f1, f2, f3, f4, f5;
};

// MASKED: pairs outside [0, count), not above lane_min, or outside the window
// go to the lane's own spare words past the last bin.
template <bool MASKED>
__device__ __forceinline__ PairWords pair_words(double s, int k, uint32_t lane_base, uint32_t bin_bytes, int count,
                                                int lane_min, int win0, uint32_t bins, uint32_t spare) {
  const float magic = 0x1.8p+23f;
  PairWords p;
  const float fb = __builtin_truncf(__builtin_amdgcn_sqrtf(static_cast<float>(s)));
  const float tc = fb + 0.5f;
  const double tcd = static_cast<double>(tc);
  const float d = static_cast<float>(fma(-tcd, tcd, s));
  const float u = d * __builtin_amdgcn_rcpf(tc);
  const float u2 = u * u, u3 = u2 * u, u4 = u2 * u2, u5 = u4 * u;
  p.f1 = __float_as_uint(fmaf(u, static_cast<float>(1 << kBinBits1), magic));
  p.f2 = __float_as_uint(fmaf(u2, static_cast<float>(1 << kBinBits2), magic));
  p.f3 = __float_as_uint(fmaf(u3, static_cast<float>(1 << kBinBits3), magic));
  p.f4 = __float_as_uint(fmaf(u4, static_cast<float>(1 << kBinBits4), magic)) << kBinShift4;
  p.f5 = __float_as_uint(fmaf(u5, static_cast<float>(1 << kBinBits5), magic)) << kBinShift5;
  if (MASKED) {
    const uint32_t bin = static_cast<uint32_t>(static_cast<int>(fb) - win0);
    p.at = bin < bins && k < count && k > lane_min ? __umul24(bin, bin_bytes) + lane_base : spare;
  } else {
    p.at = __umul24(static_cast<uint32_t>(fb), bin_bytes) + lane_base;
  }
  return p;
}

__device__ __forceinline__ void deposit(unsigned char* hb, const PairWords& p) {
  auto* to = reinterpret_cast<unsigned long long*>(hb + p.at);
  atomicAdd(to, (1ull << (32 + kBinCountShift)) | p.f1);
  atomicAdd(to + 1, (static_cast<unsigned long long>(p.f5) << 32) | p.f2);
  atomicAdd(to + 2, (static_cast<unsigned long long>(p.f4) << 32) | p.f3);
}

template <bool MASKED>
__device__ __forceinline__ void sweep(const double* __restrict__ xs, unsigned char* hb, const BinSeg& sg, int i, int j0,
                                      int j1, bool diag, uint32_t lane_base, uint32_t bin_bytes) {
  using ConstDouble = const __attribute__((address_space(4))) double;
  ConstDouble* xj = (ConstDouble*)(xs + 3 * (static_cast<int64_t>(sg.b0) + j0));
  const double* pi = xs + 3 * (static_cast<int64_t>(sg.a0) + i);
  const double xi = pi[0], yi = pi[1], zi = pi[2];
  const uint32_t spare = 24u * (kBinCap + threadIdx.x % kWave);
  double cj[3 * kBinBatch];
#pragma unroll
  for (int k = 0; k < 3 * kBinBatch; ++k) cj[k] = xj[k];
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
#pragma unroll 1
  for (int j = j0; j < j1; j += kBinBatch) {
    double s[kBinBatch];
#pragma unroll
    for (int k = 0; k < kBinBatch; ++k) {
      const double dx = xi - cj[3 * k], dy = yi - cj[3 * k + 1], dz = zi - cj[3 * k + 2];
      s[k] = fma(dz, dz, fma(dy, dy, dx * dx));
    }
    __builtin_amdgcn_sched_barrier(0);
    // (rows past the end are other segments' or the array's padding)
    xj += 3 * kBinBatch;
#pragma unroll
    for (int k = 0; k < 3 * kBinBatch; ++k) cj[k] = xj[k];
#pragma unroll
    for (int k = 0; k < kBinBatch; ++k) {
      const PairWords p =
          pair_words<MASKED>(s[k], k, lane_base, bin_bytes, j1 - j, diag ? i - j : -1, sg.win0, sg.bins, spare);
      __builtin_amdgcn_sched_barrier(0);
      if (k == kBinBatch - 1) {
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
      }
      deposit(hb, p);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

__global__ __launch_bounds__(kBinThreads) void k_bins(BinArgs b) {
  __shared__ unsigned long long h[(kBinCap + kWave) * 3];
  __shared__ BinSeg seg[kBinSegs];
  __shared__ int32_t below, nseg_s, bins_s, big_s, next_s;
  __shared__ int64_t end_s;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int64_t items = b.meta->items;
  const int64_t w1 = items * (blockIdx.x + 1) / gridDim.x;
  int64_t w = items * blockIdx.x / gridDim.x;
  if (w >= w1) return;
  const int E = b.S * b.TP;
  // the entry that holds item w: every thread counts entries that start at or
  // before it (they are in item order; an empty one shares the next one's start)
  if (tid == 0) below = 0;
  __syncthreads();
  {
    int mine = 0;
    for (int e = tid; e < E; e += kBinThreads) mine += b.entries[e].item0 <= w;
    for (int off = kWave / 2; off > 0; off >>= 1) mine += __shfl_down(mine, off, kWave);
    if (lane == 0) atomicAdd(&below, mine);
  }
  __syncthreads();
  int e0 = below - 1;
  while (w < w1) {
    // the pass: as many consecutive type pairs as fit in LDS, by the first wave
    if (wave == 0) {
      const int e = e0 + lane;
      BinEntry en{};
      int64_t next = w1;
      if (e < E) {
        en = b.entries[e];
        next = b.entries[e + 1].item0;
      }
      int64_t s0 = en.item0 > w ? en.item0 : w;
      int64_t s1 = next < w1 ? next : w1;
      bool live = e < E && s0 < s1;
      const bool split = live && en.nbins > kBinCap;
      int win = 0;
      int32_t bins = live ? en.nbins : 0;
      if (split) {
        win = static_cast<int>((s0 - en.item0) / en.base);
        const int64_t we = en.item0 + static_cast<int64_t>(win + 1) * en.base;
        s1 = s1 < we ? s1 : we;
        bins = min(en.nbins - win * kBinCap, kBinCap);
      }
      int32_t sum = bins;  // inclusive scan of the bins
      for (int off = 1; off < kWave; off <<= 1) {
        const int32_t y = __shfl_up(sum, off, kWave);
        if (lane >= off) sum += y;
      }
      // the pass ends before the first type pair that does not fit, and after
      // a window of a split one (whose other windows come in later passes)
      const unsigned long long over = __ballot(sum > kBinCap);
      const unsigned long long cuts = __ballot(split);
      int n = over ? __ffsll(over) - 1 : kWave;
      if (cuts) n = min(n, static_cast<int>(__ffsll(cuts)));
      const bool in = lane < n;
      const unsigned long long used = __ballot(in && live);
      if (in && live) {
        const int slot = __popcll(used & ((1ull << lane) - 1));
        BinSeg g;
        g.item0 = s0;
        g.pool = en.pool + static_cast<int64_t>(win) * kBinCap;
        g.k0 = static_cast<int32_t>(s0 - en.item0 - static_cast<int64_t>(win) * en.base);
        g.a0 = en.a0;
        g.na = en.na;
        g.b0 = en.b0;
        g.nb = en.nb;
        g.diag = en.diag;
        g.lds = sum - bins;
        g.bins = bins;
        g.win0 = win * kBinCap;
        g.windowed = split;
        seg[slot] = g;
      }
      int64_t most = in && live ? s1 - s0 : 0, last = in && live ? s1 : w;
      int32_t tot = in ? sum : 0;
      for (int off = kWave / 2; off > 0; off >>= 1) {
        most = max(most, __shfl_xor(most, off, kWave));
        last = max(last, __shfl_xor(last, off, kWave));
        tot = max(tot, __shfl_xor(tot, off, kWave));
      }
      // the entry that holds the next pass's first item, as far as this wave sees
      const int step = __popcll(__ballot(e < E && en.item0 <= last)) - 1;
      if (lane == 0) {
        next_s = e0 + step;
        nseg_s = __popcll(used);
        bins_s = tot;
        end_s = last;
        big_s = most * kWave * (kWave / b.sub) > kBinMaxCount;
      }
    }
    __syncthreads();
    const int nseg = nseg_s, nbins = bins_s;
    const int64_t wend = end_s;
    const int next = next_s;
    const bool big = big_s != 0;
    // copies of each bin, for consecutive lanes: fewer conflicts and fuller
    // banks, as long as they fit and the pairs pay for emptying them
    int logR = 0;
    const int64_t pairs = (wend - w) * kWave * (kWave / b.sub);
    while (logR < 4 && (static_cast<int64_t>(nbins) << (logR + 1)) <= kBinCap &&
           (static_cast<int64_t>(nbins) << (logR + 1)) * 16 <= pairs)
      ++logR;
    for (int k = tid; k < (nbins * 3) << logR; k += kBinThreads) h[k] = 0;
    __syncthreads();
    const int64_t seg_first = lane < nseg ? seg[lane].item0 : INT64_MAX;
    for (int64_t round = w; round < wend; round += kBinWaves) {
      const int64_t item = round + wave;
      if (item < wend) {
        const int at = __builtin_amdgcn_readfirstlane(__popcll(__ballot(seg_first <= item)) - 1);
        BinSeg sg = seg[at];
        sg.a0 = __builtin_amdgcn_readfirstlane(sg.a0);
        sg.na = __builtin_amdgcn_readfirstlane(sg.na);
        sg.b0 = __builtin_amdgcn_readfirstlane(sg.b0);
        sg.nb = __builtin_amdgcn_readfirstlane(sg.nb);
        sg.bins = __builtin_amdgcn_readfirstlane(sg.bins);
        sg.win0 = __builtin_amdgcn_readfirstlane(sg.win0);
        const int diag = __builtin_amdgcn_readfirstlane(sg.diag);
        const int windowed = __builtin_amdgcn_readfirstlane(sg.windowed);
        const int lds = __builtin_amdgcn_readfirstlane(sg.lds);
        const int k = __builtin_amdgcn_readfirstlane(static_cast<int>(item - sg.item0) + sg.k0);
        const int sub = k % b.sub, kk = k / b.sub;
        int it, jt;
        if (diag) {
          tri_decode(kk, &it, &jt);
        } else {
          const int nI = (sg.na + kWave - 1) / kWave;
          jt = kk / nI;
          it = kk - jt * nI;
        }
        const int span = kWave / b.sub;
        const int j0 = jt * kWave + sub * span;
        const int j1 = min(sg.nb, j0 + span);
        const int i = it * kWave + lane;
        const uint32_t bin_bytes = 24u << logR;
        const uint32_t lane_base = static_cast<uint32_t>(lds) * bin_bytes + 24u * (lane & ((1 << logR) - 1));
        auto* hb = reinterpret_cast<unsigned char*>(h);
        if (i < sg.na) {
          if (windowed || (diag && it == jt) || (j1 - j0) % kBinBatch)
            sweep<true>(b.xs, hb, sg, i, j0, j1, diag, lane_base, bin_bytes);
          else
            sweep<false>(b.xs, hb, sg, i, j0, j1, false, lane_base, bin_bytes);
        }
      }
      // (a type pair with few items cannot fill a bin's fields)
      if (big && round + kBinWaves < wend) {
        __syncthreads();
        empty_bins(h, seg, nseg, nbins, logR, kBinSpill, b.pool);
        __syncthreads();
      }
    }
    __syncthreads();
    empty_bins(h, seg, nseg, nbins, logR, 1, b.pool);
    __syncthreads();
    w = wend;
    // (the same entry while its windows last)
    e0 = next;
    while (e0 + 1 < E && b.entries[e0 + 1].item0 <= w) ++e0;
  }
}

hipError_t launch_bins(const BinArgs& b, hipStream_t st) {
  hipLaunchKernelGGL(k_bins, dim3(static_cast<uint32_t>(b.pair_wgs)), dim3(kBinThreads), 0, st, b);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The final sums.
// ---------------------------------------------------------------------------
// Roots of P_6 (Gauss-Legendre nodes), and the coefficient of v^k in the
// Lagrange polynomial of node j as kBinL[k][j] (fit_bins.py prints both).
__constant__ double kBinNode[kBinMoments] = {-0x1.dd6ca4e80a01ep-1, -0x1.528a09655c95ep-1, -0x1.e8b12d03675c5p-3,
                                             0x1.e8b12d03675c5p-3,  0x1.528a09655c95ep-1,  0x1.dd6ca4e80a01ep-1};
__constant__ double kBinL[kBinMoments][kBinMoments] = {
    {0x1.2245d507008b9p-5, -0x1.34665409dfb7ap-3, 0x1.3af537b207e53p-1, 0x1.3af537b207e53p-1, -0x1.34665409dfb7ap-3,
     0x1.2245d507008b9p-5},
    {-0x1.374b6eefbfc8bp-5, 0x1.d26aea47f8130p-3, -0x1.49fac8e7b3fd5p+1, 0x1.49fac8e7b3fd5p+1, -0x1.d26aea47f8130p-3,
     0x1.374b6eefbfc8bp-5},
    {-0x1.681e3b2e235dbp-1, 0x1.68afe49455d52p+1, -0x1.0ea855c8ccfdcp+1, -0x1.0ea855c8ccfdcp+1, 0x1.68afe49455d52p+1,
     -0x1.681e3b2e235dbp-1},
    {0x1.8232c03a4b15ap-1, -0x1.10bf7d3b27a67p+2, 0x1.1b91014927dc9p+3, -0x1.1b91014927dc9p+3, 0x1.10bf7d3b27a67p+2,
     -0x1.8232c03a4b15ap-1},
    {0x1.6c64161173aecp+0, -0x1.855396d36ffd5p+1, 0x1.9e4317956c4bep+0, 0x1.9e4317956c4bep+0, -0x1.855396d36ffd5p+1,
     0x1.6c64161173aecp+0},
    {-0x1.86c7d2f9ece58p+0, 0x1.2667a539aebf1p+2, -0x1.b205245a3fbddp+2, 0x1.b205245a3fbddp+2, -0x1.2667a539aebf1p+2,
     0x1.86c7d2f9ece58p+0}};

// sin(x) / x for 0 <= x < 1.6e6, given 1/x (any finite value at x = 0).
__device__ __forceinline__ double sinc_f64(double x, double ix) {
  const double v = sincos_any(x).s * ix;
  return x == 0.0 ? 1.0 : v;
}

// One work-group (four waves): the groups first, first + b.wgs, ... of a
// structure for 64 q values, TPG type pairs at a time.  Per node a reduction
// and a polynomial for the sine (about 35 FP64 instructions) and one FMA per
// type pair, the weights read from LDS as broadcasts; three nodes in flight
// per wave hide the sine's serial chain.
template <int TPG, bool SPART>
__device__ void bins_sum(const BinArgs& b, int s, int first, const float* __restrict__ table, int32_t Nq, double q0,
                         double dq, const double* __restrict__ qdev) {
  constexpr int kNodes = kBinChunk * kBinMoments;
  __shared__ double W[kNodes][TPG];
  __shared__ double R[kNodes], iR[kNodes];
  __shared__ double red[4][kWave];
  const int nbins = b.nbins[s];
  const int64_t pool0 = b.pool_off[s];
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int m = blockIdx.y * kWave + lane;
  const double qm = m < Nq ? (qdev ? qdev[m] : q0 + m * dq) : 0.0;
  const double iq = qm > 0.0 ? 1.0 / qm : 0.0;
  const int chunks = (nbins + kBinChunk - 1) / kBinChunk;
  const int groups = min(kBinGroups, chunks);
  double sum = 0.0;
  for (int g = first; g < groups; g += b.wgs) {
    double total = 0.0;
    for (int tp0 = 0; tp0 < b.TP; tp0 += TPG) {
      const int ntp = min(TPG, b.TP - tp0);
      // form factor products of the type pairs (2 f_a f_b), loaded together
      double ff[TPG];
      {
        int ta, tb;
        tri_decode(tp0, &ta, &tb);
        float fa[TPG], fb[TPG];
#pragma unroll
        for (int k = 0; k < TPG; ++k) {
          const int64_t mc = m < Nq ? m : 0;
          fa[k] = table[static_cast<int64_t>(min(ta, b.T - 1)) * Nq + mc];
          fb[k] = table[static_cast<int64_t>(min(tb, b.T - 1)) * Nq + mc];
          ++ta;
          if (ta > tb) {
            ta = 0;
            ++tb;
          }
        }
#pragma unroll
        for (int k = 0; k < TPG; ++k) ff[k] = 2.0 * static_cast<double>(fa[k]) * static_cast<double>(fb[k]);
      }
      double acc[TPG];
#pragma unroll
      for (int k = 0; k < TPG; ++k) acc[k] = 0.0;
      // (a chunk's integer sums are read while the last one's nodes run)
      const int bl = tid % kBinChunk, tl = tid / kBinChunk;
      const bool mine = tid < kBinChunk * TPG && tl < ntp;
      unsigned long long next[kBinMoments] = {};
      auto fetch = [&](int ch) {
        const int bin = ch * kBinChunk + bl;
        const bool have = mine && bin < nbins;
        const unsigned long long* p =
            b.pool + (pool0 + static_cast<int64_t>(tp0 + (have ? tl : 0)) * nbins + (have ? bin : 0)) * kBinMoments;
#pragma unroll
        for (int k = 0; k < kBinMoments; ++k) next[k] = have ? p[k] : 0;
      };
      fetch(g);
      for (int ch = g; ch < chunks; ch += kBinGroups) {
        __syncthreads();
        if (tid < kBinChunk * TPG) {
          double wn[kBinMoments];
          bin_node_weights(next, ch * kBinChunk + bl, kBinL, wn);
#pragma unroll
          for (int j = 0; j < kBinMoments; ++j) W[bl * kBinMoments + j][tl] = wn[j];
        } else if (tid >= 192 && tid < 192 + kNodes) {
          const int nd = tid - 192;
          const double r = bin_node_radius(ch * kBinChunk + nd / kBinMoments, kBinNode[nd % kBinMoments]) / b.invh;
          R[nd] = r;
          iR[nd] = 1.0 / r;
        }
        if (ch + kBinGroups < chunks) fetch(ch + kBinGroups);
        __syncthreads();
#pragma unroll 3
        for (int x = 0; x < kNodes / 4; ++x) {
          const int nd = 4 * x + wave;
          const double f = sinc_f64(qm * R[nd], iq * iR[nd]);
#pragma unroll
          for (int k = 0; k < TPG; ++k) acc[k] = fma(W[nd][k], f, acc[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < TPG; ++k) {
        if (SPART && k < ntp) {
          // (the four waves' sums, one row per type pair)
          __syncthreads();
          red[wave][lane] = acc[k];
          __syncthreads();
          if (wave == 0 && m < Nq)
            b.spart[(static_cast<int64_t>(g) * b.TP + tp0 + k) * Nq + m] =
                ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
        }
        // (acc is zero past the last type pair, the table values there finite
        // or not: they are left out)
        total = k < ntp ? fma(ff[k], acc[k], total) : total;
      }
    }
    __syncthreads();
    red[wave][lane] = total;
    __syncthreads();
    sum += ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    if (b.rows > 1) {
      if (wave == 0 && m < Nq) b.part[(static_cast<int64_t>(s) * b.rows + g) * Nq + m] = sum;
      sum = 0.0;
    }
  }
  if (b.rows == 1 && wave == 0 && m < Nq) b.part[static_cast<int64_t>(s) * Nq + m] = sum;
}

template <int TPG, bool SPART>
__global__ __launch_bounds__(256) void k_bins_sum(BinArgs b, DescView sd, const double* __restrict__ partial,
                                                  double* __restrict__ slices, const float* __restrict__ table,
                                                  int32_t Nq, double q0, double dq, const double* __restrict__ qdev) {
  const int64_t nb = static_cast<int64_t>(b.S) * b.wgs;
  if (blockIdx.x < nb) {
    const int s = static_cast<int>(blockIdx.x / b.wgs), g = static_cast<int>(blockIdx.x % b.wgs);
    if (b.route[s]) bins_sum<TPG, SPART>(b, s, g, table, Nq, q0, dq, qdev);
    return;
  }
  const int64_t sl = blockIdx.x - nb;
  if (b.meta->fallback == 0 || b.route[find_struct_by_slice(sd, sl)]) return;
  reduce_slice(sd, sl, partial, Nq, slices);
}

hipError_t launch_bins_reduce(const BinArgs& b, const DescView& sd, int64_t n_slices, const double* partial,
                              double* slices, const int32_t* toff, const float* table, int32_t Nq, double q0, double dq,
                              const double* qdev, double* I_out, hipStream_t st) {
  const uint32_t qgroups = static_cast<uint32_t>(ceil_div(Nq, kWave));
  const dim3 grid(static_cast<uint32_t>(static_cast<int64_t>(b.S) * b.wgs + n_slices), qgroups);
  auto go = [&](auto* k) {
    hipLaunchKernelGGL(k, grid, dim3(256), 0, st, b, sd, partial, slices, table, Nq, q0, dq, qdev);
  };
  // (as many type pairs at a time as there are, to 16: each pass repeats the sines)
  if (b.TP == 1)
    b.spart ? go(&k_bins_sum<1, true>) : go(&k_bins_sum<1, false>);
  else if (b.TP <= 6)
    b.spart ? go(&k_bins_sum<6, true>) : go(&k_bins_sum<6, false>);
  else
    b.spart ? go(&k_bins_sum<16, true>) : go(&k_bins_sum<16, false>);
  if (I_out)
    return launch_reduce_final(sd, b.S, slices, toff, nullptr, table, b.T, Nq, q0, dq, qdev, &b, I_out, st);
  return hipGetLastError();
}

}  // namespace sas
