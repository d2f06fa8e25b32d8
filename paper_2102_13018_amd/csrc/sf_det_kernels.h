// sf_det_kernels.h -- device kernels of the deterministic path used by
// both the direct and the partitioned launchers (templates: each
// translation unit instantiates what it launches).
#pragma once

#include "sf_device.h"

namespace sfi {

// One wavefront per aligned chunk of at most kChunk elements.  Lane l holds
// elements [l*LPT, (l+1)*LPT) of the chunk; the lane's block is reduced in
// registers, then lanes combine at distances 1, 2, ..., 32 -- all nodes of
// the canonical pairwise tree of the chunk.  Level 0 reads leaves through
// the sorted slot list; later levels read the previous level's results.
template <typename T, int OP>
__global__ __launch_bounds__(kBlock) void k_det_chunk(const DevChunk *__restrict__ chunks, int nchunks,
                                                      const int32_t *__restrict__ sl, const T *__restrict__ src,
                                                      T *__restrict__ dst_seq, T *__restrict__ root, int bs) {
  constexpr int LPT = kChunkLPT;
  const int lane = threadIdx.x & 63;
  const int wid = (int)(((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6);
  if (wid >= nchunks) return;
  const DevChunk ch = chunks[wid];
  int32_t idx[LPT];
#pragma unroll
  for (int s = 0; s < LPT; s++) {
    const int e = lane * LPT + s;
    idx[s] = e < ch.n ? (sl ? sl[ch.src + e] : ch.src + e) : 0;
  }
  const int m = ch.n - lane * LPT;  // valid elements of this lane (may be <= 0)
  for (int c = 0; c < bs; c++) {
    T x[LPT];
#pragma unroll
    for (int s = 0; s < LPT; s++)
      if (s < m) x[s] = ld(src + (int64_t)idx[s] * bs + c);
#pragma unroll
    for (int d = 1; d < LPT; d *= 2)
#pragma unroll
      for (int p = 0; p + d < LPT; p += 2 * d)
        if (p + d < m) x[p] = Op<OP, T>::apply(x[p], x[p + d]);
    T v = x[0];
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
      const T o = shfl_down(v, d);
      if ((lane & (2 * d - 1)) == 0 && (lane + d) * LPT < ch.n) v = Op<OP, T>::apply(v, o);
    }
    if (lane == 0) {
      if (ch.dst < 0) {
        T *rp = root + (int64_t)(-ch.dst - 1) * bs + c;
        st(rp, Op<OP, T>::apply(ld(rp), v));
      } else {
        st(dst_seq + (int64_t)ch.dst * bs + c, v);
      }
    }
  }
}

// The canonical pairwise tree of the n <= kChunk values load(0) .. load(n - 1)
// over a wavefront, as in k_det_chunk; the result is in lane 0.
template <typename T, int OP, typename Load>
__device__ __forceinline__ T wave_chunk_tree(int lane, int n, Load load) {
  constexpr int LPT = kChunkLPT;
  const int m = n - lane * LPT;
  T x[LPT];
#pragma unroll
  for (int s = 0; s < LPT; s++) x[s] = load(min(lane * LPT + s, n - 1));
#pragma unroll
  for (int d = 1; d < LPT; d *= 2)
#pragma unroll
    for (int p = 0; p + d < LPT; p += 2 * d)
      if (p + d < m) x[p] = Op<OP, T>::apply(x[p], x[p + d]);
  T v = x[0];
#pragma unroll
  for (int d = 1; d < 64; d *= 2) {
    const T o = shfl_down(v, d);
    if ((lane & (2 * d - 1)) == 0 && (lane + d) * LPT < n) v = Op<OP, T>::apply(v, o);
  }
  return v;
}

// Every level above level 0 in one launch: a wavefront per root of at most
// kChunk level-0 results, a block per (root, unit component) of more (at most
// kOneLaunchResults), whose wavefronts take its level-1 chunks and leave their
// results in the LDS for the last tree.  The chunk boundaries and trees are
// those of k_det_chunk level by level.  Bound by the latency of its few
// dependent loads, which is why one launch replaces one per level: 1.2M Zipf
// leaves of f32 2.1 + 3.0 -> 3.5 us (the Reduce 22.3 -> 19.2), MAXLOC of 2M
// 35.4 -> 32.5, 16M f64 4.6 + 4.8 -> 4.9 (123.3 -> 120.8).  Blocks of 16
// wavefronts, so that the level-1 chunks of such a root take at most two
// rounds: with more a launch per level is as fast or faster (all leaves on one
// root, f64: 2M leaves 22.6 us here, 22.7 with a launch per level; 4M leaves
// 31.4 and 31.0; 16M leaves of two f32 147 and 97).  A block per component,
// because the components of a wide unit would else wait for each other's
// barriers (2M leaves of four f64 on one root 46.9 -> 32.1, a launch per level
// 34.5; 300K of sixteen f32 43.5 -> 23.0, 38.4).
constexpr int kLevelThreads = 1024;
static_assert(kOneLaunchResults <= kChunk * kChunk, "one last tree per block");
template <typename T, int OP>
__global__ __launch_bounds__(kLevelThreads) void k_det_levels(const DevChunk *__restrict__ tops, int nbig, int ntops,
                                                              const T *__restrict__ seq, T *__restrict__ root, int bs) {
  constexpr int kWaves = kLevelThreads / 64;
  __shared__ __align__(16) unsigned char raw[kChunk * sizeof(T)];
  T *part = reinterpret_cast<T *>(raw);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const unsigned nb = (unsigned)nbig * (unsigned)bs;
  if (blockIdx.x >= nb) {
    const int64_t i = nbig + (int64_t)(blockIdx.x - nb) * kWaves + wv;
    if (i >= ntops) return;
    const DevChunk ch = tops[i];
    for (int c = 0; c < bs; c++) {
      T *rp = root + (int64_t)ch.dst * bs + c;
      const T r = ld(rp);
      const T v = wave_chunk_tree<T, OP>(lane, ch.n, [&](int e) { return ld(seq + (int64_t)(ch.src + e) * bs + c); });
      if (lane == 0) st(rp, Op<OP, T>::apply(r, v));
    }
    return;
  }
  const DevChunk ch = tops[blockIdx.x / (unsigned)bs];
  const int c = (int)(blockIdx.x % (unsigned)bs);
  const int nc = (ch.n + kChunk - 1) / kChunk;
  T *rp = root + (int64_t)ch.dst * bs + c;
  const T r = ld(rp);
  for (int j = wv; j < nc; j += kWaves) {
    const int64_t e0 = (int64_t)ch.src + j * kChunk;
    const T v = wave_chunk_tree<T, OP>(lane, min(kChunk, ch.n - j * kChunk),
                                       [&](int e) { return ld(seq + (e0 + e) * bs + c); });
    if (lane == 0) st(part + j, v);
  }
  __syncthreads();
  if (wv == 0) {
    const T v = wave_chunk_tree<T, OP>(lane, nc, [&](int e) { return ld(part + e); });
    if (lane == 0) st(rp, Op<OP, T>::apply(r, v));
  }
}
template <typename T, int OP>
void launch_levels(const sf_s *sf, const T *seq, T *root, int bs, hipStream_t st) {
  const int n = (int)sf->hp.tops.size(), nbig = sf->hp.ntops_big;
  constexpr int kWaves = kLevelThreads / 64;
  if (n == 0) return;
  const unsigned g = (unsigned)nbig * (unsigned)bs + (unsigned)((n - nbig + kWaves - 1) / kWaves);
  hipLaunchKernelGGL((k_det_levels<T, OP>), dim3(g), dim3(kLevelThreads), 0, st, sf->dp.tops, nbig, n, seq, root, bs);
}

// Large roots, pass 2: one wavefront per large root turns its chunk sums
// into chunk bases (root value + exclusive prefix) and writes the final
// root.  Each iteration scans 64*kScanPer chunk sums: kScanPer consecutive
// ones per lane in registers, the lane totals with shuffles.
constexpr int kScanPer = 8;
template <typename T>
__global__ __launch_bounds__(kBlock) void k_fop_root_scan(const int32_t *__restrict__ first, int nlarge,
                                                          const DevChunk *__restrict__ chunks, T *__restrict__ sums,
                                                          T *__restrict__ root, int bs) {
  const int lane = threadIdx.x & 63;
  const int k = (int)(((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6);
  if (k >= nlarge) return;
  const int c0 = first[k], c1 = first[k + 1];
  const int32_t r = chunks[c0].dst;
  for (int c = 0; c < bs; c++) {
    T carry = root[(int64_t)r * bs + c];
    for (int base = c0; base < c1; base += 64 * kScanPer) {
      T x[kScanPer];
      T s = T(0);
#pragma unroll
      for (int j = 0; j < kScanPer; j++) {
        const int i = base + lane * kScanPer + j;
        x[j] = i < c1 ? sums[(int64_t)i * bs + c] : T(0);
        s = Op<OP_SUM, T>::apply(s, x[j]);
      }
      T inc = s;
#pragma unroll
      for (int d = 1; d < 64; d *= 2) {
        const T o = shfl_up(inc, d);
        if (lane >= d) inc = Op<OP_SUM, T>::apply(inc, o);
      }
      T a = Op<OP_SUM, T>::apply(carry, wrap_sub(inc, s));
#pragma unroll
      for (int j = 0; j < kScanPer; j++) {
        const int i = base + lane * kScanPer + j;
        if (i < c1) sums[(int64_t)i * bs + c] = a;
        a = Op<OP_SUM, T>::apply(a, x[j]);
      }
      carry = Op<OP_SUM, T>::apply(carry, __shfl(inc, 63));
    }
    if (lane == 0) root[(int64_t)r * bs + c] = carry;
  }
}

}  // namespace sfi
