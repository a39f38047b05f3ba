// Device helpers shared by the Lanczos and tridiagonal kernels.
#pragma once

#include "internal.h"

namespace ebtc {

constexpr int kWaves = kBlock / 64;

// Workgroups are dispatched round-robin over the eight XCDs (workgroup id mod 8). Map them so that
// each XCD walks a contiguous range of logical workgroups: the workgroups of one realization then
// share one XCD's L2, where the gathered vector v_j stays resident.
__device__ inline int logical_block(int b, int G) {
  const int x = b & 7, q = b >> 3;
  const int base = G >> 3, rem = G & 7;
  return x * base + (x < rem ? x : rem) + q;
}

__device__ inline int logical_block() { return logical_block(blockIdx.x, gridDim.x); }

struct Ref {
  int task;
  int blk;
};

// True when a realization takes no part in step j: finished, or (second pass of the memory-bounded
// form) past the last step whose basis vector the combination needs.
__device__ inline bool step_skipped(const LzArgs& a, const RState* st, int j) {
  return st->done || (a.stop_mused && j + 1 >= st->m_used);
}

// The same for the kernels that form step j's product. Their launch also closes step j - 1, and its first workgroup may
// record a stop while the others start: a stop found by this launch does not count, so that all threads of a workgroup
// see the same (barriers follow); the closing, which every workgroup does for itself, then ends them.
__device__ inline bool product_skipped(const LzArgs& a, const RState* st, int j) {
  return (unsigned)(st->done - 1) < (unsigned)(j + 1) || (a.stop_mused && j + 1 >= st->m_used);  // 1 or 2 + i, i < j
}

// True when every realization of the launch stopped at step j - 1's adaptive check: the launch's
// workgroups return before reading anything else (the captured sequence runs to the step cap).
__device__ inline bool all_stopped(const LzArgs& a, int j) {
  return a.live != nullptr && j > 0 && a.live[j - 1] == 0;
}

// The same map with every XCD's range walked from its end.
__device__ inline int logical_block_back() {
  const int G = gridDim.x, b = blockIdx.x;
  const int x = b & 7, q = b >> 3;
  const int base = G >> 3, rem = G & 7, cnt = base + (x < rem ? 1 : 0);
  return x * base + (x < rem ? x : rem) + cnt - 1 - q;
}

__device__ inline Ref resolve(const LzArgs& a, bool back = false) {
  const int lb = back ? logical_block_back() : logical_block();
  if (a.blkmap == nullptr) return {a.single_task, lb};
  const int gb = a.sub_blocks ? a.sub_blocks[lb] : lb;
  const int t = a.blkmap[gb];
  return {t, gb - a.tasks[t].blk_begin};
}

// x of lane ^ M, in registers: quad permutes, a half-row mirror or a rotation of the rows of 16 lanes, and the
// row swaps (each leaves one register with the even rows, or halves, of x twice and one with the odd ones). The
// shuffle through the LDS crossbar that it replaces takes about a hundred cycles.
template <int M>
__device__ inline int lane_xor32(int x) {
  static_assert(M == 1 || M == 2 || M == 4 || M == 8 || M == 16 || M == 32, "one bit of the lane");
  if constexpr (M == 1) return __builtin_amdgcn_update_dpp(0, x, 0xb1, 0xf, 0xf, false);  // quad_perm 1 0 3 2
  if constexpr (M == 2) return __builtin_amdgcn_update_dpp(0, x, 0x4e, 0xf, 0xf, false);  // quad_perm 2 3 0 1
  if constexpr (M == 4) {  // lane ^ 7, then ^ 3
    const int h = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, false);  // row_half_mirror
    return __builtin_amdgcn_update_dpp(0, h, 0x1b, 0xf, 0xf, false);          // quad_perm 3 2 1 0
  }
  if constexpr (M == 8) return __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, false);  // row_ror:8
  if constexpr (M == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return (threadIdx.x & 16) ? (int)r[0] : (int)r[1];
  }
  if constexpr (M == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return (threadIdx.x & 32) ? (int)r[0] : (int)r[1];
  }
}
template <int M>
__device__ inline double lane_xor(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)lane_xor32<M>((int)(uint32_t)b), hi = (uint32_t)lane_xor32<M>((int)(uint32_t)(b >> 32));
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Lanes without bit M: a + a of lane ^ M; lanes with it: b + b of lane ^ M.
template <int M>
__device__ inline double lane_exchange_add(double a, double b, int lane) {
  if constexpr (M >= 16) {  // the row swaps do the selection themselves
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    uint32_t lo[2], hi[2];
    if constexpr (M == 32) {
      const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
      const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
      lo[0] = l[0], lo[1] = l[1], hi[0] = h[0], hi[1] = h[1];
    } else {
      const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
      const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
      lo[0] = l[0], lo[1] = l[1], hi[0] = h[0], hi[1] = h[1];
    }
    return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) +
           __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
  } else {
    const bool up = (lane & M) != 0;
    return (up ? b : a) + lane_xor<M>(up ? a : b);
  }
}

__device__ inline double wave_sum(double v) {
  v += lane_xor<32>(v);
  v += lane_xor<16>(v);
  v += lane_xor<8>(v);
  v += lane_xor<4>(v);
  v += lane_xor<2>(v);
  v += lane_xor<1>(v);
  return v;
}

// Sum of one double over the workgroup of NT threads; every thread gets the result. red: NT/64 doubles.
template <int NT = kBlock>
__device__ inline double block_sum(double v, double* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) t += red[i];
  return t;
}

// Butterfly reduce-scatter of P values per lane over the 64 lanes of a wave: after the call v[0]
// of lane l holds the wave-wide sum of value index (P == 64 ? l : l >> 1). Costs P - 1 (+1)
// shuffles instead of 6 P for P separate reductions.
template <int P, int M>
struct ReduceScatter {
  __device__ static inline void run(double* v, int lane) {
    if constexpr (P > 1) {
      constexpr int h = P / 2;
#pragma unroll
      for (int k = 0; k < h; ++k) v[k] = lane_exchange_add<M>(v[k], v[k + h], lane);
    } else {
      v[0] += lane_xor<M>(v[0]);
    }
    if constexpr (M > 1) ReduceScatter<(P > 1 ? P / 2 : 1), M / 2>::run(v, lane);
  }
};



// Chunking of per-workgroup partial sums: a realization with nblk workgroups sums its partials in
// chunks of kernel-independent size (left to right inside a chunk, then chunk sums left to right).
// Every kernel that needs the same total therefore gets the same bits, whatever its thread count.
__device__ inline int part_chunk(int nblk) { return (nblk + kMaxChunks - 1) / kMaxChunks; }

// Total of x[b * stride], b < count, in the canonical order. All threads of the block call it and
// all get the result. lds: >= kMaxChunks doubles of scratch.
__device__ inline double canonical_sum(const double* x, int count, int stride, double* lds) {
  const int chunk = part_chunk(count);
  const int nch = (count + chunk - 1) / chunk;
  for (int c = threadIdx.x; c < nch; c += blockDim.x) {
    double s = 0.0;
    const int b1 = min(count, (c + 1) * chunk);
    for (int b = c * chunk; b < b1; ++b) s += x[(size_t)b * stride];
    lds[c] = s;
  }
  __syncthreads();
  double t = 0.0;
  for (int c = 0; c < nch; ++c) t += lds[c];
  __syncthreads();
  return t;
}

struct StepClose {
  double beta;
  int flags;  // EBTC_FLAG_BREAKDOWN / EBTC_FLAG_NONFINITE when the realization stops here
};

// Closes Lanczos step j from its norm partials: beta_j = ||v~_{j+1}|| and the breakdown test
// beta_j <= 64 eps scal[j], scal[j] = max(|alpha_0..j|, beta_0..j-1) (recorded by the update kernel
// that finished alpha_j). Reads only values written by earlier kernels. ss: their canonical sum.
__device__ inline StepClose close_sum(const RState* st, double ss, int j, double eps) {
  StepClose c;
  c.beta = sqrt(ss);
  const double scale = st->scal[j];
  c.flags = 0;
  if (!isfinite(c.beta) || !isfinite(scale)) c.flags = EBTC_FLAG_NONFINITE;
  else if (!(c.beta > 64.0 * eps * scale)) c.flags = EBTC_FLAG_BREAKDOWN;
  return c;
}
__device__ inline StepClose close_step(const RState* st, const double* norm_part, int nblk, int j, double eps,
                                       double* lds) {
  return close_sum(st, canonical_sum(norm_part, nblk, 1, lds), j, eps);
}

}  // namespace ebtc
