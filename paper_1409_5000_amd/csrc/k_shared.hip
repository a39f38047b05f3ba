// Products of several Lanczos processes with one matrix (subgraph centrality: a process per node, started at
// e_i), w_p = s_p A v_p for all p at once.
//
// Process by process, the CSR-stream form fetches every entry's vector element as a gather of its own: 100M
// gathers per step for 50 processes on n=1e5 at degree 20, 0.54 ms at the rate the L2 takes them. Here
// k_shared_pack first lays the current basis vectors out node by node, up to 64 processes side by side, and
// k_shared_spmm gives every process a lane: one wavefront load brings an entry's element of all of them, a
// contiguous 64 to 512 bytes, and the entries are read once per 64 processes: 0.07 ms and 0.017 for the packing.
// Every product is rounded as in the stream form and each row's products are added in entry order in FP64, so
// the results are the stream form's, bit for bit; rows of more than kSharedLong entries take its code.
#include <algorithm>

#include "internal.h"
#include "step_device.h"

namespace ebtc {
namespace {

constexpr int kSharedLong = 1024;  // longer rows: the stream form's workgroup per row and process (one wavefront
                                   // in entry order would hold up the launch)
constexpr int kSharedU = 16;       // entries per load group, two groups in flight
template <typename T>
constexpr int kTileRows = 64 / sizeof(T);  // rows a wavefront collects before it writes them, 64 bytes per process
                                           // (17 KB of LDS per workgroup: 32 wavefronts fit a compute unit)

template <typename T>
__device__ inline int shared_stride(int cnt) {  // whole 64-byte pieces
  constexpr int E = 64 / sizeof(T);
  return (cnt + E - 1) / E * E;
}

// Row bounds of the wavefronts' shares: equal sums of entries + rows. Thread `shares` + 1 starts the list.
__global__ __launch_bounds__(kBlock) void k_shared_cut(int32_t n, const int32_t* rp, SharedMat q) {
  const int s = blockIdx.x * kBlock + threadIdx.x;
  if (s > q.shares) {
    if (s == q.shares + 1) *q.seen = {0, rp[n] - rp[0], 0, 0, 0, 0, 0};
    return;
  }
  const int32_t z = rp[0];
  const int64_t want = ((int64_t)(rp[n] - z) + n) * s / q.shares;
  int lo = 0, hi = n;  // first row r with rp[r] - z + r >= want
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if ((int64_t)(rp[mid] - z) + mid >= want) hi = mid; else lo = mid + 1;
  }
  q.cut[s] = s == q.shares ? n : lo;
}

// The long rows, in any order (each is a result of its own), and the rest of SharedSeen: a workgroup per group of rows
// of the stream form, whose walk one thread repeats where there are rows to wait for. cap: that form's capacity.
__global__ __launch_bounds__(kBlock) void k_shared_long(int32_t n, const int32_t* rp, SharedMat q, int cap) {
  static_assert(kBlock == kStreamRows, "a thread per row of a group");
  const int r = blockIdx.x * kBlock + threadIdx.x;
  SharedSeen* seen = q.seen;
  int len = r < n ? rp[r + 1] - rp[r] : 0;
  if (len > kSharedLong) {
    q.longs[atomicAdd(&seen->rows, 1)] = r;
    atomicAdd(&seen->longs, len > cap ? len / 16 : len);
    if (len > cap) atomicMax(&seen->big, len / 16);
  }
  __shared__ int top, most, lens[kBlock];
  if (threadIdx.x == 0) top = most = 0;
  lens[threadIdx.x] = len;
  __syncthreads();
  atomicMax(&top, len);
  if (len <= cap) atomicMax(&most, len);
  __syncthreads();
  if (threadIdx.x != 0) return;
  // most groups have nothing larger to say, and thousands of atomics on one word take longer than the rest
  auto raise = [](int32_t* x, int v) {
    if (__hip_atomic_load(x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < v) atomicMax(x, v);
  };
  raise(&seen->row, most);
  int cost = top;
  if (top > 256) {
    int held = 0, longest = 0;  // of the chunk
    cost = 0;
    for (int i = 0; i < kBlock; ++i) {
      const int l = lens[i];
      if (l > cap || held + l > cap) {
        cost += longest + (l > cap ? l / 16 : 0);
        held = longest = 0;
      }
      if (l <= cap) {
        held += l;
        longest = max(longest, l);
      }
    }
    cost += longest;
    atomicAdd(&seen->groups, cost);
  }
  raise(&seen->group, cost);
}

// Node-major copy of the processes' current vectors, and their scales: workgroups [0, count) close the last step
// of one process each, as the product kernels of the other forms do; the rest transpose 64 nodes of up to 64
// processes. Bandwidth-bound.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_shared_pack(LzArgs a, SharedMat q, int32_t n, int j) {
  __shared__ double chunks[kMaxChunks];
  __shared__ T tile[64][65];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if ((int)blockIdx.x < q.count) {
    const Task tk = a.tasks[blockIdx.x];
    double sj;
    const bool go = open_step(a, tk, a.state + blockIdx.x, 0, j, chunks, &sj);
    if (tid == 0) q.s[blockIdx.x] = go ? sj : kSharedStopped;
    return;
  }
  const int tiles = (n + 63) / 64, b = blockIdx.x - q.count, g = b / tiles, v0 = (b - g * tiles) * 64;
  const int cnt = min(64, q.count - 64 * g), S = shared_stride<T>(cnt);
  for (int p = wv; p < S; p += kWaves)
    tile[lane][p] =
        p < cnt && v0 + lane < n ? ((const T*)a.V + a.tasks[64 * g + p].vec_off + vslot(a, j) * n)[v0 + lane] : (T)0;
  __syncthreads();
  T* x = (T*)q.x + (size_t)64 * g * n;
  if (lane < S)
    for (int r = wv; r < min(64, n - v0); r += kWaves) x[(size_t)(v0 + r) * S + lane] = tile[r][lane];
}

__device__ inline int64_t wave_uniform(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ inline float lane_value(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ inline double lane_value(double v, int l) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
// An element of every process, at byte `at` (uniform) of the packed vectors plus the lane's own.
__device__ inline float load_piece(__amdgpu_buffer_rsrc_t r, int own, int at, float) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, own, at, 0));
}
__device__ inline double load_piece(__amdgpu_buffer_rsrc_t r, int own, int at, double) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, own, at, 0));
}
__device__ inline void wave_tile_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The long rows, a workgroup per row and process, by `blocks` workgroups.
template <typename T, bool HAS_VAL>
__device__ inline void long_rows(const LzArgs& a, const SharedMat& q, int32_t n, int j, int blocks, T* prod) {
  __shared__ int rp_lds[2];
  __shared__ double red[kWaves];
  for (int64_t k = blockIdx.x; k < (int64_t)q.rows * q.count; k += blocks) {
    const int h = (int)(k / q.count), p = (int)(k - (int64_t)h * q.count), row = q.longs[h];
    const double sj = q.s[p];
    if (sj == kSharedStopped) continue;
    const Task tk = a.tasks[p];
    spmv_stream_rows<T, HAS_VAL>(a.row_ptr, a.col_idx, (const T*)a.values, (const T*)a.V + tk.vec_off + vslot(a, j) * n,
                                 row, 1, sj, rp_lds, prod, (T*)a.W + tk.w_off + row, red);
    __syncthreads();
  }
}

// A wavefront per share of rows, a lane per process of group blockIdx.y. ROWS: the first row_blocks
// workgroups (of group 0) take the long rows instead, beside the others. What bounds it: 50 FP32 processes at
// n=1e5, degree 20, read 512 MB of pieces in 70 us, 7.3 TB/s, nearly all from the last-level cache (the packed
// vectors, 26 MB, do not fit an L2); few processes, or neighbours close together, the 12 cycles that a compute unit
// takes for a load of 64 lanes (FP64 23). Two groups of 16 loads are in flight per wavefront.
template <typename T, bool HAS_VAL, bool ROWS>
__global__ __launch_bounds__(kBlock) void k_shared_spmm(LzArgs a, SharedMat q, int32_t n, int j, int row_blocks) {
#pragma clang fp contract(off)
  constexpr int U = kSharedU;
  constexpr int R = kTileRows<T>;
  __shared__ T lds[ROWS ? std::max(kWaves * R * 65, StreamShape<T>::CAP) : kWaves * R * 65];
  if constexpr (ROWS) {
    if ((int)blockIdx.x < row_blocks) {
      if (blockIdx.y == 0) long_rows<T, HAS_VAL>(a, q, n, j, row_blocks, lds);
      return;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = blockIdx.y, cnt = min(64, q.count - 64 * g), S = shared_stride<T>(cnt);
  const double sj = lane < cnt ? q.s[64 * g + lane] : kSharedStopped;
  const uint64_t act = __ballot(!(sj == kSharedStopped));
  const int share = logical_block(blockIdx.x - row_blocks, gridDim.x - row_blocks) * kWaves + wv;
  if (act == 0 || share >= q.shares) return;
  const int32_t* __restrict__ rp = a.row_ptr;
  const int32_t* __restrict__ ci = a.col_idx;
  const T* __restrict__ va = (const T*)a.values;
  const int64_t x = wave_uniform((int64_t)((T*)q.x + (size_t)64 * g * n));
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)x, (short)0, __builtin_amdgcn_readfirstlane((int)((uint32_t)n * S * sizeof(T))), 0x00020000);
  T* W = (T*)a.W + (int64_t)64 * g * q.wstep;
  const int own = min(lane, S - 1) * (int)sizeof(T);
  T* tile = lds + wv * R * 65;
  const int r0 = __builtin_amdgcn_readfirstlane(q.cut[share]);
  const int r1 = __builtin_amdgcn_readfirstlane(q.cut[share + 1]);
  for (int rw = r0; rw < r1; rw += 63) {  // windows of rows whose bounds the lanes hold
    const int wr = min(63, r1 - rw);
    const int bnd = rp[rw + min(lane, wr)];
    const int nxt = __shfl_down(bnd, 1, 64);
    const uint64_t lm = __ballot(lane < wr && nxt - bnd > kSharedLong);
    int i = 0;
    while (i < wr) {  // runs of rows that are not long
      if ((lm >> i) & 1ull) {
        ++i;
        continue;
      }
      const uint64_t rest = lm >> i;
      const int end = rest ? min(wr, i + (int)__builtin_ctzll(rest)) : wr;
      const int e0 = __builtin_amdgcn_readlane(bnd, i), e1 = __builtin_amdgcn_readlane(bnd, end);
      int cur = i, rend = __builtin_amdgcn_readlane(bnd, i + 1), trows = 0, tbase = rw + i;
      double acc = 0.0;
      auto write = [&] {
        wave_tile_sync();
        const int row = lane & (R - 1);
        for (int p = lane / R; p < cnt; p += 64 / R)
          if (row < trows && ((act >> p) & 1ull)) W[p * q.wstep + tbase + row] = tile[row * 65 + p];
        wave_tile_sync();
        tbase += trows;
        trows = 0;
      };
      auto flush = [&] {  // row cur is complete
        tile[trows * 65 + lane] = (T)(acc * sj);
        acc = 0.0;
        ++cur;
        if (++trows == R) write();
        rend = cur < end ? __builtin_amdgcn_readlane(bnd, cur + 1) : 0x7fffffff;
      };
      // 32 entries' places in x and values, one per lane (past the end: the last entry again)
      auto fetch = [&](int k, int& c, T& v) {
        const int at = min(k + (lane & 31), e1 - 1);
        c = (int)((uint32_t)__builtin_nontemporal_load(ci + at) * (uint32_t)(S * sizeof(T)));
        if constexpr (HAS_VAL) v = __builtin_nontemporal_load(va + at);
      };
      // loads are issued without a condition, so that their number between two uses is known
      auto issue = [&](T (&s)[U], int c, int l0) {
#pragma unroll
        for (int u = 0; u < U; ++u) s[u] = load_piece(xr, own, __builtin_amdgcn_readlane(c, l0 + u), T{});
      };
      auto consume = [&](const T (&s)[U], T v, int l0, int k) {  // past e1: added after the last row
#pragma unroll
        for (int u = 0; u < U; ++u) {
          while (k + u >= rend) flush();
          if constexpr (HAS_VAL) acc += (double)(lane_value(v, l0 + u) * s[u]); else acc += (double)s[u];
        }
      };
      if (e0 < e1) {
        T sa[U], sb[U], v0 = 0, v1 = 0;
        int c0, c1;
        fetch(e0, c0, v0);
        fetch(e0 + 32, c1, v1);
        issue(sa, c0, 0);
        for (int k = e0; k < e1; k += 2 * U) {
          int c2;
          T v2 = 0;
          fetch(k + 64, c2, v2);
          issue(sb, c0, U);
          consume(sa, v0, 0, k);
          issue(sa, c1, 0);
          consume(sb, v0, U, k + U);
          c0 = c1, v0 = v1;
          c1 = c2, v1 = v2;
        }
      }
      while (cur < end) flush();
      if (trows) write();
      i = end;
    }
  }
}

template <typename T>
hipError_t step_t(bool has_val, const LzArgs& a, const SharedMat& q, int32_t n, int j, hipStream_t s) {
  const int groups = (q.count + 63) / 64;
  hipLaunchKernelGGL((k_shared_pack<T>), dim3((unsigned)(q.count + (int64_t)groups * ((n + 63) / 64))), dim3(kBlock), 0,
                     s, a, q, n, j);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int row_blocks = (int)std::min<int64_t>((int64_t)q.rows * q.count, 4096);
  const dim3 grid((unsigned)(row_blocks + (q.shares + kWaves - 1) / kWaves), (unsigned)groups);
  auto* spmm = q.rows > 0 ? (has_val ? k_shared_spmm<T, true, true> : k_shared_spmm<T, false, true>)
                          : (has_val ? k_shared_spmm<T, true, false> : k_shared_spmm<T, false, false>);
  hipLaunchKernelGGL(spmm, grid, dim3(kBlock), 0, s, a, q, n, j, row_blocks);
  return hipGetLastError();
}
}  // namespace

int32_t shared_shares(int dtype, int32_t n) {
  // rounds of the wavefronts that are resident at once (8 and 5 per SIMD, by registers), 16 rows each at most
  // and 4 at least
  const int64_t resident = 1024 * (dtype == EBTC_F64 ? 5 : 8), full = (n + 16 * resident - 1) / (16 * resident);
  return (int32_t)std::min<int64_t>(((int64_t)n + 3) / 4, resident * full);
}

size_t shared_stride_bytes(int dtype, int32_t count) {
  const size_t es = dtype == EBTC_F64 ? 8 : 4;
  const int32_t full = count / 64 * 64, rem = count - full;
  return es * full + (rem * es + 63) / 64 * 64;
}

hipError_t launch_shared_prepare(int dtype, const int32_t* row_ptr, const SharedMat& q, int32_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_shared_cut, dim3((unsigned)((q.shares + 2 + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, n,
                     row_ptr, q);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_shared_long, dim3((unsigned)(((int64_t)n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, n,
                     row_ptr, q, dtype == EBTC_F64 ? StreamShape<double>::CAP : StreamShape<float>::CAP);
  return hipGetLastError();
}

hipError_t launch_shared_step(int dtype, bool has_val, int j, const LzArgs& a, const SharedMat& q, int32_t n,
                              hipStream_t s) {
  return dtype == EBTC_F64 ? step_t<double>(has_val, a, q, n, j, s) : step_t<float>(has_val, a, q, n, j, s);
}

}  // namespace ebtc
