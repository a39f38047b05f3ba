// The whole Lanczos process of one realization of a few row blocks in one workgroup of 1024 threads (gfx950): the
// identification-rate backgrounds of 2049 to about 1e4 nodes, where the per-phase schedule spends most of a call on
// launches of a few microseconds each, and on those of the steps up to an adaptive run's cap.
//
// As in the one-row-block solve, barriers take the place of kernel boundaries and every phase keeps the per-phase
// kernels' arithmetic in their thread order, so the results are theirs bit for bit: the CSR-stream product, the dot
// partials of a row block in the order of 1024 or 256 threads (four row blocks side by side in the latter case), the
// canonical sums over the row blocks, the squared norms in the order of the 256-thread update. v_j and the row
// pointers stay in LDS, the basis and the product in the workspace.
// What bounds it: the basis, read twice per step by one compute unit (45 GB/s each, 4.5 TB/s together), the entries
// from the L2, and 14 us of barriers and dependent chains per step.
// 200 x n=9000, degree 2.1, FP64, 14 adaptive steps: 1.56 to 0.80 ms; FP32 1.31 to 0.60.
#include <algorithm>

#include "step_device.h"

namespace ebtc {
namespace {

constexpr int kWideThreads = 1024, kWideWaves = kWideThreads / 64;
constexpr int kWideBlocks = 8;  // row blocks at most (the LDS holds fewer in FP64)

struct WideLds {
  int32_t x_off, rp_off, work_off, bytes;  // v_j (n_max), row pointers (n_max + 1), products / dot sums
};

// Work area: the product slots of a chunk, or the dot sums of up to 64 vectors.
template <typename T>
constexpr size_t wide_work() {
  const size_t prod = sizeof(T) * StreamShape<T>::CAP;
  // FP64: 8 vectors of 16 wavefronts or 64 of 4; FP32: 32 of 16 or 64 of 4 (per row block)
  const size_t dots = sizeof(double) * kWideBlocks * (sizeof(T) == 8 ? 256 : 512);
  return prod > dots ? prod : dots;
}

__device__ inline int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)((uint64_t)hi << 32 | lo);
}

// The thread's index, computed anew, so that what follows from it is not carried around the step loop.
__device__ inline int fresh_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

constexpr int kWideRow = 128;  // entries of a row that one thread sums

// w = s_j A v_j: a thread per row, eight entries at a time (their columns with two wide loads; lanes walk rows side by
// side, so that a line is used again at once); rows of more than kWideRow entries, dealt out row by row to the
// wavefronts, 64 products at a time through LDS and summed by one lane. Each sum in entry order in FP64, products
// rounded to T first: the stream form's bits. Rows beyond the stream form's capacity, any number of them, take that
// form's other order there: the sums of 256 threads in T, four threads to a lane, reduced wavefront by wavefront
// (`first`: in entry order like all others, as in the first-product kernels). No barriers: chunks of product slots
// with two each took 2 to 3 us per 3072 entries, 390 us for 351000 entries where this takes 40.
template <typename T, bool HAS_VAL>
__device__ inline void wide_spmv(const int* rp_l, const int32_t* __restrict__ ci, const T* __restrict__ va, const T* xs,
                                 int n, double sj, T* W, T* prod, bool first) {
  constexpr int CAP = StreamShape<T>::CAP;
  struct __attribute__((packed, aligned(4))) Cols { int32_t c[8]; };
  struct __attribute__((packed, aligned(sizeof(T)))) Vals { T v[8]; };
  const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int row = tid; row < n; row += kWideThreads) {
    const int e0 = rp_l[row], e1 = rp_l[row + 1];
    if (e1 - e0 > kWideRow) continue;
    double acc = 0.0;
    int k = e0;
    for (; k + 8 <= e1; k += 8) {
      const Cols c = *(const Cols*)(ci + k);
      Vals v;
      if constexpr (HAS_VAL) v = *(const Vals*)(va + k);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        T pr = xs[c.c[u]];
        if constexpr (HAS_VAL) pr = v.v[u] * pr;
        acc += (double)pr;
      }
    }
    for (; k < e1; k += 4) {
      int c[4];
      T v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = min(k + u, e1 - 1);
        c[u] = ci[e];
        if constexpr (HAS_VAL) v[u] = va[e];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        T pr = xs[c[u]];
        if constexpr (HAS_VAL) pr = v[u] * pr;
        const double t = acc + (double)pr;
        acc = k + u < e1 ? t : acc;
      }
    }
    W[row] = (T)(acc * sj);
  }
  T* slots = prod + wave * 64;
  for (int t = 0; t < n; t += kWideThreads) {
    const int mine = t + lane * kWideWaves + wave;
    const int len = mine < n ? rp_l[mine + 1] - rp_l[mine] : 0;
    uint64_t m = __ballot(len > kWideRow);
    while (m) {
      const int row = t + __builtin_ctzll(m) * kWideWaves + wave;
      m &= m - 1;
      const int e0 = __builtin_amdgcn_readfirstlane(rp_l[row]), e1 = __builtin_amdgcn_readfirstlane(rp_l[row + 1]);
      double acc = 0.0;
      if (e1 - e0 > CAP && !first) {
        T p[4] = {0, 0, 0, 0};
        for (int k = e0 + lane; k - lane < e1; k += 256) {
          int c[4];
          T v[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int e = min(k + q * 64, e1 - 1);
            c[q] = ci[e];
            if constexpr (HAS_VAL) v[q] = va[e];
          }
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (k + q * 64 < e1) {
              const T xv = xs[c[q]];
              if constexpr (HAS_VAL) p[q] += v[q] * xv; else p[q] += xv;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) acc += wave_sum((double)p[q]);
        if (lane == 0) W[row] = (T)(acc * sj);
        continue;
      }
      int c = ci[e0 + lane];  // more than 64 entries
      T v = 0;
      if constexpr (HAS_VAL) v = va[e0 + lane];
      for (int k = e0; k < e1; k += 64) {
        T pr = xs[c];
        if constexpr (HAS_VAL) pr = v * pr;
        slots[lane] = pr;
        const int e = min(k + 64 + lane, e1 - 1);  // the next 64
        c = ci[e];
        if constexpr (HAS_VAL) v = va[e];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int cnt = min(64, e1 - k);
        int i = 0;
        for (; i + 8 <= cnt; i += 8) {
          T q[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) q[u] = slots[i + u];
#pragma unroll
          for (int u = 0; u < 8; ++u) acc += (double)q[u];
        }
        for (; i < cnt; ++i) acc += (double)slots[i];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
      if (lane == 0) W[row] = (T)(acc * sj);
    }
  }
}

// Dot sums of step j, wavefront by wavefront of NT virtual threads: red[((c * nblk + blk) * NT / 64 + w) * 8 + i] of
// vector 8 c + i.
template <typename T, int NT>
__device__ inline void wide_dots(const T* V, const T* W, int n, int nblk, int j, double* red) {
  constexpr int G = kWideThreads / NT, RPT = kRowsPerBlock / NT, NW = NT / 64;
  const int tid = fresh_tid(), lane = tid & 63, cnt = j + 1;
  const int g = tid / NT, vt = tid % NT, wave = vt >> 6;
#pragma unroll 1
  for (int c0 = 0; c0 < cnt; c0 += 8) {
#pragma unroll 1
    for (int blk = g; blk < nblk; blk += G) {  // uniform in a wavefront
      const int r0 = blk * kRowsPerBlock, r1 = min(n, r0 + kRowsPerBlock);
      T p[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) p[c] = 0;
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        const int r = r0 + q * NT + vt;
        if (r0 + q * NT < r1) {
          const uint32_t rc = (uint32_t)min(r, r1 - 1);
          const T w = W[rc];
          T v[8];
#pragma unroll
          for (int c = 0; c < 8; ++c) v[c] = (V + (size_t)min(c0 + c, j) * n)[rc];
#pragma unroll
          for (int c = 0; c < 8; ++c) p[c] += r < r1 && c0 + c < cnt ? v[c] * w : (T)0;
        }
      }
      double pd[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) pd[c] = (double)p[c];
      ReduceScatter<8, 32>::run(pd, lane);
      if (lane % 8 == 0) red[(((c0 >> 3) * nblk + blk) * NW + wave) * 8 + lane / 8] = pd[0];
    }
  }
}

template <typename T, bool HAS_VAL>
__global__ __launch_bounds__(kWideThreads) void k_solve_wide(LzArgs a, WideLds L, int steps, int shift, double tol,
                                                             ebtc_diag* diag, double* ckpt) {
  extern __shared__ __align__(16) unsigned char dyn[];
  __shared__ double part[kWideBlocks][kDotsWindow];
  __shared__ double cs[kDotsWindow];
  __shared__ double ta[kDotsWindow];
  __shared__ double tb[kDotsWindow];
  __shared__ double nsum[kWideBlocks * 4];
  __shared__ double chunks[kMaxChunks];
  __shared__ double npart_l[1];
  __shared__ RState st_l;
  constexpr bool F64 = sizeof(T) == 8;
  const int64_t r = blockIdx.x;
  const Task& tk = a.tasks[r];
  const int n = __builtin_amdgcn_readfirstlane(tk.n), tid = threadIdx.x;
  const int nblk = (n + kRowsPerBlock - 1) / kRowsPerBlock;
  T* xs = (T*)(dyn + L.x_off);
  int* rp_l = (int*)(dyn + L.rp_off);
  T* prod = (T*)(dyn + L.work_off);
  double* wred = (double*)(dyn + L.work_off);
  T* V = (T*)a.V + uniform64(tk.vec_off);
  T* W = (T*)a.W + uniform64(tk.w_off);
  T* u = (T*)a.U + uniform64(tk.u_off);
  const int64_t nz = uniform64(tk.nnz_off);
  const int32_t* rp = a.row_ptr + uniform64(tk.rowptr_off);
  const int32_t* ci = a.col_idx + nz;
  const T* va = HAS_VAL ? (const T*)a.values + nz : nullptr;
  for (int i = tid; i <= n; i += kWideThreads) rp_l[i] = rp[i];
  // start (k_start): raw v_0 = 1 with scale s_0 = 1/sqrt(n)
  for (int i = tid; i < n; i += kWideThreads) {
    V[i] = (T)1;
    xs[i] = (T)1;
  }
  RState* st = &st_l;
  if (tid == 0) {
    st->beta0 = sqrt((double)n);
    st->s[0] = 1.0 / st->beta0;
    st->theta = 0.0;
    st->est = 0.0;
    st->m_used = 0;
    st->flags = 0;
    st->done = 0;
  }
  __syncthreads();
  StepClose c{0.0, 0};  // the last step's, in every thread
  for (int j = 0; j < steps; ++j) {
    double sj = 0.0;
    if (j == 0) {
      sj = st->s[0];
    } else {
      if (tid == 0) record_close(st, c, j);
      if (c.flags) break;
      sj = 1.0 / c.beta;
    }
    wide_spmv<T, HAS_VAL>(rp_l, ci, va, xs, n, sj, W, prod, j == 0);
    __syncthreads();
    // the dot kernel's thread count for this window (dots_threads of its window class)
    const int cnt = j + 1, P = cnt <= 8 ? 8 : cnt <= 16 ? 16 : cnt <= 32 ? 32 : 64;
    const bool wide = dots_threads(P, F64 ? 8 : 4) == kDotsThreads;
    if (wide) wide_dots<T, kDotsThreads>(V, W, n, nblk, j, wred);
    else wide_dots<T, kBlock>(V, W, n, nblk, j, wred);
    __syncthreads();
    const int nw = (wide ? kDotsThreads : kBlock) / 64;
    if (tid < cnt * nblk) {  // at most 64 x 8
      const int b = tid / cnt, d = tid - b * cnt;
      const double* q = wred + ((size_t)((d >> 3) * nblk + b) * nw) * 8 + (d & 7);
      double s = 0.0;
      for (int w = 0; w < nw; ++w) s += q[w * 8];
      part[b][d] = s;
    }
    __syncthreads();
    if (tid < kDotsWindow) {  // the update kernel's coefficients (chunks of one row block)
      double coef = 0.0;
      if (tid < cnt) {
        double t = 0.0;
        for (int b = 0; b < nblk; ++b) t += 0.0 + part[b][tid];
        const double si = st->s[tid], h = si * t;
        coef = h * si;
        if (tid == j) {
          st->alpha[j] = h;
          double sc = fabs(h);  // breakdown reference of step j: max(|alpha_0..j|, beta_0..j-1)
          if (j > 0) sc = fmax(sc, fmax(st->scal[j - 1], st->beta[j - 1]));
          st->scal[j] = isfinite(h) ? sc : h;
        }
      }
      cs[tid] = coef;
    }
    __syncthreads();
    {  // v~_{j+1} = w - sum_i c_i Vraw_i, two rows per thread at a time
      constexpr int RQ = 2;
      const int t = fresh_tid();
      T* dst = V + (size_t)(j + 1) * n;
#pragma unroll 1
      for (int h = 0; h < n; h += RQ * kWideThreads) {
        uint32_t row[RQ];
        double acc[RQ];
#pragma unroll
        for (int q = 0; q < RQ; ++q) {
          row[q] = (uint32_t)min(h + q * kWideThreads + t, n - 1);
          acc[q] = (double)W[row[q]];
        }
#pragma unroll 1
        for (int c0 = 0; c0 < cnt; c0 += 8) {
          T v[RQ][8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const T* vi = V + (size_t)min(c0 + i, j) * n;
#pragma unroll
            for (int q = 0; q < RQ; ++q) v[q][i] = vi[row[q]];
          }
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const double k = cs[c0 + i];
#pragma unroll
            for (int q = 0; q < RQ; ++q) acc[q] -= k * (double)v[q][i];
          }
        }
#pragma unroll
        for (int q = 0; q < RQ; ++q)
          if (h + q * kWideThreads + t < n) {
            const T out = (T)acc[q];
            dst[row[q]] = out;
            xs[row[q]] = out;
          }
      }
    }
    __syncthreads();
    {  // squared norms of the row blocks, in the order of the 256-thread update
      const int t = fresh_tid(), vt = t % kBlock;
      for (int b = t / kBlock; b < nblk; b += kWideThreads / kBlock) {
        const int r0 = b * kRowsPerBlock, r1 = min(n, r0 + kRowsPerBlock);
        double nrm = 0.0;
        for (int i = r0 + vt; i < r1; i += kBlock) {
          const T out = xs[i];
          nrm += (double)out * (double)out;
        }
        nrm = wave_sum(nrm);
        if ((t & 63) == 0) nsum[b * 4 + (vt >> 6)] = nrm;
      }
    }
    __syncthreads();
    double ss = 0.0;
    for (int b = 0; b < nblk; ++b) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < 4; ++w) s += nsum[b * 4 + w];
      ss += 0.0 + s;
    }
    if (tid == 0) npart_l[0] = ss;
    c = close_sum(st, ss, j, a.eps);
    if (a.m_fixed == 0) {  // the adaptive check, by the first wavefront
      if (tid < 64) {
        const TriPrep p{j + 1, c.beta, st->flags, false};
        if (c.flags) {
          if (tid == 0) {
            st->beta[j] = c.beta;
            st->flags |= c.flags;
            st->done = 1;
            st->m_used = j + 1;
          }
        } else {
          tridiag_load(st, p, ta, tb);
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          tridiag_finish<kDotsWindow>(a, st, r, 1, j, p, ta, tb, shift, tol, nullptr, nullptr);
        }
      }
      __syncthreads();
      if (st->done) break;
    }
  }
  __syncthreads();
  const TriPrep p = tridiag_prepare(a, st, npart_l, 1, r, 0, 0, steps, diag, chunks);
  if (!p.exit) {
    if (tid < 64) tridiag_load(st, p, ta, tb);
    __syncthreads();
    if (tid < 64) tridiag_finish<kDotsWindow>(a, st, r, 0, 0, p, ta, tb, shift, tol, diag, ckpt);
  }
  __syncthreads();
  // combination (k_combine): u = sum_i (beta0 y_i s_i) Vraw_i, FP64, i ascending
  const int k = st->m_used;
  if (tid < k) cs[tid] = st->beta0 * st->y[tid] * st->s[tid];
  __syncthreads();
  bool finite = true;
  for (int row = tid; row < n; row += kWideThreads) {
    double acc = 0.0;
#pragma unroll 8
    for (int i = 0; i < k; ++i) acc += cs[i] * (double)V[(size_t)i * n + row];
    const T out = (T)acc;
    u[row] = out;
    finite = finite && isfinite((double)out);
  }
  if (__syncthreads_or(!finite) && tid == 0) {
    st->flags |= EBTC_FLAG_NONFINITE;
    if (diag) atomicOr(&diag[r].flags, EBTC_FLAG_NONFINITE);
  }
  __syncthreads();
  // the state to the workspace (the realization sum reads theta)
  const double* src = (const double*)st;
  double* dst = (double*)(a.state + r);
  static_assert(sizeof(RState) % sizeof(double) == 0, "state copy");
  for (int i = tid; i < (int)(sizeof(RState) / sizeof(double)); i += kWideThreads) dst[i] = src[i];
}

size_t align16(size_t x) { return (x + 15) / 16 * 16; }

template <typename T>
WideLds wide_lds(int n_max) {
  WideLds L{};
  L.rp_off = (int32_t)align16((size_t)n_max * sizeof(T));
  L.work_off = (int32_t)align16(L.rp_off + ((size_t)n_max + 1) * 4);
  L.bytes = (int32_t)(L.work_off + align16(wide_work<T>()));
  return L;
}

template <typename T, bool HAS_VAL>
hipError_t wide_t(const LzArgs& a, int64_t count, int steps, int shift, double tol, ebtc_diag* diag, double* ckpt,
                  int n_max, hipStream_t s) {
  const WideLds L = wide_lds<T>(n_max);
  hipLaunchKernelGGL((k_solve_wide<T, HAS_VAL>), dim3((unsigned)count), dim3(kWideThreads), (size_t)L.bytes, s, a, L,
                     steps, shift, tol, diag, ckpt);
  return hipGetLastError();
}

constexpr size_t kWideStatic = 16 * 1024;  // the kernels' static LDS at most
}  // namespace

bool wide_fits(int dtype, int n_max) {
  if (n_max < 1 || n_max > kWideBlocks * kRowsPerBlock) return false;
  const WideLds L = dtype == EBTC_F64 ? wide_lds<double>(n_max) : wide_lds<float>(n_max);
  return (size_t)L.bytes + kWideStatic <= kLdsBytes;
}

hipError_t prepare_wide_kernels() {
  static const hipError_t e = [] {
    const int dyn = (int)(kLdsBytes - kWideStatic);
    hipError_t r = hipFuncSetAttribute((const void*)k_solve_wide<float, true>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    if (r == hipSuccess)
      r = hipFuncSetAttribute((const void*)k_solve_wide<float, false>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    if (r == hipSuccess)
      r = hipFuncSetAttribute((const void*)k_solve_wide<double, true>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    if (r == hipSuccess)
      r = hipFuncSetAttribute((const void*)k_solve_wide<double, false>, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    return r;
  }();
  return e;
}

hipError_t launch_solve_wide(int dtype, bool has_val, const LzArgs& a, int64_t count, int steps, int shift, double tol,
                             ebtc_diag* diag, double* ckpt, int n_max, hipStream_t s) {
  if (a.window != 0 || !wide_fits(dtype, n_max) || steps < 1 || steps > kDotsWindow) return hipErrorInvalidValue;
  if (dtype == EBTC_F64)
    return has_val ? wide_t<double, true>(a, count, steps, shift, tol, diag, ckpt, n_max, s)
                   : wide_t<double, false>(a, count, steps, shift, tol, diag, ckpt, n_max, s);
  return has_val ? wide_t<float, true>(a, count, steps, shift, tol, diag, ckpt, n_max, s)
                 : wide_t<float, false>(a, count, steps, shift, tol, diag, ckpt, n_max, s);
}

}  // namespace ebtc
