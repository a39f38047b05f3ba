// The whole Lanczos process of one realization in one workgroup (gfx950, 256 threads), for batches
// whose realizations each fit one row block (n <= kRowsPerBlock) and need at most 64 steps: the tiny
// plain-method workload and the identification-rate experiments (backgrounds of 1024-9000 nodes,
// "Multiple backgrounds scenario"), where each phase of the per-phase schedule is a launch over a few
// kilobytes and the run is launch latency.
//
// One launch replaces the per-phase sequence start, [SpMV, Gram-Schmidt dots and update, adaptive
// check] x m, small exponential, basis combination: workgroup barriers take the place of kernel
// boundaries, and the realization's working set stays in LDS -- the state, the partial sums, the row
// pointers, the gathered vector v_j and the product w always; the CSR entries where they fit, and the
// basis where it fits beside them and costs no round of workgroups (solve_lds, per launch), else the input
// arrays and the workspace.
// Every phase keeps the per-phase kernels' arithmetic in their thread order: the CSR-stream SpMV's (which the
// column-segmented and entry-balanced forms share bit for bit), the dot partials of the dot kernel the window would
// get (1024 or 256 threads; a partial's bits do not depend on how many vectors one pass covers, so they are formed
// eight vectors at a time), the update and norm of the 256-thread update kernel, the same small exponential and
// combination. So a realization's results equal the per-phase schedule's bit for bit whichever schedule its batch
// takes; only where the data lives changes.
// What bounds it: few realizations (20 x n=200: 0.151 to 0.115 ms) one workgroup's chain of dependent LDS reads,
// reductions and barriers, 10000 cycles a step; many (2000 x n=1024, FP64, 13 adaptive steps: 1.69 to 0.57 ms) the
// adaptive check's chain, 10000 of a step's 37000 cycles, and the basis, read twice per step from the last-level
// cache. Four workgroups to a compute unit hide some of each, for which the LDS holds 16-bit columns and no product
// slots beside the entries, and the step loop's registers stay within 128 (three: 0.61 ms).
#include <algorithm>

#include "step_device.h"

namespace ebtc {
namespace {

constexpr int kSolveCap = kRowsPerBlock;  // product slots: every row of a simple graph on <= 2048 nodes fits
// Wavefronts per SIMD, workgroups per compute unit. FP32 without the entries in LDS two, for whose registers more of the
// product's loads are in flight (n=1500, degree 60, m=20: 4.42 to 3.94 ms; FP64 would lose 7%).
constexpr int solve_occ(bool csr_lds, size_t es) { return csr_lds || es == 8 ? 4 : 2; }
constexpr int kSolveUnits = 256;  // compute units
constexpr int kSolveRed = (kDotsThreads / 64) * 16;

// Dynamic LDS of one launch (byte offsets, host-computed from the largest realization).
struct SolveLds {
  int32_t x_off, w_off, rp_off;  // v_j, w (n_max elements each), row pointers (n_max + 1)
  int32_t v_off;                 // basis ((steps + 1) x n_max elements), or -1: in the workspace
  int32_t c_off, val_off;        // CSR columns and values (z_max each), or -1: read from the input
  int32_t z_max;
  int32_t bytes;
};

// The thread's index, computed anew: what follows from it is then not carried in registers around the step loop,
// which costs more (spilled, in scratch memory) than forming it again.
__device__ inline int fresh_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Eight vectors of up to four rows per thread, rows h + q kBlock + tid (clamped: the callers mask), all loads at
// once.
template <typename T>
__device__ inline void load_rows(const T* V, int n, int tid, int c0, int j, int h, T (&v)[4][8]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (h + q * kBlock < n) {  // uniform
      const uint32_t r = (uint32_t)min(h + q * kBlock + tid, n - 1);
#pragma unroll
      for (int c = 0; c < 8; ++c) v[q][c] = (V + (size_t)min(c0 + c, j) * n)[r];
    } else {
#pragma unroll
      for (int c = 0; c < 8; ++c) v[q][c] = 0;
    }
  }
}

// Dot partials of step j over the workgroup's n rows, 16 vectors between barriers: block_dots' arithmetic for NT
// threads (thread t of NT sums rows t, t + NT, ... in order, the sums go wave by wave, then over the waves in order).
template <typename T, int NT>
__device__ inline void solve_dots(const T* V, int n, int j, const T* ws, double* part, double* red) {
  constexpr int PASSES = NT / kBlock, RPT = kRowsPerBlock / NT, NW = NT / 64;
  const int tid = fresh_tid(), lane = tid & 63, wave = tid >> 6, cnt = j + 1;
  for (int d0 = 0; d0 < cnt; d0 += 16) {
#pragma unroll 1
    for (int c0 = d0; c0 < min(cnt, d0 + 16); c0 += 8) {
      double* out = red + ((c0 - d0) >> 3) * NW * 8;
      T v[8], vn[8];
      auto load = [&](T (&x)[8], int r0) {  // vectors c0 .. c0 + 7 of rows r0 + tid (clamped: masked below)
        const uint32_t rc = (uint32_t)min(r0 + tid, n - 1);
#pragma unroll
        for (int c = 0; c < 8; ++c) x[c] = (V + (size_t)min(c0 + c, j) * n)[rc];
      };
      auto add = [&](T (&p)[8], const T (&x)[8], int r0) {
        const int r = r0 + tid;
        const T w = ws[min(r, n - 1)];
#pragma unroll
        for (int c = 0; c < 8; ++c) p[c] += r < n && c0 + c < cnt ? x[c] * w : (T)0;
      };
      load(v, 0);
#pragma unroll 1
      for (int t0 = 0; t0 < NT; t0 += kBlock) {
        T p[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) p[c] = 0;
        if (t0 < n) {  // else no rows: zeros
          if constexpr (PASSES == 1) {  // row by row of the thread, the next row's loads ahead
#pragma unroll
            for (int q = 0; q < RPT; q += 2) {
              if (q * NT < n) {
                if ((q + 1) * NT < n) load(vn, (q + 1) * NT);
                add(p, v, q * NT);
                if ((q + 2) * NT < n) load(v, (q + 2) * NT);
                if ((q + 1) * NT < n) add(p, vn, (q + 1) * NT);
              }
            }
          } else {
            if (t0 + kBlock < min(n, NT)) load(vn, t0 + kBlock);  // the next pass's
            add(p, v, t0);
            if (NT + t0 < n) {
              load(v, NT + t0);
              add(p, v, NT + t0);
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) v[c] = vn[c];
          }
        }
        double pd[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) pd[c] = (double)p[c];
        if (t0 < n) ReduceScatter<8, 32>::run(pd, lane);
        if (lane % 8 == 0) out[(t0 / 64 + wave) * 8 + lane / 8] = pd[0];
      }
    }
    __syncthreads();
    if (tid < 16 && d0 + tid < cnt) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += red[((tid >> 3) * NW + w) * 8 + (tid & 7)];
      part[d0 + tid] = s;
    }
    __syncthreads();
  }
}

// v~_{j+1} = w - sum_i c_i Vraw_i and its squared norm: update_body's arithmetic for one row block, eight vectors
// of up to four rows per thread loaded at a time. xs also receives v~_{j+1}. Returns the norm's square.
template <typename T>
__device__ inline double solve_update(RState* st, T* V, int n, int j, const double* part, double* cs, double* red,
                                    const T* ws, T* xs) {
  const int tid = fresh_tid(), cnt = j + 1;
  if (tid < kDotsWindow) {
    double coef = 0.0;
    if (tid < cnt) {
      const double t = 0.0 + part[tid], si = st->s[tid], h = si * t;
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
  T* dst = V + (size_t)(j + 1) * n;
  double nrm = 0.0;
#pragma unroll 1
  for (int h = 0; h < n; h += 4 * kBlock) {
    double acc[4];
    int rc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      rc[q] = min(h + q * kBlock + tid, n - 1);
      acc[q] = (double)ws[rc[q]];
    }
#pragma unroll 1
    for (int c0 = 0; c0 < cnt; c0 += 8) {
      T v[4][8];
      load_rows(V, n, tid, c0, j, h, v);
      double k[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) k[c] = cs[c0 + c];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (h + q * kBlock < n) {
#pragma unroll
          for (int c = 0; c < 8; ++c) acc[q] -= k[c] * (double)v[q][c];
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = h + q * kBlock + tid;
      if (r < n) {
        const T out = (T)acc[q];
        dst[r] = out;
        xs[r] = out;
        nrm += (double)out * (double)out;
      }
    }
  }
  return block_sum<kBlock>(nrm, red);
}

__device__ inline void solve_tridiag(const LzArgs& a, RState* st, const double* npart, int64_t r, int steps, int shift,
                                     double tol, ebtc_diag* diag, double* ckpt, double* chunks, double* ta, double* tb) {
  const TriPrep p = tridiag_prepare(a, st, npart, 1, r, 0, 0, steps, diag, chunks);
  if (!p.exit) {
    if (threadIdx.x < 64) tridiag_load(st, p, ta, tb);
    __syncthreads();
    if (threadIdx.x < 64) tridiag_finish<kDotsWindow>(a, st, r, 0, 0, p, ta, tb, shift, tol, diag, ckpt);
  }
  __syncthreads();
}

// w = s_j A v_j with the realization's entries in LDS: one thread per row, the row's products in entry
// order, each rounded to T before its FP64 add -- the CSR-stream form's arithmetic (its products are
// staged in LDS before the sum) -- eight entries' loads issued ahead of the adds.
template <typename T, bool HAS_VAL>
__device__ inline void solve_spmv_lds(const int* rp_l, const uint16_t* cl, const T* vl, const T* xs, int n, double sj,
                                      T* ws) {
  for (int row = fresh_tid(); row < n; row += kBlock) {
    double acc = 0.0;
    const int e1 = rp_l[row + 1];
    int k = rp_l[row];
    for (; k + 24 <= e1; k += 8) {  // of long rows, without the tests (stars of n=1500, FP64, m=20: 1.20 to 0.79 ms)
      T x[8], v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        x[u] = xs[cl[k + u]];
        if constexpr (HAS_VAL) v[u] = vl[k + u];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        T pr = x[u];
        if constexpr (HAS_VAL) pr = v[u] * x[u];
        acc += (double)pr;
      }
    }
    for (; k < e1; k += 8) {
      T x[8], v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int e = min(k + u, e1 - 1);
        x[u] = xs[cl[e]];
        if constexpr (HAS_VAL) v[u] = vl[e];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        T pr = x[u];
        if constexpr (HAS_VAL) pr = v[u] * x[u];
        acc += (double)(k + u < e1 ? pr : (T)0);  // the sum starts at +0, which adding +0 keeps
      }
    }
    ws[row] = (T)(acc * sj);
  }
}

template <typename T, bool HAS_VAL, bool CSR_LDS>
__device__ inline void solve_spmv(int j, const int32_t* ci, const uint16_t* cl, const T* va, const T* xs, int n, double sj, int* rp_l,
                                  T* prod, T* ws, double* red) {
  if constexpr (CSR_LDS) {
    solve_spmv_lds<T, HAS_VAL>(rp_l, cl, va, xs, n, sj, ws);  // v_0 = 1: the row sums of the values
    return;
  }
  if (j == 0)  // A 1: each row's values summed in FP64 in entry order (the first-product kernels)
    spmv_stream_rows<T, HAS_VAL, kBlock, kSolveCap, true, true, !CSR_LDS>(nullptr, ci, va, xs, 0, n, sj, rp_l, prod,
                                                                          ws, red);
  else
    spmv_stream_rows<T, HAS_VAL, kBlock, kSolveCap, false, true, !CSR_LDS>(nullptr, ci, va, xs, 0, n, sj, rp_l, prod,
                                                                           ws, red);
}

__device__ inline int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ inline Task uniform_task(const Task& t) {
  Task u = t;
  u.rowptr_off = uniform64(t.rowptr_off);
  u.nnz_off = uniform64(t.nnz_off);
  u.vec_off = uniform64(t.vec_off);
  u.u_off = uniform64(t.u_off);
  u.n = __builtin_amdgcn_readfirstlane(t.n);
  return u;
}

template <typename T, bool HAS_VAL, bool CSR_LDS, bool V_LDS>
__global__ __launch_bounds__(kBlock, solve_occ(CSR_LDS, sizeof(T))) void k_solve_1(LzArgs a, SolveLds L, int steps, int shift, double tol,
                                                    ebtc_diag* diag, double* ckpt) {
  extern __shared__ __align__(16) unsigned char dyn[];
  __shared__ T prod[CSR_LDS ? 1 : kSolveCap];
  __shared__ double red_d[kSolveRed];
  __shared__ double cs[kDotsWindow];
  __shared__ double red[kWaves];
  __shared__ double chunks[kMaxChunks];
  __shared__ double ta[kDotsWindow];
  __shared__ double tb[kDotsWindow];
  double* dcoef = ta;
  __shared__ double part_l[kPartStride];
  __shared__ double npart_l[1];
  __shared__ RState st_l;
  const int64_t r = logical_block();  // one row block per realization
  // in scalar registers, where the compiler does not put what it loads: the loads of the basis then take their
  // addresses from them
  const Task tk = uniform_task(a.tasks[r]);
  const int n = tk.n, tid = threadIdx.x;
  T* xs = (T*)(dyn + L.x_off);
  T* ws = (T*)(dyn + L.w_off);
  int* rp_l = (int*)(dyn + L.rp_off);
  T* V;  // one address space: loads that could be either wait for both
  if constexpr (V_LDS) V = (T*)(dyn + L.v_off); else V = (T*)a.V + tk.vec_off;
  const int32_t* rp = a.row_ptr + tk.rowptr_off;
  for (int i = tid; i <= n; i += kBlock) rp_l[i] = rp[i];
  const int32_t* ci = a.col_idx + tk.nnz_off;
  const T* va = HAS_VAL ? (const T*)a.values + tk.nnz_off : nullptr;
  uint16_t* cl = (uint16_t*)(dyn + L.c_off);  // n <= 2048
  if constexpr (CSR_LDS) {  // the realization's entries, once, into LDS
    const int z = min(rp[n], L.z_max);
    for (int e = tid; e < z; e += kBlock) cl[e] = (uint16_t)__builtin_nontemporal_load(ci + e);
    if constexpr (HAS_VAL) {
      T* vl = (T*)(dyn + L.val_off);
      for (int e = tid; e < z; e += kBlock) vl[e] = __builtin_nontemporal_load(va + e);
      va = vl;
    }
  }
  // start (k_start): raw v_0 = 1 with scale s_0 = 1/sqrt(n)
  for (int i = tid; i < n; i += kBlock) {
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
  constexpr bool F64 = sizeof(T) == 8;
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
    solve_spmv<T, HAS_VAL, CSR_LDS>(j, ci, cl, va, xs, n, sj, rp_l, prod, ws, red);
    __syncthreads();
    // the dot kernel's thread count for this window (dots_threads of its window class)
    const int cnt = j + 1, P = cnt <= 8 ? 8 : cnt <= 16 ? 16 : cnt <= 32 ? 32 : 64;
    if (dots_threads(P, F64 ? 8 : 4) == kDotsThreads) solve_dots<T, kDotsThreads>(V, n, j, ws, part_l, red_d);
    else solve_dots<T, kBlock>(V, n, j, ws, part_l, red_d);
    const double ss = solve_update<T>(st, V, n, j, part_l, cs, red, ws, xs);
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
  solve_tridiag(a, st, npart_l, r, steps, shift, tol, diag, ckpt, chunks, ta, tb);
  // combination (k_combine): u = sum_i (beta0 y_i s_i) Vraw_i, FP64, i ascending
  const int k = st->m_used;
  if (tid < k) dcoef[tid] = st->beta0 * st->y[tid] * st->s[tid];
  __syncthreads();
  T* u = (T*)a.U + tk.u_off;
  bool finite = true;
#pragma unroll
  for (int q = 0; q < kRowsPerThread; ++q) {
    const int row = q * kBlock + tid;
    if (row < n) {
      double acc = 0.0;
#pragma unroll 8
      for (int i = 0; i < k; ++i) acc += dcoef[i] * (double)V[(size_t)i * n + row];
      const T out = (T)acc;
      u[row] = out;
      finite = finite && isfinite((double)out);
    }
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
  for (int i = tid; i < (int)(sizeof(RState) / sizeof(double)); i += kBlock) dst[i] = src[i];
}

// Static LDS of an instantiation (queried once) and its opt-in to the rest of the 160 KB as dynamic LDS.
template <typename T, bool HAS_VAL, bool CSR_LDS, bool V_LDS>
size_t solve_static_bytes(hipError_t* err) {
  static size_t bytes = 0;
  static const hipError_t e = [] {
    const void* k = (const void*)k_solve_1<T, HAS_VAL, CSR_LDS, V_LDS>;
    hipFuncAttributes fa{};
    hipError_t r = hipFuncGetAttributes(&fa, k);
    if (r != hipSuccess) return r;
    bytes = fa.sharedSizeBytes;
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kLdsBytes - bytes));
  }();
  if (e != hipSuccess) *err = e;
  return bytes;
}

// The largest static LDS of the instantiations that a launch chooses from.
template <typename T, bool HAS_VAL>
hipError_t prepare_solve_t(size_t* bytes = nullptr, size_t* csr = nullptr) {
  hipError_t e = hipSuccess;
  const size_t b = std::max(std::max(solve_static_bytes<T, HAS_VAL, true, true>(&e), solve_static_bytes<T, HAS_VAL, true, false>(&e)),
                            std::max(solve_static_bytes<T, HAS_VAL, false, true>(&e), solve_static_bytes<T, HAS_VAL, false, false>(&e)));
  if (bytes) *bytes = b;
  if (csr) *csr = solve_static_bytes<T, HAS_VAL, true, true>(&e);
  return e;
}

size_t align16(size_t x) { return (x + 15) / 16 * 16; }

// LDS plan of a launch: v_j, w and the row pointers always, then the CSR entries where they fit, then the basis where it
// fits beside them (or, without them, alone). The entries come first: read from memory the product walks them chunk by
// chunk with barriers (300 x n=700, degree 20, FP64, m=20: 1.03 ms with the basis in LDS, 0.41 with the entries). The
// basis stays in the workspace, too, where a compute unit then holds so many more workgroups that the launch takes fewer
// rounds (1500 x n=1200, degree 3, FP64, m=10: 0.93 ms with the basis in LDS, 0.56 without; 300 x n=1500, degree 60, FP32,
// m=20, no entries in LDS: 9.67 and 4.71; in one round either way, 300 of n=300: 0.20 and 0.22). fixed, fixed_csr: static
// LDS at most, and with the entries in LDS.
SolveLds solve_lds(size_t es, bool has_val, int n_max, int64_t z_max, int steps, int64_t count, size_t fixed,
                   size_t fixed_csr) {
  const size_t budget = kLdsBytes - fixed;
  SolveLds L{};
  size_t off = 0;
  L.x_off = (int32_t)off;
  off = align16(off + (size_t)n_max * es);
  L.w_off = (int32_t)off;
  off = align16(off + (size_t)n_max * es);
  L.rp_off = (int32_t)off;
  off = align16(off + (size_t)(n_max + 1) * 4);
  const size_t vb = (size_t)(steps + 1) * n_max * es;
  const size_t cb = align16((size_t)z_max * 2) + (has_val ? (size_t)z_max * es : 0);
  L.v_off = L.c_off = L.val_off = -1;
  const bool csr = off + cb <= budget;
  const size_t rest = csr ? align16(off + cb) : off;  // beside the basis
  const auto held = [&](size_t bytes) {  // workgroups of a compute unit
    return std::min<int64_t>(solve_occ(csr, es), kLdsBytes / (bytes + (csr ? fixed_csr : fixed)));
  };
  const auto rounds = [&](size_t bytes) {
    const int64_t once = kSolveUnits * held(bytes);
    return (count + once - 1) / once;
  };
  const bool basis = rest + vb <= budget && rounds(rest + vb) <= rounds(rest);
  if (csr) {
    L.c_off = (int32_t)off;
    off = align16(off + (size_t)z_max * 2);
    if (has_val) {
      L.val_off = (int32_t)off;
      off = align16(off + (size_t)z_max * es);
    }
  }
  if (basis) {
    L.v_off = (int32_t)off;
    off = align16(off + vb);
  }
  L.z_max = (int32_t)std::min<int64_t>(z_max, INT32_MAX);
  L.bytes = (int32_t)off;
  return L;
}

template <typename T, bool HAS_VAL>
hipError_t solve_t(const LzArgs& a, int64_t count, int steps, int shift, double tol, ebtc_diag* diag, double* ckpt,
                   int n_max, int64_t z_max, hipStream_t s) {
  size_t fixed = 0, fixed_csr = 0;
  const hipError_t e = prepare_solve_t<T, HAS_VAL>(&fixed, &fixed_csr);
  if (e != hipSuccess) return e;
  const SolveLds L = solve_lds(sizeof(T), HAS_VAL, n_max, z_max, steps, count, fixed, fixed_csr);
  auto* solve = L.v_off >= 0 ? (L.c_off >= 0 ? k_solve_1<T, HAS_VAL, true, true> : k_solve_1<T, HAS_VAL, false, true>)
                             : (L.c_off >= 0 ? k_solve_1<T, HAS_VAL, true, false> : k_solve_1<T, HAS_VAL, false, false>);
  hipLaunchKernelGGL(solve, dim3((unsigned)count), dim3(kBlock), (size_t)L.bytes, s, a, L, steps, shift, tol, diag, ckpt);
  return hipGetLastError();
}

}  // namespace

hipError_t prepare_solve_kernels() {
  static const hipError_t e = [] {
    hipError_t r = prepare_solve_t<float, true>();
    if (r == hipSuccess) r = prepare_solve_t<float, false>();
    if (r == hipSuccess) r = prepare_solve_t<double, true>();
    if (r == hipSuccess) r = prepare_solve_t<double, false>();
    return r;
  }();
  return e;
}

hipError_t launch_solve_1(int dtype, bool has_val, const LzArgs& a, int64_t count, int steps, int shift, double tol,
                          ebtc_diag* diag, double* ckpt, int n_max, int64_t z_max, hipStream_t s) {
  if (a.window != 0 || n_max < 1 || n_max > kRowsPerBlock || steps < 1 || steps > kDotsWindow)
    return hipErrorInvalidValue;
  if (dtype == EBTC_F64)
    return has_val ? solve_t<double, true>(a, count, steps, shift, tol, diag, ckpt, n_max, z_max, s)
                   : solve_t<double, false>(a, count, steps, shift, tol, diag, ckpt, n_max, z_max, s);
  return has_val ? solve_t<float, true>(a, count, steps, shift, tol, diag, ckpt, n_max, z_max, s)
                 : solve_t<float, false>(a, count, steps, shift, tol, diag, ckpt, n_max, z_max, s);
}

}  // namespace ebtc
