// Device steps of the Lanczos process shared by the per-phase kernels (one launch per phase over
// every realization) and the single-kernel solve (one workgroup runs a realization's whole process):
// both call these functions, so they compute the same bits.
#pragma once

#include "device_common.h"

namespace ebtc {
namespace {

// ------------------------------------------------------------------------------- phase A: SpMV
// Records the close of step j - 1, by step j's product launch, in the realization's state (one thread).
__device__ inline void record_close(RState* st, const StepClose& c, int j) {
  st->beta[j - 1] = c.beta;
  if (c.flags) {
    st->flags |= c.flags;
    st->done = 2 + j;
    st->m_used = j;
  } else {
    st->s[j] = 1.0 / c.beta;
  }
}

// Opens phase A of step j: closes step j-1 from its norm partials (all workgroups of the
// realization compute the same bits; workgroup 0 records them). Returns false when the
// realization is finished; *sj = 1/beta_{j-1} (or s_0 at j = 0).
__device__ inline bool open_step(const LzArgs& a, const Task& tk, RState* st, int blk, int j, double* chunks,
                                 double* sj, const double* npart = nullptr) {
  if (product_skipped(a, st, j)) return false;
  if (j == 0) {
    *sj = st->s[0];
    return true;
  }
  const StepClose c = close_step(st, npart ? npart : a.npart + tk.part_off / kPartStride, tk.nblk, j - 1, a.eps, chunks);
  if (blk == 0 && threadIdx.x == 0) record_close(st, c, j);
  if (c.flags) return false;
  *sj = 1.0 / c.beta;
  return true;
}

constexpr int kStreamRows = 256;
constexpr int kStreamU = 8;
template <typename T>
struct StreamShape {
  static constexpr int CAP = sizeof(T) == 8 ? 3072 : 6144;  // product slots (24 KB)
};

// Paneled form: rows with more entries are summed apart: than kTileHubMin and six times the realization's mean, or than
// the stream form's capacity, beyond which that form's sums are not in entry order.
constexpr int kTileHubMin = 256;
template <typename T>
__device__ inline int tile_hub(int64_t n, int64_t z) {
  return (int)max((int64_t)kTileHubMin, min((int64_t)StreamShape<T>::CAP, 6 * z / max(n, (int64_t)1)));
}

// SEQ_HUB: a row beyond the capacity is summed by one thread in entry order instead (the first
// product's arithmetic, for a caller that must reproduce it).
// RP_LDS: rp_lds already holds the rows' pointers (rp unused). NT_LOADS: the entries are read with the
// non-temporal policy (they live in HBM and are read once per product); off when they sit in LDS.
// HUB_NT: a row beyond the capacity is reduced in the order of a workgroup of HUB_NT threads (the
// first HUB_NT threads form the per-thread sums; the other waves add exact zeros).
template <typename T, bool HAS_VAL, int NT = kBlock, int CAP = StreamShape<T>::CAP, bool SEQ_HUB = false,
          bool RP_LDS = false, bool NT_LOADS = true, int HUB_NT = NT>
__device__ inline void spmv_stream_rows(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                        const T* __restrict__ va, const T* __restrict__ x, int r0, int rows,
                                        double scale, int* rp_lds, T* prod, T* w_out, double* red) {
  constexpr int U = kStreamU;
  const int tid = threadIdx.x;
  if constexpr (!RP_LDS) {
    for (int i = tid; i <= rows; i += NT) rp_lds[i] = rp[r0 + i];
    __syncthreads();
  }
  int ra = 0;
  while (ra < rows) {
    const int nz0 = rp_lds[ra];
    if (SEQ_HUB && rp_lds[ra + 1] - nz0 > CAP) {
      if (tid == 0) {
        double acc = 0.0;
        for (int k = nz0; k < rp_lds[ra + 1]; ++k) {
          const T xv = x[ci[k]];
          if constexpr (HAS_VAL) acc += (double)(va[k] * xv); else acc += (double)xv;
        }
        w_out[ra] = (T)(acc * scale);
      }
      ++ra;
      continue;
    }
    if (rp_lds[ra + 1] - nz0 > CAP) {  // hub row: whole workgroup, direct gathers
      static_assert(HUB_NT <= NT && HUB_NT % 64 == 0, "hub reduction layout");
      const int e = rp_lds[ra + 1];
      T acc = 0;
      if (tid < HUB_NT)
        for (int k = nz0 + tid; k < e; k += HUB_NT) {
          const T xv = x[ci[k]];
          if constexpr (HAS_VAL) acc += va[k] * xv; else acc += xv;
        }
      const double tot = block_sum<NT>((double)acc, red);
      if (tid == 0) w_out[ra] = (T)(tot * scale);
      ++ra;
      continue;
    }
    // largest rb with rp[rb] - rp[ra] <= CAP (every thread finds the same rb)
    int lo = ra + 1, hi = rows;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (rp_lds[mid] - nz0 <= CAP) lo = mid; else hi = mid - 1;
    }
    const int rb = lo;
    const int cnt = rp_lds[rb] - nz0;
    for (int k0 = tid; k0 < cnt; k0 += NT * U) {
      int c[U];
      T v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = k0 + u * NT;
        // the matrix is read once per product: non-temporal loads leave the cache lines of the
        // gathered vector resident
        if constexpr (NT_LOADS) {
          c[u] = k < cnt ? __builtin_nontemporal_load(ci + nz0 + k) : -1;
          if constexpr (HAS_VAL) v[u] = k < cnt ? __builtin_nontemporal_load(va + nz0 + k) : (T)0;
        } else {
          c[u] = k < cnt ? ci[nz0 + k] : -1;
          if constexpr (HAS_VAL) v[u] = k < cnt ? va[nz0 + k] : (T)0;
        }
      }
      T xv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) xv[u] = c[u] >= 0 ? x[c[u]] : (T)0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = k0 + u * NT;
        if (k < cnt) {
          if constexpr (HAS_VAL) prod[k] = v[u] * xv[u]; else prod[k] = xv[u];
        }
      }
    }
    __syncthreads();
    for (int r = ra + tid; r < rb; r += NT) {
      double acc = 0.0;  // FP64: sequential sums over long (BA hub) rows stay accurate
      if constexpr (NT != kBlock) {
        const int e = rp_lds[r + 1] - nz0;
        for (int k = rp_lds[r] - nz0; k < e; ++k) acc += (double)prod[k];
      } else {
        // The loop within one 64-byte line of instructions: across two, a long row's chain takes up to 13% more time
        // (entry-balanced form, n=1e6 Barabasi-Albert, FP64: 0.241 and 0.275 ms a product).
        int k = (rp_lds[r] - nz0) * (int)sizeof(T);
        const int e = (rp_lds[r + 1] - nz0) * (int)sizeof(T);
        if (k < e) {
          asm volatile(".p2align 6" : "+v"(k), "+v"(acc));
          do {
            acc += (double)*(const T*)((const char*)prod + k);
            k += (int)sizeof(T);
          } while (k < e);
        }
      }
      w_out[r] = (T)(acc * scale);
    }
    __syncthreads();
    ra = rb;
  }
}

// ------------------------------------------------------------------------------- phase B: Gram-Schmidt
// Partial dots p_d = sum_rows Vraw_{lo+d}[r] * w[r] (d < cnt = j - lo + 1 <= P) of this workgroup's
// rows, reduced over the workgroup and stored to part_blk[d]. NT fixes the arithmetic: thread t of NT
// sums rows r0 + t, r0 + t + NT, ... and the per-thread sums are reduced wave by wave, then wave by
// wave in order. The workgroup runs it with NREAL threads (NT a multiple of NREAL), each taking the
// NT / NREAL threads t = tid, tid + NREAL, ... in turn, so a smaller workgroup computes the same
// bits. Basis loads are issued min(P, 8) vectors at a time (clamped to the last one, whose extra
// contributions are masked) so that many loads are in flight per thread. RING > 0: vector i lives in
// slot i % RING (the ring of the memory-bounded form). red: (NT / 64) * P doubles of LDS.
template <typename T, int P, int NT, int RING, int NREAL = NT>
__device__ inline void block_dots(const T* __restrict__ Vr, int n, int lo, int j, int r0, int r1,
                                  const T* wsrc, double* part_blk, double* red) {
  static_assert(P == 2 || P == 8 || P == 16 || P == 32 || P == 64, "lane layout of ReduceScatter");
  static_assert(NT % NREAL == 0 && NREAL % 64 == 0, "virtual thread layout");
  constexpr int RPT = kRowsPerBlock / NT;
  constexpr int CH = P < 8 ? P : 8;
  const int tid = threadIdx.x, cnt = j - lo + 1;
  // one pass of NREAL threads, forming the sums of threads t0 + tid of NT
  auto pass = [&](int t0) {
    const int vt = t0 + tid;  // the thread of NT whose sums this pass forms
    constexpr int LP0 = 64 / P;
    if (NREAL < NT && t0 >= r1 - r0) {  // no rows in this pass: its partials are zeros
      if ((tid & 63) % LP0 == 0) red[(vt >> 6) * P + (tid & 63) / LP0] = 0.0;
      return;
    }
    T p[P];
#pragma unroll
    for (int i = 0; i < P; ++i) p[i] = 0;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const int r = r0 + q * NT + vt;
      if (r < r1) {
        const T wv = wsrc[r];
#pragma unroll
        for (int d0 = 0; d0 < P; d0 += CH) {
          if (d0 < cnt) {
            T v[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c) {
              const int i = lo + min(d0 + c, cnt - 1);
              v[c] = Vr[(size_t)(RING ? i % RING : i) * n + r];
            }
#pragma unroll
            for (int c = 0; c < CH; ++c) p[d0 + c] += (d0 + c < cnt) ? v[c] * wv : (T)0;
          }
        }
      }
    }
    double pd[P];
#pragma unroll
    for (int i = 0; i < P; ++i) pd[i] = (double)p[i];
    const int lane = tid & 63, wave = vt >> 6;
    ReduceScatter<P, 32>::run(pd, lane);
    constexpr int LP = 64 / P;  // lanes per value after the reduce-scatter: lane l holds value l / LP
    if (lane % LP == 0) red[wave * P + lane / LP] = pd[0];
  };
  if constexpr (NREAL == NT) {
    pass(0);  // straight-line code for the usual case: a loop, even of one trip, costs the scheduling
  } else {
#pragma unroll 1
    for (int t0 = 0; t0 < NT; t0 += NREAL) pass(t0);
  }
  __syncthreads();
  if (tid < P && tid < cnt) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) s += red[w * P + tid];
    part_blk[tid] = s;
  }
}

// First basis vector of the Gram-Schmidt window of step j (all of v_0..v_j without a window).
__device__ inline int window_lo(const LzArgs& a, int j) { return a.window > 0 ? max(0, j - a.window + 1) : 0; }

// Workgroup size of the step's dot partials for windows of P vectors of es-byte elements: the
// two-vector ring, windows of up to 8 vectors and FP32 windows of up to 32 take kDotsThreads (two
// rows per thread, 64 registers, eight waves per SIMD); the rest 256 threads (their accumulators need
// the registers). The first steps use windows of 8 and 16 vectors: a 32-vector one would reduce and
// store 32 partials per workgroup for one to sixteen dots.
__host__ __device__ constexpr int dots_threads(int P, int es) {
  return (P <= 8 || (es == 4 && P <= 32)) ? kDotsThreads : kBlock;
}

// Phase B of step j: every workgroup reduces the dot partials of all workgroups of its realization
// in the canonical order (identical coefficients everywhere, no inter-workgroup synchronisation),
// then v~_{j+1} = src - sum_i c_i Vraw_i over the window (FP64 accumulation, rounded once), plus
// the partial squared norm on the final pass.
// Where one realization's step data lives: its workspace blocks, or LDS in the single-kernel solve.
template <typename T>
struct StepMem {
  RState* st;    // Lanczos state
  T* V;          // raw basis, vector-major (n elements per vector)
  double* part;  // dot partials, kPartStride per row block
  double* npart; // norm partials, one per row block
};

template <typename T>
__device__ inline StepMem<T> step_mem(const LzArgs& a, const Task& tk, int task) {
  return {a.state + task, (T*)a.V + tk.vec_off, a.part + tk.part_off, a.npart + tk.part_off / kPartStride};
}

// The arithmetic of a row is the same for every P >= the window.
template <typename T, int P, int RING>
__device__ inline void update_body(const LzArgs& a, const Task& tk, const StepMem<T>& mem, int blk, int j, int from_w,
                                   int final_pass, int second, double* cs, double (*csum)[kMaxChunks], double* red) {
  RState* st = mem.st;
  constexpr int CH = P < 8 ? P : 8;
  const int tid = threadIdx.x, lo = window_lo(a, j), cnt = j - lo + 1;
  const double* part = mem.part;
  const int nblk = tk.nblk, chunk = part_chunk(nblk), nch = (nblk + chunk - 1) / chunk;
  for (int item = tid; item < nch * cnt; item += kBlock) {
    const int c = item / cnt, d = item - c * cnt;
    double s = 0.0;
    const int b1 = min(nblk, (c + 1) * chunk);
    for (int b = c * chunk; b < b1; ++b) s += part[(size_t)b * kPartStride + d];
    csum[d][c] = s;
  }
  __syncthreads();
  if (tid < P) {
    double coef = 0.0;
    if (tid < cnt) {
      double t = 0.0;
      for (int c = 0; c < nch; ++c) t += csum[tid][c];
      const double si = st->s[lo + tid];
      const double h = si * t;
      coef = h * si;
      if (lo + tid == j && blk == 0) {
        const double alpha = second ? st->alpha[j] + h : h;
        st->alpha[j] = alpha;
        if (final_pass) {  // breakdown reference of step j: max(|alpha_0..j|, beta_0..j-1)
          double sc = fabs(alpha);
          if (j > 0) sc = fmax(sc, fmax(st->scal[j - 1], st->beta[j - 1]));
          st->scal[j] = isfinite(alpha) ? sc : alpha;
        }
      }
    }
    cs[tid] = coef;
  }
  __syncthreads();
  const int n = tk.n, r0 = blk * kRowsPerBlock, r1 = min(n, r0 + kRowsPerBlock);
  T* Vr = mem.V;
  const T* src = from_w ? (const T*)a.W + tk.w_off : Vr + vslot(a, j + 1) * n;
  T* dst = Vr + vslot(a, j + 1) * n;
  double nrm = 0.0;
  // RQ rows per thread at a time, RQ x CH loads in flight (12 mixed graphs of 1e4 to 5e5 nodes: 5.71 ms of updates,
  // one row 6.02, four 5.73 on half the wavefronts)
  constexpr int RQ = 2;
#pragma unroll 1
  for (int q = 0; q < kRowsPerThread && r0 + q * kBlock < r1; q += RQ) {
    int row[RQ];
    double acc[RQ];
    int z = 0;  // the coefficients are read anew for every group of rows: held over them they spill
    asm volatile("" : "+v"(z));
#pragma unroll
    for (int u = 0; u < RQ; ++u) {
      row[u] = min(r0 + (q + u) * kBlock + tid, r1 - 1);
      acc[u] = (double)src[row[u]];
    }
#pragma unroll
    for (int d0 = 0; d0 < P; d0 += CH) {
      if (d0 < cnt) {
        T v[RQ][CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          const int i = lo + min(d0 + c, cnt - 1);
          const T* vi = Vr + (size_t)(RING ? i % RING : i) * n;
#pragma unroll
          for (int u = 0; u < RQ; ++u) v[u][c] = vi[row[u]];
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          const double k = cs[z + d0 + c];
#pragma unroll
          for (int u = 0; u < RQ; ++u) acc[u] -= k * (double)v[u][c];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < RQ; ++u)
      if (r0 + (q + u) * kBlock + tid < r1) {
        const T out = (T)acc[u];
        dst[row[u]] = out;
        nrm += (double)out * (double)out;
      }
  }
  if (!final_pass) return;
  nrm = block_sum<kBlock>(nrm, red);
  if (tid == 0) mem.npart[blk] = nrm;
}

// ------------------------------------------------------------------------------- small exponential
constexpr int kChebMax = 1 << 16;  // Chebyshev terms of the small exponential (d up to 5e7)

__device__ inline double wave_max(double v) {
  v = fmax(v, lane_xor<32>(v));
  v = fmax(v, lane_xor<16>(v));
  v = fmax(v, lane_xor<8>(v));
  v = fmax(v, lane_xor<4>(v));
  v = fmax(v, lane_xor<2>(v));
  return fmax(v, lane_xor<1>(v));
}
__device__ inline double wave_min(double v) { return -wave_max(-v); }

// v of the lane before (lane 0: 0) and of the lane after (lane 63: 0), in registers: a few cycles, where a shuffle
// through the LDS crossbar takes about a hundred.
template <int CTRL>
__device__ inline double lane_shift(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ inline double lane_before(double v) { return lane_shift<0x138>(v); }  // wave_shr:1
__device__ inline double lane_after(double v) { return lane_shift<0x130>(v); }   // wave_shl:1
__device__ inline double lane_read(double v, int l) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// True when every eigenvalue of the tridiagonal (a, b) lies below x: the leading principal minors of x I - T are
// then all positive. Their three-term recurrence has no division, which a ratio of successive minors would put into
// a chain of k dependent steps. g: a power of two of about 1 / the spectrum's width, so that the factors are at
// most about 1; the pair is rescaled every eight steps.
__device__ inline bool above_spectrum(const double* a, const double* b, int k, double x, double g) {
  double q0 = 1.0, q1 = (x - a[0]) * g;
  bool above = q1 > 0.0;
  auto step = [&](int i) {
    const double s = b[i - 1] * g, u = (x - a[i]) * g;
    const double q2 = u * q1 - (s * s) * q0;
    above = above && q2 > 0.0;
    q0 = q1;
    q1 = q2;
  };
  int i = 1;
  for (; i + 8 <= k; i += 8) {
#pragma unroll
    for (int u = 0; u < 8; ++u) step(i + u);
    const int e = -__builtin_amdgcn_frexp_exp(q1);
    q0 = __builtin_amdgcn_ldexp(q0, e);
    q1 = __builtin_amdgcn_ldexp(q1, e);
  }
  for (; i < k; ++i) step(i);
  return above;
}

struct ExpvOut {
  double theta;
  double y0, y1;  // this lane's components: rows lane and lane + 64 (0 beyond k)
  double ynorm;   // ||y||_2
  bool finite;
};

// exp(M) e1 for the tridiagonal M = T - theta I whose spectrum lies in [c - d, c + d] (sc = 1 / d, or 1 for a d that
// vanishes), the expansion below; lane l owns row l, and row l + 64 when TWO; (ta, tl, tr): the rows of t. One
// wavefront runs one chain of dependent operations, so every instruction of a term counts: neighbours by register
// moves, the factors 2 of Clenshaw's recurrence in t, the terms four at a time with one look at their size (470
// cycles a term with shuffles, branches per term and copies; 130 now).
template <bool TWO>
__device__ inline void cheb_exp(double ta_0, double tl_0, double tr_0, double ta_1, double tl_1, double tr_1, double c,
                                double d, double sc, double top, double& x0, double& x1) {
  const int lane = threadIdx.x & 63;
  const double e0 = lane == 0 ? 1.0 : 0.0;
  // o += f (t v), for f t given; rows 63 and 64 are neighbours across the lane's two halves
  auto tmul = [&](double a0, double l0, double r0, double a1, double l1, double r1, double v0, double v1, double& o0,
                  double& o1) {
    double dn0 = lane_after(v0);
    if constexpr (TWO) {
      const double dn1 = lane_after(v1);
      double up1 = lane_before(v1);
      const double row64 = lane_read(v1, 0), row63 = lane_read(v0, 63);
      dn0 = lane == 63 ? row64 : dn0;
      up1 = lane == 0 ? row63 : up1;
      o1 = fma(a1, v1, o1);
      o1 = fma(l1, up1, o1);
      o1 = fma(r1, dn1, o1);
    }
    o0 = fma(a0, v0, o0);
    o0 = fma(l0, lane_before(v0), o0);
    o0 = fma(r0, dn0, o0);
  };
  if (!(d > 1e-10)) {  // M within 1e-10 of c I: second-order Taylor (error below d^3 / 6)
    double p0 = 0.0, p1 = 0.0, r0 = 0.0, r1 = 0.0;
    tmul(ta_0, tl_0, tr_0, ta_1, tl_1, tr_1, e0, 0.0, p0, p1);
    tmul(ta_0, tl_0, tr_0, ta_1, tl_1, tr_1, p0, p1, r0, r1);
    const double ec = exp(c);
    x0 = ec * (e0 + p0 + 0.5 * r0);
    x1 = ec * (p1 + 0.5 * r1);
    return;
  }
  const int K = __builtin_amdgcn_readfirstlane(min((int)ceil(sqrt(84.0 * d)) + 12, kChebMax));
  const double a0 = 2.0 * ta_0, l0 = 2.0 * tl_0, r0 = 2.0 * tr_0, a1 = 2.0 * ta_1, l1 = 2.0 * tl_1, r1 = 2.0 * tr_1;
  const double two0 = 2.0 * e0;
  // mA, mB: m_k and m_{k+1}; (p, q): b_{k+1} and b_{k+2}; S: the sum of the m so far; f: 2 k
  double mA = 1e-200, mB = 0.0, S = 0.0, f = 2.0 * K;
  double p_0 = 0.0, p_1 = 0.0, q_0 = 0.0, q_1 = 0.0;
  auto term = [&](double& m, double& mn, double& b1_0, double& b1_1, double& b2_0, double& b2_1) {
    b2_0 = fma(two0, m, -b2_0);
    b2_1 = -b2_1;
    tmul(a0, l0, r0, a1, l1, r1, b1_0, b1_1, b2_0, b2_1);
    S += m;
    mn = fma(f * sc, m, mn);
    f -= 2.0;
  };
  int kk = K;  // terms k = K .. 1
  auto rescale = [&] {  // the unnormalised recurrence in range: a term grows it less than 1e12-fold
    if (__builtin_amdgcn_ballot_w64(mA > 1e150)) {
      constexpr double z = 0x1p-600;
      mA *= z, mB *= z, S *= z, p_0 *= z, p_1 *= z, q_0 *= z, q_1 *= z;
    }
  };
  for (; kk >= 4; kk -= 4) {
    term(mA, mB, p_0, p_1, q_0, q_1);
    term(mB, mA, q_0, q_1, p_0, p_1);
    term(mA, mB, p_0, p_1, q_0, q_1);
    term(mB, mA, q_0, q_1, p_0, p_1);
    rescale();
  }
  if (kk >= 2) {
    term(mA, mB, p_0, p_1, q_0, q_1);
    term(mB, mA, q_0, q_1, p_0, p_1);
    kk -= 2;
  }
  if (kk == 1) {
    term(mA, mB, p_0, p_1, q_0, q_1);
    const double m = mA, b_0 = p_0, b_1 = p_1;
    mA = mB, mB = m;
    p_0 = q_0, p_1 = q_1;
    q_0 = b_0, q_1 = b_1;
  }
  // f = b_0 - t b_1 = m_0 e1 + t b_1 - b_2
  const double e = top == 0.0 ? 1.0 : exp(top);
  S = 2.0 * S + mA;
  double o0 = fma(e0, mA, -q_0), o1 = -q_1;
  tmul(ta_0, tl_0, tr_0, ta_1, tl_1, tr_1, p_0, p_1, o0, o1);
  x0 = e * o0 / S;
  x1 = e * o1 / S;
}

// a, b: LDS arrays (k diagonal, k-1 off-diagonal entries), k <= 128. Called by all 64 lanes of a
// wave; lane l owns rows l and l + 64 of T. rough: the caller wants only ynorm and ratios of y's components, which
// do not depend on the shift: an upper bound of lambda_max within 1/2 takes its place (theta: that bound), one or
// two of the bisection's eight or nine rounds. It must not lie much further above, where the expansion loses
// exp(theta - lambda_max) in precision; without a shift the same bound ends the interval.
// KMAX: k is at most that (64: no second row per lane in the code).
template <int KMAX = kMLimit>
__device__ ExpvOut tridiag_expv_wave(const double* a, const double* b, int k, bool shift, bool rough = false) {
  const int lane = threadIdx.x & 63;
  k = __builtin_amdgcn_readfirstlane(k);
  const int q0 = lane, q1 = lane + 64;
  constexpr bool SECOND = KMAX > 64;
  const double ai0_0 = q0 < k ? a[q0] : 0.0, ai0_1 = SECOND && q1 < k ? a[q1] : 0.0;
  const double bl_0 = (q0 >= 1 && q0 < k) ? b[q0 - 1] : 0.0, bl_1 = SECOND && q1 < k ? b[q1 - 1] : 0.0;
  const double br_0 = (q0 + 1 < k) ? b[q0] : 0.0, br_1 = SECOND && q1 + 1 < k ? b[q1] : 0.0;
  const double rad0 = fabs(bl_0) + fabs(br_0), rad1 = fabs(bl_1) + fabs(br_1);  // Gershgorin
  const double low = wave_min(fmin(q0 < k ? ai0_0 - rad0 : INFINITY, SECOND && q1 < k ? ai0_1 - rad1 : INFINITY));
  const double high = wave_max(fmax(q0 < k ? ai0_0 + rad0 : -INFINITY, SECOND && q1 < k ? ai0_1 + rad1 : -INFINITY));
  double theta = 0.0, top = 0.0;
  if (k == 1) {
    (shift ? theta : top) = a[0];
  } else {
    const double eps = 1.1102230246251565e-16;
    double hi = high + 4.0 * eps * fmax(fabs(high), fabs(low)), lo = low - 4.0 * eps * fmax(fabs(hi), fabs(low));
    const double g = __builtin_amdgcn_ldexp(1.0, -__builtin_amdgcn_frexp_exp(hi - lo));
    for (int it = 0; it < 40; ++it) {
      if (hi - lo <= (rough || !shift ? 0.5 : 0.0) + 4.0 * eps * fmax(fabs(lo), fabs(hi))) break;
      const double w = hi - lo;
      const double x = (lane == 63) ? hi : lo + w * (double)(lane + 1) * (1.0 / 64.0);
      const unsigned long long mask = __ballot(above_spectrum(a, b, k, x, g));
      const int first = mask ? (__ffsll((long long)mask) - 1) : 63;
      const double nhi = (first == 63) ? hi : lo + w * (double)(first + 1) * (1.0 / 64.0);
      const double nlo = (first == 0) ? lo : lo + w * (double)first * (1.0 / 64.0);
      lo = nlo;
      hi = nhi;
    }
    if (shift) theta = rough ? hi : 0.5 * (lo + hi); else top = hi;
  }
  // y = exp(M) e1, M = T - theta I, by the Chebyshev expansion of exp on [bot, top], an interval that
  // holds the spectrum of M (below by Gershgorin; top = 0 with the shift): with x = c + d t,
  //   exp(x) = e^top (i_0 + 2 sum_{k>=1} i_k T_k(t)),  i_k = e^-d I_k(d)  (I_k modified Bessel),
  // and i_k falls like e^{-k^2 / 2d}, so sqrt(84 d) + 12 terms reach double precision (those beyond sum to less
  // than 3e-20 for every d up to 1e5). The i_k come
  // from Miller's backward recurrence I_{k-1} = I_{k+1} + (2k/d) I_k, unnormalised and in the order
  // Clenshaw's recurrence b_k = c_k e1 + 2 t b_{k+1} - b_{k+2} consumes them, so one backward loop does
  // both and the sum divides by the normalisation sum_k c_k T_k(1) = 1 at the end.
  const double ai_0 = q0 < k ? ai0_0 - theta : 0.0, ai_1 = SECOND && q1 < k ? ai0_1 - theta : 0.0;
  const double bot = fmin(low - theta, top);
  const double c = 0.5 * (bot + top), d = 0.5 * (top - bot);
  // t = (M - c I) / d, row by row (rows beyond k stay zero: no coupling, no diagonal)
  const double sc = d > 1e-10 ? 1.0 / d : 1.0;
  const double ta_0 = q0 < k ? (ai_0 - c) * sc : 0.0, ta_1 = SECOND && q1 < k ? (ai_1 - c) * sc : 0.0;
  const double tl_0 = bl_0 * sc, tl_1 = bl_1 * sc, tr_0 = br_0 * sc, tr_1 = br_1 * sc;
  double x0, x1;
  if (!SECOND || k <= 64) {
    cheb_exp<false>(ta_0, tl_0, tr_0, 0.0, 0.0, 0.0, c, d, sc, top, x0, x1);
  } else if constexpr (SECOND) {
    cheb_exp<true>(ta_0, tl_0, tr_0, ta_1, tl_1, tr_1, c, d, sc, top, x0, x1);
  }
  x0 = q0 < k ? x0 : 0.0;
  x1 = SECOND && q1 < k ? x1 : 0.0;
  ExpvOut o;
  o.theta = theta;
  o.y0 = x0;
  o.y1 = x1;
  o.ynorm = sqrt(wave_sum(x0 * x0 + x1 * x1));
  o.finite = isfinite(o.ynorm) && isfinite(theta);
  return o;
}

// The small exponential of one realization after its last step (mode 0) or after step j of an
// adaptive run (mode 1), in three parts so that a workgroup of any size can run it:
//   tridiag_prepare  every thread of the workgroup (close_step reduces with all of them): the order k
//                    of T, the last beta and the flags. mode 1 closes step j and stops the
//                    realization on breakdown; mode 0 closes the last step of a realization still
//                    open after m_steps (fixed m). exit: nothing more to do here (thread 0 has
//                    recorded any stop);
//   tridiag_load     the lanes of the first wave copy T to LDS (then a workgroup barrier);
//   tridiag_finish   the first wave: theta*, y = exp(T - theta* I) e1, Saad's estimate. mode 1 stops
//                    the realization when the estimate is below tol or k reached m_max (CAPPED); a
//                    realization that goes on is closed again, with the same bits, by the next phase
//                    A. mode 0 records y, theta, the estimate, diag and the checkpoint when given.
struct TriPrep {
  int k;
  double beta_last;
  int flags;
  bool exit;
};

__device__ inline TriPrep tridiag_prepare(const LzArgs& args, RState* st, const double* npart, int nblk, int64_t r,
                                          int mode, int j, int m_steps, ebtc_diag* diag, double* chunks) {
  TriPrep p{0, 0.0, st->flags, false};
  if (mode == 1) {
    if (st->done) {
      p.exit = true;
      return p;
    }
    p.k = j + 1;
    const StepClose c = close_step(st, npart, nblk, j, args.eps, chunks);
    p.beta_last = c.beta;
    if (c.flags) {
      if (threadIdx.x == 0) {
        st->beta[j] = c.beta;
        st->flags = p.flags | c.flags;
        st->done = 1;
        st->m_used = p.k;
      }
      p.exit = true;
    }
    return p;
  }
  if (st->done && st->m_used < 1) {
    // nothing to expand (an adjoint started at a zero cotangent): empty result
    if (threadIdx.x == 0) {
      st->theta = 0.0;
      st->est = 0.0;
      if (diag) {
        diag[r].m_used = 0;
        diag[r].flags = st->flags;
        diag[r].theta = 0.0;
        diag[r].est = 0.0;
      }
    }
    p.exit = true;
  } else if (st->done) {
    p.k = st->m_used;
    p.beta_last = st->beta[p.k - 1];
  } else {
    p.k = m_steps;
    const StepClose c = close_step(st, npart, nblk, p.k - 1, args.eps, chunks);
    p.beta_last = c.beta;
    p.flags |= c.flags;
  }
  return p;
}

__device__ inline void tridiag_load(const RState* st, const TriPrep& p, double* a, double* b) {
  for (int i = threadIdx.x; i < p.k; i += 64) {
    a[i] = st->alpha[i];
    b[i] = i < p.k - 1 ? st->beta[i] : p.beta_last;
  }
}

template <int KMAX = kMLimit>
__device__ inline void tridiag_finish(const LzArgs& args, RState* st, int64_t r, int mode, int j, const TriPrep& p,
                                      const double* a, const double* b, int shift, double tol, ebtc_diag* diag,
                                      double* ckpt) {
  const int lane = threadIdx.x, k = p.k;
  const double beta_last = p.beta_last;
  int flags = p.flags;
  const ExpvOut o = tridiag_expv_wave<KMAX>(a, b, k, shift != 0, mode == 1);
  const double ylast = KMAX <= 64 || k <= 64 ? __shfl(o.y0, k - 1, 64) : __shfl(o.y1, k - 65, 64);
  const double est = (o.ynorm > 0.0) ? beta_last * fabs(ylast) / o.ynorm : 0.0;
  if (mode == 1) {
    if (lane == 0) {
      int stop = 0;
      if (!o.finite) {
        flags |= EBTC_FLAG_NONFINITE;
        stop = 1;
      } else if (est < tol) {
        stop = 1;
      } else if (k >= args.m_max) {
        flags |= EBTC_FLAG_CAPPED;
        stop = 1;
      }
      if (stop) {
        st->beta[j] = beta_last;
        st->flags = flags;
        st->done = 1;
        st->m_used = k;
      } else if (args.live != nullptr) {
        // the count of realizations still running after step j (an integer, so its value does not
        // depend on the order of the adds); the next step's kernels read it after the launch boundary
        atomicAdd(&args.live[j], 1);
      }
    }
    return;
  }
  if (lane < k) st->y[lane] = o.y0;
  if (lane + 64 < k) st->y[lane + 64] = o.y1;
  if (lane == 0) {
    if (!o.finite) flags |= EBTC_FLAG_NONFINITE;
    const double e = (flags & EBTC_FLAG_BREAKDOWN) ? 0.0 : est;
    st->beta[k - 1] = beta_last;
    st->m_used = k;
    st->done = 1;
    st->flags = flags;
    st->theta = o.theta;
    st->est = e;
    if (diag) {
      diag[r].m_used = k;
      diag[r].flags = flags;
      diag[r].theta = o.theta;
      diag[r].est = e;
    }
  }
  if (ckpt) {
    double* c = ckpt + r * kCkptDoubles;
    for (int i = lane; i < kMLimit; i += 64) {
      c[i] = i < k ? a[i] : 0.0;
      c[kMLimit + i] = i < k ? b[i] : 0.0;
    }
    if (lane == 0) {
      c[2 * kMLimit] = o.theta;
      c[2 * kMLimit + 1] = st->beta0;
      c[2 * kMLimit + 2] = (double)k;
      c[2 * kMLimit + 3] = (double)flags;
    }
  }
}

}  // namespace
}  // namespace ebtc
