// Paneled SpMV form, w = s_j A v_j with every gather and every row sum in LDS.
//
// The CSR-stream form pays one L2 request per gathered element (138 G entries/s on graphs of 1e4 to 5e5
// nodes). Here the matrix is cut into tiles of one share of rows (up to 12160) by one panel of columns (up
// to 8192 FP32 / 4096 FP64 elements, 32 KB): the rows' FP64 sums stay in LDS for a whole product, the
// panels' vector slices pass through two LDS buffers, and an entry costs one LDS read (the gather) and one
// LDS add (its row's sum). Once per call the entries are put in that order:
//   cut    a realization's rows into shares of at most tile_rows rows and a quarter more entries than the
//          mean share's (k_tile_cut, k_tile_pack, k_tile_fill: a dense list of the shares of the launch);
//   sort   each share's rows are cut into kTileBands equal bands, one per wave of the product. A band's
//          entries, panel by panel, replace its CSR range (k_tile_sort): one word per entry (column in the
//          panel, row in the band, rank) and its value.
// A row belongs to one wave, whose LDS operations execute in order, so its products are added in entry
// order: the CSR-stream form's sums, bit for bit. Two entries of one row must not meet in one LDS
// instruction, where the order of the adds is not defined: the sort places the rows' first entries of a panel
// before the second ones and so on (kTileClasses), so that they seldom do, and where they do the entry's rank
// (the number of its row's earlier entries in its group of 64) puts it in a later add.
// Long rows (tile_hub) would fill whole groups, one add per entry; they are listed apart and summed by
// workgroups of their own in the same launch from products staged in LDS, one thread per row.
//
// Bound by the entry stream and, for few entries per tile, by the slices. Per product, FP32 (us; before: the
// fastest other form):
//   64 x n=1e5, degree 20, values         229   before 336 (column-segmented); its bytes alone take 148
//   24 x n=99991, degree 15, values        72   before 131 (column-segmented)
//   16 x n=2e5, degree 16, values         115   before 224 (column-segmented)
//   8 x n=4e5, degree 24, pattern         151   before 590 (entry-balanced)
//   8 x n=436472, degree 20, pattern, BA  194   before 520 (entry-balanced)
//   3 x n=1e6, degree 10, values          209   before 257 (entry-balanced), and 1.2 ms for step 0
// and 1.2 ms for the sort of the first (128M entries, 20 bytes of traffic each).
#include <algorithm>
#include <type_traits>

#include "step_device.h"

namespace ebtc {
namespace {

constexpr int kTileThreads = 1024;
constexpr int kTileBands = kTileBandsHost;                    // waves that add entries
constexpr int kTileLoaders = kTileThreads / 64 - kTileBands;  // waves that stage the slices
// Workgroups of a product that take the long rows, one per compute unit: 32 took 956 us where 64 took 545 and 256
// take 505 (24 x n=436472 Barabasi-Albert); where there are none they return at once (64 x n=1e5: 233 us with both).
constexpr int kTileHubGroups = 256;
constexpr int kSortThreads = 512;                             // one band per workgroup of the sort
constexpr int kTileClasses = 4;  // 2: 1.8 and 1.4 adds per group in the two examples; 6: 1.09 and 1.18
constexpr int kWin = 16, kWinStride = 17;  // entries of a row staged at a time by the sort, and their stride (odd)
static_assert((kTileMaxRows + kTileBands - 1) / kTileBands <= 1024, "10 bits of row in the band");

template <typename T>
struct TileShape {
  static constexpr int COLS = sizeof(T) == 8 ? 4096 : 8192;   // a slice buffer: 32 KB
  static constexpr int HCAP = 128 * 1024 / sizeof(T);         // products of a batch of long rows
  static constexpr int UL = COLS * (int)sizeof(T) / 16 / (kTileLoaders * 64);  // 16-byte loads per loader lane
};

// word of an entry: column in the panel << 2 (13 bits), row in the band << 16 (10 bits), rank << 26
__device__ inline uint32_t tile_word(int col, int row, int rank) {
  return (uint32_t)col << 2 | (uint32_t)row << 16 | (uint32_t)rank << 26;
}

// LDS operations of the workgroup before it complete; loads from memory may stay in flight across it.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS writes of this wave visible to its lanes.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Panel of column c: the FP32 quotient, then one step of correction (c < 2^24).
__device__ inline int panel_of(int c, int C, float inv) {
  int q = (int)((float)c * inv);
  q -= q * C > c ? 1 : 0;
  q += (q + 1) * C <= c ? 1 : 0;
  return q;
}

// A value every lane of the wave holds, in a scalar register: buffer resources must be wave-uniform, and a field
// read with a vector load would make every access through them a loop over the wave's lanes.
__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline int64_t uniform(int64_t v) {
  const uint32_t lo = (uint32_t)uniform((int)(uint32_t)v), hi = (uint32_t)uniform((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Workgroup b of a launch over `used` items, each XCD on a contiguous range of them; -1 past the end.
__device__ inline int spread(int used, int b) {
  const int x = b & 7, q = b >> 3, base = used >> 3, rem = used & 7;
  return q < base + (x < rem ? 1 : 0) ? x * base + min(x, rem) + q : -1;
}

// ------------------------------------------------------------------------------- cut into shares
// One wave per realization: share after share, the most rows from its first one on that keep both limits.
// Lanes try 64 consecutive full shares at once; where the entries stop one, a 64-way search finds its end.
// again: with the rows per share that k_tile_pack chose, where it chose others.
__global__ __launch_bounds__(64) void k_tile_cut(LzArgs a, int t0, int again) {
  const int t = t0 + blockIdx.x, lane = threadIdx.x;
  const int Rs = again ? a.tile_count[3] : a.tile_rows;
  if (again && Rs == a.tile_rows) return;
  const Task tk = a.tasks[t];
  const int32_t* rp = a.row_ptr + tk.rowptr_off;
  const int n = tk.n;
  const int64_t p0 = a.tile_begin[t];
  const int slots = (int)(a.tile_begin[t + 1] - p0);
  const int64_t emax = tile_entries(Rs, n, rp[n]);
  TileCut* out = a.tile_cut + p0;
  int i = 0, q = 0;
  while (i < n && q < slots) {
    const int64_t lo64 = (int64_t)i + (int64_t)lane * Rs;
    const int lo = (int)min((int64_t)n, lo64), hi = (int)min((int64_t)n, lo64 + Rs);
    const bool ok = lo < n && rp[hi] - rp[lo] <= emax && q + lane < slots;
    const unsigned long long m = __ballot(ok);
    const int f = m == ~0ull ? 64 : __ffsll((long long)~m) - 1;
    if (lane < f) out[q + lane] = {lo, hi};
    q += f;
    i = (int)min((int64_t)n, (int64_t)i + (int64_t)f * Rs);
    if (f == 64 || i >= n || q >= slots) continue;
    // too many entries: the largest end in [i + 1, b) whose rows keep within emax, at least one row
    int e = i + 1, b = min(n, i + Rs);
    const int base = rp[i];
    while (b - e > 1) {
      const int step = (b - e + 63) / 64, p = e + (lane + 1) * step;
      const unsigned long long g = __ballot(p < b && rp[min(p, n)] - base <= emax);
      const int c = g == ~0ull ? 64 : __ffsll((long long)~g) - 1;
      const int ne = e + c * step;
      b = min(b, ne + step);
      e = ne;
    }
    if (lane == 0) out[q] = {i, e};
    ++q;
    i = e;
  }
  if (lane == 0) a.tile_ncut[t] = q;
}

// again = 1: the realizations' share counts to offsets in the launch. Before that the rows per share: where
// shares end early they come on top of the rounds of kTileUnits that the host filled, and a few shares over
// would cost a whole round, so every share takes more rows, or, at the most a unit holds, one round more is
// filled (8 x n=436472 Barabasi-Albert: 560 shares of 6821 rows took 3 rounds, 316 us a product; two rounds now,
// 194 us). 15% to spare: such graphs have shares of few, long rows, which take longer (three n=1e6 graphs:
// 224 us a product with 6%, 209 with 15, 215 with 25). Never fewer rows than the host sized the slots for.
__global__ __launch_bounds__(1024) void k_tile_pack(LzArgs a, int t0, int count, int again) {
  __shared__ int wsum[16];
  __shared__ double su[16], sf[16];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (!again) {
    double used = 0.0, full = 0.0;
    for (int i = tid; i < count; i += 1024) {
      used += (double)a.tile_ncut[t0 + i];
      full += (double)((a.tasks[t0 + i].n + a.tile_rows - 1) / a.tile_rows);
    }
    used = block_sum<1024>(used, su);
    full = block_sum<1024>(full, sf);
    if (tid == 0) {
      int rows = a.tile_rows;
      if (used > full) {
        const double rounds = fmax(1.0, ceil(full / kTileUnits)), need = 1.15 * used * a.tile_rows / kTileUnits;
        double r = ceil(need / rounds);
        if (r > kTileMaxRows) r = ceil(need / (rounds + 1.0));
        rows = (int)fmin((double)kTileMaxRows, fmax((double)a.tile_least, r));
      }
      a.tile_count[3] = rows;
      a.tile_count[1] = 0;  // long rows
      a.tile_count[2] = 0;  // batches of them
    }
    return;
  }
  int carry = 0;
  for (int c0 = 0; c0 < count; c0 += 1024) {
    const int i = c0 + tid, v = i < count ? a.tile_ncut[t0 + i] : 0;
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int x = __shfl_up(inc, o, 64);
      if (lane >= o) inc += x;
    }
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    int before = 0, all = 0;
    for (int k = 0; k < 16; ++k) {
      before += k < w ? wsum[k] : 0;
      all += wsum[k];
    }
    if (i < count) a.tile_ncut[t0 + i] = carry + before + inc - v;
    carry += all;
    __syncthreads();
  }
  if (tid == 0) {
    a.tile_ncut[t0 + count] = carry;
    a.tile_count[0] = carry;
  }
}

// The launch's shares in launch order: place b of the grid takes the share whose turn it is on b's XCD.
__global__ __launch_bounds__(kBlock) void k_tile_fill(LzArgs a, int t0, int count, int places) {
  const int b = blockIdx.x * kBlock + threadIdx.x;
  if (b >= places) return;
  const int l = spread(a.tile_count[0], b);
  TileShare s{};
  s.task = -1;
  if (l >= 0) {
    int lo = 0, hi = count;  // the realization of share l: ncut[lo] <= l < ncut[lo + 1]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (a.tile_ncut[t0 + mid] <= l) lo = mid; else hi = mid;
    }
    const int t = t0 + lo, q = l - a.tile_ncut[t];
    const TileCut c = a.tile_cut[a.tile_begin[t] + q];
    const Task tk = a.tasks[t];
    s.task = t;
    s.q = q;
    s.r_begin = c.r_begin;
    s.rows = c.r_end - c.r_begin;
    s.n = tk.n;
    s.nblk = tk.nblk;
    s.vec_off = tk.vec_off;
    s.w_off = tk.w_off + c.r_begin;
    s.rowptr_off = tk.rowptr_off;
    s.part_off = tk.part_off;
  }
  a.tile_share[b] = s;
}

// ------------------------------------------------------------------------------- sort
// One workgroup per band of a share. Counts the band's entries per panel and class (a row's first, second, third
// and later entries of a panel), then places them, a row per lane and kWin entries of each row staged in LDS at a
// time: every lane walks its row and takes the next place of each entry's panel and class (an LDS counter). Which
// rows' entries stand beside each other varies from run to run, but a row's entries keep their order, and so do
// the sums.
// The classes keep two entries of one row out of one group of 64: rows with a late first entry of a panel have no
// early second one, so that even the groups where classes meet seldom hold a row twice. Adds per group for 64 x
// n=1e5, degree 20: 1.23 (first come, first placed: 1.90); n=4e5, degree 24: 1.17 (2.44).
// Reads the columns twice and the values once, writes words and values: 20 bytes per weighted entry.
template <typename T, bool HAS_VAL>
__global__ __launch_bounds__(kSortThreads) void k_tile_sort(LzArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NT = kSortThreads, U = 8, K = kTileClasses;
  // the count's groups of 64 entries overlap by the K - 1 that decide their first entries' classes
  constexpr int H = K - 1, G = 64 - H, NG = NT / 64 * U, SEG = 4 * NG * G;
  static_assert(SEG + H <= 32 * NT * kWinStride, "a bit per entry of a segment in s_col");
  __shared__ uint32_t s_col[NT * kWinStride];
  __shared__ T s_val[HAS_VAL ? NT * kWinStride : 1];
  __shared__ int s_first[NT], s_len[NT];
  __shared__ int s_bad;
  // eight places, one per XCD, then their next bands
  const int band = (blockIdx.x >> 3) % kTileBands, sh = (blockIdx.x >> 3) / kTileBands * 8 + (blockIdx.x & 7);
  const TileShare share = a.tile_share[sh];
  if (share.task < 0) return;
  const int tid = threadIdx.x, lane = tid & 63, w0r = tid - lane;  // w0r: the wave's first row slot
  const Task tk = a.tasks[share.task];
  const int n = tk.n, C = a.pan_cols, S = (n + C - 1) / C, P = a.pan_pmax;
  const float inv = 1.0f / (float)C;
  int* start = (int*)smem;  // [S] first place of each panel in the band
  int* next = start + P;    // [K][P] entries, then the next free place, of each class and panel
  const int brows = (share.rows + kTileBands - 1) / kTileBands, r_end = share.r_begin + share.rows;
  const int rb = min(r_end, share.r_begin + band * brows), re = min(r_end, rb + brows);
  const int32_t* rp = a.row_ptr + tk.rowptr_off;
  const int32_t* ci = a.col_idx + tk.nnz_off;
  const T* va = HAS_VAL ? (const T*)a.values + tk.nnz_off : nullptr;
  const int e0 = rp[rb], e1 = rp[re], blen = e1 - e0, hub = tile_hub<T>(n, rp[n]);
  uint32_t* ent = a.tile_ent + tk.aux_off + e0;
  T* val = HAS_VAL ? (T*)a.tile_val + tk.aux_off + e0 : nullptr;
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int i = tid; i < K * P; i += NT) next[i] = 0;
  if (tid == 0) s_bad = 0;
  if (tid == 0 && band == 0) a.tile_share[sh].hub = hub;
  __syncthreads();
  bool bad = false;
  // adds (sign) the entries of lanes H to 63 to their panels and classes; top: a row's first entry
  auto count = [&](bool ok, bool top, int c, int sign) {
    const bool in = (unsigned)c < (unsigned)n;
    if (ok && !in) bad = true;
    const int p = ok ? (in ? panel_of(c, C, inv) : S - 1) : -1;
    const int prev = __shfl_up(p, 1, 64);
    const unsigned long long heads = __ballot(lane == 0 || top || p != prev);
    const int k = min((int)__clzll((long long)(heads << (63 - lane))), K - 1);
    if (ok && lane >= H) atomicAdd(&next[k * P + p], sign);
  };
  uint32_t* tops = s_col;  // a bit per entry from H before the segment on: a row's first
  for (int q0 = 0; q0 < blen; q0 += SEG) {
    const int words = (min(blen - q0, SEG) + H + 31) / 32;
    for (int i = tid; i < words; i += NT) tops[i] = 0;
    __syncthreads();
    for (int row = rb + tid; row < re; row += NT) {
      const int i = rp[row] - e0 - q0 + H;
      if (rp[row + 1] > rp[row] && i >= 0 && i < words * 32) atomicOr(&tops[i >> 5], 1u << (i & 31));
    }
    __syncthreads();
    for (int g0 = (tid >> 6) * U; g0 * G < min(blen - q0, SEG); g0 += NG) {  // uniform over the wave
      int c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = q0 + (g0 + u) * G + lane - H;
        c[u] = i >= 0 && i < blen ? ci[e0 + i] : 0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int l = (g0 + u) * G + lane, i = q0 + l - H;
        const bool ok = i >= 0 && i < blen && l < words * 32;
        count(ok, ok && ((tops[l >> 5] >> (l & 31)) & 1u), c[u], 1);
      }
    }
    __syncthreads();
  }
  // long rows leave the band: their entries are taken off the counts, the rows listed in batches
  for (int r0 = rb + w0r; r0 < re; r0 += NT) {
    const int row = r0 + lane, len = row < re ? rp[row + 1] - rp[row] : 0;
    unsigned long long hubs = __ballot(len > hub);
    if (!hubs) continue;
    int base = 0;
    if (lane == 0) base = atomicAdd(&a.tile_count[1], __popcll(hubs));
    base = __builtin_amdgcn_readfirstlane(base);
    if (len > hub) a.hub_row[base + __popcll(hubs & below)] = row;
    int at = base, cnt = 0, sum = 0;
    auto emit = [&]() {
      if (cnt && lane == 0) a.hub_batch[atomicAdd(&a.tile_count[2], 1)] = {share.task, at, cnt, sum};
      at += cnt;
      cnt = sum = 0;
    };
    while (hubs) {
      const int l = __ffsll((long long)hubs) - 1;
      hubs &= hubs - 1ull;
      const int hl = __builtin_amdgcn_readlane(len, l), hb = rp[r0 + l];
      for (int k0 = lane - H; k0 - lane + H < hl; k0 += G * U) {
        int c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = k0 + u * G >= 0 && k0 + u * G < hl ? ci[hb + k0 + u * G] : 0;
#pragma unroll
        for (int u = 0; u < U; ++u) count(k0 + u * G >= 0 && k0 + u * G < hl, k0 + u * G == 0, c[u], -1);
      }
      if (sum + hl > TileShape<T>::HCAP) emit();
      ++cnt;
      sum += hl;
    }
    emit();
    if (lane == 0) atomicOr(&a.tile_share[sh].flag, kTileFlagHubs);
  }
  __syncthreads();
  // the panels' first places; the ends go to the product's table
  if (tid < 64) {
    uint32_t* ends = a.tile_end + ((int64_t)sh * kTileBands + band) * P;
    int run = 0;
    for (int s0 = 0; s0 < S; s0 += 64) {
      const int s = s0 + lane;
      int f[K], v = 0;  // the classes' first places in the panel
#pragma unroll
      for (int k = 0; k < K; ++k) {
        f[k] = v;
        v += s < S ? next[k * P + s] : 0;
      }
      int inc = v;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(inc, o, 64);
        if (lane >= o) inc += x;
      }
      if (s < S) {
        start[s] = run + inc - v;
#pragma unroll
        for (int k = 0; k < K; ++k) next[k * P + s] = run + inc - v + f[k];
        ends[s] = (uint32_t)(run + inc);
      }
      run += __builtin_amdgcn_readlane(inc, 63);
    }
    if (lane == 0) a.tile_base[(int64_t)sh * kTileBands + band] = tk.aux_off + e0;
  }
  __syncthreads();
  // Step 0's product from the all-ones start, when the caller has it computed here: each row's values in
  // entry order in FP64, times s_0 = 1/sqrt(n) (long rows: k_tile_hub_first).
  const bool first = HAS_VAL && a.first_in_prepare;
  T* w0 = (T*)a.W + tk.w_off;
  const double s0 = 1.0 / sqrt((double)n);
  uint32_t* col_l = s_col + w0r * kWinStride;  // the wave's windows: no other wave touches them
  T* val_l = HAS_VAL ? s_val + w0r * kWinStride : nullptr;
  int *first_l = s_first + w0r, *len_l = s_len + w0r;
  // equal passes of at most NT rows
  const int brow = re - rb, passes = (brow + NT - 1) / NT, prow = passes ? (brow + passes - 1) / passes : 0;
  for (int r0 = rb; r0 < re; r0 += prow) {
    const int row = r0 + tid;
    const bool mine = tid < prow && row < re;
    const int b = mine ? rp[row] : 0, full = mine ? rp[row + 1] - b : 0, len = full > hub ? 0 : full;
    int done = 0, prev = -1, lpan = -1, lcls = 0, lgrp = 0, lrank = 0;
    double acc = 0.0;
    while (__syncthreads_or(done < len)) {
      const int w = min(len - done, kWin);
      first_l[lane] = b + done;
      len_l[lane] = w;
      wave_sync();
      for (int i0 = 0; i0 < 64 * kWin; i0 += 64 * U) {
        int c[U];
        T v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = i0 + u * 64 + lane, r = i / kWin, o = i - r * kWin;
          const bool ok = o < len_l[r];
          const int k = first_l[r] + o;
          c[u] = ok ? ci[k] : 0;
          if constexpr (HAS_VAL) v[u] = ok ? va[k] : (T)0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = i0 + u * 64 + lane, r = i / kWin, o = i - r * kWin;
          col_l[r * kWinStride + o] = (uint32_t)c[u];
          if constexpr (HAS_VAL) val_l[r * kWinStride + o] = v[u];
        }
      }
      // one entry of every row per round, the waves side by side: the barrier keeps late first entries of a panel
      // behind early ones
      for (int j = 0; j < kWin; ++j) {
        lds_barrier();
        if (j < w) {
          int c = (int)col_l[lane * kWinStride + j];
          // columns out of range or falling: the share goes to the stream arithmetic
          if ((unsigned)c >= (unsigned)n || c < prev) {
            bad = true;
            c = min(max(c, prev), n - 1);
          }
          prev = c;
          const int s = panel_of(c, C, inv);
          lcls = lpan == s ? min(lcls + 1, K - 1) : 0;
          const int pos = atomicAdd(&next[lcls * P + s], 1), grp = (pos - start[s]) >> 6;
          lrank = lpan == s && lgrp == grp ? lrank + 1 : 0;
          lpan = s;
          lgrp = grp;
          if (pos < blen) {  // always, unless the share is flagged
            ent[pos] = tile_word(c - s * C, row - rb, lrank & 63);
            if constexpr (HAS_VAL) val[pos] = val_l[lane * kWinStride + j];
          }
          if constexpr (HAS_VAL) acc += (double)val_l[lane * kWinStride + j];
        }
      }
      done += w;
    }
    if (first && mine && full <= hub) w0[row] = (T)(acc * s0);
  }
  if (bad) s_bad = 1;
  __syncthreads();
  if (tid == 0 && s_bad) atomicOr(&a.tile_share[sh].flag, kTileFlagStream);
}

// ------------------------------------------------------------------------------- long rows
// One batch of long rows of a realization (at most 64): products of all its entries in LDS (FIRST: the values
// alone), formed by the waves in chunks of 512 of one row, the next chunk's columns in flight during the gathers
// of one; then one lane per row adds them in entry order, the CSR-stream form's sum. A row beyond that
// form's capacity is reduced in that form's order instead (FIRST: in entry order, as the row-sum kernel does).
// 30 us for 32768 entries, most of it the latency of the loads and the longest row's chain of adds.
template <typename T, bool HAS_VAL, bool FIRST>
__device__ inline void tile_hub_batch(const LzArgs& a, const Task& tk, const HubBatch& hb, const T* x, double scale,
                                      T* prod, double* red) {
  constexpr int NT = kTileThreads, CAP = StreamShape<T>::CAP, HCAP = TileShape<T>::HCAP, U = 8, CH = 64 * U;
  const int tid = threadIdx.x, lane = tid & 63, wv = uniform(tid >> 6), count = uniform(hb.count);
  const int32_t* rp = a.row_ptr + tk.rowptr_off;
  const int32_t* ci = a.col_idx + tk.nnz_off;
  const T* va = HAS_VAL ? (const T*)a.values + tk.nnz_off : nullptr;
  T* w = (T*)a.W + tk.w_off;
  const int row = lane < count ? a.hub_row[hb.first + lane] : 0;
  const int b = rp[row], len = lane < count ? rp[row + 1] - b : 0;
  const int staged = len <= (FIRST ? HCAP : CAP) ? len : 0;  // entries of this lane's row in LDS
  int off = staged, chk = (staged + CH - 1) / CH;             // exclusive prefix sums over the rows
  const int nch = chk;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(off, o, 64), u = __shfl_up(chk, o, 64);
    if (lane >= o) {
      off += t;
      chk += u;
    }
  }
  const int chunks = __builtin_amdgcn_readlane(chk, 63);
  off -= staged;
  chk -= nch;
  __syncthreads();  // the previous batch's products are read
  struct Chunk {
    int src, dst, m;  // first entry, first product, entries
  };
  auto find = [&](int c) {  // uniform
    Chunk k{0, 0, 0};
    if (c >= chunks) return k;
    const int r = __popcll(__ballot(lane < count && nch > 0 && chk <= c)) - 1;
    // rows without chunks in LDS are skipped by rank among those that have them
    unsigned long long has = __ballot(nch > 0);
    for (int i = 0; i < r; ++i) has &= has - 1ull;
    const int l = __ffsll((long long)has) - 1;
    const int at = (c - __builtin_amdgcn_readlane(chk, l)) * CH;
    k.src = __builtin_amdgcn_readlane(b, l) + at;
    k.dst = __builtin_amdgcn_readlane(off, l) + at;
    k.m = min(__builtin_amdgcn_readlane(staged, l) - at, CH);
    return k;
  };
  int c[U];
  T v[U];
  auto load = [&](const Chunk& k) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = u * 64 + lane < k.m;
      if constexpr (!FIRST) c[u] = ok ? ci[k.src + u * 64 + lane] : 0;
      if constexpr (HAS_VAL) v[u] = ok ? va[k.src + u * 64 + lane] : (T)0;
    }
  };
  Chunk k = find(wv);
  load(k);
  for (int i = wv; i < chunks; i += NT / 64) {
    T p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      T xv = (T)1;
      if constexpr (!FIRST) xv = u * 64 + lane < k.m ? x[c[u]] : (T)0;
      if constexpr (FIRST) p[u] = v[u];
      else if constexpr (HAS_VAL) p[u] = v[u] * xv;
      else p[u] = xv;
    }
    const Chunk at = k;
    k = find(i + NT / 64);
    load(k);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u * 64 + lane < at.m) prod[at.dst + u * 64 + lane] = p[u];
  }
  __syncthreads();
  if (wv == 0 && staged > 0) {
    // one dependent chain of adds per row: the next eight products are read while eight are added
    double acc = 0.0;
    const int e = off + len;
    int at = off;
    T p[8], r[8];
    auto read = [&](T* t, int i) {
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = prod[min(i + u, e - 1)];
    };
    auto sum = [&](const T* t) {
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += (double)t[u];
    };
    read(p, at);
    for (; at + 16 <= e; at += 16) {
      read(r, at + 8);
      sum(p);
      read(p, at + 16);
      sum(r);
    }
    for (; at < e; ++at) acc += (double)prod[at];
    w[row] = (T)(acc * scale);
  }
  for (int i = 0; i < count; ++i) {  // rows beyond the capacity, one after the other
    const int l = __builtin_amdgcn_readlane(len, i);
    if (l <= (FIRST ? HCAP : CAP)) continue;
    const int r = __builtin_amdgcn_readlane(row, i), b0 = __builtin_amdgcn_readlane(b, i), e = b0 + l;
    __syncthreads();  // the products are read
    if constexpr (FIRST) {
      double acc = 0.0;
      for (int k0 = b0; k0 < e; k0 += HCAP) {
        const int m = min(e - k0, HCAP);
        for (int q = tid; q < m; q += NT) prod[q] = va[k0 + q];
        __syncthreads();
        if (tid == 0)
          for (int q = 0; q < m; ++q) acc += (double)prod[q];
        __syncthreads();
      }
      if (tid == 0) w[r] = (T)(acc * scale);
    } else {
      T acc = 0;
      if (tid < kBlock) {
        for (int q = b0 + tid; q < e; q += kBlock) {
          const T xv = x[ci[q]];
          if constexpr (HAS_VAL) acc += va[q] * xv; else acc += xv;
        }
      }
      const double tot = block_sum<NT>((double)acc, red);
      if (tid == 0) w[r] = (T)(tot * scale);
    }
  }
}

// Step 0's product of the long rows of weighted graphs.
template <typename T>
__global__ __launch_bounds__(kTileThreads) void k_tile_hub_first(LzArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double red[kTileThreads / 64];
  for (int i = blockIdx.x; i < a.tile_count[2]; i += gridDim.x) {
    const HubBatch hb = a.hub_batch[i];
    const Task tk = a.tasks[hb.task];
    tile_hub_batch<T, true, true>(a, tk, hb, nullptr, 1.0 / sqrt((double)tk.n), (T*)smem, red);
  }
}

// ------------------------------------------------------------------------------- product
// Raw buffer resource over [p, p + bytes): 32-bit byte offsets, reads past the end give 0.
__device__ inline __amdgpu_buffer_rsrc_t tile_rsrc(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, bytes, 0x00020000);
}
constexpr int kTileStream = 2;  // non-temporal: the matrix is read once per product

// One workgroup per share: kTileBands waves add entries, the others stage the slices two panels ahead in
// registers. One barrier per panel, which waits for LDS only. The entries of a band are one stream: chunks of
// U x 64 of one panel, D chunks in flight per wave (D U 8 bytes per lane: a stream of 7 TB/s needs about
// 64 KB in flight per compute unit; measured at D U = 8, 16 and 18: 308, 226 and 209 us at n=1e5 x 64).
// Short runs take short chunks: every chunk issues U loads, however few entries it holds (one graph of
// n=1e6: 80 us with U = 2 against 103 with U = 6). All of a share's first loads wait on its record alone; the
// step is opened from partials loaded with them and summed after the last panel.
template <typename T, bool HAS_VAL, int U, int D>
__global__ __launch_bounds__(kTileThreads) void k_spmv_tile(LzArgs a, int j) {
  if (all_stopped(a, j)) return;
  constexpr int COLS = TileShape<T>::COLS, UL = TileShape<T>::UL, NT = kTileThreads;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double chunks[kMaxChunks];
  const int tid = threadIdx.x, lane = tid & 63, wv = uniform(tid >> 6);
  T* xs = (T*)smem;                                          // two slices
  double* acc = (double*)(smem + 2 * COLS * sizeof(T));      // the rows' sums
  // scratch of the long rows and of the stream arithmetic: products from the start on, then these
  double* red = (double*)(smem + TileShape<T>::HCAP * sizeof(T));
  int* off = (int*)(red + NT / 64);
  static_assert(TileShape<T>::HCAP * sizeof(T) + NT / 64 * 8 + (kStreamRows + 1) * 4 <=
                    2 * COLS * sizeof(T) + sizeof(double) * kTileMaxRows, "scratch within the dynamic LDS");
  if (blockIdx.x < kTileHubGroups) {
    for (int i = blockIdx.x; i < a.tile_count[2]; i += kTileHubGroups) {
      const HubBatch hb = a.hub_batch[i];
      const Task tk = a.tasks[hb.task];
      double sj;
      if (!open_step(a, tk, a.state + hb.task, 1, j, chunks, &sj)) continue;
      tile_hub_batch<T, HAS_VAL, false>(a, tk, hb, (const T*)a.V + tk.vec_off + vslot(a, j) * tk.n, sj, xs, red);
    }
    return;
  }
  const int sh = blockIdx.x - kTileHubGroups;
  const TileShare share = a.tile_share[sh];
  const int task = uniform(share.task);
  if (task < 0) return;
  RState* st = a.state + task;
  if (product_skipped(a, st, j)) return;
  const int n = uniform(share.n), rows = uniform(share.rows), flag = uniform(share.flag), q = uniform(share.q);
  const int C = a.pan_cols, S = (n + C - 1) / C, brows = (rows + kTileBands - 1) / kTileBands;
  const T* x = (const T*)a.V + uniform(share.vec_off) + vslot(a, j) * n;
  T* w = (T*)a.W + uniform(share.w_off);
  const int32_t* rp = a.row_ptr + uniform(share.rowptr_off) + share.r_begin;
  // this thread's chunk of the norm partials of step j - 1 (the canonical order of canonical_sum)
  const int nblk = uniform(share.nblk), chunk = part_chunk(nblk), nch = (nblk + chunk - 1) / chunk;
  double part = 0.0;
  if (j > 0 && tid < nch) {
    const double* np = a.npart + share.part_off / kPartStride;
    for (int b = tid * chunk; b < min(nblk, (tid + 1) * chunk); ++b) part += np[b];
  }
  // closes step j - 1 as open_step does; only the first share of a realization records it (all compute it)
  auto open = [&](double* sj) {
    if (j == 0) {
      *sj = st->s[0];
      return true;
    }
    if (tid < nch) chunks[tid] = part;
    __syncthreads();
    double ss = 0.0;
    for (int c = 0; c < nch; ++c) ss += chunks[c];
    const StepClose c = close_sum(st, ss, j - 1, a.eps);
    if (q == 0 && tid == 0) record_close(st, c, j);
    *sj = 1.0 / c.beta;
    return c.flags == 0;
  };
  double sj;
  if (flag & kTileFlagStream) {  // columns out of order: the CSR-stream arithmetic
    if (!open(&sj)) return;
    const Task tk = a.tasks[task];
    const T* va = HAS_VAL ? (const T*)a.values + tk.nnz_off : nullptr;
    for (int r0 = 0; r0 < rows; r0 += kStreamRows) {
      __syncthreads();  // the previous rows' LDS readers are done
      spmv_stream_rows<T, HAS_VAL, NT, StreamShape<T>::CAP, false, false, true, kBlock>(
          rp, a.col_idx + tk.nnz_off, va, x, r0, min(rows - r0, kStreamRows), sj, off, xs, w + r0, red);
    }
    return;
  }
  for (int i = tid; i < rows; i += NT) acc[i] = 0.0;
  if (wv >= kTileBands) {
    // Stage panel s into buffer s & 1 before barrier s; its last readers (panel s - 2) are past barrier s - 1.
    const int lt = tid - kTileBands * 64;
    const __amdgpu_buffer_rsrc_t rx = tile_rsrc(x, n * (int)sizeof(T));
    float4 A[UL], B[UL];
    auto load = [&](float4* r, int s) {  // past the last panel: out of range, zeros without traffic
      const int o = s < S ? s * C * (int)sizeof(T) : n * (int)sizeof(T);
#pragma unroll
      for (int u = 0; u < UL; ++u)
        r[u] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rx, o + (lt + u * kTileLoaders * 64) * 16, 0, 0));
    };
    auto store = [&](const float4* r, int s) {
      float4* b = (float4*)(xs + (s & 1) * COLS);
#pragma unroll
      for (int u = 0; u < UL; ++u) b[lt + u * kTileLoaders * 64] = r[u];
    };
    load(A, 0);
    load(B, 1);
    for (int s = 0; s < S; s += 2) {
      store(A, s);
      load(A, s + 2);
      lds_barrier();
      if (s + 1 < S) {
        store(B, s + 1);
        load(B, s + 3);
        lds_barrier();
      }
    }
  } else {
    const int64_t tab = (int64_t)sh * kTileBands + wv;
    const int64_t base = uniform(a.tile_base[tab]);
    const uint32_t* ends = a.tile_end + tab * a.pan_pmax;
    const uint32_t* ent = a.tile_ent + base;
    const T* val = HAS_VAL ? (const T*)a.tile_val + base : nullptr;
    const char* sums = (const char*)(acc + wv * brows);
    // Panel ends of 64 panels at a time, one per lane. The move makes the wait for them part of the load: later
    // reads of the register would else wait, at every panel, for all entries in flight.
    int ev = 0;
    auto load_ends = [&](int s) {
      const int got = s + lane < S ? (int)ends[s + lane] : 0;
      asm volatile("v_mov_b32 %0, %1" : "=v"(ev) : "v"(got));
    };
    load_ends(0);
    auto end_of = [&](int s) { return __builtin_amdgcn_readlane(ev, s & 63); };
    uint32_t e[D][U];
    T v[D][U];
    int cs[D], cn[D];            // each chunk's panel and entries
    int ls = 0, lq = 0, le = 0;  // the next chunk to load: panel, first entry, end of the panel
    auto settle = [&]() {        // ls: the first panel from it on with entries left (S: none)
      while (lq >= le) {
        if (++ls >= S) return;
        if ((ls & 63) == 0) load_ends(ls);
        le = end_of(ls);
      }
    };
    le = end_of(0);
    settle();
    auto load = [&](int d) {
      const int m = ls < S ? min(le - lq, U * 64) : 0;
      cs[d] = ls;
      cn[d] = m;
      // the resource ends at the chunk's last entry: lanes past it read zeros
      const __amdgpu_buffer_rsrc_t re = tile_rsrc(ent + lq, m * 4);
      const __amdgpu_buffer_rsrc_t rv = tile_rsrc(HAS_VAL ? val + lq : nullptr, HAS_VAL ? m * (int)sizeof(T) : 0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        e[d][u] = __builtin_amdgcn_raw_buffer_load_b32(re, (u * 64 + lane) * 4, 0, kTileStream);
        if constexpr (HAS_VAL) {
          if constexpr (sizeof(T) == 8)
            v[d][u] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rv, (u * 64 + lane) * 8, 0, kTileStream));
          else
            v[d][u] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rv, (u * 64 + lane) * 4, 0, kTileStream));
        }
      }
      lq += m;
      if (ls < S) settle();
    };
    int ready = -1;  // the panel whose barrier this wave passed last
    auto add = [&](int d) {
      while (ready < cs[d]) {
        lds_barrier();
        ++ready;
      }
      const char* xb = (const char*)(xs + (ready & 1) * COLS);
      const int m = cn[d];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u * 64 < m) {  // uniform
          const bool ok = u * 64 + lane < m;
          const uint32_t word = e[d][u];
          T p = *(const T*)(xb + (word & 0x7FFCu) * (sizeof(T) / 4));
          if constexpr (HAS_VAL) p = v[d][u] * p;
          using Lds = __attribute__((address_space(3))) double*;
          const Lds at = (Lds)(sums + ((word >> 13) & 0x1FF8u));
          const int rank = (int)(word >> 26);
          if (__ballot(rank != 0) == 0ull) {
            if (ok) __builtin_amdgcn_ds_atomic_fadd_f64(at, (double)p);
          } else {
            for (int r = 0;; ++r) {
              if (ok && rank == r) __builtin_amdgcn_ds_atomic_fadd_f64(at, (double)p);
              if (__ballot(rank > r) == 0ull) break;
            }
          }
        }
      }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d);
    while (cs[0] < S) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (cs[d] < S) add(d);
        load(d);
      }
    }
    for (; ready < S - 1; ++ready) lds_barrier();
  }
  __syncthreads();
  if (!open(&sj)) return;
  if (flag & kTileFlagHubs) {  // the long rows are written by their own workgroups
    const int hub = a.tile_share[sh].hub;
    for (int i = tid; i < rows; i += NT)
      if (rp[i + 1] - rp[i] <= hub) w[i] = (T)(acc[i] * sj);
  } else {
    for (int i = tid; i < rows; i += NT) w[i] = (T)(acc[i] * sj);
  }
}

// Two slices and the sums of the largest share (k_tile_pack may choose more rows than the host).
template <typename T>
constexpr size_t tile_lds() {
  return 2 * TileShape<T>::COLS * sizeof(T) + sizeof(double) * (size_t)kTileMaxRows;
}
size_t sort_lds(int panels) { return (1 + kTileClasses) * (size_t)panels * sizeof(int); }

template <typename K>
hipError_t allow(K kernel, size_t dyn) {
  return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
}

// k_spmv_tile by the length of a band's runs per panel (LzArgs::tile_short)
template <typename T, bool HAS_VAL, typename F>
auto tile_kernel(int run_short, F f) {
  return run_short ? f(k_spmv_tile<T, HAS_VAL, 2, 6>) : f(k_spmv_tile<T, HAS_VAL, 6, 3>);
}

template <typename T>
hipError_t prepare_tile_t() {
  const size_t srt = sort_lds(kTileMaxPanels);
  hipError_t e = hipSuccess;
  for (int r = 0; r < 2; ++r) {
    if (e == hipSuccess) e = tile_kernel<T, true>(r, [](auto k) { return allow(k, tile_lds<T>()); });
    if (e == hipSuccess) e = tile_kernel<T, false>(r, [](auto k) { return allow(k, tile_lds<T>()); });
  }
  if (e == hipSuccess) e = allow(k_tile_hub_first<T>, TileShape<T>::HCAP * sizeof(T));
  if (e == hipSuccess) e = allow(k_tile_sort<T, true>, srt);
  if (e == hipSuccess) e = allow(k_tile_sort<T, false>, srt);
  return e;
}

// Places of one launch: a launch's threads number less than 2^32, so batches of some 350000 realizations and more sort
// in several launches, and those of two million multiply in several (each of which takes the long rows).
constexpr int kSortPlaces = (int)(((int64_t)1 << 32) / (kTileBands * kSortThreads) / 8 * 8 - 8);
constexpr int kTilePlaces = (int)((((int64_t)1 << 32) / kTileThreads - kTileHubGroups) / 8 * 8 - 8);

// The arguments of a launch that starts at place p0.
LzArgs from_place(const LzArgs& a, int p0) {
  LzArgs p = a;
  p.tile_share += p0;
  p.tile_base += (int64_t)p0 * kTileBands;
  p.tile_end += (int64_t)p0 * kTileBands * a.pan_pmax;
  return p;
}

template <typename T>
hipError_t hub_first_t(const LzArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((k_tile_hub_first<T>), dim3(kTileHubGroups), dim3(kTileThreads), TileShape<T>::HCAP * sizeof(T), s,
                     a);
  return hipGetLastError();
}

template <typename T, bool HAS_VAL>
hipError_t tile_prepare_t(const LzArgs& a, int t0, int count, hipStream_t s) {
  const int places = (a.ntile + 7) / 8 * 8;
  hipLaunchKernelGGL(k_tile_cut, dim3((unsigned)count), dim3(64), 0, s, a, t0, 0);
  hipLaunchKernelGGL(k_tile_pack, dim3(1), dim3(1024), 0, s, a, t0, count, 0);
  hipLaunchKernelGGL(k_tile_cut, dim3((unsigned)count), dim3(64), 0, s, a, t0, 1);
  hipLaunchKernelGGL(k_tile_pack, dim3(1), dim3(1024), 0, s, a, t0, count, 1);
  hipLaunchKernelGGL(k_tile_fill, dim3((unsigned)((places + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, a, t0, count,
                     places);
  for (int p0 = 0; p0 < places; p0 += kSortPlaces)
    hipLaunchKernelGGL((k_tile_sort<T, HAS_VAL>), dim3((unsigned)(std::min(places - p0, kSortPlaces) * kTileBands)),
                       dim3(kSortThreads), sort_lds(a.pan_pmax), s, from_place(a, p0));
  if constexpr (HAS_VAL)
    if (a.first_in_prepare) return hub_first_t<T>(a, s);
  return hipGetLastError();
}

template <typename T, bool HAS_VAL>
hipError_t spmv_tile_t(int j, const LzArgs& a, hipStream_t s) {
  const int places = (a.ntile + 7) / 8 * 8;
  return tile_kernel<T, HAS_VAL>(a.tile_short, [&](auto k) {
    for (int p0 = 0; p0 < places; p0 += kTilePlaces)
      hipLaunchKernelGGL(k, dim3((unsigned)(std::min(places - p0, kTilePlaces) + kTileHubGroups)), dim3(kTileThreads),
                         tile_lds<T>(), s, from_place(a, p0), j);
    return hipGetLastError();
  });
}

}  // namespace

hipError_t prepare_tile_kernels() {
  static hipError_t e = [] {
    hipError_t r = prepare_tile_t<float>();
    if (r == hipSuccess) r = prepare_tile_t<double>();
    return r;
  }();
  return e;
}

int tile_max_cols(int dtype) { return dtype == EBTC_F64 ? TileShape<double>::COLS : TileShape<float>::COLS; }

int64_t tile_hub_rows(int64_t entries) { return entries / (kTileHubMin + 1) + 1; }

hipError_t launch_tile_prepare(int dtype, bool has_val, const LzArgs& a, int t0, int count, hipStream_t s) {
  if (a.pan_cols <= 0 || a.pan_cols > tile_max_cols(dtype) || a.pan_pmax < 1 || a.pan_pmax > kTileMaxPanels ||
      a.tile_rows < 1 || a.tile_rows > kTileMaxRows || a.tile_least < 1 || a.tile_least > a.tile_rows ||
      a.ntile < 1 || a.ntile > kTileMaxSlots || count < 1)
    return hipErrorInvalidValue;
  if (dtype == EBTC_F64)
    return has_val ? tile_prepare_t<double, true>(a, t0, count, s) : tile_prepare_t<double, false>(a, t0, count, s);
  return has_val ? tile_prepare_t<float, true>(a, t0, count, s) : tile_prepare_t<float, false>(a, t0, count, s);
}

hipError_t launch_tile_hub_first(int dtype, const LzArgs& a, hipStream_t s) {
  return dtype == EBTC_F64 ? hub_first_t<double>(a, s) : hub_first_t<float>(a, s);
}

hipError_t launch_spmv_tile(int dtype, bool has_val, int j, const LzArgs& a, hipStream_t s) {
  if (dtype == EBTC_F64) return has_val ? spmv_tile_t<double, true>(j, a, s) : spmv_tile_t<double, false>(j, a, s);
  return has_val ? spmv_tile_t<float, true>(j, a, s) : spmv_tile_t<float, false>(j, a, s);
}

}  // namespace ebtc
