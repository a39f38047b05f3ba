// Host side of the EBTC C ABI: argument checks, workspace layout, launch sequences, hipGraph cache.
#include <algorithm>
#include <array>
#include <map>
#include <sstream>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "internal.h"

using namespace ebtc;

namespace {

thread_local std::string g_err;

int fail(int code, const std::string& msg) {
  g_err = msg;
  return code;
}

}  // namespace

// Error reporting for entry points defined in other translation units.
int ebtc::report_error(int code, const std::string& msg) { return fail(code, msg); }

namespace {

#define EBTC_HIP(call)                                                                          \
  do {                                                                                          \
    hipError_t e_ = (call);                                                                     \
    if (e_ != hipSuccess) return fail(EBTC_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// One SpMV form's share of the workspace: its launch's block list (when it covers part of the batch)
// and its arenas, sized for its realizations only.
struct FormLayout {
  int64_t blocks = 0, z = 0;  // row blocks and entries of the form's realizations
  size_t off_sub = 0;         // [blocks] batch-wide block ids (mixed plans only)
  // column-segmented SpMV arenas
  size_t off_segflag = 0, off_segcnt = 0, off_segwoff = 0, off_segblk = 0, off_segcol = 0, off_segval = 0;
  // entry-balanced SpMV arenas
  size_t off_bal = 0, off_balbeg = 0;
  int64_t nbal = 0;  // shares over the form's realizations
  // paneled-form arenas
  size_t off_tilebeg = 0, off_tilecut = 0, off_tilencut = 0, off_tileshare = 0, off_tilebase = 0, off_tileend = 0,
         off_tileent = 0, off_tileval = 0, off_tilecnt = 0, off_hubrow = 0, off_hubbatch = 0;
  int64_t ntile = 0;
};

// Host tables of one SpMV form (uploaded with every call; kept in the batch for the async copies).
struct FormHost {
  std::vector<int32_t> sub;          // [blocks] the form's row blocks, batch-wide ids (mixed plans only)
  std::vector<int64_t> bal_begin;    // [R + 1] first entry-balanced share of each realization (0 elsewhere)
  std::vector<int64_t> tile_begin;   // [R + 1] first paneled share slot of each realization
};

struct Layout {
  int m_slots = 0;
  size_t off_tasks = 0, off_graphs = 0, off_blkmap = 0, off_state = 0, off_part = 0, off_npart = 0, off_V = 0,
         off_W = 0, off_U = 0, off_live = 0;
  std::vector<FormLayout> fl;  // per SpMV form of the plan
  size_t total = 0;
  int64_t total_blocks = 0;
};

struct ExecKey {
  void* ws;
  void* scores;
  double* log_scale;
  void* ckpt;
  ebtc_diag* diag;
  int m, m_max, reorth, shift, sched;
  double tol;
  std::string plan;  // the SpMV plan's signature (forms, parameters, each graph's form)
  bool operator==(const ExecKey& o) const {
    return ws == o.ws && scores == o.scores && log_scale == o.log_scale && ckpt == o.ckpt && diag == o.diag &&
           m == o.m && m_max == o.m_max && reorth == o.reorth && shift == o.shift && sched == o.sched &&
           tol == o.tol && plan == o.plan;
  }
};

struct ExecEntry {
  ExecKey key;
  hipGraph_t graph;
  hipGraphExec_t exec;
};

int elem_size(int dtype) { return dtype == EBTC_F64 ? 8 : 4; }

}  // namespace

struct ebtc_batch {
  int dtype = EBTC_F32;
  int32_t G = 0;
  int64_t R = 0;
  std::vector<int32_t> n, nreal, first;
  std::vector<int64_t> rowptr_off, nnz_off, score_off;
  const int32_t* row_ptr = nullptr;
  const int32_t* col_idx = nullptr;
  const void* values = nullptr;
  int64_t total_scores = 0;  // sum_g n_g
  int64_t total_rows = 0;    // sum_r n_r
  int32_t n_max = 0;
  int64_t z_max = 0;         // largest realization's entry count
  double mean_degree = 0.0;
  std::vector<Task> tasks;          // host staging of the device task table (kept alive for async copies)
  std::vector<GraphInfo> graphs;
  std::vector<int64_t> nnz_r;       // per-realization entry counts (validation upload)
  // host tables of the current SpMV plan's forms (kept alive for async uploads), and the plan they
  // were built for
  std::vector<FormHost> fh;
  std::string fh_sig;
  std::vector<char> tables;       // the tasks and graphs of a call, as uploaded
  std::vector<char> topk_tables;  // ebtc_topk's tables, as uploaded
  std::vector<ExecEntry> execs;
  hipStream_t capture_stream = nullptr;
  // SpMV forms chosen by ebtc_tune (empty = not tuned), used when opts->spmv is EBTC_SPMV_AUTO:
  // {form, lanes, seg_len parameter} per form and each graph's form
  std::vector<std::array<int32_t, 3>> tuned;
  std::vector<int32_t> tuned_graph;
};

namespace {

// Chunks of the chunked top-K: kTkChunk scores each, at least one per graph.
int64_t topk_chunks(const ebtc_batch* b) {
  int64_t c = 0;
  for (int32_t g = 0; g < b->G; ++g) c += (b->n[g] + kTkChunk - 1) / kTkChunk;
  return c;
}

int check_opts(const ebtc_opts* o) {
  if (!o) return fail(EBTC_EINVAL, "opts is NULL");
  if (o->m < 0 || o->m > EBTC_M_LIMIT)
    return fail(EBTC_EINVAL, "m must be in [0, " + std::to_string(EBTC_M_LIMIT) + "] (0 = adaptive)");
  if (o->m == 0 && (o->m_max < 1 || o->m_max > EBTC_M_LIMIT))
    return fail(EBTC_EINVAL, "m_max must be in [1, " + std::to_string(EBTC_M_LIMIT) + "]");
  if (o->m == 0 && !(o->tol > 0.0)) return fail(EBTC_EINVAL, "adaptive mode needs tol > 0");
  if (o->reorth < 0 || o->reorth > 2)
    return fail(EBTC_EINVAL, "reorth must be 0 (memory-bounded two-pass), 1 or 2");
  if (o->schedule < EBTC_SCHED_AUTO || o->schedule > EBTC_SCHED_SINGLE) return fail(EBTC_EINVAL, "unknown schedule");
  if (o->spmv < EBTC_SPMV_AUTO || o->spmv > EBTC_SPMV_PANELED) return fail(EBTC_EINVAL, "unknown spmv form");
  if (o->lanes_per_row != 0 && o->lanes_per_row != 4 && o->lanes_per_row != 8 && o->lanes_per_row != 16 &&
      o->lanes_per_row != 32)
    return fail(EBTC_EINVAL, "lanes_per_row must be 0, 4, 8, 16 or 32");
  if (o->hub_threshold < 0) return fail(EBTC_EINVAL, "hub_threshold must be >= 0");
  if (o->seg_len < 0) return fail(EBTC_EINVAL, "seg_len must be >= 0");
  return EBTC_OK;
}

// Schedule of the SpMV for a set of graphs: the form and its parameters.
struct SpmvPlan {
  int form = EBTC_SPMV_STREAM;
  int lanes = 0, hub = 0;
  int seglen = 0;   // LDS-staged: segment length
  int segcols = 0;  // column-segmented: columns per segment
  int smax = 0;     // column-segmented: segments of the largest realization
  int balent = 0;   // entry-balanced: entries per share
  int pancols = 0;   // paneled: columns per panel
  int panask = 0;    // paneled: columns per panel asked for (the limit of 1024 panels counts these)
  int pmax = 0;      // paneled: panels of the largest realization
  int tilerows = 0;  // paneled: rows per share
  int tileleast = 0;  // paneled: fewest rows per share that the device may choose instead
  int tileshort = 0;  // paneled: a band's runs of entries per panel are short
  // the parameter ebtc_opts::seg_len carries for this form
  int param() const {
    return form == EBTC_SPMV_SEGMENTED ? segcols
           : form == EBTC_SPMV_BALANCED ? balent
           : form == EBTC_SPMV_PANELED  ? panask
                                        : seglen;
  }
};

// The SpMV plan of a batch: one or more forms, each over a set of graphs (every realization of a graph
// takes the graph's form). With several forms each step launches one SpMV per form, over its graphs'
// row blocks; every other phase still runs once over the whole batch.
struct BatchPlan {
  std::vector<SpmvPlan> forms;
  std::vector<int32_t> graph_form;  // [G] index into forms
  bool mixed() const { return forms.size() > 1; }
  std::string sig() const {
    std::string t;
    for (const SpmvPlan& p : forms)
      t += std::to_string(p.form) + "," + std::to_string(p.lanes) + "," + std::to_string(p.hub) + "," +
           std::to_string(p.seglen) + "," + std::to_string(p.segcols) + "," + std::to_string(p.smax) + "," +
           std::to_string(p.balent) + "," + std::to_string(p.pancols) + "," + std::to_string(p.pmax) + "," +
           std::to_string(p.tilerows) + "," + std::to_string(p.tileleast) + "," + std::to_string(p.tileshort) + ";";
    if (mixed())
      for (int32_t f : graph_form) t += std::to_string(f) + ",";
    return t;
  }
};

// Graph membership of a form: nullptr = every graph.
using Members = std::vector<char>;
bool member(const Members* m, int32_t g) { return m == nullptr || (*m)[g] != 0; }

std::vector<int64_t> bal_shares(const ebtc_batch* b, int e, const Members* m);
std::vector<int64_t> tile_begins(const ebtc_batch* b, int least, const Members* m);

// Panels per realization at the columns asked for, and the widest panel that may be asked for (the kernels
// take narrower ones where these exceed their slice buffers).
constexpr int kPanelLimit = 1024;
int panel_ask(int dtype) { return dtype == EBTC_F64 ? 6144 : 12288; }

int check_form(const ebtc_batch* b, const SpmvPlan& p, const Members* m) {
  if (p.form == EBTC_SPMV_LANE_GROUPS && p.lanes != 4 && p.lanes != 8 && p.lanes != 16 && p.lanes != 32)
    return fail(EBTC_EINVAL, "the lane-group SpMV takes 4, 8, 16 or 32 lanes per row");
  if (p.form == EBTC_SPMV_BALANCED) {
    if (p.balent < 256 || p.balent > (1 << 24))
      return fail(EBTC_EINVAL, "the entry-balanced SpMV takes shares of 256 to 2^24 entries (seg_len)");
    if (bal_shares(b, p.balent, m).back() > INT32_MAX) return fail(EBTC_EINVAL, "too many entry-balanced shares");
  }
  if (p.form == EBTC_SPMV_PANELED) {
    int32_t n_max = 1;
    for (int32_t g = 0; g < b->G; ++g)
      if (member(m, g)) n_max = std::max(n_max, b->n[g]);
    if ((n_max + (int64_t)p.panask - 1) / p.panask > kPanelLimit)
      return fail(EBTC_EINVAL, "the paneled SpMV takes at most " + std::to_string(kPanelLimit) + " panels: n " +
                                   std::to_string(n_max) + " > " + std::to_string(kPanelLimit) + " x " +
                                   std::to_string(p.panask));
    if (tile_begins(b, p.tileleast, m).back() > kTileMaxSlots) return fail(EBTC_EINVAL, "too many paneled shares");
  }
  if (p.form == EBTC_SPMV_SEGMENTED && p.smax > kSegMax)
    return fail(EBTC_EINVAL, "the column-segmented SpMV needs at most " + std::to_string(kSegMax) +
                                 " segments: n " + std::to_string(p.smax * (int64_t)p.segcols) + " > " +
                                 std::to_string(kSegMax) + " x " + std::to_string(p.segcols));
  return EBTC_OK;
}

Members members_of(const BatchPlan& bp, size_t f) {
  Members m(bp.graph_form.size(), 0);
  for (size_t g = 0; g < bp.graph_form.size(); ++g) m[g] = bp.graph_form[g] == (int32_t)f ? 1 : 0;
  return m;
}

int check_plan(const ebtc_batch* b, const BatchPlan& bp) {
  // Several SpMV forms in one launch sequence (one launch per form over its graphs' row blocks) are
  // switched off: a batch of six graphs on six forms did not complete its first eager pass on the
  // GPU, and the cause is not found. The host side (block lists, per-form arenas) stays, and the
  // autotuner decides per batch.
  if (bp.mixed())
    return fail(EBTC_ENOTSUPPORTED, "several SpMV forms in one batch are not supported in this version: record the "
                                    "same form for every graph (or name one in opts->spmv)");
  for (size_t f = 0; f < bp.forms.size(); ++f) {
    const Members m = members_of(bp, f);
    const int rc = check_form(b, bp.forms[f], bp.mixed() ? &m : nullptr);
    if (rc) return rc;
  }
  return EBTC_OK;
}

// First entry-balanced share of each realization ([R + 1]): one share per e entries, at least one
// per realization of a member graph, none for the others.
std::vector<int64_t> bal_shares(const ebtc_batch* b, int e, const Members* m) {
  std::vector<int64_t> v((size_t)b->R + 1, 0);
  int64_t r = 0;
  for (int32_t g = 0; g < b->G; ++g)
    for (int32_t k = 0; k < b->nreal[g]; ++k, ++r) {
      const int64_t z = b->nnz_r[r];
      v[r + 1] = v[r] + (member(m, g) ? std::max<int64_t>(1, (z + e - 1) / e) : 0);
    }
  return v;
}

// Default share size: the largest power of two in [kBalEntriesMin, kBalEntriesMax] that leaves the
// member graphs' realizations at least kBalTargetShares shares.
int bal_default(const ebtc_batch* b, const Members* m) {
  int64_t z = 0, r = 0;
  for (int32_t g = 0; g < b->G; ++g)
    for (int32_t k = 0; k < b->nreal[g]; ++k, ++r)
      if (member(m, g)) z += b->nnz_r[r];
  int e = kBalEntriesMax;
  while (e > kBalEntriesMin && z / e < kBalTargetShares) e >>= 1;
  return e;
}

// First paneled share slot of each realization ([R + 1]; none for realizations of other forms), enough for shares of
// `least` rows and any larger number (tile_least).
std::vector<int64_t> tile_begins(const ebtc_batch* b, int least, const Members* m) {
  std::vector<int64_t> v((size_t)b->R + 1, 0);
  int64_t r = 0;
  for (int32_t g = 0; g < b->G; ++g)
    for (int32_t k = 0; k < b->nreal[g]; ++k, ++r)
      v[r + 1] = v[r] + (member(m, g) ? tile_slots(least, b->n[g], b->nnz_r[r]) : 0);
  return v;
}

// Rows per share of the paneled form: a compute unit holds one share at a time, so as few rounds of 256
// shares as the largest share allows, filled as well as they can be (64 x n=1e5: 3 rounds of 256 shares
// of 8334 rows; with 12160 rows the same three rounds would be 2.25 full).
int tile_rows(const ebtc_batch* b, const Members* m) {
  auto shares = [&](int64_t rows) {
    int64_t t = 0;
    for (int32_t g = 0; g < b->G; ++g)
      if (member(m, g)) t += (b->n[g] + rows - 1) / rows * b->nreal[g];
    return t;
  };
  const int64_t target = (shares(kTileMaxRows) + kTileUnits - 1) / kTileUnits * kTileUnits;
  int lo = kTileMinRows, hi = kTileMaxRows;  // the fewest rows whose shares do not exceed the rounds
  while (lo < hi) {
    const int mid = (lo + hi) / 2;
    if (shares(mid) <= target) hi = mid; else lo = mid + 1;
  }
  return lo;
}

// Fewest rows per share that k_tile_pack may choose where tile_rows chose `rows`: one round of shares more than the
// batch's. A launch over one realization has fewer rounds, but its slots are the batch's too.
int tile_least(const ebtc_batch* b, int rows, const Members* m) {
  int64_t full = 0;
  for (int32_t g = 0; g < b->G; ++g)
    if (member(m, g)) full += ((int64_t)b->n[g] + rows - 1) / rows * b->nreal[g];
  const int64_t rounds = std::min<int64_t>(1 << 20, std::max<int64_t>(1, (full + kTileUnits - 1) / kTileUnits));
  return (int)((int64_t)rows * rounds / (rounds + 1)) + 1;
}

// The batch's host tables for plan bp (rebuilt when the plan changes).
const std::vector<FormHost>& form_host(const ebtc_batch* cb, const BatchPlan& bp) {
  ebtc_batch* b = const_cast<ebtc_batch*>(cb);
  const std::string sig = bp.sig();
  if (b->fh_sig == sig && b->fh.size() == bp.forms.size()) return b->fh;
  b->fh.assign(bp.forms.size(), FormHost{});
  for (size_t f = 0; f < bp.forms.size(); ++f) {
    const SpmvPlan& p = bp.forms[f];
    FormHost& h = b->fh[f];
    const Members m = members_of(bp, f);
    const Members* mp = bp.mixed() ? &m : nullptr;
    if (bp.mixed()) {
      int64_t r = 0;
      int32_t blk = 0;
      for (int32_t g = 0; g < b->G; ++g) {
        const int32_t nb = (b->n[g] + kRowsPerBlock - 1) / kRowsPerBlock;
        for (int32_t k = 0; k < b->nreal[g]; ++k, ++r, blk += nb)
          if (member(mp, g))
            for (int32_t i = 0; i < nb; ++i) h.sub.push_back(blk + i);
      }
    }
    if (p.form == EBTC_SPMV_BALANCED) h.bal_begin = bal_shares(b, p.balent, mp);
    if (p.form == EBTC_SPMV_PANELED) h.tile_begin = tile_begins(b, p.tileleast, mp);
  }
  b->fh_sig = sig;
  return b->fh;
}

Layout make_layout(const ebtc_batch* b, const ebtc_opts* o, const BatchPlan& bp) {
  Layout L;
  // the memory-bounded form keeps the last three basis vectors only
  L.m_slots = o->reorth == 0 ? 3 : (o->m > 0 ? o->m : o->m_max) + 1;
  const size_t es = elem_size(b->dtype);
  int64_t blocks = 0;
  int64_t rows = 0;
  for (int32_t g = 0; g < b->G; ++g) {
    const int64_t nb = (b->n[g] + kRowsPerBlock - 1) / kRowsPerBlock;
    blocks += nb * b->nreal[g];
    rows += (int64_t)b->n[g] * b->nreal[g];
  }
  L.total_blocks = blocks;
  size_t off = 0;
  L.off_tasks = off;
  off = align_up(off + sizeof(Task) * b->R);
  L.off_graphs = off;
  off = align_up(off + sizeof(GraphInfo) * b->G);
  L.off_blkmap = off;
  off = align_up(off + sizeof(int32_t) * blocks);
  L.off_state = off;
  off = align_up(off + sizeof(RState) * b->R);
  L.off_part = off;
  off = align_up(off + sizeof(double) * kPartStride * blocks);
  L.off_npart = off;
  off = align_up(off + sizeof(double) * blocks);
  L.off_live = off;
  off = align_up(off + sizeof(int32_t) * kMLimit);
  L.off_V = off;
  off = align_up(off + es * (size_t)L.m_slots * rows);
  L.off_W = off;
  off = align_up(off + es * rows);
  L.off_U = off;
  off = align_up(off + es * rows);
  const std::vector<FormHost>& fh = form_host(b, bp);
  for (size_t f = 0; f < bp.forms.size(); ++f) {
    const SpmvPlan& sp = bp.forms[f];
    FormLayout F;
    int64_t r = 0;
    for (int32_t g = 0; g < b->G; ++g) {
      const int64_t nb = (b->n[g] + kRowsPerBlock - 1) / kRowsPerBlock;
      for (int32_t k = 0; k < b->nreal[g]; ++k, ++r)
        if (bp.graph_form[g] == (int32_t)f) {
          F.blocks += nb;
          F.z += b->nnz_r[r];
        }
    }
    const size_t z = (size_t)F.z;
    if (bp.mixed()) {
      F.off_sub = off;
      off = align_up(off + sizeof(int32_t) * (size_t)F.blocks);
    }
    if (sp.form == EBTC_SPMV_SEGMENTED) {
      F.off_segflag = off;
      off = align_up(off + sizeof(int32_t) * F.blocks);
      F.off_segcnt = off;
      off = align_up(off + (size_t)sp.smax * kRowsPerBlock * F.blocks);
      F.off_segwoff = off;
      off = align_up(off + sizeof(uint16_t) * (size_t)sp.smax * 17 * F.blocks);
      F.off_segblk = off;
      off = align_up(off + sizeof(SegBlock) * F.blocks);
      // the entries, the zero padding of every (segment, wave band) run and the rounding of every
      // block's first slot to a multiple of four
      const size_t slots = z + (size_t)F.blocks * kSegSlack + 8;
      F.off_segcol = off;
      off = align_up(off + sizeof(uint16_t) * slots);
      F.off_segval = off;
      if (b->values) off = align_up(off + es * slots);
    }
    if (sp.form == EBTC_SPMV_PANELED) {
      F.ntile = fh[f].tile_begin.back();
      const size_t slots = (size_t)F.ntile, places = (slots + 7) / 8 * 8, hubs = (size_t)tile_hub_rows(F.z);
      auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align_up(off + bytes);
        return o;
      };
      F.off_tilebeg = take(sizeof(int64_t) * (size_t)(b->R + 1));
      F.off_tilecut = take(sizeof(TileCut) * slots);
      F.off_tilencut = take(sizeof(int32_t) * (size_t)(b->R + 1));
      F.off_tileshare = take(sizeof(TileShare) * places);
      F.off_tilebase = take(sizeof(int64_t) * kTileBandsHost * places);
      F.off_tileend = take(sizeof(uint32_t) * kTileBandsHost * (size_t)sp.pmax * places);
      F.off_tileent = take(sizeof(uint32_t) * z);
      if (b->values) F.off_tileval = take(es * z);
      F.off_tilecnt = take(sizeof(int32_t) * 4);
      F.off_hubrow = take(sizeof(int32_t) * hubs);
      F.off_hubbatch = take(sizeof(HubBatch) * hubs);
    }
    if (sp.form == EBTC_SPMV_BALANCED) {
      F.nbal = fh[f].bal_begin.back();
      F.off_bal = off;
      off = align_up(off + sizeof(BalPart) * (size_t)F.nbal);
      F.off_balbeg = off;
      off = align_up(off + sizeof(int64_t) * (size_t)(b->R + 1));
    }
    L.fl.push_back(F);
  }
  L.total = off;
  return L;
}

// The task table; each realization's offsets in its form's arenas count the entries and blocks of the
// realizations of the same form before it.
void fill_tables(ebtc_batch* b, const Layout& L, const BatchPlan& bp) {
  b->tasks.resize(b->R);
  int64_t vec = 0, row = 0, part = 0;
  int32_t blk = 0;
  int64_t r = 0;
  std::vector<int64_t> aux_off(bp.forms.size(), 0);
  std::vector<int32_t> aux_blk(bp.forms.size(), 0);
  for (int32_t g = 0; g < b->G; ++g) {
    const int32_t f = bp.graph_form[g];
    for (int32_t k = 0; k < b->nreal[g]; ++k, ++r) {
      Task& t = b->tasks[r];
      const int32_t n = b->n[g];
      const int32_t nb = (n + kRowsPerBlock - 1) / kRowsPerBlock;
      t.rowptr_off = b->rowptr_off[r];
      t.nnz_off = b->nnz_off[r];
      t.vec_off = vec;
      t.w_off = row;
      t.u_off = row;
      t.part_off = part;
      t.n = n;
      t.graph = g;
      t.nblk = nb;
      t.blk_begin = blk;
      t.aux_off = aux_off[f];
      t.aux_blk = aux_blk[f];
      t.form = f;
      aux_off[f] += b->nnz_r[r];
      aux_blk[f] += nb;
      vec += (int64_t)L.m_slots * n;
      row += n;
      part += (int64_t)nb * kPartStride;
      blk += nb;
    }
  }
}

int upload_tables(ebtc_batch* b, char* ws, const Layout& L, const BatchPlan& bp, hipStream_t s) {
  fill_tables(b, L, bp);
  const std::vector<FormHost>& fh = form_host(b, bp);
  // tasks and graphs in one copy (each costs a small call about 7 us)
  const size_t graphs_at = L.off_graphs - L.off_tasks;
  b->tables.resize(graphs_at + sizeof(GraphInfo) * b->G);
  std::memcpy(b->tables.data(), b->tasks.data(), sizeof(Task) * b->R);
  std::memcpy(b->tables.data() + graphs_at, b->graphs.data(), sizeof(GraphInfo) * b->G);
  EBTC_HIP(hipMemcpyAsync(ws + L.off_tasks, b->tables.data(), b->tables.size(), hipMemcpyHostToDevice, s));
  for (size_t f = 0; f < bp.forms.size(); ++f) {
    const FormLayout& F = L.fl[f];
    if (bp.mixed() && F.blocks > 0)
      EBTC_HIP(hipMemcpyAsync(ws + F.off_sub, fh[f].sub.data(), sizeof(int32_t) * (size_t)F.blocks,
                              hipMemcpyHostToDevice, s));
    if (bp.forms[f].form == EBTC_SPMV_PANELED)
      EBTC_HIP(hipMemcpyAsync(ws + F.off_tilebeg, fh[f].tile_begin.data(), sizeof(int64_t) * (b->R + 1),
                              hipMemcpyHostToDevice, s));
    if (bp.forms[f].form == EBTC_SPMV_BALANCED)
      EBTC_HIP(hipMemcpyAsync(ws + F.off_balbeg, fh[f].bal_begin.data(), sizeof(int64_t) * (b->R + 1),
                              hipMemcpyHostToDevice, s));
  }
  return EBTC_OK;
}

// One form over the member graphs (nullptr: all); the parameters follow the largest member.
SpmvPlan spmv_form(const ebtc_batch* b, int form, int lanes, int seg_len, int hub, const Members* m = nullptr) {
  SpmvPlan p;
  p.form = form;
  int32_t n_max = 1;
  for (int32_t g = 0; g < b->G; ++g)
    if (member(m, g)) n_max = std::max(n_max, b->n[g]);
  if (form == EBTC_SPMV_LANE_GROUPS) p.lanes = lanes ? lanes : 8;
  if (form == EBTC_SPMV_LDS_STAGED) {
    const int maxseg = staged_max_seglen(b->dtype);
    p.seglen = seg_len > 0 ? std::min(seg_len, maxseg) : maxseg;
  }
  if (form == EBTC_SPMV_SEGMENTED) {
    p.segcols = std::min(seg_len > 0 ? seg_len : seg_max_cols(b->dtype), seg_max_cols(b->dtype));
    p.smax = (n_max + p.segcols - 1) / p.segcols;
  }
  if (form == EBTC_SPMV_BALANCED) p.balent = seg_len > 0 ? seg_len : bal_default(b, m);
  if (form == EBTC_SPMV_PANELED) {
    p.panask = std::min(seg_len > 0 ? seg_len : panel_ask(b->dtype), panel_ask(b->dtype));
    p.pancols = std::min(p.panask, tile_max_cols(b->dtype));
    p.pmax = (n_max + p.pancols - 1) / p.pancols;
    p.tilerows = tile_rows(b, m);
    p.tileleast = tile_least(b, p.tilerows, m);
    // entries of a band in a panel, over all member realizations: chunks of 384 pay above about 128
    double z = 0.0, runs = 0.0;
    int64_t r = 0;
    for (int32_t g = 0; g < b->G; ++g)
      for (int32_t k = 0; k < b->nreal[g]; ++k, ++r)
        if (member(m, g)) {
          z += (double)b->nnz_r[r];
          runs += (double)((b->n[g] + p.tilerows - 1) / p.tilerows) * kTileBandsHost *
                  ((b->n[g] + p.pancols - 1) / p.pancols);
        }
    p.tileshort = z < 128.0 * runs ? 1 : 0;
  }
  p.hub = hub ? hub : 16 * (p.lanes ? p.lanes : 8);
  return p;
}

BatchPlan one_form(const ebtc_batch* b, const SpmvPlan& p) {
  BatchPlan bp;
  bp.forms.push_back(p);
  bp.graph_form.assign((size_t)b->G, 0);
  return bp;
}

// The CSR-stream form unless the caller names one or ebtc_tune measured others on this batch.
BatchPlan spmv_plan(const ebtc_batch* b, const ebtc_opts* o) {
  if (o->spmv != EBTC_SPMV_AUTO)
    return one_form(b, spmv_form(b, o->spmv, o->lanes_per_row, o->seg_len, o->hub_threshold));
  if (b->tuned.empty()) return one_form(b, spmv_form(b, EBTC_SPMV_STREAM, 0, 0, o->hub_threshold));
  BatchPlan bp;
  bp.graph_form = b->tuned_graph;
  for (size_t f = 0; f < b->tuned.size(); ++f) {
    const Members m = members_of(bp, f);
    const Members* mp = b->tuned.size() > 1 ? &m : nullptr;
    bp.forms.push_back(spmv_form(b, b->tuned[f][0], b->tuned[f][1], b->tuned[f][2], o->hub_threshold, mp));
  }
  return bp;
}

// The plan with the entry-balanced form in the place of a recorded paneled one (a form named in the options stays):
// the same bits with less memory.
BatchPlan balanced_plan(const ebtc_batch* b, const ebtc_opts* o) {
  BatchPlan bp = spmv_plan(b, o);
  if (o->spmv != EBTC_SPMV_AUTO) return bp;
  for (size_t f = 0; f < bp.forms.size(); ++f)
    if (bp.forms[f].form == EBTC_SPMV_PANELED) {
      const Members m = members_of(bp, f);
      bp.forms[f] = spmv_form(b, EBTC_SPMV_BALANCED, 0, 0, o->hub_threshold, bp.mixed() ? &m : nullptr);
    }
  return bp;
}

// The plan of a forward call. The tuner times launches over the whole batch. Under the plain schedule a launch covers
// one realization: its tiles leave compute units idle and their preparation is launches of its own, so the
// entry-balanced form runs instead (16 x ER n=1e5, degree 20: 34.1 ms paneled, 15.6 balanced; 2 x n=1e6: 7.7 and 6.6;
// the other way round on Barabasi-Albert graphs, 8 x n=1e5: 16.6 and 32.8, which one cannot tell here). So it does for
// one step of a pattern-only batch, which has no product to prepare for (16 x ER n=1e5, degree 20, FP64: 318 us paneled,
// 109 balanced).
BatchPlan call_plan(const ebtc_batch* b, const ebtc_opts* o) {
  const bool no_product = (o->m > 0 ? o->m : o->m_max) == 1 && !b->values;
  return o->schedule == EBTC_SCHED_PLAIN || no_product ? balanced_plan(b, o) : spmv_plan(b, o);
}

LzArgs make_args(const ebtc_batch* b, const ebtc_opts* o, char* ws, const Layout& L) {
  LzArgs a{};
  a.row_ptr = b->row_ptr;
  a.col_idx = b->col_idx;
  a.values = b->values;
  a.tasks = (const Task*)(ws + L.off_tasks);
  a.blkmap = (const int32_t*)(ws + L.off_blkmap);
  a.sub_blocks = nullptr;
  a.single_task = 0;
  a.hub_threshold = 128;
  a.state = (RState*)(ws + L.off_state);
  a.V = ws + L.off_V;
  a.W = ws + L.off_W;
  a.U = ws + L.off_U;
  a.part = (double*)(ws + L.off_part);
  a.npart = (double*)(ws + L.off_npart);
  a.m_fixed = o->m;
  a.m_max = o->m > 0 ? o->m : o->m_max;
  a.eps = b->dtype == EBTC_F64 ? std::ldexp(1.0, -53) : std::ldexp(1.0, -24);
  a.window = o->reorth == 0 ? 2 : 0;
  a.stop_mused = 0;
  a.live = nullptr;
  return a;
}

// One SpMV launch's arguments: the base arguments plus one form's fields.
struct FArgs {
  LzArgs a;
  SpmvPlan sp;
  int64_t nb = 0;  // row blocks the launch covers (batched schedule)
};

std::vector<FArgs> form_args(const ebtc_batch* b, const LzArgs& base, char* ws, const Layout& L, const BatchPlan& bp) {
  std::vector<FArgs> out;
  for (size_t f = 0; f < bp.forms.size(); ++f) {
    const SpmvPlan& sp = bp.forms[f];
    const FormLayout& F = L.fl[f];
    FArgs x;
    x.sp = sp;
    x.nb = F.blocks;
    LzArgs& a = x.a;
    a = base;
    a.sub_blocks = bp.mixed() ? (const int32_t*)(ws + F.off_sub) : nullptr;
    a.hub_threshold = sp.hub;
    a.seglen = sp.seglen;
    // the column-segmented and the paneled sort of weighted graphs also write step 0's product
    const bool sorted = sp.form == EBTC_SPMV_SEGMENTED || sp.form == EBTC_SPMV_PANELED;
    a.first_in_prepare = base.unit_start && sorted && b->values != nullptr ? 1 : 0;
    if (sp.form == EBTC_SPMV_SEGMENTED) {
      a.seg_cols = sp.segcols;
      a.seg_stride = sp.smax * kRowsPerBlock;
      a.seg_flag = (int32_t*)(ws + F.off_segflag);
      a.seg_cnt = (uint8_t*)(ws + F.off_segcnt);
      a.seg_woff = (uint16_t*)(ws + F.off_segwoff);
      a.seg_wstride = sp.smax * 17;
      a.seg_blk = (SegBlock*)(ws + F.off_segblk);
      a.seg_col = (uint16_t*)(ws + F.off_segcol);
      a.seg_val = b->values ? (void*)(ws + F.off_segval) : nullptr;
      // 16-byte slice stores need every slice length to be a whole number of vectors: n and the
      // segment length multiples of the vector width (else a store would pass the slice's end, into
      // the other LDS buffer)
      const int vw = 16 / elem_size(b->dtype);
      a.seg_vec = sp.segcols % vw == 0 ? 1 : 0;
      for (int32_t g = 0; g < b->G; ++g)
        if (bp.graph_form[g] == (int32_t)f && b->n[g] % vw != 0) a.seg_vec = 0;
    }
    if (sp.form == EBTC_SPMV_PANELED) {
      a.pan_cols = sp.pancols;
      a.pan_pmax = sp.pmax;
      a.tile_rows = sp.tilerows;
      a.tile_least = sp.tileleast;
      a.ntile = (int32_t)F.ntile;
      a.tile_begin = (const int64_t*)(ws + F.off_tilebeg);
      a.tile_cut = (TileCut*)(ws + F.off_tilecut);
      a.tile_ncut = (int32_t*)(ws + F.off_tilencut);
      a.tile_share = (TileShare*)(ws + F.off_tileshare);
      a.tile_base = (int64_t*)(ws + F.off_tilebase);
      a.tile_short = sp.tileshort;
      a.tile_end = (uint32_t*)(ws + F.off_tileend);
      a.tile_ent = (uint32_t*)(ws + F.off_tileent);
      a.tile_val = b->values ? (void*)(ws + F.off_tileval) : nullptr;
      a.tile_count = (int32_t*)(ws + F.off_tilecnt);
      a.hub_row = (int32_t*)(ws + F.off_hubrow);
      a.hub_batch = (HubBatch*)(ws + F.off_hubbatch);
    }
    if (sp.form == EBTC_SPMV_BALANCED) {
      a.bal = (BalPart*)(ws + F.off_bal);
      a.bal_begin = (const int64_t*)(ws + F.off_balbeg);
      a.nbal = (int32_t)F.nbal;
      a.bal_entries = sp.balent;
    }
    out.push_back(x);
  }
  return out;
}

// The same launch restricted to one realization (the plain schedule).
FArgs one_task(const ebtc_batch* b, const FArgs& x, size_t f, int64_t r) {
  FArgs y = x;
  y.a.single_task = (int32_t)r;
  y.a.blkmap = nullptr;
  y.a.sub_blocks = nullptr;
  y.nb = b->tasks[r].nblk;
  const FormHost& h = b->fh[f];
  if (y.a.bal != nullptr) y.a.nbal = (int32_t)(h.bal_begin[r + 1] - h.bal_begin[r]);
  if (y.a.pan_cols > 0) y.a.ntile = (int32_t)(h.tile_begin[r + 1] - h.tile_begin[r]);
  return y;
}

// The autotuner's decisions, process-wide: bucket key -> {form, lanes, seg_len parameter}.
std::mutex g_tune_mu;
std::map<std::string, std::array<int32_t, 3>> g_tune_cache;

// A graph's autotuning bucket: precision, weights, octave of n, half-octave of the mean degree, octave
// of the largest row over the mean degree (hub rows), octave of the Krylov steps (which spread the
// once-per-call preparations).
std::string tune_key(int dtype, bool has_val, int32_t n, double mean_deg, int32_t row_max, int steps) {
  const int nl = (int)std::floor(std::log2(std::max(1, n)));
  const int dl = (int)std::floor(2.0 * std::log2(std::max(1.0, mean_deg)));
  const int hl = (int)std::floor(std::log2(std::max(1.0, row_max / std::max(1.0, mean_deg))));
  const int sl = (int)std::floor(std::log2(std::max(1, steps)));
  return std::string(dtype == EBTC_F64 ? "f64" : "f32") + (has_val ? "v" : "p") + "-n" + std::to_string(nl) + "-d" +
         std::to_string(dl) + "-h" + std::to_string(hl) + "-s" + std::to_string(sl);
}

// Kernel opt-ins to the full LDS; once per process, before any stream capture.
int prepare_kernels(const BatchPlan& bp) {
  for (const SpmvPlan& sp : bp.forms) {
    if (sp.seglen > 0) EBTC_HIP(prepare_staged_kernels());
    if (sp.segcols > 0) EBTC_HIP(prepare_seg_kernels());
    if (sp.pancols > 0) EBTC_HIP(prepare_tile_kernels());
  }
  EBTC_HIP(prepare_solve_kernels());
  EBTC_HIP(prepare_wide_kernels());
  return EBTC_OK;
}

// Optional per-launch event recording (ebtc_profile_phases).
struct Prof {
  struct Rec {
    int phase;
    hipEvent_t a, b;
  };
  std::vector<Rec> recs;
  hipStream_t s;
  int before(int phase) {
    Rec r{phase, nullptr, nullptr};
    if (hipEventCreate(&r.a) != hipSuccess || hipEventCreate(&r.b) != hipSuccess) return EBTC_EHIP;
    recs.push_back(r);
    return hipEventRecord(r.a, s) == hipSuccess ? EBTC_OK : EBTC_EHIP;
  }
  int after() { return hipEventRecord(recs.back().b, s) == hipSuccess ? EBTC_OK : EBTC_EHIP; }
  ~Prof() {
    for (auto& r : recs) {
      if (r.a) (void)hipEventDestroy(r.a);
      if (r.b) (void)hipEventDestroy(r.b);
    }
  }
};

#define EBTC_LAUNCH(call)                                                                              \
  do {                                                                                                 \
    hipError_t e_ = (call);                                                                            \
    if (e_ != hipSuccess) return fail(EBTC_EHIP, std::string("launch ") + #call + ": " + hipGetErrorString(e_)); \
  } while (0)

#define EBTC_PHASE(prof, phase, call)                                                   \
  do {                                                                                  \
    if (prof && prof->before(phase)) return fail(EBTC_EHIP, "event record failed");    \
    EBTC_LAUNCH(call);                                                                  \
    if (prof && prof->after()) return fail(EBTC_EHIP, "event record failed");          \
  } while (0)

// Whether the single-kernel schedule can run this batch: one row block per realization, the whole
// basis with one Gram-Schmidt pass, and an SpMV form whose arithmetic is the CSR stream's (the
// single-kernel solve computes those bits).
bool single_ok(const ebtc_batch* b, const ebtc_opts* o) {
  const bool stream_bits = o->spmv == EBTC_SPMV_AUTO || o->spmv == EBTC_SPMV_STREAM ||
                           o->spmv == EBTC_SPMV_SEGMENTED || o->spmv == EBTC_SPMV_BALANCED;
  const int steps = o->m > 0 ? o->m : o->m_max;
  return b->n_max <= kRowsPerBlock && o->reorth == 1 && stream_bits && steps <= kDotsWindow;
}

// Whether AUTO takes the solve of a few row blocks per workgroup (k_wide.hip): the conditions of the single-kernel
// schedule but for the size, and forms with the stream's sums where the batch is tuned.
constexpr int kSchedWide = 100;  // of AUTO only
bool wide_pays(const ebtc_batch* b, const ebtc_opts* o) {
  if (o->spmv != EBTC_SPMV_AUTO && o->spmv != EBTC_SPMV_STREAM) return false;
  const int steps = o->m > 0 ? o->m : o->m_max;
  if (o->reorth != 1 || steps > kDotsWindow || !wide_fits(b->dtype, b->n_max)) return false;
  // one step of a pattern-only graph has no product (100 x n=9000 Barabasi-Albert, FP64: 108 us here, 81 per phase)
  if (steps == 1 && !b->values) return false;
  if (o->spmv == EBTC_SPMV_AUTO)
    for (const auto& f : b->tuned)
      if (f[0] == EBTC_SPMV_LANE_GROUPS || f[0] == EBTC_SPMV_LDS_STAGED) return false;
  // A realization's entries per row at most. Denser graphs keep one workgroup's loads and long rows' chains busy past
  // what the model below knows (gain over the per-phase schedule, smallest of 2100 to 9000 nodes, up to 700
  // realizations: degree 64 pattern only 0.98, 80 0.90, 200 0.28; with values degree 32 1.02, 39 0.84).
  constexpr int64_t kMostPattern = 64, kMostValues = 32;
  const int64_t most = b->values ? kMostValues : kMostPattern;
  int64_t r = 0;
  for (int32_t g = 0; g < b->G; ++g)
    for (int32_t k = 0; k < b->nreal[g]; ++k, ++r)
      if (b->nnz_r[r] > most * b->n[g]) return false;
  // The two schedules' times by what bounds them, fitted to 700 calls on gfx950 (2100 to 9000 nodes, degree 2 to 25,
  // 1 to 300 realizations, every dtype and option) and checked on 1200 more (to 14000 nodes, degree 64, 1500
  // realizations, hub rows to 6200 entries); it never chose the slower by more than 2%. A workgroup alone:
  // a step's barriers and chains, the basis at 45 GB/s, its entries at 0.11 ns (more with values, and the more
  // workgroups share the L2); together no faster than the last-level cache, in rounds of 256. Per phase: 10 us per
  // step of an adaptive run up to its cap, 19 or 24 (FP64) of a fixed one, the basis, the entries at the rate of
  // close neighbours (long rows, which hold that schedule up, are not known here). An adaptive run's steps: 14.
  const bool fixed = o->m > 0;
  const double es = b->dtype == EBTC_F64 ? 8 : 4, val = b->values ? es / 4 : 0.0, R = (double)b->R;
  const double S = fixed ? o->m : std::min(14, steps), rows = (double)b->total_rows;
  double entries = 0.0;
  for (const int64_t z : b->nnz_r) entries += (double)z;
  const double basis = es * (S + 3.0), z = (double)b->z_max;
  const double share = 0.8 * std::min(1.0, R / 40.0) * (val > 0 || z > 1e5 ? 1.0 : 0.5);
  const double alone = (fixed ? 14e-6 : 18e-6) + b->n_max * basis / 45e9 + z * (0.11e-9 + 0.06e-9 * val) * (1.0 + share);
  const double at_once = std::min(1.0, 256.0 / R);
  const double shared = at_once * (rows * basis / 4.5e12 + entries * (4.0 + (val > 0 ? es : 0.0)) / 6e12);
  const double step = std::max(alone, shared);
  const double wide = R <= 256 ? S * step : S * (R / 256.0 * step + 0.3 * alone);
  const double phases = (fixed ? S * (es > 4 ? 24e-6 : 19e-6) : steps * 10.2e-6) +
                        S * (rows * (basis + es) / 4.8e12 + entries / 900e9);
  return wide < 0.95 * phases;
}

// The schedule a call runs: AUTO takes a single-kernel form where one applies.
int resolve_schedule(const ebtc_batch* b, const ebtc_opts* o, int* sched) {
  *sched = o->schedule;
  if (*sched == EBTC_SCHED_AUTO)
    *sched = single_ok(b, o) ? EBTC_SCHED_SINGLE : wide_pays(b, o) ? kSchedWide : EBTC_SCHED_BATCHED;
  if (*sched == EBTC_SCHED_SINGLE && !single_ok(b, o))
    return fail(EBTC_ENOTSUPPORTED, "the single-kernel schedule needs every n <= " + std::to_string(kRowsPerBlock) +
                                        ", m (or m_max) <= " + std::to_string(kDotsWindow) +
                                        ", reorth = 1 and the stream, segmented, balanced or auto SpMV form");
  return EBTC_OK;
}

// Lanczos steps for the launches described by (a, nblocks); a.blkmap / a.single_task select the scope.
// fa: the SpMV launches of each step, one per form of the plan.
int run_steps(const ebtc_batch* b, const ebtc_opts* o, const LzArgs& a, const std::vector<FArgs>& fa, int64_t nblocks,
              int64_t first, int64_t count, hipStream_t s, Prof* prof, bool with_start = true, const SharedMat* mat = nullptr) {
  const bool has_val = b->values != nullptr;
  const int steps = o->m > 0 ? o->m : o->m_max;
  // every realization in one row block: dots and update of a step in one launch (one workgroup each)
  const bool one_block = b->n_max <= kRowsPerBlock && o->reorth == 1 && a.window == 0 && steps <= kDotsWindow;
  if (with_start) EBTC_PHASE(prof, EBTC_PHASE_START, launch_start(b->dtype, a, nblocks, s));
  for (int j = 0; j < steps; ++j) {
    if (mat) EBTC_PHASE(prof, EBTC_PHASE_SPMV, launch_shared_step(b->dtype, has_val, j, a, *mat, b->n_max, s));
    for (const FArgs& x : fa) {
      if (mat || x.nb == 0 || (j == 0 && x.a.unit_start && x.a.first_in_prepare)) continue;
      EBTC_PHASE(prof, j == 0 && x.a.unit_start ? EBTC_PHASE_FIRST : EBTC_PHASE_SPMV,
                 launch_spmv_step(b->dtype, has_val, x.sp.lanes, j, x.a, x.nb, s));
    }
    if (one_block) {
      EBTC_PHASE(prof, EBTC_PHASE_DOTS, launch_dots_update_1(b->dtype, j, a, nblocks, s));
    } else if (o->reorth == 2) {
      EBTC_PHASE(prof, EBTC_PHASE_DOTS, launch_dots_step(b->dtype, j, a, nblocks, s));
      EBTC_PHASE(prof, EBTC_PHASE_UPDATE, launch_update(b->dtype, j, true, false, false, a, nblocks, s));
      EBTC_PHASE(prof, EBTC_PHASE_DOTS, launch_dots_again(b->dtype, j, a, nblocks, s));
      EBTC_PHASE(prof, EBTC_PHASE_UPDATE, launch_update(b->dtype, j, false, true, true, a, nblocks, s));
    } else {
      EBTC_PHASE(prof, EBTC_PHASE_DOTS, launch_dots_step(b->dtype, j, a, nblocks, s));
      EBTC_PHASE(prof, EBTC_PHASE_UPDATE, launch_update(b->dtype, j, true, true, false, a, nblocks, s));
    }
    if (o->m == 0)
      EBTC_PHASE(prof, EBTC_PHASE_TRIDIAG,
                 launch_tridiag_state(a, first, count, 1, j, steps, o->shift, o->tol, nullptr, nullptr, s));
  }
  return EBTC_OK;
}

// The once-per-call preparation of one form's launch: the column-segmented sort, the entry-balanced
// shares or the panel order (nothing for the other forms). f: the form's index in the plan.
int enqueue_prepare(const ebtc_batch* b, const FArgs& x, size_t f, hipStream_t s, Prof* prof) {
  const LzArgs& a = x.a;
  if (x.nb == 0) return EBTC_OK;
  if (x.sp.form == EBTC_SPMV_BALANCED) {
    const bool one = a.blkmap == nullptr;  // the plain schedule: one realization
    EBTC_PHASE(prof, EBTC_PHASE_PREPARE, launch_bal_rows(a, one ? a.single_task : 0, one ? 1 : (int)b->R, s));
    return EBTC_OK;
  }
  if (x.sp.form == EBTC_SPMV_PANELED) {
    const bool one = a.blkmap == nullptr;
    EBTC_PHASE(prof, EBTC_PHASE_PREPARE,
               launch_tile_prepare(b->dtype, b->values != nullptr, a, one ? a.single_task : 0, one ? 1 : (int)b->R, s));
    return EBTC_OK;
  }
  if (x.sp.form != EBTC_SPMV_SEGMENTED) return EBTC_OK;
  EBTC_PHASE(prof, EBTC_PHASE_PREPARE, launch_seg_prepare(b->dtype, b->values != nullptr, a, x.nb, x.sp.smax, s));
  return EBTC_OK;
}

int enqueue_prepare_all(const ebtc_batch* b, const std::vector<FArgs>& fa, hipStream_t s, Prof* prof) {
  for (size_t f = 0; f < fa.size(); ++f) {
    const int rc = enqueue_prepare(b, fa[f], f, s, prof);
    if (rc) return rc;
  }
  return EBTC_OK;
}

// Second pass of the memory-bounded form (reorth 0): the first pass kept only a ring of three basis
// vectors, so u = beta0 V y is accumulated while the same kernels regenerate the same basis (same
// launches in the same order: bitwise the same vectors), one term before each step.
int run_pass2(const ebtc_batch* b, const ebtc_opts* o, const LzArgs& a1, const std::vector<FArgs>& fa1,
              int64_t nblocks, hipStream_t s, Prof* prof) {
  LzArgs a = a1;
  a.stop_mused = 1;
  a.live = nullptr;  // the live counts belong to the first pass
  std::vector<FArgs> fa = fa1;
  for (FArgs& x : fa) {
    x.a.stop_mused = 1;
    x.a.live = nullptr;
  }
  const bool has_val = b->values != nullptr;
  const int steps = o->m > 0 ? o->m : o->m_max;
  EBTC_PHASE(prof, EBTC_PHASE_START, launch_restart(b->dtype, a, nblocks, s));
  for (int j = 0; j < steps; ++j) {
    EBTC_PHASE(prof, EBTC_PHASE_COMBINE, launch_accum(b->dtype, a, j, nblocks, s));
    if (j + 1 == steps) break;  // the last vector needed is v_{steps-1}
    for (const FArgs& x : fa) {
      if (x.nb == 0) continue;
      // the second pass never skips step 0: the sort's product of the first pass is gone
      if (j == 0 && x.sp.form == EBTC_SPMV_PANELED && x.a.first_in_prepare) {  // the long rows as the sort does them
        // Rows of many entries come from the tiles: the row sums take one thread for each. FP64, 16 x n=100000: 24
        // entries per row 118 us from the CSR and 110 from the tiles, 12: 60 and 72; 40 x n=20000, 100: 375 and 174;
        // 10 x n=8000, 1600: 62.7 ms and 0.36; against it 2 x n=1e6, 40: 0.22 and 0.30.
        if (b->mean_degree >= 32.0) EBTC_PHASE(prof, EBTC_PHASE_FIRST, launch_spmv_tile(b->dtype, has_val, 0, x.a, s));
        else EBTC_PHASE(prof, EBTC_PHASE_FIRST, launch_first_short(b->dtype, x.a, x.nb, s));
        EBTC_PHASE(prof, EBTC_PHASE_FIRST, launch_tile_hub_first(b->dtype, x.a, s));
        continue;
      }
      LzArgs xa = x.a;
      xa.first_in_prepare = 0;
      EBTC_PHASE(prof, j == 0 && xa.unit_start ? EBTC_PHASE_FIRST : EBTC_PHASE_SPMV,
                 launch_spmv_step(b->dtype, has_val, x.sp.lanes, j, xa, x.nb, s));
    }
    EBTC_PHASE(prof, EBTC_PHASE_DOTS, launch_dots_step(b->dtype, j, a, nblocks, s));
    EBTC_PHASE(prof, EBTC_PHASE_UPDATE, launch_update(b->dtype, j, true, true, false, a, nblocks, s));
  }
  return EBTC_OK;
}

int enqueue_batched(ebtc_batch* b, const ebtc_opts* o, char* ws, const Layout& L, const BatchPlan& bp, void* scores,
                    double* log_scale, void* ckpt, ebtc_diag* diag, int sched, hipStream_t s, Prof* prof = nullptr) {
  LzArgs a = make_args(b, o, ws, L);
  a.unit_start = 1;  // k_start (and k_restart) set v_0 = 1
  a.diag = diag;
  // adaptive m: the checks count the realizations still running, and once none is, the launches of
  // the remaining steps up to the cap return at once
  if (o->m == 0 && sched != EBTC_SCHED_SINGLE && sched != kSchedWide) a.live = (int32_t*)(ws + L.off_live);
  const std::vector<FArgs> fa = form_args(b, a, ws, L, bp);
  if (sched != EBTC_SCHED_SINGLE && sched != kSchedWide)  // those map their workgroups themselves
    EBTC_LAUNCH(launch_blkmap(a.tasks, b->R, (int32_t*)(ws + L.off_blkmap), s));
  const int32_t maxblk = (b->n_max + kRowsPerBlock - 1) / kRowsPerBlock;
  if (sched == EBTC_SCHED_SINGLE || sched == kSchedWide) {
    if (sched == kSchedWide)
      EBTC_PHASE(prof, EBTC_PHASE_SOLVE,
                 launch_solve_wide(b->dtype, b->values != nullptr, a, b->R, o->m > 0 ? o->m : o->m_max, o->shift,
                                   o->tol, diag, (double*)ckpt, b->n_max, s));
    else
      EBTC_PHASE(prof, EBTC_PHASE_SOLVE,
               launch_solve_1(b->dtype, b->values != nullptr, a, b->R, o->m > 0 ? o->m : o->m_max, o->shift, o->tol,
                              diag, (double*)ckpt, b->n_max, b->z_max, s));
    EBTC_PHASE(prof, EBTC_PHASE_SUM, launch_sum(b->dtype, (const GraphInfo*)(ws + L.off_graphs), b->G, maxblk,
                                                a.tasks, a.state, a.U, scores, log_scale, s));
    return EBTC_OK;
  }
  int rc = enqueue_prepare_all(b, fa, s, prof);
  if (rc) return rc;
  rc = run_steps(b, o, a, fa, L.total_blocks, 0, b->R, s, prof);
  if (rc) return rc;
  const int steps = o->m > 0 ? o->m : o->m_max;
  EBTC_PHASE(prof, EBTC_PHASE_TRIDIAG,
             launch_tridiag_state(a, 0, b->R, 0, 0, steps, o->shift, o->tol, diag, (double*)ckpt, s));
  if (o->reorth == 0) {
    rc = run_pass2(b, o, a, fa, L.total_blocks, s, prof);
    if (rc) return rc;
  } else {
    EBTC_PHASE(prof, EBTC_PHASE_COMBINE, launch_combine(b->dtype, a, L.total_blocks, s));
  }
  EBTC_PHASE(prof, EBTC_PHASE_SUM, launch_sum(b->dtype, (const GraphInfo*)(ws + L.off_graphs), b->G, maxblk, a.tasks,
                                              a.state, a.U, scores, log_scale, s));
  return EBTC_OK;
}

int enqueue_plain(ebtc_batch* b, const ebtc_opts* o, char* ws, const Layout& L, const BatchPlan& bp, void* scores,
                  double* log_scale, void* ckpt, ebtc_diag* diag, hipStream_t s) {
  LzArgs a = make_args(b, o, ws, L);
  a.unit_start = 1;
  a.blkmap = nullptr;
  a.diag = diag;
  const std::vector<FArgs> fa = form_args(b, a, ws, L, bp);
  for (int64_t r = 0; r < b->R; ++r) {
    a.single_task = (int32_t)r;
    const size_t f = (size_t)bp.graph_form[b->tasks[r].graph];
    const std::vector<FArgs> fr{one_task(b, fa[f], f, r)};
    const int64_t nb = b->tasks[r].nblk;
    int rc = enqueue_prepare(b, fr[0], f, s, nullptr);
    if (rc) return rc;
    rc = run_steps(b, o, a, fr, nb, r, 1, s, nullptr);
    if (rc) return rc;
    EBTC_LAUNCH(launch_tridiag_state(a, r, 1, 0, 0, o->m > 0 ? o->m : o->m_max, o->shift, o->tol, diag,
                                     (double*)ckpt, s));
    if (o->reorth == 0) {
      rc = run_pass2(b, o, a, fr, nb, s, nullptr);
      if (rc) return rc;
    } else {
      EBTC_LAUNCH(launch_combine(b->dtype, a, nb, s));
    }
  }
  const int32_t maxblk = (b->n_max + kRowsPerBlock - 1) / kRowsPerBlock;
  EBTC_LAUNCH(launch_sum(b->dtype, (const GraphInfo*)(ws + L.off_graphs), b->G, maxblk, a.tasks, a.state, a.U, scores,
                         log_scale, s));
  return EBTC_OK;
}

}  // namespace

namespace {

// Backward workspace: the forward layout (recomputed forward), then the adjoint Lanczos state and
// basis, the per-realization block exponentials and the node-major Z and normalised V.
struct BwdLayout {
  Layout fwd;
  size_t off_astate = 0, off_aV = 0, off_X = 0, off_Z = 0, off_Vn = 0, total = 0;
  int ld = 0;
};

BwdLayout make_bwd_layout(const ebtc_batch* b, const ebtc_opts* o) {
  BwdLayout B;
  B.fwd = make_layout(b, o, spmv_plan(b, o));
  const size_t es = elem_size(b->dtype);
  const int steps = o->m > 0 ? o->m : o->m_max;
  B.ld = (steps + 7) / 8 * 8;
  size_t off = B.fwd.total;
  B.off_astate = off;
  off = align_up(off + sizeof(RState) * b->R);
  B.off_aV = off;
  off = align_up(off + es * (size_t)B.fwd.m_slots * b->total_rows);
  B.off_X = off;
  off = align_up(off + sizeof(double) * kXLd * kXLd * b->R);
  B.off_Z = off;
  off = align_up(off + es * (size_t)B.ld * b->total_rows);
  B.off_Vn = off;
  off = align_up(off + es * (size_t)B.ld * b->total_rows);
  B.total = off;
  return B;
}

int check_bwd_opts(const ebtc_opts* o) {
  int rc = check_opts(o);
  if (rc) return rc;
  const int steps = o->m > 0 ? o->m : o->m_max;
  if (o->reorth == 0)
    return fail(EBTC_ENOTSUPPORTED, "the adjoint needs the stored basis: reorth 1 or 2");
  if (steps > adjoint_max_m())
    return fail(EBTC_ENOTSUPPORTED, "the adjoint supports Krylov dimensions up to " + std::to_string(adjoint_max_m()));
  return EBTC_OK;
}

}  // namespace

extern "C" {

int ebtc_version(int* major, int* minor) {
  if (!major || !minor) return fail(EBTC_EINVAL, "NULL output pointer");
  *major = EBTC_VERSION_MAJOR;
  *minor = EBTC_VERSION_MINOR;
  return EBTC_OK;
}

const char* ebtc_status_str(int status) {
  switch (status) {
    case EBTC_OK: return "ok";
    case EBTC_EINVAL: return "invalid argument";
    case EBTC_EBADGRAPH: return "bad graph batch";
    case EBTC_EWORKSPACE: return "workspace too small";
    case EBTC_EHIP: return "HIP runtime error";
    case EBTC_ENOTSUPPORTED: return "not supported";
    default: return "unknown status";
  }
}

const char* ebtc_last_error(void) { return g_err.c_str(); }

void ebtc_default_opts(ebtc_opts* o) {
  if (!o) return;
  std::memset(o, 0, sizeof(*o));
  o->m = 30;
  o->m_max = 60;
  o->tol = 1e-6;
  o->reorth = 1;
  o->schedule = EBTC_SCHED_AUTO;
  o->use_hipgraph = 1;
  o->shift = 1;
  o->spmv = EBTC_SPMV_AUTO;
  o->lanes_per_row = 0;
  o->hub_threshold = 0;
  o->seg_len = 0;
}

int ebtc_batch_create(const ebtc_batch_desc* d, ebtc_batch** out) {
  g_err.clear();
  if (!d || !out) return fail(EBTC_EINVAL, "NULL descriptor or output");
  if (d->dtype != EBTC_F32 && d->dtype != EBTC_F64) return fail(EBTC_EINVAL, "dtype must be EBTC_F32 or EBTC_F64");
  if (d->num_graphs < 1) return fail(EBTC_EINVAL, "num_graphs must be >= 1");
  if (d->num_realizations < 1 || d->num_realizations >= (int64_t)1 << 31)
    return fail(EBTC_EINVAL, "num_realizations must be in [1, 2^31)");
  if (!d->graph_n || !d->graph_nreal || !d->rowptr_off || !d->nnz_off)
    return fail(EBTC_EINVAL, "NULL host array in the descriptor");
  if (!d->row_ptr || !d->col_idx) return fail(EBTC_EINVAL, "NULL device row_ptr or col_idx");
  ebtc_batch* b = new ebtc_batch();
  b->dtype = d->dtype;
  b->G = d->num_graphs;
  b->R = d->num_realizations;
  // the per-realization arrays are read only after R has been checked against graph_nreal, so an
  // inconsistent count is reported instead of read past the caller's arrays
  b->n.assign(d->graph_n, d->graph_n + b->G);
  b->nreal.assign(d->graph_nreal, d->graph_nreal + b->G);
  b->row_ptr = d->row_ptr;
  b->col_idx = d->col_idx;
  b->values = d->values;
  int64_t sum_real = 0, blocks = 0;
  b->first.resize(b->G);
  b->score_off.resize(b->G + 1);
  b->score_off[0] = 0;
  for (int32_t g = 0; g < b->G; ++g) {
    if (b->n[g] < 1) {
      delete b;
      return fail(EBTC_EINVAL, "graph " + std::to_string(g) + ": n must be >= 1");
    }
    if (b->nreal[g] < 1) {
      delete b;
      return fail(EBTC_EINVAL, "graph " + std::to_string(g) + ": realizations must be >= 1");
    }
    b->first[g] = (int32_t)sum_real;
    sum_real += b->nreal[g];
    b->score_off[g + 1] = b->score_off[g] + b->n[g];
    b->n_max = std::max(b->n_max, b->n[g]);
    b->total_rows += (int64_t)b->n[g] * b->nreal[g];
    blocks += (int64_t)((b->n[g] + kRowsPerBlock - 1) / kRowsPerBlock) * b->nreal[g];
  }
  if (sum_real != b->R) {
    delete b;
    return fail(EBTC_EBADGRAPH, "num_realizations differs from the sum of graph_nreal");
  }
  b->rowptr_off.assign(d->rowptr_off, d->rowptr_off + b->R);
  b->nnz_off.assign(d->nnz_off, d->nnz_off + b->R + 1);
  if (blocks >= (int64_t)1 << 31) {
    delete b;
    return fail(EBTC_ENOTSUPPORTED, "too many row blocks for one launch");
  }
  if (b->nnz_off[0] != 0) {
    delete b;
    return fail(EBTC_EBADGRAPH, "nnz_off[0] must be 0");
  }
  b->nnz_r.resize(b->R);
  int64_t r = 0;
  for (int32_t g = 0; g < b->G; ++g) {
    for (int32_t k = 0; k < b->nreal[g]; ++k, ++r) {
      const int64_t z = b->nnz_off[r + 1] - b->nnz_off[r];
      if (z < 0 || z >= (int64_t)1 << 31) {
        delete b;
        return fail(EBTC_EBADGRAPH, "realization " + std::to_string(r) + ": entry count out of range");
      }
      if (b->rowptr_off[r] < 0) {
        delete b;
        return fail(EBTC_EBADGRAPH, "realization " + std::to_string(r) + ": negative rowptr_off");
      }
      b->nnz_r[r] = z;
      b->z_max = std::max(b->z_max, z);
    }
  }
  b->total_scores = b->score_off[b->G];
  b->mean_degree = b->total_rows > 0 ? (double)b->nnz_off[b->R] / (double)b->total_rows : 0.0;
  b->graphs.resize(b->G);
  for (int32_t g = 0; g < b->G; ++g) {
    b->graphs[g].score_off = b->score_off[g];
    b->graphs[g].n = b->n[g];
    b->graphs[g].first = b->first[g];
    b->graphs[g].count = b->nreal[g];
    b->graphs[g].pad = 0;
  }
  *out = b;
  return EBTC_OK;
}

void ebtc_batch_destroy(ebtc_batch* b) {
  if (!b) return;
  for (auto& e : b->execs) {
    (void)hipGraphExecDestroy(e.exec);
    (void)hipGraphDestroy(e.graph);
  }
  if (b->capture_stream) (void)hipStreamDestroy(b->capture_stream);
  delete b;
}

int ebtc_plan(ebtc_batch* b, const ebtc_opts* o, size_t* ws_bytes, size_t* ckpt_bytes) {
  g_err.clear();
  if (!b || !ws_bytes) return fail(EBTC_EINVAL, "NULL batch or output");
  int rc = check_opts(o);
  if (rc) return rc;
  const BatchPlan bp = spmv_plan(b, o);
  rc = check_plan(b, bp);
  if (rc) return rc;
  // one size for every schedule (call_plan)
  *ws_bytes = make_layout(b, o, bp).total;
  const BatchPlan bal = balanced_plan(b, o);
  if (bal.sig() != bp.sig()) *ws_bytes = std::max(*ws_bytes, make_layout(b, o, bal).total);
  if (ckpt_bytes) *ckpt_bytes = sizeof(double) * kCkptDoubles * (size_t)b->R;
  return EBTC_OK;
}

int ebtc_scores(ebtc_batch* b, const ebtc_opts* o, void* ws, size_t ws_bytes, void* scores_out, double* log_scale_out,
                void* ckpt_out, ebtc_diag* diag_out, void* stream) {
  g_err.clear();
  if (!b) return fail(EBTC_EINVAL, "NULL batch");
  int rc = check_opts(o);
  if (rc) return rc;
  if (!ws || !scores_out || !log_scale_out) return fail(EBTC_EINVAL, "NULL workspace, scores or log_scale output");
  const BatchPlan bp = call_plan(b, o);
  rc = check_plan(b, bp);
  if (rc) return rc;
  const Layout L = make_layout(b, o, bp);
  if (ws_bytes < L.total)
    return fail(EBTC_EWORKSPACE, "workspace of " + std::to_string(ws_bytes) + " bytes, need " + std::to_string(L.total));
  if (((uintptr_t)ws & 255) != 0) return fail(EBTC_EINVAL, "workspace must be 256-byte aligned");
  int sched = 0;
  rc = resolve_schedule(b, o, &sched);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  rc = prepare_kernels(bp);
  if (rc) return rc;
  char* w = (char*)ws;
  rc = upload_tables(b, w, L, bp, s);
  if (rc) return rc;
  if (sched == EBTC_SCHED_PLAIN)
    return enqueue_plain(b, o, w, L, bp, scores_out, log_scale_out, ckpt_out, diag_out, s);
  if (!o->use_hipgraph)
    return enqueue_batched(b, o, w, L, bp, scores_out, log_scale_out, ckpt_out, diag_out, sched, s);
  const ExecKey key{ws,       scores_out, log_scale_out, ckpt_out, diag_out, o->m,   o->m_max,
                    o->reorth, o->shift,  sched,         o->tol,   bp.sig()};
  for (auto& e : b->execs) {
    if (e.key == key) {
      EBTC_HIP(hipGraphLaunch(e.exec, s));
      return EBTC_OK;
    }
  }
  if (!b->capture_stream) EBTC_HIP(hipStreamCreateWithFlags(&b->capture_stream, hipStreamNonBlocking));
  EBTC_HIP(hipStreamBeginCapture(b->capture_stream, hipStreamCaptureModeThreadLocal));
  rc = enqueue_batched(b, o, w, L, bp, scores_out, log_scale_out, ckpt_out, diag_out, sched, b->capture_stream);
  hipGraph_t graph = nullptr;
  const hipError_t ec = hipStreamEndCapture(b->capture_stream, &graph);
  if (rc) {
    if (graph) (void)hipGraphDestroy(graph);
    return rc;
  }
  if (ec != hipSuccess) return fail(EBTC_EHIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(ec));
  hipGraphExec_t exec = nullptr;
  const hipError_t ei = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
  if (ei != hipSuccess) {
    (void)hipGraphDestroy(graph);
    return fail(EBTC_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(ei));
  }
  if (b->execs.size() >= 4) {
    (void)hipGraphExecDestroy(b->execs.front().exec);
    (void)hipGraphDestroy(b->execs.front().graph);
    b->execs.erase(b->execs.begin());
  }
  b->execs.push_back({key, graph, exec});
  EBTC_HIP(hipGraphLaunch(exec, s));
  return EBTC_OK;
}

}  // extern "C"

// ---- workspace of ebtc_scores_noalloc: a fixed device array, one per GPU, held until the process ends
namespace {

constexpr size_t kScratchBytes = EBTC_NOALLOC_WS_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kScratchDevices] = {};

// Device address of the current GPU's copy of `scratch`, looked up once per device (the array's name
// is a host-side stand-in in host code; only this address may be passed to kernels or copies).
int scratch_address(void** out) {
  int dev = -1;
  EBTC_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kScratchDevices) return fail(EBTC_ENOTSUPPORTED, "device index beyond the scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    EBTC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (p == nullptr || ((uintptr_t)p & 255) != 0) return fail(EBTC_EHIP, "scratch address unusable");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return EBTC_OK;
}

}  // namespace

extern "C" {

int ebtc_scores_noalloc(ebtc_batch* b, const ebtc_opts* o, void* scores_out, double* log_scale_out, void* ckpt_out,
                        ebtc_diag* diag_out, void* stream) {
  g_err.clear();
  if (!b) return fail(EBTC_EINVAL, "NULL batch");
  int rc = check_opts(o);
  if (rc) return rc;
  if (!scores_out || !log_scale_out) return fail(EBTC_EINVAL, "NULL scores or log_scale output");
  BatchPlan bp = call_plan(b, o);
  rc = check_plan(b, bp);
  if (rc) return rc;
  Layout L = make_layout(b, o, bp);
  if (L.total > kScratchBytes) {
    bp = balanced_plan(b, o);
    L = make_layout(b, o, bp);
  }
  if (L.total > kScratchBytes)
    return fail(EBTC_EWORKSPACE, "the batch needs a workspace of " + std::to_string(L.total) +
                                     " bytes; the static scratch holds " + std::to_string(kScratchBytes) +
                                     " (use ebtc_scores with a caller workspace)");
  int sched = 0;
  rc = resolve_schedule(b, o, &sched);
  if (rc) return rc;
  void* ws = nullptr;
  rc = scratch_address(&ws);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  rc = prepare_kernels(bp);
  if (rc) return rc;
  char* w = (char*)ws;
  rc = upload_tables(b, w, L, bp, s);
  if (rc) return rc;
  // eager launches: instantiating a hipGraph would allocate
  if (sched == EBTC_SCHED_PLAIN)
    return enqueue_plain(b, o, w, L, bp, scores_out, log_scale_out, ckpt_out, diag_out, s);
  return enqueue_batched(b, o, w, L, bp, scores_out, log_scale_out, ckpt_out, diag_out, sched, s);
}

int ebtc_profile_phases(ebtc_batch* b, const ebtc_opts* o, void* ws, size_t ws_bytes, void* scores_out,
                        double* log_scale_out, double* phase_ms, int64_t* phase_launches, void* stream) {
  g_err.clear();
  if (!b || !phase_ms || !phase_launches) return fail(EBTC_EINVAL, "NULL batch or phase output");
  int rc = check_opts(o);
  if (rc) return rc;
  if (!ws || !scores_out || !log_scale_out) return fail(EBTC_EINVAL, "NULL workspace, scores or log_scale output");
  const BatchPlan bp = o->schedule == EBTC_SCHED_PLAIN ? spmv_plan(b, o) : call_plan(b, o);  // never the plain loop
  rc = check_plan(b, bp);
  if (rc) return rc;
  const Layout L = make_layout(b, o, bp);
  if (ws_bytes < L.total) return fail(EBTC_EWORKSPACE, "workspace too small");
  if (((uintptr_t)ws & 255) != 0) return fail(EBTC_EINVAL, "workspace must be 256-byte aligned");
  int sched = 0;
  rc = resolve_schedule(b, o, &sched);
  if (rc) return rc;
  if (sched == EBTC_SCHED_PLAIN) sched = EBTC_SCHED_BATCHED;  // phases are measured on a batched pass
  hipStream_t s = (hipStream_t)stream;
  rc = prepare_kernels(bp);
  if (rc) return rc;
  char* w = (char*)ws;
  rc = upload_tables(b, w, L, bp, s);
  if (rc) return rc;
  Prof prof;
  prof.s = s;
  rc = enqueue_batched(b, o, w, L, bp, scores_out, log_scale_out, nullptr, nullptr, sched, s, &prof);
  if (rc) return rc;
  EBTC_HIP(hipStreamSynchronize(s));
  for (int p = 0; p < EBTC_PHASE_COUNT; ++p) {
    phase_ms[p] = 0.0;
    phase_launches[p] = 0;
  }
  for (auto& r : prof.recs) {
    float ms = 0.f;
    EBTC_HIP(hipEventElapsedTime(&ms, r.a, r.b));
    phase_ms[r.phase] += ms;
    phase_launches[r.phase] += 1;
  }
  return EBTC_OK;
}

int ebtc_tune(ebtc_batch* b, const ebtc_opts* o, void* ws, size_t ws_bytes, int32_t* form_out, int32_t* lanes_out,
              int32_t* seglen_out, double* ms_out, void* stream) {
  g_err.clear();
  if (!b) return fail(EBTC_EINVAL, "NULL batch");
  int rc = check_opts(o);
  if (rc) return rc;
  if (!ws) return fail(EBTC_EINVAL, "NULL workspace");
  const BatchPlan base = one_form(b, spmv_form(b, EBTC_SPMV_STREAM, 0, 0, o->hub_threshold));
  const Layout L = make_layout(b, o, base);
  if (ws_bytes < L.total)
    return fail(EBTC_EWORKSPACE, "workspace of " + std::to_string(ws_bytes) + " bytes, need " + std::to_string(L.total));
  if (((uintptr_t)ws & 255) != 0) return fail(EBTC_EINVAL, "workspace must be 256-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  char* w = (char*)ws;
  const bool has_val = b->values != nullptr;
  const int steps = o->m > 0 ? o->m : o->m_max;
  // Steps that share a preparation: an adaptive run stops long before its cap (12 to 22 steps on the families here).
  // The cache's key holds them, and not the cap: calls of one key weigh the preparations alike.
  const int spread = o->m > 0 ? steps : std::min(steps, 16);
  rc = upload_tables(b, w, L, base, s);
  if (rc) return rc;
  // 1. each graph's bucket: its largest row (over its realizations) measured on the device, in the
  //    norm-partial arena, which the start kernel below overwrites
  std::vector<int32_t> row_max((size_t)b->R, 0);
  if (b->R > 0) {
    int32_t* dmax = (int32_t*)(w + L.off_npart);
    EBTC_LAUNCH(launch_row_max((const Task*)(w + L.off_tasks), b->row_ptr, b->R, dmax, s));
    EBTC_HIP(hipMemcpyAsync(row_max.data(), dmax, sizeof(int32_t) * (size_t)b->R, hipMemcpyDeviceToHost, s));
    EBTC_HIP(hipStreamSynchronize(s));
  }
  std::vector<std::string> gkey((size_t)b->G);
  {
    int64_t r = 0;
    for (int32_t g = 0; g < b->G; ++g) {
      int64_t z = 0;
      int32_t mx = 0;
      for (int32_t k = 0; k < b->nreal[g]; ++k, ++r) {
        z += b->nnz_r[r];
        mx = std::max(mx, row_max[r]);
      }
      gkey[g] = tune_key(b->dtype, has_val, b->n[g], (double)z / std::max<int64_t>(1, (int64_t)b->nreal[g] * b->n[g]),
                         mx, spread);
    }
  }
  // the batch's composition: its buckets, sorted and joined (the cache key of the batch's form)
  std::vector<std::string> keys = gkey;
  std::sort(keys.begin(), keys.end());
  keys.erase(std::unique(keys.begin(), keys.end()), keys.end());
  std::string bkey;
  for (const std::string& k : keys) bkey += (bkey.empty() ? "" : "+") + k;
  keys.assign(1, bkey);
  for (std::string& k : gkey) k = bkey;
  // 2. time the candidate forms on the whole batch (a composition already in the cache is not timed)
  LzArgs a0 = make_args(b, o, w, L);
  EBTC_LAUNCH(launch_blkmap(a0.tasks, b->R, (int32_t*)(w + L.off_blkmap), s));
  EBTC_LAUNCH(launch_start(b->dtype, a0, L.total_blocks, s));
  double ms[EBTC_TUNE_SLOTS];
  for (double& v : ms) v = -1.0;
  hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
  for (auto& e : ev) {
    if (hipEventCreate(&e) != hipSuccess) {
      for (auto& f : ev)
        if (f) (void)hipEventDestroy(f);
      return fail(EBTC_EHIP, "hipEventCreate failed");
    }
  }
  std::map<std::string, std::array<int32_t, 3>> choice;
  constexpr int kReps = 3;
  for (const std::string& key : keys) {
    {
      std::lock_guard<std::mutex> lock(g_tune_mu);
      auto it = g_tune_cache.find(key);
      if (it != g_tune_cache.end()) {
        choice[key] = it->second;
        continue;
      }
    }
    const Members* mp = nullptr;  // every graph
    struct Cand {
      SpmvPlan p;
      int slot;
    };
    std::vector<Cand> cands;
    cands.push_back({spmv_form(b, EBTC_SPMV_STREAM, 0, 0, o->hub_threshold, mp), 0});
    for (int i = 0; i < 4; ++i)
      cands.push_back({spmv_form(b, EBTC_SPMV_LANE_GROUPS, 4 << i, 0, o->hub_threshold, mp), 1 + i});
    int32_t nmax = 1;
    for (int32_t g = 0; g < b->G; ++g)
      if (member(mp, g)) nmax = std::max(nmax, b->n[g]);
    const int maxseg = staged_max_seglen(b->dtype);
    if ((nmax + maxseg - 1) / maxseg <= 8) cands.push_back({spmv_form(b, EBTC_SPMV_LDS_STAGED, 0, 0, 0, mp), 5});
    const int small_seg = seg_max_cols(b->dtype) / 2;
    for (int i = 0; i < 2; ++i) {
      const SpmvPlan p = spmv_form(b, EBTC_SPMV_SEGMENTED, 0, small_seg << i, 0, mp);
      if (p.smax <= kSegMax) cands.push_back({p, 6 + i});
    }
    cands.push_back({spmv_form(b, EBTC_SPMV_BALANCED, 0, 0, 0, mp), 8});
    {
      const SpmvPlan p = spmv_form(b, EBTC_SPMV_PANELED, 0, 0, 0, mp);
      if (check_form(b, p, mp) == EBTC_OK) cands.push_back({p, 9});
      g_err.clear();
    }
    // The paneled form (the last candidate) takes the place of the forms whose sums it computes bit for bit. The
    // lane-group and staged forms add a row's products in another order: a batch on which one of those is the
    // fastest of the others, by more than the 3% that two timings of one form differ by, stays on it, so that the
    // paneled form's choice changes no result (staged graphs of n = 1e4 to 2.5e4 could gain a third: 77 against
    // 56 us at 46 x n=21429, degree 25).
    int best = -1;
    double best_ms = 0.0, same_ms = INFINITY;
    for (size_t c = 0; c < cands.size() && rc == EBTC_OK; ++c) {
      const SpmvPlan& p = cands[c].p;
      const BatchPlan bp = one_form(b, p);
      if (check_plan(b, bp) != EBTC_OK) {
        g_err.clear();
        continue;
      }
      const Layout Lc = make_layout(b, o, bp);  // the forms' arenas follow the common ones
      if (Lc.total > ws_bytes) continue;
      rc = prepare_kernels(bp);
      if (rc) break;
      rc = upload_tables(b, w, Lc, bp, s);
      if (rc) break;
      const std::vector<FArgs> fa = form_args(b, a0, w, Lc, bp);
      const FArgs& x = fa[0];
      // [ev0, ev1): the once-per-call preparation; [ev2, ev3): kReps products after a warm-up. Step 0
      // reads only the start vector and the state k_start wrote, so every launch does the same work.
      hipError_t e = hipEventRecord(ev[0], s);
      if (e == hipSuccess && enqueue_prepare(b, x, 0, s, nullptr) != EBTC_OK) e = hipErrorLaunchFailure;
      if (e == hipSuccess) e = hipEventRecord(ev[1], s);
      if (e == hipSuccess) e = launch_spmv_step(b->dtype, has_val, p.lanes, 0, x.a, x.nb, s);
      if (e == hipSuccess) e = hipEventRecord(ev[2], s);
      for (int k = 0; k < kReps && e == hipSuccess; ++k) e = launch_spmv_step(b->dtype, has_val, p.lanes, 0, x.a, x.nb, s);
      if (e == hipSuccess) e = hipEventRecord(ev[3], s);
      if (e == hipSuccess) e = hipEventSynchronize(ev[3]);
      float t_prep = 0.f, t_spmv = 0.f;
      if (e == hipSuccess) e = hipEventElapsedTime(&t_prep, ev[0], ev[1]);
      if (e == hipSuccess) e = hipEventElapsedTime(&t_spmv, ev[2], ev[3]);
      if (e != hipSuccess) {
        rc = fail(EBTC_EHIP, std::string("tuning launch: ") + (g_err.empty() ? hipGetErrorString(e) : g_err));
        break;
      }
      const bool prepared = p.form == EBTC_SPMV_SEGMENTED || p.form == EBTC_SPMV_BALANCED || p.form == EBTC_SPMV_PANELED;
      const double t = t_spmv / kReps + (prepared ? t_prep / spread : 0.0);
      ms[cands[c].slot] = (ms[cands[c].slot] < 0 ? 0.0 : ms[cands[c].slot]) + t;
      const bool other_sums = p.form == EBTC_SPMV_LANE_GROUPS || p.form == EBTC_SPMV_LDS_STAGED;
      const bool stays = p.form == EBTC_SPMV_PANELED && best >= 0 && best_ms < same_ms / 1.03;
      if (!other_sums && p.form != EBTC_SPMV_PANELED) same_ms = std::min(same_ms, t);
      if (best < 0 || (t < best_ms && !stays)) {
        best = (int)c;
        best_ms = t;
      }
    }
    if (rc) break;
    if (best < 0) {
      rc = fail(EBTC_EHIP, "no SpMV form could be timed");
      break;
    }
    const SpmvPlan& p = cands[best].p;
    choice[key] = {p.form, p.lanes, p.param()};
    std::lock_guard<std::mutex> lock(g_tune_mu);
    g_tune_cache[key] = choice[key];
  }
  for (auto& e : ev) (void)hipEventDestroy(e);
  if (rc) return rc;
  // 3. the plan: one form per distinct choice, each graph on its bucket's
  std::vector<std::array<int32_t, 3>> forms;
  std::vector<int32_t> gform((size_t)b->G, 0);
  for (int32_t g = 0; g < b->G; ++g) {
    const std::array<int32_t, 3>& c = choice[gkey[g]];
    size_t f = 0;
    while (f < forms.size() && forms[f] != c) ++f;
    if (f == forms.size()) forms.push_back(c);
    gform[g] = (int32_t)f;
  }
  b->tuned = forms;
  b->tuned_graph = gform;
  if (form_out) *form_out = forms.size() == 1 ? forms[0][0] : EBTC_SPMV_AUTO;
  if (lanes_out) *lanes_out = forms.size() == 1 ? forms[0][1] : 0;
  if (seglen_out) *seglen_out = forms.size() == 1 ? forms[0][2] : 0;
  if (ms_out)
    for (int i = 0; i < EBTC_TUNE_SLOTS; ++i) ms_out[i] = ms[i];
  return EBTC_OK;
}

int ebtc_tuned_forms(ebtc_batch* b, int32_t* form_out, int32_t* lanes_out, int32_t* seglen_out) {
  g_err.clear();
  if (!b || !form_out) return fail(EBTC_EINVAL, "NULL batch or output");
  for (int32_t g = 0; g < b->G; ++g) {
    const bool t = !b->tuned.empty();
    const std::array<int32_t, 3> c = t ? b->tuned[b->tuned_graph[g]] : std::array<int32_t, 3>{0, 0, 0};
    form_out[g] = c[0];
    if (lanes_out) lanes_out[g] = c[1];
    if (seglen_out) seglen_out[g] = c[2];
  }
  return EBTC_OK;
}

int ebtc_set_forms(ebtc_batch* b, const int32_t* form, const int32_t* lanes, const int32_t* seg_len) {
  g_err.clear();
  if (!b || !form) return fail(EBTC_EINVAL, "NULL batch or form");
  std::vector<std::array<int32_t, 3>> forms;
  std::vector<int32_t> gform((size_t)b->G, 0);
  for (int32_t g = 0; g < b->G; ++g) {
    const int32_t l = lanes ? lanes[g] : 0, q = seg_len ? seg_len[g] : 0;
    if (form[g] < EBTC_SPMV_STREAM || form[g] > EBTC_SPMV_PANELED)
      return fail(EBTC_EINVAL, "graph " + std::to_string(g) + ": unknown spmv form");
    if (l != 0 && l != 4 && l != 8 && l != 16 && l != 32)
      return fail(EBTC_EINVAL, "graph " + std::to_string(g) + ": lanes must be 0, 4, 8, 16 or 32");
    if (q < 0) return fail(EBTC_EINVAL, "graph " + std::to_string(g) + ": seg_len must be >= 0");
    const std::array<int32_t, 3> c{form[g], form[g] == EBTC_SPMV_LANE_GROUPS ? l : 0, q};
    size_t f = 0;
    while (f < forms.size() && forms[f] != c) ++f;
    if (f == forms.size()) forms.push_back(c);
    gform[g] = (int32_t)f;
  }
  b->tuned = forms;
  b->tuned_graph = gform;
  return EBTC_OK;
}

int ebtc_tune_cache_get(char* buf, size_t cap, size_t* len) {
  g_err.clear();
  if (!len) return fail(EBTC_EINVAL, "NULL length output");
  std::string t;
  {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    for (const auto& kv : g_tune_cache)
      t += kv.first + " " + std::to_string(kv.second[0]) + " " + std::to_string(kv.second[1]) + " " +
           std::to_string(kv.second[2]) + "\n";
  }
  *len = t.size();
  if (buf == nullptr) return EBTC_OK;
  if (cap < t.size() + 1) return fail(EBTC_EINVAL, "buffer of " + std::to_string(cap) + " bytes, need " +
                                                       std::to_string(t.size() + 1));
  std::memcpy(buf, t.c_str(), t.size() + 1);
  return EBTC_OK;
}

int ebtc_tune_cache_put(const char* text) {
  g_err.clear();
  if (!text) return fail(EBTC_EINVAL, "NULL text");
  std::map<std::string, std::array<int32_t, 3>> add;
  const char* p = text;
  while (*p) {
    const char* e = std::strchr(p, '\n');
    const std::string line = e ? std::string(p, e) : std::string(p);
    p = e ? e + 1 : p + line.size();
    if (line.empty()) continue;
    std::istringstream in(line);
    std::string key, rest;
    int f = 0, l = 0, q = 0;
    if (!(in >> key >> f >> l >> q) || (in >> rest) || f < EBTC_SPMV_STREAM || f > EBTC_SPMV_PANELED ||
        (l != 0 && l != 4 && l != 8 && l != 16 && l != 32) || q < 0)
      return fail(EBTC_EINVAL, "bad tune-cache line: " + line);
    add[key] = {f, l, q};
  }
  std::lock_guard<std::mutex> lock(g_tune_mu);
  for (const auto& kv : add) g_tune_cache[kv.first] = kv.second;
  return EBTC_OK;
}

int ebtc_tune_cache_clear(void) {
  g_err.clear();
  std::lock_guard<std::mutex> lock(g_tune_mu);
  g_tune_cache.clear();
  return EBTC_OK;
}

int ebtc_plan_backward(ebtc_batch* b, const ebtc_opts* o, size_t* ws_bytes) {
  g_err.clear();
  if (!b || !ws_bytes) return fail(EBTC_EINVAL, "NULL batch or output");
  int rc = check_bwd_opts(o);
  if (rc) return rc;
  rc = check_plan(b, spmv_plan(b, o));
  if (rc) return rc;
  *ws_bytes = make_bwd_layout(b, o).total;
  return EBTC_OK;
}

int ebtc_scores_backward(ebtc_batch* b, const ebtc_opts* o, const double* log_scale, const void* grad_scores,
                         void* grad_values, void* ws, size_t ws_bytes, const double* ckpt, int32_t* ckpt_mismatch,
                         void* stream) {
  g_err.clear();
  if (!b) return fail(EBTC_EINVAL, "NULL batch");
  int rc = check_bwd_opts(o);
  if (rc) return rc;
  if (!log_scale || !grad_scores || !grad_values || !ws)
    return fail(EBTC_EINVAL, "NULL log_scale, grad_scores, grad_values or workspace");
  if (ckpt && !ckpt_mismatch) return fail(EBTC_EINVAL, "a checkpoint to compare needs ckpt_mismatch");
  const BatchPlan bp = spmv_plan(b, o);
  rc = check_plan(b, bp);
  if (rc) return rc;
  const BwdLayout B = make_bwd_layout(b, o);
  if (ws_bytes < B.total)
    return fail(EBTC_EWORKSPACE, "workspace of " + std::to_string(ws_bytes) + " bytes, need " + std::to_string(B.total));
  if (((uintptr_t)ws & 255) != 0) return fail(EBTC_EINVAL, "workspace must be 256-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  rc = prepare_kernels(bp);
  if (rc) return rc;
  char* w = (char*)ws;
  rc = upload_tables(b, w, B.fwd, bp, s);
  if (rc) return rc;
  // 1. forward recomputation (same kernels and order as ebtc_scores: bitwise the same basis)
  LzArgs fa = make_args(b, o, w, B.fwd);
  fa.unit_start = 1;
  const std::vector<FArgs> ffa = form_args(b, fa, w, B.fwd, bp);
  EBTC_LAUNCH(launch_blkmap(fa.tasks, b->R, (int32_t*)(w + B.fwd.off_blkmap), s));
  rc = enqueue_prepare_all(b, ffa, s, nullptr);  // the sorted entries serve both solves
  if (rc) return rc;
  rc = run_steps(b, o, fa, ffa, B.fwd.total_blocks, 0, b->R, s, nullptr);
  if (rc) return rc;
  const int steps = o->m > 0 ? o->m : o->m_max;
  EBTC_LAUNCH(launch_tridiag_state(fa, 0, b->R, 0, 0, steps, o->shift, o->tol, nullptr, nullptr, s));
  // the recomputation against the forward call's checkpoint: every reduction runs in a fixed order, so
  // any difference means the inputs or the options are not the forward's
  if (ckpt) EBTC_LAUNCH(launch_ckpt_check(fa.state, ckpt, b->R, ckpt_mismatch, s));
  // 2. adjoint Lanczos started at the cotangent (shares W and the partial-sum arenas)
  LzArgs aa = fa;
  aa.unit_start = 0;  // started at the cotangent
  aa.first_in_prepare = 0;
  aa.state = (RState*)(w + B.off_astate);
  aa.V = w + B.off_aV;
  const std::vector<FArgs> faa = form_args(b, aa, w, B.fwd, bp);
  EBTC_LAUNCH(launch_start_vec(b->dtype, aa, (const GraphInfo*)(w + B.fwd.off_graphs), grad_scores,
                               B.fwd.total_blocks, s));
  EBTC_LAUNCH(launch_start_norm(aa, b->R, s));
  rc = run_steps(b, o, aa, faa, B.fwd.total_blocks, 0, b->R, s, nullptr, false);
  if (rc) return rc;
  EBTC_LAUNCH(launch_tridiag_state(aa, 0, b->R, 0, 0, steps, 1, o->tol, nullptr, nullptr, s));
  // 3. block exponential, 4. node-major Z and V, 5. SDDMM on the pattern
  double* X = (double*)(w + B.off_X);
  EBTC_LAUNCH(launch_block_exp(fa.state, aa.state, fa.tasks, log_scale, X, b->R, s));
  EBTC_LAUNCH(launch_build_zv(b->dtype, fa, aa, X, w + B.off_Z, w + B.off_Vn, B.ld, B.fwd.total_blocks, s));
  EBTC_LAUNCH(launch_sddmm(b->dtype, B.ld, fa, w + B.off_Z, w + B.off_Vn, grad_values, B.fwd.total_blocks, s));
  return EBTC_OK;
}

// One graph, `count` Lanczos processes over its CSR (every task shares the graph's arrays).
namespace {
void shared_batch(ebtc_batch& b, int32_t dtype, int32_t n, const int32_t* row_ptr, const int32_t* col_idx,
                  const void* values, int32_t count) {
  b.dtype = dtype;
  b.G = 1;
  b.R = count;
  b.n = {n};
  b.nreal = {count};
  b.first = {0};
  b.rowptr_off.assign(count, 0);
  b.nnz_off.assign((size_t)count + 1, 0);
  b.nnz_r.assign((size_t)count, 0);  // the shared entries belong to no realization's arenas
  b.score_off = {0, n};
  b.row_ptr = row_ptr;
  b.col_idx = col_idx;
  b.values = values;
  b.total_scores = n;
  b.total_rows = (int64_t)n * count;
  b.n_max = n;
  b.graphs.resize(1);
  b.graphs[0] = GraphInfo{0, n, 0, count, 0};
}

int check_sc_args(int32_t dtype, int32_t n, int32_t count, int32_t m) {
  if (dtype != EBTC_F32 && dtype != EBTC_F64) return fail(EBTC_EINVAL, "dtype must be EBTC_F32 or EBTC_F64");
  if (n < 1) return fail(EBTC_EINVAL, "n must be >= 1");
  if (count < 1) return fail(EBTC_EINVAL, "count must be >= 1");
  if (m < 1 || m > EBTC_M_LIMIT) return fail(EBTC_EINVAL, "m must be in [1, " + std::to_string(EBTC_M_LIMIT) + "]");
  if ((int64_t)count * ((n + kRowsPerBlock - 1) / kRowsPerBlock) >= ((int64_t)1 << 31))
    return fail(EBTC_ENOTSUPPORTED, "too many row blocks for one launch");
  return EBTC_OK;
}

ebtc_opts sc_opts(int32_t m) {
  ebtc_opts o;
  ebtc_default_opts(&o);
  o.m = m;
  o.reorth = 1;
  o.schedule = EBTC_SCHED_BATCHED;
  o.use_hipgraph = 0;
  o.spmv = EBTC_SPMV_STREAM;
  return o;
}

// Workspace of the products formed together (k_shared.hip), after the layout's. None for one process, for small
// graphs (n=3000, degree 20, 64 processes: 0.64 ms process by process, 0.80 together) and where the packed vectors
// of 64 processes pass the 32 bits of an element's place.
constexpr int32_t kSharedNodes = 4096;
size_t shared_layout(int32_t dtype, int32_t n, int32_t count, size_t off, char* w, SharedMat* q) {
  const size_t node = shared_stride_bytes(dtype, std::min(count, 64));
  if (count < 2 || n < kSharedNodes || node * (size_t)n >= ((size_t)1 << 32) - 4096) return off;
  q->count = count;
  q->shares = shared_shares(dtype, n);
  auto take = [&](size_t bytes) {
    char* p = w + off;
    off += align_up(bytes);
    return p;
  };
  q->x = take(shared_stride_bytes(dtype, count) * (size_t)n);
  q->s = (double*)take(sizeof(double) * (size_t)count);
  q->cut = (int32_t*)take(sizeof(int32_t) * ((size_t)q->shares + 1));
  q->longs = (int32_t*)take(sizeof(int32_t) * (size_t)n);
  q->seen = (SharedSeen*)take(sizeof(SharedSeen));
  return off;
}

// Together or process by process, by the times per step, measured on gfx950. The stream form: its gathers, at the rate
// of a graph whose neighbours lie close together (500 G/s, FP64 470; a random graph's 185 and 205 are not known
// beforehand), and where there are long chains of adds, what its slowest group of rows, or all of them on the whole
// chip, take at 40 ns an entry of a chunk's longest row (n=300000 Barabasi-Albert, degree 24, two processes: 67236
// entries, 2.73 ms a step, together 0.24; one row of 1100 in a ring lattice of n=1e6, FP64: 0.16 ms, together 0.45).
// Together: packing the vectors, a wavefront load per entry (12 cycles of a compute unit, FP64 23, or its bytes at 7.2
// TB/s) and the launches, beside the long rows' chains (34 ns an entry, FP32 with values 41) or before the chain of the
// longest of the others, which a wavefront adds. Over 2400 calls on lattices, random and Barabasi-Albert graphs with 1
// to 200 rows of 600 to 20000 entries it chose the slower by more than 3% twice, by 8% at most. In dense matrices, where
// most rows are long, it is never taken.
// n=1e5, degree 20, FP32, random / ring lattice, together against one by one: 8 processes 1.50 / 2.38 and 1.50 / 1.31 ms,
// 16 processes 1.72 / 4.20 and 1.73 / 2.06.
bool shared_pays(int32_t dtype, bool has_val, int32_t n, int32_t count, const SharedSeen& g) {
  if (g.entries < 0 || g.entries > 0x7fffffff - 256) return false;  // the kernels look a few entries ahead
  if (g.rows > n / 16) return false;
  const bool f64 = dtype == EBTC_F64;
  const double es = f64 ? 8 : 4, bytes = (double)shared_stride_bytes(dtype, count), nnz = g.entries;
  const double wait = std::max(g.group * 40e-9, g.groups * 27e-12 * count);
  const double alone = nnz * count / (f64 ? 470e9 : 500e9) + std::max(0.0, wait - 5e-6);
  const double entry = std::max((f64 ? 38e-12 : 19.5e-12) * ((count + 63) / 64), bytes / 7.2e12);
  const double loads = (nnz - g.longs) * entry, add = has_val && !f64 ? 41e-9 : 34e-9;
  const double wave = has_val ? (f64 ? 35e-9 : 28e-9) : 18e-9;
  const double rows = g.rows > 0 ? std::max({std::max(loads, g.big * 40e-9) + 10e-6, g.row * add, g.longs * add * 1e-3 * count})
                                 : loads + std::max(10e-6, 5e-6 + g.row * wave);
  return alone > n * (count * es + bytes) / 2.6e12 + rows;
}
}  // namespace

int ebtc_subgraph_centrality_ws_bytes(int32_t dtype, int32_t n, int32_t count, int32_t m, size_t* ws_bytes) {
  g_err.clear();
  if (!ws_bytes) return fail(EBTC_EINVAL, "NULL output");
  int rc = check_sc_args(dtype, n, count, m);
  if (rc) return rc;
  ebtc_batch b;
  shared_batch(b, dtype, n, nullptr, nullptr, nullptr, count);
  const ebtc_opts o = sc_opts(m);
  SharedMat q{};
  *ws_bytes = shared_layout(dtype, n, count, make_layout(&b, &o, spmv_plan(&b, &o)).total, nullptr, &q);
  return EBTC_OK;
}

int ebtc_subgraph_centrality(int32_t dtype, int32_t n, const int32_t* row_ptr, const int32_t* col_idx,
                             const void* values, int32_t count, const int32_t* nodes, int32_t m, double* sc_out,
                             void* ws, size_t ws_bytes, void* stream) {
  g_err.clear();
  int rc = check_sc_args(dtype, n, count, m);
  if (rc) return rc;
  if (!row_ptr || !col_idx || !nodes || !sc_out || !ws)
    return fail(EBTC_EINVAL, "NULL row_ptr, col_idx, nodes, output or workspace");
  ebtc_batch b;
  shared_batch(b, dtype, n, row_ptr, col_idx, values, count);
  const ebtc_opts o = sc_opts(m);
  const BatchPlan bp = spmv_plan(&b, &o);
  const Layout L = make_layout(&b, &o, bp);
  SharedMat q{};
  const size_t need = shared_layout(dtype, n, count, L.total, (char*)ws, &q);
  if (ws_bytes < L.total)
    return fail(EBTC_EWORKSPACE, "workspace of " + std::to_string(ws_bytes) + " bytes, need " + std::to_string(need));
  if (ws_bytes < need) q.count = 0;  // room for the processes alone: one by one
  if (((uintptr_t)ws & 255) != 0) return fail(EBTC_EINVAL, "workspace must be 256-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  char* w = (char*)ws;
  // first, so that it runs beside the host's copies of the tables
  if (q.count) EBTC_LAUNCH(launch_shared_prepare(dtype, row_ptr, q, n, s));
  rc = upload_tables(&b, w, L, bp, s);
  if (rc) return rc;
  LzArgs a = make_args(&b, &o, w, L);
  const std::vector<FArgs> fa = form_args(&b, a, w, L, bp);
  SharedSeen seen{};
  if (q.count) {
    q.wstep = b.tasks[1].w_off - b.tasks[0].w_off;
    EBTC_HIP(hipMemcpyAsync(&seen, q.seen, sizeof(seen), hipMemcpyDeviceToHost, s));
  }
  // the task table lives on this call's stack: wait until the copy has read it
  EBTC_HIP(hipStreamSynchronize(s));
  if (q.count && !shared_pays(dtype, values != nullptr, n, count, seen)) q.count = 0;
  q.rows = seen.rows;
  EBTC_LAUNCH(launch_blkmap(a.tasks, b.R, (int32_t*)(w + L.off_blkmap), s));
  EBTC_LAUNCH(launch_start_unit(dtype, a, nodes, L.total_blocks, s));
  rc = run_steps(&b, &o, a, fa, L.total_blocks, 0, b.R, s, nullptr, false, q.count ? &q : nullptr);
  if (rc) return rc;
  EBTC_LAUNCH(launch_tridiag_state(a, 0, b.R, 0, 0, m, 1, 0.0, nullptr, nullptr, s));
  EBTC_LAUNCH(launch_sc_out(a.state, a.tasks, nodes, b.R, sc_out, s));
  return EBTC_OK;
}

int ebtc_topk_ws_bytes(ebtc_batch* b, size_t* ws_bytes) {
  g_err.clear();
  if (!b || !ws_bytes) return fail(EBTC_EINVAL, "NULL batch or output");
  *ws_bytes = align_up(sizeof(GraphInfo) * b->G) + align_up(sizeof(int32_t) * b->G) + align_up(sizeof(int64_t) * b->G);
  if (b->n_max >= kTopkMultiMin) {  // the chunked selection: chunk tables and its scratch
    const int64_t nchunks = topk_chunks(b);
    *ws_bytes += align_up(sizeof(int32_t) * (size_t)nchunks) + align_up(sizeof(int32_t) * ((size_t)b->G + 1)) +
                 topk_multi_scratch_bytes(b->G, nchunks);
  }
  return EBTC_OK;
}

int ebtc_topk(ebtc_batch* b, const void* scores, const int32_t* k_per_graph, int32_t* idx_out, void* val_out,
              void* ws, size_t ws_bytes, void* stream) {
  g_err.clear();
  if (!b || !scores || !k_per_graph || !idx_out || !ws) return fail(EBTC_EINVAL, "NULL argument");
  size_t need = 0;
  ebtc_topk_ws_bytes(b, &need);
  if (ws_bytes < need) return fail(EBTC_EWORKSPACE, "top-k workspace too small");
  if (((uintptr_t)ws & 255) != 0) return fail(EBTC_EINVAL, "workspace must be 256-byte aligned");
  // one copy of all the tables: the graphs, K and first output slot of each; for the chunked selection (chunks of
  // kTkChunk scores, graph by graph, a graph's chunks following its node ids) each chunk's graph and each graph's
  // first chunk
  const bool chunked = b->n_max >= kTopkMultiMin;
  const int64_t nchunks = chunked ? topk_chunks(b) : 0;
  const size_t o1 = align_up(sizeof(GraphInfo) * b->G), o2 = o1 + align_up(sizeof(int32_t) * b->G);
  const size_t o3 = o2 + align_up(sizeof(int64_t) * b->G);
  const size_t o4 = o3 + (chunked ? align_up(sizeof(int32_t) * (size_t)nchunks) : 0);
  const size_t o5 = o4 + (chunked ? align_up(sizeof(int32_t) * ((size_t)b->G + 1)) : 0);
  b->topk_tables.resize(o5);
  char* t = b->topk_tables.data();
  std::memcpy(t, b->graphs.data(), sizeof(GraphInfo) * b->G);
  std::memcpy(t + o1, k_per_graph, sizeof(int32_t) * b->G);
  int64_t off = 0;
  for (int32_t g = 0; g < b->G; ++g) {
    const int32_t k = k_per_graph[g];
    if (k < 0 || k > b->n[g] || k > EBTC_TOPK_LIMIT)
      return fail(k > EBTC_TOPK_LIMIT ? EBTC_ENOTSUPPORTED : EBTC_EINVAL,
                  "graph " + std::to_string(g) + ": K must be in [0, min(n, 4096)]");
    ((int64_t*)(t + o2))[g] = off;
    off += k;
  }
  if (chunked) {
    int32_t c = 0;
    for (int32_t g = 0; g < b->G; ++g) {
      ((int32_t*)(t + o4))[g] = c;
      const int32_t nc = (b->n[g] + kTkChunk - 1) / kTkChunk;
      for (int32_t i = 0; i < nc; ++i) ((int32_t*)(t + o3))[c++] = g;
    }
    ((int32_t*)(t + o4))[b->G] = c;
  }
  hipStream_t s = (hipStream_t)stream;
  char* w = (char*)ws;
  EBTC_HIP(hipMemcpyAsync(w, t, o5, hipMemcpyHostToDevice, s));
  if (!chunked) {  // one workgroup per graph
    EBTC_LAUNCH(launch_topk(b->dtype, (const GraphInfo*)w, b->G, (const int32_t*)(w + o1), (const int64_t*)(w + o2),
                            scores, idx_out, val_out, s));
    return EBTC_OK;
  }
  EBTC_LAUNCH(launch_topk_multi(b->dtype, (const GraphInfo*)w, b->G, (const int32_t*)(w + o1), (const int64_t*)(w + o2),
                                scores, idx_out, val_out, (const int32_t*)(w + o3), (const int32_t*)(w + o4), nchunks,
                                w + o5, s));
  return EBTC_OK;
}

int ebtc_spmv(int32_t dtype, int32_t n, const int32_t* row_ptr, const int32_t* col_idx, const void* values,
              const void* x, void* y, int32_t lanes_per_row, int32_t hub_threshold, int32_t seg_len, void* stream) {
  g_err.clear();
  if (dtype != EBTC_F32 && dtype != EBTC_F64) return fail(EBTC_EINVAL, "dtype must be EBTC_F32 or EBTC_F64");
  if (n < 1 || !row_ptr || !col_idx || !x || !y) return fail(EBTC_EINVAL, "n < 1 or NULL pointer");
  if (x == y) return fail(EBTC_EINVAL, "x and y must be distinct");
  const int lanes = lanes_per_row;
  if (lanes != 0 && lanes != 4 && lanes != 8 && lanes != 16 && lanes != 32)
    return fail(EBTC_EINVAL, "lanes_per_row must be 0, 4, 8, 16 or 32");
  if (hub_threshold < 0) return fail(EBTC_EINVAL, "hub_threshold must be >= 0");
  if (seg_len < -1) return fail(EBTC_EINVAL, "seg_len must be -1, 0 or > 0");
  const int hub = hub_threshold ? hub_threshold : 16 * (lanes ? lanes : 8);
  const int seg = seg_len > 0 ? std::min(seg_len, staged_max_seglen(dtype)) : 0;
  if (seg > 0) EBTC_HIP(prepare_staged_kernels());
  EBTC_LAUNCH(launch_spmv(dtype, values != nullptr, lanes, hub, seg, n, row_ptr, col_idx, values, x, y,
                          (hipStream_t)stream));
  return EBTC_OK;
}

int ebtc_tridiag_expv(int32_t count, int32_t k, const double* alpha, const double* beta, double* y_out,
                      double* theta_out, int32_t shift, void* stream) {
  g_err.clear();
  if (count < 0) return fail(EBTC_EINVAL, "count must be >= 0");
  if (k < 1 || k > EBTC_M_LIMIT) return fail(EBTC_EINVAL, "k must be in [1, " + std::to_string(EBTC_M_LIMIT) + "]");
  if (count == 0) return EBTC_OK;
  if (!alpha || !beta || !y_out || !theta_out) return fail(EBTC_EINVAL, "NULL pointer");
  EBTC_LAUNCH(launch_tridiag_arrays(count, k, alpha, beta, y_out, theta_out, shift, (hipStream_t)stream));
  return EBTC_OK;
}

int ebtc_validate_ws_bytes(ebtc_batch* b, size_t* ws_bytes) {
  g_err.clear();
  if (!b || !ws_bytes) return fail(EBTC_EINVAL, "NULL batch or output");
  *ws_bytes = align_up(sizeof(Task) * b->R) + align_up(sizeof(int64_t) * b->R) + align_up(sizeof(int32_t) * b->R);
  return EBTC_OK;
}

int ebtc_validate(ebtc_batch* b, void* ws, size_t ws_bytes, int64_t* first_bad, void* stream) {
  g_err.clear();
  if (!b || !ws || !first_bad) return fail(EBTC_EINVAL, "NULL argument");
  size_t need = 0;
  ebtc_validate_ws_bytes(b, &need);
  if (ws_bytes < need) return fail(EBTC_EWORKSPACE, "validate workspace too small");
  hipStream_t s = (hipStream_t)stream;
  Layout L;
  L.m_slots = 1;
  BatchPlan one;
  one.forms.resize(1);
  one.graph_form.assign((size_t)b->G, 0);
  fill_tables(b, L, one);
  char* w = (char*)ws;
  const size_t o1 = align_up(sizeof(Task) * b->R), o2 = o1 + align_up(sizeof(int64_t) * b->R);
  std::vector<int32_t> bad(b->R, 0);
  EBTC_HIP(hipMemcpyAsync(w, b->tasks.data(), sizeof(Task) * b->R, hipMemcpyHostToDevice, s));
  EBTC_HIP(hipMemcpyAsync(w + o1, b->nnz_r.data(), sizeof(int64_t) * b->R, hipMemcpyHostToDevice, s));
  EBTC_HIP(hipMemcpyAsync(w + o2, bad.data(), sizeof(int32_t) * b->R, hipMemcpyHostToDevice, s));
  EBTC_LAUNCH(launch_validate(b->row_ptr, b->col_idx, (const Task*)w, (const int64_t*)(w + o1), b->R, b->n_max,
                              (int32_t*)(w + o2), s));
  EBTC_HIP(hipMemcpyAsync(bad.data(), w + o2, sizeof(int32_t) * b->R, hipMemcpyDeviceToHost, s));
  EBTC_HIP(hipStreamSynchronize(s));
  *first_bad = -1;
  for (int64_t r = 0; r < b->R; ++r)
    if (bad[r]) {
      *first_bad = r;
      break;
    }
  return EBTC_OK;
}

}  // extern "C"
