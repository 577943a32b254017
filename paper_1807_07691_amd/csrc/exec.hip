// Query execution (paper Sec. 6.3 and Sec. 7.2): runs a plan's steps over
// device-resident binding tables.
//
// A binding table is columnar int32 (one array per bound variable).  Each
// step follows the preallocation scheme of Algorithm "Pre-allocating result
// matrix space": per input row, count the output rows (N_i); exclusive prefix
// sum (P_i, int64); allocate exactly P_n rows; write every input row's
// outputs at its offset.  Expansions write through a merge path over
// (row ends, output indices) so hub rows are split across workgroups; filters
// and star-centre intersections write through a stable ballot compaction.
// When a step's output exceeds the byte budget it is cut into output ranges,
// each carried through the remaining steps before the next one is produced
// (chunked expansion); the final table may therefore consist of segments.
#include <algorithm>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>

#include "batch.hpp"
#include "exec.hpp"
#include "host_area.hpp"
#include "small.hpp"

using namespace gsmat;

namespace {

template <class T>
struct Tmp {
  DeviceMem* mem;
  hipStream_t s;
  T* p = nullptr;
  size_t bytes = 0;
  Tmp(DeviceMem* m, int64_t n, hipStream_t st) : mem(m), s(st) {
    bytes = sizeof(T) * (size_t)std::max<int64_t>(n, 1);
    p = (T*)mem->alloc(bytes, s);
    if (!p) throw OomFail{bytes};
  }
  ~Tmp() {
    if (p) mem->free(p, bytes, s);
  }
  Tmp(const Tmp&) = delete;
  Tmp& operator=(const Tmp&) = delete;
};

// Per-thread pinned host area that kernels write small results into (sizes
// of the next step, lookups, fan-out samples); read after the stream syncs.
struct PinnedArea {
  int64_t total[8];
  LookupRes res[kMaxLookups];
  int64_t part[kMaxPats * kSampleBlocks];
  uint32_t word;  // report of the launches that fill the other fields
  uint32_t words[kMaxPats * kSampleBlocks];
  // a small join's query and report (host memory only)
  SmallReport small;
  SmallArgs query;
};

static_assert(offsetof(PinnedArea, small) <= kStageBytes, "staged results must fit the staging area");

// The calling thread's area; with `make` unset, null when it has none yet.
PinnedArea* pinned(bool make = true) {
  thread_local PinnedArea* a = nullptr;
  if (!a && make) {
    GS_HIP(hipHostMalloc((void**)&a, sizeof(PinnedArea), hipHostMallocDefault));
    std::memset(a, 0, sizeof(PinnedArea));
  }
  return a;
}

// Host memory of a batch's queries and reports (at most kSmallBatch of them),
// per thread.
struct QueryArea {
  char* p = nullptr;
  size_t bytes = 0;
  char* get(size_t want) {
    if (want <= bytes) return p;
    if (p) (void)hipHostFree(p);
    p = nullptr;
    bytes = 0;
    size_t b = 1 << 16;
    while (b < want) b <<= 1;
    GS_HIP(hipHostMalloc((void**)&p, b, hipHostMallocDefault));
    bytes = b;
    return p;
  }
  ~QueryArea() {
    if (p) (void)hipHostFree(p);
  }
};
QueryArea& query_area() {
  thread_local QueryArea a;
  return a;
}

uint32_t all_of(const gsmat_query_plan* pl) {
  return pl->pats.size() >= 32 ? 0xFFFFFFFFu : ((1u << pl->pats.size()) - 1);
}

SmallStore small_store(const gsmat_store* st) {
  return SmallStore{st->out.d_desc, st->in.d_desc, st->out.ptrs(), st->in.ptrs(), st->out.src};
}

struct Exec {
  gsmat_store* st;
  const gsmat_query_plan* pl;
  hipStream_t s;
  int64_t budget;
  int64_t max_rows;
  gsmat_result* res;
  bool adaptive;

  // table allocations not yet released or handed to the result
  std::vector<std::pair<void*, size_t>> live;

  // Device memory of the tables and step scratch (null: the store's), and
  // where kernels leave small results for the host: null means pinned host
  // memory; otherwise this device area, copied to the host after the stream
  // synchronises (the allocation-free entry point uses both).
  DeviceMem* dm = nullptr;
  PinnedArea* dev_area = nullptr;
  // set: final tables are appended here rather than added to res
  std::vector<Table>* collect = nullptr;

  bool small = true;     // tables of few rows run in one launch (small.hip)
  size_t* small_bytes = nullptr;  // set: what those launches' areas took in all
  bool settled = true;   // everything launched so far has been waited for

  DeviceMem* mem() { return dm ? dm : st->mem.get(); }

  // Copies `bytes` of the device area at `p` to host memory at `h` (staged
  // small results) and waits for the stream.
  void stage_back(void* h, const void* p, size_t bytes) {
    GS_HIP(hipMemcpyAsync(h, p, bytes, hipMemcpyDeviceToHost, s));
    host_sync(s);
  }

  // Scans the tile sums in place and returns the grand total.
  int64_t scan_total(int64_t* ts, int64_t nt, hipStream_t st_) {
    if (dev_area) {
      launch_scan_tile_sums(ts, nt, ts + nt, st_, nullptr);
      int64_t v = 0;
      stage_back(&v, ts + nt, sizeof(v));
      return v;
    }
    PinnedArea* h = pinned();
    const uint32_t report = next_report();
    launch_scan_tile_sums(ts, nt, ts + nt, st_, &h->total[0], &h->word, report);
    host_wait_words(&h->word, 1, report, st_);
    return h->total[0];
  }

  void forget(void* p) {
    for (size_t i = 0; i < live.size(); ++i)
      if (live[i].first == p) {
        live[i] = live.back();
        live.pop_back();
        return;
      }
  }

  void release(Table& t) {
    if (t.owned) {
      forget(t.owned);
      mem()->free(t.owned, t.owned_bytes, s);
    }
    t.owned = nullptr;
    t.keep.reset();
  }

  // frees every table still alive (error paths)
  void release_all() {
    for (auto& a : live) mem()->free(a.first, a.second, s);
    live.clear();
  }

  // Allocates a table of n rows for the given variables (columns in order).
  // Columns start on 256-byte boundaries (stride rounded up to 64 values) so
  // that a wave's 64 stores of one column cover whole cache lines.
  Table alloc_table(int64_t n, const int* vars, int k) {
    Table t;
    t.n = n;
    t.k = k;
    const int64_t stride = col_stride(n);
    const size_t bytes = sizeof(int32_t) * (size_t)stride * (size_t)std::max(k, 1);
    if (k > 0) {
      t.owned = mem()->alloc(bytes, s);
      if (!t.owned) throw OomFail{bytes};
      t.owned_bytes = bytes;
      live.push_back({t.owned, bytes});
    }
    for (int c = 0; c < k; ++c) {
      t.var[c] = vars[c];
      t.col[c] = (int32_t*)t.owned + (size_t)c * (size_t)stride;
    }
    return t;
  }

  // Lookup of pattern tp's constant endpoint(s): the plan's, when it was
  // planned on this store, else one device lookup.
  LookupRes lookup_tp(int tp, int orient, int32_t p, int32_t v, int32_t member) {
    if (pl->lk_store == st->uid && tp < (int)pl->lk.size() && pl->lk[tp].valid) {
      const gsmat_pat_lookup& l = pl->lk[tp];
      return LookupRes{l.start, l.len, l.found, 0};
    }
    return lookup(orient, p, v, member);
  }

  LookupRes lookup(int orient, int32_t p, int32_t v, int32_t member) {
    LookupBatch b{};
    b.req[0] = LookupReq{orient, p, v, member};
    b.n = 1;
    if (dev_area) {
      launch_lookup(b, st->out.d_desc, st->in.d_desc, st->out.ptrs(), st->in.ptrs(),
                    dev_area->res, s);
      LookupRes r;
      stage_back(&r, dev_area->res, sizeof(r));
      return r;
    }
    PinnedArea* h = pinned();
    const uint32_t report = next_report();
    launch_lookup(b, st->out.d_desc, st->in.d_desc, st->out.ptrs(), st->in.ptrs(), h->res, s,
                  &h->word, report);
    host_wait_words(&h->word, 1, report, s);
    return h->res[0];
  }

  void emit(Table& t) {
    if (collect) {
      if (t.owned) forget(t.owned);
      collect->push_back(t);
      t.owned = nullptr;
      return;
    }
    const int nv = pl->n_vars;
    Segment seg;
    seg.rows = t.n;
    for (int v = 0; v < nv; ++v) {
      const int c = t.col_of(v);
      if (c < 0) throw StatusFail{GSMAT_EHIP, "internal: unbound variable at the end of the plan"};
      seg.col[v] = t.col[c];
    }
    seg.owned = t.owned;
    seg.owned_bytes = t.owned_bytes;
    seg.keep = t.keep;
    if (t.owned) forget(t.owned);
    t.owned = nullptr;
    res->rows += seg.rows;
    res->segs.push_back(seg);
    if (max_rows >= 0 && res->rows > max_rows)
      throw StatusFail{GSMAT_ETOOBIG, "result exceeds max_rows (" + std::to_string(max_rows) + ")"};
  }

  int64_t chunk_rows(int width) {
    if (budget <= 0) return INT64_MAX;
    const int64_t r = budget / (4 * (int64_t)std::max(width, 1));
    if (r < 1) throw StatusFail{GSMAT_ENOMEM, "budget_bytes cannot hold one output row"};
    return r;
  }

  // The relation of one TP on its own (views into the store where possible).
  Table tp_relation(int tp) {
    const gsmat_pattern& q = pl->pats[tp];
    const int32_t p = q.p;
    Table t;
    if (is_var(q.s) && is_var(q.o)) {
      const PredView pv = st->out.view(p);
      if (q.s != q.o) {
        t.n = pv.nnz;
        t.k = 2;
        t.col[0] = pv.src;
        t.var[0] = var_of(q.s);
        t.col[1] = pv.nbr;
        t.var[1] = var_of(q.o);
        return t;
      }
      // (?x p ?x): the diagonal
      settled = false;
      const int64_t n = pv.nnz;
      const int64_t nt = ceil_div(std::max<int64_t>(n, 1), kTile);
      Tmp<uint8_t> flags(mem(), n, s);
      Tmp<int64_t> ts(mem(), nt + 1, s);
      if (n > 0) launch_flag_diag(pv.src, pv.nbr, n, flags.p, ts.p, s);
      const int64_t m = n > 0 ? scan_total(ts.p, nt, s) : 0;
      int v = var_of(q.s);
      Table o = alloc_table(m, &v, 1);
      if (m > 0) {
        ColSet in{};
        in.c[0] = pv.src;
        OutSet out{};
        out.c[0] = const_cast<int32_t*>(o.col[0]);
        launch_compact_cols(in, 1, flags.p, n, ts.p, out, s);
      }
      return o;
    }
    if (!is_var(q.s) && is_var(q.o)) {
      const LookupRes r = lookup_tp(tp, 0, p, q.s, -1);
      const PredView pv = st->out.view(p);
      t.n = r.len;
      t.k = 1;
      t.col[0] = pv.nbr + r.start;
      t.var[0] = var_of(q.o);
      return t;
    }
    if (is_var(q.s) && !is_var(q.o)) {
      const LookupRes r = lookup_tp(tp, 1, p, q.o, -1);
      const PredView pv = st->in.view(p);
      t.n = r.len;
      t.k = 1;
      t.col[0] = pv.nbr + r.start;
      t.var[0] = var_of(q.s);
      return t;
    }
    const LookupRes r = lookup_tp(tp, 0, p, q.s, q.o);
    t.n = r.found ? 1 : 0;
    t.k = 0;
    return t;
  }

  uint32_t completes(const gsmat_step_info& sp) const { return step_completes(pl, sp); }

  // Adaptive choice of the next step on the bound table t (fan-out samples
  // of the candidate expansions are taken on the device).
  gsmat_step_info choose(const Table& t, uint32_t rem) {
    StepChoice c;
    step_candidates(st, pl, t, rem, c);
    if (c.has_filter) return c.filter;
    if (c.nc == 0) return c.cartesian;
    if (c.nc == 1) return step_pick(pl, c, nullptr);
    SampleSet ss{};
    for (int i = 0; i < c.nc; ++i) candidate_view(st, pl, t, c, i, &ss.col[i], &ss.pv[i]);
    ss.n = t.n;
    ss.ncand = c.nc;
    int64_t part[kMaxPats * kSampleBlocks];
    if (dev_area) {
      launch_sample_fanout(ss, dev_area->part, s);
      stage_back(part, dev_area->part, sizeof(int64_t) * c.nc * kSampleBlocks);
    } else {
      PinnedArea* h = pinned();
      const uint32_t report = next_report();
      launch_sample_fanout(ss, h->part, s, h->words, report);
      host_wait_words(h->words, c.nc * kSampleBlocks, report, s);
      std::copy(h->part, h->part + c.nc * kSampleBlocks, part);
    }
    int64_t sum[kMaxPats];
    for (int i = 0; i < c.nc; ++i) {
      sum[i] = 0;
      for (int b = 0; b < kSampleBlocks; ++b) sum[i] += part[i * kSampleBlocks + b];
    }
    return step_pick(pl, c, sum);
  }

  void run(int si, Table& t, uint32_t rem) {
    if (t.n == 0) {
      release(t);
      return;
    }
    if (rem == 0) {
      emit(t);
      return;
    }
    if (small && small_fits(si, t, rem) && run_small(si, t, rem)) return;
    const gsmat_step_info sp =
        (adaptive && !t.unit()) ? choose(t, rem) : pl->steps[std::min<size_t>(si, pl->steps.size() - 1)];
    const uint32_t next = rem & ~completes(sp);
    if (si < res->n_steps) res->step_in[si] += t.n;
    // a scan alone is a view: nothing is launched
    if (!t.unit() || sp.kind == GSMAT_STEP_INTERSECT) settled = false;
    switch (sp.kind) {
      case GSMAT_STEP_SCAN:
      case GSMAT_STEP_CARTESIAN: {
        Table r = tp_relation(sp.tp);
        combine(si, t, r, next);
        break;
      }
      case GSMAT_STEP_INTERSECT: {
        Table r = intersect(sp);
        combine(si, t, r, next);
        break;
      }
      case GSMAT_STEP_FILTER:
        filter(si, sp, t, next);
        break;
      case GSMAT_STEP_EXPAND:
        expand(si, sp, t, next);
        break;
      default:
        throw StatusFail{GSMAT_EINVAL, "unknown step kind"};
    }
  }

  // Whether the steps from si on are tried in one launch: the table has at
  // most kSmallRows rows, and the next step is one the launch takes.  A first
  // step must not list more rows, and one that the host answers from the plan's
  // lookups needs no launch: a scan of known length is a view, a constant
  // pattern known to hold or not to hold decides by itself (5 us against 15).
  // From a bound table some pattern left must be connected to it: a Cartesian
  // product only hands the table back (two constants' rows: 19 us against 34).
  // A table of so few rows costs the
  // general path 25 us to 60 us a step whatever its size; the launch takes 14 us
  // for one or two steps and 23 us for four.  Sixteen queries, planned, joined
  // and fetched, on 20 million triples, with the fetch in reported packs: 4.6 -> 1.4
  // ms (3 to 5 patterns, 300 to 30 000 rows), 1.65 -> 0.6 ms (1 or 2 patterns, up to
  // 100 rows).
  bool small_fits(int si, const Table& t, uint32_t rem) const {
    if (t.n > kSmallRows) return false;
    const gsmat_step_info& sp = pl->steps[std::min<size_t>(si, pl->steps.size() - 1)];
    if (!t.unit()) {
      if (!adaptive) return sp.kind == GSMAT_STEP_EXPAND || sp.kind == GSMAT_STEP_FILTER;
      for (int tp = 0; tp < (int)pl->pats.size(); ++tp) {
        const gsmat_pattern& q = pl->pats[tp];
        if (!(rem >> tp & 1)) continue;
        if (is_var(q.s) ? t.col_of(var_of(q.s)) >= 0 : !is_var(q.o)) return true;
        if (is_var(q.o) && t.col_of(var_of(q.o)) >= 0) return true;
      }
      return false;
    }
    const bool known = pl->lk_store == st->uid && pl->lk.size() == pl->pats.size();
    if (sp.kind == GSMAT_STEP_FILTER) return !(known && pl->lk[sp.tp].valid);
    if (sp.kind == GSMAT_STEP_SCAN || sp.kind == GSMAT_STEP_CARTESIAN) {
      const gsmat_pattern& q = pl->pats[sp.tp];
      return !known && (!is_var(q.s) || !is_var(q.o));
    }
    if (sp.kind != GSMAT_STEP_INTERSECT) return false;
    const int32_t cterm = -(sp.var + 1);
    for (int tp = 0; tp < (int)pl->pats.size(); ++tp) {
      if (!(sp.members >> tp & 1)) continue;
      const gsmat_pattern& q = pl->pats[tp];
      int64_t len;
      if (q.s == cterm && is_var(q.o)) len = st->out.desc[q.p].nr;
      else if (q.o == cterm && is_var(q.s)) len = st->in.desc[q.p].nr;
      else if (known && pl->lk[tp].valid) len = pl->lk[tp].len;
      else return true;
      if (len <= kSmallRows) return true;
    }
    return false;
  }

  // Whether the query's answer is a relation of the store, or nothing, as far as
  // is known without a launch.
  bool is_view() const {
    if (pl->pats.size() != 1) return false;
    const gsmat_pattern& q = pl->pats[0];
    if (is_var(q.s) && is_var(q.o)) return q.s != q.o;
    return pl->lk_store == st->uid && pl->lk.size() == 1 && pl->lk[0].valid;
  }

  // Whether a batch tries the whole query in one launch: its first relation
  // has at most kSmallRows rows, as far as is known without a lookup.
  bool small_first() const {
    Table unit;
    unit.n = 1;
    if (small_fits(0, unit, all_of(pl))) return true;
    const gsmat_step_info& sp = pl->steps[0];
    if (sp.kind != GSMAT_STEP_SCAN) return false;
    const gsmat_pattern& q = pl->pats[sp.tp];
    if (is_var(q.s) && is_var(q.o)) return q.s != q.o && st->out.desc[q.p].nnz <= kSmallRows;
    return pl->lk[sp.tp].valid && pl->lk[sp.tp].len <= kSmallRows;
  }

  // Memory of a small join: one query's own blocks, or parts of what a batch
  // holds (`hold` set: nothing is freed here).
  struct SmallMem {
    void* work = nullptr;
    size_t work_bytes = 0;
    void* fin[kSmallFins] = {};
    std::shared_ptr<Arena> work_hold, fin_hold;
  };

  int final_cols(const Table& t) const {
    return std::min<int>(t.k + (int)pl->pats.size(), kMaxCols);
  }

  void fill_small(SmallArgs& a, int si, const Table& t, uint32_t rem, const SmallLayout& l,
                  const SmallMem& sm) const {
    a.np = (int32_t)pl->pats.size();
    a.nsteps = (int32_t)pl->steps.size();
    a.adaptive = adaptive;
    a.k = t.k;
    a.si = si;
    a.rem = rem;
    a.n = t.n;
    a.budget = budget;
    a.work = (char*)sm.work;
    a.tab = l.tab;
    a.starts = l.starts;
    a.lens = l.lens;
    a.offs = l.offs;
    for (int f = 0; f < kSmallFins; ++f) a.fin[f] = (char*)sm.fin[f];
    a.lk_valid = 0;
    const bool known = pl->lk_store == st->uid && pl->lk.size() == pl->pats.size();
    for (int i = 0; i < a.np; ++i) {
      const gsmat_pattern& q = pl->pats[i];
      a.pats[i] = SmallPat{q.s, q.p, q.o};
      a.lk[i] = LookupRes{0, 0, 0, 0};
      if (known && pl->lk[i].valid) {
        a.lk[i] = LookupRes{pl->lk[i].start, pl->lk[i].len, pl->lk[i].found, 0};
        a.lk_valid |= 1u << i;
      }
    }
    for (int i = 0; i < a.nsteps; ++i) {
      const gsmat_step_info& sp = pl->steps[i];
      a.steps[i] = SmallStep{(int8_t)sp.kind, (int8_t)sp.tp, (int8_t)sp.orient, (int8_t)sp.var,
                             sp.members};
    }
    for (int c = 0; c < t.k; ++c) {
      a.col[c] = t.col[c];
      a.var[c] = (int8_t)t.var[c];
    }
  }

  // Takes the table t through the steps from si on in one launch.  True: the
  // query is finished (its answer, if any, emitted); false: the general path
  // goes on from si, t and rem, which now tell how far the launch came.
  bool run_small(int& si, Table& t, uint32_t& rem) {
    // the calling thread's area exists once it has planned a query
    PinnedArea* h = pinned(!dev_area);
    if (!h) return false;
    const SmallLayout l((int)pl->pats.size(), final_cols(t));
    SmallMem sm;
    sm.work_bytes = (size_t)l.bytes;
    sm.work = mem()->alloc(sm.work_bytes, s);
    if (!sm.work) return false;  // the general path may need less
    live.push_back({sm.work, sm.work_bytes});
    size_t fins = 0;
    for (int f = 0; f < kSmallFins; ++f) {
      if (dm && kFinBytes[f] < kSmallFin) continue;  // nothing is kept there
      sm.fin[f] = mem()->alloc(kFinBytes[f], s);
      if (!sm.fin[f]) {
        drop_fins(sm);
        drop(sm.work, sm.work_bytes);
        return false;
      }
      live.push_back({sm.fin[f], (size_t)kFinBytes[f]});
      fins += kFinBytes[f];
    }
    if (small_bytes) *small_bytes += sm.work_bytes + fins;
    fill_small(h->query, si, t, rem, l, sm);
    const uint32_t seq = next_report();
    launch_small(small_store(st), &h->query, &h->small, 1, seq, s);
    host_wait_words(&h->small.seq, 1, seq, s);
    settled = true;
    const SmallReport r = h->small;  // the area is used again by the steps below
    return finish_small(r, (int64_t*)((char*)sm.work + l.offs), sm, si, t, rem);
  }

  // idle: all work on the block has been waited for
  void drop(void* p, size_t bytes, bool idle = false) {
    forget(p);
    if (idle) mem()->free_idle(p, bytes, s);
    else mem()->free(p, bytes, s);
  }
  void drop_fins(const SmallMem& sm, int but = -1) {
    for (int f = 0; f < kSmallFins; ++f)
      if (f != but && sm.fin[f]) drop(sm.fin[f], kFinBytes[f], true);
  }

  // What a small join leaves to be written, the expansion it counted or an
  // answer to be moved out of its work area: rows and columns.
  static bool counted(const SmallReport& r) { return r.status == kSmallWrite; }
  static int64_t out_rows(const SmallReport& r) { return counted(r) ? r.m : r.n; }
  static int out_cols(const SmallReport& r) { return counted(r) ? r.k + 1 : r.k; }
  static int64_t out_bytes(const SmallReport& r) {
    return 4 * col_stride(out_rows(r)) * out_cols(r);
  }
  // Its task, and its table o, whose columns are at `to`.
  void prepare_write(const SmallReport& r, const int64_t* offs, int32_t* to, SmallWriteTask& w,
                     Table& o) {
    o.n = out_rows(r);
    o.k = out_cols(r);
    for (int c = 0; c < r.k; ++c) o.var[c] = r.var[c];
    w.offs = nullptr;
    if (counted(r)) {
      const gsmat_pattern& q = pl->pats[r.tp];
      o.from = r.n;
      o.var[r.k] = r.orient == 0 ? var_of(q.o) : var_of(q.s);
      w.offs = offs;
      w.start = r.start;
      w.nbr = r.orient == 0 ? st->out.view(q.p).nbr : st->in.view(q.p).nbr;
    }
    w.out = to;
    w.m = o.n;
    w.stride = col_stride(o.n);
    w.n = (int32_t)r.n;
    w.k = r.k;
    for (int c = 0; c < r.k; ++c) w.col[c] = r.col[c];
    for (int c = 0; c < o.k; ++c) o.col[c] = to + c * w.stride;
  }
  static double write_bytes(const SmallReport& r) {
    if (!counted(r)) return 8.0 * (double)r.n * r.k;
    return 4.0 * (double)r.m * (r.k + 2) + (double)r.n * (4.0 * r.k + 12.0);
  }
  // The same written at once, into memory of its own.
  Table write_own(const SmallReport& r, const int64_t* offs) {
    Table o = alloc_table(out_rows(r), r.var, out_cols(r));
    SmallWriteTask w;
    prepare_write(r, offs, (int32_t*)o.owned, w, o);
    launch_small_write(&w, 1, o.n, write_bytes(r), s);
    return o;
  }
  // Whether the write is one piece within the step budget.
  bool one_piece(const SmallReport& r) const {
    return budget <= 0 || r.m <= budget / (4 * (int64_t)(r.k + 1));
  }

  // Takes over what a small join reports (as run_small); written: the table
  // of its counted expansion or of its answer, where that has been written.
  bool finish_small(const SmallReport& r, const int64_t* offs, const SmallMem& sm, int& si,
                    Table& t, uint32_t& rem, Table* written = nullptr) {
    for (int i = 0; i < res->n_steps && i <= kMaxPats; ++i) {
      res->step_in[i] += r.step_in[i];
      res->step_out[i] += r.step_out[i];
    }
    const bool done = r.status == kSmallDone;
    const bool own = !sm.work_hold;
    Table o;
    o.n = r.n;
    o.k = r.k;
    for (int c = 0; c < o.k; ++c) {
      o.col[c] = r.col[c];
      o.var[c] = r.var[c];
    }
    si = r.si;
    rem = r.rem;
    bool keep_work = false;
    const int fin = r.n > 0 && r.place >= kAtFin ? r.place - kAtFin : -1;
    if (o.n == 0) {
    } else if (r.place == kAtWork && done) {
      // the answer leaves the work area for memory of its own size
      o = written ? *written : write_own(r, offs);
      settled = false;
    } else if (r.place == kAtWork) {
      keep_work = true;
      o.keep = sm.work_hold;
      if (own) {
        o.owned = sm.work;
        o.owned_bytes = sm.work_bytes;
      }
    } else if (fin >= 0) {
      o.keep = sm.fin_hold;
      o.owned_bytes = kFinBytes[fin];
      if (own) o.owned = sm.fin[fin];
    } else {  // t's own columns, or views into the store
      o.owned = t.owned;
      o.owned_bytes = t.owned_bytes;
      o.keep = t.keep;
      t.owned = nullptr;
    }
    if (own) drop_fins(sm, fin);
    if (own && !keep_work && !counted(r))
      drop(sm.work, sm.work_bytes, !done || r.place != kAtWork || r.n == 0);
    release(t);
    t = o;
    if (counted(r)) {
      // the step is counted: its outputs are written as any expansion's
      settled = false;
      if (si < res->n_steps) res->step_in[si] += t.n;
      add_out(si, r.m);
      const uint32_t next = rem & ~(1u << r.tp);
      if (written || one_piece(r)) {
        Table x = written ? *written : write_own(r, offs);
        run(si + 1, x, next);
        release(t);
      } else {
        expand_write(si, r.tp, r.orient, t, next, offs, r.start, r.m);
      }
      if (own && !keep_work) drop(sm.work, sm.work_bytes);
      return true;
    }
    if (!done) return false;
    if (t.n > 0) emit(t);
    return true;
  }

  void add_out(int si, int64_t m) {
    if (si < res->n_steps) res->step_out[si] += m;
  }

  // t x r: r alone when t is the unit table, else the Cartesian product.
  void combine(int si, Table& t, Table& r, uint32_t next) {
    if (t.unit()) {
      add_out(si, r.n);
      release(t);
      run(si + 1, r, next);
      return;
    }
    if (r.n == 0) {
      release(t);
      release(r);
      return;
    }
    if (t.k + r.k > kMaxCols) throw StatusFail{GSMAT_EUNSUPPORTED, "too many columns"};
    if (r.n > 0 && t.n > INT64_MAX / r.n) throw StatusFail{GSMAT_ETOOBIG, "Cartesian product overflows"};
    const int64_t m = t.n * r.n;
    add_out(si, m);
    int vars[kMaxCols];
    for (int c = 0; c < t.k; ++c) vars[c] = t.var[c];
    for (int c = 0; c < r.k; ++c) vars[t.k + c] = r.var[c];
    const int k = t.k + r.k;
    const int64_t rpc = chunk_rows(k);
    ColSet a{}, b{};
    for (int c = 0; c < t.k; ++c) a.c[c] = t.col[c];
    for (int c = 0; c < r.k; ++c) b.c[c] = r.col[c];
    for (int64_t J0 = 0; J0 < m; J0 += rpc) {
      const int64_t J1 = std::min(m, J0 + rpc);
      Table o = alloc_table(J1 - J0, vars, k);
      OutSet out{};
      for (int c = 0; c < k; ++c) out.c[c] = const_cast<int32_t*>(o.col[c]);
      if (k > 0) launch_cartesian(a, t.k, t.n, b, r.k, r.n, J0, J1, out, s);
      run(si + 1, o, next);
    }
    release(t);
    release(r);
  }

  Table intersect(const gsmat_step_info& sp) {
    const int32_t cterm = -(sp.var + 1);
    struct L {
      ListRef ref;
      const int32_t* ids;  // the list as an array (row ids or segment)
    };
    std::vector<L> lists;
    for (int tp = 0; tp < (int)pl->pats.size(); ++tp) {
      if (!(sp.members >> tp & 1)) continue;
      const gsmat_pattern& q = pl->pats[tp];
      L l{};
      if (q.s == cterm && is_var(q.o)) {
        l.ref.pv = st->out.view(q.p);
        l.ref.is_keys = 1;
        l.ref.len = l.ref.pv.nr;
        l.ids = l.ref.pv.keys;
      } else if (q.o == cterm && is_var(q.s)) {
        l.ref.pv = st->in.view(q.p);
        l.ref.is_keys = 1;
        l.ref.len = l.ref.pv.nr;
        l.ids = l.ref.pv.keys;
      } else if (q.s == cterm) {  // (v p c): v among the subjects of object c
        const LookupRes r = lookup_tp(tp, 1, q.p, q.o, -1);
        l.ref.seg = st->in.view(q.p).nbr + r.start;
        l.ref.bm = st->in.row_bitmap(q.p, q.o);
        l.ref.len = r.len;
        l.ids = l.ref.seg;
      } else {  // (c p v): v among the objects of subject c
        const LookupRes r = lookup_tp(tp, 0, q.p, q.s, -1);
        l.ref.seg = st->out.view(q.p).nbr + r.start;
        l.ref.bm = st->out.row_bitmap(q.p, q.s);
        l.ref.len = r.len;
        l.ids = l.ref.seg;
      }
      lists.push_back(l);
    }
    Table t;
    t.k = 1;
    t.var[0] = sp.var;
    size_t d = 0;
    for (size_t i = 1; i < lists.size(); ++i)
      if (lists[i].ref.len < lists[d].ref.len) d = i;
    const int64_t n = lists[d].ref.len;
    if (n == 0) {
      t.n = 0;
      return t;
    }
    ListSet ls{};
    for (size_t i = 0; i < lists.size(); ++i)
      if (i != d) ls.l[ls.n++] = lists[i].ref;
    const int64_t nt = ceil_div(n, kTile);
    Tmp<uint8_t> flags(mem(), n, s);
    Tmp<int64_t> ts(mem(), nt + 1, s);
    launch_flag_intersect(lists[d].ids, n, ls, flags.p, ts.p, s);
    const int64_t m = scan_total(ts.p, nt, s);
    if (m == n) {  // every driver id survives: the driver list itself
      t.n = n;
      t.col[0] = lists[d].ids;
      return t;
    }
    int v = sp.var;
    Table o = alloc_table(m, &v, 1);
    if (m > 0) {
      ColSet in{};
      in.c[0] = lists[d].ids;
      OutSet out{};
      out.c[0] = const_cast<int32_t*>(o.col[0]);
      launch_compact_cols(in, 1, flags.p, n, ts.p, out, s);
    }
    return o;
  }

  void filter(int si, const gsmat_step_info& sp, Table& t, uint32_t next) {
    const gsmat_pattern& q = pl->pats[sp.tp];
    if (!is_var(q.s) && !is_var(q.o)) {
      const LookupRes r = lookup_tp(sp.tp, 0, q.p, q.s, q.o);
      if (r.found) {
        add_out(si, t.n);
        run(si + 1, t, next);
      } else {
        release(t);
      }
      return;
    }
    const int cs = is_var(q.s) ? t.col_of(var_of(q.s)) : -1;
    const int co = is_var(q.o) ? t.col_of(var_of(q.o)) : -1;
    // The pair (s, o) is looked for among the members of row s, or of row o in
    // the other orientation.  Right after an expansion to s by 2 rows and more
    // for each of its table, o is the same for runs of rows and s is not: o's
    // row pointers and the upper levels of the search are then read once for a
    // run.  33 million rows: by s 206 us, by o 131 us; 1.4 million rows of runs
    // of 2 to 4: 24.8 and 20.5 us.  Without runs both are scattered, and the rows of
    // s, which the hubs among the older columns do not lengthen, are kept.
    const bool by_o = co >= 0 && cs == t.k - 1 && t.from > 0 && t.n / t.from >= 2;
    ProbeArgs pa{};
    if (cs >= 0) (by_o ? pa.o_col : pa.s_col) = t.col[cs];
    else pa.s_const = q.s;
    if (co >= 0) (by_o ? pa.s_col : pa.o_col) = t.col[co];
    else (by_o ? pa.s_const : pa.o_const) = q.o;
    const PredView pv = (by_o ? st->in : st->out).view(q.p);
    const int64_t n = t.n;
    const int64_t nt = ceil_div(n, kTile);
    Tmp<uint8_t> flags(mem(), n, s);
    Tmp<int64_t> ts(mem(), nt + 1, s);
    launch_flag_filter(pa, n, pv, flags.p, ts.p, s);
    const int64_t m = scan_total(ts.p, nt, s);
    add_out(si, m);
    if (m == n) {  // nothing removed: pass the table on unchanged
      run(si + 1, t, next);
      return;
    }
    if (m == 0) {
      release(t);
      return;
    }
    Table o = alloc_table(m, t.var, t.k);
    o.from = t.from;
    ColSet in{};
    OutSet out{};
    for (int c = 0; c < t.k; ++c) {
      in.c[c] = t.col[c];
      out.c[c] = const_cast<int32_t*>(o.col[c]);
    }
    launch_compact_cols(in, t.k, flags.p, n, ts.p, out, s);
    release(t);
    run(si + 1, o, next);
  }

  void expand(int si, const gsmat_step_info& sp, Table& t, uint32_t next) {
    const gsmat_pattern& q = pl->pats[sp.tp];
    const int bound_var = sp.orient == 0 ? var_of(q.s) : var_of(q.o);
    const int bc = t.col_of(bound_var);
    if (bc < 0) throw StatusFail{GSMAT_EHIP, "internal: expansion from an unbound variable"};
    if (t.k + 1 > kMaxCols) throw StatusFail{GSMAT_EUNSUPPORTED, "too many columns"};
    const PredView pv = sp.orient == 0 ? st->out.view(q.p) : st->in.view(q.p);
    const int64_t n = t.n;
    const int64_t nt = ceil_div(n, kTile);
    Tmp<int32_t> N(mem(), n, s), start(mem(), n, s);
    Tmp<int64_t> ts(mem(), nt + 1, s), P(mem(), n + 1, s);
    launch_count_expand(t.col[bc], n, pv, N.p, start.p, ts.p, s);
    int64_t m;
    PinnedArea* h = dev_area ? nullptr : pinned();
    const uint32_t report = next_report();
    const bool scanned =
        h && launch_scan_rows(N.p, n, ts.p, P.p, &h->total[0], &h->word, report, s);
    if (scanned) {
      host_wait_words(&h->word, 1, report, s);
      m = h->total[0];
    } else {
      m = scan_total(ts.p, nt, s);
    }
    add_out(si, m);
    if (m == 0) {
      release(t);
      return;
    }
    if (!scanned) launch_scan_add_i32(N.p, n, ts.p, P.p, s);
    expand_write(si, sp.tp, sp.orient, t, next, P.p, start.p, m);
  }

  // The outputs of a counted expansion (offsets P, row starts start, m > 0
  // rows), in pieces within the budget, each carried through the remaining
  // steps; releases t.
  void expand_write(int si, int tp, int orient, Table& t, uint32_t next, const int64_t* P,
                    const int32_t* start, int64_t m) {
    const gsmat_pattern& q = pl->pats[tp];
    const PredView pv = orient == 0 ? st->out.view(q.p) : st->in.view(q.p);
    const int64_t n = t.n;
    int vars[kMaxCols];
    for (int c = 0; c < t.k; ++c) vars[c] = t.var[c];
    vars[t.k] = orient == 0 ? var_of(q.o) : var_of(q.s);
    const int k = t.k;
    const int64_t rpc = chunk_rows(k + 1);
    ColSet in{};
    for (int c = 0; c < k; ++c) in.c[c] = t.col[c];
    for (int64_t J0 = 0; J0 < m; J0 += rpc) {
      const int64_t J1 = std::min(m, J0 + rpc);
      const int64_t ntiles = ceil_div(n + (J1 - J0), kTile);
      Tmp<int64_t> split(mem(), ntiles + 1, s);
      launch_mp_partition(P, n, J0, J1, split.p, ntiles, s);
      Table o = alloc_table(J1 - J0, vars, k + 1);
      OutSet out{};
      for (int c = 0; c <= k; ++c) out.c[c] = const_cast<int32_t*>(o.col[c]);
      const double parents = (double)n * (double)(J1 - J0) / (double)m;
      o.from = std::max<int64_t>(1, (int64_t)parents);
      const double bytes = 4.0 * (double)(J1 - J0) * (k + 2) + parents * (4.0 * k + 12.0);
      launch_write_expand(in, k, P, start, n, pv.nbr, J0, J1, split.p, ntiles, out, bytes, s);
      run(si + 1, o, next);
    }
    release(t);
  }
};

}  // namespace

namespace gsmat {

HostNote host_note() {
  PinnedArea* h = pinned();
  return HostNote{&h->total[0], &h->word};
}

Arena::Arena(DeviceMem* m, size_t b, hipStream_t st) : mem(m), bytes(b), s(st) {
  p = mem->alloc(bytes, s);
  if (!p) throw OomFail{bytes};
}
Arena::~Arena() {
  if (idle) mem->free_idle(p, bytes, s);
  else mem->free(p, bytes, s);
}

uint32_t step_completes(const gsmat_query_plan* pl, const gsmat_step_info& sp) {
  if (sp.kind != GSMAT_STEP_INTERSECT) return 1u << sp.tp;
  uint32_t m = 0;
  const int32_t cterm = -(sp.var + 1);
  for (int tp = 0; tp < (int)pl->pats.size(); ++tp) {
    if (!(sp.members >> tp & 1)) continue;
    const gsmat_pattern& q = pl->pats[tp];
    const int32_t other = q.s == cterm ? q.o : q.s;
    if (!is_var(other)) m |= 1u << tp;
  }
  return m;
}

void step_candidates(const gsmat_store* st, const gsmat_query_plan* pl, const Table& t,
                     uint32_t rem, StepChoice& ch) {
  uint64_t bound = 0;
  for (int c = 0; c < t.k; ++c) bound |= 1ull << t.var[c];
  auto is_bound = [&](int32_t term) { return !is_var(term) || (bound >> var_of(term) & 1); };
  ch.has_filter = false;
  ch.nc = 0;
  const int np = (int)pl->pats.size();
  for (int tp = 0; tp < np; ++tp) {
    if (!(rem >> tp & 1)) continue;
    const gsmat_pattern& q = pl->pats[tp];
    const bool connected = (is_var(q.s) && (bound >> var_of(q.s) & 1)) ||
                           (is_var(q.o) && (bound >> var_of(q.o) & 1));
    const bool all_const = !is_var(q.s) && !is_var(q.o);
    if ((connected || all_const) && is_bound(q.s) && is_bound(q.o)) {
      std::memset(&ch.filter, 0, sizeof(ch.filter));
      ch.filter.kind = GSMAT_STEP_FILTER;
      ch.filter.tp = tp;
      ch.filter.orient = -1;
      ch.filter.var = -1;
      ch.has_filter = true;
      return;
    }
  }
  for (int tp = 0; tp < np; ++tp) {
    if (!(rem >> tp & 1)) continue;
    const gsmat_pattern& q = pl->pats[tp];
    const bool sb = is_var(q.s) && (bound >> var_of(q.s) & 1);
    const bool ob = is_var(q.o) && (bound >> var_of(q.o) & 1);
    if (sb == ob) continue;  // not connected (both bound were handled above)
    const int32_t free_term = sb ? q.o : q.s;
    if (!is_var(free_term)) continue;
    ch.cand_tp[ch.nc] = (int8_t)tp;
    ch.cand_or[ch.nc] = sb ? 0 : 1;
    ++ch.nc;
  }
  int pick = -1;
  int64_t best_nnz = INT64_MAX;
  for (int tp = 0; tp < np; ++tp) {
    if (!(rem >> tp & 1)) continue;
    const int64_t z = st->out.desc[pl->pats[tp].p].nnz;
    if (z < best_nnz) {
      best_nnz = z;
      pick = tp;
    }
  }
  std::memset(&ch.cartesian, 0, sizeof(ch.cartesian));
  ch.cartesian.kind = GSMAT_STEP_CARTESIAN;
  ch.cartesian.tp = pick;
  ch.cartesian.orient = -1;
  ch.cartesian.var = -1;
}

void candidate_view(const gsmat_store* st, const gsmat_query_plan* pl, const Table& t,
                    const StepChoice& c, int i, const int32_t** col, PredView* pv) {
  const gsmat_pattern& q = pl->pats[c.cand_tp[i]];
  const bool from_s = c.cand_or[i] == 0;
  *col = t.col[t.col_of(var_of(from_s ? q.s : q.o))];
  *pv = from_s ? st->out.view(q.p) : st->in.view(q.p);
}

gsmat_step_info step_pick(const gsmat_query_plan* pl, const StepChoice& c, const int64_t* sums) {
  int best = 0;
  if (sums)
    for (int i = 1; i < c.nc; ++i)
      if (sums[i] < sums[best]) best = i;
  const gsmat_pattern& q = pl->pats[c.cand_tp[best]];
  gsmat_step_info sp;
  std::memset(&sp, 0, sizeof(sp));
  sp.kind = GSMAT_STEP_EXPAND;
  sp.tp = c.cand_tp[best];
  sp.orient = c.cand_or[best];
  sp.var = c.cand_or[best] == 0 ? var_of(q.o) : var_of(q.s);
  return sp;
}

bool run_query(gsmat_store* st, const gsmat_query_plan* pl, int64_t budget_bytes,
               int64_t max_rows, hipStream_t s, gsmat_result* res, DeviceMem* mem,
               void* dev_area, bool small, size_t* small_bytes) {
  // a pattern over an absent predicate or vertex matches nothing
  for (const gsmat_pattern& q : pl->pats) {
    if (q.p >= st->P) return true;
    if (!is_var(q.s) && q.s >= st->V) return true;
    if (!is_var(q.o) && q.o >= st->V) return true;
  }
  Exec ex{st, pl, s, budget_bytes, max_rows, res, pl->mode == GSMAT_PLAN_ADAPTIVE, {},
          mem, (PinnedArea*)dev_area};
  ex.small = small && st->small_joins;
  ex.small_bytes = small_bytes;
  Table unit;
  unit.n = 1;
  unit.k = 0;
  try {
    ex.run(0, unit, all_of(pl));
  } catch (...) {
    ex.release_all();
    throw;
  }
  return ex.settled;
}

SmallBatchEnd run_small_batch(gsmat_store* st, const gsmat_query_plan* const* plans, int32_t nq,
                              const SmallBatchRun& run, hipStream_t s,
                              std::vector<DevQueryOut>& out) {
  const int64_t budget = run.budget, max_rows = run.max_rows;
  const bool server = run.server;
  out.clear();
  out.resize(nq);
  for (DevQueryOut& o : out) o.state = kDevFallback;
  struct One {
    int q;  // the query
    SmallLayout l;
    std::unique_ptr<gsmat_result> res;
    std::unique_ptr<Exec> ex;
    Table t;
    Exec::SmallMem sm;
    int64_t at = -1;    // its table's place in the batch's outputs (-1: none)
    Table w;            // that table
    bool skip = false;  // left to the rounds
  };
  // How each query starts, and whether the launch is made.
  enum : char { kAbsent, kView, kIn, kRest };
  std::vector<char> how(nq);
  // Every query's own final block, of a size that keeps the batch's within
  // kSmallBatchFins (an answer in its block needs no write of its own: 17 queries of
  // 137 to 2192 rows 195 us with 4 KiB, 176 with 64).
  int tier = kSmallFins - 1;
  while (tier > 0 && nq * kFinBytes[tier] > kSmallBatchFins) --tier;
  const int64_t work_most = std::min(kSmallBatchWork, run.room);
  int64_t work_bytes = 0, room = run.room;
  int n = 0, most_pats = 0, rest_pats = 0, rest_steps = 0, unsure = 0;
  auto adaptive = [&](int i) { return plans[i]->mode == GSMAT_PLAN_ADAPTIVE; };
  // a pattern after the first adds one variable at most
  auto layout = [&](int i) {
    const int np = (int)plans[i]->pats.size();
    return SmallLayout(np, np + 1);
  };
  for (int i = 0; i < nq; ++i) {
    const gsmat_query_plan* pl = plans[i];
    const Exec ex{st, pl, s, budget, max_rows, nullptr, adaptive(i)};
    const int np = (int)pl->pats.size();
    bool absent = false;
    for (const gsmat_pattern& q : pl->pats)
      absent |= q.p >= st->P || (!is_var(q.s) && q.s >= st->V) || (!is_var(q.o) && q.o >= st->V);
    how[i] = absent ? kAbsent
             : ex.is_view() ? kView
             : ex.small_first() && work_bytes + layout(i).bytes + kFinBytes[tier] <= work_most
                 ? kIn : kRest;
    if (how[i] == kIn) {
      work_bytes += layout(i).bytes;
      room -= layout(i).bytes + kFinBytes[tier];
      most_pats = std::max(most_pats, np);
      unsure += np >= 3;
      ++n;
    } else if (how[i] == kRest) {
      rest_pats = std::max(rest_pats, np);
      rest_steps += np;
    }
  }
  // Steps that may be taken alone: a third more than the rounds the longest
  // query takes, which cost a third more each; two more if there is no launch.
  const int alone = 4 * std::max(most_pats, rest_pats) / 3 + (n > 0 ? 0 : 2);
  if (server ? rest_pats >= most_pats : rest_steps > alone || unsure > kSmallUnsure)
    return {false, true};
  std::vector<One> v;
  v.reserve(n);
  auto finish = [&](One& o, auto&& f) {
    const gsmat_status rc = guarded([&]() -> gsmat_status {
      try {
        f();
      } catch (...) {
        o.ex->release_all();
        throw;
      }
      return GSMAT_OK;
    });
    out[o.q] = rc == GSMAT_OK ? DevQueryOut{std::move(o.res), kDevDone, GSMAT_OK}
                              : DevQueryOut{nullptr, kDevFailed, rc};
    return rc == GSMAT_OK && o.ex->settled;
  };
  for (int i = 0; i < nq; ++i) {
    if (how[i] == kRest) continue;
    One o{i, layout(i)};
    o.res.reset(new gsmat_result);
    o.res->st = st;
    o.res->stream = s;
    o.res->n_vars = plans[i]->n_vars;
    o.res->reset_steps(plans[i]->steps.size());
    o.ex.reset(new Exec{st, plans[i], s, budget, max_rows, o.res.get(), adaptive(i)});
    o.t.n = 1;
    o.t.k = 0;
    if (how[i] == kIn) v.push_back(std::move(o));
    else finish(o, [&] { if (how[i] == kView) o.ex->run(0, o.t, all_of(plans[i])); });
  }
  if (n == 0) return {!server, true};
  DeviceMem* mem = st->mem.get();
  std::shared_ptr<Arena> work, fin, outs;
  try {
    work = std::make_shared<Arena>(mem, (size_t)work_bytes, s);
    fin = std::make_shared<Arena>(mem, (size_t)kFinBytes[tier] * n, s);
  } catch (const OomFail&) {
    return {false, true};  // the rounds may need less
  }
  SmallReport* reps =
      (SmallReport*)query_area().get((sizeof(SmallArgs) + sizeof(SmallReport) +
                                      sizeof(SmallWriteTask)) * (size_t)n);
  SmallArgs* args = (SmallArgs*)(reps + n);
  char* at = (char*)work->p;
  for (int i = 0; i < n; ++i) {
    One& o = v[i];
    o.sm.work = at;
    o.sm.work_bytes = (size_t)o.l.bytes;
    at += o.l.bytes;
    o.sm.fin[tier] = (char*)fin->p + kFinBytes[tier] * i;
    o.sm.work_hold = work;
    o.sm.fin_hold = fin;
    o.ex->fill_small(args[i], 0, o.t, all_of(plans[o.q]), o.l, o.sm);
    reps[i].seq = 0;
  }
  const uint32_t seq = next_report();
  launch_small(small_store(st), args, reps, n, seq, s);
  host_wait_words(&reps[0].seq, n, seq, s, sizeof(SmallReport) / sizeof(uint32_t));
  // Finished here: what is done, what only has to be written, and with few
  // steps left in all the queries left on the way.
  auto left = [&](const SmallReport& r) {
    return r.status == kSmallMore || (r.status == kSmallWrite && (r.rem & ~(1u << r.tp)) != 0);
  };
  for (int i = 0; i < n; ++i)
    if (left(reps[i]))
      rest_steps += __builtin_popcount(reps[i].rem) - (reps[i].status == kSmallWrite);
  bool go_alone = !server && rest_steps <= alone;
  // everything to be written goes out in one launch, into one block, as the
  // outputs of a round do
  int64_t written = 0, total = 0, most = 0;
  double alg = 0;
  int nw = 0;
  SmallWriteTask* tasks = (SmallWriteTask*)(args + n);
  for (int i = 0; i < n; ++i) {
    One& o = v[i];
    const SmallReport& r = reps[i];
    const int64_t bytes = Exec::out_bytes(r);
    o.skip = left(r) && !go_alone;
    if (o.skip) continue;
    const bool pieces = Exec::counted(r) && !o.ex->one_piece(r);
    if (pieces) {  // each within the step budget
      o.skip = bytes > room - total;
      continue;
    }
    if (run.outputs > 0 && written > 0 && written + bytes > run.outputs) {
      o.skip = true;
      go_alone = false;  // the rounds take it, and what is found left from here on
      continue;
    }
    written += bytes;
    const bool move = r.status == kSmallDone && r.n > 0 && r.place == kAtWork;
    if (!move && !Exec::counted(r)) continue;
    if (bytes > room - total) {
      o.skip = true;
      go_alone = false;
      continue;
    }
    o.at = total;
    total += bytes;
  }
  try {
    if (total > 0) outs = std::make_shared<Arena>(mem, (size_t)total, s);
  } catch (const OomFail&) {  // the rounds may need less
  }
  for (int i = 0; i < n; ++i) {
    One& o = v[i];
    const SmallReport& r = reps[i];
    if (o.at < 0) continue;
    if (!outs) {
      o.skip = true;
      go_alone = false;
      continue;
    }
    o.ex->prepare_write(r, (const int64_t*)((char*)o.sm.work + o.l.offs),
                        (int32_t*)((char*)outs->p + o.at), tasks[nw++], o.w);
    o.w.keep = outs;
    most = std::max(most, o.w.n);
    alg += Exec::write_bytes(r);
  }
  launch_small_write(tasks, nw, most, alg, s);
  bool settled = nw == 0;
  for (int i = 0; i < n; ++i) {
    One& o = v[i];
    const SmallReport& r = reps[i];
    if (o.skip) continue;
    settled &= finish(o, [&] {
      int si = 0;
      uint32_t rem = 0;
      if (!o.ex->finish_small(r, (const int64_t*)((char*)o.sm.work + o.l.offs), o.sm, si, o.t, rem,
                              o.at >= 0 ? &o.w : nullptr))
        o.ex->run(si, o.t, rem);
    });
  }
  return {go_alone, settled};
}

void run_collect(gsmat_store* st, const gsmat_query_plan* pl, const Table* t0,
                 int64_t budget_bytes, hipStream_t s, std::vector<Table>* out) {
  for (const gsmat_pattern& q : pl->pats) {
    if (q.p >= st->P) return;
    if (!is_var(q.s) && q.s >= st->V) return;
    if (!is_var(q.o) && q.o >= st->V) return;
  }
  gsmat_result counters;  // step counters only (no steps kept)
  counters.st = st;
  counters.stream = s;
  Exec ex{st, pl, s, budget_bytes, -1, &counters, true, {}, nullptr, nullptr, out};
  ex.small = st->small_joins;
  Table t;
  if (t0) {
    if (t0->owned) throw StatusFail{GSMAT_EHIP, "internal: a starting table must not own memory"};
    t = *t0;
  } else {
    t.n = 1;
    t.k = 0;
  }
  const size_t first = out->size();
  try {
    ex.run(0, t, all_of(pl));
  } catch (...) {
    ex.release_all();
    for (size_t i = first; i < out->size(); ++i)
      if ((*out)[i].owned) st->mem->free((*out)[i].owned, (*out)[i].owned_bytes, s);
    out->resize(first);
    throw;
  }
}

// Statistics of each pattern for the planner.
std::vector<TpStat> pattern_stats(const gsmat_store* st, const gsmat_pattern* pats, int n,
                                  int mode, hipStream_t s, std::vector<gsmat_pat_lookup>* lk) {
  std::vector<TpStat> out(n);
  if (lk) lk->assign(n, gsmat_pat_lookup{});
  std::vector<LookupReq> reqs;
  std::vector<int> req_of(n, -1);
  for (int i = 0; i < n; ++i) {
    const gsmat_pattern& q = pats[i];
    TpStat& t = out[i];
    if (q.p < 0 || q.p >= st->P) continue;  // absent predicate: empty relation
    const PredDesc& dout = st->out.desc[q.p];
    const PredDesc& din = st->in.desc[q.p];
    t.stat = dout.nnz;
    t.rows_s = dout.nr;
    t.rows_o = din.nr;
    if (mode == GSMAT_PLAN_PAPER) continue;
    const bool sc = !is_var(q.s), oc = !is_var(q.o);
    if ((sc && q.s >= st->V) || (oc && q.o >= st->V)) {
      t.stat = t.rows_s = t.rows_o = 0;
      continue;
    }
    if (sc && oc) {
      req_of[i] = (int)reqs.size();
      reqs.push_back({0, q.p, q.s, q.o});
    } else if (sc) {
      req_of[i] = (int)reqs.size();
      reqs.push_back({0, q.p, q.s, -1});
    } else if (oc) {
      req_of[i] = (int)reqs.size();
      reqs.push_back({1, q.p, q.o, -1});
    }
  }
  if (!reqs.empty()) {
    LookupBatch b{};
    for (size_t i = 0; i < reqs.size(); ++i) b.req[i] = reqs[i];
    b.n = (int32_t)reqs.size();
    PinnedArea* h = pinned();
    const uint32_t report = next_report();
    launch_lookup(b, st->out.d_desc, st->in.d_desc, st->out.ptrs(), st->in.ptrs(), h->res, s,
                  &h->word, report);
    host_wait_words(&h->word, 1, report, s);
    std::vector<LookupRes> res(h->res, h->res + reqs.size());
    for (int i = 0; i < n; ++i) {
      if (req_of[i] < 0) continue;
      const LookupRes& r = res[req_of[i]];
      if (lk) (*lk)[i] = gsmat_pat_lookup{r.start, r.len, r.found, 1};
      const gsmat_pattern& q = pats[i];
      const bool sc = !is_var(q.s), oc = !is_var(q.o);
      const int64_t v = (sc && oc) ? r.found : r.len;
      out[i].stat = v;
      out[i].rows_s = v;
      out[i].rows_o = v;
    }
  }
  return out;
}

}  // namespace gsmat

extern "C" gsmat_status gsmat_plan(const gsmat_store* st, const gsmat_pattern* pats,
                                   int32_t n_pats, int32_t mode, void* stream, gsmat_query_plan** out) {
  return guarded([&]() -> gsmat_status {
    if (!out) throw StatusFail{GSMAT_EINVAL, "out is NULL"};
    *out = nullptr;
    if (!st) throw StatusFail{GSMAT_EINVAL, "store is NULL"};
    std::string err;
    int32_t nv = 0;
    gsmat_status rc = validate_patterns(pats, n_pats, &nv, &err);
    if (rc != GSMAT_OK) throw StatusFail{rc, err};
    if (!st->built) throw StatusFail{GSMAT_ESTATE, "index not built"};
    (void)pinned();  // here, not in a join that must not allocate
    std::vector<gsmat_pat_lookup> lk;
    std::vector<TpStat> ts = pattern_stats(st, pats, n_pats, mode, (hipStream_t)stream, &lk);
    std::unique_ptr<gsmat_query_plan> pl(new gsmat_query_plan);
    rc = build_plan(pats, n_pats, mode, ts.data(), pl.get(), &err);
    if (rc != GSMAT_OK) throw StatusFail{rc, err};
    if (mode != GSMAT_PLAN_PAPER) {
      pl->lk = std::move(lk);
      pl->lk_store = st->uid;
    }
    *out = pl.release();
    return GSMAT_OK;
  });
}

extern "C" gsmat_status gsmat_join(gsmat_store* st, const gsmat_query_plan* pl, int64_t budget_bytes,
                                   int64_t max_rows, void* stream, gsmat_result** out) {
  return guarded([&]() -> gsmat_status {
    if (!out) throw StatusFail{GSMAT_EINVAL, "out is NULL"};
    *out = nullptr;
    if (!st || !pl) throw StatusFail{GSMAT_EINVAL, "store or plan is NULL"};
    if (!st->built) throw StatusFail{GSMAT_ESTATE, "index not built"};
    hipStream_t s = (hipStream_t)stream;
    std::unique_ptr<gsmat_result> res(new gsmat_result);
    res->st = st;
    res->stream = s;
    res->n_vars = pl->n_vars;
    res->reset_steps(pl->steps.size());
    if (!run_query(st, pl, budget_bytes, max_rows, s, res.get())) GS_HIP(hipStreamSynchronize(s));
    *out = res.release();
    return GSMAT_OK;
  });
}

// ---------------------------------------------------------- allocation-free join
//
// gsmat_join_noalloc keeps every intermediate table and every step's scratch
// in one file-scope device array of kNoAllocBytes (each GPU the library runs
// on has its own copy, held until the process ends).  Host code never uses
// the array's name as a device address: the address comes from
// hipGetSymbolAddress, taken once per device with that device current.

namespace {

constexpr size_t kNoAllocBytes = (size_t)64 << 20;
static __device__ __align__(256) char scratch[kNoAllocBytes];

struct NoAllocDevice {
  std::mutex mu;          // serialises the calls on this device
  char* base = nullptr;   // the array's device address
};

NoAllocDevice* noalloc_device(int dev) {
  static std::mutex mu;
  static std::map<int, NoAllocDevice*> devs;
  std::lock_guard<std::mutex> g(mu);
  NoAllocDevice*& d = devs[dev];
  if (!d) {
    std::unique_ptr<NoAllocDevice> nd(new NoAllocDevice);
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      throw StatusFail{GSMAT_EHIP, std::string("no-alloc scratch: hipGetSymbolAddress failed: ") +
                                       hipGetErrorString(e)};
    nd->base = (char*)p;
    d = nd.release();
  }
  return d;
}

// Stack allocator over the array: blocks come off the top; a free marks its
// block, and the top drops past every freed block at the top (the executor
// frees in nearly reverse order).  The first kStageBytes hold the staged
// small results.
struct ScratchStack {
  char* base = nullptr;
  size_t top = kStageBytes;
  size_t want = 0;  // largest request that did not fit
  size_t over = 0;  // bytes the last of them was over
  std::vector<size_t> off, len;
  std::vector<char> freed;

  void* alloc(size_t bytes) {
    const size_t b = (std::max<size_t>(bytes, 1) + 255) / 256 * 256;
    if (b > kNoAllocBytes - top) {
      want = std::max(want, b);
      over = b - (kNoAllocBytes - top);
      return nullptr;
    }
    off.push_back(top);
    len.push_back(b);
    freed.push_back(0);
    void* p = base + top;
    top += b;
    return p;
  }
  void free(void* p) {
    const size_t o = (size_t)((char*)p - base);
    for (size_t i = off.size(); i-- > 0;)
      if (off[i] == o && !freed[i]) {
        freed[i] = 1;
        break;
      }
    while (!off.empty() && freed.back()) {
      top = off.back();
      off.pop_back();
      len.pop_back();
      freed.pop_back();
    }
  }
  static void* alloc_cb(size_t bytes, void* stream, void* ctx) {
    (void)stream;
    return ((ScratchStack*)ctx)->alloc(bytes);
  }
  static void free_cb(void* p, size_t bytes, void* stream, void* ctx) {
    (void)bytes;
    (void)stream;
    ((ScratchStack*)ctx)->free(p);
  }
};

}  // namespace

extern "C" gsmat_status gsmat_join_noalloc(gsmat_store* st, const gsmat_query_plan* pl,
                                           int32_t* out, int64_t out_stride, int64_t out_cap,
                                           int64_t* n_rows, void* stream) {
  return guarded([&]() -> gsmat_status {
    if (!st || !pl || !n_rows) throw StatusFail{GSMAT_EINVAL, "store, plan or n_rows is NULL"};
    *n_rows = 0;
    if (!st->built) throw StatusFail{GSMAT_ESTATE, "index not built"};
    if (out_cap < 0 || out_stride < out_cap)
      throw StatusFail{GSMAT_EINVAL, "out_cap must be >= 0 and out_stride >= out_cap"};
    if (!out && out_cap > 0 && pl->n_vars > 0) throw StatusFail{GSMAT_EINVAL, "out is NULL"};
    hipStream_t s = (hipStream_t)stream;
    int dev = 0;
    GS_HIP(hipGetDevice(&dev));
    NoAllocDevice* nd = noalloc_device(dev);
    std::lock_guard<std::mutex> lock(nd->mu);
    ScratchStack stack;
    stack.base = nd->base;
    const gsmat_allocator a{&ScratchStack::alloc_cb, &ScratchStack::free_cb, &stack};
    DeviceMem mem(&a);
    gsmat_result res;
    res.st = st;
    res.stream = s;
    res.n_vars = pl->n_vars;
    res.reset_steps(pl->steps.size());
    struct Drop {  // the segments live in the array: nothing to free
      gsmat_result& r;
      ~Drop() {
        for (Segment& g : r.segs) g.owned = nullptr;
      }
    } drop{res};
    size_t small_bytes = 0;
    try {
      try {
        run_query(st, pl, 0, -1, s, &res, &mem, nd->base, true, &small_bytes);
      } catch (const OomFail&) {
        // the small launches' areas may be what did not fit: once without them
        if (stack.over > small_bytes) throw;
        (void)hipStreamSynchronize(s);
        stack = ScratchStack();
        stack.base = nd->base;
        res.segs.clear();
        res.rows = 0;
        res.reset_steps(pl->steps.size());
        run_query(st, pl, 0, -1, s, &res, &mem, nd->base, false);
      }
    } catch (const OomFail&) {
      (void)hipStreamSynchronize(s);  // nothing may still use the array
      throw StatusFail{GSMAT_ENOMEM,
                       "the join needs more than the " + std::to_string(kNoAllocBytes >> 20) +
                           " MiB of the allocation-free scratch (a block of " +
                           std::to_string(stack.want) + " bytes did not fit)"};
    } catch (...) {
      (void)hipStreamSynchronize(s);
      throw;
    }
    *n_rows = res.rows;
    if (res.rows > out_cap) {
      host_sync(s);
      throw StatusFail{GSMAT_ETOOBIG, "result has " + std::to_string(res.rows) +
                                          " rows, more than out_cap (" + std::to_string(out_cap) +
                                          ")"};
    }
    int64_t at = 0;
    for (const Segment& g : res.segs) {
      for (int v = 0; v < pl->n_vars && g.rows > 0; ++v)
        GS_HIP(hipMemcpyAsync(out + (int64_t)v * out_stride + at, g.col[v],
                              sizeof(int32_t) * (size_t)g.rows, hipMemcpyDeviceToDevice, s));
      at += g.rows;
    }
    // the array is reused by the next call: its work ends before this returns
    host_sync(s);
    return GSMAT_OK;
  });
}

extern "C" gsmat_status gsmat_result_info(const gsmat_result* r, int64_t* n_rows, int32_t* n_vars,
                                          int32_t* n_steps, int64_t* step_rows_in,
                                          int64_t* step_rows_out) {
  return guarded([&]() -> gsmat_status {
    if (!r) throw StatusFail{GSMAT_EINVAL, "result is NULL"};
    if (n_rows) *n_rows = r->rows;
    if (n_vars) *n_vars = r->n_vars;
    if (n_steps) *n_steps = r->n_steps;
    if (step_rows_in) std::copy(r->step_in, r->step_in + r->n_steps, step_rows_in);
    if (step_rows_out) std::copy(r->step_out, r->step_out + r->n_steps, step_rows_out);
    return GSMAT_OK;
  });
}

namespace {

// Rows [lo, hi) of a result to host memory.
struct FetchSpan {
  const gsmat_result* r;
  int64_t lo, hi;
  int32_t* to;
};

// Fetches the spans through the calling thread's transfer area: pieces of at
// most one part, in order, as many in a launch as fit the part, a part packed
// by the device while the other is copied out.  Sixty answers of a batch, 4.1 MB:
// 1.0 ms one by one, 0.31 ms together.
void fetch_spans(const FetchSpan* sp, int n, hipStream_t s) {
  uint64_t bytes = 0;
  for (int i = 0; i < n; ++i)
    bytes += sizeof(int32_t) * (uint64_t)(sp[i].hi - sp[i].lo) * sp[i].r->n_vars;
  if (bytes == 0) return;
  FetchArea& fa = fetch_area();
  fa.reserve(std::min<uint64_t>(bytes, FetchArea::kLarge));
  struct Piece {
    int32_t* from;
    int32_t* to;
    int64_t bytes;
  };
  struct Group {
    std::vector<Piece> pieces;
    int64_t bytes = 0;
    int words = 0;
    uint32_t report = 0;
  } gr[2];
  // the next row to pack: row `at` of span si, in segment seg_i (first row seg_lo)
  int si = 0;
  size_t seg_i = 0;
  int64_t seg_lo = 0, at = sp[0].lo;
  auto pack_next = [&](int i) {
    Group& g = gr[i];
    g.pieces.clear();
    g.bytes = 0;
    size_t used = 0;
    while ((int)g.pieces.size() < kPackGroups) {
      while (si < n && at >= sp[si].hi) {
        ++si;
        seg_i = 0;
        seg_lo = 0;
        if (si < n) at = sp[si].lo;
      }
      if (si >= n) break;
      const gsmat_result* r = sp[si].r;
      const int nv = r->n_vars;
      const int64_t fit = (int64_t)((fa.part - used) / (sizeof(int32_t) * nv));
      if (fit < std::min<int64_t>(sp[si].hi - at, 256)) break;  // the next part's
      while (at >= seg_lo + r->segs[seg_i].rows) seg_lo += r->segs[seg_i++].rows;
      const Segment& seg = r->segs[seg_i];
      PackTask& t = fa.tasks(i)[g.pieces.size()];
      for (int v = 0; v < nv; ++v) t.cols.c[v] = seg.col[v];
      t.k = nv;
      t.row0 = at - seg_lo;
      t.rows = std::min(std::min(sp[si].hi, seg_lo + seg.rows) - at, fit);
      t.out = (int32_t*)((char*)fa.rows(i) + used);
      const int64_t b = sizeof(int32_t) * t.rows * nv;
      g.pieces.push_back(Piece{t.out, sp[si].to + (at - sp[si].lo) * nv, b});
      g.bytes += b;
      used += (size_t)(b + 15) / 16 * 16;
      if (used > fa.part) used = fa.part;
      at += t.rows;
    }
    if (g.pieces.empty()) return;
    g.report = next_report();
    g.words =
        launch_pack_rows(fa.tasks(i), (int)g.pieces.size(), fa.words(i), g.report, s);
  };
  try {
    pack_next(0);
    pack_next(1);
    char* const end = n == 1 ? (char*)(sp[0].to + (sp[0].hi - sp[0].lo) * sp[0].r->n_vars) : nullptr;
    char* mapped = n == 1 ? (char*)sp[0].to : nullptr;
    for (int i = 0; !gr[i].pieces.empty(); i ^= 1) {
      Group& g = gr[i];
      if (n == 1 && (char*)g.pieces.back().to + g.pieces.back().bytes > mapped)
        mapped = map_ahead(mapped, end);
      host_wait_words(fa.words(i), g.words, g.report, s);
      if (g.pieces.size() == 1) {
        copy_host((char*)g.pieces[0].to, (const char*)g.pieces[0].from, g.pieces[0].bytes);
      } else {  // at least 512 KiB a thread
        const int64_t np = (int64_t)g.pieces.size();
        host_parallel_for(np, ceil_div(np * (512 << 10), std::max<int64_t>(g.bytes, 1)),
                          [&](int64_t a, int64_t b) {
                            for (; a < b; ++a)
                              std::memcpy(g.pieces[a].to, g.pieces[a].from, (size_t)g.pieces[a].bytes);
                          });
      }
      pack_next(i);
    }
  } catch (...) {
    (void)hipStreamSynchronize(s);  // nothing may still write the area
    throw;
  }
}

}  // namespace

extern "C" gsmat_status gsmat_fetch_bindings(const gsmat_result* r, int64_t row_offset,
                                             int64_t max_rows, int32_t* host_rows,
                                             int64_t* n_written, void* stream) {
  return guarded([&]() -> gsmat_status {
    if (!r) throw StatusFail{GSMAT_EINVAL, "result is NULL"};
    if (row_offset < 0 || max_rows < 0) throw StatusFail{GSMAT_EINVAL, "negative offset or count"};
    const int64_t lo = std::min(row_offset, r->rows);
    const int64_t hi = std::min(r->rows, lo + max_rows);
    if (n_written) *n_written = hi - lo;
    if (hi <= lo || r->n_vars == 0) return GSMAT_OK;
    if (!host_rows) throw StatusFail{GSMAT_EINVAL, "host_rows is NULL"};
    const FetchSpan sp{r, lo, hi, host_rows};
    fetch_spans(&sp, 1, (hipStream_t)stream);
    return GSMAT_OK;
  });
}

extern "C" gsmat_status gsmat_fetch_bindings_many(const gsmat_result* const* results, int32_t n,
                                                  int32_t* const* host_rows, void* stream) {
  return guarded([&]() -> gsmat_status {
    if (n < 0) throw StatusFail{GSMAT_EINVAL, "negative count"};
    if (n > 0 && (!results || !host_rows))
      throw StatusFail{GSMAT_EINVAL, "results or host_rows is NULL"};
    std::vector<FetchSpan> sp;
    sp.reserve(n);
    for (int32_t i = 0; i < n; ++i) {
      const gsmat_result* r = results[i];
      if (!r || r->rows == 0 || r->n_vars == 0) continue;
      if (!host_rows[i])
        throw StatusFail{GSMAT_EINVAL, "host_rows[" + std::to_string(i) + "] is NULL"};
      sp.push_back(FetchSpan{r, 0, r->rows, host_rows[i]});
    }
    if (!sp.empty()) fetch_spans(sp.data(), (int)sp.size(), (hipStream_t)stream);
    return GSMAT_OK;
  });
}

extern "C" void gsmat_result_free(gsmat_result* r) { delete r; }
