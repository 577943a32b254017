// Small joins in one launch (paper Sec. 6.3 and Sec. 7.2 for tables of a few
// thousand rows).
//
// What bounds a small query is not its bytes but the chain of launches and
// host waits of the general path: four to six launches and one or two waits
// per step, each wait about 15 us with what it drains, for kernels of 2 to 5
// us.  Here one workgroup of 16 waves takes the query from its starting table
// to its answer: it chooses every step by the same rule, counts, scans,
// writes its tables in a work area and reports once.  The rules and the order
// of the rows are those of the general path:
//   * adaptive choice: with at most kSmallRows (below kSampleRows) rows the
//     sampled fan-out is the exact output of every candidate, so one pass
//     over all candidates is the sample and the count;
//   * an expansion's output j belongs to the last row whose offset is at most
//     j (binary search over the offsets in LDS), rows in order, members in
//     order;
//   * filters and intersections keep their rows in order.
// A step that is a Cartesian product or a (?x p ?x) scan, or that enters with
// more than kSmallRows rows, is left to the general path, which goes on from
// the table reported.  An expansion of more than kSmallRows rows, or an answer
// above kSmallFin bytes, is counted here and written by k_small_write into
// memory of its exact size: one CU writes about 50 GB/s, the launch and wait
// cost 15 us.  4096 rows are 16 waves of 4 rows a lane.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "small.hpp"

namespace gsmat {

namespace {

using namespace dev;

constexpr int kST = 1024;           // threads
constexpr int kSW = kST / 64;       // waves
constexpr int kSU = 4;              // rows per lane of a chunk
constexpr int kSChunk = 64 * kSU;   // rows per wave and chunk
static_assert(kSmallRows == kSW * kSChunk, "one chunk per wave covers a table");
static_assert(kSmallRows <= kSampleRows, "the candidates' sums must equal their samples");

// What row lookups need of a predicate in one orientation.
struct SmallPred {
  const int32_t *keys, *ptr, *nbr, *dense, *dir;
  int32_t nr, shift;
};

struct SmallList {
  const int32_t* ids;
  int64_t len;
  int32_t pred;  // row keys: the pattern (by subject), or kMaxPats + pattern; else -1
};

struct SmallLds {
  int32_t P[kSmallRows];   // output offset of every row (before: candidates' lengths)
  int32_t rb[kSmallRows];  // member base of every row, less its offset (before: starts)
  SmallArgs a;
  SmallPred pred[2 * kMaxPats];  // of pattern i by subject, by object at kMaxPats + i
  LookupRes lk[kMaxPats];
  const int32_t* col[kMaxCols];
  int32_t var[kMaxCols];
  int32_t col_of[kMaxCols];
  unsigned long long tot[kMaxPats];
  int32_t cand[kMaxPats];
  int32_t wsum[kSW];
  int64_t wsum64[kSW];
  SmallList list[kMaxLists];
  int64_t in[kMaxPats + 1], out[kMaxPats + 1];
};

__device__ inline int64_t s_stride(int64_t n) { return (n + 63) / 64 * 64; }

// Where the next table (of at most kSmallRows rows) goes: the smallest final
// block that holds it when it is the answer, else the half of the work area the
// current table is not in.
__device__ inline char* s_place(const SmallArgs& A, int64_t bytes, bool last, int half, int* place,
                                int* next_half) {
  if (last && bytes <= kSmallFin) {
    for (int f = 0; f < kSmallFins; ++f)
      if (bytes <= kFinBytes[f] && A.fin[f]) {
        *place = kAtFin + f;
        return A.fin[f];
      }
  }
  *place = kAtWork;
  *next_half = half ^ 1;
  return A.work + (half ^ 1) * A.tab;
}

__device__ inline PredView s_view(const SmallPred& p) {
  PredView v{};
  v.keys = p.keys;
  v.ptr = p.ptr;
  v.nbr = p.nbr;
  v.dense = p.dense;
  v.dir = p.dir;
  v.nr = p.nr;
  v.dir_shift = p.shift;
  return v;
}

// Keeps the rows whose flag is set, in order: the wave's rows are
// w * kSChunk + u * 64 + lane.  base receives the wave's first place; the
// total is returned.  Barriers inside.
__device__ inline int s_rank(SmallLds& L, const bool (&keep)[kSU], int (&pos)[kSU]) {
  int cnt = 0;
#pragma unroll
  for (int u = 0; u < kSU; ++u) {
    const uint64_t b = __ballot(keep[u]);
    pos[u] = cnt + (int)mbcnt(b);
    cnt += (int)__popcll(b);
  }
  if (lane_id() == 0) L.wsum[wave_id()] = cnt;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kSW; ++w) {
    const int c = L.wsum[w];
    if (w < wave_id()) base += c;
    tot += c;
  }
#pragma unroll
  for (int u = 0; u < kSU; ++u) pos[u] += base;
  __syncthreads();
  return tot;
}

__global__ __launch_bounds__(kST) void k_small_join(SmallStore S,
                                                    const SmallArgs* __restrict__ args,
                                                    SmallReport* reps, uint32_t seq) {
  __shared__ SmallLds L;
  SmallReport* const rep = reps + blockIdx.x;
  const int tid = (int)threadIdx.x, lane = lane_id(), wave = wave_id();
  {  // the query comes over in one trip to host memory
    static_assert(sizeof(SmallArgs) % 4 == 0 && sizeof(SmallArgs) / 4 <= kST, "one word a thread");
    const uint32_t* src = (const uint32_t*)(args + blockIdx.x);
    if (tid < (int)(sizeof(SmallArgs) / 4)) ((uint32_t*)&L.a)[tid] = src[tid];
  }
  __syncthreads();
  const SmallArgs& A = L.a;
  const int np = A.np;
  if (tid < np) {
    const SmallPat q = A.pats[tid];
    LookupRes r = A.lk[tid];
    if (!(A.lk_valid >> tid & 1) && (q.s >= 0 || q.o >= 0)) {
      LookupReq lq{q.s >= 0 ? 0 : 1, q.p, q.s >= 0 ? q.s : q.o, q.s >= 0 && q.o >= 0 ? q.o : -1};
      r = lookup_one(lq, S.dout, S.din, S.out, S.in);
    }
    L.lk[tid] = r;
  }
  // the predicates' descriptors, by two waves while the first looks up
  if (wave == 1 || wave == 2) {
    if (lane < np) {
      const PredView v = wave == 1 ? view_of(S.dout[A.pats[lane].p], S.out)
                                   : view_of(S.din[A.pats[lane].p], S.in);
      L.pred[(wave - 1) * kMaxPats + lane] =
          SmallPred{v.keys, v.ptr, v.nbr, v.dense, v.dir, v.nr, v.dir_shift};
    }
  }
  if (tid < kMaxPats + 1) L.in[tid] = L.out[tid] = 0;
  if (tid < kMaxCols) {
    L.col_of[tid] = -1;
    L.col[tid] = nullptr;
    L.var[tid] = 0;
  }
  __syncthreads();
  if (tid < A.k) {
    L.col[tid] = A.col[tid];
    L.var[tid] = A.var[tid];
    if (A.var[tid] < kMaxCols) L.col_of[A.var[tid]] = tid;
  }
  __syncthreads();

  // the state, alike in every thread
  int64_t n = A.n;
  int k = A.k, si = A.si, status = kSmallMore, place = kAtStart, half = 1;
  uint32_t rem = A.rem;
  int left_tp = -1, left_orient = -1;  // an expansion counted and left to be written
  int64_t left_m = 0;
  const int32_t* left_start = nullptr;
  uint64_t bound = 0;
  for (int c = 0; c < k; ++c) bound |= 1ull << L.var[c];

  const SmallPat my = lane < np ? A.pats[lane] : SmallPat{0, 0, 0};
  for (;;) {
    if (n == 0 || rem == 0) {
      status = kSmallDone;
      break;
    }
    if (n > kSmallRows) break;
    const bool unit = n == 1 && k == 0;
    int kind, tp = 0, var = -1;
    uint32_t members = 0, cmask = 0, smask = 0;  // candidates; those bound at their subject
    if (A.adaptive && !unit) {
      const bool in = lane < np && (rem >> (lane & 31) & 1);
      const bool vs = my.s < 0 && (bound >> (-my.s - 1) & 1);
      const bool vo = my.o < 0 && (bound >> (-my.o - 1) & 1);
      const bool full = in && (my.s >= 0 || vs) && (my.o >= 0 || vo);
      const uint64_t mf = __ballot(full);
      if (mf) {
        kind = GSMAT_STEP_FILTER;
        tp = __ffsll((unsigned long long)mf) - 1;
      } else {
        const bool cand = in && vs != vo && (vs ? my.o < 0 : my.s < 0);
        cmask = (uint32_t)__ballot(cand);
        smask = (uint32_t)__ballot(cand && vs);
        if (!cmask) break;  // a Cartesian product
        kind = GSMAT_STEP_EXPAND;
      }
    } else {
      const SmallStep sp = A.steps[si < A.nsteps ? si : A.nsteps - 1];
      kind = sp.kind;
      tp = sp.tp;
      var = sp.var;
      members = sp.members;
      if (kind == GSMAT_STEP_EXPAND) {
        cmask = 1u << tp;
        smask = sp.orient == 0 ? cmask : 0u;
        const int32_t b = sp.orient == 0 ? A.pats[tp].s : A.pats[tp].o;
        if (b >= 0 || !(bound >> (-b - 1) & 1)) break;
      }
    }

    if (kind == GSMAT_STEP_SCAN || kind == GSMAT_STEP_CARTESIAN) {
      const SmallPat q = A.pats[tp];
      if (!unit || (q.s < 0 && q.s == q.o)) break;
      const LookupRes lk = L.lk[tp];
      __syncthreads();
      if (q.s < 0 && q.o < 0) {
        n = S.dout[q.p].nnz;
        k = 2;
        if (tid == 0) {
          L.col[0] = S.out_src + S.dout[q.p].nbr_base;
          L.col[1] = L.pred[tp].nbr;
          L.var[0] = -q.s - 1;
          L.var[1] = -q.o - 1;
          L.col_of[-q.s - 1] = 0;
          L.col_of[-q.o - 1] = 1;
        }
        bound = 1ull << (-q.s - 1) | 1ull << (-q.o - 1);
      } else if (q.s >= 0 && q.o >= 0) {
        n = lk.found ? 1 : 0;
      } else {
        const int v = q.s >= 0 ? -q.o - 1 : -q.s - 1;
        n = lk.len;
        k = 1;
        if (tid == 0) {
          L.col[0] = L.pred[q.s >= 0 ? tp : kMaxPats + tp].nbr + lk.start;
          L.var[0] = v;
          L.col_of[v] = 0;
        }
        bound = 1ull << v;
      }
      if (tid == 0 && si < A.nsteps) {
        L.in[si] += 1;
        L.out[si] += n;
      }
      rem &= ~(1u << tp);
      ++si;
      __syncthreads();
      continue;
    }

    if (kind == GSMAT_STEP_INTERSECT) {
      if (!unit) break;
      const int32_t cterm = -(var + 1);
      const bool mem = lane < np && (members >> (lane & 31) & 1);
      const uint32_t fin_of = (uint32_t)__ballot(mem && (my.s == cterm ? my.o : my.s) >= 0);
      const uint64_t mm = __ballot(mem);
      const int nl = (int)__popcll(mm);
      if (nl > kMaxLists || nl < 1) break;
      if (wave == 0 && mem) {
        SmallList l;
        const bool subj = my.s == cterm;  // the centre is the subject
        if (subj ? my.o < 0 : my.s < 0) {
          l.pred = subj ? lane : kMaxPats + lane;
          l.len = L.pred[l.pred].nr;
          l.ids = L.pred[l.pred].keys;
        } else {
          l.pred = -1;
          l.len = L.lk[lane].len;
          l.ids = L.pred[subj ? kMaxPats + lane : lane].nbr + L.lk[lane].start;
        }
        L.list[mbcnt(mm)] = l;
      }
      __syncthreads();
      int d = 0;  // the shortest list drives, the first on ties
      for (int i = 1; i < nl; ++i)
        if (L.list[i].len < L.list[d].len) d = i;
      const int64_t dn = L.list[d].len;
      if (dn > kSmallRows) break;
      const int32_t* ids = L.list[d].ids;
      int32_t x[kSU];
      bool keep[kSU];
      int pos[kSU];
#pragma unroll
      for (int u = 0; u < kSU; ++u) {
        const int r = wave * kSChunk + u * 64 + lane;
        keep[u] = r < dn;
        x[u] = keep[u] ? ids[r] : 0;
      }
      for (int i = 0; i < nl; ++i) {
        if (i == d) continue;
        int32_t a[kSU], b[kSU];
        if (L.list[i].pred >= 0) {
          const PredView pv = s_view(L.pred[L.list[i].pred]);
          row_lookup_n<kSU>(pv, x, keep, a, b);
#pragma unroll
          for (int u = 0; u < kSU; ++u) keep[u] = keep[u] && b[u] > 0;
        } else {
          const int32_t* seg = L.list[i].ids;
          const int32_t len = (int32_t)L.list[i].len;
#pragma unroll
          for (int u = 0; u < kSU; ++u) {
            a[u] = 0;
            b[u] = keep[u] ? len : 0;
          }
          lower_bound_n<kSU>(seg, x, a, b);
#pragma unroll
          for (int u = 0; u < kSU; ++u) keep[u] = keep[u] && a[u] < len && seg[a[u]] == x[u];
        }
      }
      const int m = s_rank(L, keep, pos);
      if (m == dn || m == 0) {
        if (tid == 0) L.col[0] = ids;
      } else {
        int pl = place, hf = half;
        char* to = s_place(A, 4 * s_stride(m), (rem & ~fin_of) == 0, half, &pl, &hf);
        int32_t* o = (int32_t*)to;  // at most kSmallRows values: fits
#pragma unroll
        for (int u = 0; u < kSU; ++u)
          if (keep[u]) o[pos[u]] = x[u];
        place = pl;
        half = hf;
        if (tid == 0) L.col[0] = o;
      }
      if (tid == 0) {
        L.var[0] = var;
        L.col_of[var] = 0;
        if (si < A.nsteps) {
          L.in[si] += 1;
          L.out[si] += m;
        }
      }
      n = m;
      k = 1;
      bound = 1ull << var;
      rem &= ~fin_of;
      ++si;
      __syncthreads();
      continue;
    }

    if (kind == GSMAT_STEP_FILTER) {
      const SmallPat q = A.pats[tp];
      const uint32_t next = rem & ~(1u << tp);
      int64_t m = n;
      if (q.s >= 0 && q.o >= 0) {
        if (!L.lk[tp].found) m = 0;
      } else {
        const int cs = q.s < 0 ? L.col_of[-q.s - 1] : -1, co = q.o < 0 ? L.col_of[-q.o - 1] : -1;
        if ((q.s < 0 && cs < 0) || (q.o < 0 && co < 0)) break;
        const int32_t* sc = cs >= 0 ? L.col[cs] : nullptr;
        const int32_t* oc = co >= 0 ? L.col[co] : nullptr;
        const PredView pv = s_view(L.pred[tp]);
        int32_t sv[kSU], ov[kSU], st[kSU], len[kSU], lo[kSU], cnt[kSU];
        bool keep[kSU];
        int pos[kSU];
#pragma unroll
        for (int u = 0; u < kSU; ++u) {
          const int r = wave * kSChunk + u * 64 + lane;
          keep[u] = r < n;
          sv[u] = keep[u] ? (sc ? sc[r] : q.s) : 0;
          ov[u] = keep[u] ? (oc ? oc[r] : q.o) : 0;
        }
        row_lookup_n<kSU>(pv, sv, keep, st, len);
#pragma unroll
        for (int u = 0; u < kSU; ++u) {
          lo[u] = st[u];
          cnt[u] = len[u];
        }
        lower_bound_n<kSU>(pv.nbr, ov, lo, cnt);
#pragma unroll
        for (int u = 0; u < kSU; ++u)
          keep[u] = len[u] > 0 && lo[u] < st[u] + len[u] && pv.nbr[lo[u]] == ov[u];
        m = s_rank(L, keep, pos);
        if (m > 0 && m < n) {
          const int64_t stride = s_stride(m);
          int pl = place, hf = half;
          char* to = s_place(A, 4 * stride * k, next == 0, half, &pl, &hf);
          int32_t* o = (int32_t*)to;
          for (int c = 0; c < k; ++c) {
            const int32_t* src = L.col[c];
#pragma unroll
            for (int u = 0; u < kSU; ++u)
              if (keep[u]) o[c * stride + pos[u]] = src[wave * kSChunk + u * 64 + lane];
          }
          __syncthreads();
          if (tid < k) L.col[tid] = o + tid * stride;
          place = pl;
          half = hf;
        }
      }
      if (tid == 0 && si < A.nsteps) {
        L.in[si] += n;
        L.out[si] += m;
      }
      n = m;
      rem = next;
      ++si;
      __syncthreads();
      continue;
    }

    if (kind != GSMAT_STEP_EXPAND || k + 1 > kMaxCols) break;
    // every candidate's row extents and output size
    const int nc = __popc(cmask);
    const int per = (int)((n + kSChunk - 1) / kSChunk);  // chunks of a candidate
    // kept in LDS when a chunk a wave covers them all
    const bool in_lds = nc * per <= kSW;
    const int cstride = in_lds ? per * kSChunk : (int)kSmallRows;
    int32_t* const starts = in_lds ? L.rb : (int32_t*)(A.work + A.starts);
    int32_t* const lens = in_lds ? L.P : (int32_t*)(A.work + A.lens);
    if (wave == 0 && (cmask >> (lane & 31) & 1) && lane < 32) L.cand[mbcnt(cmask)] = lane;
    if (tid < kMaxPats) L.tot[tid] = 0;
    __syncthreads();
    for (int qi = wave; qi < nc * per; qi += kSW) {
      const int c = qi / per, row0 = (qi - c * per) * kSChunk;
      const int ct = L.cand[c];
      const SmallPat q = A.pats[ct];
      const bool from_s = smask >> ct & 1;
      const int32_t* col = L.col[L.col_of[from_s ? -q.s - 1 : -q.o - 1]];
      const PredView pv = s_view(L.pred[from_s ? ct : kMaxPats + ct]);
      int32_t v[kSU], st[kSU], len[kSU];
      bool ok[kSU];
#pragma unroll
      for (int u = 0; u < kSU; ++u) {
        const int r = row0 + u * 64 + lane;
        ok[u] = r < n;
        v[u] = ok[u] ? col[r] : 0;
      }
      row_lookup_n<kSU>(pv, v, ok, st, len);
      int64_t loc = 0;
#pragma unroll
      for (int u = 0; u < kSU; ++u) {
        const int r = row0 + u * 64 + lane;  // below per * kSChunk
        starts[c * cstride + r] = st[u];
        lens[c * cstride + r] = len[u];
        loc += len[u];
      }
      loc = wave_sum(loc);
      if (lane == 0) atomicAdd(&L.tot[c], (unsigned long long)loc);
    }
    __syncthreads();
    int best = 0;  // the smallest output, the first on ties
    for (int c = 1; c < nc; ++c)
      if (L.tot[c] < L.tot[best]) best = c;
    const int64_t m = (int64_t)L.tot[best];
    tp = L.cand[best];
    const SmallPat q = A.pats[tp];
    const bool from_s = smask >> tp & 1;
    const int nv = from_s ? -q.o - 1 : -q.s - 1;
    const uint32_t next = rem & ~(1u << tp);
    if (m > 0) {
      const int64_t stride = s_stride(m);
      const bool leave = m > kSmallRows || (next == 0 && 4 * stride * (k + 1) > kSmallFin) ||
                         (A.budget > 0 && m > A.budget / (4 * (int64_t)(k + 1)));
      // offsets: four consecutive rows per thread
      int32_t len[4], st[4];
      int64_t sum = 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = tid * 4 + u;
        const bool ok = r < n;
        len[u] = ok ? lens[best * cstride + r] : 0;
        st[u] = ok ? starts[best * cstride + r] : 0;
        sum += len[u];
      }
      const int64_t inc = wave_incl_scan(sum);
      if (lane == 63) L.wsum64[wave] = inc;
      __syncthreads();
      int64_t ex = inc - sum;
#pragma unroll
      for (int w = 0; w < kSW; ++w)
        if (w < wave) ex += L.wsum64[w];
      if (leave) {
        int64_t* const offs = (int64_t*)(A.work + A.offs);
        int32_t* const sts = (int32_t*)(A.work + A.starts);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r = tid * 4 + u;
          if (r < n) {
            offs[r] = ex;
            sts[r] = st[u];
          }
          ex += len[u];
        }
        if (tid == 0) offs[n] = m;
        status = kSmallWrite;
        left_tp = tp;
        left_orient = from_s ? 0 : 1;
        left_m = m;
        left_start = sts;
        break;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = tid * 4 + u;
        if (r < n) {
          L.P[r] = (int32_t)ex;
          L.rb[r] = st[u] - (int32_t)ex;
        }
        ex += len[u];
      }
      int pl = place, hf = half;
      int32_t* const o = (int32_t*)s_place(A, 4 * stride * (k + 1), next == 0, half, &pl, &hf);
      __syncthreads();
      const int32_t* nbr = L.pred[from_s ? tp : kMaxPats + tp].nbr;
      int top = 1;
      while (top * 2 < (int)n) top *= 2;
      for (int j0 = tid; j0 < (int)m; j0 += kST * kSU) {
        int r[kSU], v[kSU];
#pragma unroll
        for (int u = 0; u < kSU; ++u) r[u] = 0;
        for (int sft = top; sft > 0; sft >>= 1) {
#pragma unroll
          for (int u = 0; u < kSU; ++u) {
            const int t = r[u] + sft;
            if (t < (int)n && L.P[t] <= j0 + u * kST) r[u] = t;
          }
        }
#pragma unroll
        for (int u = 0; u < kSU; ++u) {
          const int j = j0 + u * kST;
          v[u] = j < (int)m ? nbr[L.rb[r[u]] + j] : 0;
        }
        for (int c0 = 0; c0 < k; c0 += 4) {  // four columns' loads in flight
          int32_t x[4][kSU];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int32_t* src = L.col[min(c0 + c, k - 1)];
#pragma unroll
            for (int u = 0; u < kSU; ++u) x[c][u] = src[r[u]];
          }
#pragma unroll
          for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int u = 0; u < kSU; ++u)
              if (c0 + c < k && j0 + u * kST < (int)m) o[(c0 + c) * stride + j0 + u * kST] = x[c][u];
        }
#pragma unroll
        for (int u = 0; u < kSU; ++u)
          if (j0 + u * kST < (int)m) o[k * stride + j0 + u * kST] = v[u];
      }
      __syncthreads();
      if (tid <= k) L.col[tid] = o + tid * stride;
      if (tid == 0) {
        L.var[k] = nv;
        L.col_of[nv] = k;
      }
      place = pl;
      half = hf;
      k += 1;
      bound |= 1ull << nv;
    }
    if (tid == 0 && si < A.nsteps) {
      L.in[si] += n;
      L.out[si] += m;
    }
    n = m;
    rem = next;
    ++si;
    __syncthreads();
  }

  // The tables' stores have to be complete before the report can be seen: each
  // wave waits for its own to reach the L2, and the reporting wave's release
  // writes that back (a fence in all 16 waves cost 2 us).
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's stores are in the L2
  __syncthreads();
  if (wave == 0) {
    if (lane < kMaxCols) {
      rep->col[lane] = L.col[lane];
      rep->var[lane] = L.var[lane];
    }
    if (lane < kMaxPats + 1) {
      rep->step_in[lane] = L.in[lane];
      rep->step_out[lane] = L.out[lane];
    }
    if (lane == 0) {
      rep->n = n;
      rep->k = k;
      rep->si = si;
      rep->rem = rem;
      rep->status = status;
      rep->place = place;
      rep->tp = left_tp;
      rep->orient = left_orient;
      rep->m = left_m;
      rep->start = left_start;
    }
    report_wave(&rep->seq, seq);
  }
}

// The outputs of counted expansions: blockIdx.y is the task, the workgroups of
// a row stride over its tiles of kTile outputs.  With at most kSmallRows rows
// the tile's rows are found by two searches of a wave over the offsets (64 at
// a time, two rounds) and staged in LDS, so no split kernel and no path over
// the rows comes before the outputs.
struct SmallWriteLds {
  SmallWriteTask t;
  int32_t end[kSmallRows];  // offset of the row after, from the tile's first output
  int32_t rb[kSmallRows];   // member base, likewise
  int32_t lim[2];
};

__global__ __launch_bounds__(kBlock) void k_small_write(SmallWriteTask one,
                                                        const SmallWriteTask* __restrict__ many) {
  __shared__ SmallWriteLds L;
  const int tid = (int)threadIdx.x, lane = lane_id(), wave = wave_id();
  static_assert(sizeof(SmallWriteTask) % 4 == 0 && sizeof(SmallWriteTask) / 4 <= kBlock,
                "one word a thread");
  if (many) {
    if (tid < (int)(sizeof(SmallWriteTask) / 4))
      ((uint32_t*)&L.t)[tid] = ((const uint32_t*)(many + blockIdx.y))[tid];
  } else if (tid == 0) {
    L.t = one;
  }
  __syncthreads();
  const int n = L.t.n, k = L.t.k;
  const int64_t m = L.t.m, stride = L.t.stride;
  const int64_t* const offs = L.t.offs;
  const int32_t* const nbr = L.t.nbr;
  if (!offs) {  // an answer moved out of its work area
    for (int64_t j = (int64_t)blockIdx.x * kBlock + tid; j < m; j += (int64_t)gridDim.x * kBlock)
      for (int c = 0; c < k; ++c) L.t.out[c * stride + j] = L.t.col[c][j];
    return;
  }
  for (int64_t j0 = (int64_t)blockIdx.x * kTile; j0 < m; j0 += (int64_t)gridDim.x * kTile) {
    const int nj = (int)min((int64_t)kTile, m - j0);
    if (wave < 2) {  // the rows of the tile's first and last output
      const int64_t j = wave == 0 ? j0 : j0 + nj - 1;
      int lo = 0, len = n;  // the last row with offs <= j is in [lo, lo + len)
      while (len > 1) {
        const int step = (len + 63) / 64;
        const int i = lo + lane * step;
        const bool le = i < lo + len && offs[i] <= j;  // lanes' rows ascend: a prefix holds
        const int c = (int)__popcll(__ballot(le));
        lo += (c - 1) * step;
        len = min(step, n - lo);
      }
      if (lane == 0) L.lim[wave] = lo;
    }
    __syncthreads();
    const int r0 = L.lim[0], nr = L.lim[1] - r0 + 1;
    for (int i = tid; i < nr; i += kBlock) {
      const int64_t e = offs[r0 + i + 1] - j0;
      L.end[i] = e > kTile ? kTile : (int32_t)e;
      L.rb[i] = (int32_t)((int64_t)L.t.start[r0 + i] + (j0 - offs[r0 + i]));
    }
    __syncthreads();
    int top = 1;
    while (top * 2 < nr) top *= 2;
    constexpr int U = 4;
    int32_t* const o = L.t.out + j0;
    for (int q = tid; q < nj; q += kBlock * U) {
      int r[U], v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) r[u] = 0;
      // the first row whose end is past the output
      for (int sft = top; sft > 0; sft >>= 1) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int t = r[u] + sft;
          if (t < nr && L.end[t - 1] <= q + u * kBlock) r[u] = t;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = q + u * kBlock;
        v[u] = j < nj ? nbr[L.rb[r[u]] + j] : 0;
      }
      for (int c = 0; c < k; ++c) {
        const int32_t* src = L.t.col[c] + r0;
        int32_t x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = src[r[u]];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (q + u * kBlock < nj)
            __builtin_nontemporal_store(x[u], &o[c * stride + q + u * kBlock]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (q + u * kBlock < nj)
          __builtin_nontemporal_store(v[u], &o[k * stride + q + u * kBlock]);
    }
    __syncthreads();  // the next tile reuses the LDS
  }
}

}  // namespace

void launch_small_write(const SmallWriteTask* tasks, int n, int64_t most, double bytes,
                        hipStream_t s) {
  if (n <= 0) return;
  // enough workgroups to fill the device; few tasks take more each
  const int64_t cap = std::max<int64_t>(16, 4096 / n);
  const unsigned gx = (unsigned)std::min<int64_t>(std::max<int64_t>(ceil_div(most, kTile), 1), cap);
  const bool prof = prof_on(GSMAT_K_WRITE);
  if (prof) prof_begin(s, GSMAT_K_WRITE);
  hipLaunchKernelGGL(k_small_write, dim3(gx, (unsigned)n), dim3(kBlock), 0, s, tasks[0],
                     n > 1 ? tasks : nullptr);
  GS_HIP(hipGetLastError());
  if (prof) prof_end(s, GSMAT_K_WRITE, bytes);
}

void launch_small(const SmallStore& st, const SmallArgs* args, SmallReport* reps, int n,
                  uint32_t seq, hipStream_t s) {
  if (n <= 0) return;
  const bool prof = prof_on(GSMAT_K_OTHER);
  if (prof) prof_begin(s, GSMAT_K_OTHER);
  hipLaunchKernelGGL(k_small_join, dim3((unsigned)n), dim3(kST), 0, s, st, args, reps, seq);
  GS_HIP(hipGetLastError());
  if (prof) prof_end(s, GSMAT_K_OTHER, 0.0);
}

}  // namespace gsmat
