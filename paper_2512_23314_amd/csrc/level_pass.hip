// The passes over a level's blocks between its scans: runs, scan segments,
// marks, the split into the next level and the level's outputs (Section 4.1).
// Each that needs a prefix sum makes its inputs, sums them and uses the result in
// one launch (scan_pass.hpp).  Before that a level took about 49 launches and two
// read-backs, 5.6 us each on the host whatever the blocks: 391 of them, 2.2 ms,
// for a 4 KiB text of 9 levels, and 3 ms of a 12 ms build at 256 MiB.
#include "common.hpp"
#include "internal.hpp"
#include "scan_pass.hpp"

namespace bt {

static unsigned grid_for(uint64_t n, unsigned threads, unsigned cap = 8192) {
  uint64_t g = (n + threads - 1) / threads;
  if (g == 0) g = 1;
  return (unsigned)(g < cap ? g : cap);
}
static unsigned pass_grid(uint64_t n) { return (unsigned)scan_pass_tiles(n); }

// Launch kernel<ROWS> for n elements.
#define BT_PASS(kernel, n, ...)                                                             \
  do {                                                                                      \
    const unsigned g_ = pass_grid(n);                                                       \
    const int r_ = scan_pass_rows(n);                                                       \
    if (r_ == 1) kernel<1><<<g_, kPassThreads, 0, s>>>(__VA_ARGS__);                        \
    else if (r_ == 2) kernel<2><<<g_, kPassThreads, 0, s>>>(__VA_ARGS__);                   \
    else kernel<8><<<g_, kPassThreads, 0, s>>>(__VA_ARGS__);                                \
  } while (0)

#define GRID_STRIDE(i, n)                                                        \
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); \
       i += (uint64_t)gridDim.x * blockDim.x)

__device__ __forceinline__ uint64_t block_len(const LevelDev& lv, const TextsDev& tx, uint64_t j) {
  const uint64_t st = lv.st[j];
  const uint64_t te = tx.tend[lv.text[j]];
  return te - st < lv.b ? te - st : lv.b;
}

// ---------------------------------------------------------------- runs

// Runs of a level: maximal sequences of consecutive blocks of one text.
struct RunPass {
  const uint64_t* st;
  const uint32_t* text;
  uint64_t c, b;
  TextsDev tx;
  uint32_t* run;
  uint64_t *rs, *re;
  uint32_t* rtext;
  uint64_t* total_out;
  __device__ bool head(uint64_t j) const {
    return j == 0 || text[j] != text[j - 1] || st[j] != st[j - 1] + b;
  }
  __device__ void value(uint64_t j, uint64_t* v) const { v[0] = head(j) ? 1 : 0; }
  __device__ void apply(uint64_t j, const uint64_t* ex, const uint64_t* v) const {
    const uint64_t r = ex[0] + v[0] - 1;
    run[j] = (uint32_t)r;
    if (v[0]) {
      rs[r] = st[j];
      rtext[r] = text[j];
    }
    if (j + 1 == c || head(j + 1)) {
      const uint64_t te = tx.tend[text[j]];
      re[r] = st[j] + (te - st[j] < b ? te - st[j] : b);
    }
  }
  __device__ void total(const uint64_t* sum) const {
    if (total_out) *total_out = sum[0];
  }
};
template <int ROWS>
__global__ __launch_bounds__(kPassThreads) void k_runs(RunPass p, ScanDev sd) {
  scan_pass<1, 1u, ROWS>(p.c, sd, p);
}

hipError_t launch_runs(const uint64_t* st, const uint32_t* text, uint64_t c, uint64_t b,
                       const TextsDev& tx, uint32_t* run, uint64_t* rs, uint64_t* re,
                       uint32_t* rtext, uint64_t* total, const ScanDev& sd, hipStream_t s) {
  const RunPass p{st, text, c, b, tx, run, rs, re, rtext, total};
  BT_PASS(k_runs, c, p, sd);
  return hipGetLastError();
}

// ---------------------------------------------------------------- scan segments
//
// The probe scan walks "segments": ranges of window starts, each inside one run.
// A window whose content also occurs earlier can never be the leftmost
// occurrence of anything, so the previous level's results prune segments.  For
// a marked parent block P (all windows of this level start inside some parent):
//   - if the pair (P, P+1) has an earlier occurrence, every window starting in
//     P lies inside a copy of it (windows are at most one parent long);
//   - if the pair (P-1, P) has an earlier occurrence, or P itself does, every
//     window that ends inside P is a copy.
// Entries describe parents (or whole texts where there is no parent level) as
// [a, e) plus these two facts.
//
// Phase 1: an entry's windows.  An entry whose starts continue those of the
// previous entry (same run, first start one past the previous entry's last:
// adjacent parents that no fact cut apart) joins its segment: per entry, the
// scan's tiles would cross several of them at the lower levels.
// Phase 2: a window of length b that starts in block Q lies inside the pair
// (Q, Q+1), so if that pair occurs earlier, so does the window: Q contributes no
// window starts.  Consecutive blocks of a run that keep their starts join.
// Both: segment g = window starts [ws[g], ...) numbered from woff[g], bounded by
// the run end sre[g], of text stext[g]; segn = {segments, windows}, woff[segments]
// = windows.

struct SegPiece {
  uint64_t lo, cnt, re;
  uint32_t t, r;
};

__device__ __forceinline__ uint64_t shortest_key(const PhaseArgs& a, uint32_t t) {
  const uint64_t oL = a.odd.L[t];
  return oL && oL < a.Lmain ? oL : a.Lmain;
}

struct EntryPieces {
  const PhaseArgs& a;
  const SegDev& sg;
  __device__ SegPiece piece(uint64_t k) const {
    SegPiece p;
    p.r = a.lv.run[sg.echild[k]];
    p.t = a.lv.rtext[p.r];
    p.re = a.lv.re[p.r];
    const uint64_t Lmin = shortest_key(a, p.t), L = a.Lmain;
    const uint8_t f = sg.ef[k];
    const uint64_t ee = sg.ee[k];
    p.lo = sg.ea[k];
    if (f & kSkipInterior) {
      const uint64_t x = ee + 1 > L ? ee + 1 - L : 0;  // first start crossing e
      if (x > p.lo) p.lo = x;
    }
    p.cnt = 0;
    if (a.odd.nkeys[p.t] && !(f & kSkipCross) && p.re >= Lmin) {
      uint64_t hi = ee - 1;
      if (p.re - Lmin < hi) hi = p.re - Lmin;
      if (hi >= p.lo && ee > p.lo) p.cnt = hi - p.lo + 1;
    }
    return p;
  }
  __device__ bool joins(const SegPiece& q, const SegPiece& p) const {
    return q.cnt && q.r == p.r && q.lo + q.cnt == p.lo;
  }
};

struct BlockPieces {
  const PhaseArgs& a;
  const uint8_t* pf;
  __device__ SegPiece piece(uint64_t Q) const {
    SegPiece p;
    p.r = a.lv.run[Q];
    p.t = a.lv.text[Q];
    p.re = a.lv.re[p.r];
    const uint64_t Lmin = shortest_key(a, p.t);
    p.lo = a.lv.st[Q];
    p.cnt = 0;
    if (a.odd.nkeys[p.t] && !(pf[Q] & 1) && p.re >= Lmin) {
      uint64_t hi = p.lo + block_len(a.lv, a.tx, Q) - 1;
      if (p.re - Lmin < hi) hi = p.re - Lmin;
      if (hi >= p.lo) p.cnt = hi - p.lo + 1;
    }
    return p;
  }
  // (a block whose starts stop short of its end is the run's last with any)
  __device__ bool joins(const SegPiece& q, const SegPiece& p) const { return q.cnt && q.r == p.r; }
};

template <class Pieces>
struct SegPass {
  Pieces src;
  SegOut o;
  uint64_t* wst;
  __device__ void value(uint64_t k, uint64_t* v) const {
    const SegPiece p = src.piece(k);
    v[0] = p.cnt;
    v[1] = p.cnt && !(k > 0 && src.joins(src.piece(k - 1), p)) ? 1 : 0;
  }
  __device__ void apply(uint64_t k, const uint64_t* ex, const uint64_t* v) const {
    if (o.tseg && v[0]) {
      // tiles whose first window is one of this piece's
      const uint32_t g = (uint32_t)(ex[1] + v[1] - 1);
      for (uint64_t t = (ex[0] + kProbeTile - 1) / kProbeTile; t * kProbeTile < ex[0] + v[0]; ++t) o.tseg[t] = g;
    }
    if (!v[1]) return;
    const SegPiece p = src.piece(k);
    const uint64_t g = ex[1];
    o.woff[g] = ex[0];
    o.ws[g] = p.lo;
    o.sre[g] = p.re;
    o.stext[g] = p.t;
  }
  __device__ void total(const uint64_t* sum) const {
    o.segn[0] = sum[1];
    o.segn[1] = sum[0];
    o.woff[sum[1]] = sum[0];
    if (wst) *wst = sum[0];
  }
};

template <int ROWS>
__global__ __launch_bounds__(kPassThreads) void k_entry_segs(PhaseArgs a, SegDev sg, SegOut o,
                                                             uint64_t* wst, ScanDev sd) {
  scan_pass<2, 2u, ROWS>(sg.E, sd, SegPass<EntryPieces>{{a, sg}, o, wst});
}
template <int ROWS>
__global__ __launch_bounds__(kPassThreads) void k_block_segs(PhaseArgs a, const uint8_t* pf, SegOut o,
                                                             uint64_t* wst, ScanDev sd) {
  scan_pass<2, 2u, ROWS>(a.lv.c, sd, SegPass<BlockPieces>{{a, pf}, o, wst});
}

hipError_t launch_entry_segs(const PhaseArgs& a, const SegDev& sg, const SegOut& o, uint64_t* wst,
                             const ScanDev& sd, hipStream_t s) {
  BT_PASS(k_entry_segs, sg.E, a, sg, o, wst, sd);
  return hipGetLastError();
}
hipError_t launch_block_segs(const PhaseArgs& a, const uint8_t* pf, const SegOut& o, uint64_t* wst,
                             const ScanDev& sd, hipStream_t s) {
  BT_PASS(k_block_segs, a.lv.c, a, pf, o, wst, sd);
  return hipGetLastError();
}

// ---------------------------------------------------------------- marks (a5)

__device__ __forceinline__ void host_totals(const TextStep& ts, uint64_t unmarked, uint64_t next_runs) {
  ts.h_totals[0] = unmarked;
  ts.h_totals[1] = next_runs;
  ts.h_totals[2] = ts.totals[2];  // this level's runs
  if (ts.seen)
    for (int k = 0; k < 4; ++k) ts.h_totals[3 + k] = ts.seen[k];
}

// After phase 1: the marks (a block's pair or its left neighbour's pair is
// leftmost, or it has no consecutive neighbour), the pair facts (bit 0 of pf[j]:
// the pair (j, j+1) occurs earlier), the unmarked ranks that pointers are stored
// by, the children's ranks, and the number of runs of the next level (the
// children of a maximal group of consecutive marked blocks of one run are
// consecutive blocks of one run).
struct MarkPass {
  PhaseArgs a;
  uint64_t bn;
  uint8_t *marked, *pf;
  uint64_t *uoff, *cs, *totals;
  uint32_t* rnum;
  TextStep ts;
  __device__ bool leftmost(uint64_t q) const {
    return a.k.slot[q] != kNoKey && a.k.lm[q] == a.lv.st[q];
  }
  __device__ bool mark(uint64_t j) const {
    const LevelDev& lv = a.lv;
    if (leftmost(j) || (j > 0 && leftmost(j - 1))) return true;
    const uint32_t r = lv.run[j];
    const bool left = j > 0 && lv.run[j - 1] == r;
    const bool right = j + 1 < lv.c && lv.run[j + 1] == r;
    return !left && !right;
  }
  __device__ void value(uint64_t j, uint64_t* v) const {
    const LevelDev& lv = a.lv;
    const bool m = mark(j);
    marked[j] = m ? 1 : 0;
    pf[j] = (a.k.slot[j] != kNoKey && a.k.lm[j] < lv.st[j]) ? 1 : 0;
    v[0] = m ? 0 : 1;
    v[1] = (m && (j == 0 || lv.run[j - 1] != lv.run[j] || !mark(j - 1))) ? 1 : 0;
    v[2] = m ? (block_len(lv, a.tx, j) + bn - 1) / bn : 0;
  }
  __device__ void apply(uint64_t j, const uint64_t* ex, const uint64_t* v) const {
    uoff[j] = ex[0];
    cs[j] = ex[2];
    if (rnum) rnum[j] = (uint32_t)(ex[1] + v[1] - 1);
  }
  __device__ void total(const uint64_t* sum) const {
    uoff[a.lv.c] = sum[0];
    cs[a.lv.c] = sum[2];
    totals[0] = sum[0];
    totals[1] = sum[1];
    if (!rnum) return;
    // one text: the step of TextPass (nothing enters below its first level)
    ts.ncount[0] = sum[2];
    ts.nfirst[0] = 0;
    ts.nfirst[1] = sum[2];
    ts.woff[0] = 0;
    ts.woff[1] = (a.lv.c + 63) / 64;
    ts.h_ncount[0] = sum[2];
    ts.h_tu[0] = sum[0];
    host_totals(ts, sum[0], sum[1]);
  }
};
template <int ROWS>
__global__ __launch_bounds__(kPassThreads) void k_marks(MarkPass p, FillList f, ScanDev sd) {
  scan_pass<3, 3u, ROWS>(p.a.lv.c, sd, p);
  fill_share(f, (uint64_t)blockIdx.x * kPassThreads + threadIdx.x, (uint64_t)gridDim.x * kPassThreads);
}

hipError_t launch_marks(const PhaseArgs& a, uint64_t bn, uint8_t* marked, uint8_t* pf, uint64_t* uoff,
                        uint64_t* cs, uint64_t* totals, uint32_t* rnum, const TextStep& ts,
                        const FillList& fill, const ScanDev& sd, hipStream_t s) {
  if (rnum && a.tx.T != 1) return hipErrorInvalidValue;
  const MarkPass p{a, bn, marked, pf, uoff, cs, totals, rnum, ts};
  BT_PASS(k_marks, a.lv.c, p, fill, sd);
  return hipGetLastError();
}

// Per text: blocks of the next level (children, or the text's own blocks where
// it enters there), their prefix, the words of the marks and their prefix, the
// unmarked blocks.  The host's copies go straight to pinned memory.
struct TextPass {
  TextsDev tx;
  TextStep ts;
  __device__ void value(uint64_t t, uint64_t* v) const {
    const uint64_t n = ts.tcount[t], f = ts.tfirst[t], e = f + n;
    uint64_t nc = ts.cs[e] - ts.cs[f];
    if (ts.estep[t] == ts.enter) nc += (tx.tend[t] - tx.tstart[t] + ts.bn - 1) / ts.bn;
    v[0] = nc;
    v[1] = (n + 63) / 64;
    ts.h_tu[t] = ts.uoff[e] - ts.uoff[f];
    ts.h_ncount[t] = nc;
  }
  __device__ void apply(uint64_t t, const uint64_t* ex, const uint64_t* v) const {
    ts.ncount[t] = v[0];
    ts.nfirst[t] = ex[0];
    ts.woff[t] = ex[1];
  }
  __device__ void total(const uint64_t* sum) const {
    ts.nfirst[tx.T] = sum[0];
    ts.woff[tx.T] = sum[1];
    host_totals(ts, ts.totals[0], ts.totals[1]);
  }
};
template <int ROWS>
__global__ __launch_bounds__(kPassThreads) void k_texts(TextPass p, ScanDev sd) {
  scan_pass<2, 0u, ROWS>(p.tx.T, sd, p);
}

hipError_t launch_texts(const TextsDev& tx, const TextStep& ts, const ScanDev& sd, hipStream_t s) {
  const TextPass p{tx, ts};
  BT_PASS(k_texts, tx.T, p, sd);
  return hipGetLastError();
}

// ---------------------------------------------------------------- pointers (a7), split (a8)

// Block j (unmarked): its pointer, and the device-side check of its target.
__device__ __forceinline__ void write_pointer(const PhaseArgs& a, uint64_t j, const uint8_t* marked,
                                              const uint64_t* uoff, const uint64_t* tfirst,
                                              uint64_t* pb, uint64_t* po, uint32_t* err) {
  const LevelDev& lv = a.lv;
  const uint64_t p = a.k.lm[j];
  const uint32_t tx = lv.text[j];
  // the target block: the last one starting at or before p, searched among
  // the blocks of j's own text before j (an occurrence lies in its text and
  // ends by j's start; the checks below catch anything else)
  uint64_t lo = tfirst[tx], hi = j;
  while (hi - lo > 1) {
    const uint64_t mid = (lo + hi) >> 1;
    if (lv.st[mid] <= p) lo = mid; else hi = mid;
  }
  const uint64_t t = lo;
  const uint64_t lj = block_len(lv, a.tx, j), lt = block_len(lv, a.tx, t);
  bool ok = lv.st[t] <= p && p < lv.st[t] + lt && marked[t] && lv.text[t] == tx &&
            p + lj <= lv.st[j];
  if (ok && p + lj > lv.st[t] + lt)
    ok = t + 1 < lv.c && lv.run[t + 1] == lv.run[t] && marked[t + 1];
  if (!ok) *err = 1;
  const uint64_t u = uoff[j];
  pb[u] = t - tfirst[tx];
  po[u] = p - lv.st[t];
}

__global__ void k_pointers(PhaseArgs a, const uint8_t* marked, const uint64_t* uoff,
                           const uint64_t* tfirst, uint64_t* pb, uint64_t* po, uint32_t* err) {
  GRID_STRIDE(j, a.lv.c) {
    if (!marked[j]) write_pointer(a, j, marked, uoff, tfirst, pb, po, err);
  }
}

hipError_t launch_pointers(const PhaseArgs& a, const uint8_t* marked, const uint64_t* uoff,
                           const uint64_t* tfirst, uint64_t* ptr_block, uint64_t* ptr_off,
                           uint32_t* err, hipStream_t s) {
  k_pointers<<<grid_for(a.lv.c, 256), 256, 0, s>>>(a, marked, uoff, tfirst, ptr_block, ptr_off,
                                                    err);
  return hipGetLastError();
}

// The marks of each text packed into its own words, one wave per word, and the
// marks before each word: its first block's index in the text less the unmarked
// blocks before it.  Wave gw of nw.
__device__ __forceinline__ void store_marks(const uint8_t* marked, const StoreMarks& m, uint64_t gw,
                                            uint64_t nw) {
  const int lane = lane_id();
  for (uint64_t wi = gw; wi < m.nwords; wi += nw) {
    uint64_t lo = 0, hi = m.T;
    while (hi - lo > 1) {
      const uint64_t mid = (lo + hi) >> 1;
      if (m.woff[mid] <= wi) lo = mid; else hi = mid;
    }
    // (texts with no words share an offset with the next: the last one is taken)
    const uint64_t j = (wi - m.woff[lo]) * 64, f = m.tfirst[lo];
    const uint64_t word = __ballot(j + lane < m.tcount[lo] && marked[f + j + lane]);
    if (lane == 0) {
      m.words[wi] = word;
      m.wrank[wi] = j - (m.uoff[f + j] - m.uoff[f]);
    }
  }
}

// Marked blocks: their children (the next level's blocks, each with its parent's
// facts and, for one text, its run) and their scan entry; unmarked ones (with pb):
// their pointer.  After a phase 2 over all blocks (blocks != 0) a block's own
// earlier occurrence is a fact too.  Then the stored marks, and the next level's
// scratch cleared: each took a launch of its own, with the runs and (one text) the
// per-text counts five a level.
// WIDE (an arity of kWideSplit or more): a wave writes the children of one of its
// blocks after another, 64 together; with fewer children a thread writes its own
// block's.  A 16 MiB text, tau 65536: 2.92 -> 1.1 ms; tau 1024: 0.71 -> 0.31;
// tau 64: 0.47 -> 0.44.
constexpr uint64_t kWideSplit = 64;
template <bool WIDE>
__global__ __launch_bounds__(256) void k_split(PhaseArgs a, const uint8_t* pf, const uint64_t* cs,
                                               const uint64_t* ntfirst, uint64_t bn, uint32_t blocks,
                                               const uint32_t* rnum, NextLevel o, StoreMarks m,
                                               uint64_t* pb, uint64_t* po, uint32_t* err, FillList f) {
  const LevelDev lv = a.lv;
  // block j: its pointer, or its entry and what `children` and `runs` do with its nk
  // children from `base` on
  const auto block = [&](uint64_t j, auto&& children, auto&& runs) {
    if (!a.marked[j]) {
      if (pb) write_pointer(a, j, a.marked, m.uoff, m.tfirst, pb, po, err);
      return;
    }
    const uint32_t t = lv.text[j];
    const uint64_t c0 = cs[j], nk = cs[j + 1] - c0, st = lv.st[j], te = a.tx.tend[t];
    const uint64_t end = st + (te - st < lv.b ? te - st : lv.b);
    const uint64_t base = ntfirst[t] + (c0 - cs[m.tfirst[t]]);
    const bool again = blocks && a.k.slot[j] != kNoKey && a.k.lm[j] < st;
    uint8_t fl = 0;
    if (pf[j] & 1) fl |= kSkipCross;
    if (again || (j > 0 && (pf[j - 1] & 1))) fl |= kSkipInterior;
    children(base, nk, st, t, fl);
    const uint64_t e = j - m.uoff[j];
    o.ea[e] = st;
    o.ee[e] = end;
    o.ef[e] = fl;
    o.echild[e] = base;
    if (o.run) {
      const uint32_t r = rnum[j], here = lv.run[j];
      runs(base, nk, r);
      if (j == 0 || lv.run[j - 1] != here || !a.marked[j - 1]) {
        o.rs[r] = st;
        o.rtext[r] = t;
      }
      if (j + 1 == lv.c || lv.run[j + 1] != here || !a.marked[j + 1]) o.re[r] = end;
    }
  };
  const auto child = [&](uint64_t base, uint64_t k, uint64_t nk, uint64_t st, uint32_t t, uint8_t fl) {
    o.st[base + k] = st + k * bn;
    o.text[base + k] = t;
    o.cflag[base + k] = fl ? fl | (k + 1 == nk ? kLastChild : 0) : 0;
  };
  if (WIDE) {
    const uint64_t lane = lane_id();
    for (uint64_t j0 = (uint64_t)blockIdx.x * 256 + (threadIdx.x & ~63u); j0 < lv.c; j0 += (uint64_t)gridDim.x * 256) {
      uint64_t base = 0, nk = 0, st = 0;
      uint32_t t = 0, fl = 0, r = 0;
      if (j0 + lane < lv.c)
        block(j0 + lane,
              [&](uint64_t base_, uint64_t nk_, uint64_t st_, uint32_t t_, uint8_t fl_) {
                base = base_, nk = nk_, st = st_, t = t_, fl = fl_;
              },
              [&](uint64_t, uint64_t, uint32_t r_) { r = r_; });
      for (uint64_t bal = __ballot(nk != 0); bal; bal &= bal - 1) {
        const uint32_t src = (uint32_t)(__ffsll((unsigned long long)bal) - 1);
        const uint64_t sb = shfl64(base, src), sn = shfl64(nk, src), ss = shfl64(st, src);
        const uint32_t tt = __shfl(t, (int)src), ff = __shfl(fl, (int)src), rr = __shfl(r, (int)src);
        for (uint64_t k = lane; k < sn; k += 64) {
          child(sb, k, sn, ss, tt, (uint8_t)ff);
          if (o.run) o.run[sb + k] = rr;
        }
      }
    }
  } else {
    GRID_STRIDE(j, lv.c)
      block(j,
            [&](uint64_t base, uint64_t nk, uint64_t st, uint32_t t, uint8_t fl) {
              for (uint64_t k = 0; k < nk; ++k) child(base, k, nk, st, t, fl);
            },
            [&](uint64_t base, uint64_t nk, uint32_t r) {
              for (uint64_t k = 0; k < nk; ++k) o.run[base + k] = r;
            });
  }
  store_marks(a.marked, m, (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6),
              (uint64_t)gridDim.x * 4);
  fill_share(f, (uint64_t)blockIdx.x * 256 + threadIdx.x, (uint64_t)gridDim.x * 256);
}

hipError_t launch_split(const PhaseArgs& a, const uint8_t* pf, const uint64_t* cs,
                        const uint64_t* ntfirst, uint64_t bn, uint32_t blocks, const uint32_t* rnum,
                        const NextLevel& o, const StoreMarks& m, uint64_t* pb, uint64_t* po,
                        uint32_t* err, const FillList& fill, hipStream_t s) {
  // (a level may be far larger than the one above where texts enter)
  const uint64_t by_fill = fill.total() / (4 * 256 * 16);
  const unsigned g = grid_for(a.lv.c, 256), gf = by_fill < 4096 ? (unsigned)by_fill : 4096u;
  const unsigned grid = g > gf ? g : gf;
  if (a.lv.b / bn >= kWideSplit)
    k_split<true><<<grid, 256, 0, s>>>(a, pf, cs, ntfirst, bn, blocks, rnum, o, m, pb, po, err, fill);
  else
    k_split<false><<<grid, 256, 0, s>>>(a, pf, cs, ntfirst, bn, blocks, rnum, o, m, pb, po, err, fill);
  return hipGetLastError();
}

// Texts whose level 1 is the next level: their blocks and one entry each, from
// entry `base` on (whole text, nothing skipped).  Several workgroups take a text of
// many blocks (a root of many: s_hint, a small root_block_len): with one alone, a
// 256 MiB text whose 2^24 root blocks are its leaves took 4.4 ms, now 0.98.
__global__ void k_enter(const uint32_t* ids, TextsDev tx, uint64_t bn, const uint64_t* ntfirst,
                        uint64_t base, NextLevel o) {
  const uint32_t t = ids[blockIdx.x];
  const uint64_t ts = tx.tstart[t], te = tx.tend[t];
  const uint64_t nb = (te - ts + bn - 1) / bn;
  const uint64_t first = ntfirst[t];
  for (uint64_t k = (uint64_t)blockIdx.y * blockDim.x + threadIdx.x; k < nb; k += (uint64_t)gridDim.y * blockDim.x) {
    o.st[first + k] = ts + k * bn;
    o.text[first + k] = t;
    o.cflag[first + k] = 0;
    if (o.run) o.run[first + k] = 0;  // one text: one run
  }
  if (blockIdx.y == 0 && threadIdx.x == 0) {
    const uint64_t e = base + blockIdx.x;
    o.ea[e] = ts;
    o.ee[e] = te;
    o.ef[e] = 0;
    o.echild[e] = first;
    if (o.run) {
      o.rs[0] = ts;
      o.re[0] = te;
      o.rtext[0] = t;
    }
  }
}

hipError_t launch_enter(const uint32_t* ids, uint32_t E, uint64_t most, const TextsDev& tx, uint64_t bn,
                        const uint64_t* ntfirst, uint64_t base, const NextLevel& o, hipStream_t s) {
  if (!E) return hipSuccess;
  const unsigned threads = most <= 64 ? 64 : 256;
  const uint64_t want = (most + 4 * threads - 1) / (4 * threads), cap = E < 4096 ? 4096 / E : 1;
  const unsigned y = (unsigned)(want < 1 ? 1 : want < cap ? want : cap);
  k_enter<<<dim3(E, y), threads, 0, s>>>(ids, tx, bn, ntfirst, base, o);
  return hipGetLastError();
}

// ---------------------------------------------------------------- outputs

__global__ __launch_bounds__(256) void k_store_marks(const uint8_t* marked, StoreMarks m) {
  store_marks(marked, m, (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6),
              (uint64_t)gridDim.x * 4);
}

hipError_t launch_store_marks(const uint8_t* marked, const StoreMarks& m, hipStream_t s) {
  if (!m.nwords) return hipSuccess;
  k_store_marks<<<grid_for(m.nwords, 4, 16384), 256, 0, s>>>(marked, m);
  return hipGetLastError();
}

}  // namespace bt
