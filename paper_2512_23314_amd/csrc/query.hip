// Queries on a finished tree (Section 1: access, rank, select) and small
// auxiliary kernels of the build.
//
// access(i): start in level-1 block i / b1 at offset i mod b1.  In a marked
// block move to the child that holds the offset (its index is tau times the
// number of marked blocks before it, plus the child number).  In an unmarked
// block follow the pointer (t, off): the content continues at offset off + o
// of block t, or of block t+1 when that passes the end of t; both are marked,
// so the walk then descends from there.  At the last level read the leaf byte.
#include "common.hpp"
#include "internal.hpp"
#include "query.hpp"

namespace bt {

static unsigned grid_for(uint64_t n, unsigned threads, unsigned cap = 8192) {
  uint64_t g = (n + threads - 1) / threads;
  if (g == 0) g = 1;
  return (unsigned)(g < cap ? g : cap);
}

#define GRID_STRIDE(i, n)                                                        \
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); \
       i += (uint64_t)gridDim.x * blockDim.x)

// Queries are chains of dependent loads, one or two per level, so what they cost
// is latency times the length of the chain.  The level table is read at every
// step, by lanes on different levels: it lies in LDS.  Block lengths are mostly
// powers of two, where a shift replaces a 64-bit division.  Measured on a 64 MiB
// text of 96 symbols, 2^20 queries: access 82 -> 61 us, rank 337 -> 185 us, select
// 535 -> 469 us (which is bound by the lines it reads, about 100 per query).
constexpr uint32_t kMaxLevels = 64;  // block lengths are leaf tau^k < 2^64

__device__ __forceinline__ void load_levels(const QTree& q, QLevel* s_lv) {
  static_assert(sizeof(QLevel) % 8 == 0, "copied as words");
  const uint64_t* src = reinterpret_cast<const uint64_t*>(q.lv);
  uint64_t* dst = reinterpret_cast<uint64_t*>(s_lv);
  for (uint32_t k = threadIdx.x; k < q.h * (sizeof(QLevel) / 8); k += blockDim.x) dst[k] = src[k];
  __syncthreads();
}

// x / b, and the remainder in x
__device__ __forceinline__ uint64_t take_div(uint64_t& x, uint64_t b) {
  if ((b & (b - 1)) == 0) {
    const uint64_t k = x >> (63 - __builtin_clzll(b));
    x &= b - 1;
    return k;
  }
  const uint64_t k = x / b;
  x -= k * b;
  return k;
}

// Marks before block j of a level, and whether j is marked.
struct Mark {
  uint64_t before;
  bool marked;
};
__device__ __forceinline__ Mark mark_at(const QLevel& L, uint64_t j) {
  const uint64_t w = L.words[j >> 6], r = L.wrank[j >> 6];
  const uint32_t k = (uint32_t)j & 63;
  return {r + __popcll(w & ((1ull << k) - 1)), ((w >> k) & 1) != 0};
}

__global__ void k_access(QTree q, const uint64_t* __restrict__ pos, uint64_t m,
                         uint8_t* __restrict__ out, uint32_t* bad) {
  __shared__ QLevel lv[kMaxLevels];
  load_levels(q, lv);
  GRID_STRIDE(k, m) {
    uint64_t o = pos[k];
    if (o >= q.n) {
      out[k] = 0;
      *bad = 1;
      continue;
    }
    uint64_t j = take_div(o, lv[0].b);
    uint32_t l = 0;
    while (l + 1 < q.h) {
      const QLevel& L = lv[l];
      const Mark mk = mark_at(L, j);
      if (mk.marked) {
        ++l;
        j = mk.before * q.tau + take_div(o, lv[l].b);
      } else {
        const uint64_t u = j - mk.before;
        j = L.pb[u];
        o += L.po[u];
        if (o >= L.b) {
          o -= L.b;
          ++j;
        }
      }
    }
    out[k] = q.leaves[j * q.leaf_len + o];
  }
}

hipError_t launch_access(QTree t, const uint64_t* pos, uint64_t m, uint8_t* out, uint32_t* bad,
                         hipStream_t s) {
  if (!m) return hipSuccess;
  if (t.h > kMaxLevels) return hipErrorInvalidValue;
  k_access<<<grid_for(m, 256), 256, 0, s>>>(t, pos, m, out, bad);
  return hipGetLastError();
}

// The top bit of each byte of w that equals ch (exact: no carry crosses bytes).
__device__ __forceinline__ uint64_t equal_bytes(uint64_t w, uint8_t ch) {
  const uint64_t x = w ^ (0x0101010101010101ull * ch), low = 0x7F7F7F7F7F7F7F7Full;
  return ~(((x & low) + low) | x | low);
}

// Eight bytes of a leaf (unaligned).
__device__ __forceinline__ uint64_t leaf_word(const uint8_t* p) {
  uint64_t w;
  __builtin_memcpy(&w, p, 8);
  return w;
}

// Counter of width w at index idx.
__device__ __forceinline__ uint64_t narrow_at(const uint8_t* p, uint32_t w, uint64_t idx) {
  return w == 1 ? p[idx]
                : w == 2 ? reinterpret_cast<const uint16_t*>(p)[idx]
                         : reinterpret_cast<const uint32_t*>(p)[idx];
}

// Occurrences of symbol s between the starts of a marked block and of its child
// x, where j0 is its first child (which starts where it does), on level N.
__device__ __forceinline__ uint64_t child_count(const QLevel& N, uint64_t j0, uint64_t x, uint32_t S,
                                                uint32_t s) {
  if (N.acnt) return N.acnt[(j0 + x) * S + s] - N.acnt[j0 * S + s];
  return narrow_at(N.qc, N.qw, (j0 + x) * S + s);
}

// Occurrences of symbol s in block t of level l, whose right neighbour t + 1
// starts where it ends.  Counts relative to the parent give it where both have
// one parent; else t is the last child of its parent and t + 1 the first of the
// next one, and the parent's count less what lies before t is left (one more
// level in one of tau cases).  A tree's first levels hold absolute counts.
__device__ uint64_t block_occ(const QTree& q, const QLevel* lv, uint32_t l, uint64_t t, uint32_t s) {
  int64_t sub = 0;
  while (true) {
    const QLevel& L = lv[l];
    if (L.acnt) return (uint64_t)(L.acnt[(t + 1) * q.S + s] - L.acnt[t * q.S + s] - sub);
    const uint64_t mine = narrow_at(L.qc, L.qw, t * q.S + s);
    const uint64_t p = t / q.tau;
    if ((t + 1) / q.tau == p) return narrow_at(L.qc, L.qw, (t + 1) * q.S + s) - mine - sub;
    sub += mine;
    t = lv[l - 1].msel[p];
    --l;
  }
}

// rank(c, i): the walk of access.  Let D be the count before the current block
// plus what the pointers followed have shifted it by, so that the answer is D
// plus the occurrences in the current block before the offset.  Moving to child
// x adds the occurrences between the two starts; following a pointer of block j
// to offset off of block t replaces "before block j" by "before the source", which
// lies P[u] occurrences into t: D - P[u] is the new D, whatever the counts of j
// and t are.  Spilling into t + 1 adds the occurrences in t.  (Carrying the
// absolute counts of j and t instead took a climb to the nearest absolute level
// at every pointer.)
__global__ void k_rank(QTree q, const uint8_t* __restrict__ cs, const uint64_t* __restrict__ pos,
                       uint64_t m, uint64_t* __restrict__ out) {
  __shared__ QLevel lv[kMaxLevels];
  load_levels(q, lv);
  const uint32_t S = q.S;
  GRID_STRIDE(k, m) {
    const uint64_t i = pos[k];
    const uint8_t ch = cs[k];
    const int s = q.sym[ch];
    if (i > q.n) {
      out[k] = ~0ull;
      continue;
    }
    if (s < 0) {
      out[k] = 0;
      continue;
    }
    if (i == q.n) {
      out[k] = q.total[s];
      continue;
    }
    uint64_t o = i;
    uint64_t j = take_div(o, lv[0].b);
    int64_t D = lv[0].acnt[j * S + s];
    uint32_t l = 0;
    while (l + 1 < q.h) {
      const QLevel& L = lv[l];
      const Mark mk = mark_at(L, j);
      if (mk.marked) {
        const QLevel& N = lv[++l];
        const uint64_t j0 = mk.before * q.tau, x = take_div(o, N.b);
        if (x) D += (int64_t)child_count(N, j0, x, S, s);
        j = j0 + x;
      } else {
        const uint64_t u = j - mk.before;
        D -= (int64_t)narrow_at(L.pc, L.pw, u * S + s);
        j = L.pb[u];
        o += L.po[u];
        if (o >= L.b) {
          o -= L.b;
          D += (int64_t)block_occ(q, lv, l, j, s);
          ++j;
        }
      }
    }
    const uint8_t* lb = q.leaves + j * q.leaf_len;
    uint64_t r = 0;
    for (; r + 8 <= o; r += 8) D += __popcll(equal_bytes(leaf_word(lb + r), ch));
    for (; r < o; ++r) D += lb[r] == ch;
    out[k] = (uint64_t)D;
  }
}

hipError_t launch_rank(QTree t, const uint8_t* cs, const uint64_t* pos, uint64_t m, uint64_t* out,
                       hipStream_t s) {
  if (!m) return hipSuccess;
  if (t.h > kMaxLevels) return hipErrorInvalidValue;
  k_rank<<<grid_for(m, 256), 256, 0, s>>>(t, cs, pos, m, out);
  return hipGetLastError();
}

// select(c, k): the wanted occurrence is the k-th inside the current block.
// Level 1: binary search over the blocks.  Marked block: the last child with
// fewer than k occurrences before it.  Unmarked block with pointer (t, off): the
// (P[u] + k)-th of block t, or, past t's occurrences, one of block t + 1; the
// answer moves by (start of the block) - (source position).  At the leaf, scan
// its bytes.
__global__ void k_select(QTree q, const uint8_t* __restrict__ cs, const uint64_t* __restrict__ ks,
                         uint64_t m, uint64_t* __restrict__ out) {
  __shared__ QLevel lv[kMaxLevels];
  load_levels(q, lv);
  const uint32_t S = q.S;
  GRID_STRIDE(qi, m) {
    const uint8_t ch = cs[qi];
    uint64_t k = ks[qi];
    const int s = q.sym[ch];
    if (s < 0 || k == 0 || k > q.total[s]) {
      out[qi] = ~0ull;
      continue;
    }
    uint64_t lo = 0, hi = lv[0].c;
    while (hi - lo > 1) {
      const uint64_t mid = (lo + hi) >> 1;
      if (lv[0].acnt[mid * S + s] < k) lo = mid; else hi = mid;
    }
    uint64_t j = lo;
    k -= lv[0].acnt[j * S + s];
    uint32_t l = 0;
    uint64_t shift = 0;
    while (l + 1 < q.h) {
      const QLevel& L = lv[l];
      const Mark mk = mark_at(L, j);
      if (mk.marked) {
        const QLevel& N = lv[++l];
        const uint64_t j0 = mk.before * q.tau;
        uint64_t nch = N.c - j0;
        if (nch > q.tau) nch = q.tau;
        // the last child with fewer than k before it, by quarters: a round's three
        // counts leave together.  (Four counts at a time from the first child on
        // took lines in proportion to the arity: 2^18 queries on 16 MiB, 250 symbols,
        // tau 16 0.130 ms, now 0.093; tau 64, 200 symbols 0.30, now 0.107.)
        uint64_t x = 0, before = 0;
        while (nch > 1) {
          const uint64_t step = (nch + 3) / 4;
          uint64_t v[3];
#pragma unroll
          for (int e = 0; e < 3; ++e)
            v[e] = (e + 1) * step < nch ? child_count(N, j0, x + (e + 1) * step, S, s) : ~0ull;
          uint64_t skip = 0;
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (v[e] < k) {  // (counts do not decrease)
              before = v[e];
              skip = (e + 1) * step;
            }
          x += skip;
          nch = nch - skip < step ? nch - skip : step;
        }
        j = j0 + x;
        k -= before;
      } else {
        const uint64_t u = j - mk.before;
        const uint64_t t = L.pb[u];
        const uint64_t off = L.po[u], sj = L.st[j];
        k += narrow_at(L.pc, L.pw, u * S + s);
        const uint64_t st = L.st[t];
        // (a source that starts with t ends with it)
        const bool next = off && t + 1 < L.c && L.st[t + 1] == st + L.b;
        shift += sj - (st + off);
        j = t;
        if (next) {
          const uint64_t occ = block_occ(q, lv, l, t, s);
          if (occ < k) {
            k -= occ;
            j = t + 1;
          }
        }
      }
    }
    const QLevel& LH = lv[q.h - 1];
    uint64_t need = k;
    const uint8_t* lb = q.leaves + j * q.leaf_len;
    uint64_t res = ~0ull;
    const uint64_t rest = q.tstart + q.n - LH.st[j];
    const uint64_t llen = rest < q.leaf_len ? rest : q.leaf_len;
    uint64_t o = 0;
    for (; o + 8 <= llen; o += 8) {  // the word that holds it
      const uint32_t n = (uint32_t)__popcll(equal_bytes(leaf_word(lb + o), ch));
      if (n >= need) break;
      need -= n;
    }
    for (; o < llen; ++o) {
      if (lb[o] == ch && --need == 0) {
        res = LH.st[j] + o + shift - q.tstart;
        break;
      }
    }
    out[qi] = res;
  }
}

hipError_t launch_select(QTree t, const uint8_t* cs, const uint64_t* ks, uint64_t m, uint64_t* out,
                         hipStream_t s) {
  if (!m) return hipSuccess;
  if (t.h > kMaxLevels) return hipErrorInvalidValue;
  k_select<<<grid_for(m, 256), 256, 0, s>>>(t, cs, ks, m, out);
  return hipGetLastError();
}

__global__ void k_rank_empty(const uint64_t* pos, uint64_t m, uint64_t* out) {
  GRID_STRIDE(k, m) out[k] = pos[k] == 0 ? 0 : ~0ull;
}

hipError_t launch_rank_empty(const uint64_t* pos, uint64_t m, uint64_t* out, hipStream_t s) {
  if (!m) return hipSuccess;
  k_rank_empty<<<grid_for(m, 256), 256, 0, s>>>(pos, m, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- auxiliary

// Each thread keeps its own 256-bit set in LDS column t (word k of thread t at
// s[k][t]: a wave's lanes touch 64 different banks); 16 bytes per load.  The
// columns are then ORed and merged into the global set, which is read first so
// that most workgroups skip the atomic.
__global__ __launch_bounds__(256) void k_byte_presence(const uint8_t* __restrict__ T, uint64_t n,
                                                       uint32_t* __restrict__ seen) {
  __shared__ uint32_t s[8][256];
  const int t = threadIdx.x;
#pragma unroll
  for (int k = 0; k < 8; ++k) s[k][t] = 0;
  const auto add = [&](uint32_t c) { atomicOr(&s[c >> 5][t], 1u << (c & 31)); };
  const uint64_t mis = reinterpret_cast<uintptr_t>(T) & 15;
  const uint64_t head = mis ? (16 - mis < n ? 16 - mis : n) : 0;
  const uint64_t body = (n - head) / 16;
  const uint4* __restrict__ B = reinterpret_cast<const uint4*>(T + head);
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + t; i < body; i += (uint64_t)gridDim.x * 256) {
    const uint4 v = B[i];
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int k = 0; k < 4; ++k) add((w[q] >> (8 * k)) & 0xFFu);
  }
  if (blockIdx.x == 0) {
    for (uint64_t i = t; i < head; i += 256) add(T[i]);
    for (uint64_t i = head + body * 16 + t; i < n; i += 256) add(T[i]);
  }
  __syncthreads();
  // word k = t / 32 over the 256 columns: eight per lane, then 32 lanes
  const int k = t >> 5, part = t & 31;
  uint32_t m = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) m |= s[k][part * 8 + e];
#pragma unroll
  for (int d = 16; d >= 1; d >>= 1) m |= __shfl_xor(m, d);
  if (part == 0 && m && (seen[k] | m) != seen[k]) atomicOr(&seen[k], m);
}

hipError_t launch_byte_presence(const uint8_t* T, uint64_t n, uint32_t* seen, hipStream_t s) {
  if (!n) return hipSuccess;
  k_byte_presence<<<grid_for((n + 15) / 16, 256, 1024), 256, 0, s>>>(T, n, seen);
  return hipGetLastError();
}

__global__ void k_last_block_len(LevelDev lv, TextsDev tx, const uint64_t* tfirst,
                                 const uint64_t* tcount, uint64_t* out) {
  GRID_STRIDE(t, tx.T) {
    if (!tcount[t]) {
      out[t] = 0;
      continue;
    }
    const uint64_t j = tfirst[t] + tcount[t] - 1;
    const uint64_t st = lv.st[j], te = tx.tend[t];
    out[t] = te - st < lv.b ? te - st : lv.b;
  }
}

hipError_t launch_last_block_len(const LevelDev& lv, const TextsDev& tx, const uint64_t* tfirst,
                                 const uint64_t* tcount, uint64_t* out, hipStream_t s) {
  k_last_block_len<<<grid_for(tx.T, 256), 256, 0, s>>>(lv, tx, tfirst, tcount, out);
  return hipGetLastError();
}

__global__ void k_text_deltas(const uint64_t* scanned, const uint64_t* tfirst,
                              const uint64_t* tcount, uint32_t T, uint64_t* out) {
  GRID_STRIDE(t, T) out[t] = scanned[tfirst[t] + tcount[t]] - scanned[tfirst[t]];
}

hipError_t launch_text_deltas(const uint64_t* scanned, const uint64_t* tfirst,
                              const uint64_t* tcount, uint32_t T, uint64_t* out, hipStream_t s) {
  k_text_deltas<<<grid_for(T, 256), 256, 0, s>>>(scanned, tfirst, tcount, T, out);
  return hipGetLastError();
}

}  // namespace bt
