// One level of block-tree construction (Section 4.1): both phases, the split
// into the next level, and the level's outputs.
//
// Phase 1 (a3-a5): the key of every pair of consecutive blocks goes into an
// open-addressing table; every window of length 2b inside a run of consecutive
// blocks is fingerprinted from the prefix fingerprints and probed; a hit at
// position i lowers the slot's smallest position with atomicMin.  Phase 2
// (a6-a7) does the same for unmarked blocks with windows of length b.  Keys
// with the same fingerprint share a slot, so a slot's minimum is the leftmost
// position with that fingerprint; each key then compares its bytes with that
// position (a4 verification).  A mismatch -- a fingerprint collision -- sends
// the key to an exact fallback scan that walks the text from just past the
// false hit and verifies every further hit, so the result is the leftmost
// occurrence whatever the hash does.
//
// Only windows inside runs are scanned: for tau >= 2 the leftmost occurrence in
// T of any string no longer than b_{l-1} lies inside a run of level l (it is
// covered by two consecutive marked blocks of level l-1, whose children are
// present), so "leftmost on this level" and "leftmost in T" coincide.
#include "common.hpp"
#include "internal.hpp"
#include "lean.hpp"
#include "probe.hpp"
#include "window.hpp"

namespace bt {

static unsigned grid_for(uint64_t n, unsigned threads, unsigned cap = 8192) {
  uint64_t g = (n + threads - 1) / threads;
  if (g == 0) g = 1;
  return (unsigned)(g < cap ? g : cap);
}

#define GRID_STRIDE(i, n)                                                        \
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); \
       i += (uint64_t)gridDim.x * blockDim.x)

__device__ __forceinline__ uint64_t block_len(const LevelDev& lv, const TextsDev& tx,
                                              uint64_t j) {
  const uint64_t st = lv.st[j];
  const uint64_t te = tx.tend[lv.text[j]];
  return te - st < lv.b ? te - st : lv.b;
}

// ---------------------------------------------------------------- keys (a3, a6)

// The key at st (at least 8 bytes long) in the byte scan's prefix filter.
__device__ __forceinline__ void set_prefix_bit(const PhaseArgs& a, uint64_t st) {
  uint32_t lo = 0, hi = 0;
  for (int k = 0; k < 4; ++k) {
    lo |= (uint32_t)a.T[st + k] << (8 * k);
    hi |= (uint32_t)a.T[st + 4 + k] << (8 * k);
  }
  const uint32_t bit = prefix8_bit(lo, hi, a.bfilt_bits);
  atomicOr(&a.bfilt[bit >> 5], 1u << (bit & 31));
}

// Profiling: add a per-thread count to *p, one atomic per wave.
__device__ __forceinline__ void wave_count(uint64_t* p, uint64_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
  if ((threadIdx.x & 63) == 0 && v) atomicAdd((unsigned long long*)p, (unsigned long long)v);
}

__global__ void k_keys(PhaseArgs a) {
  const LevelDev lv = a.lv;
  uint64_t inserted = 0;
  GRID_STRIDE(j, lv.c) {
    const uint32_t t = lv.text[j];
    const uint64_t st = lv.st[j];
    const uint64_t len = block_len(lv, a.tx, j);
    uint64_t L = 0;
    bool valid;
    if (a.phase == 1) {
      valid = (j + 1 < lv.c) && lv.run[j + 1] == lv.run[j];
      if (valid) L = len + block_len(lv, a.tx, j + 1);
    } else {
      valid = a.all_blocks || !a.marked[j];
      L = len;
    }
    if (!valid) {
      a.k.slot[j] = kNoKey;
      continue;
    }
    if (a.cflag) {
      // Strings inside a parent region that occurs earlier occur earlier too:
      // a pair window of length 2b <= b_parent starting in a parent whose pair
      // with the next parent occurs earlier, or lying inside a parent that
      // occurs earlier (itself, or as part of its pair with the previous one).
      // Marks and facts only need "before its start" for these; phase 2 needs
      // exact positions for unmarked blocks, and for all blocks when pruning.
      const uint8_t f = a.cflag[j];
      const bool copy = (a.phase == 1)
                            ? ((f & kSkipCross) || ((f & kSkipInterior) && !(f & kLastChild)))
                            : (!a.exact_all && a.marked[j] && (f & (kSkipCross | kSkipInterior)));
      if (copy) {
        a.k.slot[j] = kCopyKey;
        a.k.lm[j] = st - 1;
        continue;
      }
    }
    ++inserted;
    const uint64_t xp = (L == a.Lmain) ? a.xLmain : pow61(a.x, L);
    const uint64_t fp = finish_fp(win61_any(a, st, L, xp), a.tx.tsalt[t], a.fpmask);
    a.k.fp[j] = fp;
    a.k.len[j] = L;
    if (a.k.done) a.k.done[j] = 0;
    // (a flag: written once, not by every key of the text into one word)
    if (!a.odd.nkeys[t]) a.odd.nkeys[t] = 1;
    if (L == a.Lmain) {
      uint64_t h = slot_of(fp, a.tab.mask);
      while (true) {
        const uint64_t prev = atomicCAS((unsigned long long*)&a.tab.slots[h].fp,
                                        (unsigned long long)kEmpty, (unsigned long long)fp);
        if (prev == kEmpty || prev == fp) break;
        h = (h + 1) & a.tab.mask;
      }
      a.k.slot[j] = (uint32_t)h;
      atomicMin((unsigned long long*)&a.tab.slots[h].best, (unsigned long long)st);
      if (a.tf_words) {
        // text-local filter: this text's keys only
        const uint32_t h = win32_any(a, st, L, a.x32L) + (uint32_t)a.tx.tsalt[t];
        const uint32_t p = tfilter_hash(h);
        atomicOr(a.tf_words + a.tf_off[t] + block_word(p, a.tf_wl[t]), tfilter_mask(p, h));
      }
      if (a.filt_bits) {
        if (a.pre32) {
          const uint32_t h = win32_any(a, st, L, a.x32L) + (uint32_t)a.tx.tsalt[t];
          if (a.k.h32) a.k.h32[j] = h;
          atomicOr(&a.filt[filter32_word(h, a.filt_bits)], filter32_mask(h, a.filt_bits, a.filt_two));
          if (a.filt2_words) {
            const uint32_t p = filter2_hash(h);
            atomicOr(reinterpret_cast<unsigned long long*>(a.filt2) + block_word(p, a.filt2_words),
                     (unsigned long long)filter2_mask(p, h));
          }
        } else {
          const uint64_t f1 = filter_bit(fp, a.filt_bits), f2 = filter_bit2(fp, a.filt_bits);
          atomicOr(&a.filt[f1 >> 5], 1u << (f1 & 31));
          if (a.filt_two) atomicOr(&a.filt[f2 >> 5], 1u << (f2 & 31));
        }
      }
      if (a.bfilt_bits) set_prefix_bit(a, st);
    } else {
      // the one key of this text that ends at the text's end with a short block
      a.k.slot[j] = kOddKey;
      a.odd.L[t] = L;
      a.odd.xp[t] = xp;
      a.odd.fp[t] = fp;
      a.odd.pos[t] = st;
      a.odd.best[t] = st;
      const auto hash_of = [&](uint64_t len) {  // its first len bytes: hash, x32^len
        uint32_t xp32 = 1, base = a.x32;
        for (uint64_t e = len; e; e >>= 1) {
          if (e & 1) xp32 *= base;
          base *= base;
        }
        const uint32_t h = win32_any(a, st, len, xp32) + (uint32_t)a.tx.tsalt[t];
        return (uint64_t)h | ((uint64_t)xp32 << 32);
      };
      a.odd.h32[t] = hash_of(L);
      a.odd.anc[t] = hash_of(L < kOddAnchor ? L : kOddAnchor);
      if (a.bfilt_bits) set_prefix_bit(a, st);
    }
  }
  if (a.pc) wave_count(a.pc + kPcKeys, inserted);
}

hipError_t launch_keys(const PhaseArgs& a, hipStream_t s) {
  k_keys<<<grid_for(a.lv.c, 256), 256, 0, s>>>(a);
  return hipGetLastError();
}

// ---------------------------------------------------------------- probe scan (a4, a6)

constexpr int kScanK = 16;                      // windows per lane per chunk
constexpr int kScanSlowGroup = 8;                // steps whose loads leave together where a chunk crosses segments
constexpr uint64_t kScanChunk = 64ull * kScanK;  // windows per wave per chunk
static_assert(kScanChunk == kProbeTile, "the host counts algorithmic bytes per tile of kProbeTile windows");
static_assert(kLeanK == kScanK, "lean scans take the same chunks");

// Windows are numbered run after run (woff = exclusive prefix of per-run window
// counts).  Each wave takes chunks of 64*kScanK consecutive window numbers;
// in step k lane l handles window chunk + 64k + l, so consecutive lanes read
// consecutive prefix fingerprints.
//
// Before touching the table, a window's hash is tested against a bit filter of
// the phase's keys (one or two bits per key, set by k_keys) that every
// workgroup first copies into LDS.  A clear bit proves that no key has this
// hash.  The windows that pass are appended to a per-wave queue in LDS (ballot
// + prefix popcount) and probed 64 at a time.
constexpr int kProbeThreads = 1024;

__device__ __forceinline__ bool filter_has(const uint32_t* s_filt, uint64_t b1, uint64_t b2) {
  return ((s_filt[b1 >> 5] >> (b1 & 31)) & (s_filt[b2 >> 5] >> (b2 & 31)) & 1) != 0;
}


// The queued scans: filter, and the windows that pass go to a per-wave LDS
// queue; 64 queued windows at a time then form their fingerprints and probe
// together, so a wave waits for one round of loads per 64 candidates rather
// than per step.  The filter holds bits of the keys' 32-bit hashes (H[i+L] -
// H[i] x32^L mod 2^32), and the scan reads only H for every window; the 61-bit
// fingerprint is formed for queued windows alone.  Equal strings have equal
// hashes of both kinds, so every occurrence of a key still reaches the table; a
// window that agrees with a key in both hashes without being an occurrence is
// a collision, caught by the same verification as before.
//
// One wave's queue and what a queued window does.
template <bool SALT>
struct ProbeQueue {
  const PhaseArgs& a;
  uint64_t* q;
  const int lane;
  uint32_t qn = 0;     // wave-uniform queue length
  uint64_t ncand = 0;  // wave-uniform: windows that passed the filters
  __device__ ProbeQueue(const PhaseArgs& args, uint64_t* queue) : a(args), q(queue), lane(lane_id()) {}
  // the entry this lane holds: form its fingerprint and probe
  __device__ __forceinline__ void probe_entry(uint64_t e) const {
    const uint64_t i = e & kQPosMask;
    uint64_t f = a.P ? sub61(a.P[i + a.Lmain], mul61(a.P[i], a.xLmain)) : win61<true>(a, i, a.Lmain, a.xLmain);
    if (SALT) f = add61(f, a.tx.tsalt[e >> kQPosBits]);
    probe(a.tab.slots, a.tab.mask, f & a.fpmask, i);
  }
  // whole wave: append the lanes' candidates; probe 64 once 64 are waiting
  __device__ __forceinline__ void push(bool cand, uint64_t i, uint32_t t) {
    const uint64_t bal = __ballot(cand);
    if (!bal) return;
    const uint32_t my = (uint32_t)__popcll(bal & ((1ull << lane) - 1));
    if (cand) q[qn + my] = ((uint64_t)t << kQPosBits) | i;
    qn += (uint32_t)__popcll(bal);
    ncand += (uint64_t)__popcll(bal);
    if (qn >= 64) {
      wave_sync();
      const uint64_t e = q[lane];
      const bool mv = (uint32_t)lane < qn - 64;
      const uint64_t e2 = mv ? q[64 + lane] : 0;
      wave_sync();
      if (mv) q[lane] = e2;
      qn -= 64;
      probe_entry(e);
      wave_sync();
    }
  }
  __device__ __forceinline__ void finish() {
    if (qn) {
      wave_sync();
      if ((uint32_t)lane < qn) probe_entry(q[lane]);
    }
    if (a.pc && lane == 0 && ncand) atomicAdd((unsigned long long*)(a.pc + kPcCand), (unsigned long long)ncand);
  }
};

// Copy the phase's key filter into LDS.
__device__ __forceinline__ void load_filter(const PhaseArgs& a, uint32_t* s_filt) {
  const uint32_t nq = 1u << (a.filt_bits - 7);  // uint4 words
  const uint4* src = reinterpret_cast<const uint4*>(a.filt);
  uint4* dst = reinterpret_cast<uint4*>(s_filt);
  for (uint32_t q = threadIdx.x; q < nq; q += blockDim.x) dst[q] = src[q];
  __syncthreads();
}

// The first tile of 64th f of the scan (f = 64: past the last).
__device__ __forceinline__ uint64_t round_tile(uint64_t W, uint32_t f) {
  const uint64_t tiles = (W + kScanChunk - 1) / kScanChunk;
  return tiles / 64 * f + tiles % 64 * f / 64;
}

// Rounds.  Windows are numbered in the order of their positions, so once the
// tiles below some tile are scanned, a key whose smallest position lies below
// that tile's first one has its leftmost occurrence: no later window can improve
// it.  The filters of the next round hold the other keys only.  In a repetitive
// text most keys occur in its first copies, and the windows of all later copies,
// true occurrences that would each read a slot and two prefix values for
// nothing, now fail the filter; and of the keys that occur nowhere earlier, those
// that start before the round drop out.
__global__ void k_refilter(PhaseArgs a, const uint64_t* __restrict__ woff, uint32_t f0) {
  const uint64_t R = a.segn[0], W = a.segn[1];
  const uint64_t w = round_tile(W, f0) * kScanChunk;
  if (w >= W) return;
  const uint64_t r = segment_of(woff, R, w);
  const uint64_t from = a.lv.rs[r] + (w - woff[r]);
  GRID_STRIDE(j, a.lv.c) {
    const uint32_t s = a.k.slot[j];
    if (s == kNoKey || s == kOddKey || s == kCopyKey || a.lv.st[j] < from) continue;
    if (a.tab.slots[s].best < from) continue;
    const uint32_t h = a.k.h32[j];
    atomicOr(&a.filt[filter32_word(h, a.filt_bits)], filter32_mask(h, a.filt_bits, a.filt_two));
    if (a.filt2_words) {
      const uint32_t p = filter2_hash(h);
      atomicOr(reinterpret_cast<unsigned long long*>(a.filt2) + block_word(p, a.filt2_words),
               (unsigned long long)filter2_mask(p, h));
    }
  }
}

hipError_t launch_refilter(const PhaseArgs& a, const uint64_t* woff, uint32_t f0, hipStream_t s) {
  if (!a.pre32 || !a.filt_bits || !a.k.h32) return hipErrorInvalidValue;
  k_refilter<<<grid_for(a.lv.c, 256), 256, 0, s>>>(a, woff, f0);
  return hipGetLastError();
}

// The segment of each tile's first window (tile ch: window number ch kScanChunk),
// one thread per tile, so that a wave of the scan reads it with one load instead
// of searching for it in log2(R) dependent ones.
__global__ void k_tile_segs(const uint64_t* __restrict__ woff, const uint64_t* __restrict__ segn,
                            uint32_t* __restrict__ tseg) {
  const uint64_t R = segn[0], W = segn[1];
  GRID_STRIDE(ch, (W + kScanChunk - 1) / kScanChunk) tseg[ch] = (uint32_t)segment_of(woff, R, ch * kScanChunk);
}

// The scan of a single text with dense 32-bit hashes (SALT: of a batch with
// shared filters).
//
// What bounds it: at the upper levels the hash streams, at the lower ones (many
// candidates) random reads.  Measured on 2^28 windows of the 256 MiB text,
// reading H[i] and H[i+L] for every window ran at the fabric's 5.5 TB/s, 0.39 ms,
// whatever L: the second stream is the first one L later, and few lines survive
// in an XCD's L2 until then.  So where L is a multiple of the tile, a wave walks
// a column: the tiles at i, i+L, i+2L, ..., `rows` of them, and the H[i+L] of one
// row is the H[i] of the next, kept in registers.  That reads (rows + 1) / rows
// streams in place of two.  Tiles are taken by their window numbers (units of
// rows x stride tiles, stride = L / tile); a tile whose windows do not lie in one
// segment, or do not continue the row above, loads both values as any tile did.
// Measured, kernel time before and after (with the filter test of one LDS read
// and candidates popped per lane): 2^28 windows at L = 2^21 0.393 -> 0.244 ms, at
// L = 2^17 0.417 -> 0.265 ms; 2^31 windows at L = 2^19 3.32 -> 1.75 ms; 10^8
// windows of a text with a short final key at L = 2^18 0.256 -> 0.150 ms.
//
// One 1024-thread workgroup per CU at up to 128 VGPRs: a lane's sixteen hashes of
// a row and of the row before stay in registers and its loads leave together; the
// LDS holds a 128 KiB filter (2^20 bits).  A text's short final key is tested by
// its anchor, H[i + 64] (the value the lane holds for the next step).
template <bool ODD, bool SALT>
__global__ __launch_bounds__(kProbeThreads) __attribute__((amdgpu_waves_per_eu(4)))
void k_probe_dense(PhaseArgs a, const uint64_t* __restrict__ woff, uint32_t f0, uint32_t f1,
                   const uint32_t* __restrict__ tseg, uint64_t stride, uint64_t rows) {
  extern __shared__ uint64_t s_lds[];
  uint32_t* s_filt = reinterpret_cast<uint32_t*>(s_lds);
  load_filter(a, s_filt);
  const uint32_t fbits = a.filt_bits;
  const bool two = a.filt_two != 0;
  const int lane = lane_id();
  uint64_t* waves = s_lds + (1ull << (fbits - 6));
  ProbeQueue<SALT> queue(a, waves + (uint64_t)(threadIdx.x >> 6) * kQueue);
  // the wave's segment map of a tile that crosses segments
  uint64_t* s_map = waves + (kProbeThreads / 64) * kQueue + (threadIdx.x >> 6) * kScanK;

  const uint64_t R = a.segn[0], W = a.segn[1];
  const uint64_t t0 = round_tile(W, f0), t1 = round_tile(W, f1);
  // wave-uniform (all of a wave's lanes share threadIdx.x / 64)
  const uint64_t gw = (uint64_t)blockIdx.x * (kProbeThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t nw = (uint64_t)gridDim.x * (kProbeThreads / 64);
  const uint32_t* __restrict__ H = a.P32;
  const uint64_t* __restrict__ rs_ = a.lv.rs;
  const uint64_t* __restrict__ re_ = a.lv.re;
  const uint64_t L = a.Lmain;
  const uint32_t x32L = a.x32L;
  const uint64_t* __restrict__ filt2 = reinterpret_cast<const uint64_t*>(a.filt2);
  const uint32_t f2words = a.filt2_words;
  const uint32_t s1 = 32 - fbits, s2 = two ? 27 - fbits : s1;
  const auto pass32 = [&](uint32_t h) { return filter32_has(s_filt[filter32_word(h, fbits)], h, s1, s2); };
  const auto pass2 = [&](uint32_t h) {
    const uint32_t p = filter2_hash(h);
    return filter2_has(filt2[block_word(p, f2words)], p, h);
  };
  // the second filter for the steps in okm, their loads issued together
  const auto second = [&](auto& hv, uint32_t okm) {
    constexpr int K = sizeof(hv) / sizeof(hv[0]);
    uint64_t wv[K];
#pragma unroll
    for (int k = 0; k < K; ++k)
      wv[k] = (okm >> k) & 1 ? filt2[block_word(filter2_hash(hv[k]), f2words)] : 0ull;
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) m |= filter2_has(wv[k], filter2_hash(hv[k]), hv[k]) << k;
    return m;
  };

  // the text t's short final key, if any: its length, its position, and the
  // length, hash and power of its anchor
  uint32_t t = 0;
  uint64_t salt = 0, oL = 0, opos = 0;
  uint32_t oA = 0, oh = 0, ox = 0;
  const auto load_text = [&](uint32_t nt) {
    t = nt;
    if (SALT) salt = a.tx.tsalt[t];
    if (ODD) {
      oL = a.odd.L[t];
      if (oL) {
        oA = (uint32_t)(oL < kOddAnchor ? oL : kOddAnchor);
        opos = a.odd.pos[t];
        const uint64_t hx = a.odd.anc[t];
        oh = (uint32_t)hx;
        ox = (uint32_t)(hx >> 32);
      }
    }
  };
  // a window at i that matches the anchor: the whole key's 32-bit hash, then
  // its 61-bit fingerprint
  const auto odd61 = [&](uint64_t i) {
    const uint64_t hx = a.odd.h32[t];
    if (H[i + oL] - H[i] * (uint32_t)(hx >> 32) + (uint32_t)salt != (uint32_t)hx) return;
    uint64_t g = a.P ? sub61(a.P[i + oL], mul61(a.P[i], a.odd.xp[t])) : win61<true>(a, i, oL, a.odd.xp[t]);
    if (SALT) g = add61(g, salt);
    if ((g & a.fpmask) == a.odd.fp[t] && i < a.odd.best[t])
      atomicMin((unsigned long long*)&a.odd.best[t], (unsigned long long)i);
  };

  const uint64_t units = (t1 - t0 + rows * stride - 1) / (rows * stride) * stride;
  for (uint64_t u = gw; u < units; u += nw) {
    uint32_t hp[kScanK];     // H[i + L] of the row above
    uint64_t next = ~0ull;   // the position whose H they are (of lane 0, step 0)
    uint64_t ch = t0 + u / stride * (rows * stride) + u % stride;
    for (uint64_t row = 0; row < rows && ch < t1; ++row, ch += stride) {
      const uint64_t wb = ch * kScanChunk;
      const uint64_t r0 = tseg ? tseg[ch] : segment_of(woff, R, wb);
      const uint64_t wo0 = woff[r0], wn0 = woff[r0 + 1], rs0 = rs_[r0], re0 = re_[r0];
      if (wb + kScanChunk <= wn0 && rs0 + (wb + kScanChunk - 1 - wo0) + L <= re0) {
        // the tile's windows are consecutive positions of one segment
        if (ODD || SALT) load_text(a.lv.rtext[r0]);
        const uint64_t ib = rs0 + (wb - wo0);
        const uint64_t i0 = ib + lane;
        uint32_t ha[kScanK], hb[kScanK];
        const bool keep = ib == next;
#pragma unroll
        for (int k = 0; k < kScanK; ++k) hb[k] = H[i0 + L + 64ull * k];
        if (keep) {
#pragma unroll
          for (int k = 0; k < kScanK; ++k) ha[k] = hp[k];
        } else {
#pragma unroll
          for (int k = 0; k < kScanK; ++k) ha[k] = H[i0 + 64ull * k];
        }
        const uint32_t s32 = SALT ? (uint32_t)salt : 0u;
        if (ODD && oL) {
          uint32_t om = 0;
          if (oA == kOddAnchor) {  // H[i + 64] is the next step's H[i]
            const uint32_t hl = H[i0 + 64ull * kScanK];
#pragma unroll
            for (int k = 0; k < kScanK; ++k) {
              const uint32_t hc = k + 1 < kScanK ? ha[k + 1 < kScanK ? k + 1 : k] : hl;
              if (hc - ha[k] * ox + s32 == oh) om |= 1u << k;
            }
          } else {
#pragma unroll
            for (int k = 0; k < kScanK; ++k)
              if (H[i0 + 64ull * k + oA] - ha[k] * ox + s32 == oh) om |= 1u << k;
          }
          while (om) {
            const int k = __builtin_ctz(om);
            om &= om - 1;
            if (i0 + 64ull * k < opos) odd61(i0 + 64ull * k);
          }
        }
        uint32_t hv[kScanK];
        uint32_t okm = 0;  // bit k: the lane's window of step k passes
#pragma unroll
        for (int k = 0; k < kScanK; ++k) {
          hv[k] = hb[k] - ha[k] * x32L + s32;
          hp[k] = hb[k];
          okm |= pass32(hv[k]) << k;
        }
        next = ib + L;
        if (!__ballot(okm != 0)) continue;
        if (f2words) okm = second(hv, okm);
        // as many rounds as the lane with the most candidates has
        while (__ballot(okm != 0)) {
          queue.push(okm != 0, i0 + 64ull * (okm ? __builtin_ctz(okm) : 0), t);
          okm &= okm - 1;
        }
        continue;
      }

      // the tile crosses segments (or holds windows that do not fit, or ends
      // the scan)
      next = ~0ull;
      const uint64_t w0 = wb + lane;
      if constexpr (!SALT) {
        // One text (its short key stays).  The starts of the segments inside the
        // tile become bits of a map, so that a window's segment is the first
        // one's number plus the bits up to it: no lane walks the segments, one
        // dependent read per boundary.  Then a group's segments are read
        // together, and its hashes.  (Scans of L = 64: 256 MiB text 0.26 -> 0.22
        // ms, 2 GiB 3.0 -> 2.3 ms, 100 MB tau 2 0.186 -> 0.153 ms.)
        if (ODD) load_text(0);
        const uint64_t rl = tseg ? (wb + kScanChunk < W ? (uint64_t)tseg[ch + 1] : R - 1)
                                 : segment_in(woff, r0, R, wb + kScanChunk - 1);
        if (lane < kScanK) s_map[lane] = 0;
        wave_sync();
        for (uint64_t r = r0 + 1 + lane; r <= rl; r += 64) {
          const uint64_t at = woff[r] - wb;
          if (at < kScanChunk) atomicOr(reinterpret_cast<unsigned long long*>(&s_map[at >> 6]), 1ull << (at & 63));
        }
        wave_sync();
        uint64_t r = r0;  // the segment before the step's first start
#pragma unroll 1
        for (int k0 = 0; k0 < kScanK; k0 += kScanSlowGroup) {
          uint64_t ik[kScanSlowGroup];
          uint32_t vm = 0, om = 0;  // steps with a main-length window, with a short-key window
#pragma unroll
          for (int k = 0; k < kScanSlowGroup; ++k) {
            const uint64_t map = s_map[k0 + k];
            const uint64_t w = w0 + 64ull * (k0 + k);
            const uint64_t rk = r + __popcll(map & (~0ull >> (63 - lane)));
            r += __popcll(map);
            const bool live = w < W;
            const uint64_t i = rs_[rk] + (w - woff[rk]);
            ik[k] = i;
            if (ODD) {
              // (without a short key every window of a segment fits its run)
              const uint64_t re = re_[rk];
              if (live && i + L <= re) vm |= 1u << k;
              if (live && oL && i + oL <= re && i < opos) om |= 1u << k;
            } else if (live) {
              vm |= 1u << k;
            }
          }
          uint32_t ha[kScanSlowGroup], hb[kScanSlowGroup], hc[kScanSlowGroup];
#pragma unroll
          for (int k = 0; k < kScanSlowGroup; ++k) {
            hb[k] = ((vm >> k) & 1) ? H[ik[k] + L] : 0u;
            ha[k] = (((vm | om) >> k) & 1) ? H[ik[k]] : 0u;
            if (ODD) hc[k] = ((om >> k) & 1) ? H[ik[k] + oA] : 0u;
          }
          __builtin_amdgcn_sched_barrier(0);
          if (ODD) {
            uint32_t mm = 0;
#pragma unroll
            for (int k = 0; k < kScanSlowGroup; ++k)
              if (((om >> k) & 1) && hc[k] - ha[k] * ox == oh) mm |= 1u << k;
            while (mm) {
              const int k = __builtin_ctz(mm);
              mm &= mm - 1;
              odd61(ik[k]);
            }
          }
          uint32_t hv[kScanSlowGroup];
          uint32_t okm = 0;
#pragma unroll
          for (int k = 0; k < kScanSlowGroup; ++k) {
            hv[k] = hb[k] - ha[k] * x32L;
            okm |= (pass32(hv[k]) & (vm >> k)) << k;
          }
          if (!__ballot(okm != 0)) continue;
          if (f2words) okm = second(hv, okm);
#pragma unroll
          for (int k = 0; k < kScanSlowGroup; ++k) queue.push((okm >> k) & 1, ik[k], 0);
        }
        wave_sync();  // the map is cleared again by the next such tile
      } else {
        // each lane follows its windows across segments and texts
        const uint64_t rh = tseg && wb + kScanChunk < W ? (uint64_t)tseg[ch + 1] + 1 : R;
        uint64_t r = segment_in(woff, r0, rh, w0);
        uint64_t wo = woff[r], wn = woff[r + 1], rs = rs_[r], re = re_[r];
        // lanes past the last window hold no segment: they read no text entry
        oL = 0;
        if (w0 < W) load_text(a.lv.rtext[r]);
        for (int k = 0; k < kScanK; ++k) {
          const uint64_t w = w0 + (uint64_t)k * 64;
          const bool live = w < W;  // every lane stays in the loop (the queue is wave-wide)
          if (live && w >= wn) {
            do {
              ++r;
              wo = wn;
              wn = woff[r + 1];
            } while (w >= wn);
            rs = rs_[r];
            re = re_[r];
            load_text(a.lv.rtext[r]);
          }
          const uint64_t i = rs + (w - wo);
          bool cand = false;
          if (live && i + L <= re) {
            const uint32_t h = H[i + L] - H[i] * x32L + (uint32_t)salt;
            cand = pass32(h) && (!f2words || pass2(h));
          }
          queue.push(cand, i, t);
          if (ODD && live && oL && i + oL <= re && i < opos) {
            if (H[i + oA] - H[i] * ox + (uint32_t)salt == oh) odd61(i);
          }
        }
      }
    }
  }
  queue.finish();
}

// The scan of memory-lean builds (LEAN: the 32-bit hashes are sampled and lanes
// roll them along consecutive windows, lean.hpp; queued windows form their
// 61-bit fingerprints from the samples), and the scan without queues (every
// window's 61-bit fingerprint against the filter, candidates probe at once) for
// texts beyond the queue's packing.
//
// Instances without a short final key hold their registers (SGPRs included)
// to two 1024-thread workgroups per CU, 8 waves per SIMD.  Instances with one
// carry more live values: they run one workgroup per CU with up to 128 VGPRs,
// which measured faster than spilling at 64.
template <bool ODD, bool SALT, bool LEAN>
__global__ __launch_bounds__(kProbeThreads) __attribute__((amdgpu_waves_per_eu(ODD ? 4 : 8)))
void k_probe_scan(PhaseArgs a, const uint64_t* __restrict__ woff, uint32_t f0, uint32_t f1) {
  extern __shared__ uint64_t s_lds[];
  uint32_t* s_filt = reinterpret_cast<uint32_t*>(s_lds);
  load_filter(a, s_filt);
  const uint32_t fbits = a.filt_bits;
  const bool two = a.filt_two != 0;
  const int lane = lane_id();
  const uint64_t R = a.segn[0], W = a.segn[1];
  const uint64_t gw = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint64_t nw = ((uint64_t)gridDim.x * blockDim.x) >> 6;

  if constexpr (LEAN) {
    ProbeQueue<SALT> queue(a, s_lds + (1ull << (fbits - 6)) + (uint64_t)(threadIdx.x >> 6) * kQueue);
    const uint64_t* __restrict__ filt2 = reinterpret_cast<const uint64_t*>(a.filt2);
    const uint32_t s1 = 32 - fbits, s2 = two ? 27 - fbits : s1;
    const uint32_t f2words = a.filt2_words;
    const auto pass32 = [&](uint32_t h) { return filter32_has(s_filt[filter32_word(h, fbits)], h, s1, s2) != 0; };
    const auto test8 = [&](const uint32_t* hv, bool* ok) {
#pragma unroll
      for (int k = 0; k < 8; ++k) ok[k] = pass32(hv[k]);
      if (f2words) {
        uint64_t wv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) wv[k] = ok[k] ? filt2[block_word(filter2_hash(hv[k]), f2words)] : 0ull;
#pragma unroll
        for (int k = 0; k < 8; ++k) ok[k] = filter2_has(wv[k], filter2_hash(hv[k]), hv[k]) != 0;
      }
    };
    const auto test1 = [&](uint32_t h) {
      const uint32_t p = filter2_hash(h);
      return pass32(h) && (!f2words || filter2_has(filt2[block_word(p, f2words)], p, h));
    };
    const auto push = [&](bool cand, uint64_t i, uint32_t t) { queue.push(cand, i, t); };
    const uint64_t t1 = round_tile(W, f1);
    for (uint64_t ch = round_tile(W, f0) + gw; ch < t1; ch += nw)
      lean_chunk<ODD, ODD || SALT, SALT>(a, woff, 0, R, W, ch * kScanChunk + (uint64_t)lane * kLeanK,
                                         [](uint32_t) {}, test8, test1, push);
    queue.finish();
    return;
  }

  uint64_t ncand = 0;
  const uint64_t* __restrict__ P = a.P;
  const uint64_t L = a.Lmain, xL = a.xLmain, fmask = a.fpmask;
  for (uint64_t ch = gw; ch * kScanChunk < W; ch += nw) {
    const uint64_t w0 = ch * kScanChunk + lane;
    uint64_t r = segment_of(woff, R, w0);
    uint64_t wo = woff[r], wn = woff[r + 1], rs = a.lv.rs[r], re = a.lv.re[r];
    // lanes past the last window hold no segment: they read no text entry
    uint32_t t = ((ODD || SALT) && w0 < W) ? a.lv.rtext[r] : 0;
    uint64_t salt = SALT ? a.tx.tsalt[t] : 0;
    uint64_t oL = (ODD && w0 < W) ? a.odd.L[t] : 0;
    const auto fp_of = [&](uint64_t i, uint64_t len, uint64_t xp) {
      uint64_t f = sub61(P[i + len], mul61(P[i], xp));
      if (SALT) f = add61(f, salt);
      return f & fmask;
    };
    for (int k = 0; k < kScanK; ++k) {
      const uint64_t w = w0 + (uint64_t)k * 64;
      if (w >= W) break;
      if (w >= wn) {
        do {
          ++r;
          wo = wn;
          wn = woff[r + 1];
        } while (w >= wn);
        rs = a.lv.rs[r];
        re = a.lv.re[r];
        if (ODD || SALT) t = a.lv.rtext[r];
        if (SALT) salt = a.tx.tsalt[t];
        if (ODD) oL = a.odd.L[t];
      }
      const uint64_t i = rs + (w - wo);
      if (i + L <= re) {
        const uint64_t f = fp_of(i, L, xL);
        const uint64_t b1 = filter_bit(f, fbits);
        if (filter_has(s_filt, b1, two ? filter_bit2(f, fbits) : b1)) {
          ++ncand;
          probe(a.tab.slots, a.tab.mask, f, i);
        }
      }
      if (ODD && oL && i + oL <= re && i < a.odd.pos[t] && fp_of(i, oL, a.odd.xp[t]) == a.odd.fp[t] &&
          i < a.odd.best[t])
        atomicMin((unsigned long long*)&a.odd.best[t], (unsigned long long)i);
    }
  }
  if (a.pc) wave_count(a.pc + kPcCand, ncand);
}

// Dynamic LDS beyond 64 KiB has to be allowed per kernel.
static hipError_t allow_lds(const void* fn, size_t bytes) {
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Rows of a column walk: as many as leave every resident wave (256 workgroups of
// 16) four units, at most 16 (17/16 streams).
uint64_t probe_scan_rows(uint64_t L, uint64_t tiles) {
  const uint64_t stride = L / kScanChunk;
  if (L % kScanChunk || !stride || (stride >= tiles && stride > 1)) return 1;
  uint64_t rows = tiles / (4 * 256 * (kProbeThreads / 64));
  if (rows > 16) rows = 16;
  if (rows * stride > tiles) rows = tiles / stride;
  return rows ? rows : 1;
}

hipError_t launch_probe_scan(const PhaseArgs& a, const uint64_t* woff, bool has_odd,
                             bool has_salt, uint64_t max_windows, int mode, uint32_t* tseg,
                             uint32_t f0, uint32_t f1, bool find_segs, hipStream_t s) {
  if (f0 >= f1 || f1 > 64 || (mode != 1 && (f0 != 0 || f1 != 64))) return hipErrorInvalidValue;
  const uint64_t all = (max_windows + kScanChunk - 1) / kScanChunk;
  const uint64_t tiles = (all * (f1 - f0) + 63) / 64;
  // the filter, and in queued scans 16 KiB of queues (and 2 KiB of segment maps
  // with dense hashes)
  const bool lean = a.P32 == nullptr;
  const size_t lds = ((size_t)1 << (a.filt_bits - 3)) +
                     (mode == 1 ? (size_t)(kProbeThreads / 64) * (kQueue + (lean ? 0 : kScanK)) * 8 : 0);
  // queued scans pre-filter on 32-bit hashes; sampled fingerprints serve queued
  // candidates only
  if ((mode == 1) != (a.pre32 != 0) || (mode != 1 && mode != 2) || (a.P == nullptr && mode != 1))
    return hipErrorInvalidValue;
  const auto launch = [&](auto* fn, unsigned grid, auto... args) {
    if (lds > 65536) {
      const hipError_t e = allow_lds(reinterpret_cast<const void*>(fn), lds);
      if (e != hipSuccess) return e;
    }
    fn<<<grid, kProbeThreads, lds, s>>>(a, woff, f0, f1, args...);
    return hipGetLastError();
  };
  if (mode == 1 && !lean) {
    if (tseg && f0 == 0 && find_segs) k_tile_segs<<<grid_for(all, 256), 256, 0, s>>>(woff, a.segn, tseg);
    const uint64_t rows = probe_scan_rows(a.Lmain, tiles);
    const uint64_t stride = a.Lmain % kScanChunk == 0 && a.Lmain / kScanChunk < tiles ? a.Lmain / kScanChunk : 1;
    const unsigned grid = grid_for(tiles * 64, kProbeThreads, 256);
    const uint32_t* ts = tseg;
    if (has_odd)
      return has_salt ? launch(&k_probe_dense<true, true>, grid, ts, stride, rows)
                      : launch(&k_probe_dense<true, false>, grid, ts, stride, rows);
    return has_salt ? launch(&k_probe_dense<false, true>, grid, ts, stride, rows)
                    : launch(&k_probe_dense<false, false>, grid, ts, stride, rows);
  }
  // two 1024-thread workgroups per CU: LDS of at most 80 KiB each
  const unsigned grid = grid_for(tiles * 64, kProbeThreads, 512);
  if (mode == 1) {
    if (has_odd) return has_salt ? launch(&k_probe_scan<true, true, true>, grid) : launch(&k_probe_scan<true, false, true>, grid);
    return has_salt ? launch(&k_probe_scan<false, true, true>, grid) : launch(&k_probe_scan<false, false, true>, grid);
  }
  if (has_odd) return has_salt ? launch(&k_probe_scan<true, true, false>, grid) : launch(&k_probe_scan<true, false, false>, grid);
  return has_salt ? launch(&k_probe_scan<false, true, false>, grid) : launch(&k_probe_scan<false, false, false>, grid);
}

// ---------------------------------------------------------------- byte scan (a4)
//
// For phases with few keys (the upper levels, whose blocks are longer than the
// spacing of the text's differences, so that no window is skipped), reading
// two prefix hashes per window is the whole cost.  Here a window is first
// tested on its own first eight bytes against a filter of the keys' first
// eight bytes: 1 byte of text per window instead of 8 bytes of hashes.  Equal
// strings share their first eight bytes, so every occurrence of a key passes.
// The windows that pass (in a repetitive text, mostly true copies of a key's
// first eight bytes) go to the per-wave LDS queue of the probe scan and form
// their 61-bit fingerprints 64 at a time.
//
// A wave takes 2048 consecutive window numbers; lane l takes 32 consecutive
// ones.  When they lie in one segment the lane loads the 44 aligned bytes that
// cover them and takes each window's eight bytes with byte-aligns.  Bound by the
// bytes in flight (a segment search, a load and 32 tests per wave and round) and
// by the candidates: with 16 windows per lane, and the candidates queued in a step
// per window, 2 GiB of DNA took 1.02 / 1.37 / 1.83 ms with 4 / 16 / 64 keys
// (now 0.67 / 0.85 / 1.07); one multiplication per test in place of two, and one search per wave
// in place of one per lane, changed nothing by themselves.
constexpr int kByteThreads = 1024;
constexpr int kByteK = 32;  // windows per lane
// Queue entries: position in bits 0..39, text in bits 40..62, and bit 63 set
// when the main-length window does not fit its run.
constexpr uint64_t kByteTextMask = (1ull << 23) - 1;

template <bool ODD, bool SALT, bool LEAN>
__global__ __launch_bounds__(kByteThreads) __attribute__((amdgpu_waves_per_eu(8)))
void k_byte_scan(PhaseArgs a, const uint64_t* __restrict__ woff) {
  extern __shared__ uint64_t s_lds[];
  uint32_t* s_bf = reinterpret_cast<uint32_t*>(s_lds);
  const uint32_t bits = a.bfilt_bits;
  {
    const uint32_t nq = 1u << (bits - 7);  // uint4 words
    const uint4* src = reinterpret_cast<const uint4*>(a.bfilt);
    uint4* dst = reinterpret_cast<uint4*>(s_bf);
    for (uint32_t k = threadIdx.x; k < nq; k += blockDim.x) dst[k] = src[k];
    __syncthreads();
  }
  const int lane = lane_id();
  uint64_t* q = s_lds + (1ull << (bits - 6)) + (uint64_t)(threadIdx.x >> 6) * kQueue;
  uint32_t qn = 0;  // wave-uniform queue length
  const uint64_t R = a.segn[0], W = a.segn[1];
  const uint32_t gw = __builtin_amdgcn_readfirstlane((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const uint32_t nw = (gridDim.x * blockDim.x) >> 6;
  const uint8_t* __restrict__ T = a.T;
  const uint64_t* __restrict__ P = a.P;
  const uint64_t L = a.Lmain, xL = a.xLmain, fmask = a.fpmask;
  Slot* __restrict__ slots = a.tab.slots;
  const uint64_t mask = a.tab.mask;
  const auto has = [&](uint32_t lo, uint32_t hi) {
    const uint32_t b = prefix8_bit(lo, hi, bits);
    return ((s_bf[b >> 5] >> (b & 31)) & 1u) != 0;
  };
  // A queued window: its fingerprints against the keys.  Bit 63 of the entry
  // says whether the main-length window fits its run.  A window of the short
  // final key's length always fits (segments hold the windows of the shorter
  // of the two lengths), so only the text's end bounds it.
  const auto check = [&](uint64_t e) {
    const uint64_t i = e & kQPosMask;
    const uint32_t t = (uint32_t)((e >> kQPosBits) & kByteTextMask);  // bit 63 is the fit bit
    const uint64_t salt = SALT ? a.tx.tsalt[t] : 0;
    if (!(e >> 63)) {
      uint64_t f = P ? sub61(P[i + L], mul61(P[i], xL)) : win61<true>(a, i, L, xL);
      if (SALT) f = add61(f, salt);
      probe(slots, mask, f & fmask, i);
    }
    if (ODD) {
      const uint64_t oL = a.odd.L[t];
      if (oL && i + oL <= a.tx.tend[t] && i < a.odd.pos[t]) {
        uint64_t g = P ? sub61(P[i + oL], mul61(P[i], a.odd.xp[t])) : win61<true>(a, i, oL, a.odd.xp[t]);
        if (SALT) g = add61(g, salt);
        if ((g & fmask) == a.odd.fp[t] && i < a.odd.best[t])
          atomicMin((unsigned long long*)&a.odd.best[t], (unsigned long long)i);
      }
    }
  };
  // whole wave: append the lanes' candidates; check 64 once 64 are waiting, a full
  // wave of them at once.  Bit 63 of an entry: the main-length window does not fit the run.
  uint64_t ncand = 0;  // wave-uniform: windows that passed the filter
  const auto push = [&](bool cand, uint64_t e) {
    const uint64_t bal = __ballot(cand);
    if (!bal) return;
    ncand += (uint64_t)__popcll(bal);
    if (bal != ~0ull) {
      const uint32_t my = (uint32_t)__popcll(bal & ((1ull << lane) - 1));
      if (cand) q[qn + my] = e;
      qn += (uint32_t)__popcll(bal);
      if (qn < 64) return;
      wave_sync();
      e = q[lane];
      const bool mv = (uint32_t)lane < qn - 64;
      const uint64_t e2 = mv ? q[64 + lane] : 0;
      wave_sync();
      if (mv) q[lane] = e2;
      qn -= 64;
    }
    check(e);
    wave_sync();
  };

  for (uint64_t ch = gw; ch * (64ull * kByteK) < W; ch += nw) {
    const uint64_t w0 = ch * (64ull * kByteK) + (uint64_t)lane * kByteK;
    const bool any = w0 < W;  // lanes past the last window hold no segment
    // the segment of the chunk's first window, once for the wave; lanes look for
    // their own from there on only where the chunk does not lie in it
    const uint64_t c0 = ch * (64ull * kByteK);
    uint64_t r = 0;
    for (uint64_t hi = R; hi - r > 1;) {
      const uint64_t mid = (r + hi) >> 1;
      if (woff[mid] <= c0) r = mid; else hi = mid;
    }
    uint64_t wo = woff[r], wn = woff[r + 1], rs = a.lv.rs[r], re = a.lv.re[r];
    uint32_t t = a.lv.rtext[r];
    const bool whole = c0 + 64ull * kByteK <= wn;  // the chunk lies in that segment
    if (!whole && any) {
      for (uint64_t hi = R; hi - r > 1;) {
        const uint64_t mid = (r + hi) >> 1;
        if (woff[mid] <= w0) r = mid; else hi = mid;
      }
      wo = woff[r];
      wn = woff[r + 1];
      rs = a.lv.rs[r];
      re = a.lv.re[r];
      t = a.lv.rtext[r];
    }
    const uint64_t i0 = rs + (w0 - wo);
    // the lane's 32 windows in one segment, all of main length inside the run
    const bool fast = any && w0 + (kByteK - 1) < wn && i0 + (kByteK - 1) + L <= re;
    uint32_t m = 0;  // bit k: window w0 + k passes
    if (fast) {
      // The 44 bytes from the 4-byte aligned address at or below T + i0 cover
      // [i0, i0 + 39).  They end inside the lane's last window, which starts 31
      // bytes on and ends at or before the run end (31 + L >= 47: keys of the byte
      // scan are pairs of blocks of b >= 16, or longer than one), and they start no
      // lower than the aligned base of the allocation holding the text.
      const uintptr_t ad = reinterpret_cast<uintptr_t>(T + i0);
      const uint32_t* wp = reinterpret_cast<const uint32_t*>(ad & ~(uintptr_t)3);
      uint32_t w[kByteK / 4 + 3];
#pragma unroll
      for (int k = 0; k < kByteK / 4 + 3; ++k) w[k] = wp[k];
      const uint32_t sh = (uint32_t)(ad & 3);
      uint32_t x[kByteK / 4 + 2];  // x[k] = bytes [i0 + 4k, i0 + 4k + 4)
#pragma unroll
      for (int k = 0; k < kByteK / 4 + 2; ++k) x[k] = __builtin_amdgcn_alignbyte(w[k + 1], w[k], sh);
#pragma unroll
      for (int k = 0; k < kByteK; ++k) {
        const int qq = k >> 2, o = k & 3;
        const uint32_t l4 = o ? __builtin_amdgcn_alignbyte(x[qq + 1], x[qq], o) : x[qq];
        const uint32_t h4 = o ? __builtin_amdgcn_alignbyte(x[qq + 2], x[qq + 1], o) : x[qq + 1];
        m |= (has(l4, h4) ? 1u : 0u) << k;
      }
    } else if (any) {
      // windows across segment ends: walk them one by one (this lane only)
      uint64_t r2 = r, wo2 = wo, wn2 = wn, rs2 = rs;
      for (int k = 0; k < kByteK; ++k) {
        const uint64_t wi = w0 + k;
        if (wi >= W) break;
        while (wi >= wn2) {
          ++r2;
          wo2 = wn2;
          wn2 = woff[r2 + 1];
          rs2 = a.lv.rs[r2];
        }
        // every window of a segment has at least 8 bytes before the run end
        const uint64_t i = rs2 + (wi - wo2);
        uint64_t v;
        __builtin_memcpy(&v, T + i, 8);
        m |= (has((uint32_t)v, (uint32_t)(v >> 32)) ? 1u : 0u) << k;
      }
    }
    if (!__ballot(m != 0)) continue;  // most chunks hold no candidate
    // Where many windows pass (runs and other strings that a key's first eight
    // bytes repeat), a step takes windows one sample of the prefix fingerprints
    // apart: the lanes read consecutive samples and add the same number of bytes to
    // them.  (The lanes' next candidates lie 32 bytes apart, two to eight samples.)
    // In chunks of one segment, from 16 lanes with a quarter of their windows each;
    // below that the other order takes fewer steps.  64 MiB with one byte in 256 not
    // zero: 8 launches at tau 2 13.4 -> 6.4 ms, 4 memory-lean ones 7.8 -> 6.0.
    if (__builtin_expect(whole && __popcll(__ballot(fast && __popc(m) >= kByteK / 4)) >= 16, 0)) {
      const uint32_t sh = LEAN ? a.pshift : 0;
      const uint64_t e0 = ((uint64_t)t << kQPosBits) | (rs + (c0 - wo));  // the first window's entry
      for (uint32_t step = 0; step < kByteK; ++step) {
        const uint32_t w = ((step >> sh) << (6 + sh)) + ((uint32_t)lane << sh) + (step & ((1u << sh) - 1));
        push((__shfl(fast ? m : 0u, (int)(w / kByteK)) >> (w % kByteK)) & 1, e0 + w);
      }
      if (fast) m = 0;
    }
    // queue the candidates, each lane's next one in a step: as many steps as the
    // lane with the most has, one or two; lanes that walked segments walk them
    // again, now with the run end and text of each window
    while (__ballot(m != 0)) {
      uint64_t e = 0;
      const bool c = m != 0;
      if (c) {
        const uint64_t wi = w0 + (uint32_t)__builtin_ctz(m);
        m &= m - 1;
        if (!fast) {
          while (wi >= wn) {
            ++r;
            wo = wn;
            wn = woff[r + 1];
            rs = a.lv.rs[r];
            re = a.lv.re[r];
            t = a.lv.rtext[r];
          }
        }
        const uint64_t i = rs + (wi - wo);
        e = ((i + L > re) ? (1ull << 63) : 0) | ((uint64_t)t << kQPosBits) | i;
      }
      push(c, e);
    }
  }
  if (qn) {
    wave_sync();
    if ((uint32_t)lane < qn) check(q[lane]);
  }
  if (a.pc && lane == 0 && ncand) atomicAdd((unsigned long long*)(a.pc + kPcCand), (unsigned long long)ncand);
}

hipError_t launch_byte_scan(const PhaseArgs& a, const uint64_t* woff, bool has_odd, bool has_salt,
                            uint64_t max_windows, hipStream_t s) {
  if (a.bfilt_bits < 12 || a.bfilt_bits > 19) return hipErrorInvalidValue;
  const uint64_t waves = (max_windows + 64 * kByteK - 1) / (64 * kByteK);
  const unsigned grid = grid_for(waves * 64, kByteThreads, 512);
  // filter up to 64 KiB + queues 16 KiB: two 1024-thread workgroups per CU
  const size_t lds = ((size_t)1 << (a.bfilt_bits - 3)) + (size_t)(kByteThreads / 64) * kQueue * 8;
#define BT_BYTE_LAUNCH(O, S, LN)                                                           \
  do {                                                                                     \
    if (lds > 65536) {                                                                     \
      const hipError_t e = allow_lds(reinterpret_cast<const void*>(&k_byte_scan<O, S, LN>), lds); \
      if (e != hipSuccess) return e;                                                       \
    }                                                                                      \
    k_byte_scan<O, S, LN><<<grid, kByteThreads, lds, s>>>(a, woff);                        \
  } while (0)
#define BT_BYTE_SALT(O, LN) \
  if (has_salt) BT_BYTE_LAUNCH(O, true, LN); else BT_BYTE_LAUNCH(O, false, LN);
  if (a.P == nullptr) {
    if (has_odd) {
      BT_BYTE_SALT(true, true)
    } else {
      BT_BYTE_SALT(false, true)
    }
  } else if (has_odd) {
    BT_BYTE_SALT(true, false)
  } else {
    BT_BYTE_SALT(false, false)
  }
#undef BT_BYTE_SALT
#undef BT_BYTE_LAUNCH
  return hipGetLastError();
}

// ---------------------------------------------------------------- verification
//
// A key whose slot minimum is its own position is its own leftmost occurrence;
// any other compares its bytes with the slot's position (verification), and a
// mismatch, a collision, sends it on an exact walk.

constexpr uint64_t kVChunk = kSettleMax;  // bytes compared per work item

__global__ void k_phase_record(uint64_t* pc, const uint64_t* windows, const uint64_t* counts) {
  if (threadIdx.x == 0) {
    pc[kPcWindows] = windows ? *windows : 0;
    pc[kPcVerified] = counts[0];
    pc[kPcCollisions] = counts[1];
  }
}

hipError_t launch_phase_record(uint64_t* pc, const uint64_t* windows, const VerifyBufs& v,
                               hipStream_t s) {
  k_phase_record<<<1, 64, 0, s>>>(pc, windows, v.counts);
  return hipGetLastError();
}

// One wave compares bytes [off, end) of a key with the candidate occurrence, 4 KiB
// requested together.
__device__ __forceinline__ bool wave_bytes_differ(const uint8_t* __restrict__ T, uint64_t a0,
                                                  uint64_t b0, uint64_t off, uint64_t end) {
  bool diff = false;
  for (; off + 4096 <= end; off += 4096) {
    const uint64_t o = off + (uint64_t)lane_id() * 16;
    uint4 x[4], y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[e] = load16(T + a0 + o + 1024 * e);
      y[e] = load16(T + b0 + o + 1024 * e);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      diff |= (x[e].x != y[e].x) | (x[e].y != y[e].y) | (x[e].z != y[e].z) | (x[e].w != y[e].w);
    if (__any(diff)) return true;
  }
  for (uint64_t o = off + (uint64_t)lane_id() * 16; o < end; o += 64 * 16) {
    if (o + 16 <= end) {
      const uint4 x = load16(T + a0 + o);
      const uint4 y = load16(T + b0 + o);
      diff |= (x.x != y.x) | (x.y != y.y) | (x.z != y.z) | (x.w != y.w);
    } else {
      for (uint64_t q = o; q < end; ++q) diff |= T[a0 + q] != T[b0 + q];
    }
  }
  return __any(diff);
}

// Exact fallback after a collision: the wave walks positions lb, lb+1, ... up to
// the start of key j, fingerprints each window, and verifies hits in increasing
// order; the first verified hit is the leftmost occurrence (no true occurrence
// lies before lb, see the file header of bt_host.cpp).  The key's own start
// always verifies, so the walk ends.  Every lane returns it.
__device__ uint64_t wave_walk(const PhaseArgs& a, uint64_t j, uint64_t lb) {
  const int lane = lane_id();
  const uint64_t pos = a.lv.st[j];
  const uint64_t L = a.k.len[j];
  const uint64_t fpk = a.k.fp[j];
  const uint64_t salt = a.tx.tsalt[a.lv.text[j]];
  const uint64_t xp = pow61(a.x, L);
  for (uint64_t p0 = lb; p0 <= pos; p0 += 64) {
    const uint64_t p = p0 + lane;
    const bool m = p <= pos && finish_fp(win61_any(a, p, L, xp), salt, a.fpmask) == fpk;
    uint64_t bal = __ballot(m);
    while (bal) {
      const uint64_t q = p0 + (uint64_t)(__ffsll((unsigned long long)bal) - 1);
      bool diff = false;
      for (uint64_t off = 0; off < L && !diff; off += kVChunk) {
        const uint64_t end = L - off < kVChunk ? L : off + kVChunk;
        diff = wave_bytes_differ(a.T, q, pos, off, end);
      }
      if (!diff) return q;
      bal &= bal - 1;
    }
  }
  return pos;
}

__device__ __forceinline__ uint64_t slot_best(const PhaseArgs& a, uint64_t j, uint32_t s) {
  return s == kOddKey ? a.odd.best[a.lv.text[j]] : a.tab.slots[s].best;
}

// Profiling: add each wave's count n to *p, one update per workgroup (they serialize).
__device__ __forceinline__ void block_count(uint64_t* p, uint64_t n) {
  __shared__ unsigned long long s_n;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  if (lane_id() == 0 && n) atomicAdd(&s_n, (unsigned long long)n);
  __syncthreads();
  if (threadIdx.x == 0 && s_n) atomicAdd((unsigned long long*)p, s_n);
}

// Keys of at most kVChunk bytes: resolved, verified and settled in one launch
// (before, a list of the keys to verify, its verification and its results, each
// writing and reading the list).  A wave takes 64 keys, one per lane; those
// to verify are compared by groups of G lanes, 16 bytes per lane and step, 64 / G
// keys at a time (G: about a key's 16-byte words, 64 for 1 KiB or more), four such
// batches' first words loaded together.  Bound by the random lines it reads (slot,
// occurrence, key).  Builds with one launch in place of three: 256 MiB 8.99 ->
// 8.72 ms, 2 GiB 94.4 -> 91.9 ms, 1 MiB 2.22 -> 2.09 ms.  Walking in this kernel took
// its registers from 79 to 104; held to 64 it spilled, and ran 1.5x slower.
template <int G>
__global__ __launch_bounds__(256) void k_settle(PhaseArgs a, VerifyBufs v) {
  const int lane = lane_id();
  const int sub = lane % G, grp = lane / G;
  constexpr uint32_t per = 64 / G;
  constexpr int kBatch = 4;
  const uint64_t c = a.lv.c;
  uint64_t verified = 0;
  for (uint64_t j0 = ((uint64_t)blockIdx.x * 256 + (threadIdx.x & ~63u)); j0 < c;
       j0 += (uint64_t)gridDim.x * 256) {
    const uint64_t j = j0 + lane;
    bool need = false, bad = false;
    uint64_t best = 0, pos = 0;
    uint32_t len = 0;
    if (j < c) {
      const uint32_t s = a.k.slot[j];
      if (s != kNoKey && s != kCopyKey) {
        pos = a.lv.st[j];
        best = slot_best(a, j, s);
        need = best != pos;
        if (need) {
          len = (uint32_t)a.k.len[j];
          bad = best < a.tx.tstart[a.lv.text[j]];  // hit in another text: a collision
        } else {
          a.k.lm[j] = pos;
        }
      }
    }
    const uint64_t bal = __ballot(need && !bad);
    const uint32_t n = (uint32_t)__popcll(bal);
    const uint32_t rank = (uint32_t)__popcll(bal & ((1ull << lane) - 1));
    verified += (uint64_t)__popcll(__ballot(need));
    // lane k of `order` holds the lane of the k-th key to compare
    const int order = __builtin_amdgcn_ds_permute((need && !bad ? (int)rank : 63) << 2, lane);
    for (uint32_t k0 = 0; k0 < n; k0 += kBatch * per) {
      // kBatch keys per group, their first 16 bytes per lane loaded together
      uint64_t b0[kBatch], p0[kBatch];
      uint32_t L[kBatch];
      uint4 x[kBatch], y[kBatch];
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        const uint32_t k = k0 + e * per + grp;
        const uint32_t src = (uint32_t)__shfl(order, (int)(k < n ? k : 0));
        b0[e] = shfl64(best, src);
        p0[e] = shfl64(pos, src);
        L[e] = __shfl(len, (int)src);
        if (k >= n) L[e] = 0;
        if ((uint32_t)sub * 16 + 16 <= L[e]) {
          x[e] = load16(a.T + b0[e] + sub * 16);
          y[e] = load16(a.T + p0[e] + sub * 16);
        } else {
          x[e] = y[e] = make_uint4(0, 0, 0, 0);
        }
      }
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        bool diff = (x[e].x != y[e].x) | (x[e].y != y[e].y) | (x[e].z != y[e].z) | (x[e].w != y[e].w);
        for (uint32_t o = (uint32_t)sub * 16 + ((uint32_t)sub * 16 + 16 <= L[e] ? G * 16 : 0); o < L[e];
             o += G * 16) {
          if (o + 16 <= L[e]) {
            const uint4 u = load16(a.T + b0[e] + o);
            const uint4 w = load16(a.T + p0[e] + o);
            diff |= (u.x != w.x) | (u.y != w.y) | (u.z != w.z) | (u.w != w.w);
          } else {
            for (uint32_t q = o; q < L[e]; ++q) diff |= a.T[b0[e] + q] != a.T[p0[e] + q];
          }
        }
        const uint64_t dm = __ballot(diff);
        const uint32_t r0 = k0 + e * per;  // the ranks compared here: r0 .. r0 + per - 1
        if (need && !bad && rank >= r0 && rank < r0 + per) {
          const uint64_t mine = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1) << ((rank - r0) * (G & 63));
          if (dm & mine) bad = true;
          else a.k.lm[j] = best;
        }
      }
    }
    if (bad) {  // rare: listed for k_walk, whose registers would halve this kernel's waves
      const uint64_t at = atomicAdd((unsigned long long*)&v.counts[1], 1ull);
      v.vlist[at] = (uint32_t)j;
      v.vbest[at] = best;
    }
  }
  if (a.pc) block_count(&v.counts[0], verified);
}

// The walks of the keys that failed (counts[1] of them listed), one wave each.
__global__ __launch_bounds__(256) void k_walk(PhaseArgs a, VerifyBufs v) {
  const uint64_t cnt = v.counts[1];
  const uint64_t gw = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint64_t nw = ((uint64_t)gridDim.x * blockDim.x) >> 6;
  for (uint64_t i = gw; i < cnt; i += nw) {
    const uint64_t j = v.vlist[i], ts = a.tx.tstart[a.lv.text[j]], lb = v.vbest[i] + 1;
    const uint64_t found = wave_walk(a, j, lb > ts ? lb : ts);
    if (lane_id() == 0) a.k.lm[j] = found;
  }
}

// Longer keys, in chunks of at least kVChunk bytes: item (j, chunk) is one wave's, and
// the wave that ends a key's last chunk (KeysDev.done) settles it, or walks.  A lane
// looks its item up and the wave then takes those to compare in turn, so keys that
// are their own first occurrence cost a lane only; items of a wave are a grid apart,
// which spreads runs of keys to compare over the chip.  At most kMaxChunks chunks a
// key: its waves' counter updates serialize.  Bound by the launch at these lengths (few
// keys).  One launch in place of a list of the keys, its comparison and its results:
// 1 MiB build 1.44 -> 1.32 ms; from 16 MiB on, where the host is behind on these
// levels anyway, 0 to 1%.
constexpr uint64_t kMaxChunks = 2048;  // below 2^16: KeysDev.done counts in 16 bits

__global__ __launch_bounds__(256) void k_settle_long(PhaseArgs a, VerifyBufs v, uint64_t cpk,
                                                     uint64_t chunk) {
  const int lane = lane_id();
  const uint64_t items = a.lv.c * cpk;
  const uint64_t gw = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint64_t nw = ((uint64_t)gridDim.x * blockDim.x) >> 6;
  uint64_t verified = 0;
  for (uint64_t i0 = gw; i0 < items; i0 += nw * 64) {
    const uint64_t it = i0 + (uint64_t)lane * nw;
    bool need = false, other = false;
    uint64_t j = 0, off = 0, best = 0, pos = 0, L = 0;
    if (it < items) {
      j = it / cpk;
      off = (it - j * cpk) * chunk;
      const uint32_t s = a.k.slot[j];
      if (s != kNoKey && s != kCopyKey) {
        pos = a.lv.st[j];
        L = a.k.len[j];
        best = slot_best(a, j, s);
        other = best < a.tx.tstart[a.lv.text[j]];  // hit in another text: a collision
        need = best != pos && off < L;
        if (best == pos && off == 0) a.k.lm[j] = pos;
      }
    }
    verified += (uint64_t)__popcll(__ballot(need && off == 0));
    for (uint64_t m = __ballot(need); m; m &= m - 1) {
      const uint32_t src = (uint32_t)(__ffsll((unsigned long long)m) - 1);
      const uint64_t kj = shfl64(j, src), ko = shfl64(off, src), kl = shfl64(L, src);
      const uint64_t kb = shfl64(best, src), kp = shfl64(pos, src);
      bool bad = __shfl((int)other, (int)src) != 0;
      if (!bad) bad = wave_bytes_differ(a.T, kb, kp, ko, kl - ko < chunk ? kl : ko + chunk);
      const uint32_t nch = (uint32_t)((kl + chunk - 1) / chunk);
      if (nch > 1) {
        uint32_t old = 0;
        if (lane == 0) old = atomicAdd(&a.k.done[kj], bad ? 0x10001u : 1u);
        old = __shfl(old, 0);
        if ((old & 0xFFFFu) + 1 < nch) continue;
        bad |= (old >> 16) != 0;
      }
      uint64_t found = kb;
      if (bad) {
        const uint64_t ts = a.tx.tstart[a.lv.text[kj]];
        found = wave_walk(a, kj, kb + 1 > ts ? kb + 1 : ts);
        if (lane == 0) atomicAdd((unsigned long long*)&v.counts[1], 1ull);
      }
      if (lane == 0) a.k.lm[kj] = found;
    }
  }
  if (a.pc) block_count(&v.counts[0], verified);
}

hipError_t launch_settle(const PhaseArgs& a, const VerifyBufs& v, uint64_t max_len, hipStream_t s) {
  if (max_len > kVChunk) {
    const uint64_t chunk = ((max_len + kMaxChunks - 1) / kMaxChunks + kVChunk - 1) / kVChunk * kVChunk;
    const uint64_t cpk = (max_len + chunk - 1) / chunk;
    if (!a.k.done) return hipErrorInvalidValue;
    k_settle_long<<<grid_for(a.lv.c * cpk * 64, 256, 2048), 256, 0, s>>>(a, v, cpk, chunk);
    return hipGetLastError();
  }
  const unsigned g = grid_for(a.lv.c, 256, 8192);
  // lanes per key: about one 16-byte word per lane, at least 4 lanes
  if (max_len <= 64) k_settle<4><<<g, 256, 0, s>>>(a, v);
  else if (max_len <= 128) k_settle<8><<<g, 256, 0, s>>>(a, v);
  else if (max_len <= 256) k_settle<16><<<g, 256, 0, s>>>(a, v);
  else if (max_len <= 512) k_settle<32><<<g, 256, 0, s>>>(a, v);
  else k_settle<64><<<g, 256, 0, s>>>(a, v);
  k_walk<<<grid_for(a.lv.c * 64, 256, 1024), 256, 0, s>>>(a, v);
  return hipGetLastError();
}

// ---------------------------------------------------------------- leaves (a8)

// Leaf bytes: block j of the last level lands at j*b (texts' regions are
// contiguous; only a text-final block is short, and it ends its region; the
// bytes after its end are written as zeros).  Thread k writes output bytes
// [16k, 16k + 16) with one 16-byte store (the last, partial chunk byte by
// byte).  A chunk inside one block, with 24 bytes of the buffer after its
// source, is read as three aligned 8-byte words; any other chunk byte by byte.
__global__ void k_leaves(const uint8_t* __restrict__ T, LevelDev lv, TextsDev tx,
                         uint8_t* __restrict__ out) {
  const uint64_t total = lv.c * lv.b;
  const uint64_t end = tx.tend[tx.T - 1];  // the buffer's end (texts are in order)
  GRID_STRIDE(k, (total + 15) / 16) {
    const uint64_t p = 16 * k;
    uint64_t j = p / lv.b, r = p - j * lv.b;
    uint64_t len = block_len(lv, tx, j), src = lv.st[j];
    uint64_t lo = 0, hi = 0;
    if (r + 16 <= len && src + r + 24 <= end) {
      bytes16_at(T, end, src + r, lo, hi);
    } else {
      for (int e = 0; e < 16 && p + e < total; ++e) {
        if (r == lv.b) {
          ++j;
          r = 0;
          len = block_len(lv, tx, j);
          src = lv.st[j];
        }
        const uint64_t v = r < len ? T[src + r] : 0;
        (e < 8 ? lo : hi) |= v << (8 * (e & 7));
        ++r;
      }
    }
    if (p + 16 <= total) {
      uint4 w;
      w.x = (uint32_t)lo;
      w.y = (uint32_t)(lo >> 32);
      w.z = (uint32_t)hi;
      w.w = (uint32_t)(hi >> 32);
      *reinterpret_cast<uint4*>(out + p) = w;
    } else {
      for (uint64_t e = 0; p + e < total; ++e) out[p + e] = (uint8_t)((e < 8 ? lo : hi) >> (8 * (e & 7)));
    }
  }
}

hipError_t launch_leaves(const uint8_t* T, const LevelDev& lv, const TextsDev& tx, uint8_t* out,
                         hipStream_t s) {
  if (!lv.c) return hipSuccess;
  k_leaves<<<grid_for((lv.c * lv.b + 15) / 16, 256), 256, 0, s>>>(T, lv, tx, out);
  return hipGetLastError();
}

}  // namespace bt
