// xmem_prep.hip -- trace preparation upstream of the Memory Simulator, on MI355X (gfx950).
//
//   xmem_lifecycles   Section 3.2: pair raw allocator events by address into
//                     memory blocks.  A stable sort by a hash of (trace, address)
//                     puts every address's events next to each other in stream
//                     order; an allocation is closed by the next event of its
//                     address when that is a free.
//   xmem_attribute    Section 3.2: link each block to the operator window it
//                     belongs to.  Per block: a binary search for the last
//                     window of its trace that starts no later than the
//                     allocation, a climb to the innermost window containing
//                     it, then the two rules tried outward.  Section 3.3 item
//                     5: the sizes of each trace's parameter blocks go into a
//                     per-trace open-addressing hash set, and a product
//                     allocated in an optimizer.step() phase whose size is in
//                     it becomes an optimizer state.  Kept blocks are
//                     compacted by a scan.
//   xmem_orchestrate  Section 3.3: retime each block's free by category, then
//                     a stable sort of the allocations and frees by (trace,
//                     time, rank) gives the Simulator's event order, and a
//                     scatter writes the event words.
//
// Long batches are HBM-bound, short ones bound by launches.  The sort is an LSD radix sort of
// (64-bit key, 32-bit value) pairs, 9 bits a pass (35 bits of (trace, time) in four passes, where
// 8-bit digits took five), in three kernels per pass:
//   k_rs_hist     digit histogram of each 4096-element tile;
//   k_rs_rows     one workgroup per digit: exclusive scan of its tiles' counts;
//   k_rs_scatter  each wavefront ranks its 64-element steps with nine
//                 ballots (lanes with the same digit; stable by lane order),
//                 the tile is reordered by digit in LDS, and each digit's run
//                 is written to consecutive addresses.
// The pairing needs equal keys to meet, not an order, so it sorts by 18, 27 or 36 bits of a hash:
// the passes are known on the host, whatever the addresses span.  The orchestration sorts by time,
// rebased to its batch's minimum, over the passes its span needs.  Up to 8,192 records are sorted
// by one workgroup in one launch, and no flags are scanned: per tile counts, added up by the
// kernels that use them.  One profile of 4,001 events takes 15 launches instead of 148: 535 -> 200 us
// for the three steps (with their host calls); 128 profiles of 65,536 events 2,045 -> 1,585 us.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <stddef.h>
#include <stdint.h>

#include "xmem.h"
#include "xmem_prep.h"

namespace {

constexpr int kThreads = 256;             // 4 wavefronts
constexpr int kItems = 16;                // elements per lane per tile
constexpr int kTileN = kThreads * kItems;  // 4096
constexpr int kDigit = 9;                 // bits a radix pass sorts by
constexpr int kBins = 1 << kDigit;
constexpr int kSteps = kTileN / 64;       // 64-record steps of a tile
constexpr int kWaves = kThreads / 64;
constexpr int kScanThreads = 1024;
constexpr int kXcds = 8;
// the kernels that work on records (not the sort's passes): a tile per workgroup of 1024, whose
// chains of dependent loads (window climbs, marker searches) need the wavefronts
constexpr int kRecThreads = 1024;
constexpr int kRecItems = kTileN / kRecThreads;
constexpr int64_t kPersist = INT64_MAX;
constexpr uint64_t kFree = 1ull << 63;

__host__ __device__ inline size_t al256(size_t x) { return (x + 255) & ~size_t(255); }
__host__ __device__ inline int64_t tiles_of(int64_t n) { return (n + kTileN - 1) / kTileN; }

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
// a sort pass over bits [sh, sh + kDigit) runs only below the key width found on the device (*gate)
__device__ __forceinline__ bool gated(const int32_t* gate, int sh) { return gate && sh >= *gate; }

// ---------------------------------------------------------------- scans
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t old, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xf, false);
}
// inclusive scan up the wavefront in lane order on DPP alone: shifts by 1, 2, 4 and 8 lanes within
// each row of 16, then row 0's total into row 1 and row 2's into row 3 (row_bcast:15), then rows
// 0-1's total into rows 2-3 (row_bcast:31).  All lanes active.
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t x) {
  x += dpp_u32<0x111, 0xf>(0, x);
  x += dpp_u32<0x112, 0xf>(0, x);
  x += dpp_u32<0x114, 0xf>(0, x);
  x += dpp_u32<0x118, 0xf>(0, x);
  x += dpp_u32<0x142, 0xa>(0, x);
  x += dpp_u32<0x143, 0xc>(0, x);
  return x;
}
// exclusive scan of v over the workgroup's kThreads threads; *total gets the sum (s: kWaves words)
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* s, uint32_t* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t x = wave_scan_u32(v);
  if (lane == 63) s[wv] = x;
  __syncthreads();
  uint32_t before = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) {
    before += k < wv ? s[k] : 0u;
    tot += s[k];
  }
  __syncthreads();
  *total = tot;
  return before + x - v;
}
// exclusive scan of part[0..np) in place, one workgroup
__global__ __launch_bounds__(kScanThreads) void k_scan_top(uint32_t* part, int64_t np) {
  __shared__ uint32_t s[kScanThreads / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t per = (np + kScanThreads - 1) / kScanThreads;
  const int64_t lo = (int64_t)threadIdx.x * per;
  uint32_t acc = 0;
  for (int64_t i = lo; i < lo + per && i < np; ++i) acc += part[i];
  const uint32_t x = wave_scan_u32(acc);
  if (lane == 63) s[wv] = x;
  __syncthreads();
  uint32_t run = x - acc;
#pragma unroll
  for (int k = 0; k < kScanThreads / 64; ++k) run += k < wv ? s[k] : 0u;
  for (int64_t i = lo; i < lo + per && i < np; ++i) {
    const uint32_t v = part[i];
    part[i] = run;
    run += v;
  }
}

// Flags of a tile's records (record kRecThreads i + thread of the tile: every load coalesced), as one
// ballot per 64-record step, and the flagged records before each step.
struct TileFlags {
  uint64_t m[kSteps];
  uint32_t before[kSteps + 1];  // [kSteps]: all of the tile
};
__device__ __forceinline__ void flags_put(TileFlags& f, int i, bool flag) {
  const uint64_t m = ballot(flag);
  if ((threadIdx.x & 63) == 0) f.m[i * (kRecThreads / 64) + (threadIdx.x >> 6)] = m;
}
__device__ __forceinline__ void flags_scan(TileFlags& f) {
  static_assert(kSteps == 64, "one wavefront scans the steps");
  __syncthreads();
  if (threadIdx.x < 64) {
    const uint32_t c = (uint32_t)__builtin_popcountll(f.m[threadIdx.x]);
    const uint32_t x = wave_scan_u32(c);
    f.before[threadIdx.x] = x - c;
    if (threadIdx.x == 63) f.before[kSteps] = x;
  }
  __syncthreads();
}
// flagged records of the tile before its record r <= kTileN
__device__ __forceinline__ uint32_t flags_before(const TileFlags& f, int r) {
  if (r >= kTileN) return f.before[kSteps];
  return f.before[r >> 6] + (uint32_t)__builtin_popcountll(f.m[r >> 6] & ((1ull << (r & 63)) - 1));
}

// What the tiles before this one hold: part scanned by k_scan_top, or, up to kPartTiles tiles,
// added up here (one load a thread instead of a launch).  Every thread of the kRecThreads calls it.
constexpr int64_t kPartTiles = kRecThreads;
__device__ __forceinline__ uint32_t tile_before(const uint32_t* part, int64_t ntiles) {
  if (ntiles > kPartTiles) return part[blockIdx.x];
  __shared__ uint32_t s[kRecThreads / 64];
  const uint32_t x = wave_scan_u32((int)threadIdx.x < (int)blockIdx.x ? part[threadIdx.x] : 0u);
  if ((threadIdx.x & 63) == 63) s[threadIdx.x >> 6] = x;
  __syncthreads();
  uint32_t t = 0;
#pragma unroll
  for (int k = 0; k < kRecThreads / 64; ++k) t += s[k];
  return t;
}
void scan_parts(uint32_t* part, int64_t ntiles, hipStream_t st) {
  if (ntiles > kPartTiles) k_scan_top<<<1, kScanThreads, 0, st>>>(part, ntiles);
}

// ---------------------------------------------------------------- traces of records
// The first index i in [0, n] with v[i] >= x (v ascending, n: none), found by one whole wavefront:
// each round looks at 64 evenly spaced entries, where a binary search takes a dependent load a
// halving.
__device__ __forceinline__ int64_t wave_lower_bound(const int64_t* v, int64_t n, int64_t x) {
  const int lane = threadIdx.x & 63;
  int64_t lo = 0, hi = n;  // the answer is in [lo, hi]
  while (lo < hi) {
    const int64_t step = (hi - lo + 63) / 64;
    const int64_t p = lo + lane * step;
    const uint64_t m = ballot(p < hi && v[p] < x);  // a prefix of the lanes
    if (m == 0) return lo;
    const int64_t last = lo + (63 - __builtin_clzll(m)) * step;
    const int64_t next = last + step;
    lo = last + 1;
    hi = next < hi ? next : hi;
  }
  return lo;
}
// The last trace that starts at or before record base (workgroup-wide; every thread calls it).
__device__ __forceinline__ int64_t tile_trace(const int64_t* off, int64_t T, int64_t base) {
  __shared__ int64_t s_t;
  if (threadIdx.x < 64) {
    const int64_t t = wave_lower_bound(off, T, base + 1) - 1;  // off[0] == 0
    if (threadIdx.x == 0) s_t = t;
  }
  __syncthreads();
  return s_t;
}
// A thread's walk over its records in ascending order: the trace of each, the last one that starts
// at or before it (which steps over empty traces).  The steps double and are then halved: a tile of
// short traces, or with many empty ones between its records, takes a few dependent loads a record
// where a step a trace took one for each of them (1,000,000 traces, 50,000 of them of one event and
// the others empty: the three steps 181 -> 0.9 ms; 200,000 of 0 to 5 events: 2.8 -> 0.57 ms).
struct TraceStep {
  int64_t t, next;
  __device__ __forceinline__ TraceStep(const int64_t* off, int64_t T, int64_t t0) : t(t0) {
    next = t + 1 < T ? off[t + 1] : INT64_MAX;
  }
  __device__ __forceinline__ void to(const int64_t* off, int64_t T, int64_t k) {
    if (k < next) return;
    int64_t lo = t + 1, hi = lo + 1;  // trace lo starts at or before k
    next = hi < T ? off[hi] : INT64_MAX;
    while (k >= next) {
      const int64_t step = 2 * (hi - t);
      lo = hi;
      hi = lo + step < T ? lo + step : T;
      next = hi < T ? off[hi] : INT64_MAX;
    }
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1, o = off[mid];
      if (o <= k) {
        lo = mid;
      } else {
        hi = mid;
        next = o;
      }
    }
    t = lo;
  }
};
// The traces that start in the tile [base, base + kTileN) of n records, with those that start at n
// (and the end, T) in the last tile: out[t] = at + per * (records of the tile before it) + its flagged ones.
__device__ __forceinline__ void tile_offsets(const int64_t* off, int64_t T, int64_t n, int64_t base, const TileFlags& f,
                                             uint32_t at, int per, int64_t* out) {
  __shared__ int64_t s_r[2];
  const bool last = base + kTileN >= n;
  if (threadIdx.x < 64) {
    const int64_t a = wave_lower_bound(off, T + 1, base), b = last ? T + 1 : wave_lower_bound(off, T + 1, base + kTileN);
    if (threadIdx.x == 0) { s_r[0] = a; s_r[1] = b; }
  }
  __syncthreads();
  for (int64_t t = s_r[0] + threadIdx.x; t < s_r[1]; t += kRecThreads) {
    const int r = (int)(off[t] - base);
    out[t] = (int64_t)at + (int64_t)per * r + flags_before(f, r);
  }
}

// ---------------------------------------------------------------- LSD radix sort
// One record's digit into the tile's histogram.  A wavefront whose elements share one digit (the
// high digits of keys sorted by the low ones) adds once: 64 atomics on one LDS word would be serialized.
__device__ __forceinline__ void hist_add(uint32_t* h, bool ok, uint32_t d) {
  const uint64_t act = ballot(ok);
  const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
  const uint64_t same = ballot(ok && d == d0);
  if (same == act) {
    if (act && (threadIdx.x & 63) == (uint32_t)__builtin_ctzll(act)) atomicAdd(&h[d0], (uint32_t)__builtin_popcountll(act));
  } else if (ok) {
    atomicAdd(&h[d], 1u);
  }
}
__device__ __forceinline__ void hist_clear(uint32_t* h) {
  for (int d = threadIdx.x; d < kBins; d += blockDim.x) h[d] = 0;
  __syncthreads();
}
// digit-major: hist[d * ntiles + tile]
__device__ __forceinline__ void hist_store(const uint32_t* h, uint32_t* hist, int64_t ntiles) {
  __syncthreads();
  for (int d = threadIdx.x; d < kBins; d += blockDim.x) hist[(int64_t)d * ntiles + blockIdx.x] = h[d];
}
// The digit of a key: its own bits, or (HASHED) those of a hash of it without its lowest bit, where
// the order of different keys does not matter but only that equal ones meet (kHashBits bits spread
// evenly, so the passes are known beforehand, whatever the keys span).
constexpr int kHashBits = 4 * kDigit;
template <bool HASHED>
__device__ __forceinline__ uint32_t digit_of(uint64_t key, int shift) {
  const uint64_t x = HASHED ? ((key | 1) * 0x9E3779B97F4A7C15ull) >> (64 - kHashBits) : key;
  return (uint32_t)(x >> shift) & (kBins - 1);
}
// digit histogram of each tile
template <bool HASHED>
__global__ __launch_bounds__(kThreads) void k_rs_hist(const uint64_t* keys, int64_t n, int shift, uint32_t* hist,
                                                      int64_t ntiles, const int32_t* gate) {
  if (gated(gate, shift)) return;
  __shared__ uint32_t h[kBins];
  hist_clear(h);
  const int64_t base = (int64_t)blockIdx.x * kTileN;
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const int64_t k = base + (int64_t)i * kThreads + threadIdx.x;
    const bool ok = k < n;
    hist_add(h, ok, ok ? digit_of<HASHED>(keys[k], shift) : 0u);
  }
  hist_store(h, hist, ntiles);
}
// one workgroup per digit: its tiles' counts become an exclusive scan, its total goes to tot
__global__ __launch_bounds__(kThreads) void k_rs_rows(uint32_t* hist, int64_t ntiles, uint32_t* tot, const int32_t* gate,
                                                      int shift) {
  if (gated(gate, shift)) return;
  __shared__ uint32_t s[kWaves];
  uint32_t* row = hist + (int64_t)blockIdx.x * ntiles;
  constexpr int kPer = 8;
  uint32_t carry = 0;
  for (int64_t b = 0; b < ntiles; b += kThreads * kPer) {
    const int64_t i0 = b + (int64_t)threadIdx.x * kPer;
    uint32_t v[kPer], acc = 0, total;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      v[j] = i0 + j < ntiles ? row[i0 + j] : 0u;
      acc += v[j];
    }
    uint32_t run = carry + block_excl_scan(acc, s, &total);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      if (i0 + j < ntiles) row[i0 + j] = run;
      run += v[j];
    }
    carry += total;
  }
  if (threadIdx.x == 0) tot[blockIdx.x] = carry;
}

// Stable scatter of one tile by one digit.  off[d * ntiles + tile]: this tile's elements of digit d
// go after that many of the digit's; tot[d]: the digit's elements.
template <bool HASHED>
__global__ __launch_bounds__(kThreads, 4) void k_rs_scatter(const uint64_t* kin, const uint32_t* vin, uint64_t* kout,
                                                         uint32_t* vout, int64_t n, int shift, const uint32_t* off,
                                                         const uint32_t* tot, int64_t ntiles, const int32_t* gate) {
  if (gated(gate, shift)) return;
  // workgroups go round-robin over the 8 XCDs: each takes a contiguous eighth of the tiles, so that
  // the lines shared by the runs of neighbouring tiles fill up in one L2 (128 profiles of 65,536
  // events: 1,658 -> 1,610 us for the three steps)
  const int64_t tile = (int64_t)(blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
  if (tile >= ntiles) return;
  // the tile in output order: keys, then values (two phases); before that, per-wavefront digit
  // counts and their exclusive scan (so that the LDS allows four workgroups per CU)
  __shared__ uint64_t sk[kTileN];
  uint32_t(*wcnt)[kBins] = reinterpret_cast<uint32_t(*)[kBins]>(sk);
  static_assert(sizeof(uint32_t) * kWaves * kBins <= sizeof(sk), "the counts fit in the tile");
  __shared__ uint32_t tbase[kBins];  // start of each digit in the tile's local order
  __shared__ uint32_t gbase[kBins];  // where the digit's run starts in the output, less tbase
  __shared__ uint32_t s_w[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint64_t below = (1ull << lane) - 1;
  for (int d = lane; d < kBins; d += 64) wcnt[wv][d] = 0;
  const int64_t base = tile * kTileN + (int64_t)wv * (kTileN / kWaves);
  uint64_t key[kItems];
  uint32_t val[kItems], rd[kItems];  // rank in the wavefront's digit run | digit << 16 (kBins: no element)
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const int64_t k = base + (int64_t)i * 64 + lane;
    const bool ok = k < n;
    key[i] = ok ? kin[k] : 0;
    val[i] = ok ? vin[k] : 0;
    const uint32_t d = digit_of<HASHED>(key[i], shift);
    uint64_t peers = ballot(ok);
#pragma unroll
    for (int b = 0; b < kDigit; ++b) {
      const uint64_t bb = ballot((d >> b) & 1u);
      peers &= ((d >> b) & 1u) ? bb : ~bb;
    }
    const uint32_t before = (uint32_t)__builtin_popcountll(peers & below);
    const uint32_t c = wcnt[wv][d];
    rd[i] = (c + before) | ((ok ? d : (uint32_t)kBins) << 16);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    if (ok && before == 0) wcnt[wv][d] = c + (uint32_t)__builtin_popcountll(peers);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  }
  __syncthreads();
  {  // thread tid owns digits 2 tid and 2 tid + 1: exclusive scans over the wavefronts, then over the digits
    uint32_t cnt[2], all[2], t;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int d = 2 * tid + j;
      uint32_t s = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = wcnt[w][d];
        wcnt[w][d] = s;
        s += c;
      }
      cnt[j] = s;
      all[j] = tot[d];
    }
    static_assert(kBins == 2 * kThreads, "two digits a thread");
    const uint32_t local = block_excl_scan(cnt[0] + cnt[1], s_w, &t), global = block_excl_scan(all[0] + all[1], s_w, &t);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int d = 2 * tid + j;
      const uint32_t tb = local + (j ? cnt[0] : 0u);
      tbase[d] = tb;
      gbase[d] = global + (j ? all[0] : 0u) + off[(int64_t)d * ntiles + tile] - tb;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kItems; ++i) {  // rd becomes the element's place in the tile (all ones: no element)
    const uint32_t d = rd[i] >> 16;
    rd[i] = d < kBins ? tbase[d] + wcnt[wv][d] + (rd[i] & 0xffffu) : 0xffffffffu;
  }
  __syncthreads();  // the counts are read: the keys take their place
#pragma unroll
  for (int i = 0; i < kItems; ++i)
    if (rd[i] != 0xffffffffu) sk[rd[i]] = key[i];
  __syncthreads();
  const int64_t cnt = n - tile * kTileN < kTileN ? n - tile * kTileN : kTileN;
  // sorted place tid + kThreads j of the tile: its output index (below XMEM_PREP_MAX_RECORDS)
  uint32_t out_at[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {  // digit runs go to consecutive output addresses
    const int i = tid + j * kThreads;
    out_at[j] = 0xffffffffu;
    if (i < cnt) {
      const uint64_t k = sk[i];
      out_at[j] = gbase[digit_of<HASHED>(k, shift)] + (uint32_t)i;
      kout[out_at[j]] = k;
    }
  }
  __syncthreads();
  uint32_t* sv = reinterpret_cast<uint32_t*>(sk);
#pragma unroll
  for (int i = 0; i < kItems; ++i)
    if (rd[i] != 0xffffffffu) sv[rd[i]] = val[i];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j)
    if (out_at[j] != 0xffffffffu) vout[out_at[j]] = sv[tid + j * kThreads];
}

struct SortWs {
  uint64_t *ka, *kb;
  uint32_t *va, *vb;
  uint32_t* hist;
  uint32_t* tot;  // kBins
};

// Sorts (ka, va)[0..n) by key bits [lo, hi), stably; returns true when the
// result is in (kb, vb), false when in (ka, va).  With a gate, the passes at and
// above bit *gate (found on the device) exit at once.  hist_done: the first
// pass's histogram is in place.
template <bool HASHED>
bool sort_bits(SortWs& w, int64_t n, int lo, int hi, bool in_b, hipStream_t st, const int32_t* gate, bool hist_done = false) {
  const int64_t nt = tiles_of(n);
  for (int sh = lo; sh < hi; sh += kDigit) {
    uint64_t* kin = in_b ? w.kb : w.ka;
    uint32_t* vin = in_b ? w.vb : w.va;
    uint64_t* kout = in_b ? w.ka : w.kb;
    uint32_t* vout = in_b ? w.va : w.vb;
    if (sh > lo || !hist_done) k_rs_hist<HASHED><<<(unsigned)nt, kThreads, 0, st>>>(kin, n, sh, w.hist, nt, gate);
    k_rs_rows<<<kBins, kThreads, 0, st>>>(w.hist, nt, w.tot, gate, sh);
    k_rs_scatter<HASHED><<<(unsigned)((nt + kXcds - 1) / kXcds * kXcds), kThreads, 0, st>>>(kin, vin, kout, vout, n, sh, w.hist, w.tot, nt, gate);
    in_b = !in_b;
  }
  return in_b;
}
constexpr int kAllBits = (64 + kDigit - 1) / kDigit * kDigit;

int passes_for(int64_t maxval) {  // passes that values 0..maxval take
  int b = 0;
  while (b < 63 && (maxval >> b) != 0) ++b;
  return (b + kDigit - 1) / kDigit;
}

// The same sort of at most kOneRecords records by one workgroup, pass after pass in one launch (a
// pass of the kernels above costs its three launches, 3 to 4 us each, however few the records).
// Sorts from (ka, va) or (kb, vb) by bits [lo, hi) and returns where the result lies.  Every
// thread calls it.
constexpr int kOneThreads = 1024, kOneWaves = kOneThreads / 64, kOneItems = 8;
constexpr int64_t kOneRecords = kOneThreads * kOneItems;
struct OneLds {
  uint32_t cnt[kOneWaves][kBins];  // a wavefront's digit counts, then where its run of each digit starts
  uint32_t w[kOneWaves];
};
template <bool HASHED>
__device__ __forceinline__ bool sort_one(OneLds& s, uint64_t* ka, uint32_t* va, uint64_t* kb, uint32_t* vb, int n, int lo,
                                         int hi, bool in_b) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint64_t below = (1ull << lane) - 1;
  for (int sh = lo; sh < hi; sh += kDigit) {
    const uint64_t* kin = in_b ? kb : ka;
    const uint32_t* vin = in_b ? vb : va;
    uint64_t* kout = in_b ? ka : kb;
    uint32_t* vout = in_b ? va : vb;
    for (int d = lane; d < kBins; d += 64) s.cnt[wv][d] = 0;
    uint64_t key[kOneItems];
    uint32_t val[kOneItems], rd[kOneItems];  // rank in the wavefront's digit run | digit << 16
#pragma unroll
    for (int i = 0; i < kOneItems; ++i) {  // each wavefront its 512 consecutive records
      const int k = wv * (64 * kOneItems) + i * 64 + lane;
      const bool ok = k < n;
      key[i] = ok ? kin[k] : 0;
      val[i] = ok ? vin[k] : 0;
      const uint32_t d = digit_of<HASHED>(key[i], sh);
      uint64_t peers = ballot(ok);
#pragma unroll
      for (int b = 0; b < kDigit; ++b) {
        const uint64_t bb = ballot((d >> b) & 1u);
        peers &= ((d >> b) & 1u) ? bb : ~bb;
      }
      const uint32_t before = (uint32_t)__builtin_popcountll(peers & below), c = s.cnt[wv][d];
      rd[i] = (c + before) | (d << 16);
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      if (ok && before == 0) s.cnt[wv][d] = c + (uint32_t)__builtin_popcountll(peers);
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    __syncthreads();
    {  // thread tid owns digit tid: a scan over the digits, then over the wavefronts
      uint32_t c = 0;
      if (tid < kBins)
        for (int q = 0; q < kOneWaves; ++q) c += s.cnt[q][tid];
      const uint32_t x = wave_scan_u32(c);
      if (lane == 63) s.w[wv] = x;
      __syncthreads();
      if (tid < kBins) {
        uint32_t run = x - c;
        for (int k = 0; k < wv; ++k) run += s.w[k];
        for (int q = 0; q < kOneWaves; ++q) {
          const uint32_t m = s.cnt[q][tid];
          s.cnt[q][tid] = run;
          run += m;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kOneItems; ++i) {
      if (wv * (64 * kOneItems) + i * 64 + lane < n) {
        const uint32_t at = s.cnt[wv][rd[i] >> 16] + (rd[i] & 0xffffu);
        kout[at] = key[i];
        vout[at] = val[i];
      }
    }
    __syncthreads();
    in_b = !in_b;
  }
  return in_b;
}

// ---------------------------------------------------------------- workspace
struct PrepWs {
  SortWs s;
  uint32_t* part;    // tiles: flagged records of each tile, then their exclusive scan
  uint32_t* total;   // 1: their sum
  uint32_t* tid;     // n: trace of each record (separate key layouts), or the attribution's kept flags
  int64_t* t64;      // n: per-record int64 scratch (free time of an allocation / retimed free of a block),
                     // or the attribution's parameter-size hash sets (2 u32 slots per block)
  uint32_t* apos;    // n: position of an allocation word within its trace
  int32_t* bad;      // 1
  uint64_t* kr;      // 8: the orchestration's times on the device: kr[0] their minimum, kr[1] their maximum; its
                     // sorts' gates (32 bits each, from kr[3] on); their layout (kr[5], see k_orch_keys)
};

size_t carve(void* base, int64_t T, int64_t n, PrepWs* w) {
  size_t o = 0;
  char* b = static_cast<char*>(base);
  auto take = [&](size_t bytes) { char* p = b ? b + o : nullptr; o += al256(bytes); return p; };
  const int64_t nt = tiles_of(n > 0 ? n : 1);
  const int64_t hist_n = (int64_t)kBins * nt;
  PrepWs x;
  x.s.ka = reinterpret_cast<uint64_t*>(take(8 * n));
  x.s.kb = reinterpret_cast<uint64_t*>(take(8 * n));
  x.s.va = reinterpret_cast<uint32_t*>(take(4 * n));
  x.s.vb = reinterpret_cast<uint32_t*>(take(4 * n));
  x.s.hist = reinterpret_cast<uint32_t*>(take(4 * hist_n));
  x.s.tot = reinterpret_cast<uint32_t*>(take(4 * kBins));
  x.part = reinterpret_cast<uint32_t*>(take(4 * nt));
  x.total = reinterpret_cast<uint32_t*>(take(4));
  x.tid = reinterpret_cast<uint32_t*>(take(4 * n));
  x.t64 = reinterpret_cast<int64_t*>(take(8 * n));
  x.apos = reinterpret_cast<uint32_t*>(take(4 * n));
  x.bad = reinterpret_cast<int32_t*>(take(4));
  x.kr = reinterpret_cast<uint64_t*>(take(64));
  (void)T;
  if (w) *w = x;
  return o;
}

// ---------------------------------------------------------------- the start of a call
// One of a call's offset arrays: valid when off[0] == 0, non-decreasing, off[T] == n (n < 0: any end).
struct Offsets { const int64_t* off; int64_t n; };
__device__ __forceinline__ bool offsets_bad(const Offsets& o, int64_t T, int64_t i) {
  if (!o.off) return false;
  return (i == 0 && (o.off[0] != 0 || (o.n >= 0 && o.off[T] != o.n))) || (i < T && o.off[i + 1] < o.off[i]);
}
// Checks the offsets, clears the key range and zeroes zero[0..T).  One workgroup (at most
// kBeginTraces traces) also settles the rest: *bad, the status, and zero output offsets when the
// batch is rejected or empty.  More workgroups find *bad zeroed, and k_finish settles it.
constexpr int64_t kBeginTraces = 16384;
__global__ __launch_bounds__(kScanThreads) void k_begin(Offsets a, Offsets b, Offsets c, int64_t T, bool empty, int64_t* zero,
                                                       uint64_t* kr, int32_t* bad, int32_t* status, int64_t* out) {
  __shared__ int s_bad;
  if (threadIdx.x == 0) s_bad = 0;
  __syncthreads();
  bool mine = false;
  for (int64_t i = (int64_t)blockIdx.x * kScanThreads + threadIdx.x; i <= T; i += (int64_t)gridDim.x * kScanThreads) {
    mine = mine || offsets_bad(a, T, i) || offsets_bad(b, T, i) || offsets_bad(c, T, i);
    if (zero && i < T) zero[i] = 0;
  }
  if (mine) s_bad = 1;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    kr[0] = ~0ull;
    kr[1] = 0;
  }
  __syncthreads();
  if (gridDim.x > 1) {
    if (threadIdx.x == 0 && s_bad) atomicOr(bad, 1);
    return;
  }
  if (threadIdx.x == 0) {
    *bad = s_bad;
    *status = s_bad ? XMEM_T_BAD_BATCH : 0;
  }
  if (s_bad || empty)
    for (int64_t i = threadIdx.x; i <= T; i += kScanThreads) out[i] = 0;
}
__global__ void k_zero_i32(int32_t* p) { *p = 0; }
__global__ __launch_bounds__(kThreads) void k_finish(int64_t T, bool empty, const int32_t* bad, int32_t* status, int64_t* out) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i == 0) *status = *bad ? XMEM_T_BAD_BATCH : 0;
  if ((*bad || empty) && i <= T) out[i] = 0;
}

unsigned grid_of(int64_t n, int t) { return (unsigned)((n + t - 1) / t > 0 ? (n + t - 1) / t : 1); }

void begin(Offsets a, Offsets b, Offsets c, int64_t T, bool empty, int64_t* zero, const PrepWs& w, int32_t* status,
           int64_t* out, hipStream_t st) {
  const unsigned g = T <= kBeginTraces ? 1u : grid_of(T + 1, kScanThreads);
  if (g > 1) k_zero_i32<<<1, 1, 0, st>>>(w.bad);
  k_begin<<<g, kScanThreads, 0, st>>>(a, b, c, T, empty, zero, w.kr, w.bad, status, out);
}
void finish(int64_t T, bool empty, const PrepWs& w, int32_t* status, int64_t* out, hipStream_t st) {
  if (T > kBeginTraces) k_finish<<<grid_of(T + 1, kThreads), kThreads, 0, st>>>(T, empty, w.bad, status, out);
}

// ---------------------------------------------------------------- key ranges
// A sort key spans fewer bits than its 64: kr receives the minimum and maximum of the keys that
// take part.  The key then sorts as key - min, over the passes its width needs.
// a thread's running part of a range
struct RangePart {
  uint64_t mn = ~0ull, mx = 0;
  __device__ void add(bool in, uint64_t v) {
    mn = in && v < mn ? v : mn;
    mx = in && v > mx ? v : mx;
  }
};
// the workgroup's parts combined (wavefront butterflies, then LDS), then one atomic per word
__device__ __forceinline__ void range_commit(uint64_t* kr, RangePart p) {
  __shared__ uint64_t s[2][kRecThreads / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t a = __shfl_xor(p.mn, o, 64), b = __shfl_xor(p.mx, o, 64);
    p.mn = a < p.mn ? a : p.mn;
    p.mx = b > p.mx ? b : p.mx;
  }
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { s[0][wv] = p.mn; s[1][wv] = p.mx; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < (int)blockDim.x / 64; ++k) {
      p.mn = s[0][k] < p.mn ? s[0][k] : p.mn;
      p.mx = s[1][k] > p.mx ? s[1][k] : p.mx;
    }
    if (p.mn <= p.mx) {
      atomicMin((unsigned long long*)&kr[0], (unsigned long long)p.mn);
      atomicMax((unsigned long long*)&kr[1], (unsigned long long)p.mx);
    }
  }
}
// bits of max - min
__device__ __forceinline__ int range_bits(const uint64_t* kr) {
  const uint64_t span = kr[0] <= kr[1] ? kr[1] - kr[0] : 0;
  return span ? 64 - __builtin_clzll(span) : 0;
}
// the pass gate of a range: an even number of passes, so that a gated sort ends in the buffer it
// started from
__device__ __forceinline__ int32_t range_gate(const uint64_t* kr) {
  const int passes = (range_bits(kr) + kDigit - 1) / kDigit;
  return kDigit * (passes + (passes & 1));
}

constexpr uint64_t kJoint = 1, kJointBuf = 2;  // orchestration: the sort's layout (kr[5], k_orch_keys)
// A record's key: equal exactly for the allocations and frees of one (trace, address), but for the
// lowest bit, which marks a free.  (trace, address) itself when the address is below 2^47 and the
// trace below 2^15; else (kWide) 61 bits mixed from both, whose equality the pairing verifies on
// the records.  A 0-byte record takes no part: a key of its own (kNone).
constexpr uint64_t kNone = 3ull << 62, kWide = 1ull << 63;
__device__ __forceinline__ uint64_t life_key(uint64_t t, uint64_t addr, int64_t bytes, int64_t k) {
  const uint64_t free = bytes < 0 ? 1u : 0u;
  if (bytes == 0) return kNone | ((uint64_t)k << 1);
  if (addr < (1ull << 47) && t < (1ull << 15)) return (t << 48) | (addr << 1) | free;
  uint64_t x = (addr ^ (t * 0xD6E8FEB86659FD93ull)) * 0xD6E8FEB86659FD93ull;
  x = (x ^ (x >> 32)) * 0xD6E8FEB86659FD93ull;
  return kWide | (((x ^ (x >> 32)) & ((1ull << 61) - 1)) << 1) | free;
}
// Keys and record indices, per tile its allocations (part), and the first pass's digit histogram.
__global__ __launch_bounds__(kRecThreads) void k_life_keys(const xmem_raw_event* raw, const int64_t* off, int64_t n, int64_t T,
                                                           const int32_t* bad, uint64_t* key, uint32_t* val, int shift,
                                                           uint32_t* hist, int64_t ntiles, uint32_t* part) {
  if (*bad) return;
  __shared__ uint32_t h[kBins];
  __shared__ uint32_t s_cnt;
  if (threadIdx.x == 0) s_cnt = 0;
  hist_clear(h);
  const int64_t base = (int64_t)blockIdx.x * kTileN;
  TraceStep tr(off, T, tile_trace(off, T, base));
  uint32_t allocs = 0;
#pragma unroll
  for (int i = 0; i < kRecItems; ++i) {
    const int64_t k = base + (int64_t)i * kRecThreads + threadIdx.x;
    const bool ok = k < n;
    uint64_t x = 0;
    if (ok) {
      tr.to(off, T, k);
      const int64_t bytes = raw[k].bytes;
      x = life_key((uint64_t)tr.t, raw[k].addr, bytes, k);
      key[k] = x;
      val[k] = (uint32_t)k;
      allocs += bytes > 0 ? 1u : 0u;
    }
    hist_add(h, ok, digit_of<true>(x, shift));
  }
  atomicAdd(&s_cnt, allocs);
  hist_store(h, hist, ntiles);
  if (threadIdx.x == 0) part[blockIdx.x] = s_cnt;
}
__global__ __launch_bounds__(kOneThreads) void k_life_sort_one(int64_t n, int shift0, const int32_t* bad, uint64_t* ka,
                                                               uint32_t* va, uint64_t* kb, uint32_t* vb) {
  if (*bad) return;
  __shared__ OneLds s;
  sort_one<true>(s, ka, va, kb, vb, (int)n, shift0, kHashBits, false);
}
// whether records i and j (keys equal but for the lowest bit) are of one trace and address
__device__ __forceinline__ bool life_same(const xmem_raw_event* raw, const int64_t* off, int64_t T, uint64_t key, uint32_t i,
                                          uint32_t j) {
  if (!(key & kWide)) return true;
  if (raw[i].addr != raw[j].addr) return false;
  // of one trace: no trace starts in (min, max]
  const int64_t a = i < j ? i : j, b = i < j ? j : i;
  int64_t lo = 0, hi = T;  // the first trace that starts past a
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (off[mid] > a) hi = mid; else lo = mid + 1;
  }
  return lo >= T || off[lo] > b;
}
// Sorted by the key's hash, stably: the records of one key meet in stream order, among those of the
// few other keys with the same hash (bits below shift0 unsorted): a run.  An allocation is closed by
// the next record of its key when that is a free; a free is unmatched unless the record of its key
// before it is an allocation.  Few other keys may still be many records: where one address is taken
// and freed again all the time, its records lie between those of any other that shares its hash.  So
// a thread looks at its kNear next records only, its wavefront at the 64 after them, and then its
// workgroup goes on through the run, 2,048 records a step.  2^20 events, half of them at one address,
// 30 others sharing its hash: the call takes 260 us, by threads alone 57 ms; 110 us either way where
// none shares it.  (64 records a thread: 16 profiles of 20,011 events 103 -> 111 us a call; 512 or
// 1,024 threads 110 or 115 us.  Without the wavefronts' part a batch whose runs are a little longer
// than a thread's part waits for its workgroups: 40 profiles of 2,000 events 97 us a call, 88 with it.)
constexpr int kNear = 16, kFarItems = 8;
constexpr int64_t kNoPartner = -1, kFarPartner = -2;
__device__ __forceinline__ uint64_t run_of(uint64_t key, int shift0) {
  return ((key | 1) * 0x9E3779B97F4A7C15ull) >> (64 - kHashBits + shift0);
}
struct LifeRun {
  const xmem_raw_event* raw;
  const int64_t* off;
  int64_t T;
  const uint64_t* key;
  const uint32_t* val;
  int64_t n;
  int shift0;
};
// what place q says to the search of record k (key x): it holds the partner (1), ends the run (0), neither (-1)
__device__ __forceinline__ int life_look(const LifeRun& r, uint64_t x, uint32_t k, int64_t q, uint64_t y) {
  if ((y | 1) == (x | 1)) return life_same(r.raw, r.off, r.T, x, k, r.val[q]) ? 1 : -1;
  return run_of(y, r.shift0) != run_of(x, r.shift0) ? 0 : -1;
}
// the place of the record of x's trace and address next to place p (an allocation looks forward, a
// free back), kNoPartner, or kFarPartner: not among the kNear next ones
__device__ __forceinline__ int64_t life_near(const LifeRun& r, int64_t p, uint64_t x, uint32_t k) {
  const int64_t dir = (x & 1) ? -1 : 1;
  for (int i = 1; i <= kNear; ++i) {
    const int64_t q = p + dir * i;
    if (q < 0 || q >= r.n) return kNoPartner;
    const int look = life_look(r, x, k, q, r.key[q]);
    if (look >= 0) return look ? q : kNoPartner;
  }
  return kFarPartner;
}
__device__ __forceinline__ uint64_t lane_u64(uint64_t v, int lane) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), lane) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
// the same among the 64 after those, by one wavefront (p, x and k wave-uniform)
__device__ __forceinline__ int64_t life_wave(const LifeRun& r, int64_t p, uint64_t x, uint32_t k) {
  const int64_t dir = (x & 1) ? -1 : 1, from = p + dir * (kNear + 1), q = from + dir * (int64_t)(threadIdx.x & 63);
  const uint64_t y = q >= 0 && q < r.n ? r.key[q] : x;  // (x: past the records the search ends)
  for (uint64_t m = ballot((y | 1) == (x | 1) || run_of(y, r.shift0) != run_of(x, r.shift0)); m; m &= m - 1) {
    const int64_t at = from + dir * (int64_t)__builtin_ctzll(m);
    if (at < 0 || at >= r.n) return kNoPartner;
    const int look = life_look(r, x, k, at, r.key[at]);
    if (look >= 0) return look ? at : kNoPartner;
  }
  return kFarPartner;
}
// the same past the kNear + 64 next ones, by the whole workgroup (s_hit: one word; every thread calls it):
// the nearest place that holds x's key or ends the run, then whether that is of x's trace and address
__device__ int64_t life_far(const LifeRun& r, int64_t p, uint64_t x, uint32_t k, uint32_t* s_hit) {
  const int64_t dir = (x & 1) ? -1 : 1;
  const uint64_t run = run_of(x, r.shift0);
  for (int64_t from = p + dir * (kNear + 64 + 1);;) {
    uint64_t y[kFarItems];
#pragma unroll
    for (int i = 0; i < kFarItems; ++i) {
      const int64_t q = from + dir * (i * kThreads + (int)threadIdx.x);
      y[i] = q >= 0 && q < r.n ? r.key[q] : x;  // (x: past the records the search ends)
    }
    uint32_t hit = ~0u;  // the distance
#pragma unroll
    for (int i = kFarItems - 1; i >= 0; --i)
      hit = (y[i] | 1) == (x | 1) || run_of(y[i], r.shift0) != run ? (uint32_t)(i * kThreads) + threadIdx.x : hit;
    if (threadIdx.x == 0) *s_hit = ~0u;
    __syncthreads();
    if (hit != ~0u) atomicMin(s_hit, hit);
    __syncthreads();
    const uint32_t first = *s_hit;
    __syncthreads();
    if (first == ~0u) {
      from += dir * (kThreads * kFarItems);
    } else {
      const int64_t q = from + dir * (int64_t)first;
      const int look = q >= 0 && q < r.n ? life_look(r, x, k, q, r.key[q]) : 0;
      if (look >= 0) return look ? q : kNoPartner;
      from = q + dir;  // another trace's or address's, of the same 61 mixed bits
    }
  }
}
// record k (key x), its partner at place q (kNoPartner: none)
__device__ __forceinline__ void life_settle(const LifeRun& r, uint64_t x, uint32_t k, int64_t q, int64_t* tfree,
                                            int64_t* unmatched) {
  const bool other = q >= 0 && ((r.key[q] ^ x) & 1);  // of the other kind: the two are one block's
  if (!(x & 1)) {
    tfree[k] = other ? r.raw[r.val[q]].ts : kPersist;
  } else if (!other) {
    int64_t lo = 0, hi = r.T - 1;  // the last trace that starts at or before the record
    while (lo < hi) {
      const int64_t mid = (lo + hi + 1) >> 1;
      if (r.off[mid] <= (int64_t)k) lo = mid; else hi = mid - 1;
    }
    atomicAdd((unsigned long long*)&unmatched[lo], 1ull);
  }
}
__global__ __launch_bounds__(kThreads, 8) void k_life_pair(const xmem_raw_event* raw, const int64_t* off, int64_t T,
                                                        const uint64_t* key, const uint32_t* val, int64_t n, int shift0,
                                                        const int32_t* bad, int64_t* tfree, int64_t* unmatched) {
  if (*bad) return;
  __shared__ uint32_t s_far[kThreads], s_nfar, s_hit;  // the threads whose partners are far
  const LifeRun r{raw, off, T, key, val, n, shift0};
  const int64_t base = (int64_t)blockIdx.x * kThreads, p = base + threadIdx.x;
  if (threadIdx.x == 0) s_nfar = 0;
  __syncthreads();
  const uint64_t x = p < n ? key[p] : kNone;
  const bool search = (x & kNone) != kNone && (!(x & 1) || unmatched);
  const uint32_t k = search ? val[p] : 0;
  int64_t q = search ? life_near(r, p, x, k) : kNoPartner;
  for (uint64_t far = ballot(q == kFarPartner); far; far &= far - 1) {
    const int l = __builtin_ctzll(far);
    const int64_t found = life_wave(r, base + (int)(threadIdx.x & ~63u) + l, lane_u64(x, l),
                                    (uint32_t)__builtin_amdgcn_readlane((int)k, l));
    if ((int)(threadIdx.x & 63) == l) q = found;
  }
  if (q == kFarPartner) s_far[atomicAdd(&s_nfar, 1u)] = threadIdx.x;
  else if (search) life_settle(r, x, k, q, tfree, unmatched);
  __syncthreads();
  const uint32_t nfar = s_nfar;
  for (uint32_t i = 0; i < nfar; ++i) {
    const int64_t pf = base + s_far[i];
    const uint64_t xf = key[pf];
    const uint32_t kf = val[pf];
    const int64_t q = life_far(r, pf, xf, kf, &s_hit);
    if (threadIdx.x == 0) life_settle(r, xf, kf, q, tfree, unmatched);
  }
}
// the blocks in allocation order (part: allocations before each tile), and the traces' offsets
__global__ __launch_bounds__(kRecThreads) void k_life_emit(const xmem_raw_event* raw, const int32_t* cat, const int64_t* off,
                                                        int64_t T, int64_t n, const int32_t* bad, const uint32_t* part,
                                                        const int64_t* tfree, xmem_block* blocks, int64_t* boff) {
  if (*bad) return;
  __shared__ TileFlags f;
  const int64_t base = (int64_t)blockIdx.x * kTileN;
  int64_t bytes[kRecItems];
#pragma unroll
  for (int i = 0; i < kRecItems; ++i) {
    const int64_t k = base + (int64_t)i * kRecThreads + threadIdx.x;
    bytes[i] = k < n ? raw[k].bytes : 0;
    flags_put(f, i, bytes[i] > 0);
  }
  flags_scan(f);
  const uint32_t at = tile_before(part, gridDim.x);
#pragma unroll 4
  for (int i = 0; i < kRecItems; ++i) {
    const int r = i * kRecThreads + threadIdx.x;
    const int64_t k = base + r;
    if (bytes[i] > 0) {
      xmem_block b;
      b.size = bytes[i];
      b.t_alloc = raw[k].ts;
      b.t_free = tfree[k];
      b.category = cat ? cat[k] : XMEM_CAT_OTHER;
      b.pad = 0;
      blocks[at + flags_before(f, r)] = b;
    }
  }
  tile_offsets(off, T, n, base, f, at, 0, boff);
}

// ---------------------------------------------------------------- attribution (Section 3.2)
// the enclosing window of window i of a trace whose windows start at w (-1: a root)
__device__ __forceinline__ int64_t win_parent(const xmem_window* w, int64_t i) {
  const int64_t p = w[i].parent;
  return (p >= 0 && p < i) ? p : -1;
}
// per window: the end of its nearest enclosing component (kPersist: none), and whether it lies in
// an optimizer.step() phase (itself or an enclosing window is a component of category optimizer);
// and two empty slots of the parameter-size sets per block
__global__ __launch_bounds__(kRecThreads) void k_att_windows(const xmem_window* win, const int64_t* woff, int64_t T, int64_t nw,
                                                          int64_t nb, const int32_t* bad, int64_t* comp_end,
                                                          uint32_t* in_step, uint64_t* tab) {
  if (*bad) return;
  const int64_t base = (int64_t)blockIdx.x * kTileN;
#pragma unroll
  for (int i = 0; i < kRecItems; ++i) {
    const int64_t k = base + (int64_t)i * kRecThreads + threadIdx.x;
    if (k < nb) tab[k] = 0;
  }
  if (base >= nw) return;
  TraceStep tr(woff, T, tile_trace(woff, T, base));
#pragma unroll 2
  for (int i = 0; i < kRecItems; ++i) {
    const int64_t g = base + (int64_t)i * kRecThreads + threadIdx.x;
    if (g >= nw) break;
    tr.to(woff, T, g);
    const xmem_window* w = win + woff[tr.t];
    const int64_t me = g - woff[tr.t];
    // one climb for both: up to the nearest component for its end, on to the root for the phase
    int64_t end = kPersist;
    bool found = false;
    uint32_t step = w[me].kind == XMEM_WIN_COMPONENT && w[me].category == XMEM_CAT_OPTIMIZER;
    for (int64_t a = win_parent(w, me); a >= 0 && !(found && step); a = win_parent(w, a)) {
      const bool comp = w[a].kind == XMEM_WIN_COMPONENT;
      if (comp && !found) {
        end = w[a].end;
        found = true;
      }
      step |= comp && w[a].category == XMEM_CAT_OPTIMIZER;
    }
    comp_end[g] = end;
    in_step[g] = step;
  }
}
// Section 3.3 item 5: the parameter sizes of each trace as an open-addressing hash set of block
// indices + 1 (0: empty), at two slots per block of the trace, so at most half full: every probe
// sequence reaches an empty slot.
struct ParamSet { int64_t base, cap; };
__device__ __forceinline__ ParamSet param_set(const int64_t* boff, int64_t t) {
  return ParamSet{2 * boff[t], 2 * (boff[t + 1] - boff[t])};
}
__device__ __forceinline__ uint64_t size_hash(int64_t size) {
  return ((uint64_t)size * 0x9E3779B97F4A7C15ull) >> 32;
}
constexpr uint32_t kKept = 1u << 31, kStepCandidate = 1u << 30;  // role word: linked; a product in an optimizer.step() phase
// The window each block links to (index in its trace, -1 if none) and its role by the operator rule
// (role: the category below kStepCandidate's bit); a parameter's size goes into its trace's set.
// Per tile its kept blocks (part).
__global__ __launch_bounds__(kRecThreads) void k_att_blocks(const xmem_block* blocks, const int64_t* boff, int64_t T, int64_t nb,
                                                         const xmem_window* win, const int64_t* woff,
                                                         const int64_t* comp_end, const uint32_t* in_step,
                                                         const int32_t* bad, int32_t* bwin, uint32_t* role, int32_t* cats,
                                                         uint32_t* tab, uint32_t* part) {
  if (*bad) return;
  __shared__ uint32_t s_cnt;
  if (threadIdx.x == 0) s_cnt = 0;
  const int64_t base = (int64_t)blockIdx.x * kTileN;
  TraceStep tr(boff, T, tile_trace(boff, T, base));  // (its barrier orders s_cnt too)
  uint32_t kept = 0;
  for (int i = 0; i < kRecItems; ++i) {
    const int64_t b = base + (int64_t)i * kRecThreads + threadIdx.x;
    if (b >= nb) break;
    tr.to(boff, T, b);
    const int64_t wbase = woff[tr.t], n = woff[tr.t + 1] - wbase;
    const xmem_window* w = win + wbase;
    const int64_t ta = blocks[b].t_alloc, tf = blocks[b].t_free, size = blocks[b].size;
    int64_t lo = 0, hi = n;  // last window that starts no later than the allocation
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (w[mid].start <= ta) lo = mid + 1; else hi = mid;
    }
    int64_t j = lo - 1;
    while (j >= 0 && w[j].end < ta) j = win_parent(w, j);  // up to the innermost window containing it
    const bool step = j >= 0 && in_step[wbase + j];
    int32_t link = -1, cat = XMEM_CAT_OTHER;
    bool product = false;
    for (; j >= 0; j = win_parent(w, j)) {
      const xmem_window x = w[j];
      if (x.kind != XMEM_WIN_OPERATOR) continue;
      if (x.start < ta && tf < x.end) { link = (int32_t)j; break; }  // (i) a temporary: strictly inside the window
      if (tf > comp_end[wbase + j]) {                                  // (ii) a product
        link = (int32_t)j;
        cat = x.category;
        product = true;
        break;
      }
    }
    if (bwin) bwin[b] = link;
    role[b] = (link >= 0 ? kKept : 0u) | (product && step ? kStepCandidate : 0u);
    cats[b] = cat;
    kept += link >= 0 ? 1u : 0u;
    if (product && cat == XMEM_CAT_PARAMETER) {
      const ParamSet ps = param_set(boff, tr.t);
      for (int64_t s = (int64_t)(size_hash(size) % (uint64_t)ps.cap);; s = s + 1 == ps.cap ? 0 : s + 1) {
        const uint32_t old = atomicCAS(&tab[ps.base + s], 0u, (uint32_t)(b + 1));
        if (old == 0 || blocks[old - 1].size == size) break;  // inserted, or the size is there already
      }
    }
  }
  atomicAdd(&s_cnt, kept);
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = s_cnt;
}
// The kept blocks in order with their roles (a product in an optimizer.step() phase whose size is a
// parameter's is an optimizer state), and the traces' offsets.
__global__ __launch_bounds__(kRecThreads) void k_att_emit(const xmem_block* blocks, const int64_t* boff, int64_t T, int64_t nb,
                                                       const int32_t* bad, const uint32_t* role, const int32_t* cats,
                                                       const uint32_t* tab, const uint32_t* part, xmem_block* kept,
                                                       int64_t* koff) {
  if (*bad) return;
  __shared__ TileFlags f;
  const int64_t base = (int64_t)blockIdx.x * kTileN;
  uint32_t rl[kRecItems];
#pragma unroll
  for (int i = 0; i < kRecItems; ++i) {
    const int64_t b = base + (int64_t)i * kRecThreads + threadIdx.x;
    rl[i] = b < nb ? role[b] : 0u;
    flags_put(f, i, rl[i] & kKept);
  }
  flags_scan(f);
  const uint32_t at = tile_before(part, gridDim.x);
  TraceStep tr(boff, T, tile_trace(boff, T, base));
#pragma unroll 4
  for (int i = 0; i < kRecItems; ++i) {
    const int r = i * kRecThreads + threadIdx.x;
    const int64_t b = base + r;
    if (rl[i] & kKept) {
      xmem_block x = blocks[b];
      x.category = cats[b];
      if (rl[i] & kStepCandidate) {
        tr.to(boff, T, b);
        const ParamSet ps = param_set(boff, tr.t);
        for (int64_t s = (int64_t)(size_hash(x.size) % (uint64_t)ps.cap);; s = s + 1 == ps.cap ? 0 : s + 1) {
          const uint32_t v = tab[ps.base + s];
          if (v == 0) break;
          if (blocks[v - 1].size == x.size) { x.category = XMEM_CAT_OPTIMIZER; break; }
        }
      }
      kept[at + flags_before(f, r)] = x;
    }
  }
  tile_offsets(boff, T, nb, base, f, at, 0, koff);
}

// ---------------------------------------------------------------- orchestration (Section 3.3)
// first value > t in the ascending v[lo, hi), or kPersist
__device__ __forceinline__ int64_t next_marker(const int64_t* v, int64_t lo, int64_t hi, int64_t t) {
  int64_t a = lo, b = hi;
  while (a < b) {
    const int64_t mid = (a + b) >> 1;
    if (v[mid] > t) b = mid; else a = mid + 1;
  }
  return a < hi ? v[a] : kPersist;
}
// Retimed free of each block; the range of the times (sign bit flipped: signed order as unsigned) of
// the allocation and free records that take part (a persistent block's free does not: it sorts
// last by its trace); per tile the blocks that are freed (part).
__global__ __launch_bounds__(kRecThreads) void k_orch_retime(const xmem_block* blocks, const int64_t* boff, int64_t T, int64_t nb,
                                                          const int64_t* steps, const int64_t* soff, const int64_t* zg,
                                                          const int64_t* zoff, const int32_t* bad, int64_t* tfr, uint64_t* kr,
                                                          uint32_t* part) {
  if (*bad) return;
  __shared__ uint32_t s_cnt;
  if (threadIdx.x == 0) s_cnt = 0;
  const int64_t base = (int64_t)blockIdx.x * kTileN;
  TraceStep tr(boff, T, tile_trace(boff, T, base));  // (its barrier orders s_cnt too)
  RangePart p;
  uint32_t freed = 0;
#pragma unroll 4
  for (int i = 0; i < kRecItems; ++i) {
    const int64_t b = base + (int64_t)i * kRecThreads + threadIdx.x;
    if (b >= nb) break;
    tr.to(boff, T, b);
    const xmem_block x = blocks[b];
    int64_t f = x.t_free;
    switch (x.category) {
      case XMEM_CAT_PARAMETER:
      case XMEM_CAT_OPTIMIZER:
        f = kPersist;
        break;
      case XMEM_CAT_BATCH: {
        const int64_t e = next_marker(steps, soff[tr.t], soff[tr.t + 1], x.t_alloc);
        f = f < e ? f : e;
        break;
      }
      case XMEM_CAT_GRADIENT:
        f = next_marker(zg, zoff[tr.t], zoff[tr.t + 1], x.t_alloc);
        break;
      default:
        break;
    }
    if (f != kPersist && f < x.t_alloc) f = x.t_alloc;
    tfr[b] = f;
    p.add(true, (uint64_t)x.t_alloc ^ (1ull << 63));
    p.add(f != kPersist, (uint64_t)f ^ (1ull << 63));
    freed += f != kPersist ? 1u : 0u;
  }
  atomicAdd(&s_cnt, freed);
  range_commit(kr, p);  // (its barrier orders s_cnt too)
  if (threadIdx.x == 0) part[blockIdx.x] = s_cnt;
}
// The sort records of each block (2b: its allocation, 2b + 1: its free) and the traces' word offsets.
// The layout is chosen on the device from the time range (kr[5]: bit 0 set for the joint key, bit 1
// when the sorted records end in the second buffer, bits 8.. the time bits tb).  Joint key, when
// trace, time and rank fit in 64 bits together: (trace << (tb + 2)) | (time << 2) | rank, the free of a
// persistent block last (T << (tb + 2)); one sort of tbits + tb + 2 bits, from the second buffer.
// Rank at equal times: a free of an earlier block 0, an allocation 1, a free of a block allocated at
// that time 2.  Otherwise three key groups as separate sorts: the rank (here, in the first buffer),
// the time in an even number of passes, then the trace.  The host launches the same kernels either
// way; the gates skip the passes a layout does not take: gate[0] the time sort (or the joint sort),
// gate[1] the rank sort, gate[2] the trace sort.
__global__ __launch_bounds__(kRecThreads) void k_orch_keys(const xmem_block* blocks, const int64_t* boff, int64_t T, int64_t nb,
                                                        const int64_t* tfr, int tbits, bool trace_odd, const int32_t* bad,
                                                        uint64_t* kr, int32_t* gate, uint64_t* ka, uint32_t* va,
                                                        uint64_t* kb, uint32_t* vb, uint32_t* tid, const uint32_t* part,
                                                        uint32_t* total, int64_t* eoff) {
  if (*bad) return;
  __shared__ TileFlags f;
  const int64_t base = (int64_t)blockIdx.x * kTileN;
  const int tb = range_bits(kr);
  const bool joint = tbits + tb + 2 <= 64;
  const uint64_t lowest = kr[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const int jp = (tbits + tb + 2 + kDigit - 1) / kDigit;
    gate[0] = joint ? kDigit * jp : range_gate(kr);
    gate[1] = joint ? 0 : 64;
    gate[2] = joint ? 0 : 64;
    // the time sort starts in the second buffer; the separate layout then takes the trace passes
    const bool in_b = joint ? !(jp & 1) : !trace_odd;
    kr[5] = (joint ? kJoint : 0) | (in_b ? kJointBuf : 0) | ((uint64_t)tb << 8);
  }
  TraceStep tr(boff, T, tile_trace(boff, T, base));
#pragma unroll 4
  for (int i = 0; i < kRecItems; ++i) {
    const int64_t b = base + (int64_t)i * kRecThreads + threadIdx.x;
    const bool ok = b < nb;
    const int64_t fr = ok ? tfr[b] : kPersist;
    flags_put(f, i, fr != kPersist);
    if (ok) {
      tr.to(boff, T, b);
      const int64_t ta = blocks[b].t_alloc;
      if (joint) {
        const uint64_t t = (uint64_t)tr.t << (tb + 2);
        kb[2 * b] = t | ((((uint64_t)ta ^ (1ull << 63)) - lowest) << 2) | 1u;
        kb[2 * b + 1] = fr == kPersist ? (uint64_t)T << (tb + 2)
                                       : t | ((((uint64_t)fr ^ (1ull << 63)) - lowest) << 2) | (fr == ta ? 2u : 0u);
        vb[2 * b] = (uint32_t)(2 * b);
        vb[2 * b + 1] = (uint32_t)(2 * b + 1);
      } else {
        ka[2 * b] = 1;
        ka[2 * b + 1] = fr == ta ? 2 : 0;
        va[2 * b] = (uint32_t)(2 * b);
        va[2 * b + 1] = (uint32_t)(2 * b + 1);
        tid[b] = (uint32_t)tr.t;
      }
    }
  }
  flags_scan(f);
  const uint32_t frees = tile_before(part, gridDim.x);
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = (uint32_t)nb + frees + f.before[kSteps];
  tile_offsets(boff, T, nb, base, f, (uint32_t)base + frees, 1, eoff);
}
// second key group of the separate layout: the time, rebased to the batch's earliest
__global__ void k_orch_time_keys(const xmem_block* blocks, const int64_t* tfr, int64_t n, const int32_t* bad,
                                 const uint64_t* kr, const uint32_t* val, uint64_t* key) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n || *bad || (kr[5] & kJoint)) return;
  const uint32_t r = val[p];
  const int64_t tm = (r & 1) ? tfr[r >> 1] : blocks[r >> 1].t_alloc;
  key[p] = ((r & 1) && tm == kPersist) ? 0 : ((uint64_t)tm ^ (1ull << 63)) - kr[0];
}
// third key group: the trace, T for the free of a persistent block (sorts last)
__global__ void k_orch_trace_keys(const uint32_t* btid, const int64_t* tfr, int64_t n, int64_t T, const int32_t* bad,
                                  const uint64_t* kr, const uint32_t* val, uint64_t* key) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n || *bad || (kr[5] & kJoint)) return;
  const uint32_t r = val[p];
  key[p] = ((r & 1) && tfr[r >> 1] == kPersist) ? (uint64_t)T : (uint64_t)btid[r >> 1];
}
// Few records: whichever sorts the layout takes, by one workgroup; the result lies where kr[5] says.
__global__ __launch_bounds__(kOneThreads) void k_orch_sort_one(const xmem_block* blocks, const uint32_t* btid,
                                                               const int64_t* tfr, int64_t n, int64_t T, int tp,
                                                               const int32_t* bad, const uint64_t* kr, const int32_t* gate,
                                                               uint64_t* ka, uint32_t* va, uint64_t* kb, uint32_t* vb) {
  if (*bad) return;
  __shared__ OneLds s;
  if (kr[5] & kJoint) {
    sort_one<false>(s, ka, va, kb, vb, (int)n, 0, gate[0], true);
    return;
  }
  sort_one<false>(s, ka, va, kb, vb, (int)n, 0, kDigit, false);  // the rank, to (kb, vb)
  __syncthreads();
  for (int64_t p = threadIdx.x; p < n; p += kOneThreads) {
    const uint32_t r = vb[p];
    const int64_t tm = (r & 1) ? tfr[r >> 1] : blocks[r >> 1].t_alloc;
    kb[p] = ((r & 1) && tm == kPersist) ? 0 : ((uint64_t)tm ^ (1ull << 63)) - kr[0];
  }
  __syncthreads();
  sort_one<false>(s, ka, va, kb, vb, (int)n, 0, gate[0], true);  // the time, an even number of passes
  __syncthreads();
  for (int64_t p = threadIdx.x; p < n; p += kOneThreads) {
    const uint32_t r = vb[p];
    kb[p] = ((r & 1) && tfr[r >> 1] == kPersist) ? (uint64_t)T : (uint64_t)btid[r >> 1];
  }
  __syncthreads();
  sort_one<false>(s, ka, va, kb, vb, (int)n, 0, tp * kDigit, true);
}
// position of each allocation's word within its trace
__global__ __launch_bounds__(kRecThreads) void k_orch_apos(const int64_t* eoff, int64_t T, const uint32_t* total,
                                                        const int32_t* bad, const uint64_t* kr, const uint32_t* va,
                                                        const uint32_t* vb, uint32_t* apos) {
  const int64_t base = (int64_t)blockIdx.x * kTileN;
  if (*bad || base >= (int64_t)*total) return;
  const int64_t m = (int64_t)*total;
  const uint32_t* val = (kr[5] & kJointBuf) ? vb : va;
  TraceStep tr(eoff, T, tile_trace(eoff, T, base));
#pragma unroll 4
  for (int i = 0; i < kRecItems; ++i) {
    const int64_t p = base + (int64_t)i * kRecThreads + threadIdx.x;
    if (p >= m) break;
    const uint32_t r = val[p];
    if (r & 1) continue;
    tr.to(eoff, T, p);
    apos[r >> 1] = (uint32_t)(p - eoff[tr.t]);
  }
}
__global__ void k_orch_words(const xmem_block* blocks, const uint32_t* total, const int32_t* bad, const uint64_t* kr,
                             const uint32_t* va, const uint32_t* vb, const uint32_t* apos, uint64_t* events) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (*bad || p >= (int64_t)*total) return;
  const uint32_t r = ((kr[5] & kJointBuf) ? vb : va)[p];
  events[p] = (r & 1) ? (kFree | (uint64_t)apos[r >> 1]) : (uint64_t)blocks[r >> 1].size;
}

bool aligned256(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 255) == 0; }

}  // namespace

extern "C" {

size_t xmem_prep_workspace_bytes(int64_t n_traces, int64_t n_records) {
  if (n_traces < 0 || n_records < 0 || n_records > XMEM_PREP_MAX_RECORDS || n_traces > INT32_MAX - 1) return 0;
  return carve(nullptr, n_traces, n_records, nullptr);
}

int xmem_lifecycles(const xmem_raw_event* d_raw, const int32_t* d_category, const int64_t* d_raw_offsets,
                    int64_t n_traces, int64_t total_raw, xmem_block* d_blocks, int64_t* d_block_offsets,
                    int64_t* d_unmatched_frees, int32_t* d_status, void* d_workspace, size_t workspace_bytes,
                    void* hip_stream) {
  if (n_traces < 0 || total_raw < 0 || total_raw > XMEM_PREP_MAX_RECORDS || n_traces > INT32_MAX - 1) return XMEM_EINVAL;
  if (!d_raw_offsets || !d_block_offsets || !d_status || (total_raw > 0 && (!d_raw || !d_blocks))) return XMEM_EINVAL;
  const size_t need = carve(nullptr, n_traces, total_raw, nullptr);
  if (!d_workspace || workspace_bytes < need || !aligned256(d_workspace)) return XMEM_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  PrepWs w;
  carve(d_workspace, n_traces, total_raw, &w);
  const int64_t T = n_traces, n = total_raw;
  const bool empty = n == 0 || T == 0;
  begin({d_raw_offsets, n}, {nullptr, 0}, {nullptr, 0}, T, empty, d_unmatched_frees, w, d_status, d_block_offsets, st);
  if (!empty) {
    const int64_t nt = tiles_of(n);
    // digits of the hash: enough that a key shares all of them with few others.  320,160 events in
    // two digits rather than three: 1,027 -> 1,014 us for a whole estimate; 8.4M in two rather than
    // three: 1,610 -> 1,665 us (the pairing then looks past more of the others)
    const int shift0 = kHashBits - kDigit * (n <= (1 << 20) ? 2 : n <= (1 << 25) ? 3 : 4);
    k_life_keys<<<(unsigned)nt, kRecThreads, 0, st>>>(d_raw, d_raw_offsets, n, T, w.bad, w.s.ka, w.s.va, shift0, w.s.hist, nt,
                                                      w.part);
    scan_parts(w.part, nt, st);
    bool in_b = ((kHashBits - shift0) / kDigit) & 1;
    if (n <= kOneRecords)
      k_life_sort_one<<<1, kOneThreads, 0, st>>>(n, shift0, w.bad, w.s.ka, w.s.va, w.s.kb, w.s.vb);
    else
      in_b = sort_bits<true>(w.s, n, shift0, kHashBits, false, st, nullptr, true);
    k_life_pair<<<grid_of(n, kThreads), kThreads, 0, st>>>(d_raw, d_raw_offsets, T, in_b ? w.s.kb : w.s.ka,
                                                           in_b ? w.s.vb : w.s.va, n, shift0, w.bad, w.t64, d_unmatched_frees);
    k_life_emit<<<(unsigned)nt, kRecThreads, 0, st>>>(d_raw, d_category, d_raw_offsets, T, n, w.bad, w.part, w.t64, d_blocks,
                                                   d_block_offsets);
  }
  finish(T, empty, w, d_status, d_block_offsets, st);
  return hipGetLastError() == hipSuccess ? XMEM_OK : XMEM_EHIP;
}

int xmem_attribute(const xmem_block* d_blocks, const int64_t* d_block_offsets, int64_t n_traces,
                   int64_t total_blocks, const xmem_window* d_windows, const int64_t* d_window_offsets,
                   int64_t total_windows, xmem_block* d_kept, int64_t* d_kept_offsets, int32_t* d_block_window,
                   int32_t* d_status, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  if (n_traces < 0 || total_blocks < 0 || total_windows < 0 || n_traces > INT32_MAX - 1) return XMEM_EINVAL;
  const int64_t n = total_blocks > total_windows ? total_blocks : total_windows;
  if (n > XMEM_PREP_MAX_RECORDS) return XMEM_EINVAL;
  if (!d_block_offsets || !d_window_offsets || !d_kept_offsets || !d_status) return XMEM_EINVAL;
  if ((total_blocks > 0 && (!d_blocks || !d_kept)) || (total_windows > 0 && !d_windows)) return XMEM_EINVAL;
  const int64_t T = n_traces, nb = total_blocks, nw = total_windows;
  const size_t need = carve(nullptr, T, n, nullptr);
  if (!d_workspace || workspace_bytes < need || !aligned256(d_workspace)) return XMEM_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  PrepWs w;
  carve(d_workspace, T, n, &w);
  int64_t* comp_end = reinterpret_cast<int64_t*>(w.s.ka);  // the sort buffers are free here: per window
  uint32_t* in_step = w.apos;                                  // per window
  int32_t* cats = reinterpret_cast<int32_t*>(w.s.va);          // per block
  uint64_t* tab = reinterpret_cast<uint64_t*>(w.t64);          // per block: two slots of the parameter-size sets
  const bool empty = nb == 0 || T == 0;
  begin({d_block_offsets, nb}, {d_window_offsets, nw}, {nullptr, 0}, T, empty, nullptr, w, d_status, d_kept_offsets, st);
  if (!empty) {
    const int64_t nt = tiles_of(nb);
    k_att_windows<<<(unsigned)tiles_of(n), kRecThreads, 0, st>>>(d_windows, d_window_offsets, T, nw, nb, w.bad, comp_end, in_step,
                                                              tab);
    k_att_blocks<<<(unsigned)nt, kRecThreads, 0, st>>>(d_blocks, d_block_offsets, T, nb, d_windows, d_window_offsets, comp_end,
                                                    in_step, w.bad, d_block_window, w.tid, cats,
                                                    reinterpret_cast<uint32_t*>(tab), w.part);
    scan_parts(w.part, nt, st);
    k_att_emit<<<(unsigned)nt, kRecThreads, 0, st>>>(d_blocks, d_block_offsets, T, nb, w.bad, w.tid, cats,
                                                  reinterpret_cast<uint32_t*>(tab), w.part, d_kept, d_kept_offsets);
  }
  finish(T, empty, w, d_status, d_kept_offsets, st);
  return hipGetLastError() == hipSuccess ? XMEM_OK : XMEM_EHIP;
}

int xmem_orchestrate(const xmem_block* d_blocks, const int64_t* d_block_offsets, int64_t n_traces,
                     int64_t total_blocks, const int64_t* d_step_ts, const int64_t* d_step_offsets,
                     const int64_t* d_zero_grad_ts, const int64_t* d_zero_grad_offsets, uint64_t* d_events,
                     int64_t* d_event_offsets, int32_t* d_status, void* d_workspace, size_t workspace_bytes,
                     void* hip_stream) {
  if (n_traces < 0 || total_blocks < 0 || 2 * total_blocks > XMEM_PREP_MAX_RECORDS || n_traces > INT32_MAX - 1)
    return XMEM_EINVAL;
  if (!d_block_offsets || !d_step_offsets || !d_zero_grad_offsets || !d_event_offsets || !d_status) return XMEM_EINVAL;
  if (total_blocks > 0 && (!d_blocks || !d_events)) return XMEM_EINVAL;
  const int64_t T = n_traces, nb = total_blocks, n = 2 * total_blocks;
  const size_t need = carve(nullptr, T, n, nullptr);
  if (!d_workspace || workspace_bytes < need || !aligned256(d_workspace)) return XMEM_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  PrepWs w;
  carve(d_workspace, T, n, &w);
  const bool empty = nb == 0 || T == 0;
  begin({d_block_offsets, nb}, {d_step_offsets, -1}, {d_zero_grad_offsets, -1}, T, empty, nullptr, w, d_status, d_event_offsets,
        st);
  if (!empty) {
    const int64_t nt = tiles_of(nb);
    // gate[0]: the time (or joint) sort, gate[1]: the rank sort, gate[2]: the trace sort
    int32_t* gate = reinterpret_cast<int32_t*>(w.kr + 3);
    int tbits = 0;
    while (tbits < 63 && (T >> tbits) != 0) ++tbits;  // bits of the trace field (0..T)
    const int tp = passes_for(T);
    k_orch_retime<<<(unsigned)nt, kRecThreads, 0, st>>>(d_blocks, d_block_offsets, T, nb, d_step_ts, d_step_offsets,
                                                     d_zero_grad_ts, d_zero_grad_offsets, w.bad, w.t64, w.kr, w.part);
    scan_parts(w.part, nt, st);
    k_orch_keys<<<(unsigned)nt, kRecThreads, 0, st>>>(d_blocks, d_block_offsets, T, nb, w.t64, tbits, tp & 1, w.bad, w.kr, gate,
                                                   w.s.ka, w.s.va, w.s.kb, w.s.vb, w.tid, w.part, w.total, d_event_offsets);
    if (n <= kOneRecords) {
      k_orch_sort_one<<<1, kOneThreads, 0, st>>>(d_blocks, w.tid, w.t64, n, T, tp, w.bad, w.kr, gate, w.s.ka, w.s.va, w.s.kb,
                                                 w.s.vb);
    } else {
      sort_bits<false>(w.s, n, 0, kDigit, false, st, gate + 1);  // rank at equal times (separate layout)
      k_orch_time_keys<<<grid_of(n, 256), 256, 0, st>>>(d_blocks, w.t64, n, w.bad, w.kr, w.s.vb, w.s.kb);
      sort_bits<false>(w.s, n, 0, kAllBits, true, st, gate);  // time (its span only), or the joint key
      k_orch_trace_keys<<<grid_of(n, 256), 256, 0, st>>>(w.tid, w.t64, n, T, w.bad, w.kr, w.s.vb, w.s.kb);
      sort_bits<false>(w.s, n, 0, tp * kDigit, true, st, gate + 2);  // trace; persistent blocks' frees last
    }
    k_orch_apos<<<(unsigned)tiles_of(n), kRecThreads, 0, st>>>(d_event_offsets, T, w.total, w.bad, w.kr, w.s.va, w.s.vb, w.apos);
    k_orch_words<<<grid_of(n, 256), 256, 0, st>>>(d_blocks, w.total, w.bad, w.kr, w.s.va, w.s.vb, w.apos, d_events);
  }
  finish(T, empty, w, d_status, d_event_offsets, st);
  return hipGetLastError() == hipSuccess ? XMEM_OK : XMEM_EHIP;
}

}  // extern "C"
