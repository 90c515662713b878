// LDS sorts of final segments (one workgroup per segment) and the
// global-memory fallback for segments longer than the LDS capacity.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "device.hpp"
#include "engine.hpp"
#include "internal.hpp"

namespace rs {

static inline uint32_t grid_for(uint64_t work, uint32_t per_cu) {
  const uint64_t g = std::min<uint64_t>(work, (uint64_t)num_cu_cached() * per_cu);
  return (uint32_t)std::max<uint64_t>(g, 1);
}

// ---------------------------------------------------------------------------
// The merge sort of (key, position) pairs in LDS: exact for every input,
// whatever its keys.  Thread t holds elements i * THREADS + t of len <=
// THREADS * ITEMS.  Rank r ends at place lpad(r) of sa, its payload in sa.p.
// Called by every thread of the block; ends with a barrier.
template <typename K, bool PAY, int THREADS, int ITEMS>
__device__ __forceinline__ void merge_pairs(K (&k)[ITEMS], uint32_t (&v)[ITEMS], uint32_t (&p)[ITEMS], uint32_t len,
                                            const LdsArr<K>& sa) {
  // (the sort takes its elements in any order)
#pragma unroll
  for (int i = 0; i < ITEMS; i++) {
    if (i * THREADS + threadIdx.x >= len) {
      k[i] = KMax<K>::v;
      v[i] = kPadIdx;
    }
  }
  lds_merge_sort<K, THREADS, ITEMS, PAY>(k, v, p, sa);
#pragma unroll
  for (int i = 0; i < ITEMS; i++) {
    const int q = lpad(threadIdx.x * ITEMS + i);
    sa.put(q, k[i], v[i]);
    if constexpr (PAY) sa.p[q] = p[i];
  }
  __syncthreads();
}

// The stretch [c0, c0 + cnt) of a segment so.  A segment of at most THREADS runs
// is read through a RunMap, built in the memory at map (looking 12288 elements
// up one by one, 10 dependent loads each, takes as long as sorting them).
template <typename K, bool F32, bool PAY, int THREADS, int ITEMS>
__device__ __forceinline__ void sort_stretch(const SegReader<K, F32, PAY>& rd, uint32_t c0, uint32_t cnt,
                                             const LdsArr<K>& sa, void* map) {
  K k[ITEMS];
  uint32_t v[ITEMS], p[ITEMS];
  const FinalSeg& f = rd.f;
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));  // (addresses are not kept from one segment to the next)
  if (f.src && f.nt <= THREADS) {  // uniform
    RunMap<THREADS, THREADS * ITEMS>& m = *reinterpret_cast<RunMap<THREADS, THREADS * ITEMS>*>(map);
    const int s = (int)f.src - 1;
    const uint32_t *o = rd.w.offs[s] + f.col, r = (uint32_t)t < f.nt ? rd.w.runs[s][f.col + t] : 0u;
    const uint32_t ofs = (uint32_t)t < f.nt ? o[t] - o[0] : 0u;
    uint64_t bal;
    m.clear(t);
    __syncthreads();
    m.mark(t, t, f.nt, ofs, r & 0xFFFFu, c0, cnt, bal);
    __syncthreads();
    m.number(t, t, ofs, r >> 16, c0, rd.w.tile_log2, bal);
    __syncthreads();
    const BufView<K, PAY> bv{rd.w.buf_rec[s] + f.pstart * BufView<K, PAY>::W};
    m.each(t, cnt, [&](int i, uint32_t d) { bv.get(d, k[i], v[i], p[i]); });
  } else {
    uint32_t j[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; i++) j[i] = c0 + min((uint32_t)(i * THREADS + t), cnt - 1);
    rd.get_all(j, k, v, p);
  }
  merge_pairs<K, PAY, THREADS, ITEMS>(k, v, p, cnt, sa);
}

// The same in the smallest of four shapes that holds the stretch.
template <typename K, bool F32, bool PAY, int THREADS, int ITEMS>
__device__ __forceinline__ void sort_stretch_fit(const SegReader<K, F32, PAY>& rd, uint32_t c0, uint32_t cnt,
                                                 const LdsArr<K>& sa, void* map) {
  if (cnt <= THREADS)
    sort_stretch<K, F32, PAY, THREADS, 1>(rd, c0, cnt, sa, map);
  else if (cnt <= THREADS * ITEMS / 4)
    sort_stretch<K, F32, PAY, THREADS, ITEMS / 4>(rd, c0, cnt, sa, map);
  else if (cnt <= THREADS * ITEMS / 2)
    sort_stretch<K, F32, PAY, THREADS, ITEMS / 2>(rd, c0, cnt, sa, map);
  else
    sort_stretch<K, F32, PAY, THREADS, ITEMS>(rd, c0, cnt, sa, map);
}

// len sorted elements to the output (start of the segment).
template <typename K, bool F32, bool PAY, int THREADS>
__device__ __forceinline__ void put_pairs(const LdsArr<K>& sa, uint32_t len, K* kout, uint32_t* pout, uint32_t* yout) {
  for (uint32_t j = threadIdx.x; j < len; j += THREADS) {
    const int q = lpad(j);
    kout[j] = to_output<K, F32>(sa.key(q));
    if (pout) pout[j] = sa.v[q];
    if constexpr (PAY) yout[j] = sa.p[q];
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Final segments ranked in bins: one workgroup per segment, its elements held
// in registers from the load to the output, LDS used for 32-bit words that
// rank them and then to bring them into rank order.
//
// With d = key - lower bound of the keys (rb bits) and x = position - smallest
// position (ib bits), the element's word is the top 32 bits of the rb + ib bit
// number (d, x), which orders like (key, position).  Its top LB bits are the
// bin, of which there is one per element of a full segment.  A rank is the
// start of the bin plus the number of smaller words in it:
//   count    one LDS atomic per element gives its place in its bin,
//   scan     the bin starts, and the sum of squared bin sizes (the compares
//            ranking will take),
//   place    the words, bin by bin,
//   rank     every thread compares its own elements with their bins' words
//            (and may read past a bin's end: later bins hold larger words).
// Equal words of different elements (keys that differ in few low bits, or
// equal keys near to each other) get equal ranks, which leaves the sum of all
// ranks below len (len - 1) / 2: such a segment (uniform test) goes on with
// the next 32 bits of (d, x) among its equals (rank_ties).
//
// A key that a part of a segment shares makes a long bin and a large group of
// equal words.  Its elements lie in every wave, which then all loop as long as
// the bin is; so from kRankOwn compares per element on, and among more than
// kTiesOwn pairs of equals, a thread ranks the words at its places of the
// sorted bins and not its own (2000 segments of 8000 u64 keys, 3 % of them 0:
// 2010 -> 386 us; 4096 of 4096, 10 % of them 0: 2550 -> 386).  Where ranks are
// few compares each, the own words are ranked: by place takes more barriers and
// passes (2000 segments of 8000 gaussian u64 keys, 192 us, 206 with all equal
// words by place).
//
// A segment whose ranking would take more than kRankBudget compares per element
// or kRankTotal in all, half of it if the words drop key bits (most keys
// clustered far apart from others), is marked kPairsFlag and left to the merge
// sort of k_local_rare.  Half of kRankTotal for all would hand over the segments
// of few values that many elements share (3145728 u64 keys below 16: 112 us as
// it is, 174 so), and all of it for all would rank rows with a shared key
// (2000 of 8000 u64 keys, 10 % of them 0: 657 us as it is, 795 so).
// Where LDS and registers allow it, a segment is merge sorted on the spot
// instead: by the one-wave workgroups (16384 rows of 256 f32 keys, as many of
// every magnitude, took 1115 us when handed over, 92 so) and for a plain call's
// only workgroup, which has nothing to hand over to and gives up at a third of
// kRankBudget, or a fifth if the words drop key bits, as every compare is then
// made twice (12000 u64 keys in 300 clusters: 88 us ranked, 72 merge sorted;
// 4001 with 10 % of them 0: 41, 30).
//
// Few distinct keys need no case of their own: d then has few bits and the
// bins go on with the position.
//
// Bound: VALU issue (a wave's instruction occupies its SIMD for four cycles)
// and HBM.  Hence 32-bit words computed once, one bin per element (few
// compares), and element minima by their upper halves first.  LDS is 8 B per
// element: words and bins share the memory of the staging area.
constexpr uint32_t kRankBudget = 128, kRankTotal = 1u << 20;  // compares: per element, in all
constexpr uint32_t kRankOwn = 4, kTiesOwn = 1024;

// Exclusive scan of the THREADS * BPT bin counts in place (bin is 16-byte
// aligned, BPT a multiple of 4); returns the sum of their squares, uniformly.
template <int THREADS, int BPT>
__device__ __forceinline__ uint32_t bins_scan(uint32_t* bin, uint32_t len, uint32_t* tmp, int t) {
  constexpr int NW = THREADS / kWave;
  static_assert(BPT % 4 == 0 && NW <= 16, "bins are read by fours, the waves' sums fit one row");
  const uint32_t lane = lane_id(), wv = t / kWave;
  uint4* const b4 = reinterpret_cast<uint4*>(bin) + t * (BPT / 4);
  uint32_t sum = 0, sq = 0;
#pragma unroll
  for (int k = 0; k < BPT / 4; k++) {
    const uint4 x = b4[k];
    sum += x.x + x.y + x.z + x.w;
    sq += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
  }
  const uint32_t inc = wave_incl_scan_dpp(sum), sqi = wave_incl_scan_dpp(sq);
  if (lane == kWave - 1) {
    tmp[wv] = inc;
    tmp[NW + wv] = sqi;
  }
  __syncthreads();
  // every wave scans the waves' sums in one row of lanes
  const uint32_t ws = row_incl_scan_dpp((int)lane < NW ? tmp[lane] : 0u);
  const uint32_t wq = row_incl_scan_dpp((int)lane < NW ? tmp[NW + lane] : 0u);
  const uint32_t uw = uniform(wv);
  const uint32_t off = uw ? lane_u32(ws, (int)uw - 1) : 0u, cost = lane_u32(wq, NW - 1);
  uint32_t e = off + inc - sum;
#pragma unroll
  for (int k = 0; k < BPT / 4; k++) {  // the counts are read again: fewer registers
    uint4 x = b4[k];
    const uint32_t e1 = e + x.x, e2 = e1 + x.y, e3 = e2 + x.z;
    b4[k] = make_uint4(e, e1, e2, e3);
    e = e3 + x.w;
  }
  if (t == THREADS - 1) bin[THREADS * BPT] = len;
  __syncthreads();
  return cost;
}

// How many of a[0, n) are below v, U at a time (a[n, n + U - 1) may be read;
// PAST: they are not below v either).
template <bool PAST, int U>
__device__ __forceinline__ uint32_t count_below(const uint32_t* a, uint32_t n, uint32_t v) {
  uint32_t less = 0;
#pragma unroll 1
  for (uint32_t k = 0; k < n; k += U) {
    uint32_t x[U];
#pragma unroll
    for (int u = 0; u < U; u++) x[u] = a[k + u];
#pragma unroll
    for (int u = 0; u < U; u++) less += (x[u] < v) & (u == 0 || PAST || k + u < n) ? 1u : 0u;
  }
  return less;
}

// Ranks of a segment with equal words.  Elements of equal rank r are a group
// of m that owns the ranks r .. r + m - 1; `rounds` times, the groups are
// ordered by the next 32 bits limb(round, i), U values read at a time.  fr and
// cnt hold N values each (fr: and 3 beyond) and are free on entry and exit (a
// barrier on both sides).
// BY_PLACE: a thread counts for the values at places i * THREADS + t instead
// of for its own elements.  Neighbouring lanes are then in one group, loop
// alike and read the same word, and a large group keeps only its own waves
// busy (its elements lie in every wave), for two more barriers and passes.
template <int THREADS, int ITEMS, int U, bool BY_PLACE, typename LimbFn>
__device__ __forceinline__ void rank_ties(uint32_t* fr, uint32_t* cnt, uint32_t len, uint32_t (&rank)[ITEMS],
                                          int rounds, LimbFn limb, int t) {
#pragma unroll 1
  for (int round = 0; round < rounds; round++) {
#pragma unroll
    for (int i = 0; i < ITEMS; i++) cnt[i * THREADS + t] = 0;
    __syncthreads();
    uint32_t pl[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
      pl[i] = 0;
      if (t < (int)len - i * THREADS) pl[i] = atomicAdd(&cnt[rank[i]], 1u);
    }
    __syncthreads();
    if constexpr (BY_PLACE) {
#pragma unroll
      for (int i = 0; i < ITEMS; i++)  // the group's size joins the place in it
        if (t < (int)len - i * THREADS) pl[i] |= cnt[rank[i]] << 16;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        if (t < (int)len - i * THREADS) {
          const uint32_t p = rank[i] + (pl[i] & 0xFFFFu);
          fr[p] = limb(round, i);
          cnt[p] = (pl[i] & 0xFFFF0000u) | rank[i];
          pl[i] = p;
        }
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        if (t < (int)len - i * THREADS) {
          uint32_t* const c = cnt + i * THREADS + t;
          const uint32_t g = *c, m = g >> 16;
          *c = m > 1 ? count_below<false, U>(fr + (g & 0xFFFFu), m, fr[i * THREADS + t]) : 0u;
        }
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < ITEMS; i++)
        if (t < (int)len - i * THREADS) rank[i] += cnt[pl[i]];
    } else {
#pragma unroll
      for (int i = 0; i < ITEMS; i++)
        if (t < (int)len - i * THREADS) fr[rank[i] + pl[i]] = limb(round, i);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        if (t < (int)len - i * THREADS) {
          const uint32_t m = cnt[rank[i]];
          if (m > 1) rank[i] += count_below<false, U>(fr + rank[i], m, limb(round, i));
        }
      }
    }
    __syncthreads();
  }
}

// Ranks words in bins by place: on entry rank[i] is the place in the bin, on
// exit the bin's start plus the smaller words in it.  Returns the sum of the
// thread's ranks; a barrier must follow before fr is written.
template <int THREADS, int ITEMS>
__device__ __forceinline__ uint32_t rank_by_place(uint32_t* fr, const uint32_t* bin, uint32_t len,
                                                  uint32_t (&wd)[ITEMS], int bsh, uint32_t (&rank)[ITEMS], int t) {
#pragma unroll
  for (int i = 0; i < ITEMS; i++) {
    if (t < (int)len - i * THREADS) {
      rank[i] += bin[wd[i] >> bsh];
      fr[rank[i]] = wd[i];
    }
  }
  if (t < 3) fr[len + t] = ~0u;
  __syncthreads();
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; i++) {
    if (t < (int)len - i * THREADS) {
      const uint32_t x = fr[i * THREADS + t], b = x >> bsh, s0 = bin[b];
      wd[i] = s0 + count_below<true, 4>(fr + s0, bin[b + 1] - s0, x);
      sum += wd[i];
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ITEMS; i++)
    if (t < (int)len - i * THREADS) fr[i * THREADS + t] = wd[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ITEMS; i++)
    if (t < (int)len - i * THREADS) rank[i] = fr[rank[i]];
  return sum;
}

// Sorts the final segments of the classes in a bit mask, the longest class
// first.  DIRECT: the whole input [0, n) of a plain call instead, by one
// workgroup.
template <typename K, bool F32, bool PAY, int THREADS, int ITEMS, int WPE, bool DIRECT = false>
__global__ __launch_bounds__(THREADS, WPE) void k_local_rank(Work w, uint32_t classes, const K* in_keys,
                                                             const uint32_t* in_pay, K* keys_out, uint32_t* perm_out,
                                                             uint32_t* pay_out) {
  constexpr int N = THREADS * ITEMS;
  constexpr int LB = 31 - __builtin_clz((unsigned)N);  // 2^LB bins: one per element, or more than half
  constexpr int BPT = (1 << LB) / THREADS;
  constexpr bool PAIRS = DIRECT || THREADS == kWave;  // crowded segments are merge sorted on the spot
  constexpr int NP = lpad_size(N), KW = (int)(sizeof(K) / 4);
  // words, then bins; the staging area of the output and the pairs use the same memory
  constexpr int MEM = PAIRS ? (KW + 1 + (PAY ? 1 : 0)) * NP : 0;
  __shared__ __align__(16) uint32_t s_mem[MEM > 2 * N + 8 ? MEM : 2 * N + 8];
  __shared__ uint32_t s_red[6 * (THREADS / kWave)];
  __shared__ uint32_t s_tmp[2 * (THREADS / kWave)];
  __shared__ uint32_t s_sum, s_crowd;
  __shared__ RunMap<DIRECT ? kWave : THREADS, DIRECT ? kWave : N> map;  // of the next segment, if it lies in a buffer
  uint32_t* const fr = s_mem;           // N words, and 3 beyond
  uint32_t* const bin = s_mem + N + 4;  // 2^LB + 1 bins
  uint64_t* const st = reinterpret_cast<uint64_t*>(s_mem);
  // the (at most three) classes, the longest first, and their segment counts
  const int c0 = 31 - __builtin_clz(classes);
  const uint32_t m1 = classes & ~(1u << c0);
  const int c1 = m1 ? 31 - __builtin_clz(m1) : c0;
  const uint32_t m2 = m1 & ~(1u << c1);
  const int c2 = m2 ? 31 - __builtin_clz(m2) : c1;
  const uint32_t n0 = DIRECT ? 1u : uniform(final_count(w, c0)), n1 = n0 + uniform(m1 ? final_count(w, c1) : 0u),
                 total = n1 + uniform(m2 ? final_count(w, c2) : 0u);
  auto seg_at = [&](uint32_t q) -> FinalSeg* {
    return q < n0 ? w.cls[c0] + q : q < n1 ? w.cls[c1] + (q - n0) : w.cls[c2] + (q - n1);
  };
  K key[ITEMS];
  uint32_t idx[ITEMS], pay[ITEMS];
  // Thread t takes elements i * THREADS + t.  One source per segment
  // (uniform), every lane loads (lanes past the end reload the last element),
  // so that all loads go out before any is used.  Input segments: scalar
  // bases, 32-bit byte offsets.
  auto load = [&](const FinalSeg& f, int t) {
    if (!DIRECT && f.src) {
      const BufView<K, PAY> bv{w.buf_rec[f.src - 1] + f.pstart * BufView<K, PAY>::W};
      if (map.over != 0) {  // uniform
#pragma unroll
        for (int i = 0; i < ITEMS; i++)
          bv.get(locate(w, (int)f.src - 1, f.col, 0, f.nt - 1, min((uint32_t)(i * THREADS + t), f.len - 1)), key[i],
                 idx[i], pay[i]);
      } else if (((uint64_t)f.nt << w.tile_log2) * (4 * BufView<K, PAY>::W) <= 0xFFFFFFFFull) {  // 32-bit offsets do
        map.each(t, f.len, [&](int i, uint32_t d) { bv.get32(d, key[i], idx[i], pay[i]); });
      } else {
        map.each(t, f.len, [&](int i, uint32_t d) { bv.get(d, key[i], idx[i], pay[i]); });
      }
    } else {
      const K* const kin = in_keys + f.start;
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        const uint32_t j = min((uint32_t)(i * THREADS + t), f.len - 1);
        key[i] = at32(kin, j);  // raw bits
        idx[i] = j;
        if constexpr (PAY) pay[i] = at32(in_pay + f.start, j);
      }
    }
  };
  auto uniform_seg = [](const FinalSeg& f) -> FinalSeg {
    return FinalSeg{uniform64(f.start), uniform64(f.pstart), uniform(f.len), uniform(f.src), uniform(f.col),
                    uniform(f.nt)};
  };
  // this thread's run of a buffer segment
  struct Run {
    uint32_t ofs, e, c;
  };
  auto run_of = [&](const FinalSeg& f, uint32_t t) -> Run {
    Run r{0u, 0u, 0u};
    if (f.src && t < f.nt) {
      const uint32_t *o = w.offs[f.src - 1] + f.col, v = w.runs[f.src - 1][f.col + t];
      r.ofs = o[t] - o[0];
      r.e = v >> 16;
      r.c = v & 0xFFFFu;
    }
    return r;
  };
  uint32_t q = blockIdx.x;
  if (q >= total) return;
  if constexpr (DIRECT) direct_reset(w);
  FinalSeg f = DIRECT ? FinalSeg{0ull, 0ull, (uint32_t)w.n, 0u, 0u, 0u} : uniform_seg(*seg_at(q));
  if constexpr (!DIRECT) {
    if (f.src) {
      const int t = threadIdx.x;
      const Run r = run_of(f, t);
      uint64_t bal;
      map.clear(t);
      __syncthreads();
      map.mark(t, t, f.nt, r.ofs, r.c, 0u, f.len, bal);
      __syncthreads();
      map.number(t, t, r.ofs, r.e, 0u, w.tile_log2, bal);
      __syncthreads();
    }
  }
  load(f, threadIdx.x);
  FinalSeg f_ahead = f;  // the next segment's descriptor, loaded an iteration ahead
  if constexpr (!DIRECT) f_ahead = *seg_at(q + gridDim.x < total ? q + gridDim.x : q);
  __syncthreads();  // every wave has read the map
  for (;;) {
    const uint32_t len = f.len, src = f.src;
    const uint64_t start = f.start;
    // the next segment's runs now, its elements before the last output of
    // this one (whose registers they take): a load that follows stores waits
    // for them, and so would the start of every segment
    const uint32_t qn = q + gridDim.x;
    const bool more = qn < total;
    FinalSeg fn = f;
    Run rn{0u, 0u, 0u};
    if constexpr (!DIRECT) {
      fn = uniform_seg(f_ahead);
      f_ahead = *seg_at(qn + gridDim.x < total ? qn + gridDim.x : q);
      rn = run_of(fn, threadIdx.x);
      map.clear(threadIdx.x);
    }
    uint64_t bal = 0;
    // an opaque copy of the thread index: per-thread addresses are recomputed
    // per segment rather than hoisted out of the loop and kept live
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    K* const kout = keys_out + start;
    uint32_t* const pout = perm_out ? perm_out + start : nullptr;
    uint32_t* const yout = PAY ? pay_out + start : nullptr;
    if constexpr (F32) {
      if (!src) {
#pragma unroll
        for (int i = 0; i < ITEMS; i++) key[i] = ord_of<K, F32>(key[i]);
      }
    }
#pragma unroll
    for (int b = 0; b < BPT / 4; b++) reinterpret_cast<uint4*>(bin)[b * THREADS + t] = make_uint4(0, 0, 0, 0);
    if (t == 0) s_sum = 0;
    if (DIRECT && t == 0) s_crowd = 0;
    // bounds of the keys (64-bit keys: of their upper halves) and positions
    constexpr int KS = sizeof(K) == 8 ? 32 : 0;
    uint32_t hmn = ~0u, hmx = 0u, imn = ~0u, imx = 0u;
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
      const uint32_t h = (uint32_t)((uint64_t)key[i] >> KS);
      hmn = min(hmn, h);
      hmx = max(hmx, h);
      imn = min(imn, idx[i]);
      imx = max(imx, idx[i]);
    }
    // (the barrier of the reduction also orders the stores above before their readers)
    const Range4 br = block_range<uint32_t, THREADS>(hmn, hmx, imn, imx, s_red, t);
    imn = br.imn;
    const uint32_t ir = br.imx - br.imn;
    K mn;
    uint64_t kr;
    if constexpr (sizeof(K) == 4) {
      mn = (K)br.kmn;
      kr = br.kmx - br.kmn;
    } else {
      mn = br.kmn << 32;
      kr = ((br.kmx - br.kmn) << 32) | 0xFFFFFFFFu;
      if (br.kmx - br.kmn < (1u << LB)) {  // uniform: the upper halves tell too little
        uint64_t mn2 = ~0ull, mx2 = 0ull;
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
          mn2 = key[i] < mn2 ? key[i] : mn2;
          mx2 = key[i] > mx2 ? key[i] : mx2;
        }
        __syncthreads();  // the first reduction's values have been read
        const Range4 b2 = block_range<uint64_t, THREADS>(mn2, mx2, 0u, 0u, s_red, t);
        mn = b2.kmn;
        kr = b2.kmx - b2.kmn;
      }
    }
    const int rb = kr ? 64 - __clzll((long long)kr) : 0, ib = ir ? 32 - __clz((int)ir) : 0;
    // wd = (d >> sr) << sl | x >> si: 32 bits, or rb + ib if that is less
    const int sr = max(rb - 32, 0), sl = min(32 - min(rb, 32), ib), si = ib - sl;
    const int bsh = max(min(rb, 32) + sl - LB, 0);
    uint32_t wd[ITEMS], rank[ITEMS];
    if (sl == 0) {  // uniform: key bits only
#pragma unroll
      for (int i = 0; i < ITEMS; i++) wd[i] = (uint32_t)((uint64_t)(K)(key[i] - mn) >> sr);
    } else {
#pragma unroll
      for (int i = 0; i < ITEMS; i++)
        wd[i] = ((rb ? (uint32_t)(key[i] - mn) : 0u) << (sl & 31)) | ((idx[i] - imn) >> si);
    }
    // One workgroup alone, whose atomics would queue up at crowded bins (7 of
    // 32 us for 4001 keys): a wave of whose first elements crowd_lanes share the
    // bin of one of two of them leaves its elements out, and if those waves
    // are few their elements are counted after all.  More lanes where the words
    // hold all key bits: with 6, 12000 u64 keys below 16, which rank well, were
    // merge sorted (26 us, 74 so); with 16, 250 keys of 16 values spread over
    // the type were ranked (9.4 us, 12.4 so).
    const int crowd_lanes = sr ? 6 : 16;
    bool out = false;
    if constexpr (DIRECT) {
      const uint32_t b = wd[0] >> bsh;
      const uint64_t same = __ballot(b == lane_u32(b, 0) || b == lane_u32(b, 21));
      out = __ballot(t < (int)len) == ~0ull && __popcll(same) >= crowd_lanes;
      if (out && lane_id() == 0) atomicAdd(&s_crowd, 1u);
    }
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
      rank[i] = 0;  // first the place in the bin
      if (t < (int)len - i * THREADS && !out) rank[i] = atomicAdd(&bin[wd[i] >> bsh], 1u);
    }
    if constexpr (!DIRECT) {
      if (fn.src) map.mark(t, t, fn.nt, rn.ofs, rn.c, 0u, fn.len, bal);
    }
    __syncthreads();
    if constexpr (!DIRECT) {
      if (fn.src) map.number(t, t, rn.ofs, rn.e, 0u, w.tile_log2, bal);
    }
    bool many = false;  // uniform
    if constexpr (DIRECT) {
      const uint32_t waves = s_crowd;
      many = waves * 4 * kWave >= min(len, (uint32_t)THREADS) && waves > 0;
      if (!many && waves > 0) {
#pragma unroll
        for (int i = 0; i < ITEMS; i++)
          if (t < (int)len - i * THREADS && out) rank[i] = atomicAdd(&bin[wd[i] >> bsh], 1u);
        __syncthreads();
      }
    }
    const uint32_t cost = many ? ~0u : bins_scan<THREADS, BPT>(bin, len, s_tmp, t);  // uniform
    const uint32_t limit = min((!DIRECT ? kRankBudget : sr ? kRankBudget / 5 : kRankBudget / 3) * len,
                               sr ? kRankTotal / 2 : kRankTotal);
    const bool crowded = many || cost > limit;
    if (crowded) {
      if constexpr (!PAIRS) {
        if (t == 0) {
          seg_at(q)->src = src | kPairsFlag;
          if (src) w.ctl->pairs_in[src - 1] = 1;
        }
      } else {
        const LdsArr<K> sa{s_mem, s_mem + (KW - 1) * NP, s_mem + KW * NP, s_mem + (KW + 1) * NP};
        constexpr int H = DIRECT && ITEMS <= 8 ? ITEMS / 2 : ITEMS;
        if (H < ITEMS && len <= THREADS * H) {  // uniform
          K k[H];
          uint32_t v[H], y[H];
#pragma unroll
          for (int i = 0; i < H; i++) {
            k[i] = key[i];
            v[i] = idx[i];
            if constexpr (PAY) y[i] = pay[i];
          }
          merge_pairs<K, PAY, THREADS, H>(k, v, y, len, sa);
        } else {
          merge_pairs<K, PAY, THREADS, ITEMS>(key, idx, pay, len, sa);
        }
        put_pairs<K, F32, PAY, THREADS>(sa, len, kout, pout, yout);
      }
    } else {
    uint32_t sum = 0;
    if (cost <= kRankOwn * len) {  // uniform
#pragma unroll
      for (int i = 0; i < ITEMS; i++)
        if (t < (int)len - i * THREADS) fr[bin[wd[i] >> bsh] + rank[i]] = wd[i];
      if (t < 3) fr[len + t] = ~0u;
      __syncthreads();
      // bin start and size of every element, then its rank
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        if (t < (int)len - i * THREADS) {
          const uint32_t b = wd[i] >> bsh, s0 = bin[b];
          rank[i] = ((bin[b + 1] - s0) << 16) | s0;
        }
      }
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        if (t < (int)len - i * THREADS) {
          rank[i] = (rank[i] & 0xFFFFu) + count_below<true, 4>(fr + (rank[i] & 0xFFFFu), rank[i] >> 16, wd[i]);
          sum += rank[i];
        }
      }
    } else {
      sum = rank_by_place<THREADS, ITEMS>(fr, bin, len, wd, bsh, rank, t);
    }
    const bool exact = sr == 0 && si == 0;  // uniform: words are distinct
    if (!exact) {
      sum = wave_incl_scan_dpp(sum);
      if (lane_id() == kWave - 1) atomicAdd(&s_sum, sum);
    }
    __syncthreads();  // every word read
    const uint32_t missing = exact ? 0u : (uint32_t)(((uint64_t)len * (len - 1)) >> 1) - s_sum;  // uniform
    if (missing != 0) {
      // the bits of (d, x) below the word: those of d that were dropped (sr of
      // them), then x (all of it, or its low si bits)
      auto limb = [&](int round, int i) -> uint32_t {
        return sr && round == 0 ? (uint32_t)(key[i] - mn) : idx[i] - imn;
      };
      constexpr int U = sizeof(K) == 8 && !DIRECT ? 2 : 4;
      if (missing > kTiesOwn)
        rank_ties<THREADS, ITEMS, U, true>(fr, bin, len, rank, sr ? 2 : 1, limb, t);
      else
        rank_ties<THREADS, ITEMS, U, false>(fr, bin, len, rank, sr ? 2 : 1, limb, t);
    }
    // into rank order and out; the last array's registers are free for the
    // next segment once it is staged
    if constexpr (sizeof(K) == 4) {
#pragma unroll
      for (int i = 0; i < ITEMS; i++)
        if (t < (int)len - i * THREADS) st[rank[i]] = ((uint64_t)idx[i] << 32) | key[i];
    } else {
#pragma unroll
      for (int i = 0; i < ITEMS; i++)
        if (t < (int)len - i * THREADS) st[rank[i]] = (uint64_t)key[i];
    }
    constexpr bool TWO = sizeof(K) == 8 || PAY;  // two rounds through the staging area
    if constexpr (TWO) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        const uint32_t j = i * THREADS + t;
        if (t < (int)len - i * THREADS) {
          const uint64_t x = st[j];
          at32(kout, j) = to_output<K, F32>((K)x);
          if constexpr (sizeof(K) == 4) {
            if (pout) at32(pout, j) = (uint32_t)(x >> 32);
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        if (t < (int)len - i * THREADS) {
          if constexpr (sizeof(K) == 4)
            fr[rank[i]] = pay[i];
          else if constexpr (PAY)
            st[rank[i]] = ((uint64_t)pay[i] << 32) | idx[i];
          else
            fr[rank[i]] = idx[i];
        }
      }
    }
    }
    __syncthreads();
    if (more) load(fn, t);
    if (!crowded) {
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        const uint32_t j = i * THREADS + t;
        if (t < (int)len - i * THREADS) {
          if constexpr (sizeof(K) == 4 && !PAY) {
            const uint64_t x = st[j];
            at32(kout, j) = to_output<K, F32>((K)x);
            if (pout) at32(pout, j) = (uint32_t)(x >> 32);
          } else if constexpr (sizeof(K) == 4) {
            at32(yout, j) = fr[j];
          } else if constexpr (PAY) {
            const uint64_t x = st[j];
            if (pout) at32(pout, j) = (uint32_t)x;
            at32(yout, j) = (uint32_t)(x >> 32);
          } else {
            if (pout) at32(pout, j) = fr[j];
          }
        }
      }
    }
    if (!more) break;
    q = qn;
    f = fn;
    __syncthreads();  // the next segment clears its bins in the staging area
  }
}

// ---------------------------------------------------------------------------
// Fallback for a final segment longer than cap (the balance guarantee of the
// sampling holds only with high probability): one workgroup sorts chunks of C
// elements in LDS into the segment's own range of the buffer that does not hold
// its level's elements, and then finds every element's rank by a binary search
// in each other chunk and writes it out.  Nothing else reads or writes that
// range, so that segments are independent of each other, unless segments of
// that buffer were handed over (they may be read at the same time): then a
// sorted chunk takes the places its elements had in their own buffer, which
// costs a search for every place.  A segment seldom has more than two chunks;
// the searches (a chain of dependent loads) run for U elements at a time.
template <typename K, bool F32, bool PAY, int THREADS, int ITEMS>
__device__ __forceinline__ void sort_oversize(const Work& w, const FinalSeg& f, const LdsArr<K>& sa, void* map,
                                              const K* in_keys, const uint32_t* in_pay, K* keys_out,
                                              uint32_t* perm_out, uint32_t* pay_out) {
  using View = BufView<K, PAY>;
  // (the debug switch: smaller chunks, so that there are several)
  const uint32_t C = f.len <= THREADS * ITEMS ? THREADS * ITEMS / 4 : THREADS * ITEMS;
  const SegReader<K, F32, PAY> rd{w, f, in_keys, in_pay};
  const bool own = f.src && uniform(w.ctl->pairs_in[(f.src - 1) ^ 1]) != 0;  // uniform
  const View b{w.buf_rec[f.src == 0 ? 0u : own ? f.src - 1 : (f.src - 1) ^ 1]};
  auto at = [&](uint32_t q) -> uint64_t { return own ? rd.at(q) : f.start + q; };
  for (uint32_t c0 = 0; c0 < f.len; c0 += C) {
    const uint32_t cnt = min(C, f.len - c0);
    sort_stretch_fit<K, F32, PAY, THREADS, ITEMS>(rd, c0, cnt, sa, map);
    for (uint32_t j = threadIdx.x; j < cnt; j += THREADS) {
      const int q = lpad(j);
      b.put(at(c0 + j), sa.key(q), sa.v[q], PAY ? sa.p[q] : 0u);
    }
    __syncthreads();
  }
  constexpr int U = 4;
  for (uint32_t j0 = threadIdx.x; j0 < f.len; j0 += THREADS * U) {
    K k[U];
    uint32_t v[U], y[U], rank[U];
#pragma unroll
    for (int u = 0; u < U; u++) b.get(at(min(j0 + u * THREADS, f.len - 1)), k[u], v[u], y[u]);
#pragma unroll
    for (int u = 0; u < U; u++) rank[u] = (j0 + u * THREADS) % C;
#pragma unroll 1
    for (uint32_t c0 = 0; c0 < f.len; c0 += C) {
      // elements of the chunk below each: the first lo are, those from lo + n on are not
      uint32_t lo[U];
#pragma unroll
      for (int u = 0; u < U; u++) lo[u] = 0;
#pragma unroll 1
      for (uint32_t n = min(C, f.len - c0); n > 0;) {
        const uint32_t half = n >> 1;
#pragma unroll
        for (int u = 0; u < U; u++) {
          const uint64_t q = at(c0 + lo[u] + half);
          lo[u] += pair_less(b.key(q), b.idx(q), k[u], v[u]) ? n - half : 0u;
        }
        n = half;
      }
#pragma unroll
      for (int u = 0; u < U; u++) rank[u] += (j0 + u * THREADS) / C * C == c0 ? 0u : lo[u];
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      if (j0 + u * THREADS < f.len) {
        keys_out[f.start + rank[u]] = to_output<K, F32>(k[u]);
        if (perm_out) perm_out[f.start + rank[u]] = v[u];
        if constexpr (PAY) pay_out[f.start + rank[u]] = y[u];
      }
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// What is left after all classes, in one resident-sized launch: the segments
// k_local_rank handed over, of every class, by the merge sort of pairs, and the
// segments longer than the LDS capacity (sort_oversize).  Each thread checks
// one list entry and the marked ones are collected in LDS, so that the search
// is parallel rather than a chain of dependent loads.  No register is spilled:
// scratch memory for spills adds 4 to 6 us to a call, however empty the launch.
template <typename K, bool F32, bool PAY, int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_local_rare(Work w, const K* in_keys, const uint32_t* in_pay, K* keys_out,
                                                        uint32_t* perm_out, uint32_t* pay_out) {
  constexpr int NP = lpad_size(THREADS * ITEMS);
  __shared__ RunMap<THREADS, THREADS * ITEMS> map;  // (large enough for every shape)
  __shared__ uint32_t s_lo[NP];
  __shared__ uint32_t s_hi[sizeof(K) == 8 ? NP : 1];
  __shared__ uint32_t s_v[NP];
  __shared__ uint32_t s_p[PAY ? NP : 1];
  __shared__ uint32_t s_list[THREADS];
  __shared__ uint32_t s_n;
  const LdsArr<K> sa{s_lo, s_hi, s_v, s_p};
  for (int c = 0; c <= kNumClasses - 2; c++) {
    const uint32_t cnt = final_count(w, c);
    // neighbouring entries go to different workgroups: marked segments
    // (the tails of a distribution) often lie next to each other
    for (uint32_t q0 = 0; q0 < cnt; q0 += gridDim.x * THREADS) {
      if (threadIdx.x == 0) s_n = 0;
      __syncthreads();
      const uint32_t q = q0 + threadIdx.x * gridDim.x + blockIdx.x;
      if (q < cnt && (w.cls[c][q].src & kPairsFlag)) s_list[atomicAdd(&s_n, 1u)] = q;
      __syncthreads();
      const uint32_t n = s_n;
      for (uint32_t k = 0; k < n; k++) {
        FinalSeg f = w.cls[c][s_list[k]];
        f.src &= 0xFFu;
        const SegReader<K, F32, PAY> rd{w, f, in_keys, in_pay};
        sort_stretch_fit<K, F32, PAY, THREADS, ITEMS>(rd, 0, f.len, sa, &map);
        put_pairs<K, F32, PAY, THREADS>(sa, f.len, keys_out + f.start, perm_out ? perm_out + f.start : nullptr,
                                        PAY ? pay_out + f.start : nullptr);
      }
      __syncthreads();
    }
  }
  // a workgroup per oversize segment (8e8 u32 keys, whose mean bucket is half the
  // capacity: 13.6 ms; 225 when one workgroup took them all)
  const uint32_t cnt = final_count(w, kNumClasses - 1);
  for (uint32_t q = blockIdx.x; q < cnt; q += gridDim.x) {
    const FinalSeg f = w.cls[kNumClasses - 1][q];
    sort_oversize<K, F32, PAY, THREADS, ITEMS>(w, f, sa, &map, in_keys, in_pay, keys_out, perm_out, pay_out);
  }
}

// A plain call that fits one workgroup.  Many threads with few elements each:
// one workgroup has the GPU to itself.
template <typename K, bool F32, int T, int I>
static int direct_launch(const Work& w, const K* kin, K* kout, uint32_t* perm_out, hipStream_t st) {
  static const std::string tag =
      "(k_local_rank<K, F32, PAY, " + std::to_string(T) + ", " + std::to_string(I) + ", true>)";
  RS_LAUNCH_TAGGED((k_local_rank<K, F32, false, T, I, 4, true>), tag.c_str(), 1, T, st, w, 1u, kin, nullptr, kout,
                   perm_out, nullptr);
  return 0;
}

template <typename K, bool F32>
int launch_direct(const Work& w, const K* kin, K* kout, uint32_t* perm_out, hipStream_t st) {
  if (w.n <= 256) return direct_launch<K, F32, 64, 4>(w, kin, kout, perm_out, st);
  if (w.n <= 1024) return direct_launch<K, F32, 256, 4>(w, kin, kout, perm_out, st);
  if (w.n <= 4096) return direct_launch<K, F32, 1024, 4>(w, kin, kout, perm_out, st);
  if (w.n <= 8192) return direct_launch<K, F32, 1024, 8>(w, kin, kout, perm_out, st);
  return direct_launch<K, F32, 1024, 12>(w, kin, kout, perm_out, st);
}

// Classes sorted by one launch of k_local_rank, on workgroups of T threads
// with I elements each, per_cu of them per CU: four times what a CU holds (each
// takes several segments, the next one's elements in flight while it writes
// out; once or twice as many measured the same), fewer of the one-wave
// workgroups, whose dispatch alone took 8 us when there were 32768.
template <typename K, bool F32, bool PAY, int T, int I, int WPE>
static int rank_launch(uint32_t classes, uint32_t per_cu, const Work& w, const K* kin, const uint32_t* pay_in,
                       K* kout, uint32_t* perm_out, uint32_t* pay_out, hipStream_t st) {
  static const std::string tag =
      "(k_local_rank<K, F32, PAY, " + std::to_string(T) + ", " + std::to_string(I) + ">)";
  if (!classes) return 0;
  uint64_t cap = 0;
  for (int c = 0; c < kNumClasses - 1; c++) cap += (classes >> c) & 1u ? w.cls_cap[c] : 0;
  RS_LAUNCH_TAGGED((k_local_rank<K, F32, PAY, T, I, WPE>), tag.c_str(), grid_for(cap, per_cu), T, st, w, classes,
                   kin, pay_in, kout, perm_out, pay_out);
  return 0;
}

// Shapes.  What counts is how many elements a CU has in flight without
// register spills (a spilled register's reload waits for the output stores:
// 512 x 8 bounded to 64 registers took 856 instead of 547 us on the buckets
// of at most 4096 of 2^28 u64 keys).  512 x 8 (80 registers, 33 KB) runs
// three workgroups per CU, 512 x 12 (109 registers, 49 KB) two: the buckets of
// 4097 to 6144 of that sort took 1230 us in 1024 x 8 workgroups, 1150 us in
// 512 x 16 and 751 us in 512 x 12.  With a payload 512 x 8 keeps its 97
// registers (297 us on the 1 GiB batch; 327 at 80).
template <typename K, bool F32, bool PAY>
int launch_local_ranks(uint32_t classes, const Work& w, const K* kin, const uint32_t* pay_in, K* kout,
                       uint32_t* perm_out, uint32_t* pay_out, hipStream_t st) {
  int rc = 0;
  // longest segments first (a payload call has no class of 12288)
  if constexpr (PAY)
    rc = rank_launch<K, F32, PAY, 1024, 8, 4>(classes & 0x80u, 4, w, kin, pay_in, kout, perm_out, pay_out, st);
  else
    rc = rank_launch<K, F32, PAY, 1024, 12, 4>(classes & 0x180u, 4, w, kin, pay_in, kout, perm_out, pay_out, st);
  if (!rc) rc = rank_launch<K, F32, PAY, 512, 12, 4>(classes & 0x40u, 8, w, kin, pay_in, kout, perm_out, pay_out, st);
  if (!rc)
    rc = rank_launch<K, F32, PAY, 512, 8, PAY ? 4 : 6>(classes & 0x38u, 12, w, kin, pay_in, kout, perm_out, pay_out,
                                                       st);
  if (!rc) rc = rank_launch<K, F32, PAY, 256, 4, 8>(classes & 0x04u, 16, w, kin, pay_in, kout, perm_out, pay_out, st);
  if (!rc)  // (seven waves per SIMD where the pairs would spill registers at eight)
    rc = rank_launch<K, F32, PAY, 64, 4, PAY || sizeof(K) == 8 ? 7 : 8>(classes & 0x03u, 32, w, kin, pay_in, kout,
                                                                       perm_out, pay_out, st);
  if (rc) return rc;
  if constexpr (PAY)
    RS_LAUNCH((k_local_rare<K, F32, PAY, 1024, 8>), grid_for(1u << 30, 1), 1024, st, w, kin, pay_in, kout, perm_out,
              pay_out);
  else
    RS_LAUNCH((k_local_rare<K, F32, PAY, 768, 16>), grid_for(1u << 30, 1), 768, st, w, kin, pay_in, kout, perm_out,
              pay_out);
  return 0;
}

#define RS_INST_LOCAL(K, F, P)                                                                                    \
  template int launch_local_ranks<K, F, P>(uint32_t, const Work&, const K*, const uint32_t*, K*, uint32_t*,        \
                                           uint32_t*, hipStream_t);
RS_INST_LOCAL(uint32_t, false, false)
RS_INST_LOCAL(uint32_t, true, false)
RS_INST_LOCAL(uint64_t, false, false)
RS_INST_LOCAL(uint32_t, false, true)
RS_INST_LOCAL(uint32_t, true, true)
RS_INST_LOCAL(uint64_t, false, true)

template int launch_direct<uint32_t, false>(const Work&, const uint32_t*, uint32_t*, uint32_t*, hipStream_t);
template int launch_direct<uint32_t, true>(const Work&, const uint32_t*, uint32_t*, uint32_t*, hipStream_t);
template int launch_direct<uint64_t, false>(const Work&, const uint64_t*, uint64_t*, uint32_t*, hipStream_t);

}  // namespace rs
