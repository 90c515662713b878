// Multilevel sample sort engine (paper Appendix G: robust multi-level sample
// sort, RAMS) for one GPU, plus the LDS sort of its final buckets.
//
// One level splits every "big" segment (more than `cap` elements) into
// k = 2^logk buckets:
//   splitters  draw a*k random sample positions per segment, gather
//              (key, position) pairs, sort them in LDS and keep every a-th
//              as a splitter (positions break key ties, Appendix G);
//   split      classify every element with a branchless descent of the
//              splitter tree held in LDS (a Super Scalar Sample Sort style
//              classifier; a key equal to a splitter key is resolved by the
//              positions), rank inside (tile, bucket) with LDS atomics, stage
//              the tile in LDS grouped by bucket and write it back as one
//              contiguous piece, with the length of each bucket's run;
//   scan       exclusive prefix sum of the [segment][bucket][tile] run
//              lengths: the bucket bounds, and where each run's elements
//              stand in their bucket;
//   route      the level's buckets: split again or sort in LDS.
// The paper's all-to-all exchange is thus done by the readers: the next level
// and the local sorts gather a bucket's runs, one per tile (32 elements each
// where 256 buckets share a tile of 8192).  Elements are read and written
// once per level; no pass counts them first.
// Buckets at most `cap` long become final segments and are sorted, one
// workgroup each, in LDS; the rest are split again at the next level.
// Everything is sized on the device: no bucket size returns to the host.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>

#include "device.hpp"
#include "engine.hpp"
#include "internal.hpp"

namespace rs {

// Size classes of final segments (upper bounds); the last is "oversize".
__constant__ uint32_t c_class_max[kNumClasses] = {64, 256, 1024, 2048, 3072, 4096, 6144, 8192, 12288, 0xFFFFFFFFu};
static const uint32_t h_class_max[kNumClasses] = {64, 256, 1024, 2048, 3072, 4096, 6144, 8192, 12288, 0xFFFFFFFFu};

uint32_t class_max(int c) { return (c >= 0 && c < kNumClasses) ? h_class_max[c] : 0u; }

// cmin: the smallest class used.  A sort with few final buckets routes them
// all to one or two large classes, so that they run in one launch that fills
// the GPU instead of several nearly idle ones.
__device__ __forceinline__ uint32_t class_of(uint32_t len, uint32_t cap, uint32_t force_fallback, uint32_t cmin) {
  if (len > cap || (force_fallback && len > 64)) return kNumClasses - 1;
  uint32_t c = cmin;
  while (len > c_class_max[c]) c++;
  return c;
}

// log2 of the bucket count for a segment of len keys that still has `left`
// levels (this one included) to reach buckets of about `target` keys: the
// 2^lq buckets needed are shared out over the levels the segment needs, the
// upper levels taking the smaller share (fewer buckets where the data is
// largest keeps the runs of a tile long).  Only a plan with extra levels
// (`spread`) spreads them over more levels than the fewest that reach the
// target, at least 4 buckets per level; otherwise a segment of a batch that
// needs one level takes one, however many the batch's largest needs.
__device__ __forceinline__ uint32_t logk_for(uint32_t len, uint32_t target, uint32_t left, uint32_t spread) {
  const uint32_t q = (len + target - 1) / target;  // buckets wanted
  const uint32_t lq = q <= 1 ? 0u : 32u - __clz(q - 1);
  const uint32_t need = (lq + kMaxLogK - 1) / kMaxLogK;
  const uint32_t fewest = max(need, 1u);
  const uint32_t lv = left < need ? left : (spread ? max(fewest, min(left, lq / 2)) : fewest);
  uint32_t lk = lv > 1 ? lq / lv : lq;
  lk = lk < 1u ? 1u : lk;
  return lk > (uint32_t)kMaxLogK ? (uint32_t)kMaxLogK : lk;
}

__device__ __forceinline__ void set_status(Ctl* ctl, int32_t code) { atomicCAS(&ctl->status, 0, code); }

// Tiles of a segment of len elements.
__device__ __forceinline__ uint32_t tiles_of(const Work& w, uint32_t len) {
  return (uint32_t)(((uint64_t)len + (1u << w.tile_log2) - 1) >> w.tile_log2);
}


// Routing of a block's segments to the list of segments to split (index
// kNumClasses) or to the final lists by size class, aggregated per block:
// slots are counted in LDS (one LDS atomic per segment), then one global
// atomic per list and block reserves them.  Every thread of the block
// calls once per iteration of a block-uniform loop; `lds` is zeroed before
// the first call (route_lds_init) and is left zeroed.
struct RouteLds {
  uint32_t cnt[kNumClasses + 1];
  uint32_t base[kNumClasses + 1];
  unsigned long long keys[kNumClasses];
  uint32_t tiles, entries, tile_base, entry_base;  // of the segments to split
};

__device__ __forceinline__ void route_lds_init(RouteLds& L) {
  if (threadIdx.x <= (unsigned)kNumClasses) {
    L.cnt[threadIdx.x] = 0;
    if (threadIdx.x < (unsigned)kNumClasses) L.keys[threadIdx.x] = 0;
  }
  if (threadIdx.x == 0) L.tiles = L.entries = 0;
  __syncthreads();
}

__device__ __forceinline__ void route(const Work& w, RouteLds& L, int next, bool active, bool to_big, FinalSeg f,
                                      uint64_t ubase, uint32_t cap, uint32_t ff, uint32_t target, uint32_t left,
                                      uint32_t cmin) {
  const uint32_t c = (active && !to_big) ? class_of(f.len, cap, ff, cmin) : 0u;
  const uint32_t dest = to_big ? (uint32_t)kNumClasses : c;
  const uint32_t li = active ? atomicAdd(&L.cnt[dest], 1u) : 0u;
  // a segment to split takes its tiles and matrix entries of the next level
  const bool big = active && to_big;
  uint32_t logk = 0, tb = 0, cb = 0;
  if (big) {
    const uint32_t nt = tiles_of(w, f.len);
    logk = logk_for(f.len, target, left, w.spread);
    tb = atomicAdd(&L.tiles, nt);
    cb = atomicAdd(&L.entries, nt << logk);
  }
  if (active && !to_big) atomicAdd(&L.keys[c], (unsigned long long)f.len);  // (statistics)
  __syncthreads();
  if (threadIdx.x <= (unsigned)kNumClasses) {
    const uint32_t t = threadIdx.x, n = L.cnt[t];
    uint32_t* ctr = t == (uint32_t)kNumClasses ? &w.ctl->big_count[next] : &w.ctl->class_count[t];
    L.base[t] = n ? atomicAdd(ctr, n) : 0u;
    if (t < (uint32_t)kNumClasses && L.keys[t]) atomicAdd((unsigned long long*)&w.ctl->class_keys[t], L.keys[t]);
    L.cnt[t] = 0;
    if (t < (uint32_t)kNumClasses) L.keys[t] = 0;
    if (t == (uint32_t)kNumClasses && n) {
      L.tile_base = atomicAdd(&w.ctl->tiles[next], L.tiles);
      L.entry_base = atomicAdd(&w.ctl->entries[next], L.entries);
      L.tiles = L.entries = 0;
    }
  }
  __syncthreads();
  if (active) {
    const uint32_t i = L.base[dest] + li;
    if (to_big) {
      if (i < w.big_max)
        w.big[next][i] = BigSeg{f.start, ubase, f.pstart, f.len, logk, f.col, f.nt, L.tile_base + tb, L.entry_base + cb};
      else
        set_status(w.ctl, -3);  // capacity bound violated: internal error
    } else {
      if (i < w.cls_cap[c])
        w.cls[c][i] = f;
      else
        set_status(w.ctl, -3);
    }
  }
}

// ---------------------------------------------------------------------------
__global__ void k_reset(Ctl* ctl, uint32_t levels) {
  uint32_t* p = reinterpret_cast<uint32_t*>(ctl);
  const uint32_t nw = (uint32_t)(offsetof(Ctl, l0_spl_key) / 4);
  for (uint32_t i = threadIdx.x; i < nw; i += blockDim.x) p[i] = (i == 1) ? levels : 0u;
}

// Route every user segment: split it (big list 0) or sort it directly.  With
// bad offsets (status -1) no segment is split: overlapping ones would take more
// tiles and matrix entries than the workspace has room for.  The last workgroup
// to come through sees the status of all.
__global__ void k_init(Work w, const uint64_t* seg_off, uint32_t num_segs, uint64_t n_total, uint32_t cap,
                       uint32_t target, uint32_t levels, uint32_t ff, uint32_t cmin) {
  __shared__ RouteLds L;
  route_lds_init(L);
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t s0 = blockIdx.x * blockDim.x; s0 < num_segs; s0 += stride) {
    const uint32_t s = s0 + threadIdx.x;
    bool active = s < num_segs;
    uint64_t a = 0, b = 0;
    if (active) {
      a = seg_off ? seg_off[s] : 0ull;
      b = seg_off ? seg_off[s + 1] : n_total;
      if (b < a || b > n_total || (s == 0 && a != 0) || (s + 1 == num_segs && b != n_total) ||
          b - a >= 0xFFFFFFFFull) {
        atomicExch(&w.ctl->status, -1);  // (whatever else was found)
        __threadfence();                 // before the workgroup is counted below
        active = false;
      }
    }
    const uint32_t len = active ? (uint32_t)(b - a) : 0u;
    active = active && len > 0;
    route(w, L, 0, active, len > cap && levels > 0, FinalSeg{a, 0ull, len, 0u, 0u, 0u}, a, cap, ff, target, levels,
          cmin);
  }
  __syncthreads();  // (the counts' atomics have returned their values)
  if (threadIdx.x != 0 || atomicAdd(&w.ctl->init_done, 1u) + 1u != gridDim.x) return;
  if (atomicAdd(&w.ctl->status, 0) != 0) {
    atomicExch(&w.ctl->big_count[0], 0u);
    atomicExch(&w.ctl->tiles[0], 0u);
    atomicExch(&w.ctl->entries[0], 0u);
  }
}

// The splitter kernel's shape: up to kSplThreads * kSplItems samples per segment.
constexpr int kSplThreads = 1024, kSplItems = 8;  // (a = 32 at k = 256, 16 at 512)
constexpr uint32_t kStartThreads = 256;

// A plain sort's start in one launch: reset the control block, route the one
// segment [0, n) (split it, or sort it in its class), and give it its tiles.
// With `staged` (a split sort of at least kSplThreads * kSplItems keys), the
// workgroups also draw the first level's sample, the same a0 * k positions
// the splitter kernel would, and store the (raw key, position) records at the
// front of buffer B, which the first level does not touch before its split:
// the random loads are spread over many CUs instead of coming from the
// splitter kernel's one workgroup.
template <typename K>
__global__ __launch_bounds__(kStartThreads) void k_start_plain(Work w, uint64_t n, uint32_t cap, uint32_t target,
                                                              uint32_t levels, uint32_t ff, uint32_t cmin,
                                                              const K* in_keys, uint32_t a0, uint64_t seed,
                                                              int staged) {
  if (staged) {
    const uint32_t logk = logk_for((uint32_t)n, target, levels, w.spread);
    const uint32_t S = min(a0, (uint32_t)(kSplThreads * kSplItems) >> logk) << logk;
    const uint32_t j = blockIdx.x * kStartThreads + threadIdx.x;
    if (j < S) {
      // level 0, segment start 0: the stream and position of k_splitters
      const uint64_t r = rand_at(seed, 0ull, j);
      const uint64_t pos = ((r >> 32) * n) >> 32;
      BufView<K, false>{w.buf_rec[1]}.put(j, in_keys[pos], (uint32_t)pos, 0u);
    }
    if (blockIdx.x != 0) return;
  }
  uint32_t* p = reinterpret_cast<uint32_t*>(w.ctl);
  const uint32_t nw = (uint32_t)(offsetof(Ctl, l0_spl_key) / 4);
  for (uint32_t i = threadIdx.x; i < nw; i += blockDim.x) p[i] = (i == 1) ? levels : 0u;
  __syncthreads();
  if (threadIdx.x != 0 || n == 0) return;
  const uint32_t len = (uint32_t)n;
  if (len > cap && levels > 0) {
    const uint32_t logk = logk_for(len, target, levels, w.spread);
    const uint32_t nt = tiles_of(w, len);
    w.big[0][0] = BigSeg{0ull, 0ull, 0ull, len, logk, 0u, 0u, 0u, 0u};
    w.ctl->big_count[0] = 1;
    w.ctl->tiles[0] = nt;
    w.ctl->entries[0] = nt << logk;
  } else {
    const uint32_t c = class_of(len, cap, ff, cmin);
    w.cls[c][0] = FinalSeg{0ull, 0ull, len, 0u, 0u, 0u};
    w.ctl->class_count[c] = 1;
    w.ctl->class_keys[c] = n;
  }
}

// Splitter selection: one workgroup per segment.  S = a << logk sample
// positions drawn uniformly (with replacement) from the segment; the
// (key, position) pairs are sorted in LDS and every a-th becomes a splitter.
// The k-1 splitters are stored as an implicit binary search tree: node t at
// depth d, index q = t - 2^d within its depth, holds splitter number
// (2q+1) * 2^(logk-1-d) (1-based, in sorted order).  The workgroup also writes
// down, for each of the segment's tiles, the segment and (buffer levels) the
// run that holds the tile's first element.
// Plain sorts of at least this many keys launch both forms of the first split
// (see k_split): the empty one costs 3 us, 0.15 % of such a sort (2^28 uniform
// u64 keys 4697 us with and without it), and the tiled one saves a fifth of
// the launch where splitters repeat keys.  Both forms from 2^23 keys on, and
// from 2^27 on, in us for u64 keys: uniform ones of 9000000 280 and 277, 2^25
// 732 and 730, 2^27 - 1 2511 and 2512; keys below 16 of 2^25 799 and 836, 2^27 - 1
// 2556 and 2694; 30 % one key, 2^27 - 1, 2668 and 2982.  So a lower bound gives up to 1 %
// of the smaller sorts of distinct keys for 4 to 12 % of those of repeated ones;
// distinct keys are taken to be the rule here.
constexpr uint64_t kTiledMin = 1ull << 27;
constexpr uint32_t kSplRankBudget = 64;  // compares per sample the ranking path may take
template <typename K, bool F32, bool SRC_IN, bool PAY, int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_splitters(Work w, int lev, const K* in_keys, int src_buf,
                                                       uint32_t a, uint64_t seed, int staged) {
  constexpr int N = THREADS * ITEMS;
  constexpr int NP = lpad_size(N);
  constexpr int LB = 31 - __builtin_clz((unsigned)N);  // bins of the ranking path
  constexpr int PL = (1 << LB) / THREADS;
  static_assert(PL >= 1, "one bin per thread at least");
  __shared__ uint32_t s_lo[NP];
  __shared__ uint32_t s_hi[sizeof(K) == 8 ? NP : 1];
  __shared__ uint32_t s_v[NP];
  __shared__ uint32_t s_bin[(1 << LB) + 1];
  __shared__ uint32_t s_red[6 * (THREADS / kWave)];
  __shared__ uint32_t s_tmp[THREADS / kWave + 1];
  __shared__ uint32_t s_cost;
  const LdsArr<K> sa{s_lo, s_hi, s_v, nullptr};
  const int cur = lev & 1;
  const uint32_t m = (uint32_t)min((uint64_t)w.ctl->big_count[cur], w.big_max);
  const BufView<K, PAY> bv{SRC_IN ? nullptr : w.buf_rec[src_buf]};
  K* tkey = (K*)w.tree_key;
  for (uint32_t s = blockIdx.x; s < m; s += gridDim.x) {
    const BigSeg bs = w.big[cur][s];
    // a samples per bucket, fewer when a * k would exceed the LDS sample (or a
    // short segment's length)
    uint32_t ae = min(a, (uint32_t)(THREADS * ITEMS) >> bs.logk);
    if constexpr (!SRC_IN) ae = min(ae, max(bs.len >> bs.logk, 1u));
    const uint32_t S = ae << bs.logk;
    const uint32_t ntiles = tiles_of(w, bs.len);
    if (!SRC_IN || m > 1) {  // (the tiles of an only input segment are known to be its)
      for (uint32_t i = threadIdx.x; i < ntiles; i += THREADS) w.tile_seg[bs.tb + i] = s;
    }
    if constexpr (!SRC_IN) {
      // One walk over the segment's runs finds the run that holds each tile's
      // first element and the places of the samples, which are drawn one from
      // each of S equal stretches of the segment (the first rem of them are
      // one element longer), so that a run need only look at its own
      // stretches.  (Looking each sample's run up took 8 or more dependent
      // loads: 187 us for the 256 segments of 2^28 keys.)
      constexpr int U = 8;  // runs a thread has in flight
      const uint32_t *o = w.offs[src_buf] + bs.col, *rr = w.runs[src_buf] + bs.col, o0 = o[0];
      const uint32_t wd = bs.len / S, rem = bs.len - wd * S, wide = rem * (wd + 1u);
      const uint32_t half = (1u << w.tile_log2) - 1u;
      const uint32_t stream = (uint32_t)rand_at(seed, ((uint64_t)lev << 40) ^ bs.start, 0);
      for (uint32_t t0 = threadIdx.x; t0 < bs.nt; t0 += THREADS * U) {
        uint32_t fs[U], rs_[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
          const uint32_t t = min(t0 + u * THREADS, bs.nt - 1u);
          fs[u] = o[t];
          rs_[u] = rr[t];
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
          const uint32_t t = t0 + u * THREADS, f = fs[u] - o0, c = rs_[u] & 0xFFFFu;
          if (t >= bs.nt || c == 0) continue;
          for (uint32_t i = (uint32_t)(((uint64_t)f + half) >> w.tile_log2); i <= (f + c - 1) >> w.tile_log2; i++)
            w.tile_run[bs.tb + i] = t;
          const uint32_t place = (t << w.tile_log2) + (rs_[u] >> 16) - f;
          uint32_t j = f < wide ? f / (wd + 1u) : rem + (f - wide) / wd;
          for (; j < S; j++) {
            const uint32_t lo = j * wd + min(j, rem);
            if (lo >= f + c) break;
            const uint32_t pos = lo + __umulhi(mix32(stream + j * 0x9E3779B9u), wd + (j < rem ? 1u : 0u));
            if (pos >= f && pos < f + c) s_v[j] = place + pos;
          }
        }
      }
      __syncthreads();
    }
    K k[ITEMS];
    uint32_t v[ITEMS], p[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
      const uint32_t j = threadIdx.x * ITEMS + i;
      if (SRC_IN && staged && j < S) {
        // drawn by k_start_plain (the same positions), stored in order
        BufView<K, false>{w.buf_rec[1]}.get(j, k[i], v[i], p[i]);
      } else if (j < S) {
        if constexpr (SRC_IN) {
          const uint64_t r = rand_at(seed, ((uint64_t)lev << 40) ^ bs.start, j);
          const uint32_t off = (uint32_t)(((r >> 32) * (uint64_t)bs.len) >> 32);
          k[i] = in_keys[bs.start + off];  // raw bits; mapped below once all loads are issued
          v[i] = (uint32_t)(bs.start + off - bs.ubase);
        } else {
          bv.get(bs.pstart + s_v[j], k[i], v[i], p[i]);
        }
      } else {
        k[i] = KMax<K>::v;
        v[i] = kPadIdx;
      }
      p[i] = 0;
    }
    if constexpr (SRC_IN && F32) {
#pragma unroll
      for (int i = 0; i < ITEMS; i++)
        if (threadIdx.x * ITEMS + i < S) k[i] = ord_of<K, F32>(k[i]);
    }
    const uint32_t kk = 1u << bs.logk;
    // The splitters are the samples of rank j * ae - 1 (j = 1 .. kk - 1) in
    // (key, position) order.  Ranks come from bins:
    // samples are counted into bins by the top bits of (key - min) (or, for a
    // narrow key range, key offset then position bits), and a sample's rank
    // is its bin's start plus the number of smaller samples in its bin.  If
    // that would cost more than kSplRankBudget compares per sample, the samples
    // are merge sorted instead.  As many bins as samples: the compares are a
    // serial chain per thread and the ranking's bound, so bins are small and
    // read four samples at a time (from an eighth of the bins, a sample at a
    // time: first and second level of 2^26 gaussian f32 38 + 63 -> 25 + 49 us,
    // of 2^28 u64 30 + 134 -> 20 + 120, of 2^25 u64 with duplicates 11 + 58 ->
    // 11 + 30; what is left of the second level is the samples' loads).
    bool ranked = false;
    {
      K kmn = KMax<K>::v, kmx = K(0);
      uint32_t imn = ~0u, imx = 0u;
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        if (threadIdx.x * ITEMS + i < S) {
          kmn = k[i] < kmn ? k[i] : kmn;
          kmx = k[i] > kmx ? k[i] : kmx;
          imn = min(imn, v[i]);
          imx = max(imx, v[i]);
        }
      }
      for (int b = threadIdx.x; b <= (1 << LB); b += THREADS) s_bin[b] = 0;
      if (threadIdx.x == 0) s_cost = 0;
      const Range4 br = block_range<K, THREADS>(kmn, kmx, imn, imx, s_red, threadIdx.x);
      kmn = (K)br.kmn;
      const uint64_t kr = (uint64_t)((K)br.kmx - kmn);
      const int rb = kr ? 64 - __clzll((long long)kr) : 0;
      BinMap bm;
      const bool narrow = rb < LB;  // bins: key offset, then the top bits of the position
      if (narrow) {
        const uint32_t ib = LB - rb, ir = br.imx - br.imn;
        const int ibits = ir ? 32 - __clz(ir) : 0;
        bm = BinMap{(uint64_t)br.imn, 32u, ib, (uint32_t)max(ibits - (int)ib, 0), (1u << ib) - 1u};
      } else {
        bm = BinMap{0ull, (uint32_t)(rb - LB), 0u, 0u, 0u};
      }
      auto bin_of = [&](K key, uint32_t idx) -> uint32_t {
        const uint64_t off = (uint64_t)(K)(key - kmn);
        return bm(narrow ? (off << 32) | idx : off);
      };
      uint32_t r[ITEMS];
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        r[i] = 0;
        if (threadIdx.x * ITEMS + i < S) r[i] = atomicAdd(&s_bin[bin_of(k[i], v[i])], 1u);
      }
      __syncthreads();
      {  // the bins' starts and the sum of their squared sizes
        uint32_t x[PL], sum = 0, sq = 0;
#pragma unroll
        for (int q = 0; q < PL; q++) {
          x[q] = s_bin[threadIdx.x * PL + q];
          sum += x[q];
          sq += x[q] * x[q];
        }
        sq = lane_u32(wave_incl_scan_dpp(sq), kWave - 1);
        if (lane_id() == 0 && sq) atomicAdd(&s_cost, sq);
        uint32_t tot, b = block_excl_scan<THREADS>(sum, s_tmp, &tot);
#pragma unroll
        for (int q = 0; q < PL; q++) {
          s_bin[threadIdx.x * PL + q] = b;
          b += x[q];
        }
        if (threadIdx.x == 0) s_bin[1 << LB] = S;
      }
      __syncthreads();
      if (s_cost <= kSplRankBudget * S) {  // uniform
        ranked = true;
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
          if (threadIdx.x * ITEMS + i < S) sa.put(s_bin[bin_of(k[i], v[i])] + r[i], k[i], v[i]);
        }
        __syncthreads();
        constexpr uint32_t U = 4;  // samples of a bin read at a time
        for (uint32_t pq = threadIdx.x; pq < S; pq += THREADS) {
          const K key = sa.key(pq);
          const uint32_t idx = s_v[pq];
          const uint32_t db = bin_of(key, idx);
          const uint32_t s0 = s_bin[db], s1 = s_bin[db + 1];
          // samples are drawn with replacement: equal samples are ranked by
          // their place in the bin, so that every rank is taken once
          uint32_t less = 0;
          for (uint32_t q = s0; q < s1; q += U) {
            K kq[U];
            uint32_t iq[U];
#pragma unroll
            for (uint32_t u = 0; u < U; u++) {
              kq[u] = sa.key(min(q + u, s1 - 1u));
              iq[u] = s_v[min(q + u, s1 - 1u)];
            }
#pragma unroll
            for (uint32_t u = 0; u < U; u++) {
              const bool below = (kq[u] < key) | ((kq[u] == key) & ((iq[u] < idx) | ((iq[u] == idx) & (q + u < pq))));
              less += (q + u < s1) & below ? 1u : 0u;
            }
          }
          const uint32_t rank = s0 + less;
          if ((rank + 1) % ae == 0) {
            const uint32_t j = (rank + 1) / ae;
            if (j < kk) {
              const uint32_t node = (j | kk) >> (__builtin_ctz(j) + 1);
              tkey[(uint64_t)s * kMaxK + node] = key;
              w.tree_idx[(uint64_t)s * kMaxK + node] = idx;
              if (lev == 0 && s == 0) {
                w.ctl->l0_spl_key[j - 1] = (uint64_t)key;
                w.ctl->l0_spl_pos[j - 1] = idx;
              }
            }
          }
        }
      }
    }
    if (!ranked) {
      lds_merge_sort<K, THREADS, ITEMS, false>(k, v, p, sa);
#pragma unroll
      for (int i = 0; i < ITEMS; i++) sa.put(lpad(threadIdx.x * ITEMS + i), k[i], v[i]);
      __syncthreads();
      for (uint32_t node = threadIdx.x + 1; node < kk; node += THREADS) {
        const uint32_t d = 31u - __clz(node);
        const uint32_t q = node - (1u << d);
        const uint32_t j = (2u * q + 1u) << (bs.logk - 1u - d);
        const uint32_t r = j * ae - 1u;
        tkey[(uint64_t)s * kMaxK + node] = sa.key(lpad(r));
        w.tree_idx[(uint64_t)s * kMaxK + node] = s_v[lpad(r)];
      }
      if (lev == 0 && s == 0) {
        for (uint32_t j = threadIdx.x + 1; j < kk; j += THREADS) {
          w.ctl->l0_spl_key[j - 1] = (uint64_t)sa.key(lpad(j * ae - 1u));
          w.ctl->l0_spl_pos[j - 1] = s_v[lpad(j * ae - 1u)];
        }
      }
    }
    if (lev == 0 && s == 0 && threadIdx.x == 0) w.ctl->l0_k = kk;
    __syncthreads();
    if (SRC_IN && m == 1 && bs.len >= kTiledMin) {  // uniform
      const uint32_t j = threadIdx.x;
      const int rep =
          __syncthreads_or(j > 0 && j + 1 < kk && w.ctl->l0_spl_key[j] == w.ctl->l0_spl_key[j - 1]);
      if (j == 0) w.ctl->l0_repeats = rep != 0;
    }
  }
}

// ---------------------------------------------------------------------------
// Classification of a thread's ITEMS elements with the splitter tree in LDS.
// tk holds 2k entries: node t of the implicit tree (t in [1, k)) at tk[t],
// and below them a leaf row, tk[k + b] = the b-th smallest splitter key for
// b < k - 1 and tk[2k - 1] = the largest (see tree_to_lds).  ti holds the
// positions of the tree nodes.  Levels are the outer loop so the ITEMS
// lookups of a level are independent.  The descent compares keys only and
// walks byte offsets into tk (one shift-add per level, no index scaling).
// It ends at the leaf k + b where b is the number of splitter keys strictly
// below the key, so the key can only equal a splitter key on its path if it
// equals that leaf's (the smallest splitter key >= key; the last leaf repeats
// the largest splitter key, which a key in bucket k - 1 exceeds).  Such an
// element is classified again comparing (key, position) pairs (the tie-break
// of Appendix G: positions are looked at only when keys are equal).  `pairs`
// (uniform over the wave, kept by the caller across tiles) skips the key-only
// descent for a tile after one in which every element of the wave tied, as
// on inputs of few distinct keys.
// Result: bucket = number of splitters strictly below (key, position).
template <typename K, int ITEMS, typename IdxFn>
__device__ __forceinline__ void classify_batch(const K* tk, const uint32_t* ti, uint32_t logk, const K (&key)[ITEMS],
                                               const bool (&valid)[ITEMS], IdxFn idx_of, uint32_t (&b)[ITEMS],
                                               bool& pairs) {
  constexpr uint32_t KB = (uint32_t)sizeof(K);
  const uint32_t kk = 1u << logk;
  // level-major descent comparing (key, position) for the elements in m
  auto pair_descent = [&](const bool (&m)[ITEMS], uint32_t (&q)[ITEMS]) {
    uint32_t id[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
      id[i] = m[i] ? idx_of(i) : 0u;  // positions first (independent loads)
      q[i] = 1;
    }
    for (uint32_t l = 0; l < logk; l++) {
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        const K t = tk[q[i]];
        const uint32_t u = ti[q[i]];
        q[i] = 2u * q[i] + ((key[i] > t) | ((key[i] == t) & (id[i] > u)) ? 1u : 0u);
      }
    }
  };
  uint32_t j[ITEMS];
  if (pairs) {  // uniform
    // every element of this wave's previous tile tied: the (key, position)
    // descent alone gives the bucket.  A splitter key equals the key exactly
    // when one of the two splitters around the result does (the leaf row
    // holds them), which decides the mode of the next tile.
    pair_descent(valid, j);
    bool untied = false;
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
      const bool t = key[i] == tk[j[i]] || (j[i] > kk && key[i] == tk[j[i] - 1]);
      untied = untied | (valid[i] & !t);
    }
    pairs = !__any(untied);
  } else {
    // the current node's LDS address; twice it, less the tree's (once) and
    // plus a node's size for the right child, is the child's: no addition of
    // the tree's base per step (with the ranks below, the second level of 2^28
    // u64 keys, bound by its vector instructions: 1869 -> 1806 us)
    const uint32_t tb = uniform(lds_address(tk)), left = 0u - tb, right = KB - tb;
    uint32_t a[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; i++) a[i] = tb + KB;
    for (uint32_t l = 0; l < logk; l++) {
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        const K t = lds_at<K>(a[i]);
        a[i] = 2u * a[i] + (key[i] > t ? right : left);
      }
    }
    K leaf[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; i++) leaf[i] = lds_at<K>(a[i]);
    bool eq[ITEMS];
    bool tie = false, untied = false;
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
      eq[i] = (key[i] == leaf[i]) & valid[i];
      tie = tie | eq[i];
      untied = untied | (valid[i] & !eq[i]);
      j[i] = (a[i] - tb) / KB;
    }
    if (__any(tie)) {
      uint32_t q[ITEMS];
      pair_descent(eq, q);
#pragma unroll
      for (int i = 0; i < ITEMS; i++) j[i] = eq[i] ? q[i] : j[i];
    }
    pairs = !__any(untied);
  }
#pragma unroll
  for (int i = 0; i < ITEMS; i++) b[i] = j[i] - kk;
}

// Classification of a tile whose splitters lie in order of (key, position)
// all before or all after its elements' positions wherever keys are equal
// (see TileTree): u holds at node t the least key that goes right.
template <typename K, int ITEMS>
__device__ __forceinline__ void classify_tile(const K* u, uint32_t logk, const K (&key)[ITEMS], uint32_t (&b)[ITEMS]) {
  constexpr uint32_t KB = (uint32_t)sizeof(K);
  const uint32_t ub = uniform(lds_address(u)), left = 0u - ub, right = KB - ub;
  uint32_t a[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; i++) a[i] = ub + KB;
  for (uint32_t l = 0; l < logk; l++) {
#pragma unroll
    for (int i = 0; i < ITEMS; i++) {
      const K t = lds_at<K>(a[i]);
      a[i] = 2u * a[i] + (key[i] >= t ? right : left);
    }
  }
#pragma unroll
  for (int i = 0; i < ITEMS; i++) b[i] = (a[i] - ub) / KB - (1u << logk);
}

// The elements of an input tile have consecutive positions p0 .. last, and a
// splitter's position is seldom among them: then "(key, position) above the
// splitter (t, q)" is "key >= t" for the whole tile if q < p0 and "key >= t +
// 1" if q >= last, and ties need no positions.  set() writes the tree of such
// thresholds; flags gets kBuilt, and kInside if one threshold does not exist.
// First level of 2^28 u64 keys, all equal 1470 -> 1124 us, of 16 values
// 1882 -> 1498.
template <typename K>
struct TileTree {
  static constexpr uint32_t kBuilt = 1, kInside = 2;
  // Thread i of at least k.
  static __device__ __forceinline__ void set(const K* tk, const uint32_t* ti, uint32_t logk, uint32_t i, uint32_t p0,
                                             uint32_t last, K* u, uint32_t* flags) {
    const bool node = i > 0 && i < (1u << logk);
    const K t = node ? tk[i] : K(0);
    const uint32_t q = node ? ti[i] : 0u;
    if (node) u[i] = q < p0 ? t : t + 1;
    const bool inside = node && q >= p0 && (q < last || t == KMax<K>::v);
    const uint32_t f = (i == 0 ? kBuilt : 0u) | (__any(inside) ? kInside : 0u);
    if (f && lane_id() == 0) atomicOr(flags, f);
  }
};

// Splitter tree of a segment (2^logk buckets): nodes tk[1, k) / ti[1, k) and
// the leaf row tk[k, 2k) (see classify_batch); splitter j (1-based, in sorted
// order) is tree node (j | k) >> (ctz(j) + 1).  A thread's part of the copy
// from global memory, at least kMaxK threads: fetch, then store.
template <typename K>
struct TreePart {
  K node, leaf;
  uint32_t pos;
  __device__ __forceinline__ void fetch(const Work& w, uint32_t s, uint32_t logk, uint32_t i) {
    const K* tkey = (const K*)w.tree_key;
    const uint32_t kk = 1u << logk;
    const uint64_t o = (uint64_t)s * kMaxK;
    node = leaf = K(0);
    pos = 0;
    if (i >= kk) return;
    const uint32_t j = i ? i : kk - 1;  // thread 0: the last leaf repeats the largest
    leaf = tkey[o + ((j | kk) >> (__builtin_ctz(j) + 1))];
    if (i) {
      node = tkey[o + i];
      pos = w.tree_idx[o + i];
    }
  }
  __device__ __forceinline__ void store(uint32_t logk, uint32_t i, K* tk, uint32_t* ti) const {
    const uint32_t kk = 1u << logk;
    if (i >= kk) return;
    tk[i ? kk + i - 1 : 2 * kk - 1] = leaf;
    if (i) {
      tk[i] = node;
      ti[i] = pos;
    }
  }
};

// ---------------------------------------------------------------------------
// Exclusive scan of a level's run lengths into offs in one launch: a chained
// scan with decoupled look-back.  Workgroups take chunks of run lengths in
// order from a counter; each publishes its chunk's sum at once and, after
// looking back at its predecessors' published sums (or inclusive prefixes),
// its inclusive prefix.  The first wave looks back, at 64 predecessors at a
// time: by one thread, a predecessor at a time, the scan of a 2^20-key sort
// took 9.3 us and larger ones were better off in three launches.  A status
// word holds all that is passed on (flag << 32 | value, flag 1 = the chunk's
// sum, 2 = the inclusive prefix through the chunk; zeroed before each level),
// so relaxed loads and stores do.  A chunk's predecessors are held by
// workgroups that are already running, so every wait ends; the wait is bounded
// all the same (status set to an internal error after kScanSpinMax polls).
// Sums are taken modulo 2^32: offsets are only ever subtracted from offsets of
// the same segment, which is shorter than 2^32.
// Chunks: 16 run lengths per thread of 256 threads, or of 1024 for matrices of
// more than 2^21 entries (two of 2^23: 74 instead of 109 us; one of 2^17 entries:
// 7.7 instead of 5.5 us).
constexpr int kScanItems = 16, kScanChunk = 256 * kScanItems;  // (the smallest)
constexpr uint32_t kScanSpinMax = 1u << 26;

template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_scan(Work w, int lev) {
  constexpr uint32_t CHUNK = THREADS * kScanItems;
  __shared__ uint32_t tmp[THREADS / kWave + 1];
  __shared__ uint32_t s_chunk, s_prefix;
  const uint32_t M = w.ctl->entries[lev & 1];
  const uint32_t *const runs = w.runs[lev & 1], len_mask = 0xFFFFu;
  uint32_t* const offs = w.offs[lev & 1];
  const uint32_t nb = (M + CHUNK - 1) / CHUNK;
  // as many workgroups as chunks take part (the others would only queue for
  // the chunk counter, at about 10 ns each)
  if (blockIdx.x >= nb) return;
  for (;;) {
    if (threadIdx.x == 0) s_chunk = atomicAdd(&w.ctl->scan_next, 1u);
    __syncthreads();
    const uint32_t c = s_chunk;
    if (c >= nb) break;
    const uint32_t b0 = c * CHUNK + threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
#pragma unroll
    for (int q = 0; q < kScanItems / 4; q++) {
      const uint32_t j = b0 + 4 * q;
      if (j + 4 <= M) {
        const uint4 x = *reinterpret_cast<const uint4*>(runs + j);  // j % 4 == 0: 16-byte aligned
        v[4 * q] = x.x & len_mask;
        v[4 * q + 1] = x.y & len_mask;
        v[4 * q + 2] = x.z & len_mask;
        v[4 * q + 3] = x.w & len_mask;
      } else {
#pragma unroll
        for (int r = 0; r < 4; r++) v[4 * q + r] = j + r < M ? runs[j + r] & len_mask : 0u;
      }
    }
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; i++) sum += v[i];
    uint32_t tot;
    uint32_t e = block_excl_scan<THREADS>(sum, tmp, &tot);
    if (threadIdx.x < kWave) {  // the first wave
      const uint32_t lane = threadIdx.x;
      auto publish = [&](uint64_t flag, uint32_t v) {
        if (lane == 0)
          __hip_atomic_store(&w.scan_flags[c], (flag << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      uint32_t prefix = 0, spins = 0;
      if (c > 0) {
        publish(1, tot);
        for (uint32_t end = c;;) {  // lane l looks at chunk end - 1 - l; below chunk 0 lies the prefix 0
          const uint64_t s = lane < end ? __hip_atomic_load(&w.scan_flags[end - 1 - lane], __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT)
                                        : 2ull << 32;
          const uint32_t flag = (uint32_t)(s >> 32);
          const uint64_t done = __ballot(flag == 2);
          // lanes up to the nearest prefix, whose values are added up
          const uint64_t need = done ? (done & (0ull - done)) * 2 - 1 : ~0ull;
          if (__ballot(flag == 0) & need) {  // one of them is not published yet
            if (++spins > kScanSpinMax) {
              if (lane == 0) set_status(w.ctl, -3);
              break;
            }
            __builtin_amdgcn_s_sleep(1);
            continue;
          }
          prefix += lane_u32(wave_incl_scan_dpp((need >> lane) & 1ull ? (uint32_t)s : 0u), kWave - 1);
          if (done) break;
          end -= kWave;
        }
      }
      publish(2, prefix + tot);
      if (lane == 0) s_prefix = prefix;
    }
    __syncthreads();
    e += s_prefix;
#pragma unroll
    for (int i = 0; i < kScanItems; i++) {
      const uint32_t x = v[i];
      v[i] = e;
      e += x;
    }
#pragma unroll
    for (int q = 0; q < kScanItems / 4; q++) {
      const uint32_t j = b0 + 4 * q;
      if (j + 4 <= M) {
        *reinterpret_cast<uint4*>(offs + j) = make_uint4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
      } else {
#pragma unroll
        for (int r = 0; r < 4; r++)
          if (j + r < M) offs[j + r] = v[4 * q + r];
      }
    }
    __syncthreads();  // s_chunk / s_prefix are rewritten next
  }
}

// ---------------------------------------------------------------------------
// Split: one tile at a time, classify, rank inside (tile, bucket), stage by
// bucket in LDS and write the tile back as one contiguous piece, with each
// bucket's run (its start in the tile and length) into the level's matrix.
//
// Tiles are dealt out so that the workgroups of an XCD (dispatch is
// round-robin over the 8 XCDs) work on consecutive tiles: their entries of a
// matrix row are then written through one L2, and they share the segment's
// splitter tree and, on a buffer level, neighbouring runs.
//
// The next tile's elements are loaded once this tile's are staged (into the
// same registers) and arrive while it is written out; on a buffer level their
// places come from a RunMap that is built between this tile's barriers.  The
// tile after that has its segment's descriptor loaded meanwhile, and a new
// segment's splitter tree is fetched a tile ahead.  All LDS that a tile's
// first phase writes is kept twice, so that no barrier closes the loop (one
// tree only where two do not fit, with its load and a barrier exposed).
// With TILED, an input tile's keys are classified by a TileTree.  That form is
// a kernel of its own because a branch on it in the loop costs other inputs
// 3 % of the launch, and is launched beside the ordinary one (`both`): the one
// that does not suit the tree returns at once.
template <typename K, bool F32, bool SRC_IN, bool PAY, int THREADS, int ITEMS, bool TILED = false>
__global__ __launch_bounds__(THREADS) void k_split(Work w, int lev, const K* in_keys, const uint32_t* in_pay,
                                                   int src_buf, int dst_buf, int both) {
  using View = BufView<K, PAY>;
  constexpr uint32_t TILE = THREADS * ITEMS;
  constexpr int W = View::W;
  constexpr int MAPS = SRC_IN ? 1 : 2;
  using Map = RunMap<SRC_IN ? kWave : THREADS, SRC_IN ? kWave : (int)TILE>;
  static_assert(THREADS >= kMaxK, "one histogram bin per thread");
  static_assert(TILE <= (1u << 14), "run starts, lengths and ranks fit 16 bits");
  constexpr int TREES = SRC_IN || W < 4 ? 2 : 1;
  __shared__ K tk[TREES][2 * kMaxK];
  __shared__ uint32_t ti[TREES][kMaxK];
  __shared__ K tile_tree[TILED ? kMaxK : 1];
  __shared__ uint32_t tile_flags[2];
  __shared__ uint32_t hist[2][kMaxK];
  __shared__ uint32_t tmp[THREADS / kWave + 1];
  __shared__ Map map[MAPS];
  __shared__ __align__(16) uint32_t stage[TILE * W];

  if (SRC_IN && both && (w.ctl->l0_repeats != 0) != TILED) return;
  const int cur = lev & 1;
  const uint32_t m = (uint32_t)min((uint64_t)w.ctl->big_count[cur], w.big_max);
  const uint32_t G = w.ctl->tiles[cur];
  {  // for this level's scan and the next level's lists
    const uint32_t nb = (w.ctl->entries[cur] + kScanChunk - 1) / kScanChunk;
    for (uint32_t i = blockIdx.x * THREADS + threadIdx.x; i < nb; i += gridDim.x * THREADS) w.scan_flags[i] = 0ull;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      w.ctl->scan_next = 0;
      w.ctl->big_count[cur ^ 1] = 0;
      w.ctl->tiles[cur ^ 1] = 0;
      w.ctl->entries[cur ^ 1] = 0;
    }
  }
  // the XCD's share of the tiles, dealt to its workgroups in turn
  const uint32_t x = blockIdx.x & 7u, step = gridDim.x >> 3;
  const uint32_t hi = (uint32_t)(((uint64_t)G * (x + 1)) >> 3);
  uint32_t g = (uint32_t)(((uint64_t)G * x) >> 3) + (blockIdx.x >> 3);
  if (g >= hi) return;

  const int t = threadIdx.x;
  for (int i = t; i < 2 * kMaxK; i += THREADS) (&hist[0][0])[i] = 0;
  auto seg_of = [&](uint32_t gg) -> uint32_t { return m == 1 ? 0u : uniform(w.tile_seg[gg]); };
  const uint32_t* const runs_in = SRC_IN ? nullptr : w.runs[src_buf];
  const uint32_t* const offs_in = SRC_IN ? nullptr : w.offs[src_buf];
  uint32_t* const runs_out = w.runs[cur];
  K key[ITEMS];
  uint32_t idx[ITEMS], pay[ITEMS];
  // a buffer level's run of this thread for the tile to be loaded
  struct Run {
    uint32_t run, ofs, e, c;
  };
  auto run_of = [&](const BigSeg& b, uint32_t first) -> Run {
    Run r{first + (uint32_t)t, 0u, 0u, 0u};
    if (r.run < b.nt) {
      const uint32_t v = runs_in[b.col + r.run];
      r.ofs = offs_in[b.col + r.run] - offs_in[b.col];
      r.e = v >> 16;
      r.c = v & 0xFFFFu;
    }
    return r;
  };
  auto load = [&](const BigSeg& b, uint32_t tl, const Map& mp) {
    const uint32_t cnt = min(TILE, b.len - tl * TILE);
    if constexpr (SRC_IN) {
      const uint64_t base = b.start + (uint64_t)tl * TILE;
      const K* const kin = in_keys + base;
      const uint32_t ib = (uint32_t)(base - b.ubase);
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        const uint32_t p = min((uint32_t)(i * THREADS + t), cnt - 1u);
        key[i] = at32(kin, p);  // raw bits: mapped when the tile is used, so the loads are not waited for
        idx[i] = ib + p;
        if constexpr (PAY) pay[i] = at32(in_pay + base, p);
      }
    } else {
      const View bv{w.buf_rec[src_buf] + b.pstart * W};
      if (mp.over != 0) {  // uniform
#pragma unroll
        for (int i = 0; i < ITEMS; i++) {
          const uint32_t p = min((uint32_t)(i * THREADS + t), cnt - 1u);
          bv.get(locate(w, src_buf, b.col, 0, b.nt - 1, tl * TILE + p), key[i], idx[i], pay[i]);
        }
      } else if (((uint64_t)b.nt << w.tile_log2) * (4 * W) <= 0xFFFFFFFFull) {  // uniform: 32-bit offsets do
        mp.each(t, cnt, [&](int i, uint32_t d) { bv.get32(d, key[i], idx[i], pay[i]); });
      } else {
        mp.each(t, cnt, [&](int i, uint32_t d) { bv.get(d, key[i], idx[i], pay[i]); });
      }
    }
  };
  auto uniform_seg = [](const BigSeg& b) -> BigSeg {
    return BigSeg{uniform64(b.start), uniform64(b.ubase), uniform64(b.pstart), uniform(b.len), uniform(b.logk),
                  uniform(b.col),     uniform(b.nt),      uniform(b.tb),       uniform(b.cb)};
  };

  uint32_t s = seg_of(g);
  BigSeg bs = uniform_seg(w.big[cur][s]);
  TreePart<K> tree;
  tree.fetch(w, s, bs.logk, t);
  tree.store(bs.logk, t, tk[0], ti[0]);
  if constexpr (TILED) {
    if (t < 2) tile_flags[t] = 0;
    __syncthreads();
  }
  auto tile_thresholds = [&](uint32_t tl, int at) {
    const uint32_t p0 = (uint32_t)(bs.start - bs.ubase) + tl * TILE;
    if (t < kMaxK)
      TileTree<K>::set(tk[0], ti[0], bs.logk, t, p0, p0 + min(TILE, bs.len - tl * TILE) - 1u, tile_tree,
                       &tile_flags[at]);
  };
  if constexpr (TILED) tile_thresholds(g - bs.tb, 0);
  int par = 0, tp = 0;
  if constexpr (!SRC_IN) {
    const Run r = run_of(bs, uniform(w.tile_run[g]));
    const uint32_t j0 = (g - bs.tb) * TILE, cnt = min(TILE, bs.len - j0);
    uint64_t bal;
    map[0].clear(t);
    __syncthreads();
    map[0].mark(t, r.run, bs.nt, r.ofs, r.c, j0, cnt, bal);
    __syncthreads();
    map[0].number(t, r.run, r.ofs, r.e, j0, w.tile_log2, bal);
  }
  // the next tile's segment and first run
  uint32_t sn = s, first = 0;
  BigSeg bn = bs;
  if (g + step < hi) {
    sn = seg_of(g + step);
    if (m > 1) bn = uniform_seg(w.big[cur][sn]);
    if constexpr (!SRC_IN) first = uniform(w.tile_run[g + step]);
  }
  __syncthreads();
  load(bs, g - bs.tb, map[0]);
  bool pairs = false;  // classification mode of this wave's next tile
  for (;;) {
    const uint32_t tl = g - bs.tb, cnt = min(TILE, bs.len - tl * TILE), kk = 1u << bs.logk;
    uint32_t* const h = hist[par];
    const uint32_t gn = g + step, g2 = gn + step;
    const bool more = gn < hi, more2 = g2 < hi;
    // on their way while this tile is classified: the next tile's runs and, if
    // it is of another segment, tree; the segment of the tile after that
    Run rn{0u, 0u, 0u, 0u};
    uint32_t j0 = 0, cn = 0;
    if constexpr (!SRC_IN) {
      if (more) {
        rn = run_of(bn, first);
        j0 = (gn - bn.tb) * TILE;
        cn = min(TILE, bn.len - j0);
      }
    }
    const bool new_tree = sn != s;  // uniform
    if (TREES == 2 && new_tree) tree.fetch(w, sn, bn.logk, t);
    uint32_t s2 = sn, first2 = 0;
    if (more2) {
      if (m > 1) s2 = w.tile_seg[g2];
      if constexpr (!SRC_IN) first2 = w.tile_run[g2];
    }
    if constexpr (!SRC_IN) map[(par ^ 1) & (MAPS - 1)].clear(t);
    if (t < kMaxK) hist[par ^ 1][t] = 0;
    bool valid[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; i++) valid[i] = t < (int)cnt - i * THREADS;
    if constexpr (SRC_IN && F32) {
#pragma unroll
      for (int i = 0; i < ITEMS; i++) key[i] = ord_of<K, F32>(key[i]);
    }
    uint32_t pos[ITEMS];  // bucket, then place in the staged tile
    if (TILED && tile_flags[par] == TileTree<K>::kBuilt)  // uniform
      classify_tile<K, ITEMS>(tile_tree, bs.logk, key, pos);
    else
      classify_batch<K, ITEMS>(tk[tp], ti[tp], bs.logk, key, valid, [&](int i) -> uint32_t { return idx[i]; }, pos,
                               pairs);
    // rank inside (tile, bucket): one LDS atomic per element; where the
    // wave's first 64 elements all fall into one bucket (skewed inputs), it
    // looks for one bucket among each 64 and takes one atomic for them.  A
    // wave's valid elements are a prefix of its lanes, so lane 0 holds one
    // whenever any lane does.
    const uint32_t lane = lane_id();
    if (__ballot(valid[0] && pos[0] != uniform(pos[0])) != 0) {
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        uint32_t r = 0;
        if (valid[i]) r = atomicAdd(&h[pos[i]], 1u);
        pos[i] = (pos[i] << 18) | r;  // 4 * bucket << 16, r < TILE
      }
    } else {
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        const uint32_t b0 = uniform(pos[i]);
        uint32_t r = 0;
        if (__ballot(valid[i] && pos[i] != b0) == 0) {
          const uint64_t act = __ballot(valid[i]);
          uint32_t basev = 0;
          if (lane == 0 && act) basev = atomicAdd(&h[b0], (uint32_t)__popcll(act));
          r = uniform(basev) + (uint32_t)__popcll(act & ((1ull << lane) - 1ull));
        } else if (valid[i]) {
          r = atomicAdd(&h[pos[i]], 1u);
        }
        pos[i] = (pos[i] << 18) | r;
      }
    }
    // the next tile's runs are touched line by line, so that their elements
    // come from the L2 when they are loaded, after this tile is staged (second
    // level of 2^28 u64 keys: 2034 -> 1901 us)
    constexpr int TOUCH = SRC_IN ? 1 : 5;
    uint32_t touched[TOUCH];
    if constexpr (!SRC_IN) {
      const bool in = rn.c > 0 && rn.ofs < j0 + cn && rn.ofs + rn.c > j0;
      const uint32_t bytes = in ? rn.c * (4 * W) : 4u;
      const char* line = reinterpret_cast<const char*>(w.buf_rec[src_buf] +
                                                       (bn.pstart + (in ? (rn.run << w.tile_log2) + rn.e : 0u)) * W);
#pragma unroll
      for (int k = 0; k < TOUCH; k++)
        touched[k] = *reinterpret_cast<const uint32_t*>(line + min((uint32_t)k * 128u, bytes - 4u));
    }
    s2 = uniform(s2);
    BigSeg b2 = bn;
    if (m > 1) b2 = w.big[cur][s2];
    if (TREES == 2 && new_tree) tree.store(bn.logk, t, tk[(tp ^ 1) & (TREES - 1)], ti[(tp ^ 1) & (TREES - 1)]);
    __syncthreads();
    if constexpr (TILED) {  // every wave has classified this tile
      if (more) tile_thresholds(gn - bs.tb, par ^ 1);
      if (t == 0) tile_flags[par] = 0;  // (for the tile after the next)
    }
    // exclusive scan of the tile histogram -> tile-local bucket starts
    const uint32_t hv = t < (int)kk ? h[t] : 0u;
    const uint32_t inc = wave_incl_scan_dpp(hv);
    if (t < kMaxK && lane == kWave - 1) tmp[t / kWave] = inc;
    uint64_t bal = 0;
    if constexpr (!SRC_IN) {
      if (more) map[par ^ 1].mark(t, rn.run, bn.nt, rn.ofs, rn.c, j0, cn, bal);
    }
    __syncthreads();
    if (t < kMaxK) {
      uint32_t ex = inc - hv;
      for (int q = 0; q < t / kWave; q++) ex += tmp[q];
      h[t] = ex;
      if (t < (int)kk) runs_out[bs.cb + t * tiles_of(w, bs.len) + tl] = (ex << 16) | hv;
    }
    if constexpr (!SRC_IN) {
      if (more) map[par ^ 1].number(t, rn.run, rn.ofs, rn.e, j0, w.tile_log2, bal);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; i++) pos[i] = at32(h, pos[i] >> 18) + (pos[i] & 0xFFFFu);
#pragma unroll
    for (int i = 0; i < ITEMS; i++)
      if (valid[i]) View{stage}.put(pos[i], key[i], idx[i], pay[i]);
    if constexpr (!SRC_IN) {
#pragma unroll
      for (int k = 0; k < TOUCH; k++) asm volatile("" ::"v"(touched[k]));
    }
    if (more) load(bn, gn - bn.tb, map[(par ^ 1) & (MAPS - 1)]);
    __syncthreads();
    // the tile, as it lies
    {
      uint32_t* const out = w.buf_rec[dst_buf] + (bs.start + (uint64_t)tl * TILE) * W;
      const uint32_t words = cnt * W, quads = words / 4;
      struct __attribute__((aligned(4))) Quad {
        uint32_t x[4];
      };
      for (uint32_t q = t; q < quads; q += THREADS) {
        const uint4 v = reinterpret_cast<const uint4*>(stage)[q];
        at32(reinterpret_cast<Quad*>(out), q) = Quad{{v.x, v.y, v.z, v.w}};
      }
      if (t < (int)(words & 3u)) out[4 * quads + t] = stage[4 * quads + t];
    }
    if (!more) break;
    if (new_tree) {
      if constexpr (TREES == 2) {
        tp ^= 1;
      } else {  // (every wave has classified this tile)
        tree.fetch(w, sn, bn.logk, t);
        tree.store(bn.logk, t, tk[0], ti[0]);
        __syncthreads();
      }
    }
    g = gn;
    s = sn;
    bs = bn;
    sn = s2;
    if (m > 1) bn = uniform_seg(b2);
    first = uniform(first2);
    par ^= 1;
  }
}

// Buckets of the finished level lev: split again or sort in LDS.  A workgroup
// takes WAVES segments of at most 64 buckets at a time, a wave each, or one
// with a thread per bucket.  Bound by the atomics on the lists' counters, a few
// addresses for the whole chip, so a workgroup adds up what it has: 4000
// segments of 16 to 64 buckets, 78 -> 23 us (a workgroup per segment before).
// A workgroup with one segment (every plain sort up to 2^28) does not look at
// its width: 2 us for a load and a barrier.
struct LevelEnd {
  uint32_t cap, target, last, dst_code, ff, left, cmin;
};
constexpr int kRouteThreads = kMaxK;
__global__ __launch_bounds__(kRouteThreads) void k_route(Work w, int lev, LevelEnd a) {
  __shared__ RouteLds L;
  __shared__ uint32_t most, filled;
  const int cur = lev & 1;
  const uint32_t m = (uint32_t)min((uint64_t)w.ctl->big_count[cur], w.big_max);
  if (blockIdx.x >= m) return;
  if (threadIdx.x == 0) most = filled = 0;
  route_lds_init(L);
  const uint32_t* const offs = w.offs[cur];
  const uint32_t wave = threadIdx.x / kWave, lane = lane_id();
  constexpr uint32_t WAVES = kRouteThreads / kWave;
  const uint32_t own = (m - blockIdx.x + gridDim.x - 1) / gridDim.x;  // segments blockIdx.x + q * gridDim.x, q < own
  uint32_t mx = 0, nz = 0;
  for (uint32_t q = 0; q < own;) {
    // the next WAVES segments if all of them have a bucket per lane at most
    const bool narrow = own > 1 && !__syncthreads_or(q + wave < own &&
                                                     w.big[cur][blockIdx.x + (q + wave) * gridDim.x].logk >
                                                         (uint32_t)__builtin_ctz(kWave));
    const uint32_t sq = narrow ? q + wave : q, b = narrow ? lane : threadIdx.x;
    const uint32_t s = blockIdx.x + min(sq, own - 1) * gridDim.x;
    const BigSeg bs = w.big[cur][s];
    const uint32_t kk = 1u << bs.logk, nt = tiles_of(w, bs.len);
    bool active = sq < own && b < kk;
    uint32_t len = 0, lo = 0;
    if (active) {
      const uint32_t seg0 = offs[bs.cb];
      lo = offs[bs.cb + b * nt] - seg0;
      const uint32_t hi = (b + 1 < kk) ? offs[bs.cb + (b + 1) * nt] - seg0 : bs.len;
      len = hi - lo;
      if (lev == 0 && s == 0) w.ctl->l0_bucket[b] = len;
    }
    mx = max(mx, len);
    nz += len ? 1u : 0u;
    active = active && len > 0;
    // (the debug switch for the global-memory sort holds at the last level)
    route(w, L, cur ^ 1, active, len > a.cap && !a.last,
          FinalSeg{bs.start + lo, bs.start, len, a.dst_code, bs.cb + b * nt, nt}, bs.ubase, a.cap, a.last ? a.ff : 0u,
          a.target, a.left, a.cmin);
    __syncthreads();  // L.base is rewritten next
    q += narrow ? WAVES : 1;
  }
  if (lev < kMaxLevels) {  // statistics: the workgroup's, then one atomic each
    for (int d = kWave / 2; d > 0; d >>= 1) {
      mx = max(mx, (uint32_t)__shfl_xor(mx, d, kWave));
      nz += (uint32_t)__shfl_xor(nz, d, kWave);
    }
    if (lane == 0 && nz) {
      atomicMax(&most, mx);
      atomicAdd(&filled, nz);
    }
    __syncthreads();
    if (threadIdx.x == 0 && filled) {
      atomicMax(&w.ctl->level_max[lev], most);
      atomicAdd(&w.ctl->level_buckets[lev], filled);
    }
  }
}

// Before a later level reuses the buffer that holds sorted final segments
// (three levels or more): they leave the lists, counted.
__global__ void k_flush(Ctl* ctl) {
  if (threadIdx.x < (unsigned)kNumClasses) {
    ctl->class_done[threadIdx.x] += ctl->class_count[threadIdx.x];
    ctl->class_count[threadIdx.x] = 0;
  }
  if (threadIdx.x < 2) ctl->pairs_in[threadIdx.x] = 0;
}

// ===========================================================================
// Host side
// ===========================================================================
static Tuning g_tuning;

Tuning& tuning() { return g_tuning; }

static inline uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

// Bucket size the levels aim for: at most half the LDS capacity, so that the
// spread of bucket sizes around it stays below the capacity.
static uint32_t effective_target(const Tuning& t, uint32_t cap) {
  return std::max<uint32_t>(64u, std::min<uint32_t>(t.target, cap / 2));
}

uint32_t plan_levels(uint64_t n, const Tuning& t, uint32_t cap) {
  if (n <= cap) return 0;
  uint32_t L = 0;
  uint64_t reach = effective_target(t, cap);
  while (reach < n) {
    reach <<= kMaxLogK;
    L++;
  }
  L = std::max<uint32_t>(L, 1);
  // extra levels, while every level still gets at least 4 buckets
  uint32_t lq = 0;
  for (uint64_t q = (n + effective_target(t, cap) - 1) / effective_target(t, cap); (1ull << lq) < q;) lq++;
  for (uint32_t e = 0; e < t.extra_levels && 2 * (L + 1) <= lq; e++) L++;
  return std::min<uint32_t>(L, std::min<uint32_t>(t.max_levels, kMaxLevels));
}

uint32_t effective_cap(const Tuning& t, bool pay) {
  uint32_t cap = std::min<uint32_t>(t.cap, pay ? 8192u : 12288u);
  return std::max<uint32_t>(cap, 64u);
}

// Elements per tile: 2^13, or 2^12 where that would leave CUs without a tile
// (or by the tuning's choice).
static uint32_t tile_log2_for(uint64_t n, const Tuning& t) {
  return (t.tile_log2 == 12 || n < (uint64_t)num_cu_cached() * 4 << 13) ? 12u : 13u;
}

// The class that takes every bucket of a single-level plain sort of few
// buckets: the first that holds cap, at most that of 8192 (what is longer goes
// to the next).
static int few_class(uint32_t cap) {
  int c = 0;
  while (c < 7 && h_class_max[c] < cap) c++;
  return c;
}

// Workspace layout: returns total bytes; fills w (pointers relative to base).
size_t layout(int kt, uint64_t n, uint32_t num_segs, bool pay, const Tuning& t, char* base, Work* w,
              uint32_t* levels_out) {
  const uint64_t ks = kt == 1 ? 8 : 4;
  const uint32_t cap = effective_cap(t, pay);
  const uint32_t levels = plan_levels(n, t, cap);
  // segments to split: each longer than cap, and of a level's at most kMaxK
  // per segment of the level before
  uint64_t big_max = levels ? n / (cap + 1) + 1 : 0, most = num_segs;
  for (uint32_t l = 1; l < levels && most < big_max; l++) most *= kMaxK;
  big_max = std::min(big_max, std::max<uint64_t>(most, levels ? 1 : 0));
  const uint32_t tlog = tile_log2_for(n, t);
  const uint64_t tiles_max = levels ? (n >> tlog) + big_max + 1 : 0;
  // matrix entries: tiles * k per segment, at most kMaxK per full tile and, for
  // the partial tile of each segment, its k (2^lq < 2 len / target + 2, see logk_for)
  // (part: a bound of all buckets of a level)
  const uint64_t part = std::min<uint64_t>(big_max * kMaxK, 2 * (n / effective_target(t, cap)) + 4 * big_max);
  const uint64_t count_max = levels ? (n >> tlog) * kMaxK + part + kMaxK : 0;
  const uint64_t scan_blocks = count_max / kScanChunk + 2;
  const uint64_t final_max = (uint64_t)num_segs + (uint64_t)levels * part + 1;
  uint64_t off = 0;
  auto take = [&](uint64_t bytes) {
    uint64_t o = off;
    off = align_up(off + bytes, 256);
    return o;
  };
  const uint64_t o_ctl = take(sizeof(Ctl));
  const uint64_t o_big0 = take(big_max * sizeof(BigSeg));
  const uint64_t o_big1 = take(big_max * sizeof(BigSeg));
  const uint64_t o_tk = take(big_max * kMaxK * ks);
  const uint64_t o_ti = take(big_max * kMaxK * 4);
  uint64_t o_run[2], o_ofs[2];
  for (int b = 0; b < 2; b++) {  // (a second pair from two levels on)
    o_run[b] = take((uint32_t)b < levels ? count_max * 4 : 0);
    o_ofs[b] = take((uint32_t)b < levels ? count_max * 4 : 0);
  }
  const uint64_t o_ts = take(tiles_max * 4);
  const uint64_t o_tr = take(levels >= 2 ? tiles_max * 4 : 0);
  const uint64_t o_par = take(scan_blocks * 8);
  uint64_t o_cls[kNumClasses], cls_cap[kNumClasses];
  for (int c = 0; c < kNumClasses; c++) {
    const uint64_t lo = c == 0 ? 0 : h_class_max[c - 1];
    uint64_t bound = n / (lo + 1) + 1;
    if (c == kNumClasses - 1) bound = n / (std::min<uint64_t>(cap, 64) + 1) + 1;
    // a single-level plain sort of few buckets routes all of them (at most
    // kMaxK, however short) to few_class(cap).  Plain sorts that leave out the
    // classes below 2048 fill no list beyond its bound: a split segment has at
    // most 2 len / target <= len / 2048 buckets, and with those of the levels
    // above (512 at most of the first, 512 for each of the second) they are
    // fewer than n / 1025.
    cls_cap[c] = std::min<uint64_t>(final_max, std::max<uint64_t>(bound, c >= few_class(cap) ? kMaxK + 1 : 0));
    o_cls[c] = take(cls_cap[c] * sizeof(FinalSeg));
  }
  const uint64_t nb = (levels || t.force_fallback) ? n : 0;
  uint64_t o_bk[2];
  for (int b = 0; b < 2; b++) o_bk[b] = take(nb * (ks + 4 + (pay ? 4 : 0)));
  if (w) {
    w->ctl = (Ctl*)(base + o_ctl);
    w->big[0] = (BigSeg*)(base + o_big0);
    w->big[1] = (BigSeg*)(base + o_big1);
    w->tree_key = base + o_tk;
    w->tree_idx = (uint32_t*)(base + o_ti);
    for (int b = 0; b < 2; b++) {
      w->runs[b] = (uint32_t*)(base + o_run[b]);
      w->offs[b] = (uint32_t*)(base + o_ofs[b]);
    }
    w->tile_seg = (uint32_t*)(base + o_ts);
    w->tile_run = (uint32_t*)(base + o_tr);
    w->scan_flags = (uint64_t*)(base + o_par);
    for (int c = 0; c < kNumClasses; c++) {
      w->cls[c] = (FinalSeg*)(base + o_cls[c]);
      w->cls_cap[c] = cls_cap[c];
    }
    for (int b = 0; b < 2; b++) w->buf_rec[b] = (uint32_t*)(base + o_bk[b]);
    w->big_max = big_max;
    w->tiles_max = tiles_max;
    w->tile_log2 = tlog;
    w->spread = t.extra_levels > 0 ? 1u : 0u;
    w->count_max = count_max;
    w->scan_blocks = scan_blocks;
    w->n = n;
  }
  if (levels_out) *levels_out = levels;
  return off;
}

static int g_num_cu = 0;
uint32_t num_cu_cached();
static int num_cu() {
  if (!g_num_cu) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    hipDeviceProp_t p;
    if (hipGetDeviceProperties(&p, dev) == hipSuccess)
      g_num_cu = p.multiProcessorCount;
    else
      g_num_cu = 256;
  }
  return g_num_cu;
}

uint32_t num_cu_cached() { return (uint32_t)num_cu(); }

static inline uint32_t grid_for(uint64_t work, uint32_t per_cu) {
  const uint64_t g = std::min<uint64_t>(work, (uint64_t)num_cu() * per_cu);
  return (uint32_t)std::max<uint64_t>(g, 1);
}




// Algorithm of a size class: RFIS (classes 0 to 2) or RQuick (classes 3 to 5)
// up to the tuning's thresholds, else the ranking in bins.
enum class ClassAlgo { kRank, kRfis, kRquick };
static ClassAlgo class_algo(int c, const Tuning& t) {
  if (h_class_max[c] <= t.rfis_max) return c <= 2 ? ClassAlgo::kRfis : ClassAlgo::kRank;
  if (h_class_max[c] <= t.rquick_max) return c >= 3 && c <= 5 ? ClassAlgo::kRquick : ClassAlgo::kRank;
  return ClassAlgo::kRank;
}

template <typename K, bool F32, bool PAY>
static int enqueue_typed(const void* keys_in, const uint32_t* pay_in, const uint64_t* seg_off, uint32_t num_segs,
                         uint64_t n, void* keys_out, uint32_t* perm_out, uint32_t* pay_out, void* ws,
                         size_t ws_bytes, hipStream_t st) {
  const Tuning t = g_tuning;
  Work w;
  uint32_t levels = 0;
  const size_t need = layout(F32 ? 2 : (sizeof(K) == 8 ? 1 : 0), n, num_segs, PAY, t, (char*)ws, &w, &levels);
  if (ws_bytes < need) return -2;
  const uint32_t cap = effective_cap(t, PAY);
  const uint32_t a = std::min<uint32_t>(std::max<uint32_t>(t.oversample, 1), kMaxOversample);
  const uint32_t ff = t.force_fallback;
  const uint32_t target = effective_target(t, cap);
  const K* kin = (const K*)keys_in;
  K* kout = (K*)keys_out;

  if (!seg_off && levels == 0 && !ff && n <= cap) {
    // the whole input fits one workgroup: one launch, no segment lists
    int c = 0;
    while (n > h_class_max[c]) c++;
    const ClassAlgo al = class_algo(c, t);
    if (al == ClassAlgo::kRfis)
      return launch_rfis_class<K, F32, PAY>(c | kDirect, w, kin, pay_in, kout, perm_out, pay_out, 1, st);
    if (al == ClassAlgo::kRquick)
      return launch_rquick_class<K, F32, PAY>(c | kDirect, w, kin, pay_in, kout, perm_out, pay_out, 1, st);
    if constexpr (!PAY) return launch_direct<K, F32>(w, kin, kout, perm_out, st);
  }
  // A single-level plain sort with at most about two final buckets per CU
  // routes all of them to the largest class group that runs two workgroups
  // per CU (and the class above it), so the local sorts run in one or two
  // launches.  Other plain sorts leave out the classes of at most 1024 keys
  // (three launches, 17 us of a 320 us sort): their buckets are about the
  // target size, whatever the keys, so hardly any is that short.
  uint32_t cmin = 0;
  const bool few = !seg_off && levels == 1 && n <= (uint64_t)target * 2 * num_cu();
  if (few) {
    cmin = (uint32_t)few_class(cap);
  } else if (!seg_off && levels > 0 && target >= 4096 && t.rfis_max <= 64 && t.rquick_max <= 64) {
    cmin = 3;
  }
  // a single-level sort of few buckets is latency-bound on its
  // one-workgroup sample sort: 16 samples per bucket keep its buckets
  // within twice the target while halving that step
  const uint32_t a0 = few ? std::min<uint32_t>(a, 16u) : a;
  // the first level's sample drawn at the start (k_start_plain), room in buffer B
  const int staged = (!seg_off && levels > 0 && n >= (uint64_t)kSplThreads * kSplItems) ? 1 : 0;
  if (!seg_off) {
    RS_LAUNCH(k_start_plain<K>, staged ? (uint32_t)(kSplThreads * kSplItems / kStartThreads) : 1u, kStartThreads,
              st, w, n, cap, target, levels, ff, cmin, kin, a0, t.seed, staged);
  } else {
    RS_LAUNCH(k_reset, 1, 256, st, w.ctl, levels);
    RS_LAUNCH(k_init, grid_for((num_segs + 1023) / 1024, 1), 1024, st, w, seg_off, num_segs, n, cap, target, levels,
              ff, cmin);
  }

  // the local sorts of every final segment listed
  auto local_sorts = [&]() -> int {
    uint32_t ranked = 0;  // classes ranked in bins
    for (int c = (int)cmin; c < kNumClasses - 1; c++) {
      // (a class can only be non-empty if its lower bound is below cap)
      if (c > 0 && h_class_max[c - 1] >= cap) break;
      const ClassAlgo al = class_algo(c, t);
      int rc = 0;
      if (al == ClassAlgo::kRank)
        ranked |= 1u << c;
      else if (al == ClassAlgo::kRfis)
        rc = launch_rfis_class<K, F32, PAY>(c, w, kin, pay_in, kout, perm_out, pay_out, w.cls_cap[c], st);
      else
        rc = launch_rquick_class<K, F32, PAY>(c, w, kin, pay_in, kout, perm_out, pay_out, w.cls_cap[c], st);
      if (rc) return rc;
    }
    return launch_local_ranks<K, F32, PAY>(ranked, w, kin, pay_in, kout, perm_out, pay_out, st);
  };
  for (uint32_t lev = 0; lev < levels; lev++) {
    const int dst = lev & 1;
    const int src = (lev + 1) & 1;  // buffer written by the previous level
    const bool last = lev + 1 == levels;
    const LevelEnd le{cap, target, last ? 1u : 0u, (uint32_t)(dst + 1), ff, levels - lev - 1, cmin};
    const uint32_t gs = grid_for(w.big_max, 1);
    if (lev == 0)
      RS_LAUNCH((k_splitters<K, F32, true, PAY, kSplThreads, kSplItems>), gs, kSplThreads, st, w, (int)lev, kin, src,
                a0, t.seed, staged);
    else
      RS_LAUNCH((k_splitters<K, false, false, PAY, kSplThreads, kSplItems>), gs, kSplThreads, st, w, (int)lev, kin,
                src, a, t.seed, 0);
    if (lev >= 2) {  // the level writes over the buffer and matrices of level lev - 2
      const int rc = local_sorts();
      if (rc) return rc;
      RS_LAUNCH(k_flush, 1, kWave, st, w.ctl);
    }
    // resident-sized grids, multiples of 8 for the XCD-aware walk
    if (w.tile_log2 == 12) {
      const uint32_t g = std::max<uint32_t>(8u, grid_for(w.tiles_max, 2) & ~7u);
      if (lev == 0)
        RS_LAUNCH((k_split<K, F32, true, PAY, 512, 8>), g, 512, st, w, (int)lev, kin, pay_in, src, dst, 0);
      else
        RS_LAUNCH((k_split<K, false, false, PAY, 512, 8>), g, 512, st, w, (int)lev, kin, pay_in, src, dst, 0);
    } else {
      const uint32_t g = std::max<uint32_t>(8u, grid_for(w.tiles_max, 1) & ~7u);
      if (lev == 0) {
        const int both = !PAY && seg_off == nullptr && n >= kTiledMin;
        RS_LAUNCH((k_split<K, F32, true, PAY, 1024, 8>), g, 1024, st, w, (int)lev, kin, pay_in, src, dst, both);
        if constexpr (!PAY) {
          if (both)
            RS_LAUNCH((k_split<K, F32, true, false, 1024, 8, true>), g, 1024, st, w, (int)lev, kin, nullptr, src, dst,
                      1);
        }
      } else
        RS_LAUNCH((k_split<K, false, false, PAY, 1024, 8>), g, 1024, st, w, (int)lev, kin, pay_in, src, dst, 0);
    }
    if (w.count_max > 1ull << 21)
      RS_LAUNCH(k_scan<1024>, grid_for(w.count_max / (1024 * kScanItems) + 1, 2), 1024, st, w, (int)lev);
    else
      RS_LAUNCH(k_scan<256>, grid_for(w.count_max / kScanChunk + 1, 4), 256, st, w, (int)lev);
    RS_LAUNCH(k_route, grid_for(w.big_max, 2), kRouteThreads, st, w, (int)lev, le);
  }
  return local_sorts();
}

int enqueue_sort(int kt, const void* keys_in, const uint32_t* pay_in, const uint64_t* seg_off, uint32_t num_segs,
                 uint64_t n, void* keys_out, uint32_t* perm_out, uint32_t* pay_out, void* ws, size_t ws_bytes,
                 hipStream_t st) {
  const bool pay = pay_in && pay_out;
  if (!pay) {
    pay_in = nullptr;
    pay_out = nullptr;
  }
  switch (kt) {
    case 0:
      return pay ? enqueue_typed<uint32_t, false, true>(keys_in, pay_in, seg_off, num_segs, n, keys_out, perm_out,
                                                         pay_out, ws, ws_bytes, st)
                 : enqueue_typed<uint32_t, false, false>(keys_in, pay_in, seg_off, num_segs, n, keys_out, perm_out,
                                                          pay_out, ws, ws_bytes, st);
    case 1:
      return pay ? enqueue_typed<uint64_t, false, true>(keys_in, pay_in, seg_off, num_segs, n, keys_out, perm_out,
                                                         pay_out, ws, ws_bytes, st)
                 : enqueue_typed<uint64_t, false, false>(keys_in, pay_in, seg_off, num_segs, n, keys_out, perm_out,
                                                          pay_out, ws, ws_bytes, st);
    case 2:
      return pay ? enqueue_typed<uint32_t, true, true>(keys_in, pay_in, seg_off, num_segs, n, keys_out, perm_out,
                                                        pay_out, ws, ws_bytes, st)
                 : enqueue_typed<uint32_t, true, false>(keys_in, pay_in, seg_off, num_segs, n, keys_out, perm_out,
                                                         pay_out, ws, ws_bytes, st);
    default:
      return -1;
  }
}

size_t workspace_bytes(int kt, uint64_t n, uint32_t num_segs, bool pay) {
  return layout(kt, n, num_segs, pay, g_tuning, nullptr, nullptr, nullptr);
}

}  // namespace rs
