// Internal layout shared by the host driver and the kernels of the
// multilevel sample sort engine.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "device.hpp"

namespace rs {

constexpr int kMaxLogK = 9;               // at most 512 buckets per level
constexpr int kMaxK = 1 << kMaxLogK;
constexpr int kMaxLevels = 8;
constexpr int kNumClasses = 10;           // final-bucket size classes (see the class table in engine.hip)
constexpr uint32_t kMaxOversample = 32;

// A level splits every segment tile by tile: each tile of 2^tile_log2
// elements is sorted by bucket and written back as one contiguous piece, and
// the level's matrices say, for every (segment, bucket, tile) in that order,
// where in the tile the bucket's run starts and how long it is (runs: start
// << 16 | length) and how many elements of the segment lie before it in bucket
// order (offs, a running sum; only differences within a segment count).  A
// bucket is read back as its runs, one per tile.

// A segment that the current level splits.
struct BigSeg {
  uint64_t start;   // global position of the first element
  uint64_t ubase;   // position of the user segment start (input-sourced levels: idx = pos - ubase)
  uint64_t pstart;  // start of the segment it is a bucket of (buffer levels)
  uint32_t len;     // number of elements
  uint32_t logk;    // this segment is split into 1 << logk buckets
  uint32_t col;     // buffer levels: its first entry in the previous level's matrices,
  uint32_t nt;      // and its runs there
  uint32_t tb;      // its first tile among the level's tiles
  uint32_t cb;      // its first entry in the level's matrices
};

// A bucket (or a whole user segment) that is sorted in one workgroup.
struct FinalSeg {
  uint64_t start;
  uint64_t pstart;  // buffer segments: start of the segment it is a bucket of
  uint32_t len;
  uint32_t src;  // low byte: 0 caller input (positions implicit), 1 buffer A, 2 buffer B (and the
                 // matrices of the same number);
                 // kPairsFlag: handed from the ranking in bins to k_local_rare
  uint32_t col, nt;  // as in BigSeg
};
constexpr uint32_t kPairsFlag = 0x100;

// Control block at the start of the workspace (all counters device-side).
struct Ctl {
  int32_t status;                  // RSORT_OK or a device-detected error
  uint32_t levels;                 // levels enqueued by the host
  uint32_t big_count[2];           // ping-pong lists of segments to split
  uint32_t tiles[2];               // tiles and matrix entries of the levels (ping-pong, as big_count)
  uint32_t entries[2];
  uint32_t scan_next;              // next chunk of the run lengths to scan (chained scan)
  uint32_t pairs_in[2];            // 1: a segment of buffer A, B was handed to k_local_rare
  uint32_t class_done[kNumClasses];   // final segments already sorted before a later level (three levels or more)
  uint32_t class_count[kNumClasses];  // final segments per size class (last = oversize)
  uint32_t level_max[kMaxLevels];  // largest bucket created per level
  uint32_t level_buckets[kMaxLevels];
  uint64_t class_keys[kNumClasses];  // keys routed to each size class
  // diagnostics of level 0, segment 0
  uint32_t l0_k;
  uint32_t l0_repeats;  // the level-0 splitters repeat keys (looked at from kTiledMin keys on)
  uint32_t init_done;              // workgroups of k_init that are through
  uint64_t l0_spl_key[kMaxK];      // ordinal keys, sorted
  uint32_t l0_spl_pos[kMaxK];
  uint32_t l0_bucket[kMaxK];
};

// Pointers into the workspace for one call.
struct Work {
  Ctl* ctl;
  BigSeg* big[2];
  void* tree_key;        // [big_max * kMaxK] (K), node t of segment s at s*kMaxK + t
  uint32_t* tree_idx;
  uint32_t* runs[2];     // [count_max] matrices of the even and odd levels
  uint32_t* offs[2];     // [count_max]
  uint32_t* tile_seg;    // [tiles_max] segment of each of the level's tiles
  uint32_t* tile_run;    // [tiles_max] buffer levels: the run that holds the tile's first element
  uint64_t* scan_flags;  // [scan_blocks] chained-scan status of each chunk of the run lengths
  FinalSeg* cls[kNumClasses];     // per size class lists
  uint64_t cls_cap[kNumClasses];
  uint32_t* buf_rec[2];  // A, B: [n] element records (ordinal key, position[, payload]; see BufView)
  uint64_t big_max, tiles_max, count_max, scan_blocks, n;
  uint32_t tile_log2;    // log2 of the elements per tile
  uint32_t spread;       // 1: the plan has extra levels, and segments spread their buckets over them
};

// a[i] with a scalar base and a 32-bit byte offset (i * sizeof(T) < 2^32).
template <typename T>
__device__ __forceinline__ T& at32(T* a, uint32_t i) {
  using C = std::conditional_t<std::is_const<T>::value, const char, char>;
  return *reinterpret_cast<T*>(reinterpret_cast<C*>(a) + (uint32_t)(i * (uint32_t)sizeof(T)));
}

// The element buffers of the levels interleave each element's ordinal key,
// its input position and, in payload calls, its payload in one record of
// 32-bit words (key low, key high for 64-bit keys, position, payload), so that
// one memory instruction moves a whole element.
template <typename K, bool PAY>
struct BufView {
  static constexpr int KW = (int)(sizeof(K) / 4);
  static constexpr int W = KW + 1 + (PAY ? 1 : 0);  // words per record
  uint32_t* p;
  struct Rec {
    uint32_t x[W];
  };
  static __device__ __forceinline__ void unpack(const Rec& r, K& k, uint32_t& v, uint32_t& y) {
    if constexpr (sizeof(K) == 8)
      k = ((uint64_t)r.x[1] << 32) | r.x[0];
    else
      k = r.x[0];
    v = r.x[KW];
    if constexpr (PAY) y = r.x[KW + 1];
  }
  __device__ __forceinline__ K key(uint64_t i) const {
    const uint32_t* r = p + i * W;
    if constexpr (sizeof(K) == 8)
      return ((uint64_t)r[1] << 32) | r[0];
    else
      return r[0];
  }
  __device__ __forceinline__ uint32_t idx(uint64_t i) const { return p[i * W + KW]; }
  __device__ __forceinline__ uint32_t pay(uint64_t i) const { return PAY ? p[i * W + W - 1] : 0u; }
  __device__ __forceinline__ void get(uint64_t i, K& k, uint32_t& v, uint32_t& y) const {
    unpack(*reinterpret_cast<const Rec*>(p + i * W), k, v, y);
  }
  // get with a scalar base and a 32-bit byte offset
  __device__ __forceinline__ void get32(uint32_t i, K& k, uint32_t& v, uint32_t& y) const {
    unpack(at32(reinterpret_cast<const Rec*>(p), i), k, v, y);
  }
  __device__ __forceinline__ void put(uint64_t i, K k, uint32_t v, uint32_t y) const {
    Rec r;
    r.x[0] = (uint32_t)k;
    if constexpr (sizeof(K) == 8) r.x[1] = (uint32_t)((uint64_t)k >> 32);
    r.x[KW] = v;
    if constexpr (PAY) r.x[KW + 1] = y;
    *reinterpret_cast<Rec*>(p + i * W) = r;
  }
};

// Place, from the start of the segment it is a bucket of, of a bucket's
// element j: in the last of its runs lo .. hi that starts at or before j.
// (For single elements; whole buckets are read through a RunMap.)
__device__ __forceinline__ uint32_t locate(const Work& w, int m, uint32_t col, uint32_t lo, uint32_t hi, uint32_t j) {
  const uint32_t* o = w.offs[m] + col;
  const uint32_t o0 = o[0];
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (o[mid] - o0 <= j)
      lo = mid;
    else
      hi = mid - 1;
  }
  return (lo << w.tile_log2) + (w.runs[m][col + lo] >> 16) + (j - (o[lo] - o0));
}

// The same for N elements of a bucket of nt runs: all of a step's loads go out
// before any is used.
template <int N>
__device__ __forceinline__ void locate_all(const Work& w, int m, uint32_t col, uint32_t nt, const uint32_t (&j)[N],
                                           uint32_t (&place)[N]) {
  const uint32_t *o = w.offs[m] + col, *r = w.runs[m] + col, o0 = o[0];
  uint32_t lo[N];
#pragma unroll
  for (int i = 0; i < N; i++) lo[i] = 0;
#pragma unroll 1
  for (uint32_t n = nt; n > 1;) {
    const uint32_t half = n >> 1;
    uint32_t x[N];
#pragma unroll
    for (int i = 0; i < N; i++) x[i] = o[lo[i] + half];
#pragma unroll
    for (int i = 0; i < N; i++) lo[i] += x[i] - o0 <= j[i] ? half : 0u;
    n -= half;
  }
#pragma unroll
  for (int i = 0; i < N; i++) place[i] = (lo[i] << w.tile_log2) + (r[lo[i]] >> 16) + (j[i] - (o[lo[i]] - o0));
}

// Reads a final segment by elements (the rare paths and the sorts of small
// classes).
template <typename K, bool F32, bool PAY>
struct SegReader {
  const Work& w;
  const FinalSeg& f;
  const K* in_keys;
  const uint32_t* in_pay;
  __device__ __forceinline__ uint64_t at(uint32_t j) const {
    return f.pstart + locate(w, (int)(f.src & 0xFFu) - 1, f.col, 0, f.nt - 1, j);
  }
  __device__ __forceinline__ void get(uint32_t j, K& k, uint32_t& v) const {
    if (f.src & 0xFFu) {
      uint32_t y;
      BufView<K, PAY>{w.buf_rec[(f.src & 0xFFu) - 1]}.get(at(j), k, v, y);
    } else {
      k = load_ord<K, F32>(in_keys, f.start + j);
      v = j;
    }
  }
  __device__ __forceinline__ uint32_t pay(uint32_t j) const {
    if constexpr (!PAY) return 0u;
    return (f.src & 0xFFu) ? BufView<K, PAY>{w.buf_rec[(f.src & 0xFFu) - 1]}.pay(at(j)) : in_pay[f.start + j];
  }
  // N elements at a time, payloads included; every j is below f.len.
  template <int N>
  __device__ __forceinline__ void get_all(const uint32_t (&j)[N], K (&k)[N], uint32_t (&v)[N], uint32_t (&y)[N]) const {
    if (f.src & 0xFFu) {  // uniform
      const int m = (int)(f.src & 0xFFu) - 1;
      uint32_t place[N];
      locate_all<N>(w, m, f.col, f.nt, j, place);
      const BufView<K, PAY> bv{w.buf_rec[m]};
#pragma unroll
      for (int i = 0; i < N; i++) bv.get(f.pstart + place[i], k[i], v[i], y[i]);
    } else {
#pragma unroll
      for (int i = 0; i < N; i++) {
        k[i] = in_keys[f.start + j[i]];
        v[i] = j[i];
        if constexpr (PAY) y[i] = in_pay[f.start + j[i]];
      }
#pragma unroll
      for (int i = 0; i < N; i++) k[i] = ord_of<K, F32>(k[i]);
    }
  }
};

// Where the elements of a bucket, or of a stretch [j0, j0 + cnt) of one, lie:
// built by a workgroup in LDS from the bucket's runs, one thread per run, in
// three steps with a barrier after each, and then read by whole waves, each
// over 64 consecutive elements at a time.  mask holds a bit for each element that is the
// first of its run (or of the stretch), base the bits before each of its
// words, delta, by run, what added to an element's place in the stretch gives
// its place in the segment.  A stretch of more runs than threads (elements
// strewn thinly over many tiles) sets over, and is read through locate.
template <int THREADS, int N>
struct RunMap {
  static constexpr int NW = THREADS / kWave, WORDS = N / kWave, PL = (WORDS + kWave - 1) / kWave;
  unsigned long long mask[WORDS];
  uint32_t base[WORDS];
  uint32_t delta[THREADS];
  uint32_t wcnt[NW];
  uint32_t over;

  __device__ __forceinline__ void clear(int t) {
    for (int i = t; i < WORDS; i += THREADS) mask[i] = 0ull;
  }
  // Thread t's run (number run of nt): ofs elements of the bucket before it,
  // e its start in its tile, c its length (0: none).
  __device__ __forceinline__ void mark(int t, uint32_t run, uint32_t nt, uint32_t ofs, uint32_t c, uint32_t j0,
                                       uint32_t cnt, uint64_t& bal) {
    const bool in = run < nt && c > 0 && ofs < j0 + cnt && ofs + c > j0;
    bal = __ballot(in);
    if ((t & (kWave - 1)) == 0) wcnt[t / kWave] = (uint32_t)__popcll(bal);
    if (in) {
      const uint32_t s = max(ofs, j0) - j0;
      atomicOr(&mask[s >> 6], 1ull << (s & 63u));
    }
    if (t == THREADS - 1) over = run + 1 < nt && ofs + c < j0 + cnt ? 1u : 0u;
  }
  __device__ __forceinline__ void number(int t, uint32_t run, uint32_t ofs, uint32_t e, uint32_t j0,
                                         uint32_t tile_log2, uint64_t bal) {
    const uint32_t lane = (uint32_t)t & (kWave - 1);
    if ((bal >> lane) & 1ull) {
      uint32_t ord = (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
      for (int q = 0; q < t / kWave; q++) ord += wcnt[q];
      delta[ord] = (run << tile_log2) + e - ofs + j0;
    }
    if (t < kWave) {
      uint32_t x[PL], sum = 0;
#pragma unroll
      for (int k = 0; k < PL; k++) {
        x[k] = t * PL + k < WORDS ? (uint32_t)__popcll(mask[t * PL + k]) : 0u;
        sum += x[k];
      }
      uint32_t s = wave_incl_scan_dpp(sum) - sum;
#pragma unroll
      for (int k = 0; k < PL; k++) {
        if (t * PL + k < WORDS) base[t * PL + k] = s;
        s += x[k];
      }
    }
  }
  // A wave's words: lane i holds what its element i * THREADS + t (one of
  // N / THREADS per thread) needs, read with one LDS access for all of them.
  struct Words {
    uint32_t lo, hi, first;
  };
  __device__ __forceinline__ Words words(int t) const {
    const int wd = min(t & (kWave - 1), N / THREADS - 1) * NW + t / kWave;
    const uint64_t m = mask[wd];
    // run of the word's first element; the bits after it, moved down one
    return Words{(uint32_t)(m >> 1), (uint32_t)(m >> 33), base[wd] + (uint32_t)(m & 1ull) - 1u};
  }
  // Place in the segment of element p = i * THREADS + t of the stretch.
  __device__ __forceinline__ uint32_t at(const Words& w, int i, uint32_t p) const {
    const uint32_t ord = __builtin_amdgcn_mbcnt_hi(
        lane_u32(w.hi, i), __builtin_amdgcn_mbcnt_lo(lane_u32(w.lo, i), lane_u32(w.first, i)));
    return delta[ord] + p;
  }
  // Loads a thread's elements of the stretch (its first cnt; a thread past the
  // end gets some element of the stretch): get(i, place).  Every lane of
  // every wave calls.
  template <typename F>
  __device__ __forceinline__ void each(int t, uint32_t cnt, F&& get) const {
    constexpr int ITEMS = N / THREADS;
    const Words w = words(t);
    if (cnt == (uint32_t)N) {  // uniform
#pragma unroll
      for (int i = 0; i < ITEMS; i++) get(i, at(w, i, i * THREADS + t));
    } else {
      const uint32_t d0 = delta[0];
#pragma unroll
      for (int i = 0; i < ITEMS; i++) {
        const uint32_t p = i * THREADS + t;
        // past the end: the wave's last element, or the stretch's first
        const uint32_t d = i * THREADS + (t & ~(kWave - 1)) < (int)cnt ? at(w, i, p) - (p < cnt ? 0u : p - cnt + 1u) : d0;
        get(i, d);
      }
    }
  }
};

// Launcher flag (or-ed into the class index): sort the whole input of a
// plain call as one segment in a single launch.  The kernels then receive a
// negative class argument.
constexpr int kDirect = 0x100;
// Final segments of class cls (cls < 0: the direct single-segment mode).
__device__ __forceinline__ uint32_t final_count(const Work& w, int cls) {
  if (cls < 0) return 1u;
  return (uint32_t)min((uint64_t)w.ctl->class_count[cls], w.cls_cap[cls]);
}
__device__ __forceinline__ FinalSeg final_at(const Work& w, int cls, uint32_t q) {
  if (cls < 0) return FinalSeg{0ull, 0ull, (uint32_t)w.n, 0u, 0u, 0u};
  return w.cls[cls][q];
}
// In the direct mode no reset kernel runs: the first thread clears the status
// and statistics of the workspace.
__device__ __forceinline__ void direct_reset(const Work& w) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    w.ctl->status = 0;
    w.ctl->levels = 0;
    w.ctl->l0_k = 0;
    for (int c = 0; c < kNumClasses; c++) {
      w.ctl->class_count[c] = 0;
      w.ctl->class_done[c] = 0;
      w.ctl->class_keys[c] = 0;
    }
  }
}

}  // namespace rs
