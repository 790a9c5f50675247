// Split sort: (key, value) pairs ordered by 64-bit key in at most two scattering
// sweeps and one pass of sorts in LDS, for sorts whose order among equal keys
// does not matter (the re-rank gives equal keys one name whatever their order).
//
// The LSD sort moves every pair once per key digit (7 or 8 sweeps of 24 bytes a
// pair for a round-0 key). Here the number of sweeps depends on the count only:
//
//   1. A stratified sample of the keys, sorted, gives F - 1 splitters (F a power
//      of two, at most 2^20): bucket b holds the keys in
//      (splitter[b - 1], splitter[b]]. Whatever the keys' distribution, a bucket
//      holds about count / F pairs (at most 1024, 1280 above 2^30 pairs). A key that the sample holds several times
//      fills several splitters; all its pairs go to the bucket that begins with
//      the second of them, which holds nothing else (an equality bucket: it is
//      sorted already, however large).
//   2. Up to kSplitMaxD buckets: one sweep scatters the pairs into them. Above:
//      F = D1 * D2, one sweep into D1 groups of D2 neighbouring buckets, one
//      inside each group.
//   3. Every bucket is sorted in LDS by one workgroup: again a sample (a key per
//      thread), a scatter into as many parts of about four pairs, and each pair's place
//      in its part by counting the smaller keys.
//
// Measured on MI355X for the 2^28 round-0 keys of a Markov text (7 varying bytes):
// 8.4 ms from the text to the SA and the survivors (sample 0.3, histograms 0.6 + 0.6,
// sweeps 1.9 + 2.1, LDS 2.9) against 14.2 ms for packing, histogram, seven LSD sweeps
// of 1.68 ms and the re-rank.
//
// Bucket counts come from a histogram before each sweep; a tile reserves its
// part of each bucket with one atomic add per bucket, so the order among equal
// keys (and inside a bucket before step 3) varies from run to run.
//
// A bucket that is no equality bucket and is larger than LDS holds
// (kSplitCap pairs, seven times the largest mean) raises kCtrSplitOver: the keys
// are then unsorted, the re-rank returns at once, and the host repeats the work
// with the LSD sort. With `over` samples per bucket the size of a bucket follows
// a Gamma(over) law; over = 12 (6 up to 1024 buckets, 4 where their mean is at
// most 512) leaves an overflow to inputs made for it. The sample positions are a
// fixed function of the count, so a given input always behaves alike.

#include <type_traits>

#include "driver.h"

namespace sa {

namespace {

constexpr int kSplitBlock = 512;
constexpr int kSplitMaxLogD = 10;
constexpr u32 kSplitMaxD = 1u << kSplitMaxLogD;
constexpr u32 kSplitOne = 4608;       // pairs of an input sorted as one bucket
constexpr u32 kSplitCap = 9216;       // pairs of a bucket sorted in LDS at most
constexpr u32 kSplitRankMax = 8192;   // samples sorted by counting at most
constexpr u32 kSplitOverOne = 6;      // samples per bucket of one sweep at most
static_assert((kSplitOverOne << kSplitMaxLogD) <= kSplitRankMax, "one sweep's samples");
constexpr u32 kSplitXcds = 8;
// Pairs per thread of a sweep over a large input: two workgroups a CU with 1024
// buckets. (8 and 10 give three and two, and 2-5% longer builds: shorter runs.)
constexpr int kSweepItems = 12;
constexpr int kPosBits = 14;          // a place in a bucket
static_assert(kSplitCap <= 1u << kPosBits, "places");
constexpr int kSearchGang = 4;        // searches of a thread side by side

__device__ inline int lane_id() { return threadIdx.x & (kWave - 1); }

__device__ inline u32 wave_inclusive_sum(u32 v) {
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const u32 t = __shfl_up(v, off, kWave);
    if (lane_id() >= off) v += t;
  }
  return v;
}

// Exclusive sum over the workgroup's kSplitBlock threads (every thread calls).
__device__ inline u32 block_exclusive_sum(u32 v, u32* s_w) {
  const int wave = threadIdx.x / kWave;
  const u32 inc = wave_inclusive_sum(v);
  if (lane_id() == kWave - 1) s_w[wave] = inc;
  __syncthreads();
  u32 off = 0;
#pragma unroll
  for (int w = 0; w < kSplitBlock / kWave; ++w)
    if (w < wave) off += s_w[w];
  __syncthreads();
  return off + inc - v;
}

// Splitters sp[0 .. D - 2] (ascending, D = 2^logd) sit in LDS as a search tree in
// breadth-first order: node k has the children 2k and 2k + 1. The nodes of one
// depth are neighbours, so the lanes' reads of a step spread over the banks (in
// sorted order, those of the first steps are multiples of a large power of two
// apart and fall on one bank).
__device__ inline u32 tree_node(u32 i, int logd) {
  const u32 t = u32(__builtin_ctz(i + 1));
  return (1u << (logd - 1 - int(t))) + ((i + 1) >> (t + 1));
}

// Bucket of every key: the number of splitters below it, or the next one when
// the key equals a splitter that fills the next splitter too (bit b of fl). The
// searches of a thread's items go side by side, so that their LDS reads overlap
// (one after the other, the reads' latency alone took longer than the sweep's
// memory traffic).
template <int ITEMS>
__device__ inline void buckets_of(const u64* tree, const u32* fl, int logd, const u64* key,
                                  u32 (&b)[ITEMS]) {
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) b[j] = 1;
  for (int d = 0; d < logd; ++d) {
    u64 x[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) x[j] = tree[b[j]];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) b[j] = 2 * b[j] + (x[j] < key[j] ? 1u : 0u);
  }
  const u32 n = 1u << logd;
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    b[j] -= n;
    if ((fl[b[j] >> 5] >> (b[j] & 31u)) & 1u)
      if (tree[tree_node(b[j], logd)] == key[j]) ++b[j];
  }
}

// Adds one to s_cnt[b] for every lane with `on` and returns the lane's place among
// all so far. Lanes of one bucket, which an LDS atomic takes one after the other, are
// common where neighbours share their top bits (the texts of a batch, repeated
// bytes): a wave of one bucket adds once.
__device__ inline u32 count_in(u32* s_cnt, u32 b, bool on) {
  const u32 b0 = u32(__builtin_amdgcn_readfirstlane(int(b)));
  if (__all(on && b == b0)) {
    u32 base = 0;
    if (lane_id() == 0) base = atomicAdd(&s_cnt[b0], u32(kWave));
    return u32(__builtin_amdgcn_readfirstlane(int(base))) + u32(lane_id());
  }
  return on ? atomicAdd(&s_cnt[b], 1u) : 0u;
}

__device__ inline void flag(u64* counters, u64 bits) {
  atomicOr(reinterpret_cast<unsigned long long*>(counters + kCtrError), (unsigned long long)bits);
}

// The 32-bit integer hash "lowbias32" (Chris Wellons, hash-prospector).
__device__ inline u32 mix32(u32 x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}

}  // namespace

// Shape of one split sort, from its count alone (host).
struct SplitShape {
  u32 count;
  int log1, log2;     // buckets of the first and the second sweep (log2; 0, 0: LDS only)
  u32 over;           // samples per bucket
  u32 samples;        // F * over
  u32 tile;           // pairs per sweep workgroup
  u32 tiles;          // of the first sweep
  u32 groups;         // tile groups of the first sweep, one per XCD (or one)
  u32 per;            // tiles per group
  u32 nb() const { return 1u << (log1 + log2); }
};

// What a round 0 in one workgroup needs besides the sort's own arguments (ctl alone:
// the sort of a later round, whose count is there).
struct SplitTiny {
  const u8* text;
  u16* code;
  SortCtl* ctl;
  u64* rc;
  int trim;
};

// An equality bucket of a round 0 (see split_equal_list_kernel).
constexpr u32 kEqualPiece = 4096;
struct SplitEqual {
  u32 bucket, piece0;
  u64 out;  // first slot of the active list
};

// Device arrays of one split sort.
struct SplitArrays {
  u64* splitters;  // [F], ascending, the last all ones
  u64* top;        // [D1] splitters between the groups of the first sweep
  u32* top_flag;   // [D1 / 32] bit i: top[i] equals the splitter after it
  u32* tot1;       // [groups][D1] counts
  u32* cur1;       // [groups][D1] pairs placed so far
  u32* tot2;       // [D1][D2]
  u32* cur2;       // [D1][D2]
  u32* start1;     // [D1 + 1] first pair of each group of buckets
  u32* tile0;      // [D1 + 1] first tile of the second sweep of each group
  u32* start;      // [F + 1] first pair of each bucket
  u32 *big, *big2;  // number of buckets left to the larger local sorts, then those
  unsigned long long* equal_head;  // round 0: the listed equality buckets
  SplitEqual* equal;               // [F]
};

// Round-0 keys read straight from a text (text == nullptr: from memory): key i is
// the codes of text[i, i + c), w bits each, 0 past the end.
struct SplitText {
  const u8* text;
  const u16* code;
  const u64* counters;  // kCtrCodeBits, kCtrChars
  int words;            // the text is 4-byte aligned
  // A batch (nl.m != 0): `text` is the arena and the keys are those of the joining
  // texts, each with its own codes, w and c and with its slot at idshift. The sort's
  // pairs are the elements from `first` on.
  TextTab tab;
  NewList nl;
  int idshift;
  u64 first;
  // A dense round (names set): key i is the names of suffixes i and i + h, `bits` each.
  const u32* names;
  const RoundCtl* rc;  // h
  int bits;
};
constexpr int kKeyHalo = 64;  // c <= 64
// Where the keys of a first sweep come from.
constexpr int kFromKeys = 0, kFromText = 1, kFromBatch = 2, kFromNames = 3;

// Key of suffix i in a dense round of n suffixes, at offset h.
__device__ inline u64 pair_key(const u32* __restrict__ names, int bits, u64 h, u32 i, u32 n) {
  const u64 j = i + h;
  return (u64(names[i]) << bits) | u64(j < n ? names[j] : 0u);
}

// The joining text that element e of the merged array is in (the last one whose
// first element is at or before e). Every lane of a wave asks for the same e: 64
// probes at a time, two reads in turn for up to 4096 texts.
__device__ inline u32 batch_text_of(const NewList& nl, u64 e) {
  u32 lo = 0, n = nl.m;
  while (n > 1) {
    const u32 step = (n + kWave - 1) / kWave;
    const u32 at = u32(lane_id()) * step;
    const u64 below = __ballot(at < n && nl.out[lo + at] <= e);
    const u32 skip = (u32(__popcll(below)) - 1) * step;  // (probe 0 is: out[lo] <= e)
    lo += skip;
    n = n - skip < step ? n - skip : step;
  }
  return lo;
}

// The same by one thread alone, between texts lo and hi.
__device__ inline u32 batch_text_between(const NewList& nl, u32 lo, u32 hi, u64 e) {
  while (lo < hi) {
    const u32 mid = lo + (hi - lo + 1) / 2;
    if (nl.out[mid] <= e) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// c codes of w bits at a time: key[j] of sym(j) .. sym(j + c - 1).
template <int ITEMS>
__device__ inline void roll_keys(const u16* sym, u32 w, u32 c, u64 tag, u64 (&key)[ITEMS]) {
  const u64 mask = c * w >= 64 ? ~u64(0) : (u64(1) << (c * w)) - 1;
  u64 k = 0;
  for (u32 j = 0; j < c; ++j) k = (k << w) | sym[j];
  key[0] = tag | k;
#pragma unroll
  for (int j = 1; j < ITEMS; ++j) {
    k = ((k << w) | sym[j + c - 1]) & mask;
    key[j] = tag | k;
  }
}

// Codes of positions base .. base + SPAN - 1 of a text of n bytes (0 past its end).
template <u32 SPAN>
__device__ inline void text_codes(const u8* text, u64 base, u64 n, bool words, const u16* s_code,
                                  u16* s_sym) {
  const u32 tid = threadIdx.x;
  if (words && base + SPAN <= n) {
    const u32* tw = reinterpret_cast<const u32*>(text + base);
    for (u32 q = tid; q < SPAN / 4; q += kSplitBlock) {
      const u32 v = tw[q];
      s_sym[4 * q] = s_code[v & 0xFFu];
      s_sym[4 * q + 1] = s_code[(v >> 8) & 0xFFu];
      s_sym[4 * q + 2] = s_code[(v >> 16) & 0xFFu];
      s_sym[4 * q + 3] = s_code[v >> 24];
    }
  } else {
    for (u32 i = tid; i < SPAN; i += kSplitBlock) {
      const u64 p = base + i;
      s_sym[i] = p < n ? s_code[text[p]] : u16(0);
    }
  }
}

// The keys of positions base + ITEMS tid .. + ITEMS - 1 of a tile of ITEMS per
// thread, rolled from the tile's codes in LDS. (Every thread calls; s_sym holds the
// codes of the tile and of kKeyHalo positions more.)
template <int ITEMS>
__device__ inline void text_keys(const SplitText& T, u32 base, u32 count, u16* s_code, u16* s_sym,
                                 u64 (&key)[ITEMS]) {
  constexpr u32 SPAN = u32(ITEMS) * kSplitBlock + kKeyHalo;
  const u32 tid = threadIdx.x;
  const u32 w = u32(T.counters[kCtrCodeBits]);
  const u32 c = u32(T.counters[kCtrChars]);
  if (tid < 256) s_code[tid] = T.code[tid];
  __syncthreads();
  text_codes<SPAN>(T.text, base, count, T.words != 0, s_code, s_sym);
  __syncthreads();
  roll_keys<ITEMS>(s_sym + tid * ITEMS, w, c, 0, key);
}

// The same for elements base + ITEMS tid .. of a batch's merged array (n of the
// tile's are there), and the suffixes' positions in their texts. A tile inside one
// text is read and rolled as above; one that several texts share (a quarter of the
// tiles at 32 KiB a text, all of them below 6 KiB) looks each byte's code up in its
// text's table, in L2. 1024 texts of 1.1e9 bytes: 42.5 -> 39.3 ms a build against
// packing the keys first (4.5 ms, and 2.9 to count them); 4096 of 1.4e8 bytes 2.82 ->
// 2.77.
struct BatchText {  // the text of a workgroup's last tile (its codes are in LDS)
  u64 begin, end;   // its elements
  u64 len;
  const u8* text;
  u32 t, wc;
};
template <int ITEMS>
__device__ inline void batch_keys(const SplitText& T, BatchText& B, u32 base0, u32 n, u16* s_code,
                                  u16* s_sym, u64 (&key)[ITEMS], u32 (&val)[ITEMS]) {
  const u64 base = T.first + base0;
  constexpr u32 TILE = u32(ITEMS) * kSplitBlock;
  const u32 tid = threadIdx.x;
  const NewList& nl = T.nl;
  const u32 first = tid * ITEMS;
  u32 i0 = 0;
  bool one = base >= B.begin && base + n <= B.end;  // all of this is uniform
  if (!one) {
    i0 = batch_text_of(nl, base);
    B.end = nl.out[i0 + 1];  // (out[m] = all elements)
    one = base + n <= B.end;
    if (one) {
      B.begin = nl.out[i0];
      B.t = nl.t[i0];
      B.len = T.tab.len[B.t];
      B.text = T.text + T.tab.base[B.t];
      B.wc = T.tab.wc[B.t];
      if (tid < 256) s_code[tid] = T.tab.code[u64(B.t) * 256 + tid];
      __syncthreads();
    } else {
      B.end = 0;
    }
  }
  if (one) {
    const u64 at = base - B.begin;
    text_codes<TILE + kKeyHalo>(B.text, at, B.len,
                                (reinterpret_cast<uintptr_t>(B.text + at) & 3) == 0, s_code,
                                s_sym);
    __syncthreads();
    roll_keys<ITEMS>(s_sym + first, B.wc & 0xFFFFu, B.wc >> 16, u64(B.t) << T.idshift, key);
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) val[j] = u32(at) + first + j;
    return;
  }
  const u32 i1 = batch_text_of(nl, base + n - 1);
  // Codes of the thread's own elements, and (64 threads) of the halo's, where only
  // the last element's text matters.
  u32 i = first < n ? batch_text_between(nl, i0, i1, base + first) : i1;
  {
    // The bytes are all requested before the first code is.
    u32 k = i, t = nl.t[k];
    u64 end = nl.out[k + 1];
    const u8* from = T.text + T.tab.base[t] - nl.out[k];  // of element 0, were it this text's
    u32 at[ITEMS];
    u8 byte[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      const u64 e = base + first + j;
      byte[j] = 0;
      if (first + j < n) {
        if (e >= end) {
          while (end <= e) end = nl.out[++k + 1];  // (ends: e < out[m])
          t = nl.t[k];
          from = T.text + T.tab.base[t] - nl.out[k];
        }
        byte[j] = from[e];
      }
      at[j] = t;
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      const u16 code = T.tab.code[u64(at[j]) * 256 + byte[j]];
      if (first + j < n) s_sym[first + j] = code;
    }
    const u64 e = base + n + tid;
    if (tid < kKeyHalo && e < nl.out[i1 + 1]) {
      const u32 t = nl.t[i1];
      s_sym[n + tid] = T.tab.code[u64(t) * 256 + T.text[T.tab.base[t] + (e - nl.out[i1])]];
    }
  }
  __syncthreads();
  u32 end = 0, w = 0, c = 0, start = 0;  // of the text in progress, in the tile
  u64 k = 0, mask = 0, tag = 0;
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const u32 q = first + j;
    key[j] = 0;
    val[j] = 0;
    if (q >= n) continue;
    if (j == 0 || q >= end) {
      while (nl.out[i + 1] <= base + q) ++i;
      const u32 t = nl.t[i];
      const u32 wc = T.tab.wc[t];
      w = wc & 0xFFFFu;
      c = wc >> 16;
      mask = c * w >= 64 ? ~u64(0) : (u64(1) << (c * w)) - 1;
      tag = u64(t) << T.idshift;
      start = u32(nl.out[i] - base);  // modulo 2^32
      const u64 e = nl.out[i + 1] - base;
      end = e < TILE + kKeyHalo ? u32(e) : TILE + kKeyHalo;
      k = 0;
      for (u32 x = q; x < q + c; ++x) k = (k << w) | (x < end ? s_sym[x] : u16(0));
    } else {
      const u32 x = q + c - 1;
      k = ((k << w) | (x < end ? s_sym[x] : u16(0))) & mask;
    }
    key[j] = tag | k;
    val[j] = q - start;
  }
}

// What the bucket sorts of a round 0 write besides the sorted keys: SA[place] =
// position for every suffix (a survivor's entry is overwritten when its name
// becomes unique), and the suffixes whose key is not unique as the active list.
// In a batch (tbase set) the key's top bits name the text, positions and names are
// local to it, and the texts' suffixes fill the sorted array in slot order: this
// sort's from place `first` on (keys, values and sa point there). `total` bounds the
// active list.
struct SplitFinal {
  u32* sa;  // nullptr: a plain sort
  u32* act_idx;
  u64* act_ti;  // batch: (text << 32) | position
  u32* act_rank;
  const u64* tbase;
  int idshift;
  u64 first, total;
};

// Code width w and characters per round-0 key c of an alphabet of sigma bytes, as
// alphabet_codes_kernel has them for one text.
__device__ inline void key_shape(u32 sigma, int trim, u32 rb, u32* w, u32* c) {
  *w = sigma ? 32 - __clz(sigma) : 1;
  *c = 64 / *w;
  const u32 used = *c * *w;
  if (trim && used % rb != 0 && used > rb) {
    const u32 full = (used / rb) * rb;
    if (full / *w >= 1) *c = full / *w;
  }
}

// Code of byte value threadIdx.x (of the first 256 threads) from its presence flag:
// 1 + the present bytes below it, 0 if absent; *sigma gets their number. Every
// thread of the workgroup calls; s_w holds four words.
__device__ inline u16 byte_code(bool present, u32* s_w, u32* sigma) {
  const u32 t = threadIdx.x;
  const u32 p = t < 256 && present ? 1u : 0u;
  const u32 inc = wave_inclusive_sum(p);
  if (t < 256 && lane_id() == kWave - 1) s_w[t / kWave] = inc;
  __syncthreads();
  u32 off = 0;
  *sigma = 0;
  for (u32 w = 0; w < 4; ++w) {
    if (w < t / kWave) off += s_w[w];
    *sigma += s_w[w];
  }
  return p ? u16(off + inc) : u16(0);
}

// The sort's plan as the re-rank and the round log read it: the buffer that holds
// the output, and which digits vary (skip flags). One lane per pass.
struct SplitPlanOut {
  SortPlan* plan;  // nullptr: none (a sort of samples)
  u32* log;        // the plan log's row
  int npass, rb;
  u32 final_buf;
  const RoundCtl* rc;  // set: `log` is the whole log, the row the round's
};
__device__ inline void write_plan(const SplitPlanOut& o, u64 varying) {
  const int p = threadIdx.x;
  if (p >= kMaxPasses) return;
  u32 skip = !(p < o.npass && ((varying >> (p * o.rb)) & ((u64(1) << o.rb) - 1)) != 0);
  if (varying == 0) skip = p != o.npass - 1;  // all keys equal: the LSD sort's one copy pass
  u32* log = o.log;
  if (o.rc) log += size_t(o.rc->round < u32(kMaxRounds) ? o.rc->round : 0) * kPlanLogWords;
  o.plan->skip[p] = skip;
  log[p] = skip;
  log[kMaxPasses + p] = 0;
  log[2 * kMaxPasses + p] = 0;
  if (p == 0) {
    o.plan->final_buf = o.final_buf;
    log[3 * kMaxPasses] = o.final_buf;
  }
}

// First kernel: control words of the sort and cleared counts.
__global__ __launch_bounds__(256) void split_begin_kernel(SortCtl* __restrict__ ctl, u64 count,
                                                          u32* __restrict__ clear, u64 words,
                                                          u64* __restrict__ counters) {
  const u64 stride = u64(gridDim.x) * blockDim.x;
  for (u64 i = u64(blockIdx.x) * blockDim.x + threadIdx.x; i < words; i += stride) clear[i] = 0;
  if (!ctl || blockIdx.x != 0) return;
  if (threadIdx.x == 0) {
    ctl->count = count;
    ctl->dense = 0;
  }
  for (u32 i = threadIdx.x; i <= u32(kCtrActive); i += blockDim.x) counters[i] = 0;
}

// Position of sample i: drawn in the i-th of `samples` equal stretches.
__device__ inline u32 sample_position(u32 i, u32 count, u32 samples) {
  const u32 lo = u32(u64(i) * count / samples), hi = u32(u64(i + 1) * count / samples);
  const u32 w = hi > lo ? hi - lo : 1;
  const u32 p = lo + mix32(i + 0x9e3779b9u) % w;
  return p < count ? p : count - 1;
}

__global__ __launch_bounds__(256) void split_sample_kernel(const u64* __restrict__ keys,
                                                           SplitText T, u32 count, u32 samples,
                                                           u64* __restrict__ out) {
  __shared__ u16 s_code[256];
  if (T.text && !T.nl.m) {
    s_code[threadIdx.x] = T.code[threadIdx.x];
    __syncthreads();
  }
  const u32 i = blockIdx.x * 256 + threadIdx.x;
  if (i >= samples) return;
  const u32 p = sample_position(i, count, samples);
  if (!T.text) {
    out[i] = T.names ? pair_key(T.names, T.bits, T.rc->h, p, count) : keys[p];
    return;
  }
  if (T.nl.m) {
    const u64 e0 = T.first + p;
    const u32 x = batch_text_between(T.nl, 0, T.nl.m - 1, e0);
    const u32 t = T.nl.t[x];
    const u32 w = T.tab.wc[t] & 0xFFFFu, c = T.tab.wc[t] >> 16;
    const u8* text = T.text + T.tab.base[t];
    const u64 len = T.tab.len[t];
    u64 k = 0;
    for (u64 q = e0 - T.nl.out[x], e = q + c; q < e; ++q)
      k = (k << w) | (q < len ? T.tab.code[u64(t) * 256 + text[q]] : u16(0));
    out[i] = (u64(t) << T.idshift) | k;
    return;
  }
  const u32 cw = u32(T.counters[kCtrCodeBits]), c = u32(T.counters[kCtrChars]);
  u64 k = 0;
  for (u32 q = 0; q < c; ++q) {
    const u64 x = u64(p) + q;
    k = (k << cw) | (x < count ? s_code[T.text[x]] : u16(0));
  }
  out[i] = k;
}

// Sorts up to kSplitRankMax samples by counting, for each, the smaller ones
// (ties by index): 16 samples per workgroup, each counted by 32 threads that
// read neighbouring samples, so that 8192 samples occupy every CU.
// Every over-th sorted sample is a splitter of the f buckets, written to `out` by
// itself (and the last, all ones); the lists of larger buckets start empty and
// `present`, if any, is cleared for the next build. (So many samples at most only an
// input of one sweep has: two sweeps take 12 for each of 2048 buckets or more.)
__global__ __launch_bounds__(kSplitBlock) void split_rank_kernel(
    const u64* __restrict__ in, u32 samples, u64* __restrict__ out, u32 over, u32 f,
    u32* __restrict__ big, u32* __restrict__ big2, u32* __restrict__ present) {
  constexpr u32 PER = 16, PARTS = kSplitBlock / PER;
  __shared__ u64 s_k[kSplitRankMax];
  __shared__ u32 s_r[PER];
  for (u32 i = threadIdx.x; i < samples; i += kSplitBlock) s_k[i] = in[i];
  if (threadIdx.x < PER) s_r[threadIdx.x] = 0;
  __syncthreads();
  const u32 i = blockIdx.x * PER + threadIdx.x % PER;
  const u32 p = threadIdx.x / PER;
  if (i < samples) {
    const u64 k = s_k[i];
    u32 r = 0;
    u32 j = p;
    // Before sample i an equal one counts, after it does not.
#pragma unroll 8
    for (; j < i; j += PARTS) r += s_k[j] <= k ? 1u : 0u;
#pragma unroll 8
    for (; j < samples; j += PARTS) r += s_k[j] < k ? 1u : 0u;
    atomicAdd(&s_r[threadIdx.x % PER], r);
  }
  __syncthreads();
  if (p == 0 && i < samples) {
    const u32 r = s_r[threadIdx.x];
    if (r > 0 && r % over == 0 && r / over < f) out[r / over - 1] = s_k[i];
  }
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      out[f - 1] = ~u64(0);
      big[0] = big2[0] = 0;
    }
    if (present && threadIdx.x < 256) present[threadIdx.x] = 0;
  }
}

// Splitters from the sorted samples: every over-th, and the table of the first
// sweep (group i + 1 begins after splitter (i + 1) * D2 - 1).
__global__ __launch_bounds__(256) void split_pick_kernel(const u64* __restrict__ sorted, int log1,
                                                         int log2, u32 over, u32 samples,
                                                         SplitArrays A) {
  const u32 f = 1u << (log1 + log2);
  auto at = [&](u32 i) {
    const u64 q = u64(i + 1) * over;
    return i + 1 < f && q < samples ? sorted[q] : ~u64(0);
  };
  const u32 i = blockIdx.x * 256 + threadIdx.x;
  if (i == 0) A.big[0] = A.big2[0] = 0;
  if (i < f) A.splitters[i] = at(i);
  const u32 d1 = 1u << log1;
  if (blockIdx.x * 256 < d1) {
    const u32 last = ((i + 1) << log2) - 1;  // of group i
    const u64 k = i < d1 ? at(last) : 0;
    const bool same = i + 1 < d1 && at(last + 1) == k;
    if (i < d1) A.top[i] = k;
    const u64 m = __ballot(same);
    if ((lane_id() & 31) == 0 && i < d1) A.top_flag[i >> 5] = u32(m >> lane_id());
  }
}

// Round 0 of a text of one sweep, where the launches themselves are most of the
// time: three kernels in place of the clears, the alphabet, the sample and the
// splitters (nine kernels; 2^16 bytes: 108 -> 75 us a build with the plan written
// by the sweep and the counters mirrored by a kernel).
//
// 1. The bytes present (`present` is zero between builds: kernel 3 clears it), and
// every cleared or initial control word.
__global__ __launch_bounds__(256) void small_begin_kernel(const u8* __restrict__ text, u32 n,
                                                          int vec_ok, u32* __restrict__ present,
                                                          SortCtl* __restrict__ ctl,
                                                          u64* __restrict__ counters,
                                                          u64* __restrict__ rc,
                                                          u32* __restrict__ clear, u32 words) {
  __shared__ u32 seen[256];
  seen[threadIdx.x] = 0;
  const u32 stride = gridDim.x * 256, t = blockIdx.x * 256 + threadIdx.x;
  for (u32 i = t; i < words; i += stride) clear[i] = 0;
  if (t < u32(kCtrCount)) counters[t] = 0;
  if (t < u32(sizeof(RoundCtl) / 8)) rc[t] = 0;
  if (t == 0) {
    ctl->count = n;
    ctl->dense = 0;
  }
  __syncthreads();
  const u32 nvec = vec_ok ? n / 16 : 0;
  const uint4* v = reinterpret_cast<const uint4*>(text);
  for (u32 i = t; i < nvec; i += stride) {
    const uint4 x = v[i];
    const u32 ws[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int b = 0; b < 4; ++b) seen[(ws[q] >> (8 * b)) & 0xFFu] = 1;
    }
  }
  for (u32 i = nvec * 16 + t; i < n; i += stride) seen[text[i]] = 1;
  __syncthreads();
  if (seen[threadIdx.x]) atomicOr(&present[threadIdx.x], 1u);
}

// 2. The alphabet (every workgroup for itself, the first one for the kernels after
// it) and the sample.
__global__ __launch_bounds__(256) void small_sample_kernel(const u8* __restrict__ text, u32 n,
                                                           const u32* __restrict__ present,
                                                           int trim, int rb, u32 samples,
                                                           u16* __restrict__ code,
                                                           u64* __restrict__ counters,
                                                           u64* __restrict__ out) {
  __shared__ u16 s_code[256];
  __shared__ u32 s_w[4];
  u32 sigma, w, c;
  const u16 mine = byte_code(present[threadIdx.x] != 0, s_w, &sigma);
  key_shape(sigma, trim, u32(rb), &w, &c);
  s_code[threadIdx.x] = mine;
  if (blockIdx.x == 0) {
    code[threadIdx.x] = mine;
    if (threadIdx.x == 0) {
      counters[kCtrSigma] = sigma;
      counters[kCtrCodeBits] = w;
      counters[kCtrChars] = c;
    }
  }
  __syncthreads();
  const u32 i = blockIdx.x * 256 + threadIdx.x;
  if (i >= samples) return;
  const u32 p = sample_position(i, n, samples);
  u64 k = 0;
  for (u32 q = 0; q < c; ++q) {
    const u64 x = u64(p) + q;
    k = (k << w) | (x < n ? s_code[text[x]] : u16(0));
  }
  out[i] = k;
}

// The pairs [base, base + n) and tables of one tile, for the kernels below.
// Level 1: tile k of group g (g = workgroup mod groups, so that a group stays on
// one XCD, whose L2 joins the partial lines at the ends of neighbouring tiles'
// runs). Level 2: the workgroups of one XCD take consecutive tiles.
struct SplitTile {
  u32 row;   // row of the counts
  u32 base;  // first pair
  u32 n;     // pairs (0: none)
  u32 out0;  // level 2: first pair of the group of buckets
  bool first;
};

__device__ inline SplitTile split_tile2(const SplitArrays& A, u32 d1, u32 tile, u32 bid,
                                        u32* s_row) {
  SplitTile t{0, 0, 0, 0, false};
  const u32 total = A.tile0[d1];
  const u32 per = (total + kSplitXcds - 1) / kSplitXcds;
  const u32 id = (bid % kSplitXcds) * per + bid / kSplitXcds;
  if (bid / kSplitXcds >= per || id >= total) return t;  // uniform
  for (u32 j = threadIdx.x; j < d1; j += kSplitBlock)
    if (A.tile0[j] <= id && id < A.tile0[j + 1]) *s_row = j;
  __syncthreads();
  t.row = *s_row;
  const u32 k = id - A.tile0[t.row];
  t.out0 = A.start1[t.row];
  const u32 size = A.start1[t.row + 1] - t.out0;
  t.first = k == 0;
  t.base = t.out0 + k * tile;
  const u32 left = k * tile < size ? size - k * tile : 0;
  t.n = left < tile ? left : tile;
  return t;
}

// Splitter tree of a sweep into LDS: the first of two sweeps the `top` table and its
// flags, the second the row's own splitters, a single sweep all of them. (Bit D - 1
// of the flags is never set.)
template <bool SECOND>
__device__ inline void load_splitters(const SplitArrays& A, u32 row, int logd, bool two, u64* s_sp,
                                      u32* s_fl) {
  const u32 d = 1u << logd;
  if (!SECOND && two) {
    for (u32 i = threadIdx.x; i + 1 < d; i += kSplitBlock) s_sp[tree_node(i, logd)] = A.top[i];
    for (u32 i = threadIdx.x; i < (d + 31) / 32; i += kSplitBlock) s_fl[i] = A.top_flag[i];
  } else {
    const u64* sp = A.splitters + (SECOND ? u64(row) << logd : 0);
    for (u32 i0 = 0; i0 < d; i0 += kSplitBlock) {
      const u32 i = i0 + threadIdx.x;
      const u64 k = i < d ? sp[i] : 0;
      const bool same = i + 1 < d && sp[i + 1] == k;
      if (i + 1 < d) s_sp[tree_node(i, logd)] = k;
      const u64 m = __ballot(same);
      if ((lane_id() & 31) == 0 && i < d) s_fl[i >> 5] = u32(m >> lane_id());
    }
  }
}

// Counts per bucket. Bound by the key reads (8 bytes a pair) and the search:
// log2(D) LDS reads a pair; from a text, by one byte a pair and the search. Level 1
// also ORs the keys and their complements.
template <int ITEMS, bool SECOND, int FROM>
__global__ __launch_bounds__(kSplitBlock)
__attribute__((amdgpu_waves_per_eu(FROM == kFromBatch ? 5 : 4))) void split_hist_kernel(
    const u64* __restrict__ keys, SplitText T, SplitShape S, SplitArrays A,
    u64* __restrict__ counters) {
  constexpr bool TEXT = FROM == kFromText || FROM == kFromBatch;
  // A tile of a batch has few buckets (those of its text), on whose counts the LDS adds
  // of a wave queue: four counts for each (1.1e9 suffixes: 4.1 -> 3.5 ms).
  constexpr u32 COPIES = FROM == kFromBatch ? 4 : 1;
  __shared__ u16 s_code[TEXT ? 256 : 1];
  __shared__ u16 s_sym[TEXT ? ITEMS * kSplitBlock + kKeyHalo : 1];
  __shared__ u64 s_sp[kSplitMaxD];
  __shared__ u32 s_cnt[kSplitMaxD * COPIES];
  __shared__ u32 s_fl[kSplitMaxD / 32];
  __shared__ u32 s_row;
  __shared__ u64 s_or[kSplitBlock / kWave], s_not[kSplitBlock / kWave];
  constexpr u32 TILE = u32(ITEMS) * kSplitBlock;
  const u32 tid = threadIdx.x;
  const int logd = SECOND ? S.log2 : S.log1;
  const u32 d = 1u << logd;
  u32 row = 0, k0 = 0, kstep = 1, kend = 1;
  SplitTile t{0, 0, 0, 0, false};
  if (SECOND) {
    t = split_tile2(A, 1u << S.log1, TILE, blockIdx.x, &s_row);
    if (t.n == 0) return;
    row = t.row;
  } else {
    row = blockIdx.x % S.groups;
    k0 = blockIdx.x / S.groups;
    kstep = gridDim.x / S.groups;
    kend = S.per;
    if (FROM == kFromBatch) {  // neighbouring tiles, mostly of one text
      const u32 q = (S.per + kstep - 1) / kstep;
      k0 *= q;
      kend = k0 + q < S.per ? k0 + q : S.per;
      kstep = 1;
    }
  }
  BatchText bt{};
  const u64 h = FROM == kFromNames ? T.rc->h : 0;
  load_splitters<SECOND>(A, row, logd, S.log2 != 0, s_sp, s_fl);
  for (u32 i = tid; i < d * COPIES; i += kSplitBlock) s_cnt[i] = 0;
  __syncthreads();
  u64 kor = 0, knot = 0;
  for (u32 k = k0; k < kend; k += kstep) {
    u32 base, n;
    if (SECOND) {
      base = t.base;
      n = t.n;
    } else {
      const u64 b = (u64(row) * S.per + k) * TILE;
      if (b >= S.count) break;
      base = u32(b);
      n = S.count - base < TILE ? S.count - base : TILE;
    }
    u64 key[ITEMS];
    if constexpr (TEXT) {
      u32 unused[ITEMS];
      if constexpr (FROM == kFromBatch)
        batch_keys<ITEMS>(T, bt, base, n, s_code, s_sym, key, unused);
      else text_keys<ITEMS>(T, base, S.count, s_code, s_sym, key);
      __syncthreads();  // the next tile's codes go to the same place
    } else {
#pragma unroll
      for (int j = 0; j < ITEMS; ++j) {
        const u32 e = u32(j) * kSplitBlock + tid;
        if constexpr (FROM == kFromNames)
          key[j] = e < n ? pair_key(T.names, T.bits, h, base + e, S.count) : 0;
        else
          key[j] = e < n ? keys[u64(base) + e] : 0;
      }
    }
    u32 bk[ITEMS];
    buckets_of<ITEMS>(s_sp, s_fl, logd, key, bk);
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      const u32 e = TEXT ? tid * ITEMS + j : u32(j) * kSplitBlock + tid;
      if (COPIES == 1) {
        (void)count_in(s_cnt, bk[j], e < n);
      } else {
        const u32 b0 = u32(__builtin_amdgcn_readfirstlane(int(bk[j])));
        if (__all(e < n && bk[j] == b0)) {
          if (lane_id() == 0) atomicAdd(&s_cnt[b0 * COPIES], u32(kWave));
        } else if (e < n) {
          atomicAdd(&s_cnt[bk[j] * COPIES + tid % COPIES], 1u);
        }
      }
      if (e < n) {
        if (!SECOND) {
          kor |= key[j];
          knot |= ~key[j];
        }
      }
    }
  }
  if (!SECOND) {
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) {
      kor |= __shfl_xor(kor, off, kWave);
      knot |= __shfl_xor(knot, off, kWave);
    }
    if (lane_id() == 0) {
      s_or[tid / kWave] = kor;
      s_not[tid / kWave] = knot;
    }
  }
  __syncthreads();
  u32* tot = SECOND ? A.tot2 : A.tot1;
  for (u32 i = tid; i < d; i += kSplitBlock) {
    u32 c = 0;
    for (u32 q = 0; q < COPIES; ++q) c += s_cnt[i * COPIES + q];
    if (c) atomicAdd(&tot[(u64(row) << logd) + i], c);
  }
  if (!SECOND && counters && tid == 0) {
    u64 o = 0, n = 0;
    for (int w = 0; w < kSplitBlock / kWave; ++w) {
      o |= s_or[w];
      n |= s_not[w];
    }
    // (A word that has the bits already, as far as a plain read tells, is left
    // alone: the atomics of all workgroups on it take 12 ns each.)
    if (o & ~counters[kCtrKeyOr])
      atomicOr(reinterpret_cast<unsigned long long*>(counters + kCtrKeyOr), (unsigned long long)o);
    if (n & ~counters[kCtrKeyNot])
      atomicOr(reinterpret_cast<unsigned long long*>(counters + kCtrKeyNot),
               (unsigned long long)n);
  }
}

// One scattering sweep. Bound by memory: 24 bytes a pair (20 when the values are
// generated), each bucket's run of a tile written contiguously from LDS. A pair's
// place in its run is its LDS fetch-add on the bucket's count (no order among
// equal keys is kept, which saves the LSD sweep's ballots).
// 2^28 suffixes: 1.9 ms from the text (13 bytes a suffix), 2.1 ms the second sweep
// (24 bytes, 3.1 TB/s); 2^30 from names (20 bytes) 11.1 ms. Tiles of 12288 pairs
// (1024 threads, one workgroup a CU) made the whole build 7% slower.
template <int ITEMS, bool SECOND, int FROM>
__global__ __launch_bounds__(kSplitBlock) __attribute__((amdgpu_waves_per_eu(4)))
void split_sweep_kernel(
    const u64* __restrict__ kin, const u32* __restrict__ vin, SplitText T, u64* __restrict__ kout,
    u32* __restrict__ vout, SplitShape S, SplitArrays A, int iota, SplitPlanOut plan,
    u64* __restrict__ counters) {
  constexpr u32 TILE = u32(ITEMS) * kSplitBlock;
  constexpr bool TEXT = FROM == kFromText || FROM == kFromBatch;
  static_assert(kSplitMaxD <= 2 * kSplitBlock, "two buckets per thread");
  __shared__ u64 s_buf[TILE];       // codes of a text, then keys, then values
  static_assert(2 * (TILE + kKeyHalo) <= 8 * TILE, "the tile's codes fit");
  __shared__ u16 s_code[TEXT ? 256 : 1];
  __shared__ u16 s_dig[TILE];
  __shared__ u64 s_sp[kSplitMaxD];  // splitters, then (as u32) the output offsets
  __shared__ u32 s_cnt[kSplitMaxD];
  __shared__ u32 s_fl[kSplitMaxD / 32];
  __shared__ u32 s_w[kSplitBlock / kWave];
  __shared__ u32 s_row;
  const u32 tid = threadIdx.x;
  const int logd = SECOND ? S.log2 : S.log1;
  const u32 d = 1u << logd;
  SplitTile t{0, 0, 0, 0, false};
  if (SECOND) {
    t = split_tile2(A, 1u << S.log1, TILE, blockIdx.x, &s_row);
    if (t.n == 0 && !t.first) return;  // uniform
  } else {
    t.row = blockIdx.x % S.groups;
    const u32 k = blockIdx.x / S.groups;
    const u64 b = (u64(t.row) * S.per + k) * TILE;
    t.first = blockIdx.x == 0;
    if (k >= S.per || b >= S.count) return;  // (workgroup 0 always has a tile)
    t.base = u32(b);
    t.n = S.count - t.base < TILE ? S.count - t.base : TILE;
  }
  // The tile's pairs are requested first. Item j of a thread: striped over the
  // threads, or (from a text) consecutive.
  auto item = [&](int j) { return TEXT ? tid * ITEMS + j : u32(j) * kSplitBlock + tid; };
  u64 key[ITEMS];
  u32 val[ITEMS];
  const u64 h = FROM == kFromNames ? T.rc->h : 0;
  if constexpr (FROM == kFromBatch) {
    BatchText bt{};
    batch_keys<ITEMS>(T, bt, t.base, t.n, s_code, reinterpret_cast<u16*>(s_buf), key, val);
  } else if constexpr (TEXT) {
    text_keys<ITEMS>(T, t.base, S.count, s_code, reinterpret_cast<u16*>(s_buf), key);
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) val[j] = t.base + item(j);
  } else {
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      const u32 e = item(j);
      if constexpr (FROM == kFromNames)
        key[j] = e < t.n ? pair_key(T.names, T.bits, h, t.base + e, S.count) : 0;
      else
        key[j] = e < t.n ? __builtin_nontemporal_load(kin + t.base + e) : 0;
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      const u32 e = item(j);
      val[j] =
          iota ? t.base + e : (vin && e < t.n) ? __builtin_nontemporal_load(vin + t.base + e) : 0;
    }
  }
  load_splitters<SECOND>(A, t.row, logd, S.log2 != 0, s_sp, s_fl);
  for (u32 i = tid; i < d; i += kSplitBlock) s_cnt[i] = 0;
  // Where the buckets 2 tid and 2 tid + 1 of this row start: their totals
  // scanned, plus (level 1) what earlier groups put there.
  u32 all[2] = {0, 0}, below[2] = {0, 0};
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const u32 b = 2 * tid + q;
    if (b >= d) continue;
    if (SECOND) {
      all[q] = A.tot2[(u64(t.row) << logd) + b];
    } else {
      for (u32 g = 0; g < S.groups; ++g) {
        const u32 c = A.tot1[(g << logd) + b];
        all[q] += c;
        if (g < t.row) below[q] += c;
      }
    }
  }
  u32 at[2];
  at[0] = t.out0 + block_exclusive_sum(all[0] + all[1], s_w);  // (two barriers: the tables are set)
  at[1] = at[0] + all[0];
  if (t.first) {
    // What the next kernels read: the start of every bucket and, after the
    // first of two sweeps, the tiles of the second (at least one per group).
    if (!SECOND && plan.plan) write_plan(plan, counters[kCtrKeyOr] & counters[kCtrKeyNot]);
    u32* start = SECOND ? A.start + (u64(t.row) << logd) : S.log2 ? A.start1 : A.start;
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (2 * tid + q < d) start[2 * tid + q] = at[q];
    if (tid == 0 && (!SECOND || t.row + 1 == (1u << S.log1))) start[d] = S.count;
    if (!SECOND && S.log2) {
      u32 nt[2];
#pragma unroll
      for (int q = 0; q < 2; ++q)
        nt[q] = 2 * tid + q < d ? (all[q] ? (all[q] - 1) / S.tile + 1 : 1u) : 0u;
      const u32 t0 = block_exclusive_sum(nt[0] + nt[1], s_w);
      if (2 * tid < d) A.tile0[2 * tid] = t0;
      if (2 * tid + 1 < d) A.tile0[2 * tid + 1] = t0 + nt[0];
      if (2 * tid + 2 == d) A.tile0[d] = t0 + nt[0] + nt[1];
    }
  }
  if (t.n == 0) return;  // uniform
  u32 place[ITEMS];  // bucket, then the pair's place in the tile
  u32 rank[ITEMS];
  buckets_of<ITEMS>(s_sp, s_fl, logd, key, place);
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    rank[j] = count_in(s_cnt, place[j], item(j) < t.n);
  }
  __syncthreads();
  u32 cnt[2] = {0, 0}, off[2] = {0, 0};
  u32* cur = SECOND ? A.cur2 : A.cur1;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const u32 b = 2 * tid + q;
    if (b < d) {
      cnt[q] = s_cnt[b];
      if (cnt[q]) off[q] = at[q] + below[q] + atomicAdd(&cur[(u64(t.row) << logd) + b], cnt[q]);
    }
  }
  const u32 l0 = block_exclusive_sum(cnt[0] + cnt[1], s_w);
  u32* s_delta = reinterpret_cast<u32*>(s_sp);  // every search is done
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const u32 b = 2 * tid + q;
    if (b < d) {
      const u32 l = q ? l0 + cnt[0] : l0;
      s_cnt[b] = l;
      s_delta[b] = off[q] - l;  // modulo 2^32
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    if (item(j) < t.n) {
      const u32 b = place[j];
      const u32 p = s_cnt[b] + rank[j];  // < t.n: the counts of the tile sum to t.n
      place[j] = p;
      s_buf[p] = key[j];
      s_dig[p] = u16(b);
    }
  }
  __syncthreads();
  bool bad = false;
  u32 o[ITEMS];
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const u32 q = u32(j) * kSplitBlock + tid;
    o[j] = ~0u;
    if (q < t.n) {
      o[j] = s_delta[s_dig[q]] + q;
      if (o[j] < S.count) kout[o[j]] = s_buf[q];
      else bad = true;
    }
  }
  if (bad) flag(counters, kErrBounds);
  if (!vout) return;
  __syncthreads();
  u32* s_val = reinterpret_cast<u32*>(s_buf);
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    if (item(j) < t.n) s_val[place[j]] = val[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const u32 q = u32(j) * kSplitBlock + tid;
    if (q < t.n && o[j] < S.count) vout[o[j]] = s_val[q];
  }
}

// x of the lane whose number differs in the bits of MASK (1, 2, 3, 4, 7, 8, 15 by
// data-parallel moves inside rows of 16 lanes, others through LDS hardware).
template <int MASK>
__device__ inline u32 lane_xor(u32 x) {
  auto dpp = [](u32 v, auto ctrl) {
    return u32(__builtin_amdgcn_mov_dpp(int(v), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  if constexpr (MASK == 1) return dpp(x, std::integral_constant<int, 0xB1>{});
  else if constexpr (MASK == 2) return dpp(x, std::integral_constant<int, 0x4E>{});
  else if constexpr (MASK == 3) return dpp(x, std::integral_constant<int, 0x1B>{});
  else if constexpr (MASK == 7) return dpp(x, std::integral_constant<int, 0x141>{});
  else if constexpr (MASK == 4) return lane_xor<3>(lane_xor<7>(x));
  else if constexpr (MASK == 8) return dpp(x, std::integral_constant<int, 0x128>{});
  else if constexpr (MASK == 15) return dpp(x, std::integral_constant<int, 0x140>{});
  else return u32(__shfl_xor(int(x), MASK, kWave));
}

// One compare-exchange step with the lane MASK away: the lower lane keeps the
// smaller key.
template <int MASK>
__device__ inline u64 exchange(u64 v) {
  const u64 o = (u64(lane_xor<MASK>(u32(v >> 32))) << 32) | lane_xor<MASK>(u32(v));
  const bool lower = (lane_id() & MASK) < (MASK + 1) / 2;
  return ((o < v) == lower) ? o : v;
}

// The wave's 64 keys in ascending lane order (bitonic merges of mirrored runs).
__device__ inline u64 wave_sort(u64 v) {
  v = exchange<1>(v);
  v = exchange<3>(v); v = exchange<1>(v);
  v = exchange<7>(v); v = exchange<2>(v); v = exchange<1>(v);
  v = exchange<15>(v); v = exchange<4>(v); v = exchange<2>(v); v = exchange<1>(v);
  v = exchange<31>(v); v = exchange<8>(v); v = exchange<4>(v); v = exchange<2>(v);
  v = exchange<1>(v);
  v = exchange<63>(v); v = exchange<16>(v); v = exchange<8>(v); v = exchange<4>(v);
  v = exchange<2>(v); v = exchange<1>(v);
  return v;
}

// First place of the run of equal keys that place q of a sorted bucket is in (k: its
// key above the low sh bits): steps back that double while they stay in the run, then
// halve, so that a run of r pairs takes 2 log2(r) reads (one key at a time, a text of
// 4608 equal bytes took 1.45 ms a build).
__device__ inline u32 run_head(const u64* s_key, u32 q, int sh, u64 k) {
  u32 h = q, step = 1;
  while (step <= h && s_key[h - step] >> sh == k) {
    h -= step;
    step *= 2;
  }
  while (step >>= 1)
    if (step <= h && s_key[h - step] >> sh == k) h -= step;
  return h;
}

// Every bucket sorted in place, one workgroup each (a persistent grid strides
// over them). BLOCK of the bucket's keys, taken evenly from all of it and sorted (each
// wave its 64 in registers, then their places among the other waves' by binary search),
// are the splitters of BLOCK parts of about four pairs; the pairs go to their parts in
// LDS, and each takes its place there by counting the smaller keys of its part.
// (The bucket's first BLOCK keys are no sample where pairs come nearly in key order: 1 MiB
// of ascending numbers, a line each, took 506 us a build with them, 130 with these, and
// 318 with the LSD sort.) A bucket of fewer than BLOCK pairs has all its keys as samples,
// one of fewer than BLOCK / 4 is one part, which counting sorts sooner (1000 bytes as
// one bucket: 129 us a build as one part, 48 split).
// Bound by memory (24 bytes a pair) as long as the LDS work (about 25 reads a
// pair) and the waits between its steps stay below it: the next bucket's pairs
// are requested as soon as this one's are in LDS, and a workgroup is small (two
// waves and eight workgroups a CU for buckets of 512, four and four for 1024) so
// that others work while one waits.
// A bucket of more than CAP pairs goes to the list `big` for a launch of a larger
// shape (which takes its buckets from there: `from`), or if there is no list raises
// kCtrSplitOver. start == nullptr: the whole input (count <= CAP) is
// the one bucket, with generated values when iota is set and the key ORs left in
// the counters.
// (2^28 suffixes: 3.0 ms with FINAL, 24 bytes a suffix at 2.1 TB/s; 4.2 ms at 96
// registers, which spills.)
// FINAL (a round 0): the sorted pairs leave through LDS in order, which gives every
// pair its neighbours' keys: its name if it is not unique, as the re-rank would
// find it, without another pass over the pairs. The name is 1 + the first place of
// its run of equal keys, which lies in this bucket.
// TINY: the whole round 0 of a text of at most CAP bytes in one workgroup, from the
// control words and the alphabet on (n, text and tables in `tiny`).
template <int CAP, int BLOCK, bool FINAL, bool TINY>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(4)))
void split_local_kernel(
    u64* __restrict__ keys, u32* __restrict__ vals, u32 count, u32 nbuckets,
    const u32* __restrict__ start, const u64* __restrict__ splitters,
    const u32* __restrict__ from, u32* __restrict__ big, int iota, SplitFinal fin,
    SplitPlanOut plan, SplitTiny tiny, u64* __restrict__ counters) {
  constexpr int IT = (CAP + BLOCK * kSearchGang - 1) / (BLOCK * kSearchGang) * kSearchGang;
  constexpr int P = BLOCK;          // parts, and samples
  constexpr int NW = BLOCK / kWave;
  constexpr int LOGP = __builtin_ctz(P);
  constexpr int PER = P / kWave;    // parts per lane of the scanning wave
  constexpr int GANG = 2;           // counts of a thread side by side
  static_assert(kSearchGang % GANG == 0, "whole gangs");
  typedef typename std::conditional<(P <= 256), u8, u16>::type Part;
  __shared__ u64 s_key[CAP + 4];
  __shared__ u32 s_val[CAP];
  __shared__ Part s_part[CAP];
  __shared__ u64 s_raw[P];   // samples
  __shared__ u64 s_sp[P];    // splitter tree
  __shared__ u32 s_cnt[P];
  __shared__ u32 s_off[P + 1];
  __shared__ u32 s_fl[P / 32];
  __shared__ u32 s_left, s_taken;  // FINAL: survivors of the bucket
  __shared__ u64 s_out;
  const u32 tid = threadIdx.x;
  if (!TINY && tiny.ctl) {
    // A later round: its count (at most CAP, bounded by the host) is on the device,
    // and a dense round's values are the positions.
    count = u32(tiny.ctl->count);
    if (count == 0 || count > u32(CAP)) return;
    iota = tiny.ctl->dense != 0;
  }
  if (from) {
    nbuckets = from[0];
    if (blockIdx.x >= nbuckets) return;
  }
  // Bucket w of the launch: its first pair, its size (0: nothing to sort), the
  // key below it and whether its keys, less that one, leave the low kPosBits
  // bits free.
  auto bucket = [&](u32 w, u32& a, u32& m, u64& low, bool& narrow) {
    a = 0;
    m = 0;
    low = 0;
    narrow = false;
    if (w >= nbuckets) return;
    if (!start) {
      m = count;
      return;
    }
    const u32 f = from ? from[1 + w] : w;
    a = start[f];
    const u32 z = start[f + 1];
    low = f > 0 ? splitters[f - 1] : 0;
    const u64 width = splitters[f] - low;
    const bool same = f > 0 && width == 0;
    narrow = (width >> (64 - kPosBits)) == 0;
    if (z < a || z > count) {
      if (tid == 0) flag(counters, kErrBounds);
      return;
    }
    // An equality bucket is in order already, and so is a single pair. (FINAL:
    // split_equal_kernel takes the equality buckets, this kernel every other.)
    if (z == a || same || (!FINAL && z - a == 1)) return;
    if (z - a > u32(CAP)) {
      if (tid == 0) {
        if (big)
          big[1 + atomicAdd(&big[0], 1u)] = f;
        else
          counters[kCtrSplitOver] = 1;
      }
      return;
    }
    m = z - a;
  };
  u64 key[IT];
  u32 val[IT];
  auto load = [&](u32 a, u32 m) {
#pragma unroll
    for (int j = 0; j < IT; ++j) {
      const u32 e = u32(j) * BLOCK + tid;
      key[j] = 0;
      val[j] = 0;
      if (e < m) {
        key[j] = keys[u64(a) + e];
        val[j] = !start && iota ? e : vals ? vals[u64(a) + e] : 0;
      }
    }
  };
  u32 a, m;
  u64 low;
  bool narrow;
  bucket(blockIdx.x, a, m, low, narrow);
  if constexpr (TINY) {
    // The text in LDS (over the values), the bytes seen, the codes (over the tree).
    static_assert(BLOCK >= 256 && P >= 256, "a thread per byte value");
    u8* const s_txt = reinterpret_cast<u8*>(s_val);
    u16* const s_code = reinterpret_cast<u16*>(s_sp);
    for (u32 i = tid; i < 256; i += BLOCK) s_cnt[i] = 0;
    if (tid < u32(kCtrCount) && tid != u32(kCtrActive)) counters[tid] = 0;
    for (u32 i = tid; i < u32(sizeof(RoundCtl) / 8); i += BLOCK) tiny.rc[i] = 0;
    __syncthreads();
    for (u32 i = tid; i < count; i += BLOCK) {
      const u8 x = tiny.text[i];
      s_txt[i] = x;
      s_cnt[x] = 1;
    }
    __syncthreads();
    u32 sigma, cw, c;
    const u16 mine = byte_code(tid < 256 && s_cnt[tid & 255u] != 0, s_off, &sigma);
    key_shape(sigma, tiny.trim, u32(plan.rb), &cw, &c);
    if (tid < 256) {
      s_code[tid] = mine;
      tiny.code[tid] = mine;
    }
    if (tid == 0) {
      // (The clear of these words above is this wave's: the stores stay in order.)
      static_assert(kCtrCount <= kWave, "cleared by the first wave");
      counters[kCtrSigma] = sigma;
      counters[kCtrCodeBits] = cw;
      counters[kCtrChars] = c;
      tiny.ctl->count = count;
      tiny.ctl->dense = 0;
    }
    __syncthreads();
    u64 o = 0, n = 0;
#pragma unroll
    for (int j = 0; j < IT; ++j) {
      const u32 e = u32(j) * BLOCK + tid;
      u64 k = 0;
      if (e < count) {
        for (u32 q = 0; q < c; ++q) k = (k << cw) | (e + q < count ? s_code[s_txt[e + q]] : u16(0));
        o |= k;
        n |= ~k;
      }
      key[j] = k;
      val[j] = e;
    }
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) {
      o |= __shfl_xor(o, off, kWave);
      n |= __shfl_xor(n, off, kWave);
    }
    if (lane_id() == 0) {
      s_raw[tid / kWave] = o;
      s_raw[NW + tid / kWave] = n;
    }
    __syncthreads();
    o = n = 0;
    for (int w = 0; w < NW; ++w) {
      o |= s_raw[w];
      n |= s_raw[NW + w];
    }
    write_plan(plan, o & n);
    __syncthreads();  // the arrays are reused below
  } else {
    load(a, m);
  }
  for (u32 w = blockIdx.x; w < nbuckets; w += gridDim.x) {
    u32 na, nm;
    u64 nlow;
    bool nnarrow;
    bucket(w + gridDim.x, na, nm, nlow, nnarrow);
    if (!TINY && !start) {
      // The whole input: the bits that vary, for the plan.
      u64 o = 0, n = 0;
#pragma unroll
      for (int j = 0; j < IT; ++j)
        if (u32(j) * BLOCK + tid < m) {
          o |= key[j];
          n |= ~key[j];
        }
#pragma unroll
      for (int off = kWave / 2; off >= 1; off >>= 1) {
        o |= __shfl_xor(o, off, kWave);
        n |= __shfl_xor(n, off, kWave);
      }
      if (lane_id() == 0) {
        s_raw[tid / kWave] = o;
        s_raw[NW + tid / kWave] = n;
      }
      __syncthreads();
      o = n = 0;
      for (int w = 0; w < NW; ++w) {
        o |= s_raw[w];
        n |= s_raw[NW + w];
      }
      if (plan.plan) write_plan(plan, o & n);
      __syncthreads();
    }
    const bool split = m >= u32(P) / 4;  // fewer pairs: one part
    s_cnt[tid] = 0;
    if (split) {
      // One key of each thread, of its rows of the bucket in turn (a bit-reversed
      // thread number spreads them evenly over each row): pairs may come in the order
      // of their keys (sorted records, an earlier round's survivors), where the first P
      // alone would leave all others in one part.
      const u32 rows = (m + BLOCK - 1) / BLOCK;  // <= IT
      u32 row = __umulhi(__brev(tid), rows);
      if (row > 0 && row * BLOCK + tid >= m) --row;
      u64 k = row * BLOCK + tid < m ? key[0] : ~u64(0);
#pragma unroll
      for (int j = 1; j < IT; ++j) k = row == u32(j) ? key[j] : k;
      k = wave_sort(k);
      s_raw[tid] = k;
      __syncthreads();
      // Place among all samples: equal ones of earlier waves come first.
      const u32 wave = tid / kWave;
      u32 r = u32(lane_id());
#pragma unroll
      for (u32 o = 1; o < u32(NW); ++o) {
        const u32 other = (wave + o) % NW;
        const u64* list = s_raw + other * kWave;
        const u64 lim = other < wave ? 1 : 0;  // count keys <= k, or < k
        u32 c = 0;
#pragma unroll
        for (u32 step = kWave / 2; step; step >>= 1) {
          const u64 x = list[c + step - 1];
          c += (lim ? x <= k : x < k) ? step : 0u;
        }
        const u64 x = list[c];
        r += c + ((lim ? x <= k : x < k) ? 1u : 0u);
      }
      __syncthreads();
      // Sorted samples 1 .. P - 1 are the splitters.
      s_raw[r] = k;
      if (r > 0) s_sp[tree_node(r - 1, LOGP)] = k;
      __syncthreads();
      // Bit b: splitters b and b + 1 (sorted samples b + 1 and b + 2) are equal.
      const bool same = tid + 2 < u32(P) && s_raw[tid + 1] == s_raw[tid + 2];
      const u64 ms = __ballot(same);
      if ((lane_id() & 31) == 0) s_fl[tid >> 5] = u32(ms >> lane_id());
    }
    __syncthreads();
    u32 pr[IT];  // part | place in it << 16
    if (split) {
#pragma unroll
      for (int j = 0; j < IT; j += kSearchGang) {
        if (u32(j) * BLOCK < m) {  // uniform
          u32 part[kSearchGang];
          buckets_of<kSearchGang>(s_sp, s_fl, LOGP, key + j, part);
#pragma unroll
          for (int y = 0; y < kSearchGang; ++y) {
            const u32 e = u32(j + y) * BLOCK + tid;
            pr[j + y] = e < m ? part[y] | (atomicAdd(&s_cnt[part[y]], 1u) << 16) : 0u;
          }
        }
      }
    } else {
      pr[0] = tid << 16;  // m < P = BLOCK: one pair a thread
      if (tid == 0) s_cnt[0] = m;
    }
    __syncthreads();
    if (tid < u32(kWave)) {
      u32 c[PER], sum = 0;
#pragma unroll
      for (int y = 0; y < PER; ++y) {
        c[y] = s_cnt[PER * tid + y];
        sum += c[y];
      }
      u32 run = wave_inclusive_sum(sum) - sum;
#pragma unroll
      for (int y = 0; y < PER; ++y) {
        s_off[PER * tid + y] = run;
        run += c[y];
      }
      if (tid == u32(kWave) - 1) s_off[P] = run;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IT; ++j) {
      const u32 e = u32(j) * BLOCK + tid;
      if (e < m) {
        const u32 b = pr[j] & 0xFFFFu;
        const u32 p = s_off[b] + (pr[j] >> 16);
        // Narrow buckets: the key's offset with the place below it, so that no
        // two are equal and one comparison orders a pair.
        s_key[p] = narrow ? ((key[j] - low) << kPosBits) | p : key[j];
        s_val[p] = val[j];
        s_part[p] = Part(b);
      }
    }
    if (tid < 4u) s_key[m + tid] = ~u64(0);  // read, never counted, by the last part
    __syncthreads();
    if (!FINAL) load(na, nm);
    // Pair q: its place is its part's start plus the smaller keys of the part.
    // (Parts are ordered: keys read past the part's end are larger.) A part of
    // equal keys is in order already.
    u64 kk[FINAL ? IT : 1];
    u32 place[FINAL ? IT : 1];
#pragma unroll
    for (int j = 0; j < IT; j += GANG) {
      if (u32(j) * BLOCK >= m) break;  // uniform
      u64 k[GANG];
      u32 at[GANG], lo[GANG], longest = 0;
#pragma unroll
      for (int y = 0; y < GANG; ++y) {
        const u32 q = u32(j + y) * BLOCK + tid;
        k[y] = q < m ? s_key[q] : 0;
        const u32 b = q < m ? s_part[q] : 0u;
        lo[y] = s_off[b];
        u32 size = q < m ? s_off[b + 1] - lo[y] : 0u;
        if (split && b > 0 && ((s_fl[(b - 1) >> 5] >> ((b - 1) & 31u)) & 1u)) {
          lo[y] = q;
          size = 1;
        }
        at[y] = lo[y];
        longest = size > longest ? size : longest;
      }
      if (narrow) {
        for (u32 x = 0; x < longest; x += 4) {
#pragma unroll
          for (int y = 0; y < GANG; ++y) {
            const u32 z = lo[y] + x < m ? lo[y] + x : m;
#pragma unroll
            for (u32 i = 0; i < 4; ++i) at[y] += s_key[z + i] < k[y] ? 1u : 0u;
          }
        }
      } else {
        for (u32 x = 0; x < longest; x += 4) {
#pragma unroll
          for (int y = 0; y < GANG; ++y) {
            const u32 z = lo[y] + x < m ? lo[y] + x : m;
            const u32 before = u32(j + y) * BLOCK + tid - z;  // keys of the four before q
#pragma unroll
            for (u32 i = 0; i < 4; ++i) {
              const u64 kx = s_key[z + i];
              at[y] += (kx < k[y] || (kx == k[y] && int(i) < int(before))) ? 1u : 0u;
            }
          }
        }
      }
#pragma unroll
      for (int y = 0; y < GANG; ++y) {
        const u32 q = u32(j + y) * BLOCK + tid;
        if constexpr (FINAL) {
          kk[j + y] = k[y];
          place[j + y] = at[y];
        } else if (q < m) {
          keys[u64(a) + at[y]] = narrow ? (k[y] >> kPosBits) + low : k[y];
          if (vals) vals[u64(a) + at[y]] = s_val[q];
        }
      }
    }
    if constexpr (FINAL) {
      if (tid == 0) s_left = s_taken = 0;
      __syncthreads();
#pragma unroll
      for (int j = 0; j < IT; ++j) {
        const u32 q = u32(j) * BLOCK + tid;
        if (q < m) s_key[place[j]] = kk[j];
        if (!narrow && q < m) kk[j] = s_val[q];
      }
      __syncthreads();
      if (!narrow) {  // (a narrow key names its value's place)
#pragma unroll
        for (int j = 0; j < IT; ++j)
          if (u32(j) * BLOCK + tid < m) s_val[place[j]] = u32(kk[j]);
        __syncthreads();
      }
      load(na, nm);
      constexpr u32 PMASK = (1u << kPosBits) - 1;
      const int sh = narrow ? kPosBits : 0;
      u32 same = 0;  // bit j: item j shares its key with a neighbour
#pragma unroll
      for (int j = 0; j < IT; ++j) {
        const u32 q = u32(j) * BLOCK + tid;
        if (q < m) {
          const u64 x = s_key[q], k = x >> sh;
          const bool dup =
              (q > 0 && s_key[q - 1] >> sh == k) || (q + 1 < m && s_key[q + 1] >> sh == k);
          same |= dup ? 1u << j : 0u;
          keys[u64(a) + q] = narrow ? k + low : k;
          fin.sa[u64(a) + q] = s_val[narrow ? u32(x) & PMASK : q];
        }
      }
      if (same) atomicAdd(&s_left, u32(__popc(same)));
      __syncthreads();
      const u32 left = s_left;
      if (TINY && tid == 0) counters[kCtrActive] = left;
      if (left) {  // uniform
        if (tid == 0)
          s_out = TINY ? 0
                       : atomicAdd(reinterpret_cast<unsigned long long*>(counters + kCtrActive),
                                   (unsigned long long)left);
        __syncthreads();
        if (s_out + left > fin.total) {
          if (tid == 0) flag(counters, kErrBounds);
        } else {
#pragma unroll
          for (int j = 0; j < IT; ++j) {
            const u32 q = u32(j) * BLOCK + tid;
            if ((same >> j) & 1u) {
              const u64 x = s_key[q], k = x >> sh;
              const u32 v = s_val[narrow ? u32(x) & PMASK : q];
              const u32 h = run_head(s_key, q, sh, k);
              const u64 o = s_out + atomicAdd(&s_taken, 1u);
              u64 name = fin.first + a + h + 1;
              if (fin.tbase) {
                const u64 t = (narrow ? k + low : k) >> fin.idshift;
                name -= fin.tbase[t];
                fin.act_ti[o] = (t << 32) | v;
              } else {
                fin.act_idx[o] = v;
              }
              fin.act_rank[o] = u32(name);
            }
          }
        }
      }
    }
    __syncthreads();  // the next bucket reuses the LDS arrays
    a = na;
    m = nm;
    low = nlow;
    narrow = nnarrow;
  }
}

// Round 0, the equality buckets: their pairs are in order, and every suffix of one
// (unless it is alone) survives under the name of the bucket's first place. First
// they are listed, with their slots in the active list and their pieces of
// kEqualPiece pairs numbered in list order; then workgroups take pieces, so that a
// bucket of any size (a text of one character is one bucket) is spread over all.
__global__ __launch_bounds__(256) void split_equal_list_kernel(
    u32 nbuckets, u32 count, const u32* __restrict__ start, const u64* __restrict__ splitters,
    unsigned long long* __restrict__ head,  // entries << 32 | pieces
    SplitEqual* __restrict__ list, u64* __restrict__ counters) {
  const u32 stride = gridDim.x * 256;
  for (u32 f0 = blockIdx.x * 256; f0 < nbuckets; f0 += stride) {  // uniform trip count
    const u32 f = f0 + threadIdx.x;
    u32 m = 0;
    if (f > 0 && f < nbuckets && splitters[f - 1] == splitters[f]) {
      const u32 a = start[f], z = start[f + 1];
      if (z > a && z <= count) m = z - a;
    }
    // One pair of atomics per wave.
    const u64 any = __ballot(m != 0);
    if (any == 0) continue;  // wave-uniform
    const u32 pieces = (m + kEqualPiece - 1) / kEqualPiece;
    const u32 left = m > 1 ? m : 0;
    const u32 pinc = wave_inclusive_sum(pieces);
    u64 linc = left;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const u64 t = __shfl_up(linc, off, kWave);
      if (lane_id() >= off) linc += t;
    }
    unsigned long long h = 0, o = 0;
    if (lane_id() == kWave - 1) {
      h = atomicAdd(head, ((unsigned long long)__popcll(any) << 32) | pinc);
      o = atomicAdd(reinterpret_cast<unsigned long long*>(counters + kCtrActive),
                    (unsigned long long)linc);
    }
    h = __shfl(h, kWave - 1, kWave);
    o = __shfl(o, kWave - 1, kWave);
    if (m) {
      const u32 e = u32(h >> 32) + u32(__popcll(any & ((u64(1) << lane_id()) - 1)));
      list[e] = SplitEqual{f, u32(h) + pinc - pieces, o + linc - left};
    }
  }
}

__global__ __launch_bounds__(256) void split_equal_kernel(
    const u64* __restrict__ keys, const u32* __restrict__ vals, u32 count,
    const u32* __restrict__ start, const unsigned long long* __restrict__ head,
    const SplitEqual* __restrict__ list, SplitFinal fin, u64* __restrict__ counters) {
  const unsigned long long h = *head;
  const u32 entries = u32(h >> 32), pieces = u32(h);
  bool bad = false;
  for (u32 w = blockIdx.x; w < pieces; w += gridDim.x) {
    u32 lo = 0, hi = entries;  // the last entry whose pieces start at or before w
    while (hi - lo > 1) {
      const u32 mid = (lo + hi) >> 1;
      if (list[mid].piece0 <= w)
        lo = mid;
      else
        hi = mid;
    }
    const SplitEqual e = list[lo];
    const u32 a = start[e.bucket], m = start[e.bucket + 1] - a;
    const u32 i0 = (w - e.piece0) * kEqualPiece;
    const u32 i1 = m - i0 < kEqualPiece ? m : i0 + kEqualPiece;
    u64 name = fin.first + a + 1, t = 0;
    if (fin.tbase) {
      t = keys[a] >> fin.idshift;
      name -= fin.tbase[t];
    }
    for (u32 i = i0 + threadIdx.x; i < i1; i += 256) {
      const u32 v = vals[u64(a) + i];
      fin.sa[u64(a) + i] = v;
      if (m == 1) continue;
      const u64 o = e.out + i;
      if (o >= fin.total) {
        bad = true;
        continue;
      }
      if (fin.tbase)
        fin.act_ti[o] = (t << 32) | v;
      else
        fin.act_idx[o] = v;
      fin.act_rank[o] = u32(name);
    }
  }
  if (bad) flag(counters, kErrBounds);
}

// Control words of a build to their pinned host mirror: a kernel's writes reach it
// sooner than a copy command does.
__global__ __launch_bounds__(256) void mirror_kernel(const u64* __restrict__ from, u32 words,
                                                     u64* __restrict__ to) {
  for (u32 i = blockIdx.x * 256 + threadIdx.x; i < words; i += gridDim.x * 256) to[i] = from[i];
}

void launch_mirror(const u64* from, u64* to, u32 words, hipStream_t s) {
  hipLaunchKernelGGL(mirror_kernel, dim3(u32(ceil_div(words, 256))), dim3(256), 0, s, from, words,
                     to);
}

namespace {

SplitShape split_shape(u64 count) {
  SplitShape S{};
  S.count = u32(count);
  int lf = 0;
  if (count > kSplitOne) {
    // Buckets of at most 512 pairs on average; of up to 1024 where one sweep then
    // does for two, and above 2^29 pairs.
    while (lf < 2 * kSplitMaxLogD && (count >> 9) > (u64(1) << lf)) ++lf;
    if (lf == kSplitMaxLogD + 1 && (count >> kSplitMaxLogD) <= kSplitMaxD) lf = kSplitMaxLogD;
    // Small inputs: buckets of 256, so that more CUs take part.
    while (lf < kSplitMaxLogD && (count >> 8) > (u64(1) << lf)) ++lf;
  }
  // One sweep up to 1024 buckets; above, two, the second as wide as it can be (its
  // output stays within one group of buckets, the first one's is all over).
  if (lf <= kSplitMaxLogD) {
    S.log1 = lf;
    S.log2 = 0;
  } else {
    S.log2 = std::min(kSplitMaxLogD, lf - 3);
    S.log1 = lf - S.log2;
  }
  S.over = lf > kSplitMaxLogD ? 12 : count > (u64(512) << lf) ? kSplitOverOne : 4;
  S.samples = S.over << lf;
  // Small inputs: small tiles, so that more CUs take part.
  S.tile = count < (u64(1) << 22) ? 4 * kSplitBlock : kSweepItems * kSplitBlock;
  S.tiles = u32(ceil_div(count, S.tile));
  S.groups = S.tiles >= 16 * kSplitXcds ? kSplitXcds : 1;
  S.per = (S.tiles + S.groups - 1) / S.groups;
  return S;
}

struct Carver {
  char* p;
  size_t left;
  bool ok = true;
  void* take(size_t bytes) {
    bytes = (bytes + 255) / 256 * 256;
    if (bytes > left) {
      ok = false;
      return nullptr;
    }
    void* r = p;
    p += bytes;
    left -= bytes;
    return r;
  }
  template <typename T>
  T* get(u64 n) { return static_cast<T*>(take(size_t(n) * sizeof(T))); }
};

// Arrays of one sort; the counts to clear come first, in one piece.
SplitArrays carve(Carver& cv, const SplitShape& S, bool final, u32** clear, u64* clear_words) {
  SplitArrays A{};
  const u64 d1 = u64(1) << S.log1, f = S.nb(), rows1 = u64(S.groups) * d1;
  const u64 words = 4 + 2 * rows1 + (S.log2 ? 2 * f : 0);
  u32* p = cv.get<u32>(words);
  *clear = p;
  *clear_words = words;
  A.equal_head = reinterpret_cast<unsigned long long*>(p);
  A.tot1 = p + 4;
  A.cur1 = A.tot1 + rows1;
  A.tot2 = A.cur1 + rows1;
  A.cur2 = A.tot2 + f;
  A.splitters = cv.get<u64>(f);
  A.top = cv.get<u64>(d1);
  A.top_flag = cv.get<u32>(ceil_div(d1, 32));
  A.start1 = cv.get<u32>(d1 + 1);
  A.tile0 = cv.get<u32>(d1 + 1);
  A.start = cv.get<u32>(f + 1);
  A.big = cv.get<u32>(f + 1);
  A.big2 = cv.get<u32>(f + 1);
  if (final) A.equal = cv.get<SplitEqual>(f);
  return A;
}

}  // namespace
}  // namespace sa

namespace drv {

// Sorts `count` pairs in (kA, vA) (values optional) within `cv`'s scratch; the
// result ends in buffer A or B (*fin). top: the build's own sort, whose control
// words and plan row are set; otherwise a sort of samples inside one. T.text: the
// keys are the text's, values the positions; out.sa: a round 0 (see SplitFinal;
// values generated, or in vA for a batch).
static sa_status split_run(sa_ctx* c, const Bufs& bf, u64 count, const SplitText& T,
                           const SplitFinal& out, int iota, Carver cv, bool top, int npass,
                           int log_row, u32* fin, hipStream_t s) {
  const SplitShape S = split_shape(count);
  const bool final = out.sa != nullptr;
  u32* clear = nullptr;
  u64 words = 0;
  const SplitArrays A = carve(cv, S, final, &clear, &words);
  u64 *sk = nullptr, *sk2 = nullptr;
  if (S.log1) {
    sk = cv.get<u64>(S.samples);
    sk2 = cv.get<u64>(S.samples);
  }
  if (!cv.ok) return SA_EDEVICE;  // split_usable() has checked this
  u64* ctr = c->counters;
  u64* const ctr_top = top ? ctr : nullptr;
  *fin = 0;
  // Round 0 of a text short enough for one sweep or none starts with its own
  // kernels (see small_begin_kernel).
  const bool batch = T.nl.m != 0;
  const bool small_text = T.text && !batch && !S.log2;
  if (small_text && S.log1) {
    Tracer t(c, s, SA_KERNEL_OTHER, double(count));
    const u8* text = T.text;
    hipLaunchKernelGGL(small_begin_kernel,
                       dim3(u32(std::min<u64>(std::max<u64>(1, ceil_div(count, 256 * 32)), 256))),
                       dim3(256), 0, s, text, S.count, (reinterpret_cast<uintptr_t>(text) & 15) == 0,
                       c->present, c->ctl, ctr, reinterpret_cast<u64*>(c->rc), clear, u32(words));
  } else if (!small_text) {
    Tracer t(c, s, SA_KERNEL_OTHER, 0);
    const u32 g = u32(std::min<u64>(std::max<u64>(1, ceil_div(words, 1024)), 1024));
    // (A batch's later groups add to the counters of its first.)
    hipLaunchKernelGGL(split_begin_kernel, dim3(g), dim3(256), 0, s,
                       top && T.first == 0 ? c->ctl : nullptr, batch ? out.total : count, clear,
                       words, ctr);
  }
  const SplitPlanOut plan{top ? c->plan : nullptr, c->plan_log + size_t(log_row) * kPlanLogWords,
                          npass, c->radix_bits, S.log1 && !S.log2 ? 1u : 0u, nullptr};
#define SA_LOCAL(CAP, BL, GRID, KEYS, VALS, NB, START, SPL, FROM, BIG)                           \
  do {                                                                                           \
    if (final)                                                                                   \
      hipLaunchKernelGGL((split_local_kernel<CAP, BL, true, false>), dim3(GRID), dim3(BL), 0, s, \
                         KEYS, VALS, u32(count), NB, START, SPL, FROM, BIG, iota, out, plan,     \
                         SplitTiny{}, ctr);                                                      \
    else                                                                                         \
      hipLaunchKernelGGL((split_local_kernel<CAP, BL, false, false>), dim3(GRID), dim3(BL), 0, s, \
                         KEYS, VALS, u32(count), NB, START, SPL, FROM, BIG, iota, out, plan,     \
                         SplitTiny{}, ctr);                                                      \
  } while (0)
  if (!S.log1) {
    Tracer t(c, s, SA_KERNEL_SORT_PASS, double(count) * (T.text ? 13.0 : iota ? 20.0 : 24.0));
    if (T.text) {
      const SplitTiny tiny{T.text, c->code, c->ctl, reinterpret_cast<u64*>(c->rc), c->round0_trim};
      hipLaunchKernelGGL((split_local_kernel<int(kSplitOne), 1024, true, true>), dim3(1),
                         dim3(1024), 0, s, bf.kA, nullptr, u32(count), 1u, nullptr, nullptr,
                         nullptr, nullptr, 1, out, plan, tiny, ctr);
      return SA_OK;
    }
    SA_LOCAL(int(kSplitOne), 1024, 1, bf.kA, bf.vA, 1u, nullptr, nullptr, nullptr, nullptr);
  } else {
    {
      Tracer t(c, s, SA_KERNEL_OTHER, 0);
      if (small_text)
        hipLaunchKernelGGL(small_sample_kernel, dim3(u32(ceil_div(S.samples, 256))), dim3(256), 0,
                           s, T.text, S.count, c->present, c->round0_trim, c->radix_bits, S.samples,
                           c->code, ctr, sk);
      else
        hipLaunchKernelGGL(split_sample_kernel, dim3(u32(ceil_div(S.samples, 256))), dim3(256), 0,
                           s, bf.kA, T, S.count, S.samples, sk);
      if (!S.log2) {
        hipLaunchKernelGGL(split_rank_kernel, dim3(u32(ceil_div(S.samples, 16))),
                           dim3(kSplitBlock), 0, s, sk, S.samples, A.splitters, S.over, S.nb(),
                           A.big, A.big2, small_text ? c->present : nullptr);
      } else {
        u32 sf = 0;
        const Bufs sb{sk, sk2, nullptr, nullptr};
        const sa_status st = split_run(c, sb, S.samples, SplitText{}, SplitFinal{}, 0, cv, false, 0,
                                       0, &sf, s);
        if (st != SA_OK) return st;
        hipLaunchKernelGGL(split_pick_kernel, dim3(u32(ceil_div(S.nb(), 256))), dim3(256), 0, s,
                           sf ? sk2 : sk, S.log1, S.log2, S.over, S.samples, A);
      }
    }
    const bool small = S.tile == 4 * kSplitBlock;
    const u32 hgrid = S.groups * std::min<u32>(S.per, 4096 / S.groups);
    const u32* vin = iota ? nullptr : bf.vA;
#define SA_HIST(IT, SECOND, FROM, GRID, KEYS, CTR)                                              \
  hipLaunchKernelGGL((split_hist_kernel<IT, SECOND, FROM>), dim3(GRID), dim3(kSplitBlock), 0, s, \
                     KEYS, T, S, A, CTR)
#define SA_SWEEP(IT, SECOND, FROM, GRID, KIN, VIN, KOUT, VOUT, IOTA)                              \
  hipLaunchKernelGGL((split_sweep_kernel<IT, SECOND, FROM>), dim3(GRID), dim3(kSplitBlock), 0, s, \
                     KIN, VIN, T, KOUT, VOUT, S, A, IOTA, plan, ctr)
    {
      Tracer t(c, s, SA_KERNEL_HISTOGRAM, double(count) * (T.text ? 1.0 : 8.0));
      if (batch) {
        if (small) SA_HIST(4, false, kFromBatch, hgrid, bf.kA, ctr_top);
        else SA_HIST(kSweepItems, false, kFromBatch, hgrid, bf.kA, ctr_top);
      } else if (T.text) {
        if (small) SA_HIST(4, false, kFromText, hgrid, bf.kA, ctr_top);
        else SA_HIST(kSweepItems, false, kFromText, hgrid, bf.kA, ctr_top);
      } else if (T.names) {
        if (small) SA_HIST(4, false, kFromNames, hgrid, bf.kA, ctr_top);
        else SA_HIST(kSweepItems, false, kFromNames, hgrid, bf.kA, ctr_top);
      } else {
        if (small) SA_HIST(4, false, kFromKeys, hgrid, bf.kA, ctr_top);
        else SA_HIST(kSweepItems, false, kFromKeys, hgrid, bf.kA, ctr_top);
      }
    }
    {
      Tracer t(c, s, SA_KERNEL_SORT_PASS, double(count) * (T.text ? 13.0 : iota ? 20.0 : 24.0));
      const u32 grid = S.groups * S.per;
      if (batch) {
        if (small) SA_SWEEP(4, false, kFromBatch, grid, bf.kA, vin, bf.kB, bf.vB, iota);
        else SA_SWEEP(kSweepItems, false, kFromBatch, grid, bf.kA, vin, bf.kB, bf.vB, iota);
      } else if (T.text) {
        if (small) SA_SWEEP(4, false, kFromText, grid, bf.kA, vin, bf.kB, bf.vB, iota);
        else SA_SWEEP(kSweepItems, false, kFromText, grid, bf.kA, vin, bf.kB, bf.vB, iota);
      } else if (T.names) {
        if (small) SA_SWEEP(4, false, kFromNames, grid, bf.kA, vin, bf.kB, bf.vB, iota);
        else SA_SWEEP(kSweepItems, false, kFromNames, grid, bf.kA, vin, bf.kB, bf.vB, iota);
      } else {
        if (small) SA_SWEEP(4, false, kFromKeys, grid, bf.kA, vin, bf.kB, bf.vB, iota);
        else SA_SWEEP(kSweepItems, false, kFromKeys, grid, bf.kA, vin, bf.kB, bf.vB, iota);
      }
    }
    u64* kout = bf.kB;
    u32* vout = bf.vB;
    *fin = 1;
    if (S.log2) {
      // At most one partly filled tile per group; a multiple of the XCDs.
      const u32 grid = u32(ceil_div(u64(S.tiles) + (u64(1) << S.log1), kSplitXcds) * kSplitXcds);
      {
        Tracer t(c, s, SA_KERNEL_HISTOGRAM, double(count) * 8.0);
        if (small) SA_HIST(4, true, kFromKeys, grid, bf.kB, nullptr);
        else SA_HIST(kSweepItems, true, kFromKeys, grid, bf.kB, nullptr);
      }
      {
        Tracer t(c, s, SA_KERNEL_SORT_PASS, double(count) * 24.0);
        if (small) SA_SWEEP(4, true, kFromKeys, grid, bf.kB, bf.vB, bf.kA, bf.vA, 0);
        else SA_SWEEP(kSweepItems, true, kFromKeys, grid, bf.kB, bf.vB, bf.kA, bf.vA, 0);
      }
      kout = bf.kA;
      vout = bf.vA;
      *fin = 0;
    }
#undef SA_HIST
#undef SA_SWEEP
    Tracer t(c, s, SA_KERNEL_SORT_PASS, double(count) * 24.0);
    // Most buckets fit the first, smallest local sort; what it lists goes on to the
    // next (which is short of work, not of room: two lists).
    const u32 nb = S.nb();
    if ((count >> 9) <= nb)
      SA_LOCAL(1016, 128, std::min<u32>(nb, u32(c->num_cus) * 8), kout, vout, nb, A.start,
               A.splitters, nullptr, A.big);
    else
      SA_LOCAL(2032, 256, std::min<u32>(nb, u32(c->num_cus) * 4), kout, vout, nb, A.start,
               A.splitters, nullptr, A.big);
    // (In a single sweep of buckets of 256 pairs on average one larger shape does;
    // elsewhere what the first one leaves, about 0.3% of the buckets, is mostly
    // little larger: 16 MiB of Markov text 0.90 ms with 1024 threads for it, 0.84.)
    const bool short_buckets = (count >> 9) <= nb;
    const bool one_tier = !S.log2 && (count >> 8) <= nb;
    if (!one_tier && short_buckets && S.log2)
      SA_LOCAL(2032, 256, std::min<u32>(nb, u32(c->num_cus) * 4), kout, vout, nb, A.start,
               A.splitters, A.big, A.big2);
    else if (!one_tier)
      SA_LOCAL(3840, 512, std::min<u32>(nb, u32(c->num_cus)), kout, vout, nb, A.start,
               A.splitters, A.big, A.big2);
    SA_LOCAL(int(kSplitCap), 1024, std::min<u32>(nb, u32(c->num_cus)), kout, vout, nb, A.start,
             A.splitters, one_tier ? A.big : A.big2, nullptr);
    if (final) {
      hipLaunchKernelGGL(split_equal_list_kernel, dim3(u32(std::min<u64>(ceil_div(nb, 256), 256))),
                         dim3(256), 0, s, nb, u32(count), A.start, A.splitters, A.equal_head,
                         A.equal, ctr);
      hipLaunchKernelGGL(split_equal_kernel,
                         dim3(u32(std::min<u64>(std::max<u64>(1, count / kEqualPiece),
                                                u64(c->num_cus) * 8))),
                         dim3(256), 0, s, kout, vout, u32(count), A.start, A.equal_head, A.equal,
                         out, ctr);
    }
  }
#undef SA_LOCAL
  return SA_OK;
}

// Whether a sort of `count` pairs may take the split sort. An explicit tuning
// asks for the LSD sweeps it describes. Above 1280 * 2^20 pairs a bucket's mean
// comes too close to what the local sorts hold. The scratch is the active list's
// position array (4 bytes a suffix; no sort's input needs it any more and no
// sort's output yet). The ranks beside it stay: a multi-text round can be repeated.
// A round 0 writes the active list while it still reads the scratch, so its scratch
// is the ISA instead, which is formed after it.
constexpr u64 kSplitMost = u64(1280) << 20;

bool split_usable(const sa_ctx* c, u64 count) {
  if (c->tuning_explicit || c->force_lsd || count == 0 || count > kSplitMost) return false;
  // Arrays and samples of the sort and of the sorts of samples inside it.
  size_t need = 0;
  for (u64 n = count;;) {
    const SplitShape S = split_shape(n);
    Carver cv{nullptr, ~size_t(0)};
    u32* clear;
    u64 words;
    carve(cv, S, true, &clear, &words);
    if (S.log1) {
      cv.get<u64>(S.samples);
      cv.get<u64>(S.samples);
    }
    need += ~size_t(0) - cv.left;
    if (S.log2 == 0) break;
    n = S.samples;
  }
  return need <= size_t(c->cap) * 4;
}

sa_status split_sort(sa_ctx* c, const Bufs& bf, u64 count, int npass, int vals_present, int slot,
                     hipStream_t s) {
  u32 fin = 0;
  const Carver cv{reinterpret_cast<char*>(c->act_idx), size_t(c->cap) * 4};
  return split_run(c, bf, count, SplitText{}, SplitFinal{}, vals_present ? 0 : 1, cv, true, npass,
                   slot, &fin, s);
}

bool split_from_names(u64 count) { return split_shape(count).log1 != 0; }

sa_status split_dense(sa_ctx* c, const Bufs& bf, u64 n, int bits, int npass, int slot,
                      hipStream_t s) {
  u32 fin = 0;
  const Carver cv{reinterpret_cast<char*>(c->act_idx), size_t(c->cap) * 4};
  SplitText T{};
  T.names = c->isa;
  T.rc = c->rc;
  T.bits = bits;
  return split_run(c, bf, n, T, SplitFinal{}, 1, cv, true, npass, slot, &fin, s);
}

bool split_small_text(u64 n) { return split_shape(n).log2 == 0; }

sa_status split_round0(sa_ctx* c, const u8* text, u64 n, int npass, u32* d_sa, hipStream_t s) {
  u32 fin = 0;
  const Carver cv{reinterpret_cast<char*>(c->isa), size_t(c->cap) * 4};
  SplitText T{};
  T.text = text;
  T.code = c->code;
  T.counters = c->counters;
  T.words = (reinterpret_cast<uintptr_t>(text) & 3) == 0;
  const SplitFinal out{d_sa, c->act_idx, nullptr, c->act_rank, nullptr, 0, 0, n};
  return split_run(c, full_bufs(c), n, T, out, 1, cv, true, npass, 0, &fin, s);
}

bool split_one_fits(const sa_ctx* c, u64 bound) {
  return !c->tuning_explicit && !c->force_lsd && bound <= kSplitOne;
}

void split_one(sa_ctx* c, const Bufs& bf, int npass, int log_row, u64 trace_count, hipStream_t s) {
  Tracer t(c, s, SA_KERNEL_SORT_PASS, double(trace_count) * 24.0);
  const SplitPlanOut plan{c->plan,
                          log_row >= 0 ? c->plan_log + size_t(log_row) * kPlanLogWords : c->plan_log,
                          npass, c->radix_bits, 0u, log_row >= 0 ? nullptr : c->rc};
  SplitTiny tiny{};
  tiny.ctl = c->ctl;
  hipLaunchKernelGGL((split_local_kernel<int(kSplitOne), 1024, false, false>), dim3(1), dim3(1024),
                     0, s, bf.kA, bf.vA, u32(0), 1u, nullptr, nullptr, nullptr, nullptr, 0,
                     SplitFinal{}, plan, tiny, c->counters);
}

// A batch of more suffixes than one sort takes goes in groups, filled up to 2^29:
// buckets then hold 512 on average, above up to 1024 and more, which the next larger
// local sort takes, and in equal groups of just over half of that only 300 (4.46e9
// suffixes: LSD sort 264.9 ms, equal groups of at most 2^29 150.5, filled ones 147.7).
// Where one sort does, groups gain nothing: 1.12e9 suffixes 38.9 ms, three equal
// groups 40.5, filled ones 39.9. A group has two sweeps' worth, so that all end in the
// same buffer.
constexpr u64 kBatchGroup = u64(1) << 29;
constexpr u64 kBatchGroupMin = u64(1) << 21;

bool split_batch_groups(const sa_ctx* c, const std::vector<u64>& out, std::vector<u32>* cut) {
  const u32 m = u32(out.size() - 1);
  cut->assign(1, 0);
  if (m == 0 || !split_usable(c, 1)) return false;
  for (u32 i = 1; i < m && out[m] > kSplitMost; ++i) {
    const u64 begin = out[cut->back()];
    if (out[i + 1] - begin > kBatchGroup && out[i] - begin >= kBatchGroupMin &&
        out[m] - out[i] >= kBatchGroupMin)
      cut->push_back(i);
  }
  cut->push_back(m);
  u64 most = 0;
  for (size_t g = 0; g + 1 < cut->size(); ++g)
    most = std::max<u64>(most, out[(*cut)[g + 1]] - out[(*cut)[g]]);
  return split_usable(c, most);
}

bool split_batch_from_text(u64 n) { return split_shape(n).log1 != 0; }

sa_status split_batch0(sa_ctx* c, const std::vector<u64>& nout, const std::vector<u32>& cut,
                       int npass, const u8* arena, const TextTab& tab, const NewList& nl,
                       int idshift, u32* d_sa, hipStream_t s) {
  const u64 total = nout.back();
  for (size_t g = 0; g + 1 < cut.size(); ++g) {
    const u64 first = nout[cut[g]], n = nout[cut[g + 1]] - first;
    u32 fin = 0;
    const Carver cv{reinterpret_cast<char*>(c->isa), size_t(c->cap) * 4};
    const SplitFinal out{d_sa + first, nullptr, c->act_ti, c->act_rank, tab.base, idshift, first,
                         total};
    SplitText T{};
    if (split_batch_from_text(n)) {
      T.text = arena;
      T.tab = tab;
      T.nl = nl;
      T.nl.t += cut[g];
      T.nl.out += cut[g];
      T.nl.m = cut[g + 1] - cut[g];
      T.idshift = idshift;
      T.first = first;
    }
    Bufs b = full_bufs(c);
    b.kA += first;
    b.kB += first;
    b.vA += first;
    b.vB += first;
    const sa_status st = split_run(c, b, n, T, out, 0, cv, true, npass, 0, &fin, s);
    if (st != SA_OK) return st;
  }
  return SA_OK;
}

}  // namespace drv
