// Index structures computed on the GPU from a text and its suffix array, the
// step the paper's conclusion names after suffix sorting: the LCP array, the
// Burrows-Wheeler transform of text$, and an FM index that answers pattern
// queries by backward search over the transform.
//
// LCP array, in two parts. First, in suffix array order, LCP[j] is found by
// comparing suffixes SA[j - 1] and SA[j] directly over at most kLcpCap bytes
// (eight at a time); where they agree on all of them the entry is "long".
// Second, only for the long entries: with Phi[SA[j]] = SA[j - 1] (the suffix
// just before suffix i in sorted order), the permuted array PLCP[i] =
// lcp(suffix i, suffix Phi[i]) satisfies PLCP[i + 1] >= PLCP[i] - 1, so a
// left-to-right pass over the text positions extends each common prefix from
// the previous one minus one (Kasai et al.'s argument, in the Phi form of
// Kaerkkaeinen, Manzini and Puglisi), and a long one from at least kLcpCap.
// Each thread runs that pass over its own stretch of positions (skipping
// stretches without long positions, found in a bitmap); then LCP[j] =
// PLCP[SA[j]] for the long entries. Texts with short common prefixes take the
// first part almost alone; repetitive ones fall back to the second.
//
// FM index. Rows of the transform are the sorted suffixes of text$ (row 0 is
// $ alone, row r >= 1 is suffix SA[r - 1]); B[r] is the character before row
// r's suffix. C[c] = 1 + #{i : T[i] < c} is the first row starting with byte c
// and Occ(c, r) = #{q < r : B[q] = c}. Backward search keeps [sp, ep), the rows
// that start with the pattern's suffix read so far: sp = C[c] + Occ(c, sp),
// ep = C[c] + Occ(c, ep) for each pattern byte c from the last to the first.
// Occ comes from a table sampled every kOccBlock rows per byte present in the
// text plus a count over the rest of the block.

#include <cstring>
#include <vector>

#include "driver.h"

using namespace drv;

namespace {

constexpr u32 kNone = 0xFFFFFFFFu;  // no predecessor (SA[0]); never a position (n < 2^32)
constexpr int kLcpStretch = 512;     // positions per thread in the PLCP pass
constexpr u32 kLcpCap = 32;          // bytes compared in suffix array order
constexpr u32 kLcpLong = 0xFFFFFFFFu;  // LCP entry still to come from the PLCP pass
constexpr int kOccBlock = 256;       // rows per occurrence sample
constexpr int kOccGroup = 64;        // sample blocks per workgroup of the count kernel
constexpr int kScanChunk = 4096;     // entries per workgroup of the sample scan

__device__ inline int lane_id() { return threadIdx.x & (kWave - 1); }

__device__ inline void flag_error(u64* err) {
  atomicOr(reinterpret_cast<unsigned long long*>(err), (unsigned long long)kErrBounds);
}

// Length of the common prefix of text[x, n) and text[y, n), at most `cap`,
// comparing eight bytes at a time where whole aligned words around both
// stretches lie inside the text (byte by byte otherwise).
__device__ inline u32 common_prefix(const u8* __restrict__ text, u64 n, u64 x, u64 y, u32 cap) {
  u64 lim = n - (x > y ? x : y);
  if (lim > cap) lim = cap;
  const uintptr_t t0 = reinterpret_cast<uintptr_t>(text);
  const uintptr_t ax = (t0 + x) & ~uintptr_t(7), ay = (t0 + y) & ~uintptr_t(7);
  const u64 words = (lim + 7) / 8 + 1;  // aligned words covering lim bytes from either start
  if (ax >= t0 && ay >= t0 && ax + 8 * words <= t0 + n && ay + 8 * words <= t0 + n) {
    const u64* px = reinterpret_cast<const u64*>(ax);
    const u64* py = reinterpret_cast<const u64*>(ay);
    const u32 sx = u32(t0 + x - ax) * 8, sy = u32(t0 + y - ay) * 8;  // bit offsets
    u64 wx = px[0], wy = py[0];
    for (u64 k = 0; 8 * k < lim; ++k) {
      const u64 nx = px[k + 1], ny = py[k + 1];
      // Bytes [8k, 8k + 8) of each stretch, little-endian.
      const u64 vx = sx ? (wx >> sx) | (nx << (64 - sx)) : wx;
      const u64 vy = sy ? (wy >> sy) | (ny << (64 - sy)) : wy;
      const u64 d = vx ^ vy;
      if (d) {
        const u64 m = 8 * k + u64(__builtin_ctzll(d) / 8);
        return u32(m < lim ? m : lim);
      }
      wx = nx;
      wy = ny;
    }
    return u32(lim);
  }
  u32 m = 0;
  while (m < lim && text[x + m] == text[y + m]) ++m;
  return m;
}

// The first 16 bytes of suffix x, little-endian, 0 past the end of the text.
struct Head {
  u64 lo, hi;
};
__device__ inline Head suffix_head(const u8* __restrict__ text, u64 n, u64 x) {
  const uintptr_t t0 = reinterpret_cast<uintptr_t>(text);
  const uintptr_t ax = (t0 + x) & ~uintptr_t(7);
  Head h{0, 0};
  if (ax >= t0 && ax + 24 <= t0 + n) {
    const u64* p = reinterpret_cast<const u64*>(ax);
    const u64 w0 = p[0], w1 = p[1], w2 = p[2];
    const u32 s = u32(t0 + x - ax) * 8;
    h.lo = s ? (w0 >> s) | (w1 << (64 - s)) : w0;
    h.hi = s ? (w1 >> s) | (w2 << (64 - s)) : w1;
  } else if (x < n) {
    for (u32 q = 0; q < 16 && x + q < n; ++q) {
      if (q < 8)
        h.lo |= u64(text[x + q]) << (8 * q);
      else
        h.hi |= u64(text[x + q]) << (8 * (q - 8));
    }
  }
  return h;
}

// LCP in suffix array order up to kLcpCap; a long entry marks its position in
// `long_bits`, records Phi there and sets *any_long.
// Bound by the random reads of the text (a line per suffix): each suffix's first
// 16 bytes are read once, by one lane, and its successor takes them from that lane
// (neighbours used to read both suffixes of every pair: two lines per entry, 2^26
// suffixes of a Markov text in 1.62 ms). A wave takes kLcpRows rows of 64 consecutive
// entries, whose reads overlap. (16 rows, four at a time, save few second reads and
// leave short texts to few waves: 1000 bytes 35 us a call, 43 with 16; 2^26 the same,
// 0.74 and 0.84 ms for sorted lines.)
constexpr int kLcpRows = 4;
__global__ __launch_bounds__(256) void lcp_direct_kernel(const u8* __restrict__ text, u64 n,
                                                         const u32* __restrict__ sa,
                                                         u32* __restrict__ lcp,
                                                         u32* __restrict__ phi,
                                                         u32* __restrict__ long_bits,
                                                         u64* __restrict__ any_long,
                                                         u64* __restrict__ err) {
  const int lane = lane_id();
  const u64 wave = (u64(blockIdx.x) * blockDim.x + threadIdx.x) / kWave;
  const u64 first = wave * (u64(kLcpRows) * kWave);
  if (first >= n) return;  // wave-uniform
  // The suffix before the wave's first entry.
  u32 carry_s = first > 0 ? sa[first - 1] : 0;
  Head carry = first > 0 ? suffix_head(text, n, carry_s) : Head{0, 0};
  u32 b[kLcpRows];
  Head h[kLcpRows];
#pragma unroll
  for (int g = 0; g < kLcpRows; ++g) {
    const u64 j = first + u64(g) * kWave + lane;
    b[g] = j < n ? sa[j] : 0;
  }
#pragma unroll
  for (int g = 0; g < kLcpRows; ++g) h[g] = suffix_head(text, n, b[g]);
#pragma unroll
  for (int g = 0; g < kLcpRows; ++g) {
    const u64 j = first + u64(g) * kWave + lane;
    u32 a = __shfl_up(b[g], 1, kWave);
    Head p{__shfl_up(h[g].lo, 1, kWave), __shfl_up(h[g].hi, 1, kWave)};
    if (lane == 0) {
      a = carry_s;
      p = carry;
    }
    carry_s = __shfl(b[g], kWave - 1, kWave);
    carry.lo = __shfl(h[g].lo, kWave - 1, kWave);
    carry.hi = __shfl(h[g].hi, kWave - 1, kWave);
    if (j >= n) continue;
    if (j == 0) {
      lcp[0] = 0;
      continue;
    }
    if (a >= n || b[g] >= n || a == b[g]) {
      flag_error(err);
      lcp[j] = 0;
      continue;
    }
    const u64 room = n - (a > b[g] ? a : b[g]);
    const u64 dl = p.lo ^ h[g].lo, dh = p.hi ^ h[g].hi;
    u32 m = dl ? u32(__builtin_ctzll(dl) / 8) : dh ? 8 + u32(__builtin_ctzll(dh) / 8) : 16u;
    if (m > room) m = u32(room);
    if (m == 16) m += common_prefix(text, n, u64(a) + 16, u64(b[g]) + 16, kLcpCap - 16);
    if (m < kLcpCap) {
      lcp[j] = m;
    } else {
      lcp[j] = kLcpLong;
      phi[b[g]] = a;
      atomicOr(&long_bits[b[g] >> 5], 1u << (b[g] & 31u));
      *any_long = 1;
    }
  }
}

// PLCP at the long positions, over stretches of kLcpStretch positions, in
// place over Phi. A long position's common prefix is at least kLcpCap and at
// least the previous position's minus one when that one was long too.
__global__ __launch_bounds__(256) void plcp_long_kernel(const u8* __restrict__ text, u64 n,
                                                        const u32* __restrict__ long_bits,
                                                        const u64* __restrict__ any_long,
                                                        u32* __restrict__ phi_plcp) {
  static_assert(kLcpStretch % 32 == 0, "whole bitmap words per stretch");
  if (*any_long == 0) return;
  const u64 t = u64(blockIdx.x) * blockDim.x + threadIdx.x;
  const u64 lo = t * kLcpStretch;
  if (lo >= n) return;
  const u64 hi = lo + kLcpStretch < n ? lo + kLcpStretch : n;
  u64 l = 0;
  for (u64 w0 = lo; w0 < hi; w0 += 32) {
    u32 bits = long_bits[w0 >> 5];
    if (!bits) {
      l = 0;
      continue;
    }
    for (u64 i = w0; i < hi && i < w0 + 32; ++i) {
      if (!((bits >> (i - w0)) & 1u)) {
        l = 0;
        continue;
      }
      const u64 p = phi_plcp[i];
      if (l < kLcpCap) l = kLcpCap;
      // Extend eight bytes at a time while both stretches agree on all of them.
      for (;;) {
        const u64 room = n - (i > p ? i : p);
        if (l >= room) break;
        const u32 step = room - l < 4096 ? u32(room - l) : 4096u;
        const u32 m = common_prefix(text, n, i + l, p + l, step);
        l += m;
        if (m < step) break;
      }
      phi_plcp[i] = u32(l);
      l = l ? l - 1 : 0;
    }
  }
}

// LCP[j] = PLCP[SA[j]] for the long entries.
__global__ __launch_bounds__(256) void lcp_long_gather_kernel(const u32* __restrict__ sa, u64 n,
                                                              const u32* __restrict__ plcp,
                                                              const u64* __restrict__ any_long,
                                                              u32* __restrict__ lcp) {
  if (*any_long == 0) return;
  const u64 stride = u64(gridDim.x) * blockDim.x;
  for (u64 j = u64(blockIdx.x) * blockDim.x + threadIdx.x; j < n; j += stride) {
    if (lcp[j] != kLcpLong) continue;
    const u32 s = sa[j];
    lcp[j] = s < n ? plcp[s] : 0u;
  }
}

// The row of $ (1 + the j with SA[j] = 0) into *dollar.
__global__ __launch_bounds__(256) void find_dollar_kernel(const u32* __restrict__ sa, u64 n,
                                                          int vec_ok, u64* __restrict__ dollar) {
  const u64 stride = u64(gridDim.x) * blockDim.x;
  const u64 t = u64(blockIdx.x) * blockDim.x + threadIdx.x;
  const u64 nvec = vec_ok ? n / 4 : 0;
  const uint4* v = reinterpret_cast<const uint4*>(sa);
  for (u64 i = t; i < nvec; i += stride) {
    const uint4 x = v[i];
    if (x.x == 0 || x.y == 0 || x.z == 0 || x.w == 0)
      *dollar = 4 * i + 1 + (x.x == 0 ? 0 : x.y == 0 ? 1 : x.z == 0 ? 2 : 3);
  }
  for (u64 j = nvec * 4 + t; j < n; j += stride)
    if (sa[j] == 0) *dollar = j + 1;
}

// Transform rows r = 0 .. n: B[r] = T[n - 1] for r = 0, T[SA[r - 1] - 1]
// otherwise; the $ row either is left out (compact: rows after it move down by
// one, *dollar known) or holds the byte 0 (the FM index keeps every row and
// corrects its counts at the $ row, which goes to *dollar here).
// Bound by the random reads of the text (a line per row). A thread makes four
// neighbouring output bytes, so that four reads are in flight and they leave as one
// word (one byte a thread: 1.21 ms for 2^26 rows of a Markov text). `out` is
// 4-byte aligned when `words` is set.
__global__ __launch_bounds__(256) void bwt_kernel(const u8* __restrict__ text, u64 n,
                                                  const u32* __restrict__ sa,
                                                  u64* __restrict__ dollar, int compact,
                                                  int words, u8* __restrict__ out,
                                                  u64* __restrict__ err) {
  const u64 d = compact ? *dollar : ~u64(0);
  const u64 outs = compact ? n : n + 1;
  const u64 stride = u64(gridDim.x) * blockDim.x * 4;
  for (u64 o = (u64(blockIdx.x) * blockDim.x + threadIdx.x) * 4; o < outs; o += stride) {
    u32 s[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const u64 r = o + q + (o + q >= d ? 1 : 0);  // (n + 1 past the last row of a compact one)
      s[q] = r == 0 ? u32(n) : r <= n ? sa[r - 1] : 1u;
      if (r > 0 && s[q] >= n) s[q] = 0xFFFFFFFFu;  // not a position
    }
    u32 word = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool in = o + q < outs;
      if (in && s[q] > n) flag_error(err);
      if (in && s[q] == 0 && !compact) *dollar = o + q;
      const u8 ch = in && s[q] != 0 && s[q] <= n ? text[s[q] - 1] : u8(0);
      word |= u32(ch) << (8 * q);
    }
    if (words && o + 4 <= outs) {
      *reinterpret_cast<u32*>(out + o) = word;
    } else {
      for (int q = 0; q < 4; ++q)
        if (o + q < outs) out[o + q] = u8(word >> (8 * q));
    }
  }
}

// Byte counts of the text (for C) in LDS, a copy per wave, then one atomic per
// byte value. The text is read as 16-byte words where it is 16-byte aligned.
__global__ __launch_bounds__(256) void byte_count_kernel(const u8* __restrict__ text, u64 n,
                                                         int vec_ok, u64* __restrict__ counts) {
  __shared__ u32 h[4][256];
  for (int i = threadIdx.x; i < 4 * 256; i += 256) (&h[0][0])[i] = 0;
  __syncthreads();
  u32* mine = h[threadIdx.x / kWave];
  const u64 stride = u64(gridDim.x) * blockDim.x;
  const u64 t = u64(blockIdx.x) * blockDim.x + threadIdx.x;
  const u64 nvec = vec_ok ? n / 16 : 0;
  const uint4* v = reinterpret_cast<const uint4*>(text);
  for (u64 i = t; i < nvec; i += stride) {
    const uint4 x = v[i];
    const u32 ws[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int by = 0; by < 4; ++by) atomicAdd(&mine[(ws[k] >> (8 * by)) & 0xFFu], 1u);
    }
  }
  for (u64 i = nvec * 16 + t; i < n; i += stride) atomicAdd(&mine[text[i]], 1u);
  __syncthreads();
  const u32 c = h[0][threadIdx.x] + h[1][threadIdx.x] + h[2][threadIdx.x] + h[3][threadIdx.x];
  if (c)
    atomicAdd(reinterpret_cast<unsigned long long*>(counts + threadIdx.x), (unsigned long long)c);
}

// Per sample block b (rows [b * kOccBlock, (b + 1) * kOccBlock) of B): the
// count of each present byte, written to occ[code][b] (a later scan turns the
// counts into prefix sums). A workgroup takes kOccGroup consecutive blocks so
// that each byte's row of counts is written in runs. The $ row (byte 0 in B)
// is not counted.
// Counts are 16-bit halves, two blocks a word (a block has 256 rows), and only the
// present bytes have them: 128 * sigma bytes of LDS, which is what each workgroup
// clears and reads again (64 KB of it took twice the time of the counting).
__global__ __launch_bounds__(256) void occ_count_kernel(const u8* __restrict__ B, u64 rows,
                                                        u64 nblocks,
                                                        const u64* __restrict__ dollar_ptr,
                                                        const u16* __restrict__ code, u32 sigma,
                                                        u64 stride_b, u32* __restrict__ occ) {
  extern __shared__ u32 cnt[];  // [sigma][kOccGroup / 2]
  constexpr u32 HW = kOccGroup / 2;
  __shared__ u16 s_code[256];
  s_code[threadIdx.x] = code[threadIdx.x];
  const u64 dollar = dollar_ptr ? *dollar_ptr : ~u64(0);
  for (u32 i = threadIdx.x; i < sigma * HW; i += 256) cnt[i] = 0;
  __syncthreads();
  const u64 b0 = u64(blockIdx.x) * kOccGroup;
  const u64 r0 = b0 * kOccBlock;
  constexpr u32 kWords = kOccGroup * kOccBlock / 4;  // words of the group
  // (B is padded to whole blocks.)
  const u64 padded = nblocks * kOccBlock;
  for (u32 q = threadIdx.x; q < kWords; q += 256) {
    const u64 r = r0 + u64(q) * 4;
    if (r >= padded) continue;
    const u32 w = *reinterpret_cast<const u32*>(B + r);
    const u32 g = q * 4 / kOccBlock;
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const u32 c = s_code[(w >> (8 * y)) & 0xFFu];
      if (r + y < rows && r + y != dollar && c < sigma)
        atomicAdd(&cnt[c * HW + g / 2], 1u << (16 * (g & 1u)));
    }
  }
  __syncthreads();
  for (u32 idx = threadIdx.x; idx < sigma * kOccGroup; idx += 256) {
    const u32 c = idx / kOccGroup, g = idx % kOccGroup;
    const u64 b = b0 + g;
    if (b < nblocks)
      occ[u64(c) * stride_b + b] = (cnt[c * HW + g / 2] >> (16 * (g & 1u))) & 0xFFFFu;
  }
}

// Exclusive scan of each byte's row of block counts, in three steps: chunks
// of kScanChunk entries scanned in LDS (chunk totals saved), the totals of a
// row scanned by one workgroup, the chunk offsets added.
__global__ __launch_bounds__(256) void occ_scan_chunks_kernel(u32* __restrict__ occ, u64 entries,
                                                              u64 stride_b, u64 chunks,
                                                              u64* __restrict__ totals) {
  __shared__ u32 wsum[4];
  const u64 c = blockIdx.y;
  const u64 ch = blockIdx.x;
  u32* row = occ + c * stride_b;
  const u64 base = ch * kScanChunk;
  constexpr int IT = kScanChunk / 256;
  // (stride_b is a multiple of 64 entries: a row is padded to whole 16-byte words.)
  u32 v[IT];
  u32 sum = 0;
#pragma unroll
  for (int k = 0; k < IT; k += 4) {
    const u64 e = base + u64(threadIdx.x) * IT + k;
    const uint4 x = e < stride_b ? *reinterpret_cast<const uint4*>(row + e) : uint4{0, 0, 0, 0};
    v[k] = e < entries ? x.x : 0u;
    v[k + 1] = e + 1 < entries ? x.y : 0u;
    v[k + 2] = e + 2 < entries ? x.z : 0u;
    v[k + 3] = e + 3 < entries ? x.w : 0u;
    sum += v[k] + v[k + 1] + v[k + 2] + v[k + 3];
  }
  // Exclusive scan of the per-thread sums.
  u32 inc = sum;
  for (int off = 1; off < kWave; off <<= 1) {
    const u32 t = __shfl_up(inc, off, kWave);
    if (lane_id() >= off) inc += t;
  }
  if (lane_id() == kWave - 1) wsum[threadIdx.x / kWave] = inc;
  __syncthreads();
  u32 woff = 0, total = 0;
  for (int w = 0; w < 4; ++w) {
    if (w < int(threadIdx.x / kWave)) woff += wsum[w];
    total += wsum[w];
  }
  u32 run = woff + inc - sum;
#pragma unroll
  for (int k = 0; k < IT; k += 4) {
    const u64 e = base + u64(threadIdx.x) * IT + k;
    uint4 x;
    x.x = run;
    x.y = x.x + v[k];
    x.z = x.y + v[k + 1];
    x.w = x.z + v[k + 2];
    run = x.w + v[k + 3];
    if (e < stride_b) *reinterpret_cast<uint4*>(row + e) = x;
  }
  if (threadIdx.x == 0) totals[c * chunks + ch] = total;
}

__global__ __launch_bounds__(64) void occ_scan_totals_kernel(u64* __restrict__ totals,
                                                             u64 chunks) {
  if (threadIdx.x != 0) return;
  u64* t = totals + u64(blockIdx.x) * chunks;
  u64 run = 0;
  for (u64 k = 0; k < chunks; ++k) {
    const u64 v = t[k];
    t[k] = run;
    run += v;
  }
}

__global__ __launch_bounds__(256) void occ_scan_add_kernel(u32* __restrict__ occ, u64 entries,
                                                           u64 stride_b, u64 chunks,
                                                           const u64* __restrict__ totals) {
  const u64 c = blockIdx.y;
  const u64 ch = blockIdx.x;
  const u32 add = u32(totals[c * chunks + ch]);
  u32* row = occ + c * stride_b;
  const u64 base = ch * kScanChunk;
  for (int k = threadIdx.x; k < kScanChunk; k += 256) {
    const u64 e = base + u64(k);
    if (e < entries) row[e] += add;
  }
}

// Backward search. Occ(c, r) is the sample at r's block plus the matches of byte c
// among the block's rows before r (minus the $ row when c is the byte 0 that stands
// in for it). Bound by the latency of a chain of dependent random reads, one step
// per pattern byte, so what counts is how many chains are in flight: a bound of a
// pattern takes 16 lanes (a 256-row block is 16 bytes a lane), a wave two patterns
// (one pattern a wave: 200 us for 2^16 patterns of 16 bytes in a 2^26-byte text).
// Patterns are concatenated with offsets[num + 1].
__global__ __launch_bounds__(256) void fm_count_kernel(
    const u8* __restrict__ B, u64 n, u64 dollar, const u32* __restrict__ occ, u64 stride_b,
    const u64* __restrict__ C, const u16* __restrict__ code, const u8* __restrict__ pats,
    const u64* __restrict__ offs, u32 num, u64* __restrict__ ranges) {
  static_assert(kOccBlock == 256, "16 lanes of 16 bytes");
  __shared__ u64 s_C[256];
  __shared__ u16 s_code[256];
  s_C[threadIdx.x] = C[threadIdx.x];
  s_code[threadIdx.x] = code[threadIdx.x];
  __syncthreads();
  const int lane = lane_id();
  const bool upper = (lane >> 4) & 1;  // this quarter of the wave holds ep, else sp
  const u32 l = u32(lane & 15);
  const u64 pairs = (u64(num) + 1) / 2;
  const u64 waves = (u64(gridDim.x) * blockDim.x) / kWave;
  for (u64 w = (u64(blockIdx.x) * blockDim.x + threadIdx.x) / kWave; w < pairs; w += waves) {
    const u64 q = 2 * w + u64(lane >> 5);
    const bool have = q < num;
    const u64 a = have ? offs[q] : 0, z = have ? offs[q + 1] : 0;
    u64 pos = upper ? n + 1 : 0;
    u64 k = z;
    while (__any(k > a)) {  // wave-uniform: the shuffles below see every lane
      const bool on = k > a;
      u32 part = 0;
      u64 base = 0, sample = 0;
      bool absent = false;
      if (on) {
        --k;
        const u32 c = pats[k];
        const u32 cc = s_code[c];
        base = s_C[c];
        absent = cc == 0xFFFFu;  // the byte does not occur: no row starts with it
        if (!absent) {
          const u64 start = pos & ~u64(kOccBlock - 1);
          const uint4 x = reinterpret_cast<const uint4*>(B + start)[l];
          sample = occ[u64(cc) * stride_b + start / kOccBlock];
          const u32 before = u32(pos - start);  // rows of the block before pos
          const u32 mine = before > 16 * l ? before - 16 * l : 0u;
          const u32 cw = c * 0x01010101u;
          const u32 ws[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
          for (u32 i = 0; i < 4; ++i) {
            const u32 d = ws[i] ^ cw;
            const u32 nz = ((d & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | d | 0x7F7F7F7Fu;  // 0x7F: zero byte
            const u32 take = mine > 4 * i ? mine - 4 * i : 0u;
            const u32 keep = take >= 4 ? ~0u : (1u << (8 * take)) - 1u;
            part += u32(__popc(~nz & keep));
          }
          if (l == 0 && c == 0 && dollar >= start && dollar < pos) part -= 1;
        }
      }
#pragma unroll
      for (int off = 1; off < 16; off <<= 1) part += u32(__shfl_xor(int(part), off, kWave));
      if (on) pos = absent ? base : base + sample + u64(int(part));
    }
    if (have && l == 0) {
      // Rows 1.. are suffixes SA[0..]: the $ row never starts with a byte. The
      // empty pattern: every suffix.
      const u64 v = z > a ? pos - 1 : upper ? n : 0;
      ranges[2 * q + (upper ? 1 : 0)] = v;
    }
  }
}

__global__ __launch_bounds__(256) void fill_tail_kernel(u8* __restrict__ p, u64 from, u64 to) {
  for (u64 i = from + threadIdx.x; i < to; i += 256) p[i] = 0;
}

void launch_fill_tail(u8* p, u64 from, u64 to, hipStream_t s) {
  hipLaunchKernelGGL(fill_tail_kernel, dim3(1), dim3(256), 0, s, p, from, to);
}

u32 grid_for(u64 items, u32 per_block, u32 cap) {
  u64 g = ceil_div(std::max<u64>(items, 1), per_block);
  return u32(std::min<u64>(g, cap));
}

sa_status finish(sa_ctx* c, hipStream_t s) {
  // readback() also reports the kernels' error flag.
  return readback(c, s);
}

}  // namespace

// The FM index: the transform rows, the occurrence samples and the tables.
struct sa_fm {
  int device = 0;
  u64 n = 0, dollar = 0, nblocks = 0, stride_b = 0;
  u32 sigma = 0;
  void* dev = nullptr;
  u8* B = nullptr;
  u32* occ = nullptr;
  u64* C = nullptr;
  u16* code = nullptr;
};

extern "C" {

sa_status sa_lcp(sa_ctx* ctx, const uint8_t* d_text, uint64_t n, const uint32_t* d_sa,
                 uint32_t* d_lcp, void* stream) {
  if (!ctx) return SA_EINVAL;
  if (n == 0) return SA_OK;
  if (!d_text || !d_sa || !d_lcp) return SA_EINVAL;
  if (n >= (u64(1) << 32)) return SA_ETOOBIG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (hipSetDevice(ctx->device) != hipSuccess) return SA_EDEVICE;
  sa_status st = ensure_workspace(ctx, n);
  if (st != SA_OK) return st;
  launch_fill_u64(ctx->counters, kCtrCount, 0, s);
  u32* phi = ctx->isa;        // Phi at the long positions, then PLCP in place
  u32* long_bits = ctx->live;  // the long positions
  launch_fill_u32(long_bits, ceil_div(n, 32), 0, s);
  const u32 g = grid_for(n, 256, 8192);
  u64* any_long = ctx->counters + kCtrIndexAux;
  hipLaunchKernelGGL(lcp_direct_kernel,
                     dim3(u32(ceil_div(ceil_div(n, u64(kLcpRows) * kWave), 256 / kWave))),
                     dim3(256), 0, s, d_text, n, d_sa, d_lcp, phi, long_bits, any_long,
                     ctx->counters + kCtrError);
  const u64 threads = ceil_div(n, kLcpStretch);
  hipLaunchKernelGGL(plcp_long_kernel, dim3(u32(ceil_div(threads, 256))), dim3(256), 0, s,
                     d_text, n, long_bits, any_long, phi);
  hipLaunchKernelGGL(lcp_long_gather_kernel, dim3(g), dim3(256), 0, s, d_sa, n, phi, any_long,
                     d_lcp);
  return finish(ctx, s);
}

sa_status sa_bwt(sa_ctx* ctx, const uint8_t* d_text, uint64_t n, const uint32_t* d_sa,
                 uint8_t* d_bwt, uint64_t* dollar, void* stream) {
  if (!ctx || !dollar) return SA_EINVAL;
  *dollar = 0;
  if (n == 0) return SA_OK;
  if (!d_text || !d_sa || !d_bwt) return SA_EINVAL;
  if (n >= (u64(1) << 32)) return SA_ETOOBIG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (hipSetDevice(ctx->device) != hipSuccess) return SA_EDEVICE;
  launch_fill_u64(ctx->counters, kCtrCount, 0, s);
  u64* d_dollar = ctx->counters + kCtrIndexAux;
  hipLaunchKernelGGL(find_dollar_kernel, dim3(grid_for(n, 256 * 16, 4096)), dim3(256), 0, s, d_sa,
                     n, (reinterpret_cast<uintptr_t>(d_sa) & 15) == 0, d_dollar);
  hipLaunchKernelGGL(bwt_kernel, dim3(grid_for(n, 1024, 65536)), dim3(256), 0, s, d_text, n, d_sa,
                     d_dollar, 1, (reinterpret_cast<uintptr_t>(d_bwt) & 3) == 0, d_bwt,
                     ctx->counters + kCtrError);
  const sa_status st = finish(ctx, s);
  if (st != SA_OK) return st;
  *dollar = ctx->h_counters[kCtrIndexAux];
  if (*dollar == 0 || *dollar > n) return SA_EDEVICE;  // SA holds no 0: not a suffix array
  return SA_OK;
}

sa_status sa_fm_create(sa_fm** out, sa_ctx* ctx, const uint8_t* d_text, uint64_t n,
                       const uint32_t* d_sa, void* stream) {
  if (!out || !ctx) return SA_EINVAL;
  *out = nullptr;
  if (n >= (u64(1) << 32)) return SA_ETOOBIG;
  if (n && (!d_text || !d_sa)) return SA_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (hipSetDevice(ctx->device) != hipSuccess) return SA_EDEVICE;
  sa_fm* fm = new (std::nothrow) sa_fm();
  if (!fm) return SA_ENOMEM;
  fm->device = ctx->device;
  fm->n = n;
  const u64 rows = n + 1;
  fm->nblocks = ceil_div(rows, kOccBlock) + 1;  // one more: Occ(c, rows) when rows % 256 == 0
  // Byte counts -> C, the present bytes and their codes (on the host: 256 values).
  std::vector<u64> counts(256, 0);
  // (In the context's sample array, which only a build's rounds use.)
  u64* tmp = ctx->sample;
  static_assert(kLazySamples >= 256, "the byte counts fit");
  launch_fill_u64(tmp, 256, 0, s);
  if (n)
    hipLaunchKernelGGL(byte_count_kernel, dim3(grid_for(n, 256 * 16 * 4, 1024)), dim3(256), 0, s,
                       d_text, n, (reinterpret_cast<uintptr_t>(d_text) & 15) == 0, tmp);
  if (hipMemcpyAsync(counts.data(), tmp, 256 * sizeof(u64), hipMemcpyDeviceToHost, s) !=
          hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess) {
    delete fm;
    return SA_EDEVICE;
  }
  std::vector<u64> C(256, 0);
  std::vector<u16> code(256, 0xFFFFu);
  std::vector<u8> sym;
  u64 run = 1;  // row 0 is $
  for (int c = 0; c < 256; ++c) {
    C[c] = run;
    run += counts[c];
    if (counts[c]) {
      code[c] = u16(sym.size());
      sym.push_back(u8(c));
    }
  }
  fm->sigma = u32(sym.size());
  fm->stride_b = (fm->nblocks + 63) / 64 * 64;
  const u64 chunks = ceil_div(fm->nblocks, kScanChunk);
  // One allocation: B (rows, padded to whole blocks), occ, C, code, sym, totals.
  const size_t b_bytes = (fm->nblocks * kOccBlock + 255) / 256 * 256;
  const size_t occ_bytes = size_t(std::max<u32>(fm->sigma, 1)) * fm->stride_b * 4;
  const size_t off_occ = b_bytes, off_C = off_occ + occ_bytes, off_code = off_C + 256 * 8,
               off_tot = off_code + 512 + 256,
               total = off_tot + size_t(std::max<u32>(fm->sigma, 1)) * chunks * 8;
  if (hipMalloc(&fm->dev, total) != hipSuccess) {
    (void)hipGetLastError();
    delete fm;
    return SA_ENOMEM;
  }
  char* p = static_cast<char*>(fm->dev);
  fm->B = reinterpret_cast<u8*>(p);
  fm->occ = reinterpret_cast<u32*>(p + off_occ);
  fm->C = reinterpret_cast<u64*>(p + off_C);
  fm->code = reinterpret_cast<u16*>(p + off_code);
  u64* totals = reinterpret_cast<u64*>(p + off_tot);
  sa_status st = SA_OK;
  // The rows past the last one (the pad of its block and the last, empty block).
  launch_fill_tail(fm->B, rows, b_bytes, s);
  if (hipMemcpyAsync(fm->C, C.data(), 256 * 8, hipMemcpyHostToDevice, s) != hipSuccess ||
      hipMemcpyAsync(fm->code, code.data(), 512, hipMemcpyHostToDevice, s) != hipSuccess)
    st = SA_EDEVICE;
  u64* d_dollar = ctx->counters + kCtrIndexAux;
  if (st == SA_OK) {
    launch_fill_u64(ctx->counters, kCtrCount, 0, s);
    if (n)
      hipLaunchKernelGGL(bwt_kernel, dim3(grid_for(rows, 1024, 65536)), dim3(256), 0, s, d_text, n,
                         d_sa, d_dollar, 0, 1, fm->B, ctx->counters + kCtrError);
  }
  if (st == SA_OK && fm->sigma) {
    hipLaunchKernelGGL(occ_count_kernel, dim3(u32(ceil_div(fm->nblocks, kOccGroup))), dim3(256),
                       fm->sigma * kOccGroup * 2, s, fm->B, rows, fm->nblocks, d_dollar, fm->code,
                       fm->sigma, fm->stride_b, fm->occ);
    hipLaunchKernelGGL(occ_scan_chunks_kernel, dim3(u32(chunks), fm->sigma), dim3(256), 0, s,
                       fm->occ, fm->nblocks, fm->stride_b, chunks, totals);
    hipLaunchKernelGGL(occ_scan_totals_kernel, dim3(fm->sigma), dim3(64), 0, s, totals, chunks);
    hipLaunchKernelGGL(occ_scan_add_kernel, dim3(u32(chunks), fm->sigma), dim3(256), 0, s,
                       fm->occ, fm->nblocks, fm->stride_b, chunks, totals);
  }
  if (st == SA_OK) {
    st = finish(ctx, s);  // waits for the index and reports the kernels' errors
    if (st == SA_OK && n) {
      fm->dollar = ctx->h_counters[kCtrIndexAux];
      if (fm->dollar == 0 || fm->dollar > n) st = SA_EDEVICE;
    }
  }
  if (st != SA_OK) {
    sa_fm_destroy(fm);
    return st;
  }
  *out = fm;
  return SA_OK;
}

sa_status sa_fm_count(sa_fm* fm, const uint8_t* d_patterns, const uint64_t* d_offsets,
                      uint32_t num_patterns, uint64_t* d_ranges, void* stream) {
  if (!fm) return SA_EINVAL;
  if (num_patterns == 0) return SA_OK;
  if (!d_offsets || !d_ranges) return SA_EINVAL;
  if (hipSetDevice(fm->device) != hipSuccess) return SA_EDEVICE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const u32 g = grid_for(num_patterns, 2 * (256 / kWave), 16384);
  hipLaunchKernelGGL(fm_count_kernel, dim3(g), dim3(256), 0, s, fm->B, fm->n, fm->dollar,
                     fm->occ, fm->stride_b, fm->C, fm->code, d_patterns, d_offsets, num_patterns,
                     d_ranges);
  if (hipGetLastError() != hipSuccess) return SA_EDEVICE;
  return SA_OK;
}

sa_status sa_fm_info(const sa_fm* fm, uint64_t* n, uint64_t* dollar, uint32_t* sigma,
                     uint64_t* device_bytes) {
  if (!fm) return SA_EINVAL;
  if (n) *n = fm->n;
  if (dollar) *dollar = fm->dollar;
  if (sigma) *sigma = fm->sigma;
  if (device_bytes) {
    const u64 chunks = ceil_div(fm->nblocks, kScanChunk);
    *device_bytes = (fm->nblocks * kOccBlock + 255) / 256 * 256 +
                    u64(std::max<u32>(fm->sigma, 1)) * fm->stride_b * 4 + 256 * 8 + 512 + 256 +
                    u64(std::max<u32>(fm->sigma, 1)) * chunks * 8;
  }
  return SA_OK;
}

sa_status sa_fm_destroy(sa_fm* fm) {
  if (!fm) return SA_OK;
  (void)hipSetDevice(fm->device);
  (void)hipFree(fm->dev);
  delete fm;
  return SA_OK;
}

}  // extern "C"
