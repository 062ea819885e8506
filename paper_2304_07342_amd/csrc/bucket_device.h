// Chunk encoder for 1- and 2-byte symbols with MIN >= 2: candidates from
// 2-symbol buckets instead of comparing every position with its window.
#pragma once

#include "encode_device.h"

namespace gpulz {
namespace enc {
namespace bucket {

// A match of MIN >= 2 symbols at p with offset d has the same 2-symbol
// prefix at p - d, so it is enough to look at the earlier positions whose
// 2-symbol hash equals p's. A tile of kTile positions, and the window before
// it, is bucketed by (hash, block of kPB positions), hash first, so that the
// positions p may match are one run of the bucketed order: p's bucket and
// those of the nb blocks before it. An entry holds a position and its first
// kInline symbols (as bytes), so that a candidate costs one 8-byte LDS read
// and a dozen vector instructions. Neighbouring lanes of the search take
// neighbouring entries, so they walk the same run: their reads are broadcasts
// and their trip counts alike; the hashes are ordered by how often they occur
// (three classes), so that short runs do not wait for long ones.
//
// The search tells matches of up to kInline - 1 symbols exactly. Where a
// position's best is longer, it is only marked, and the parse works it out
// when a token really starts there: of a long match's positions the parse
// visits one. With one such candidate (the usual case) its offset is kept and
// the parse only extends it; with several, or where a match is cut by its
// own offset or the chunk end, the parse takes the per-column search.
//
// 2-byte symbols are searched through one byte of each: the low byte where the
// chunk's symbols span less than 256 values, which loses nothing, else a hash of
// both bytes (the low byte may hardly vary: big-endian values, samples scaled by
// 256). There every result is checked against the symbols and marked where
// they differ (equal symbols have equal bytes, so a result that holds is the
// best). 16 MiB of 8-bit noise scaled by 256 (C 2048, W 128): 1358 us by low
// bytes, all alike, 113 by the hash; of byte-swapped codes 331 and 195.
//
// Bound by vector instruction issue: about 420 of them per 64 positions (Zipf
// bytes), at four fifths of what the SIMDs issue (comparing every position with a window
// of 256 took over 1000). 64 MiB of Zipf bytes, C 4096, W 256: 2203 us before,
// 843 so; uint16 codes, C 2048, W 128: 1153 and 536; 1 MiB of codes 56 and 36.
// Tiles of 1024 positions with 4 waves: tiles of 2048 took 969 us (Zipf), 8
// waves 958; blocks of 64 positions 917 (shorter runs, twice the counters).
constexpr uint32_t kPB = 128;         // positions per block
constexpr uint32_t kHashBits = 8;
constexpr uint32_t kHash = 1u << kHashBits;
constexpr uint32_t kTile = 1024;      // positions searched per round
constexpr uint32_t kMaxNb = kMaxWindow / kPB;          // blocks before p's own
constexpr uint32_t kMaxIns = kTile + kMaxNb * kPB;     // positions bucketed per tile
constexpr uint32_t kMaxRow = (kTile / kPB + kMaxNb) / 2 + 1;
constexpr uint32_t kUnroll = 2;                        // candidates per step of the search
constexpr uint32_t kInline = 6;                        // symbols in an entry
constexpr uint32_t kMaxSyms = 8192;                    // chunks it takes
constexpr uint32_t kMaxWaves = 16;
// Results to be worked out at a token start (exact ones are 0 or L << 8 | d &
// 0xFF with L >= 2): kOne | d & 0xFF = the match at offset d, of at least
// kInline symbols; kAny = any match.
constexpr uint32_t kOne = 1u << 8, kAny = 1u;
constexpr uint32_t kShared = kMaxWaves + 16;           // shared words

// Blocks of the window before a position's own.
__host__ __device__ constexpr uint32_t window_blocks(uint32_t W) { return (W + kPB - 1) / kPB; }
// Words of a hash's 16-bit counters: one per block of a tile, and its end.
__host__ __device__ constexpr uint32_t row_words(uint32_t nb) { return (kTile / kPB + nb) / 2 + 1; }
__host__ __device__ constexpr uint32_t max_ins(uint32_t nb) { return kTile + nb * kPB; }
// The parse takes segments of 2^seg_shift positions, at most one per thread.
// (1024 threads: 8 positions, so that more waves share the searches at token
// starts; 256 KiB of runs of up to 8 bytes, C 2048, W 128: 125 us with 16, 74 with
// 8, 55 with 4; uint16 codes 32.5, 31.2, 35.7; 256 KiB of Zipf bytes 23.5 and 21.9.
// 1 MiB of codes goes by its slowest chunk: 35 to 41 us with 16 and 35 to 42 with 8
// over 16 draws, 37.8 and 37.6 on average.)
__host__ __device__ constexpr uint32_t seg_shift(uint32_t C, uint32_t threads) {
  return threads == 1024 && C <= 4096 ? 3u : C <= 16 * threads ? 4u : 5u;
}
// Position p's result: lanes of the parse read one segment apart, so each
// segment is followed by one unused word (a bank further each).
__host__ __device__ constexpr uint32_t res_at(uint32_t p, uint32_t sh) { return p + (p >> sh) * 2; }
__host__ __device__ constexpr uint32_t segments(uint32_t C, uint32_t sh) {
  return (uint32_t)(align_up(C, 64) >> sh);
}

// LDS after the staged chunk: [2-byte symbols: their low bytes] | results
// (u16 per position) | entries and counters of the tile, reused after the
// search for the parse: per segment its token masks, what comes before it and
// where it ends, and the flag bits | shared words.
__host__ __device__ constexpr uint64_t low_bytes(uint32_t C, uint32_t S) {
  return S == 2 ? align_up(C, 64) + 64 : 0;
}
__host__ __device__ constexpr uint64_t res_bytes(uint32_t C, uint32_t sh) {
  return segments(C, sh) * ((2ull << sh) + 4);
}
__host__ __device__ constexpr uint64_t area_bytes(uint32_t C, uint32_t sh, uint32_t nb) {
  const uint64_t tile = 8ull * (max_ins(nb) + kUnroll) + 4ull * kHash * row_words(nb);
  const uint64_t parse = segments(C, sh) * (8 + 4 + 4) + align_up(C, 64) / 8;
  return align_up(tile > parse ? tile : parse, 16);
}
__host__ __device__ constexpr uint64_t lds_bytes(uint32_t C, uint32_t S, uint32_t W, uint32_t wc,
                                                 uint32_t threads) {
  const uint32_t sh = seg_shift(C, threads);
  return pad_for(S, wc) + chunk_lds_bytes(C, S) + low_bytes(C, S) + align_up(res_bytes(C, sh), 16) +
         area_bytes(C, sh, window_blocks(W)) + 4 * kShared;
}

// LDS of one chunk, also enough for the split parse that takes over where the
// buckets are too full.
template <int S, int WC>
__host__ __device__ constexpr uint64_t chunk_lds(uint32_t C, uint32_t W, uint32_t threads) {
  const uint64_t a = lds_bytes(C, S, W, WC, threads), b = spec_lds_bytes<S, WC>(C);
  return a > b ? a : b;
}
// Window columns of that split parse for a window of wc columns: one variant
// for bytes, two for 2-byte symbols (one or two streaming columns).
template <int S, int WC> constexpr int kFallbackWC = S == 2 && WC <= 2 ? 2 : 4;
// Whether this encoder takes chunks of C symbols with these parameters. MIN = 1
// needs single symbols as candidates. C: the parse has a segment of at most 32
// positions for each of 256 threads.
__host__ constexpr bool takes(uint32_t C, uint32_t MIN, uint64_t lds) {
  return MIN >= 2 && C <= kMaxSyms && lds <= kMaxGroupLdsBytes;
}

__device__ __forceinline__ uint32_t hash2(uint32_t x) {
  return ((x & 0xFFFFu) * 40503u >> 9) & (kHash - 1);
}

// Position of the lowest set bit, ~0 if there is none.
__device__ __forceinline__ uint32_t first_bit(uint32_t x) {
  uint32_t r;
  asm("v_ffbl_b32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

// Four 1- or 2-byte symbols from symbol address p of the stage, and the leading
// equal symbols (0..4) of two such words.
template <int S>
__device__ __forceinline__ typename SymType<4 * S>::T load4(const uint8_t* stage, uint32_t p) {
  const uint32_t a = p * S;
  return load_run<S>(reinterpret_cast<const uint32_t*>(stage + (a & ~3u)), a & 3u);
}
template <int S>
__device__ __forceinline__ uint32_t equal4(typename SymType<4 * S>::T x,
                                           typename SymType<4 * S>::T y) {
  if constexpr (S == 1) {
    return min(first_bit(x ^ y), 32u) >> 3;
  } else {
    const uint64_t e = x ^ y;
    return min(min(first_bit((uint32_t)e), first_bit((uint32_t)(e >> 32)) | 32u), 64u) >> 4;
  }
}

// The second largest of a >= b and x.
__device__ __forceinline__ uint32_t second_of(uint32_t a, uint32_t b, uint32_t x) {
  uint32_t r;
  asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(x));
  return r;
}

// A byte of each staged 2-byte symbol: the low one if all symbols lie within 256
// of each other (then equal bytes mean equal symbols), which is returned,
// uniformly, else the high byte of a product. `shared` holds 2 words.
template <int NT>
__device__ __forceinline__ bool take_low_bytes(const uint8_t* stage, uint32_t c, uint8_t* low,
                                               uint32_t* shared) {
  const uint32_t tid = threadIdx.x;
  if (tid == 0) {
    shared[0] = 0xFFFFu;
    shared[1] = 0;
  }
  __syncthreads();
  uint32_t mn = 0xFFFFu, mx = 0;
  for (uint32_t k = 4 * tid; k < c; k += 4 * NT) {
    const uint2 v = *reinterpret_cast<const uint2*>(stage + 2 * k);
    *reinterpret_cast<uint32_t*>(low + k) = __builtin_amdgcn_perm(v.y, v.x, 0x06040200u);
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) {
      const uint32_t s = (e < 2 ? v.x : v.y) >> (16 * (e & 1)) & 0xFFFFu;
      if (k + e < c) {
        mn = min(mn, s);
        mx = max(mx, s);
      }
    }
  }
  mx = wave_max_u32(mx);
  mn = 0xFFFFu - wave_max_u32(0xFFFFu - mn);
  if (lane_id() == 0) {
    atomicMin(&shared[0], mn);
    atomicMax(&shared[1], mx);
  }
  __syncthreads();
  const bool exact = __builtin_amdgcn_readfirstlane(shared[1] - shared[0]) < 256u;
  if (__builtin_expect(!exact, 0)) {
    for (uint32_t k = 4 * tid; k < c; k += 4 * NT) {
      const uint2 v = *reinterpret_cast<const uint2*>(stage + 2 * k);
      uint32_t h = 0;
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e) {
        const uint32_t s = (e < 2 ? v.x : v.y) >> (16 * (e & 1)) & 0xFFFFu;
        h |= (s * 0x9E37u >> 8 & 0xFFu) << (8 * e);
      }
      *reinterpret_cast<uint32_t*>(low + k) = h;
    }
    __syncthreads();
  }
  return exact;
}

// The longest match of every position of the chunk into res (all waves).
// sym holds a byte of each symbol; exact: equal bytes mean equal symbols, else
// results are checked in the staged 2-byte symbols. Returns kSearched, or,
// uniformly, that a tile's buckets are so full that comparing every position
// with its window is cheaper (runs of few symbols: kFull) or that most of its
// positions have the same two bytes (kConstant).
// A position walks about 2 (nb + 1) candidates for each rank of the mean; of equal
// share among k hashes, n positions have a mean rank of kPB / 2k. From a mean of
// 16 / (nb + 1) on the streaming parse is the sooner one where few hashes hold the
// tile (few symbols) or one holds a third of it, and in launches of few chunks,
// whose 16 waves share the parse; else the tile is runs of many symbols, where
// streaming tokens end at their own offset and are searched again. Streaming
// against buckets, 16 MiB, C 4096, W 256, in us: bytes of 3 values (mean 7) 525 and
// 695; of 0 and 1, nine zeros of ten (mean 42) 524 and 3409; noise with 7 zero bytes
// of ten (mean 16) 516 and 1321; runs of up to 64 bytes (mean about 25, 80 hashes)
// 2308 and 1360; 256 KiB of such runs (C 2048, W 128) 109 and 178. 2-byte symbols
// always take the streaming parse: with the test in their kernel the compiler
// orders its loops otherwise, 1-3% slower on codes (128 MiB, C 2048: 1035 and 1052
// us), for runs 849 us instead of 2390. Above 48 (of at most 63.5) one hash holds
// nearly all.
enum SearchEnd { kSearched, kFull, kConstant };
// Whether few hashes hold the counted tile of n positions, or one a third of it
// (all waves; uniform; the shared words are free again).
template <int NT>
__device__ __forceinline__ bool tile_of_few(const uint32_t* cnt32, uint32_t row, uint32_t n,
                                            uint32_t* shared) {
  const uint32_t tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (wave < kHash / 64) {
    uint32_t sum = 0;
    for (uint32_t k = 0; k < row; ++k) sum += (cnt32[tid * row + k] & 0xFFFFu) + (cnt32[tid * row + k] >> 16);
    const uint32_t used = popc64(ballot(sum != 0)), largest = wave_max_u32(sum);
    if (lane_id() == 0) {
      shared[2 * wave] = used;
      shared[2 * wave + 1] = largest;
    }
  }
  __syncthreads();
  uint32_t hashes = 0, top = 0;
#pragma unroll
  for (uint32_t w = 0; w < kHash / 64; ++w) {
    hashes += shared[2 * w];
    top = max(top, shared[2 * w + 1]);
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(hashes < 32 || 3 * top > n);
}
template <int S, int NT>
__device__ __forceinline__ SearchEnd search(const uint8_t* stage, const uint8_t* sym, bool exact,
                                       uint32_t c, uint32_t W, uint32_t MIN, uint16_t* res,
                                       uint2* order, uint32_t* cnt32, uint32_t* shared,
                                       uint32_t seg_sh) {
  constexpr int kPer = (kMaxIns + NT - 1) / NT;
  static_assert(NT >= (int)kHash && kHash % 64 == 0, "one hash per thread");
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint16_t* cnt16 = reinterpret_cast<const uint16_t*>(cnt32);
  const uint32_t nb = window_blocks(W), row = row_words(nb);
  for (uint32_t t0 = 0; t0 < c; t0 += kTile) {
    const uint32_t lo = t0 > nb * kPB ? t0 - nb * kPB : 0u;  // first bucketed position
    const uint32_t hi = min(c - 1, t0 + kTile);        // past the last one (the chunk's last
                                                       // position starts no 2-symbol match)
    const uint32_t n = hi > lo ? hi - lo : 0u;
    for (uint32_t k = tid; k < kHash * row; k += NT) cnt32[k] = 0;
    if (tid == 0) shared[kMaxWaves] = 0;
    __syncthreads();
    uint32_t kr[kPer], x0[kPer], x1[kPer], ranks = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t r = tid + NT * i;
      if (r < n) {
        const uint32_t p = lo + r;
        const uint32_t* w = reinterpret_cast<const uint32_t*>(sym + (p & ~3u));
        const uint32_t w0 = w[0], w1 = w[1], w2 = w[2];
        x0[i] = __builtin_amdgcn_alignbyte(w1, w0, p);
        x1[i] = __builtin_amdgcn_perm(p, __builtin_amdgcn_alignbyte(w2, w1, p), 0x05040100u);
        const uint32_t key = hash2(x0[i]) * (2 * row) + r / kPB;
        const uint32_t sh = (key & 1u) * 16u;
        const uint32_t old = atomicAdd(&cnt32[key >> 1], 1u << sh);
        const uint32_t rank = (old >> sh) & 0xFFFFu;
        kr[i] = key << 16 | rank;
        ranks += rank;
      }
    }
    ranks = readlane(wave_incl_scan(ranks), 63);
    if (lane == 0) atomicAdd(&shared[kMaxWaves], ranks);
    __syncthreads();
    ranks = __builtin_amdgcn_readfirstlane(shared[kMaxWaves]);
    if (__builtin_expect(ranks * (nb + 1) > 16 * n, 0)) {
      if (S == 2 || NT == 1024 || tile_of_few<NT>(cnt32, row, n, shared))
        return ranks > 48 * n ? kConstant : kFull;
    }
    // exclusive scan of the counters, in place: one hash per thread, the
    // hashes with more than 24 entries first, then those with more than 8
    uint32_t wv[kMaxRow], sum = 0;
    if (tid < kHash) {
#pragma unroll
      for (uint32_t k = 0; k < kMaxRow; ++k) {
        wv[k] = k < row ? cnt32[tid * row + k] : 0u;
        sum += (wv[k] & 0xFFFFu) + (wv[k] >> 16);
      }
    }
    const uint32_t top = sum > 24 ? sum : sum > 8 ? sum << 16 : 0u;  // the first two classes
    const uint32_t incl = wave_incl_scan(sum), incl_top = wave_incl_scan(top);
    if (lane == 63 && wave < kHash / 64) {
      shared[2 * wave] = incl;
      shared[2 * wave + 1] = incl_top;
    }
    __syncthreads();
    if (tid < kHash) {
      uint32_t before = incl - sum, before_top = incl_top - top, all_top = 0;
#pragma unroll
      for (uint32_t w = 0; w < kHash / 64; ++w) {
        const uint32_t x = shared[2 * w], y = shared[2 * w + 1];
        before += w < wave ? x : 0u;
        before_top += w < wave ? y : 0u;
        all_top += y;
      }
      const uint32_t n0 = all_top & 0xFFFFu, n1 = all_top >> 16;
      const uint32_t b0 = before_top & 0xFFFFu, b1 = before_top >> 16;
      uint32_t run = sum > 24 ? b0 : sum > 8 ? n0 + b1 : n0 + n1 + before - b0 - b1;
#pragma unroll
      for (uint32_t k = 0; k < kMaxRow; ++k) {
        const uint32_t a = run, b = run + (wv[k] & 0xFFFFu);
        run = b + (wv[k] >> 16);
        if (k < row) cnt32[tid * row + k] = a | b << 16;
      }
    }
    if (tid < kUnroll) order[n + tid] = make_uint2(0u, 0xFFFF0000u);  // never in a window
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t r = tid + NT * i;
      if (r < n) order[cnt16[kr[i] >> 16] + (kr[i] & 0xFFFFu)] = make_uint2(x0[i], x1[i]);
    }
    __syncthreads();
    // ---- one bucketed entry per lane: walk its run of candidates. A lane
    // whose run is shorter than its wave's longest goes on past its end: any
    // position 1 to W before p is a true candidate, whatever its bucket.
    for (uint32_t i0 = 64 * wave; i0 < n; i0 += NT) {
      const uint2 x = order[min(i0 + lane, n - 1)];
      const uint32_t p = x.y >> 16, pm1 = p - 1;
      const bool query = i0 + lane < n && p >= t0;
      const uint32_t b = (p - lo) / kPB;
      const uint32_t kb = hash2(x.x) * (2 * row) + b;
      uint32_t j = cnt16[kb - min(b, nb)];
      const uint32_t steps = wave_max_u32(query ? cnt16[kb + 1] - j : 0u);
      uint32_t best = 0, next = 0;  // largest two of (8 x equal symbols) << 9 | d - 1
      for (uint32_t s = 0; s < steps; s += kUnroll, j += kUnroll) {
        const uint2* y = order + min(j, n);
#pragma unroll
        for (uint32_t u = 0; u < kUnroll; ++u) {
          const uint2 v = y[u];
          const uint32_t dm1 = pm1 - (v.y >> 16);
          // equal bits (the positions above the symbols differ somewhere, so
          // that more than kInline symbols mean kInline)
          const uint32_t eq = min(first_bit(v.x ^ x.x), first_bit(v.y ^ x.y) | 32u);
          const uint32_t key = dm1 < W ? (eq & 0x38u) << 9 | dm1 : 0u;
          next = second_of(best, next, key);
          best = max(best, key);
        }
      }
      if (query) {
        const uint32_t L = min(best >> 12, kInline), d = (best & 0x1FFu) + 1, cap = min(d, c - p);
        const bool one = L == kInline && next >> 12 < kInline && cap >= kInline;
        uint32_t r = one ? kOne | (d & 0xFFu) : L >= MIN ? L << 8 | (d & 0xFFu) : 0u;
        if (!one && L >= min(kInline, cap + 1)) r = kAny;
        if constexpr (S == 2) {
          if (!exact && L >= 2) {
            const uint16_t* a = reinterpret_cast<const uint16_t*>(stage) + p;
            bool same = true;
            for (uint32_t t = 0; t < min(L, c - p); ++t) same &= a[t] == *(a + t - d);
            if (!same) r = kAny;
          }
        }
        res[res_at(p, seg_sh)] = (uint16_t)r;
      }
    }
    if (t0 + kTile >= c && tid == 0) res[res_at(c - 1, seg_sh)] = 0;
    __syncthreads();
  }
  return kSearched;
}

// ---- match policy 1 (the paper's single window pass, see encode_chunk_scan) ------
//
// The walk of a position p goes through the window's slots from the oldest on:
// a slot unlike sym[p] is passed over, an equal one starts a run of L equal
// symbols (L at most p - w, 255 and what is left of the chunk), which counts
// if strictly longer than the best one, and the walk goes on past the slot
// where the run stopped. So only the equal slots matter: each lane first
// compares its symbol with 32 slots (two vector instructions a slot: compare,
// and shift the result into a mask), then takes the mask's bits in order. The
// step-by-step walk takes some twenty instructions a slot.
//
// For 1- and 2-byte symbols, where every sixth slot or so is equal, a second mask
// tells the slots whose next symbol matches, too, and only those are taken: a
// run of one symbol cannot win (MIN >= 2), and only passes over the slot after
// it. Of r equal slots right before a slot, all runs of one, every second one
// is such a start: the slot is passed over if r is odd.

// m = 2 m + (a == b).
template <int S>
__device__ __forceinline__ void push_equal(uint32_t& m, typename SymType<S>::T a,
                                           typename SymType<S>::T b) {
  if constexpr (S == 8) {
    asm("v_cmp_eq_u64 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc"
        : "+v"(m) : "v"(a), "v"(b) : "vcc");
  } else if constexpr (S == 4) {
    asm("v_cmp_eq_u32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc"
        : "+v"(m) : "v"(a), "v"(b) : "vcc");
  } else {
    asm("v_cmp_eq_u16 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc"
        : "+v"(m) : "v"((uint32_t)a), "v"((uint32_t)b) : "vcc");
  }
}

// Equality of x with the 32 symbols from symbol address w on (w may be before
// the chunk: the pad is read), the first in bit 31.
template <int S>
__device__ __forceinline__ uint32_t equal32(const uint8_t* stage, int32_t w,
                                            typename SymType<S>::T x) {
  using T = typename SymType<S>::T;
  uint32_t m = 0;
  if constexpr (S >= 4) {
    const T* y = reinterpret_cast<const T*>(stage) + w;
#pragma unroll
    for (uint32_t t = 0; t < 32; ++t) push_equal<S>(m, y[t], x);
  } else {
    const int32_t at = w * S;
    const uint32_t* y = reinterpret_cast<const uint32_t*>(stage + (at & ~3));
    uint32_t a = y[0];
#pragma unroll
    for (uint32_t t = 0; t < 8 * S; ++t) {  // a dword of 4 / S symbols at a time
      const uint32_t b = y[t + 1];
      const uint32_t v = __builtin_amdgcn_alignbyte(b, a, (uint32_t)at);
      a = b;
#pragma unroll
      for (uint32_t e = 0; e < 4 / S; ++e) push_equal<S>(m, (T)(v >> (8 * S * e)), x);
    }
  }
  return m;
}

// The walk of position p from slot w on, slot by slot (w = p: none).
template <int S>
__device__ __forceinline__ void scan_walk(const typename SymType<S>::T* sym, uint32_t p, uint32_t c,
                                          uint32_t w, uint32_t& bestL, uint32_t& bestd) {
  uint32_t b = p, len = 0, off = 0;
  while (w < p && b < c) {
    const bool eq = (len < kMaxMatch) & (sym[b] == sym[w]);
    off = (eq & (len == 0)) ? p - w : off;
    const bool better = !eq & (len > bestL);
    bestL = better ? len : bestL;
    bestd = better ? off : bestd;
    len = eq ? len + 1 : 0u;
    b = eq ? b + 1 : p;
    ++w;
  }
  if (len > bestL) {
    bestL = len;
    bestd = off;
  }
}

// Whether a wave walks a chunk of 1- or 2-byte symbols slot by slot: a block of 64
// positions in the middle of it (each wave its own) has more slots to take, by a
// sample of 8 in the middle of their windows, than the masks pay for, but not all
// (long runs, of which few slots are taken). 8 MiB of bytes, C 4096, W 256: of 2
// values (8 of 32 slots) 1640 us by the walk, 3140 by masks; nine zeros of ten 1577
// and 4400; of 3 values (3.6) 1716 and 1990, W 128 1056 and 1031; runs of up to 8
// (3) 810 and 693. (4- and 8-byte
// symbols: of 2 values 265 and 289, W 128 199 and 177.)
template <int S>
__device__ __forceinline__ bool slots_to_take(const uint8_t* stage, uint32_t c, uint32_t W) {
  using T = typename SymType<S>::T;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (S >= 4 || W < 32 || c < 1024) return false;
  const T* sym = reinterpret_cast<const T*>(stage) + c / 2 + 64 * wave + lane_id();
  const T* y = sym - W / 2 - 8;
  uint32_t n = 0;
#pragma unroll
  for (uint32_t e = 0; e < 8; ++e) n += popc64(ballot(y[e] == sym[0] && y[e + 1] == sym[1]));
  return n > (W > 128 ? 54u : 80u) && n < 480;  // of 64 * 8
}

// Policy-1 results of every position into res (all waves of NT threads).
template <int S, int NT>
__device__ __forceinline__ void scan_search(const uint8_t* stage, uint32_t c, uint32_t W,
                                            uint32_t MIN, uint16_t* res, uint32_t seg_sh) {
  using T = typename SymType<S>::T;
  const T* sym = reinterpret_cast<const T*>(stage);
  if (slots_to_take<S>(stage, c, W)) {
    for (uint32_t p = threadIdx.x; p < c; p += NT) {
      uint32_t bestL = 0, bestd = 0;
      scan_walk<S>(sym, p, c, p > W ? p - W : 0u, bestL, bestd);
      res[res_at(p, seg_sh)] = (uint16_t)(bestL >= MIN ? bestL << 8 | (bestd & 0xFFu) : 0u);
    }
    return;
  }
  for (uint32_t p = threadIdx.x; p - lane_id() < c; p += NT) {
    const bool in = p < c;
    const T x = sym[in ? p : 0u];
    [[maybe_unused]] typename SymType<S >= 4 ? 4 : 4 * S>::T x4{};
    [[maybe_unused]] T x1{};
    if constexpr (S <= 2) {
      x4 = load4<S>(stage, in ? p : 0u);
      x1 = (T)(x4 >> (8 * S));
    }
    const int32_t w0 = (int32_t)p - (int32_t)W;  // the oldest slot
    int32_t cur = w0 < 0 ? 0 : w0;               // the next slot to look at
    uint32_t bestL = 0, bestd = 0;
    bool on = in;
    for (uint32_t k = 0; k < W; k += 32) {
      const int32_t g = w0 + (int32_t)k;  // slot of bit 31
      const uint32_t n = min(32u, W - k);  // slots of this mask
      if (!ballot(on && cur < g + (int32_t)n)) continue;  // long runs: every lane is past it
      const uint32_t all = equal32<S>(stage, g, x);
      uint32_t m = all;
      if constexpr (S <= 2) m &= equal32<S>(stage, g + 1, x1);
      m &= (uint32_t)(~0ull << 32 >> n);  // the first n slots
      const int32_t skip = cur - g;
      if (skip > 0) m = skip >= 32 ? 0u : m & (~0u >> skip);
      if (!on) m = 0;
      // takes the run of L symbols at slot w
      auto take = [&](int32_t w, uint32_t d, uint32_t L) {
        if (L > bestL) {
          bestL = L;
          bestd = d;
        }
        cur = w + (int32_t)L + 1;
        on = L < d && p + L < c;  // else the walk has reached p or the chunk's end
        const uint32_t past = (uint32_t)(cur - g);
        m = !on || past >= 32 ? 0u : m & (~0u >> past);
      };
      // equal slots right before slot t of the mask, back to `cur` at most
      auto run_before = [&](uint32_t t) {
        const uint32_t ones = first_bit(~(uint32_t)((uint64_t)all >> (32 - t)));
        return min(ones, t - (uint32_t)min(max(cur - g, 0), (int32_t)t));
      };
      if constexpr (S >= 4) {
        while (m) {
          const int32_t w = g + __builtin_clz(m);
          const uint32_t d = p - (uint32_t)w, lim = min(min(d, kMaxMatch), c - p);
          // four symbols a step (those past the chunk are slack)
          const T* a = sym + p + 1;
          const T* b = sym + w + 1;
          uint32_t L = 1;
          while (L < lim) {
            uint32_t ne = 0;
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e) ne |= (a[e] != b[e] ? 1u : 0u) << e;
            const uint32_t same = min(first_bit(ne), 4u);
            L += same;
            if (same < 4) break;
            a += 4;
            b += 4;
          }
          take(w, d, min(L, lim));
        }
      } else {
        // runs of four symbols and more wait until every lane has one (or is
        // done), and are extended together
        bool waits = false;
        while (ballot(m != 0)) {
          const uint32_t t = m ? (uint32_t)__builtin_clz(m) : 0u;
          const int32_t w = g + (int32_t)t;
          const uint32_t d = p - (uint32_t)w, lim = min(min(d, kMaxMatch), c - p);
          if (ballot(m != 0 && !waits)) {
            if (m != 0 && !waits) {
              if (run_before(t) & 1u) {
                cur = w + 1;
                m &= ~(1u << (31 - t));
              } else {
                const uint32_t L = equal4<S>(x4, load4<S>(stage, (uint32_t)w));
                if (L == 4 && lim > 4) waits = true;
                else take(w, d, min(max(L, 1u), lim));
              }
            }
          } else if (waits) {
            uint32_t L = 4;
            while (L < lim) {
              const uint32_t e = equal4<S>(load4<S>(stage, p + L), load4<S>(stage, (uint32_t)w + L));
              L += e;
              if (e < 4) break;
            }
            take(w, d, min(L, lim));
            waits = false;
          }
        }
        // a run of one symbol at the mask's last slot passes over the next one
        cur = max(cur, g + (int32_t)(n + (run_before(n) & 1u)));
      }
    }
    if (in) res[res_at(p, seg_sh)] = (uint16_t)(bestL >= MIN ? bestL << 8 | (bestd & 0xFFu) : 0u);
  }
}

// LDS of a policy-1 chunk.
__host__ __device__ constexpr uint64_t scan_lds(uint32_t C, uint32_t S, uint32_t threads) {
  const uint32_t sh = seg_shift(C, threads);
  const uint64_t parse = segments(C, sh) * (8 + 4 + 4) + align_up(C, 64) / 8;
  return pad_for(S, 4) + chunk_lds_bytes(C, S) + align_up(res_bytes(C, sh), 16) +
         align_up(parse, 16) + 4 * kShared;
}
// Policy-1 chunks that have room for results and parse in LDS; at MIN = 1 a run
// of one symbol can win, so no slot may be passed over. 16 MiB of uint16 codes
// (C 2048, W 128) 865 us slot by slot, 505 so (615 with the one-symbol runs
// taken as well); 4 MiB of Zipf bytes (W 256) 1825 and 504; a 16 MiB float32
// field 565 and 126. Bound by vector issue: two instructions a slot and
// symbol, then the equal slots one by one.
__host__ constexpr bool takes_scan(uint32_t C, uint32_t S, uint32_t MIN, uint32_t threads) {
  return MIN >= 2 && C <= kMaxSyms && scan_lds(C, S, threads) <= kMaxGroupLdsBytes;
}

// Greedy parse from LDS results: lane g of the workgroup takes segment g. All
// segments are parsed at once, each as if a token started at its first
// position; then every segment is entered where the one before it ends, again
// and again until nothing changes. Two parses that meet at a token start agree
// from there on, so a changed entry is walked only until it meets the segment's
// earlier parse, and two or three rounds are enough. Each round settles at
// least one more segment. (One scalar walk per block of 128 positions instead:
// Zipf bytes 1341 us.)
template <int S, int WC> struct SegmentParse {
  using Sym = typename SymType<S>::T;
  const Sym* win;
  uint16_t* res;
  uint32_t c, W, MIN, seg_sh;
  uint64_t wmask[WC];
  uint32_t first, size;  // this lane's segment
  uint32_t T, P;         // token starts, pointer starts
  uint32_t exit;         // the token start past its end, in the chunk

  // Length of the match at chunk position pos with result r = kOne | d.
  __device__ __forceinline__ uint32_t extend(uint32_t pos, uint32_t r) const {
    constexpr uint32_t kStep = 8 / S;  // symbols a step
    const uint32_t d = ((r - 1) & 0xFFu) + 1;
    const uint32_t cap = min(min(d, kMaxMatch), c - pos);
    const uint8_t* b = reinterpret_cast<const uint8_t*>(win);
    uint32_t L = kInline;
    while (L < cap) {
      const uint32_t x = S * (pos + L), y = x - S * d;
      const uint32_t* xw = reinterpret_cast<const uint32_t*>(b + (x & ~3u));
      const uint32_t* yw = reinterpret_cast<const uint32_t*>(b + (y & ~3u));
      const uint32_t x1 = xw[1], y1 = yw[1];
      const uint32_t e0 = __builtin_amdgcn_alignbyte(x1, xw[0], x) ^ __builtin_amdgcn_alignbyte(y1, yw[0], y);
      const uint32_t e1 = __builtin_amdgcn_alignbyte(xw[2], x1, x) ^ __builtin_amdgcn_alignbyte(yw[2], y1, y);
      const uint32_t bits = min(min(first_bit(e0), first_bit(e1) | 32u), 64u);
      L += bits / (8 * S);
      if (bits < 64) break;
    }
    static_assert(kStep * S == 8, "whole symbols");
    return min(L, cap);
  }

  // Parses from position p of the segment (or past it) on, until its end or
  // a start of the parse so far. Called by all lanes of a wave; those with
  // `go` unset keep what they have. Lanes that come to a match to be extended
  // wait until no lane can go on without one, and extend theirs together.
  __device__ __forceinline__ void walk(bool go, uint32_t p) {
    const uint32_t lane = lane_id();
    uint32_t t = 0, q = 0, r = 0;
    bool waits = false;
    for (;;) {
      const bool on = go && !waits && p < size && !(T >> p & 1u);
      if (ballot(on)) {
        const uint32_t pos = first + p;
        if (on) r = res[res_at(pos, seg_sh)];
        uint64_t any = ballot(on && r == kAny);
        while (any) {
          const uint32_t j = (uint32_t)__builtin_ctzll(any);
          any &= any - 1;
          const uint32_t h = readlane(pos, j);
          const uint32_t key = search_token<S, WC>(win, h, c, W, MIN, wmask, lane);
          if (lane == j) {
            r = key ? (key >> 9) << 8 | (key & 0xFFu) : 0u;
            res[res_at(h, seg_sh)] = (uint16_t)r;
          }
        }
        waits |= on && r >> 8 == 1;
        if (on && !waits) {
          t |= 1u << p;
          q |= (r ? 1u : 0u) << p;
          p += max(r >> 8, 1u);
        }
        continue;
      }
      if (!ballot(waits)) break;
      if (waits) {
        const uint32_t pos = first + p, L = extend(pos, r);
        // a match shorter than MIN is a literal
        res[res_at(pos, seg_sh)] = (uint16_t)(L >= MIN ? L << 8 | (r & 0xFFu) : 0u);
        t |= 1u << p;
        q |= (L >= MIN ? 1u : 0u) << p;
        p += L >= MIN ? L : 1u;
        waits = false;
      }
    }
    if (!go) return;
    if (p < size) {  // met the parse so far
      const uint32_t rest = ~0u << p;
      T = t | (T & rest);
      P = q | (P & rest);
    } else {
      T = t;
      P = q;
      exit = first + p;
    }
  }
};

// Encodes one chunk (the same stream as enc::encode_chunk, or with kScan
// enc::encode_chunk_scan). All waves of the workgroup of NT threads take part
// throughout.
template <int S, int WC, int NT, bool kSinglePass, bool kScan = false>
__device__ __forceinline__ void encode_chunk(const ChunkJob& job, uint8_t* lds) {
  using Sym = typename SymType<S>::T;
  constexpr uint32_t kWaves = NT / 64;
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t c = __builtin_amdgcn_readfirstlane(job.c);
  uint8_t* stage = lds + pad_bytes<S, WC>();
  uint8_t* low = stage + chunk_lds_bytes(job.C, S);
  uint16_t* res = reinterpret_cast<uint16_t*>(low + (kScan ? 0 : low_bytes(job.C, S)));
  const uint32_t seg_sh = seg_shift(job.C, NT), seg = 1u << seg_sh;
  const uint32_t nb = window_blocks(job.W);
  uint8_t* area = reinterpret_cast<uint8_t*>(res) + align_up(res_bytes(job.C, seg_sh), 16);
  const uint32_t nsegC = segments(job.C, seg_sh);
  uint32_t* shared;
  if constexpr (kScan) {
    shared = reinterpret_cast<uint32_t*>(area + align_up(nsegC * 16 + align_up(job.C, 64) / 8, 16));
    stage_chunk<S>(job, stage);
    __syncthreads();
    scan_search<S, NT>(stage, c, job.W, job.MIN, res, seg_sh);
    __syncthreads();
  } else {
    uint2* order = reinterpret_cast<uint2*>(area);
    uint32_t* cnt32 = reinterpret_cast<uint32_t*>(order + max_ins(nb) + kUnroll);
    shared = reinterpret_cast<uint32_t*>(area + area_bytes(job.C, seg_sh, nb));
    stage_chunk<S>(job, stage);
    __syncthreads();
    bool exact = true;
    if constexpr (S == 2) exact = take_low_bytes<NT>(stage, c, low, shared);
    const SearchEnd end = search<S, NT>(stage, S == 2 ? low : stage, exact, c, job.W, job.MIN, res,
                                        order, cnt32, shared, seg_sh);
    if (end != kSearched) {
      __syncthreads();
      encode_chunk_spec<S, WC, kSinglePass, true>(job, lds, end == kConstant);
      return;
    }
  }

  // ---- parse
  const uint32_t nseg = (c + seg - 1) >> seg_sh;
  uint2* T = reinterpret_cast<uint2*>(area);  // token starts, pointer starts
  uint32_t* pre = reinterpret_cast<uint32_t*>(T + nsegC);  // tokens | pointers << 16 before it
  uint32_t* exits = pre + nsegC;
  uint32_t* flags = exits + nsegC;
  for (uint32_t k = tid; k < (job.C + 31) / 32; k += NT) flags[k] = 0;
  const Sym* win = reinterpret_cast<const Sym*>(stage);
  {
    SegmentParse<S, WC> sp;
    sp.win = win;
    sp.res = res;
    sp.c = c;
    sp.W = job.W;
    sp.MIN = job.MIN;
#pragma unroll
    for (int col = 0; col < WC; ++col) sp.wmask[col] = ballot(64u * col + lane + 1u <= job.W);
    sp.seg_sh = seg_sh;
    sp.first = tid << seg_sh;
    sp.size = tid < nseg ? min(seg, c - sp.first) : 0u;
    sp.T = sp.P = sp.exit = 0;
    uint32_t entry = sp.first;
    sp.walk(tid < nseg, 0);
    if (tid < nseg) exits[tid] = sp.exit;
    __syncthreads();
    for (uint32_t round = 0;; ++round) {
      uint32_t in = tid && tid < nseg ? exits[tid - 1] : entry;
      const uint32_t was = sp.exit;
      if (ballot(in != entry)) {
        sp.walk(in != entry, in - sp.first);
        entry = in;
        // tokens longer than segments settle one segment after the other: after
        // some rounds a wave settles all of its own in one
        if (kScan && round >= 4) {
          for (;;) {
            const uint32_t up = __shfl_up(sp.exit, 1);
            if (lane && tid < nseg) in = up;
            if (!ballot(in != entry)) break;
            sp.walk(in != entry, in - sp.first);
            entry = in;
          }
        }
      }
      __syncthreads();
      const bool changed = sp.exit != was;
      if (changed) exits[tid] = sp.exit;
      if (!__syncthreads_or(changed)) break;
    }
    // tokens and pointers before each segment
    const uint32_t v = __popc(sp.T) | __popc(sp.P) << 16;
    const uint32_t incl = wave_incl_scan(v);
    if (lane == 63) shared[wave] = incl;
    __syncthreads();
    uint32_t before = incl - v, all = 0;
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) {
      const uint32_t x = shared[w];
      before += w < wave ? x : 0u;
      all += x;
    }
    if (tid < nseg) {
      T[tid] = make_uint2(sp.T, sp.P);
      pre[tid] = before;
    }
    if (tid == 0) shared[kMaxWaves] = all;
  }
  __syncthreads();
  const uint32_t all = __builtin_amdgcn_readfirstlane(shared[kMaxWaves]);
  const uint32_t ntok = all & 0xFFFFu, nptr = all >> 16;
  const uint32_t F = (ntok + 7) / 8, P = S * (ntok - nptr) + 2 * nptr;
  const RecordPlace rec = place_record<kSinglePass>(job, F, P, shared + kMaxWaves + 4);
  if (!rec.ok) return;

  // ---- encode: one position per lane; flag bits are collected in LDS
  for (uint32_t p = tid; p < c; p += NT) {
    const uint32_t g = p >> seg_sh, bit = p & (seg - 1), below = (1u << bit) - 1u;
    const uint2 m = T[g];
    const uint32_t before = pre[g];
    const uint32_t rank = (before & 0xFFFFu) + __popc(m.x & below);
    const uint32_t np = (before >> 16) + __popc(m.y & below);
    uint8_t* dst = rec.payload + (S * (rank - np) + 2 * np);
    if (m.y >> bit & 1u) {
      const uint32_t r = res[res_at(p, seg_sh)];
      const uint16_t v = (uint16_t)(r >> 8 | r << 8);
      __builtin_memcpy(dst, &v, 2);
      atomicOr(&flags[rank >> 5], 1u << (rank & 31u));
    } else if (m.x >> bit & 1u) {
      const Sym v = win[p];
      __builtin_memcpy(dst, &v, S);
    }
  }
  __syncthreads();
  const uint8_t* fb = reinterpret_cast<const uint8_t*>(flags);
  for (uint32_t k = tid; k < F; k += NT) rec.flags[k] = fb[k];
}

}  // namespace bucket
}  // namespace enc
}  // namespace gpulz
