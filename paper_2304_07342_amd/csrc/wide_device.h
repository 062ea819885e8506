// Chunk sizing for 4- and 8-byte symbols with MIN >= 2: pointers are looked for
// only where a pair of symbols repeats, found by hashing instead of comparing
// every position with its window.
#pragma once

#include "encode_device.h"

namespace gpulz {
namespace enc {
namespace wide {

// A match of MIN >= 2 symbols starts at p only if the pair (sym[p], sym[p + 1])
// also stands at an earlier position. Repeated pairs are found by hashing the
// whole chunk: every pair sets its bit in a bitmap, and a pair that finds it set
// sets that bit in a second one; pairs whose bit is in the second bitmap go
// into the next round, with another hash and a smaller bitmap. Equal pairs
// stay together in every round, chance collisions shrink (4096 pairs: about
// 250 after the first round, 8, 0), so that a chunk of noisy data is known to be
// all literals after three rounds, without having been staged. Other chunks are
// staged, and their candidates searched exactly. Candidates of any distance are
// kept (the search decides), so the window does not matter here.
//
// 256 MiB float32 field (C 4096, W 256): 508 us with every second position
// compared with its window in look-back order; 197 us with these sizes (105-117),
// the scan (5) and the records written at copy rate (88). 100 MB of float64 104 and
// 77, 1 MiB of float32 26 and 10. A chunk takes 35 vector and 22 scalar
// instructions and 4.7 LDS accesses, most of them scattered atomics, per 64 positions
// (W / 2 vector and as many scalar ones with the window comparison); the vector
// units are busy half the time.
constexpr uint32_t kMaxVectors = 8;       // 16-byte vectors a thread of 256 holds, at most
constexpr uint32_t kMaxBytes = 16 * kMaxVectors * 256;  // largest chunk
constexpr uint32_t kBits = 1u << 16;      // first round
constexpr uint32_t kSmallBits = 1u << 13;  // later rounds
constexpr uint32_t kListMax = 1024;       // pairs in question after a round
constexpr uint32_t kKeep = 128;           // candidates handed to the searches
constexpr uint32_t kCounts = 8;           // shared words before a count per wave
constexpr uint32_t kKeepAt = kCounts + kSpecWaves;
constexpr uint32_t kShared = kKeepAt + kKeep / 2;  // shared words, then the candidates
constexpr uint32_t kRepetitive = ~0u;

// LDS: the bitmaps of the first round (after it the lists and the small bitmaps
// lie in the first of them), overlaid by the staged chunk with its hit bitmap
// and candidate list, or with what the split parse needs; then the shared words.
// (Bitmaps scaled with C leave more pairs in question: 100 MiB of sorted uint32,
// C 2048: 96 us, 88 so; 4 MiB, C 256: 38 and 36.)
__host__ __device__ constexpr uint64_t area_bytes(uint32_t C, uint32_t S, uint32_t wc) {
  const uint64_t e = align_up(encode_lds(C, S, wc, kEncodeWaves), 16), b = 2 * kBits / 8;
  return e > b ? e : b;
}
__host__ __device__ constexpr uint64_t lds_bytes(uint32_t C, uint32_t S, uint32_t wc) {
  return area_bytes(C, S, wc) + 4 * kShared;
}
__host__ __device__ constexpr bool takes(uint32_t C, uint32_t S, uint32_t MIN) {
  return S >= 4 && MIN >= 2 && (uint64_t)C * S <= kMaxBytes;
}
// Launches of few chunks: 16 waves a chunk, and the split parse for chunks of
// repeating pairs (if it takes chunks of C symbols): 64 chunks of uint32 out of
// 16 values (C 4096) 1484 us with one wave's parse, 217 so; of a half-zero field
// 341 and 89.
constexpr uint32_t kFewThreads = 64 * kSpecWaves;
template <int S, int WC>
__host__ __device__ constexpr uint64_t few_area_bytes(uint32_t C) {
  const uint64_t a = area_bytes(C, S, WC), b = align_up(spec_lds_bytes<S, WC>(C), 16);
  return C <= kSpecMaxSyms && b > a ? b : a;
}

// 16-bit hash of the pair (a, b) for round r: 24-bit multiplies (full rate),
// with the high bits folded in, as integers may differ in them only.
template <int S>
__device__ __forceinline__ uint32_t hash_pair(typename SymType<S>::T a, typename SymType<S>::T b,
                                              uint32_t r) {
  auto m24 = [](uint32_t x, uint32_t k) { return (x & 0xFFFFFFu) * k; };
  const uint32_t k0 = r == 0 ? 0x9E3779u : r == 1 ? 0x165667u : 0xBF5847u;
  const uint32_t k1 = r == 0 ? 0x85EBCBu : r == 1 ? 0xD3A265u : 0x6C8E95u;
  uint32_t h;
  if constexpr (S == 4) {
    h = m24(a ^ a >> 11, k0) + m24(b ^ b >> 11, k1);
  } else {
    const uint32_t al = (uint32_t)a, ah = (uint32_t)(a >> 32);
    const uint32_t bl = (uint32_t)b, bh = (uint32_t)(b >> 32);
    h = m24(al ^ ah >> 11, k0) + m24(ah ^ al >> 13, 0xC2B2AFu) + m24(bl ^ bh >> 11, k1) +
        m24(bh ^ bl >> 13, 0x27D4EBu);
  }
  return h >> 16;
}

// Sets bit h of `seen`, and of `twice` if it was set.
__device__ __forceinline__ void mark(uint32_t* seen, uint32_t* twice, uint32_t h) {
  const uint32_t b = 1u << (h & 31u);
  if (atomicOr(&seen[h >> 5], b) & b) atomicOr(&twice[h >> 5], b);
}
__device__ __forceinline__ bool marked(const uint32_t* twice, uint32_t h) {
  return twice[h >> 5] >> (h & 31u) & 1u;
}

// Candidate positions of the chunk at src (c symbols, at most kVectors 16-byte
// vectors per thread), whole workgroup: their number, with the positions in
// keep[], or kRepetitive if too many pairs repeat. Uniform. kRuns: runs of one
// symbol, which set one bit over and over, one lane after the other, are told
// from the first vectors: where a quarter of their pairs are such, the chunk is
// not hashed (256 KiB of uint64 half zero: 68.8 us, 74.4 hashed).
template <int S, uint32_t kVectors, uint32_t kThreads, bool kRuns>
__device__ __forceinline__ uint32_t candidates(const uint8_t* src, uint32_t c, uint8_t* area,
                                               uint32_t* shared, uint16_t* keep) {
  using T = typename SymType<S>::T;
  constexpr uint32_t V = 16 / S;
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t n = c - 1;  // pairs
  const T* sym = reinterpret_cast<const T*>(src);
  uint32_t* seen = reinterpret_cast<uint32_t*>(area);
  uint32_t* twice = seen + kBits / 32;
  uint16_t* list = reinterpret_cast<uint16_t*>(area);  // two lists of kListMax
  uint32_t* small = reinterpret_cast<uint32_t*>(list + 2 * kListMax);
  // ---- first round: V consecutive pairs per vector, hashes kept two a word
  T v[kVectors][V + 1];
#pragma unroll
  for (uint32_t k = 0; k < kVectors; ++k) {
    const uint32_t p = V * (tid + kThreads * k);
    if (p + V < c) {
      __builtin_memcpy(v[k], sym + p, 16);
      v[k][V] = sym[p + V];
    } else {
#pragma unroll
      for (uint32_t e = 0; e <= V; ++e) v[k][e] = p + e < c ? sym[p + e] : T(0);
    }
  }
  for (uint32_t k = tid; k < 2 * kBits / 128; k += kThreads)
    reinterpret_cast<uint4*>(area)[k] = make_uint4(0, 0, 0, 0);
  if (tid < 4) shared[tid] = 0;
  if constexpr (kRuns) {
    uint32_t same = 0;
#pragma unroll
    for (uint32_t e = 0; e < V; ++e) same += popc64(ballot(V * tid + e < n && v[0][e] == v[0][e + 1]));
    if (lane == 0) shared[kCounts + (tid >> 6)] = same;
  }
  __syncthreads();
  if constexpr (kRuns) {
    uint32_t same = 0;
#pragma unroll
    for (uint32_t w = 0; w < kThreads / 64; ++w) same += shared[kCounts + w];
    if (n && 4 * uniform(same) >= min(n, V * kThreads)) return kRepetitive;
  }
  uint32_t hs[kVectors][V / 2];
#pragma unroll
  for (uint32_t k = 0; k < kVectors; ++k) {
    const uint32_t p = V * (tid + kThreads * k);
    const bool whole = V * kThreads * (k + 1) <= n;  // uniform: every lane's pairs exist
#pragma unroll
    for (uint32_t e = 0; e < V; ++e) {
      const uint32_t h = hash_pair<S>(v[k][e], v[k][e + 1], 0);
      if (e % 2 == 0) hs[k][e / 2] = h;
      else hs[k][e / 2] |= h << 16;
      if (whole || p + e < n) mark(seen, twice, h);
    }
  }
  __syncthreads();
  uint32_t mine = 0;  // bit V k + e: pair e of vector k is in question
#pragma unroll
  for (uint32_t k = 0; k < kVectors; ++k) {
    const uint32_t p = V * (tid + kThreads * k);
    const bool whole = V * kThreads * (k + 1) <= n;
#pragma unroll
    for (uint32_t e = 0; e < V; ++e) {
      const uint32_t h = e % 2 ? hs[k][e / 2] >> 16 : hs[k][e / 2] & 0xFFFFu;
      const uint32_t bit = (uint32_t)marked(twice, h);
      mine |= (whole || p + e < n ? bit : 0u) << (V * k + e);
    }
  }
  {
    const uint32_t cnt = (uint32_t)__popc(mine), incl = wave_incl_scan(cnt);
    const uint32_t all = readlane(incl, 63);
    uint32_t base = 0;
    if (lane == 0 && all) base = atomicAdd(&shared[0], all);
    uint32_t at = readlane(base, 0) + incl - cnt;
    // (the lists lie in `seen`, which the marks above no longer touch)
    for (uint32_t m = mine; m; m &= m - 1, ++at) {
      const uint32_t b = (uint32_t)__builtin_ctz(m);
      if (at < kListMax) list[at] = (uint16_t)(V * (tid + kThreads * (b / V)) + b % V);
    }
  }
  for (uint32_t k = tid; k < 2 * kSmallBits / 32; k += kThreads) small[k] = 0;
  __syncthreads();
  uint32_t left = uniform(shared[0]);
  if (left > kListMax) return kRepetitive;
  // ---- later rounds: one pair of the list per thread at a time
#pragma unroll 1
  for (uint32_t r = 1; r <= 2 && left; ++r) {
    uint32_t* seen2 = small;
    uint32_t* twice2 = small + kSmallBits / 32;
    const uint16_t* from = list + (r - 1) * kListMax;
    uint16_t* to = r == 1 ? list + kListMax : keep;
    const uint32_t cap = r == 1 ? kListMax : kKeep;
    for (uint32_t k = tid; k < left; k += kThreads) {
      const uint32_t p = from[k];
      mark(seen2, twice2, hash_pair<S>(sym[p], sym[p + 1], r) % kSmallBits);
    }
    __syncthreads();
    for (uint32_t k = tid; k < left; k += kThreads) {
      const uint32_t p = from[k];
      if (marked(twice2, hash_pair<S>(sym[p], sym[p + 1], r) % kSmallBits)) {
        const uint32_t at = atomicAdd(&shared[r], 1u);
        if (at < cap) to[at] = (uint16_t)p;
      }
    }
    __syncthreads();
    left = uniform(shared[r]);
    if (left > cap) return kRepetitive;
    if (r == 1 && left) {
      for (uint32_t k = tid; k < 2 * kSmallBits / 32; k += kThreads) small[k] = 0;
      __syncthreads();
    }
  }
  return left;
}

// Sizes of a chunk's record, and whether it has pointers.
struct Sized {
  uint32_t F, P;
  bool pointers;
};

// Whether a chunk is nearly one long run: fewer than one symbol in 128 differs
// from the one before it, and the window lets a token cover so many. Its few
// long tokens are sooner found by one wave than by 16 (zero uint32 symbols, C
// 4096, W 256: 659 and 828 us; W 32: 356 and 54). Whole workgroup, uniform.
template <int S, uint32_t kThreads>
__device__ __forceinline__ bool one_run(const ChunkJob& job, uint32_t* shared) {
  using T = typename SymType<S>::T;
  if (job.W <= 128) return false;
  const T* sym = reinterpret_cast<const T*>(job.src);
  uint32_t turns = 0;
  for (uint32_t k = threadIdx.x + 1; k - lane_id() < job.c; k += kThreads)
    turns += popc64(ballot(k < job.c && sym[k] != sym[k - 1]));
  if (lane_id() == 0) shared[kCounts + (threadIdx.x >> 6)] = turns;
  __syncthreads();
  turns = 0;
#pragma unroll
  for (uint32_t w = 0; w < kThreads / 64; ++w) turns += shared[kCounts + w];
  return 128 * uniform(turns) < job.c;
}

// Sizes one chunk, whole workgroup of kThreads; a record with pointers is written
// to the chunk's slot, others are their flag zeros and the chunk itself. The
// result is wave 0's: once the parse is its work alone the other waves leave.
// kRuns: see candidates() (streams of many chunks go without: a long one of
// noisy data pays 3% for it, and one of runs gains nothing).
template <int S, int WC, uint32_t kVectors, uint32_t kThreads, bool kRuns>
__device__ __forceinline__ Sized size_chunk(ChunkJob job, uint8_t* lds) {
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr bool kFew = kThreads == kFewThreads;
  constexpr uint32_t kWaves = kThreads / 64;
  const uint32_t c = job.c;
  uint32_t* shared = reinterpret_cast<uint32_t*>(
      lds + (kFew ? few_area_bytes<S, WC>(job.C) : area_bytes(job.C, S, WC)));
  uint16_t* keep = reinterpret_cast<uint16_t*>(shared + kKeepAt);
  const Sized literals = {(c + 7) / 8, c * S, false};
  const uint32_t ncand = candidates<S, kVectors, kThreads, kRuns>(job.src, c, lds, shared, keep);
  if (ncand == 0) return literals;
  __syncthreads();
  const bool sampled = ncand == kRepetitive;
  if constexpr (kFew) {
    if (sampled && job.C <= kSpecMaxSyms && !one_run<S, kThreads>(job, shared)) {
      job.sizes = shared;
      encode_chunk_spec<S, WC, false>(job, lds);
      return {shared[0], shared[1], true};
    }
  }
  uint8_t* stage = lds + pad_bytes<S, WC>();
  uint32_t* hits = reinterpret_cast<uint32_t*>(stage + chunk_lds_bytes(job.C, S));
  const uint32_t nhw = (uint32_t)hit_words(job.C, S);
  uint32_t* list = hits + nhw;
  stage_chunk<S>(job, stage);
  for (uint32_t k = tid; k < nhw; k += kThreads) hits[k] = 0;
  __syncthreads();
  if (sampled) {  // the window comparison of every second position
    constexpr uint32_t kBlock = Geo<S>::kBlock;
    build_hits<S, WC>(stage, wave, (c + kBlock - 1) / kBlock, kWaves, job.W, c, true, hits);
  } else if (tid < ncand) {
    atomicOr(&hits[keep[tid] >> 5], 1u << (keep[tid] & 31u));
  }
  __syncthreads();
  uint64_t wmask[WC];
#pragma unroll
  for (int col = 0; col < WC; ++col) wmask[col] = ballot(64u * col + lane + 1u <= job.W);
  const bool listed = build_list<S, WC>(stage, hits, nhw, sampled, job, wmask, list, wave,
                                        kEncodeWaves);
  if (wave != 0) return literals;
  if (listed) {  // no search found a match: literals only
    const uint32_t* key = list + kEncodeWaves * kListPerWave;
    const uint32_t* cnt = key + kEncodeWaves * kListPerWave;
    bool any = false;
    for (uint32_t w = 0; w < kEncodeWaves; ++w)
      any |= lane < cnt[w] && key[w * kListPerWave + lane] != 0;
    if (ballot(any) == 0) return literals;
  }
  const Parsed r = parse_chunk<S, WC, false>(job, stage, hits, nhw, sampled, false, listed, list,
                                             wmask, kEncodeWaves);
  return {(r.ntok + 7) / 8, r.pay, true};
}

// Writes a chunk's record, whole workgroup: the table entry, the flag bytes and
// the payload, from the chunk itself (src) if it has no pointer, else from the
// slot. in_end: end of the input (no dword that reaches it is read).
__device__ __forceinline__ void put_record(const uint8_t* src, const uint8_t* in_end,
                                           const uint8_t* slot, uint64_t flag_area, const Sized& z,
                                           uint8_t* table, uint8_t* rec, uint32_t tid,
                                           uint32_t nthreads) {
  // (through values of their own: a choice between the members was compiled as one
  // between their addresses, for which every workgroup read the launch packet in
  // host memory: 4 MiB of float32 17.5 us, 4 so)
  const uint32_t F = z.F, P = z.P;
  const uint32_t e = tid < 4 ? F : P;
  if (tid < 8) table[tid] = (uint8_t)(e >> (8 * (tid & 3u)));
  if (z.pointers) {
    stream::copy_bytes(rec, slot, z.F, tid, nthreads);
    stream::copy_bytes(rec + z.F, slot + flag_area, z.P, tid, nthreads);
  } else {
    stream::fill_zero(rec, z.F, tid, nthreads);
    stream::copy_unaligned(rec + z.F, src, z.P, in_end, tid, nthreads);
  }
}

}  // namespace wide
}  // namespace enc
}  // namespace gpulz
