// Device code of the decoder, shared by the single-buffer and batch kernels.
//
// The paper states that decompression exists and is easy to parallelise
// (section 4.4) without describing it; this decoder follows from the stream
// layout:
//   header   one thread checks every header field;
//   table    the table's F_i + P_i are prefix-summed once per group of 64
//            chunks (one u64 per group; the sum must end exactly at the
//            stream's end); a chunk's record offset is its group's offset
//            plus a 64-lane prefix sum over the group's table entries;
//   chunk    (all literals: F and P say so and the flag bytes are zero) copied
//            from the stream to the output;
//   chunk    (4- and 8-byte symbols, or few chunks; at most 4096 symbols and
//            16 KiB) one workgroup of 256 threads per chunk: the record is staged into
//            LDS with 16-byte loads; block-wide scans over the flag bits and
//            the token lengths give every token's payload offset and output
//            position at once, every rule is checked and the literals are
//            written into an LDS copy of the chunk; wave 0 then copies the
//            pointers in token order (a run of pointers whose sources are
//            already final is copied together), and the chunk is written to
//            HBM with 16-byte stores;
//   chunk    (1- and 2-byte symbols in many chunks, and longer chunks) one
//            wavefront walks the tokens 64 at a time: lane l takes token t + l,
//            its flag bit gives its kind,
//            mbcnt over the literal / pointer ballots its payload offset, a
//            wave scan of the token lengths its output position. Literals are
//            written into an LDS ring of recent symbols; then the new symbols
//            are taken 64 at a time, one per lane: a pointer's symbol follows
//            its source back to a literal or out of the 64, in registers, and
//            copies it. Finished symbols stream out to HBM; the next tokens'
//            payload is loaded meanwhile. The ring keeps the last 256 symbols
//            (the largest offset), so LDS use does not depend on the chunk size.
// Every rule the encoder guarantees is checked; a broken one makes the
// stream GPULZ_ERR_CORRUPT.
#pragma once

#include "gpulz_internal.h"
#include "stream_device.h"
#include "wave.h"

namespace gpulz {
namespace dec {

constexpr uint32_t kGroup = 64;  // chunks per record-offset group

// Checks the header of a stream of in_bytes bytes (16-byte aligned, as every
// entry point requires); fills p (p.status = kOk or kCorrupt). One thread; the
// header is four 16-byte loads in flight together, its fields register words.
__device__ inline void parse_header(const uint8_t* h, uint64_t in_bytes, DecodeParams& p) {
  p = DecodeParams{};
  bool ok = in_bytes >= kHeaderBytes;
  if (ok) {
    uint4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = reinterpret_cast<const uint4*>(h)[k];
    const uint32_t w[16] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w,
                            v[2].x, v[2].y, v[2].z, v[2].w, v[3].x, v[3].y, v[3].z, v[3].w};
    ok = w[0] == 0x315A4C47u &&            // "GLZ1"
         (w[1] & 0xFFFFu) == 1u &&         // version
         w[1] >> 24 <= 1u &&               // match policy 0 or 1
         w[3] >> 24 == kMaxMatch;
    p.S = w[1] >> 16 & 0xFFu;
    p.C = w[2];
    p.W = w[3] & 0xFFFFu;
    p.MIN = w[3] >> 16 & 0xFFu;
    p.n = (uint64_t)w[5] << 32 | w[4];
    p.N = (uint64_t)w[7] << 32 | w[6];
    const uint64_t total = (uint64_t)w[9] << 32 | w[8];
    p.r = (uint16_t)(w[10] & 0xFFu);
    ok = ok && (p.S == 1 || p.S == 2 || p.S == 4 || p.S == 8) && p.C >= 1 && p.C <= (1u << 24) &&
         p.W >= 1 && p.W <= kMaxWindow && p.MIN >= 1;
    if (ok) {
      p.m = p.n / p.S;
      ok = p.r == p.n % p.S && p.N == (p.m + p.C - 1) / p.C && total == in_bytes &&
           p.N <= decode_max_chunks(in_bytes);
      // bytes 41..47 are zero, and those of 48..63 past the r tail bytes
      const uint64_t tail = (uint64_t)w[13] << 32 | w[12];
      ok = ok && w[10] >> 8 == 0 && w[11] == 0 && w[14] == 0 && w[15] == 0 &&
           (p.r >= 8 || tail >> (8 * p.r) == 0);
    }
  }
  p.status = ok ? kOk : kCorrupt;
}

// Workgroup-wide: group_off[g] = absolute offset of the first record of chunk
// group g (g = 0 .. ceil(N / 64)); returns the end of the last record. Any
// blockDim that is a multiple of 64. `scratch` holds blockDim/64 + 1 u64.
__device__ inline uint64_t scan_table_groups(const uint8_t* in, uint64_t N, uint64_t* group_off,
                                             uint64_t* scratch) {
  // each thread sums 16 consecutive entries (eight 16-byte loads; the table
  // starts 16-byte aligned), so 4 threads cover a group of 64; one block-wide
  // scan per tile of 16 blockDim entries gives every group's offset
  constexpr uint32_t kPer = 16;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
  const uint32_t nw = blockDim.x >> 6;
  const uint64_t ngroups = (N + kGroup - 1) / kGroup;
  const uint8_t* table = in + kHeaderBytes;
  const uint4* t4 = reinterpret_cast<const uint4*>(table);
  const uint64_t tile = (uint64_t)blockDim.x * kPer;
  uint64_t carry = kHeaderBytes + 8 * N;
  for (uint64_t base = 0; base < N; base += tile) {
    const uint64_t i0 = base + (uint64_t)tid * kPer;
    uint64_t v = 0;
    if (i0 + kPer <= N) {
#pragma unroll
      for (uint32_t q = 0; q < kPer / 2; ++q) {
        const uint4 e = t4[i0 / 2 + q];
        v += (uint64_t)e.x + e.y + (uint64_t)e.z + e.w;
      }
    } else {
      for (uint32_t k = 0; k < kPer && i0 + k < N; ++k) {
        const uint32_t* e = reinterpret_cast<const uint32_t*>(table + 8 * (i0 + k));
        v += (uint64_t)e[0] + e[1];
      }
    }
    const uint64_t incl = wave_incl_scan_u64(v);
    if (lane == 63) scratch[wid] = incl;
    __syncthreads();
    uint64_t before = 0, total = 0;
    for (uint32_t w = 0; w < nw; ++w) {
      const uint64_t x = scratch[w];
      before += w < wid ? x : 0ull;
      total += x;
    }
    // i0 is a multiple of 64 exactly on every fourth thread
    if ((tid & 3u) == 0 && i0 < N) group_off[i0 / kGroup] = carry + before + incl - v;
    carry += total;
    __syncthreads();
  }
  if (tid == 0) group_off[ngroups] = carry;
  return carry;
}

// Wave-wide: absolute record offset of chunk i.
__device__ inline uint64_t record_offset(const uint8_t* in, const uint64_t* group_off, uint64_t i) {
  const uint32_t lane = lane_id();
  const uint64_t g = i / kGroup;
  const uint32_t k = (uint32_t)(i % kGroup);
  uint64_t v = 0;
  if (lane < k) {
    const uint32_t* e = reinterpret_cast<const uint32_t*>(in + kHeaderBytes + 8 * (g * kGroup + lane));
    v = (uint64_t)e[0] + e[1];
  }
  const uint64_t s = wave_incl_scan_u64(v);
  return group_off[g] + __shfl(s, 63, 64);
}

// ---- wave decoder -----------------------------------------------------------

constexpr uint32_t kRingSyms = 1024;  // symbols of a wave's ring
constexpr uint32_t kFlushSyms = 256;  // symbols written out at once
// Symbols a step may add, up to 254 more for the last token's end: what is not
// written out yet (below kFlushSyms) or may be a source (the last 256) and the
// new ones fit the ring.
constexpr uint32_t kSpanSyms = kRingSyms - kFlushSyms - kMaxMatch - 1;
constexpr uint32_t kStepSyms = kSpanSyms + 256;  // symbols of a step, at most
constexpr uint32_t kFewPointers = 8;  // a lone wave copies so many one by one
constexpr uint32_t kShortFill = 8;  // longer pointers' offsets are laid out by all lanes
template <int S> struct WaveLds {
  typename SymType<S>::T ring[kRingSyms];
  uint16_t off[kStepSyms];  // offset of each new symbol's pointer, 0 for a literal
};

// 8 bytes of [p, end) from byte 8 k on (zeros past the end), any alignment.
__device__ __forceinline__ uint64_t load_bytes8(const uint8_t* p, uint32_t k, uint32_t n) {
  uint64_t v = 0;
  if (8 * k + 8 <= n) {
    __builtin_memcpy(&v, p + 8 * k, 8);
  } else {
    for (uint32_t b = 8 * k; b < n; ++b) v |= (uint64_t)p[b] << (8 * (b - 8 * k));
  }
  return v;
}

// Decode one chunk of c symbols with one wavefront; returns false (uniformly)
// if it breaks a rule. `flags` is the record (F flag bytes, then P payload
// bytes; no byte past them is read). kAlone: the wave is one of few on its compute
// unit, so the chain of a round's steps counts: a round of few pointers copies
// them one after the other (with all wave slots taken that form costs more than
// it saves).
template <int S, bool kAlone>
__device__ bool decode_chunk_wave(const uint8_t* flags, uint32_t F, uint32_t P, uint32_t c,
                                  uint32_t W, uint32_t MIN, uint8_t* dst, uint8_t* lds_bytes) {
  using T = typename SymType<S>::T;
  using V = typename SymType<S == 8 ? 8 : 4>::T;  // holds a token's payload
  WaveLds<S>& lds = *reinterpret_cast<WaveLds<S>*>(lds_bytes);
  T* const out = reinterpret_cast<T*>(dst);
  T* const ring = lds.ring;
  constexpr uint32_t M = kRingSyms - 1;
  const uint32_t lane = lane_id();
  if (F > (c + 7) / 8) return false;  // more tokens than symbols
  const uint8_t* pay = flags + F;
  const bool wide = ((uintptr_t)out & 15u) == 0;
  const uint32_t rounds = (F + 7) / 8;
  uint32_t q = 0;        // symbols decoded
  uint32_t done = 0;     // symbols written out
  uint32_t t = 0, u = 0;  // tokens taken, their payload bytes
  uint64_t fw = 0;       // flag words of 64 rounds, one per lane

  // this lane's payload at offset `off` (0 if it does not end in the payload):
  // 2 bytes of a pointer, S of a literal, in the lower bits
  auto payload = [&](bool has, bool ptr, uint32_t off) -> V {
    V v = 0;
    if (S >= 4 && has && !ptr) {
      if (off + S <= P) __builtin_memcpy(&v, pay + off, S);
    } else if (has && off + 2 <= P) {
      uint16_t x;
      __builtin_memcpy(&x, pay + off, 2);
      v = x;
    } else if (S == 1 && has && off < P) {
      v = pay[off];
    }
    return v;
  };
  auto flush = [&](uint32_t n) {  // writes out symbols [done, done + n)
    if (S <= 2 && wide && n == kFlushSyms) {  // four symbols per lane
      using Quad = typename SymType<S <= 2 ? 4 * S : S>::T;
      reinterpret_cast<Quad*>(out + done)[lane] = reinterpret_cast<const Quad*>(ring + (done & M))[lane];
    } else {
      for (uint32_t k = lane; k < n; k += 64) out[done + k] = ring[(done + k) & M];
    }
    done += n;
  };

  uint64_t pm_next = 0;
  V v_next = 0;
  uint32_t off_next = 0, u_next = 0;
  for (uint32_t r = 0; r <= rounds; ++r) {
    const uint64_t pm = pm_next;
    const V v = v_next;
    const uint32_t off = off_next;
    const uint32_t base = 64 * (r - 1);  // this round's first token (r >= 1)
    if (r < rounds) {  // the next round's flags and payload
      if ((r & 63u) == 0) fw = 8 * (r + lane) < F ? load_bytes8(flags, r + lane, F) : 0ull;
      pm_next = (uint64_t)readlane((uint32_t)(fw >> 32), r & 63u) << 32 |
                readlane((uint32_t)fw, r & 63u);
      const uint32_t left = 8 * F - 64 * r;  // tokens the flags can still describe
      const uint64_t hm = left >= 64 ? ~0ull : (1ull << left) - 1ull;
      const uint64_t lm = hm & ~pm_next;
      off_next = u_next + S * mbcnt(lm) + 2u * mbcnt(pm_next);
      v_next = payload(hm >> lane & 1, pm_next >> lane & 1, off_next);
      u_next += S * popc64(lm) + 2u * popc64(pm_next);
    }
    if (r == 0) continue;

    const uint32_t left = 8 * F - base;
    const bool has = lane < left;
    const bool ptr = pm >> lane & 1;
    const uint32_t sz = ptr ? 2u : (uint32_t)S;
    const uint32_t L = ptr ? (uint32_t)v & 0xFFu : 1u;
    const uint32_t O = ptr ? (((uint32_t)v >> 8) - 1u & 0xFFu) + 1u : 1u;
    const uint32_t len = has ? L : 0u;
    const uint32_t incl = wave_incl_scan(len);
    const uint32_t pos = q + incl - len;
    const uint32_t total = readlane(incl, 63);
    const uint64_t tm = ballot(has && pos < c);  // tokens of the chunk (a prefix)
    bool bad = off + sz > P;
    if (ptr) bad = bad || L < MIN || O > W || O > pos || L > O || pos + L > c;
    if (ballot((tm >> lane & 1) && bad)) return false;
    if (tm == 0) break;  // the chunk was complete before this round
    uint64_t todo = tm;
    if (kAlone && total <= kSpanSyms && popc64(tm & pm) <= kFewPointers) {
      if ((tm & ~pm) >> lane & 1) ring[pos & M] = (T)v;
      for (uint64_t m = tm & pm; m; m &= m - 1) {
        const uint32_t j = (uint32_t)__builtin_ctzll(m);
        const uint32_t pj = readlane(pos, j), Lj = readlane(L, j), Oj = readlane(O, j);
        wave_sync();
        for (uint32_t k = lane; k < Lj; k += 64) ring[(pj + k) & M] = ring[(pj - Oj + k) & M];
      }
      q = tm & pm ? readlane(pos + len, 63u - (uint32_t)__builtin_clzll(tm)) : q + popc64(tm);
      todo = 0;
      if (q - done >= kFlushSyms) {
        wave_sync();
        while (q - done >= kFlushSyms) flush(kFlushSyms);
      }
    }
    // usually one step; a round of long pointers takes several
    while (todo) {
      uint64_t now = todo;
      if (total > kSpanSyms) now = ballot((todo >> lane & 1) && pos < q + kSpanSyms);
      const bool mine = now >> lane & 1;
      const uint32_t at = pos - q;
      if (mine) lds.off[at] = (uint16_t)(ptr ? O : 0u);
      if (mine && !ptr) ring[pos & M] = (T)v;
      const bool fill = mine && ptr;
      for (uint32_t k = 1; ballot(fill && L <= kShortFill && k < L); ++k)
        if (fill && L <= kShortFill && k < L) lds.off[at + k] = (uint16_t)O;
      uint64_t big = ballot(fill && L > kShortFill);
      while (big) {
        const uint32_t j = (uint32_t)__builtin_ctzll(big);
        big &= big - 1;
        const uint32_t aj = readlane(at, j), Lj = readlane(L, j), Oj = readlane(O, j);
        for (uint32_t k = lane; k < Lj; k += 64) lds.off[aj + k] = (uint16_t)Oj;
      }
      wave_sync();
      const uint32_t last = 63u - (uint32_t)__builtin_clzll(now);
      const uint32_t n = readlane(pos + len, last) - q;  // new symbols
      for (uint32_t b = 0; b < n; b += 64) {
        // sources relative to this lane's 64 symbols: negative ones are final,
        // a literal is its own source; each step replaces a source by its
        // source's source, so a chain of 64 ends after 6
        const uint32_t p = q + b + lane;
        const uint32_t o = b + lane < n ? lds.off[b + lane] : 0u;
        int32_t s = (int32_t)(lane - o);
        for (;;) {
          const int32_t s2 = __builtin_amdgcn_ds_bpermute(4 * s, s);
          const bool on = s >= 0 && s2 != s;
          if (!ballot(on)) break;
          s = on ? s2 : s;
        }
        const T x = ring[(q + b + (uint32_t)s) & M];
        if (o) ring[p & M] = x;
        wave_sync();
      }
      todo &= ~now;
      q += n;
      while (q - done >= kFlushSyms) flush(kFlushSyms);
    }
    t += popc64(tm);
    u += S * popc64(tm & ~pm) + 2u * popc64(tm & pm);
    if (q >= c) break;
  }
  if (q < c) return false;  // flags exhausted before the chunk is complete
  wave_sync();
  flush(c - done);
  wave_sync();
  if ((t + 7) / 8 != F || u != P) return false;
  return t == 8 * F || flags[F - 1] >> (t - 8 * (F - 1)) == 0;
}

// ---- workgroup decoder ------------------------------------------------------

constexpr uint32_t kDecThreads = 256;
constexpr uint32_t kFastSyms = 16 * kDecThreads;          // tokens per chunk (16 per thread)
constexpr uint32_t kFastOut = kDecodeRingBytes;           // chunk bytes kept in LDS
constexpr uint32_t kFastRec = kFastSyms / 8 + kFastOut + 32;

struct BlockLds {
  uint8_t rec[kFastRec];              // staged record (16-byte aligned copy)
  uint8_t out[kFastOut];              // the chunk; the ring of the wave decoder
  uint64_t ptrbits[kFastSyms / 64];   // pointer flags of the decoded tokens
  uint32_t scratch[16];
};

// Block-wide maximum and sum of one u32 each per thread, and any of a flag.
__device__ inline void block_reduce(uint32_t& mx, uint32_t& sum, bool& any, uint32_t* scratch) {
  const uint32_t lane = lane_id(), wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const uint32_t wm = wave_max_u32(mx);
  const uint32_t ws = readlane(wave_incl_scan(sum), 63);
  const bool wa = ballot(any) != 0;
  if (lane == 0) {
    scratch[wid] = wm;
    scratch[4 + wid] = ws;
    scratch[8 + wid] = wa;
  }
  __syncthreads();
  mx = 0;
  sum = 0;
  any = false;
  for (uint32_t w = 0; w < nw; ++w) {
    mx = max(mx, scratch[w]);
    sum += scratch[4 + w];
    any = any || scratch[8 + w];
  }
  __syncthreads();
}

// Whether the workgroup decoder takes a chunk of c symbols with F flag and
// P payload bytes.
__device__ inline bool fits_block(uint32_t c, uint32_t S, uint32_t F, uint32_t P) {
  return c <= kFastSyms && c * S <= kFastOut && F <= kFastSyms / 8 && F + P + 16 <= kFastRec;
}

// One symbol of S bytes at any byte address in LDS (aligned dword reads and a
// funnel shift; up to 11 bytes past the symbol are read).
template <int S>
__device__ __forceinline__ typename SymType<S>::T load_sym(const uint8_t* p) {
  const uint32_t sh = (uint32_t)(uintptr_t)p & 3u;
  const uint32_t* w = reinterpret_cast<const uint32_t*>(__builtin_assume_aligned(p - sh, 4));
  const uint32_t lo = __builtin_amdgcn_alignbyte(w[1], w[0], sh);
  if constexpr (S == 8) {
    return (uint64_t)lo | ((uint64_t)__builtin_amdgcn_alignbyte(w[2], w[1], sh) << 32);
  } else {
    return (typename SymType<S>::T)lo;
  }
}

// Sum over the waves before this one of a wave-uniform value, and the total.
__device__ inline uint32_t waves_excl(uint32_t v, uint32_t* scratch, uint32_t& total) {
  const uint32_t wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  if (lane_id() == 0) scratch[wid] = v;
  __syncthreads();
  uint32_t before = 0;
  total = 0;
  for (uint32_t w = 0; w < nw; ++w) {
    const uint32_t x = scratch[w];
    before += w < wid ? x : 0u;
    total += x;
  }
  __syncthreads();
  return before;
}

// Decode one chunk with the whole workgroup (kDecThreads threads); returns
// false (uniformly) if the chunk breaks a rule. rec: its record in HBM;
// in_end: end of the stream (no byte at or past it is read); dst: its first
// output byte.
//
// Token i (of the 8 F the flags describe) is handled by wave i / (64 R) in
// round (i / 64) % R on lane i % 64, R = ceil(8 F / 256) rounds per wave, so
// neighbouring lanes touch neighbouring LDS bytes and small chunks still
// spread over all four waves. Payload offsets come from the literal / pointer
// counts (mbcnt within a round, running totals across rounds, one exchange
// across waves); output positions likewise from the token lengths.
template <int S>
__device__ bool decode_chunk_block(const uint8_t* rec, const uint8_t* in_end, uint32_t F,
                                   uint32_t P, uint32_t c, uint32_t W, uint32_t MIN, uint8_t* dst,
                                   BlockLds& sm) {
  using T = typename SymType<S>::T;
  const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  T* out = reinterpret_cast<T*>(sm.out);

  // stage the record; the copy keeps the record's alignment within 16 bytes
  const uint32_t a = (uint32_t)((uintptr_t)rec & 15u);
  const uint8_t* g0 = rec - a;
  const uint32_t nwords = (a + F + P + 15) / 16;
  for (uint32_t k = tid; k < nwords; k += kDecThreads) {
    const uint8_t* gp = g0 + 16 * k;
    if (gp + 16 <= in_end) {
      *reinterpret_cast<uint4*>(sm.rec + 16 * k) = *reinterpret_cast<const uint4*>(gp);
    } else {
      for (uint32_t b = 0; b < 16; ++b) sm.rec[16 * k + b] = gp + b < in_end ? gp[b] : 0;
    }
  }
  __syncthreads();
  const uint8_t* fl = sm.rec + a;
  const uint8_t* pay = fl + F;
  const uint32_t nt = 8 * F;
  // R rounds of 64 tokens per wave (R <= 16), so that small chunks spread over
  // all four waves too
  const uint32_t R = nt <= 256 ? 1u : (nt + 255) / 256;
  const uint32_t tpw = 64 * R;
  const uint32_t t0 = tpw * wave + lane;

  // token i's kind: pointer flag bit (only for i < 8 F)
  auto is_ptr = [&](uint32_t i) { return i < nt && ((fl[i >> 3] >> (i & 7)) & 1u); };
  // the wave's literal / pointer counts: lane l counts the wave's tokens
  // R l .. R l + R - 1 (R flag bits at any bit offset, at most 3 bytes)
  uint32_t np, nh;
  {
    const uint32_t i = tpw * wave + R * lane;  // first of this lane's R tokens
    const uint32_t b0 = i >> 3;
    uint32_t fb = 0;
    if (b0 < F) fb = fl[b0];
    if (b0 + 1 < F) fb |= (uint32_t)fl[b0 + 1] << 8;
    if (b0 + 2 < F) fb |= (uint32_t)fl[b0 + 2] << 16;
    fb >>= (i & 7u);
    const uint32_t cnt = i >= nt ? 0u : min(R, nt - i);
    const uint32_t hmask = (1u << cnt) - 1u;
    np = readlane(wave_incl_scan((uint32_t)__popc(fb & hmask)), 63);
    nh = readlane(wave_incl_scan((uint32_t)__popc(hmask)), 63);
  }
  uint32_t tot;
  const uint32_t x1 = waves_excl((nh - np) | (np << 16), sm.scratch, tot);
  if ((tot >> 16) == 0) {
    // no pointer: the record is valid exactly when its tokens are the chunk's
    // c literals (F = ceil(c / 8) flag bytes, P = c S payload bytes), and then
    // the payload is the chunk. It is copied out of LDS with one funnel shift
    // (its start's offset within a dword is the same for every word).
    if (F != (c + 7) / 8 || P != c * S) return false;
    const uint32_t nb = c * S, base = a + F, sh = base & 3u;
    const uint32_t* w = reinterpret_cast<const uint32_t*>(sm.rec + (base - sh));
    if (((uintptr_t)dst & 15u) == 0) {
      for (uint32_t k = tid; k < nb / 16; k += kDecThreads) {
        const uint32_t* q = w + 4 * k;
        const uint32_t q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
        const uint32_t q4 = sh ? q[4] : 0u;  // read only when it holds payload bytes
        *reinterpret_cast<uint4*>(dst + 16 * k) =
            make_uint4(__builtin_amdgcn_alignbyte(q1, q0, sh), __builtin_amdgcn_alignbyte(q2, q1, sh),
                       __builtin_amdgcn_alignbyte(q3, q2, sh), __builtin_amdgcn_alignbyte(q4, q3, sh));
      }
      for (uint32_t b = (nb & ~15u) + tid; b < nb; b += kDecThreads) dst[b] = sm.rec[base + b];
    } else {
      for (uint32_t b = tid; b < nb; b += kDecThreads) dst[b] = sm.rec[base + b];
    }
    return true;
  }
  const uint32_t lit0 = x1 & 0xFFFFu, ptr0 = x1 >> 16;
  // Pointer symbols are resolved in parallel (pointer jumping, below) when the
  // chunk has many pointers and its decoded bytes leave room in `out` for a
  // 16-bit source index per symbol; otherwise wave 0 copies them in order.
  const uint32_t src_at = (c * S + 15) & ~15u;
  const bool jump = (tot >> 16) >= 64 && src_at + 2 * c <= kFastOut;
  uint16_t* src = reinterpret_cast<uint16_t*>(sm.out + src_at);

  // this wave's total length: one per token, plus L - 1 per pointer whose
  // payload is in range
  uint32_t wlen = nh;
  {
    uint32_t lit = lit0, ptr = ptr0;
    for (uint32_t j = 0; j < R; ++j) {
      const uint32_t i = t0 + 64 * j;
      const bool isp = is_ptr(i);
      const uint64_t pmj = ballot(isp), lm = ballot(i < nt && !isp);
      if (pmj) {
        const uint32_t off = S * (lit + mbcnt(lm)) + 2 * (ptr + mbcnt(pmj));
        const uint32_t e = isp && off + 2 <= P ? pay[off] - 1u : 0u;
        wlen += readlane(wave_incl_scan(e), 63);
      }
      lit += popc64(lm);
      ptr += popc64(pmj);
    }
  }
  uint32_t pos_end;
  const uint32_t wpos0 = waves_excl(wlen, sm.scratch, pos_end);

  // positions, checks and literals; taken tokens (position < c) are a prefix
  bool bad = false;
  uint32_t taken = 0, uend = 0;
  {
    uint32_t lit = lit0, ptr = ptr0, run = wpos0;
    for (uint32_t j = 0; j < R; ++j) {
      const uint32_t i = t0 + 64 * j;
      const bool has = i < nt;
      const bool isp = is_ptr(i);
      const uint64_t pmj = ballot(isp), lm = ballot(has && !isp);
      const uint32_t off = S * (lit + mbcnt(lm)) + 2 * (ptr + mbcnt(pmj));
      const uint32_t sz = isp ? 2u : (uint32_t)S;
      const bool okp = off + sz <= P;
      uint32_t L = 1, O = 1, pos;
      if (pmj) {
        if (isp && okp) {
          L = pay[off];
          O = pay[off + 1] ? pay[off + 1] : 256u;
        }
        const uint32_t len = has ? L : 0u;
        const uint32_t inc = wave_incl_scan(len);
        pos = run + inc - len;
        run += readlane(inc, 63);
      } else {
        // no pointer in this round: consecutive positions
        pos = run + lane;
        run += popc64(lm);
      }
      const bool tk = has && pos < c;
      if (tk) {
        ++taken;
        uend = max(uend, off + sz);
        if (!okp) {
          bad = true;
        } else if (isp) {
          const bool ok = L >= MIN && O <= W && O <= pos && L <= O && pos + L <= c;
          bad = bad || !ok;
          if (ok && jump)
            for (uint32_t k = 0; k < L; ++k) src[pos + k] = (uint16_t)(pos + k - O);
        } else {
          out[pos] = load_sym<S>(pay + off);
          if (jump) src[pos] = (uint16_t)pos;
        }
      }
      const uint64_t tb = ballot(tk && isp);
      if (lane == 0 && !jump) sm.ptrbits[R * wave + j] = tb;
      lit += popc64(lm);
      ptr += popc64(pmj);
    }
  }
  uint32_t Tn = taken;
  block_reduce(uend, Tn, bad, sm.scratch);
  // every rule of the wave decoder: all checks above hold, the flags cover
  // the chunk, the tokens use exactly F flag bytes and P payload bytes, and
  // the unused flag bits are zero
  if (bad || pos_end < c || (Tn + 7) / 8 != F || uend != P) return false;
  if (Tn < nt && (fl[F - 1] >> (Tn - 8 * (F - 1))) != 0) return false;

  // pointers. Symbol p of a pointer with offset O takes the value of symbol
  // p - O (always earlier, since O <= its position), which is a literal or
  // again a pointer symbol. Replacing every source by its source's source
  // (pointer jumping) reaches a literal for every symbol within
  // ceil(log2 c) <= 12 rounds: a chain of any length halves each round. The
  // update is in place: a thread that reads an entry another thread just
  // replaced still gets an earlier symbol of the same chain. Then every
  // pointer symbol copies its literal.
  if (jump) {
    for (uint32_t round = 0; round < 13; ++round) {
      bool changed = false;
      for (uint32_t p = tid; p < c; p += kDecThreads) {
        const uint32_t s0 = src[p];
        const uint32_t s1 = src[s0];
        if (s1 != s0) {
          src[p] = (uint16_t)s1;
          changed = true;
        }
      }
      if (!__syncthreads_or(changed)) break;
    }
    for (uint32_t p = tid; p < c; p += kDecThreads) {
      const uint32_t s0 = src[p];
      if (s0 != p) out[p] = out[s0];
    }
    __syncthreads();
  }

  // pointers, 64 at a time in token order, by wave 0. A pointer is copied
  // once the last uncopied pointer before it ends at or before its source
  // starts (destinations are ordered, so no uncopied output overlaps its
  // source); the first uncopied pointer always qualifies.
  if (!jump && wave == 0) {
    const uint32_t nwd = (Tn + 63) / 64;
    const uint64_t wd = lane < nwd ? sm.ptrbits[lane] : 0ull;
    const uint32_t cnt = popc64(wd);
    const uint32_t wb_incl = wave_incl_scan(cnt);
    const uint32_t wb = wb_incl - cnt;  // pointers before flag word `lane`
    const uint32_t NP = readlane(wb_incl, 63);
    uint32_t extra = 0;
    for (uint32_t g = 0; g < NP; g += 64) {
      const uint32_t o = g + lane;  // this lane's pointer ordinal
      const bool valid = o < NP;
      // its flag word: the last word whose first ordinal is <= o
      uint32_t lo = 0, hi = 63;
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const uint32_t mid = (lo + hi + 1) / 2;
        if ((uint32_t)__shfl((int)wb, (int)mid, 64) <= o) lo = mid;
        else hi = mid - 1;
      }
      uint64_t m = __shfl((unsigned long long)wd, (int)lo, 64);
      uint32_t r = o - (uint32_t)__shfl((int)wb, (int)lo, 64);
      uint32_t bit = 0;
#pragma unroll
      for (uint32_t width = 32; width >= 1; width >>= 1) {
        const uint32_t lowc = popc64(m & ((1ull << width) - 1));
        if (r >= lowc) {
          r -= lowc;
          m >>= width;
          bit += width;
        }
      }
      const uint32_t t = 64 * lo + bit;
      uint32_t L = 0, O = 0;
      if (valid) {
        const uint32_t off = S * (t - o) + 2 * o;
        L = pay[off];
        O = pay[off + 1] ? pay[off + 1] : 256u;
      }
      const uint32_t e = valid ? L - 1 : 0u;
      const uint32_t inc = wave_incl_scan(e);
      const uint32_t pos = t + extra + inc - e;
      extra += readlane(inc, 63);
      const uint32_t end = pos + L, src = pos - O;
      uint64_t un = ballot(valid);
      while (un) {
        const uint64_t below = un & ((1ull << lane) - 1);
        const uint32_t lk = below ? 63u - (uint32_t)__clzll(below) : 0u;
        const uint32_t endk = (uint32_t)__shfl((int)end, (int)lk, 64);
        const bool ready = ((un >> lane) & 1u) && (below == 0 || endk <= src);
        const uint64_t rm = ballot(ready);
        if (popc64(rm) == 1) {
          const uint32_t j0 = (uint32_t)__ffsll((unsigned long long)rm) - 1;
          const uint32_t P0 = readlane(pos, j0), Lj = readlane(L, j0), Oj = readlane(O, j0);
          for (uint32_t k = lane; k < Lj; k += 64) out[P0 + k] = out[P0 - Oj + k];
        } else if (ready) {
          for (uint32_t k = 0; k < L; ++k) out[pos + k] = out[src + k];
        }
        wave_sync();
        un &= ~rm;
      }
    }
  }
  __syncthreads();

  // write the chunk out
  const uint32_t nb = c * S;
  if (((uintptr_t)dst & 15u) == 0) {
    for (uint32_t k = tid; k < nb / 16; k += kDecThreads)
      *reinterpret_cast<uint4*>(dst + 16 * k) = *reinterpret_cast<const uint4*>(sm.out + 16 * k);
    for (uint32_t b = (nb & ~15u) + tid; b < nb; b += kDecThreads) dst[b] = sm.out[b];
  } else {
    for (uint32_t b = tid; b < nb; b += kDecThreads) dst[b] = sm.out[b];
  }
  return true;
}

// A record sized for c literals (F = ceil(c / 8) flag bytes, P = c S payload
// bytes) whose flag bytes are all zero is valid and its payload is the chunk:
// copy it straight from the stream to the output (dword-aligned 16-byte loads,
// funnel-shifted by the payload's offset within a dword). Returns false
// (uniformly), having written nothing, if any flag bit is set. Every dword
// read holds a byte of the record; none reaches in_end.
__device__ inline bool copy_literal_chunk(const uint8_t* rec, const uint8_t* in_end, uint32_t F,
                                          uint32_t nb, uint8_t* dst) {
  const uint32_t tid = threadIdx.x;
  const uint32_t r0 = (uint32_t)((uintptr_t)rec & 3u);
  const uint32_t* fw = reinterpret_cast<const uint32_t*>(rec - r0);
  bool set = false;
  for (uint32_t k = tid; 4 * k < r0 + F; k += kDecThreads) {
    uint32_t v = 0;
    const uint8_t* wk = reinterpret_cast<const uint8_t*>(fw + k);
    if (wk + 4 <= in_end) {
      v = fw[k];
    } else {
      for (uint32_t b = 0; wk + b < in_end; ++b) v |= (uint32_t)wk[b] << (8 * b);
    }
    if (4 * k < r0) v &= ~0u << (8 * r0);                // bytes before the record
    const uint32_t in_f = r0 + F - 4 * k;                 // flag bytes in this dword, from its start
    if (in_f < 4) v &= (1u << (8 * in_f)) - 1u;           // bytes after the flags
    set = set || v != 0;
  }
  if (__syncthreads_or(set)) return false;
  const uint8_t* src = rec + F;
  const uint32_t sh = (uint32_t)((uintptr_t)src & 3u);
  const uint32_t* sw = reinterpret_cast<const uint32_t*>(src - sh);
  const uint32_t ng = ((uintptr_t)dst & 15u) == 0 ? nb / 16 : 0u;  // 16-byte groups
  // four groups per thread in flight: all loads, then all stores
  for (uint32_t k0 = tid; k0 < ng; k0 += 4 * kDecThreads) {
    uint4 g[4];
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const uint32_t k = k0 + j * kDecThreads;
      if (k < ng) g[j] = stream::load_group(sw + 4 * k, sh, in_end);
    }
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const uint32_t k = k0 + j * kDecThreads;
      if (k < ng) *reinterpret_cast<uint4*>(dst + 16 * k) = g[j];
    }
  }
  for (uint32_t b = 16 * ng + tid; b < nb; b += kDecThreads) dst[b] = src[b];
  return true;
}

// Where chunk i of a validated stream is and goes (all wave-uniform).
struct ChunkPlace {
  const uint8_t* rec;
  uint32_t F, P, c;
  uint8_t* dst;
};
__device__ inline ChunkPlace chunk_place(const uint8_t* in, const DecodeParams& p,
                                         const uint64_t* group_off, uint64_t i, uint8_t* out) {
  ChunkPlace k;
  i = uniform(i);
  const uint8_t* e = in + kHeaderBytes + 8 * i;
  k.F = uniform(*reinterpret_cast<const uint32_t*>(e));
  k.P = uniform(*reinterpret_cast<const uint32_t*>(e + 4));
  k.rec = in + uniform(record_offset(in, group_off, i));
  const uint64_t cs = i * p.C;
  k.c = (uint32_t)min<uint64_t>(p.C, p.m - cs);
  k.dst = out + cs * p.S;
  return k;
}

// LDS of one wave of decode_stream_chunk_wave.
constexpr uint32_t kWaveLds = (sizeof(WaveLds<2>) + 15) / 16 * 16;

// Decode chunk i of a validated stream of 1- or 2-byte symbols with one
// wavefront and kWaveLds bytes of LDS; false (uniformly) if it is corrupt. A record of literals alone is the chunk itself behind its zero
// flag bytes and is copied (64 MiB of random uint16, C 2048: 49 us; token by
// token 120).
__device__ inline bool decode_stream_chunk_wave(const uint8_t* in, const DecodeParams& p,
                                                const uint64_t* group_off, uint64_t i,
                                                uint8_t* out, uint8_t* lds) {
  const ChunkPlace k = chunk_place(in, p, group_off, i, out);
  const uint32_t F = k.F, P = k.P, c = k.c;
  if (F == (c + 7) / 8 && P == c * p.S) {
    const uint32_t lane = lane_id();
    uint64_t set = 0;
    for (uint32_t w = lane; 8 * w < F; w += 64) set |= load_bytes8(k.rec, w, F);
    if (!ballot(set != 0)) {
      stream::copy_unaligned<2>(k.dst, k.rec + F, P, k.rec + F + P, lane, 64);
      return true;
    }
  }
  if (p.S == 1) return decode_chunk_wave<1, false>(k.rec, F, P, c, p.W, p.MIN, k.dst, lds);
  return decode_chunk_wave<2, false>(k.rec, F, P, c, p.W, p.MIN, k.dst, lds);
}

// Whether the chunks of a validated stream are decoded by one wave each, where
// `chunks` chunks of 1- and 2-byte symbols are decoded together. A wave takes
// half the instructions of a workgroup but about 1 us per 64 tokens, so it needs
// many chunks, and the more the longer they are. Workgroup against wave, in us:
// Zipf bytes, C 4096: 1600 chunks 64 and 70, 2048 chunks 70 and 69, 4096 chunks
// 130 and 83; uint16 codes, C 4096: 1600 chunks 64 and 63; C 2048: 42 and 37.
// Where pointers save next to nothing a chunk is nearly all literals, which
// workgroups decode sooner: random bytes, C 4096: 3072 chunks 54 and 81, 8192
// chunks 130 and 125; C 2048: 3072 chunks 40 and 46, 4096 chunks 50 and 47. At 2
// bytes a symbol that can be told from single pointers: with less than one in
// 1024 symbols most chunks are copied, and the others want to end soon (64 MiB
// of random uint16 with one pointer, C 4096: 41 and 57). Chunks too long for
// the workgroup decoder are one wave's work in either kernel; the wave kernel has
// room for more of them at a time.
constexpr uint32_t kFewestForWaves = 1024;
__device__ __forceinline__ bool takes_waves(const DecodeParams& p, uint64_t in_bytes,
                                            uint64_t chunks) {
  if (p.S > 2) return false;
  if (p.C > kFastSyms) return chunks > kFewestForWaves;
  const uint64_t literals = p.m * p.S + p.m / 8 + p.N;  // record bytes without a pointer
  const uint64_t records = in_bytes - kHeaderBytes - 8 * p.N;
  const uint64_t saved = literals > records ? literals - records : 0;
  if (p.S == 2 && saved < p.m / 1024) return false;
  return chunks > (saved < p.m / 32 ? max(kFewestForWaves, 7 * p.C / 4) : 1280 + p.C / 8);
}

// Decode chunk i of a validated stream of in_bytes bytes with the whole
// workgroup; false (uniformly) if it is corrupt. Chunks the workgroup
// decoder does not take go to the wave decoder on wave 0 (1.5 MB of uint16
// codes, C 8192: 97 us; 268 with the pointers of 64 tokens copied one by one;
// 1 MiB of uint32 out of 16 values: 114 and 409).
__device__ inline bool decode_stream_chunk_block(const uint8_t* in, uint64_t in_bytes,
                                                 const DecodeParams& p, const uint64_t* group_off,
                                                 uint64_t i, uint8_t* out, BlockLds& sm) {
  const uint8_t* e = in + kHeaderBytes + 8 * i;
  const uint32_t F = *reinterpret_cast<const uint32_t*>(e);
  const uint32_t P = *reinterpret_cast<const uint32_t*>(e + 4);
  const uint8_t* rec = in + record_offset(in, group_off, i);
  const uint64_t cs = i * p.C;
  const uint32_t c = (uint32_t)min<uint64_t>(p.C, p.m - cs);
  uint8_t* dst = out + cs * p.S;
  if (F == (c + 7) / 8 && P == c * p.S && copy_literal_chunk(rec, in + in_bytes, F, P, dst)) return true;
  if (fits_block(c, p.S, F, P)) {
    switch (p.S) {
      case 1: return decode_chunk_block<1>(rec, in + in_bytes, F, P, c, p.W, p.MIN, dst, sm);
      case 2: return decode_chunk_block<2>(rec, in + in_bytes, F, P, c, p.W, p.MIN, dst, sm);
      case 4: return decode_chunk_block<4>(rec, in + in_bytes, F, P, c, p.W, p.MIN, dst, sm);
      default: return decode_chunk_block<8>(rec, in + in_bytes, F, P, c, p.W, p.MIN, dst, sm);
    }
  }
  const uint32_t wave = threadIdx.x >> 6;
  if (wave == 0) {
    bool ok;
    switch (p.S) {
      case 1: ok = decode_chunk_wave<1, true>(rec, F, P, c, p.W, p.MIN, dst, sm.out); break;
      case 2: ok = decode_chunk_wave<2, true>(rec, F, P, c, p.W, p.MIN, dst, sm.out); break;
      case 4: ok = decode_chunk_wave<4, true>(rec, F, P, c, p.W, p.MIN, dst, sm.out); break;
      default: ok = decode_chunk_wave<8, true>(rec, F, P, c, p.W, p.MIN, dst, sm.out); break;
    }
    if (lane_id() == 0) sm.scratch[15] = ok;
  }
  __syncthreads();
  const bool ok = sm.scratch[15] != 0;
  __syncthreads();
  return ok;
}

}  // namespace dec
}  // namespace gpulz
