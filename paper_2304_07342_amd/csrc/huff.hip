// Entropy stage after LZSS (gpuLZ section 4.5 pairs LZSS with a Huffman
// coder): byte Huffman coding in chunks that decode in parallel. The rules of
// the code and of the stream are in huff_internal.h and gpulz.h.
//
// Compression, five launches on one stream, no host round trip:
//   hist_kernel    per-workgroup byte histograms (32 bank-padded LDS
//                  sub-histograms, 16-byte loads);
//   build_kernel   one workgroup: sums the histograms, sorts (weight,
//                  symbol) keys, runs Huffman's merge (sorted leaves,
//                  internal nodes in creation order) many joins a round,
//                  limits the lengths, assigns canonical codes, writes the
//                  code lengths;
//   size_kernel    one wave per chunk: code bits of the chunk;
//   scan_kernel    one workgroup: record offsets and the header;
//   encode_kernel  one wave per chunk: bit offsets by a wave scan, codes
//                  ORed into LDS words, the record written once.
// Decompression:
//   dec_prepare_kernel  one workgroup: checks the header and the code,
//                       builds the lookup tables, scans the record sizes;
//   decode_kernel       one lane per 128-symbol sub-block (32 lanes per
//                       chunk): code words staged in LDS, a two-level
//                       lookup table in LDS, each lane writing its symbols
//                       with 16-byte stores.
#include "huff_internal.h"
#include "stream_device.h"
#include "wave.h"

namespace gpulz {
namespace huff {
namespace {

__device__ inline uint64_t input_size(const EncArgs& a) { return a.d_n ? *a.d_n : a.max_n; }

__device__ inline uint32_t byte_of(const uint4& q, uint32_t b) {
  const uint32_t w = b < 8 ? (b < 4 ? q.x : q.y) : (b < 12 ? q.z : q.w);
  return (w >> (8 * (b & 3))) & 0xFFu;
}

// ---- compression -----------------------------------------------------------

// 32 sub-histograms per workgroup, one per lane of a half-wave (lanes l and
// l + 32 share one), each padded by a word so that the copies of one byte
// value fall in different LDS banks: a skewed input (most bytes equal) then
// costs two-way same-address atomics instead of 64-way ones.
constexpr uint32_t kHistCopies = 32;
constexpr uint32_t kHistStride = 257;

__global__ __launch_bounds__(256) void hist_kernel(EncArgs a) {
  __shared__ uint32_t h[kHistCopies * kHistStride];
  const uint32_t tid = threadIdx.x;
  for (uint32_t k = tid; k < kHistCopies * kHistStride; k += 256) h[k] = 0;
  __syncthreads();
  uint32_t* mine = h + (tid & (kHistCopies - 1)) * kHistStride;
  const uint64_t n = input_size(a);
  if (n <= a.max_n) {
    const uint64_t words = (n + 15) / 16;
    const uint64_t per = (words + gridDim.x - 1) / gridDim.x;
    const uint64_t w0 = (uint64_t)blockIdx.x * per;
    const uint64_t w1 = w0 + per < words ? w0 + per : words;
    const uint4* in4 = reinterpret_cast<const uint4*>(a.in);
    const uint64_t wfull = n / 16;  // whole 16-byte words
    uint64_t w = w0 + tid;
    // four loads in flight per thread, then their 64 bytes counted
    for (; w + 3 * 256 < w1 && w + 3 * 256 < wfull; w += 4 * 256) {
      uint4 q[4];
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) q[u] = in4[w + u * 256];
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u)
#pragma unroll
        for (uint32_t b = 0; b < 16; ++b) atomicAdd(&mine[byte_of(q[u], b)], 1u);
    }
    for (; w < w1; w += 256) {
      if (16 * w + 16 <= n) {
        const uint4 q = in4[w];
#pragma unroll
        for (uint32_t b = 0; b < 16; ++b) atomicAdd(&mine[byte_of(q, b)], 1u);
      } else {
        for (uint64_t b = 16 * w; b < n; ++b) atomicAdd(&mine[a.in[b]], 1u);
      }
    }
  }
  __syncthreads();
  uint32_t sum = 0;
#pragma unroll 8
  for (uint32_t c = 0; c < kHistCopies; ++c) sum += h[c * kHistStride + tid];
  a.partial[(uint64_t)blockIdx.x * 256 + tid] = sum;
}

// Lanes of the wave whose code has the same length as this lane's.
__device__ __forceinline__ uint64_t same_length(uint32_t l) {
  uint64_t same = ~0ull;
#pragma unroll
  for (uint32_t b = 0; b < 4; ++b) {
    const uint64_t set = __ballot((l >> b) & 1u);
    same &= (l >> b) & 1u ? set : ~set;
  }
  return same;
}

// Codes of each length among the symbols of each 64-symbol group: the rank
// of a code among those of its length is a ballot inside its group and the
// counts of the groups before it, where a loop over the symbols before it
// took up to 256 dependent LDS reads.
struct LengthCounts {
  uint32_t n[4][16];

  // Called by threads 0..255 with symbol tid's length; returns the rank in
  // the group. `n` is zeroed before and read after a barrier.
  __device__ __forceinline__ uint32_t add(uint32_t tid, uint32_t l) {
    const uint64_t same = same_length(l);
    const uint32_t r = __popcll(same & ((1ull << (tid & 63u)) - 1));
    if (r == 0) n[tid >> 6][l] = __popcll(same);
    return r;
  }
  __device__ __forceinline__ uint32_t before(uint32_t tid, uint32_t l) const {
    uint32_t s = 0;
#pragma unroll
    for (uint32_t g = 0; g < 3; ++g) s += g < tid >> 6 ? n[g][l] : 0u;
    return s;
  }
  __device__ __forceinline__ uint32_t total(uint32_t l) const {
    return n[0][l] + n[1][l] + n[2][l] + n[3][l];
  }
};

struct BuildLds {
  uint64_t w[256];    // weight by symbol (0 = absent)
  uint64_t tmp[256];  // unsorted keys; a merge round's weights in order
  uint64_t key[256];  // weight << 8 | symbol, ascending; absent symbols last
  uint64_t iw[256];   // internal node weights in creation order
  uint16_t parent[512];
  uint16_t anc[256], dist[256];  // pointer jumping over internal nodes
  uint8_t len[256];
  LengthCounts lengths;
  uint32_t next[16];
  uint64_t total;       // sum of the weights
  uint32_t present, deepest, internal;
};

// Huffman's merge by one wave: sorted leaves, and internal nodes in creation
// order (their weights never decrease); a leaf wins a tie (its index is
// smaller). One round joins every node that is at hand and no heavier than
// the sum t of the two lightest: no node made in the round is lighter than t,
// and one of weight t comes after the others of that weight, so joining them
// two by two in ascending order is what one join after the other does. An odd
// node at the end waits. t at least doubles every second round, so the
// rounds follow the logarithm of the weights (about 20) where the joins one
// by one were up to 255 LDS round trips (build_kernel on the LZSS stream of
// 1 MiB of codes: 64 us with one join at a time and the ranks counted in a
// loop, 34 us so, of 128 MiB 73 and 44; what is left is the chain of rounds on
// one wave and the sum of the histograms). A round costs about six single joins, so few symbols are joined one
// by one (47 symbols of raw uint16 codes, built five times for the length
// limit: 1 MiB 150 us in rounds, 103 one by one), and weights that grow
// like a chain, whose rounds are a join or two: after such a round the next 8
// joins are made one by one, then 16 and so on. W is uint32_t when the weights
// sum below 2^31 (cheaper compares; below 2^31 so that no weight equals the
// 32-bit infinity), else uint64_t. Returns the number of internal nodes.
constexpr uint32_t kSingleJoins = 96;
template <typename W>
__device__ uint32_t merge(BuildLds& sm, uint32_t m, uint32_t lane) {
  const W kInf = (W)~0ull;
  W leaf[4];
#pragma unroll
  for (uint32_t q = 0; q < 4; ++q) {
    const uint32_t x = 64 * q + lane;
    leaf[q] = x < m ? (W)(sm.key[x] >> 8) : kInf;
  }
  uint32_t li = 0, kf = 0, kc = 0;  // first leaf and node at hand, nodes made
  uint32_t single = m <= kSingleJoins ? m : 0u, next_single = 8;  // joins to make one by one
  while (kc + 1 < m) {
    if (single) {
      // one lane joins the two lightest nodes, `single` times
      if (lane == 0) {
        for (; single && kc + 1 < m; --single) {
          const W l0 = li < m ? (W)(sm.key[li] >> 8) : kInf;
          const W l1 = li + 1 < m ? (W)(sm.key[li + 1] >> 8) : kInf;
          const W i0 = kf < kc ? (W)sm.iw[kf] : kInf;
          const W i1 = kf + 1 < kc ? (W)sm.iw[kf + 1] : kInf;
          uint32_t na, nb;
          W w;
          if (l0 <= i0) {
            na = li++;
            w = l0;
            if (l1 <= i0) {
              nb = li++;
              w += l1;
            } else {
              nb = 256 + kf++;
              w += i0;
            }
          } else {
            na = 256 + kf++;
            w = i0;
            if (l0 <= i1) {
              nb = li++;
              w += l0;
            } else {
              nb = 256 + kf++;
              w += i1;
            }
          }
          sm.iw[kc] = w;
          sm.parent[na] = sm.parent[nb] = (uint16_t)(256 + kc);
          ++kc;
        }
      }
      single = 0;
      li = uniform(li);
      kf = uniform(kf);
      kc = uniform(kc);
      wave_sync();
      continue;
    }
    const W l0 = li < m ? (W)(sm.key[li] >> 8) : kInf;
    const W l1 = li + 1 < m ? (W)(sm.key[li + 1] >> 8) : kInf;
    const W i0 = kf < kc ? (W)sm.iw[kf] : kInf;
    const W i1 = kf + 1 < kc ? (W)sm.iw[kf + 1] : kInf;
    const W t = l0 <= i0 ? l0 + (l1 <= i0 ? l1 : i0) : i0 + (l0 <= i1 ? l0 : i1);
    W node[4];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      const uint32_t x = 64 * q + lane;
      node[q] = x < kc ? (W)sm.iw[x] : kInf;
    }
    uint32_t le = 0, ie = 0;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      le += __popcll(__ballot(leaf[q] <= t));
      ie += __popcll(__ballot(node[q] <= t));
    }
    const uint32_t na = le - li, nb = ie - kf, k = na + nb;
    // places in the merged order: a loop over the shorter list (what was
    // joined before is no heavier than what is left, so whole counts less
    // the joined ones are counts of what is left)
    uint32_t pl[4], pn[4];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      pl[q] = 64 * q + lane - li;
      pn[q] = 64 * q + lane - kf;
    }
    if (na <= nb) {
      for (uint32_t x = li; x < le; ++x) {
        const W v = (W)(sm.key[x] >> 8);
        uint32_t c = 0;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
          c += __popcll(__ballot(node[q] < v));
          pn[q] += v <= node[q] ? 1u : 0u;
        }
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) pl[q] += 64 * q + lane == x ? c - kf : 0u;
      }
    } else {
      for (uint32_t x = kf; x < ie; ++x) {
        const W v = (W)sm.iw[x];
        uint32_t c = 0;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
          c += __popcll(__ballot(leaf[q] <= v));
          pl[q] += v < leaf[q] ? 1u : 0u;
        }
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) pn[q] += 64 * q + lane == x ? c - li : 0u;
      }
    }
    bool waits_node = false;
    if (k & 1u)
      waits_node = nb && (!na || (W)sm.iw[ie - 1] >= (W)(sm.key[le - 1] >> 8));
    const uint32_t pairs = k / 2;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      const uint32_t x = 64 * q + lane;
      if (x >= li && x < le && pl[q] < 2 * pairs) {
        sm.tmp[pl[q]] = leaf[q];
        sm.parent[x] = (uint16_t)(256 + kc + pl[q] / 2);
      }
      if (x >= kf && x < ie && pn[q] < 2 * pairs) {
        sm.tmp[pn[q]] = node[q];
        sm.parent[256 + x] = (uint16_t)(256 + kc + pn[q] / 2);
      }
    }
    wave_sync();
    for (uint32_t x = lane; x < pairs; x += 64) sm.iw[kc + x] = sm.tmp[2 * x] + sm.tmp[2 * x + 1];
    wave_sync();
    li = le - (k & 1u && !waits_node ? 1u : 0u);
    kf = ie - (waits_node ? 1u : 0u);
    kc += pairs;
    if (pairs <= 2) {
      single = next_single;
      next_single *= 2;
    } else {
      next_single = 8;
    }
  }
  return kc;
}

__global__ __launch_bounds__(1024) void build_kernel(EncArgs a) {
  __shared__ BuildLds sm;
  const uint32_t tid = threadIdx.x;
  if (input_size(a) > a.max_n) return;
  if (tid < 256) sm.w[tid] = 0;
  if (tid == 0) sm.present = 0;
  __syncthreads();
  {
    // partial histograms: 64 column groups of 4 bins x 16 row groups, 16-byte
    // loads, several in flight per thread
    const uint32_t cg = tid & 63u;
    uint64_t s0 = 0, s1 = 0, s2 = 0, s3 = 0;
    const uint4* p4 = reinterpret_cast<const uint4*>(a.partial);
#pragma unroll 8
    for (uint32_t r = tid >> 6; r < a.hist_blocks; r += 16) {
      const uint4 v = p4[(uint64_t)r * 64 + cg];
      s0 += v.x;
      s1 += v.y;
      s2 += v.z;
      s3 += v.w;
    }
    atomicAdd(reinterpret_cast<unsigned long long*>(&sm.w[4 * cg]), (unsigned long long)s0);
    atomicAdd(reinterpret_cast<unsigned long long*>(&sm.w[4 * cg + 1]), (unsigned long long)s1);
    atomicAdd(reinterpret_cast<unsigned long long*>(&sm.w[4 * cg + 2]), (unsigned long long)s2);
    atomicAdd(reinterpret_cast<unsigned long long*>(&sm.w[4 * cg + 3]), (unsigned long long)s3);
  }
  __syncthreads();
  if (tid < 256 && sm.w[tid]) atomicAdd(&sm.present, 1u);
  __syncthreads();
  const uint32_t m = sm.present;
  // weights are at most 2^40, so 41 halvings make them all 1 and the tree at
  // most 8 deep: the cap never binds for a correct build, it only guarantees
  // that the loop ends
  uint32_t rounds = 0;
  for (;; ++rounds) {
    // sort by rank: keys are distinct (absent symbols get distinct keys
    // above every present one)
    if (tid == 0) sm.total = 0;
    if (tid < 256) {
      sm.tmp[tid] = sm.w[tid] ? (sm.w[tid] << 8 | tid) : (~0ull << 8 | tid);
      sm.len[tid] = 0;
    }
    __syncthreads();
    if (tid < 256 && sm.w[tid]) atomicAdd(reinterpret_cast<unsigned long long*>(&sm.total),
                                          (unsigned long long)sm.w[tid]);
    {
      // four adjacent threads count a quarter of the keys each
      const uint64_t k = sm.tmp[tid >> 2];
      uint32_t r = 0;
#pragma unroll 16
      for (uint32_t j = 0; j < 64; ++j) r += sm.tmp[4 * j + (tid & 3u)] < k;
      r += __shfl_xor(r, 1);
      r += __shfl_xor(r, 2);
      if ((tid & 3u) == 0) sm.key[r] = k;
    }
    __syncthreads();
    if (tid < 64) {
      uint32_t kc = 0;
      if (m == 1) {
        if (tid == 0) sm.len[sm.key[0] & 255u] = 1;
      } else if (m > 1) {
        // 32-bit weights while every weight stays below the 32-bit infinity
        kc = sm.total >> 31 ? merge<uint64_t>(sm, m, tid) : merge<uint32_t>(sm, m, tid);
      }
      if (tid == 0) {
        sm.internal = kc;
        sm.deepest = m == 1 ? 1u : 0u;
      }
    }
    __syncthreads();
    // depths of the internal nodes by pointer jumping (8 rounds cover 255)
    const uint32_t kc = sm.internal;
    if (tid < kc) {
      const bool root = tid + 1 == kc;
      sm.anc[tid] = (uint16_t)(root ? tid : sm.parent[256 + tid] - 256u);
      sm.dist[tid] = root ? 0 : 1;
    }
    __syncthreads();
    for (uint32_t round = 0; round < 8; ++round) {
      uint32_t d = 0, na = 0;
      if (tid < kc) {
        const uint32_t up = sm.anc[tid];
        d = sm.dist[tid] + sm.dist[up];
        na = sm.anc[up];
      }
      __syncthreads();
      if (tid < kc) {
        sm.dist[tid] = (uint16_t)d;
        sm.anc[tid] = (uint16_t)na;
      }
      __syncthreads();
    }
    if (kc && tid < m) {
      const uint32_t d = sm.dist[sm.parent[tid] - 256u] + 1u;
      sm.len[sm.key[tid] & 255u] = (uint8_t)d;
      atomicMax(&sm.deepest, d);
    }
    __syncthreads();
    if (sm.deepest <= kLimit) break;
    if (rounds == kMaxLimitRounds) {
      if (tid == 0) a.codes[256] = 1;  // reported by scan_kernel
      return;
    }
    if (tid < 256) sm.w[tid] = (sm.w[tid] + 1) / 2;
    __syncthreads();
  }
  // canonical codes
  if (tid < 64) sm.lengths.n[tid >> 4][tid & 15u] = 0;
  __syncthreads();
  uint32_t l = 0, r = 0;
  if (tid < 256) {
    l = sm.len[tid];
    r = sm.lengths.add(tid, l);
  }
  __syncthreads();
  if (tid <= kLimit) {
    // first code of length tid: every shorter code takes 2^(tid - length)
    uint32_t c = 0;
    for (uint32_t k = 1; k < tid; ++k) c += sm.lengths.total(k) << (tid - k);
    sm.next[tid] = c;
  }
  __syncthreads();
  if (tid < 256)
    a.codes[tid] = l ? l << 16 | (sm.next[l] + sm.lengths.before(tid, l) + r) : 0u;
  if (tid < 128) a.out[64 + tid] = (uint8_t)(sm.len[2 * tid] | sm.len[2 * tid + 1] << 4);
  if (tid == 0) a.codes[256] = 0;
}

__global__ __launch_bounds__(256) void size_kernel(EncArgs a) {
  __shared__ uint32_t L[256];
  const uint64_t n = input_size(a);
  if (n > a.max_n || a.codes[256] != 0) return;
  const uint64_t N = chunks(n);
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  L[tid] = a.codes[tid] >> 16;
  __syncthreads();
  const uint64_t i = (uint64_t)blockIdx.x * 4 + (tid >> 6);
  if (i >= N) return;
  const uint64_t first = i * kChunk;
  const uint32_t c = (uint32_t)(n - first < kChunk ? n - first : kChunk);
  uint32_t bits = 0;
  if (c == kChunk) {
    const uint4* in4 = reinterpret_cast<const uint4*>(a.in + first) + 4 * lane;
#pragma unroll
    for (uint32_t v = 0; v < 4; ++v) {
      const uint4 q = in4[v];
#pragma unroll
      for (uint32_t b = 0; b < 16; ++b) bits += L[byte_of(q, b)];
    }
  } else {
    for (uint32_t b = 64 * lane; b < c && b < 64 * lane + 64; ++b) bits += L[a.in[first + b]];
  }
  bits = readlane(wave_incl_scan(bits), 63);
  if (lane == 0) {
    const uint32_t nsub = (c + kSub - 1) / kSub;
    a.sizes[2 * i] = offsets_bytes(nsub);
    a.sizes[2 * i + 1] = 4 * ((bits + 31) / 32);
    reinterpret_cast<uint32_t*>(a.out + kPre)[i] = bits;
  }
}

__device__ inline uint8_t header_byte(uint32_t b, uint64_t n, uint64_t N, uint64_t total) {
  switch (b) {
    case 0: return 'G';
    case 1: return 'L';
    case 2: return 'H';
    case 3: return '1';
    case 4: return 1;  // version
    case 6: return (uint8_t)kLimit;
    default: break;
  }
  if (b >= 8 && b < 12) return (uint8_t)(kChunk >> (8 * (b - 8)));
  if (b >= 12 && b < 16) return (uint8_t)(kSub >> (8 * (b - 12)));
  if (b >= 16 && b < 24) return (uint8_t)(n >> (8 * (b - 16)));
  if (b >= 24 && b < 32) return (uint8_t)(N >> (8 * (b - 24)));
  if (b >= 32 && b < 40) return (uint8_t)(total >> (8 * (b - 32)));
  return 0;
}

__global__ __launch_bounds__(1024) void scan_kernel(EncArgs a) {
  __shared__ uint64_t scratch[1024 / 64 + 1];
  const uint64_t n = input_size(a);
  const uint32_t tid = threadIdx.x;
  if (n > a.max_n || a.codes[256] != 0) {
    if (tid == 0) {
      *a.out_bytes = 0;
      *a.status = kInvalidArg;
    }
    return;
  }
  const uint64_t N = chunks(n);
  const uint64_t sum = stream::scan_record_sizes<16>(a.sizes, N, a.offs, scratch);
  const uint64_t total = kPre + 4 * N + sum;
  if (tid == 0) {
    a.offs[N] = sum;
    *a.out_bytes = total;
    *a.status = kOk;
  }
  if (tid < 64) a.out[tid] = header_byte(tid, n, N, total);
}

// One wave per chunk, four chunks per workgroup. Lane l codes the chunk's
// bytes [64 l, 64 l + 64): its bit count, a wave prefix sum (DPP) for its bit
// offset, then its codes ORed into the wave's LDS words through a 64-bit
// accumulator (only the first and last word of a lane's range are shared
// with a neighbour). Sub-block k starts at lane 2k's offset.
constexpr uint32_t kEncWaves = 4;

struct EncWaveLds {
  uint32_t words[kMaxWords];
  uint32_t offs32[kSubs / 2 + 1];
};

__global__ __launch_bounds__(64 * kEncWaves) void encode_kernel(EncArgs a) {
  __shared__ uint32_t code[256];
  __shared__ EncWaveLds wl[kEncWaves];
  const uint64_t n = input_size(a);
  if (n > a.max_n || a.codes[256] != 0) return;
  const uint64_t N = chunks(n);
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  code[tid] = a.codes[tid];
  __syncthreads();
  const uint64_t i = (uint64_t)blockIdx.x * kEncWaves + wave;
  if (i >= N) return;
  EncWaveLds& w = wl[wave];
  const uint64_t first = i * kChunk;
  const uint32_t c = (uint32_t)(n - first < kChunk ? n - first : kChunk);
  const uint32_t nsub = (c + kSub - 1) / kSub;
  // this lane's 64 bytes
  const uint32_t j0 = 64 * lane;
  const uint32_t cnt = j0 < c ? (c - j0 < 64 ? c - j0 : 64) : 0;
  uint4 q[4];
  if (cnt == 64) {
    const uint4* in4 = reinterpret_cast<const uint4*>(a.in + first + j0);
#pragma unroll
    for (uint32_t v = 0; v < 4; ++v) q[v] = in4[v];
  } else {
    uint32_t t[16];
#pragma unroll
    for (uint32_t v = 0; v < 16; ++v) t[v] = 0;
#pragma unroll
    for (uint32_t b = 0; b < 64; ++b)
      if (b < cnt) t[b >> 2] |= (uint32_t)a.in[first + j0 + b] << (8 * (b & 3));
#pragma unroll
    for (uint32_t v = 0; v < 4; ++v) q[v] = make_uint4(t[4 * v], t[4 * v + 1], t[4 * v + 2], t[4 * v + 3]);
  }
  uint32_t mybits = 0;
#pragma unroll
  for (uint32_t b = 0; b < 64; ++b) mybits += b < cnt ? code[byte_of(q[b >> 4], b & 15u)] >> 16 : 0u;
  const uint32_t incl = wave_incl_scan(mybits);
  const uint32_t off = incl - mybits;
  const uint32_t total = readlane(incl, 63);
  uint16_t* offs16 = reinterpret_cast<uint16_t*>(w.offs32);
  if ((lane & 1u) == 0 && j0 < c) offs16[lane >> 1] = (uint16_t)off;  // sub-block lane / 2
  if (lane == 0 && (nsub & 1u)) offs16[nsub] = 0;
  const uint32_t nwords = (total + 31) / 32;
  for (uint32_t k = lane; k < nwords; k += 64) w.words[k] = 0;
  wave_sync();
  if (cnt) {
    uint64_t acc = 0;
    uint32_t used = off & 31u, wi = off >> 5;
#pragma unroll
    for (uint32_t b = 0; b < 64; ++b) {
      if (b < cnt) {
        const uint32_t e = code[byte_of(q[b >> 4], b & 15u)];
        const uint32_t l = e >> 16;
        acc |= (uint64_t)(e & 0xFFFFu) << (64 - used - l);
        used += l;
        if (used >= 32) {
          atomicOr(&w.words[wi++], (uint32_t)(acc >> 32));
          acc <<= 32;
          used -= 32;
        }
      }
    }
    if (used) atomicOr(&w.words[wi], (uint32_t)(acc >> 32));
  }
  wave_sync();
  const uint32_t ow = offsets_bytes(nsub) / 4;
  uint32_t* rec = reinterpret_cast<uint32_t*>(a.out + kPre + 4 * N + a.offs[i]);
  for (uint32_t k = lane; k < ow + nwords; k += 64) rec[k] = k < ow ? w.offs32[k] : w.words[k - ow];
}

// ---- decompression ---------------------------------------------------------

struct PrepLds {
  DecTables t;
  LengthCounts lengths;
  uint32_t bad;
  uint64_t scratch[1024 / 64 + 1];
};

// One workgroup, so a chain of latencies bounds it: the header comes in 64
// bytes at once (checked byte by byte it was up to 24 dependent loads) and the
// ranks from ballots; 1 MiB of codes' stream 13.4 -> 8.2 us with the loop over
// the symbols gone, 128 MiB of codes' 30 -> 22.
__global__ __launch_bounds__(1024) void dec_prepare_kernel(DecArgs a) {
  __shared__ PrepLds sm;
  const uint32_t tid = threadIdx.x;
  DecTables& T = sm.t;
  if (tid == 0) {
    bool ok = a.in_bytes >= kPre;
    if (ok) {
      // the 64-byte header in four loads: magic, version, code length limit
      // and zero | chunk and sub-block symbols | n, chunks | stream bytes |
      // zeros
      const uint64_t* h = reinterpret_cast<const uint64_t*>(a.in);
      uint64_t v[8];
#pragma unroll
      for (uint32_t b = 0; b < 8; ++b) v[b] = h[b];
      ok = v[0] == (0x31484C47ull | 1ull << 32 | (uint64_t)kLimit << 48) &&
           v[1] == (kChunk | (uint64_t)kSub << 32) && (v[5] | v[6] | v[7]) == 0;
      T.n = v[2];
      T.N = v[3];
      ok = ok && v[4] == a.in_bytes && T.N == chunks(T.n) && T.N <= (a.in_bytes - kPre) / 4;
    }
    T.status = ok ? kOk : kCorrupt;
    sm.bad = 0;
  }
  if (tid < 64) sm.lengths.n[tid >> 4][tid & 15u] = 0;
  __syncthreads();
  uint32_t len = 0, rank = 0;
  if (T.status == kOk && tid < 256) {
    len = (a.in[64 + tid / 2] >> (4 * (tid & 1u))) & 15u;
    rank = sm.lengths.add(tid, len);
  }
  __syncthreads();
  if (tid <= kLimit && T.status == kOk) {
    // first code and rank of length tid, from the codes shorter than it
    uint32_t c = 0, r = 0;
    for (uint32_t k = 1; k < tid; ++k) {
      const uint32_t m = sm.lengths.total(k);
      c += m << (tid - k);
      r += m;
    }
    T.first[tid] = c;
    T.rank0[tid] = r;
    T.count[tid] = tid ? sm.lengths.total(tid) : 0u;
    if (tid == kLimit) {
      const uint32_t longest = sm.lengths.total(kLimit);
      const uint32_t present = r + longest, kraft = c + longest;
      const bool code_ok = T.n == 0 ? present == 0
                                    : (present == 1 ? sm.lengths.total(1) == 1 : kraft == (1u << kLimit));
      if (!code_ok) sm.bad = 1;
    }
  }
  __syncthreads();
  if (tid == 0 && sm.bad) {
    T.status = kCorrupt;
    sm.bad = 0;
  }
  __syncthreads();
  if (T.status != kOk) {
    if (tid == 0) {
      *a.tab = T;
      *a.out_bytes = 0;
      *a.status = kCorrupt;
    }
    return;
  }
  if (tid < 256 && len) T.by_rank[T.rank0[len] + sm.lengths.before(tid, len) + rank] = (uint8_t)tid;
  __syncthreads();
  // two-level table, every entry decoded on its own thread: an 11-bit prefix
  // holds the code of length <= 11 it starts with; prefixes from first(12) / 2
  // on (where the codes longer than 11 bits begin, being the last codes) point
  // to 16-entry subtables over the next 4 bits; anything else matches no code
  const uint32_t p0 = T.first[kLutBits + 1] >> 1;
  for (uint32_t k = tid; k < (1u << kLutBits); k += 1024) {
    uint32_t e = 0;
    for (uint32_t l = 1; l <= kLutBits; ++l) {
      const uint32_t d = (k >> (kLutBits - l)) - T.first[l];
      if (d < T.count[l]) {
        e = l << 8 | T.by_rank[T.rank0[l] + d];
        break;
      }
    }
    if (e == 0 && k >= p0 && k - p0 < kMaxSubtables) e = 0x8000u | (k - p0);
    T.lut[k] = (uint16_t)e;
  }
  for (uint32_t k = tid; k < kMaxSubtables * 16; k += 1024) {
    const uint32_t prefix = p0 + k / 16;
    uint32_t e = 0;
    if (prefix < (1u << kLutBits)) {
      const uint32_t v = prefix << 4 | (k & 15u);  // 15-bit window
      for (uint32_t l = kLutBits + 1; l <= kLimit; ++l) {
        const uint32_t d = (v >> (kLimit - l)) - T.first[l];
        if (d < T.count[l]) {
          e = l << 8 | T.by_rank[T.rank0[l] + d];
          break;
        }
      }
    }
    T.lut2[k] = (uint16_t)e;
  }
  // record sizes from the table of code bits: 8 entries per thread per
  // tile, read with 16-byte loads before any size is written (the table
  // starts 16-byte aligned; sizes is 256-byte aligned)
  const uint32_t* bits_tab = reinterpret_cast<const uint32_t*>(a.in + kPre);
  for (uint64_t base = 0; base < T.N; base += 8 * 1024) {
    const uint64_t i0 = base + 8 * (uint64_t)tid;
    if (i0 >= T.N) continue;
    uint32_t bits[8];
    if (i0 + 8 <= T.N) {
      const uint4 lo = reinterpret_cast<const uint4*>(bits_tab + i0)[0];
      const uint4 hi = reinterpret_cast<const uint4*>(bits_tab + i0)[1];
      bits[0] = lo.x, bits[1] = lo.y, bits[2] = lo.z, bits[3] = lo.w;
      bits[4] = hi.x, bits[5] = hi.y, bits[6] = hi.z, bits[7] = hi.w;
    } else {
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) bits[k] = i0 + k < T.N ? bits_tab[i0 + k] : 0u;
    }
    uint32_t sz[16];
    bool bad = false;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      const uint64_t i = i0 + k;
      const uint32_t c = i < T.N ? (uint32_t)(T.n - i * kChunk < kChunk ? T.n - i * kChunk : kChunk) : 0u;
      bad = bad || bits[k] > kLimit * c;
      sz[2 * k] = i < T.N ? offsets_bytes((c + kSub - 1) / kSub) : 0u;
      sz[2 * k + 1] = 4 * ((bits[k] + 31) / 32);
    }
    if (bad) sm.bad = 1;
    if (i0 + 8 <= T.N) {
      uint4* dst = reinterpret_cast<uint4*>(a.sizes + 2 * i0);
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) dst[q] = make_uint4(sz[4 * q], sz[4 * q + 1], sz[4 * q + 2], sz[4 * q + 3]);
    } else {
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k)
        if (i0 + k < T.N) {
          a.sizes[2 * (i0 + k)] = sz[2 * k];
          a.sizes[2 * (i0 + k) + 1] = sz[2 * k + 1];
        }
    }
  }
  __syncthreads();
  const uint64_t sum = stream::scan_record_sizes<16>(a.sizes, T.N, a.offs, sm.scratch);
  if (tid == 0) {
    if (sm.bad || kPre + 4 * T.N + sum != a.in_bytes) {
      T.status = kCorrupt;
      *a.out_bytes = 0;
    } else {
      T.status = T.n > a.capacity ? kOutOfSpace : kOk;
      *a.out_bytes = T.n;
    }
    *a.status = T.status;
  }
  __syncthreads();
  // publish the tables
  const uint32_t* src = reinterpret_cast<const uint32_t*>(&T);
  uint32_t* dst = reinterpret_cast<uint32_t*>(a.tab);
  for (uint32_t k = tid; k < sizeof(DecTables) / 4; k += 1024) dst[k] = src[k];
}

constexpr uint32_t kDecWaves = 4;                // waves per decode workgroup
constexpr uint32_t kInStageWords = 1024;         // code words staged per chunk (8 bits/symbol)
constexpr uint32_t kMaxDecodeBlocks = 16384;

struct DecLds {
  alignas(8) uint16_t lut[1u << kLutBits];
  uint16_t lut2[kMaxSubtables * 16];
  uint32_t in[kDecWaves][2][kInStageWords];  // code words of each wave's two chunks
};

struct DecCode {
  const uint16_t* lut;
  const uint16_t* lut2;
  uint32_t long0;  // first 15-bit window of the codes longer than 11 bits
};

// 16 bytes at a 4-byte boundary (chunks start 4096 bytes apart in an output
// that is 4-byte aligned).
struct __attribute__((packed, aligned(4))) Quad {
  uint32_t v[4];
};

// Decodes the `cnt` symbols of one sub-block starting at bit `start` of the
// chunk's code words `wds` (nwords >= 1 of them) and writes them at `dst`;
// returns the bit position after them, or ~0u if one of them matches no code.
// Every lane runs all 128 steps, so the loop is uniform across the wave:
// steps past `cnt` decode whatever bits follow and are not written. Word
// reads are clamped to the last word instead of branching: bits past a
// sub-block's end never decide whether it ends exactly at its end bit. The
// bit buffer is refilled once per pair of symbols (after a refill it holds at
// least 32 bits; two codes take at most 30). The chain from one code to the
// next is one table read: the second-level entry of a longer code is at a
// place that the window alone gives (those codes are the last ones, so their
// windows are consecutive), and both tables are read at once.
template <typename WordPtr>
__device__ __forceinline__ uint32_t decode_sub(const DecCode& dc, WordPtr wds, uint32_t nwords,
                                               uint32_t start, uint32_t cnt, uint8_t* dst) {
  const uint32_t last = nwords - 1;
  uint32_t wi = start >> 5;
  const uint32_t w0 = wds[wi < last ? wi : last], w1 = wds[wi + 1 < last ? wi + 1 : last];
  wi += 2;
  uint64_t buf = ((uint64_t)w0 << 32 | w1) << (start & 31u);
  uint32_t avail = 64 - (start & 31u), p = start, p_end = start;
  bool bad = false;
  for (uint32_t j = 0; j < kSub; j += 16) {
    Quad q;
#pragma unroll
    for (uint32_t v = 0; v < 4; ++v) {
      uint32_t acc = 0;
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) {
        if ((u & 1u) == 0) {
          const uint32_t w = wds[wi < last ? wi : last];
          const bool take = avail < 32;
          buf |= take ? (uint64_t)w << (32 - avail) : 0ull;
          wi += take ? 1u : 0u;
          avail += take ? 32u : 0u;
        }
        const uint32_t peek = (uint32_t)(buf >> (64 - kLimit));
        uint32_t k2 = peek - dc.long0;
        k2 = k2 < kMaxSubtables * 16 ? k2 : 0u;
        const uint32_t e1 = dc.lut[peek >> (kLimit - kLutBits)];
        const uint32_t e2 = dc.lut2[k2];
        const uint32_t e = e1 & 0x8000u ? e2 : e1;
        uint32_t l = e >> 8;
        const uint32_t sym = e & 0xFFu;
        if (l == 0) bad = bad || j + 4 * v + u < cnt;
        l = l ? l : 1u;
        buf <<= l;
        avail -= l;
        p += l;
        p_end = j + 4 * v + u + 1 == cnt ? p : p_end;
        acc |= sym << (8 * u);
      }
      q.v[v] = acc;
    }
    if (j + 16 <= cnt) {
      *reinterpret_cast<Quad*>(dst + j) = q;
    } else {
#pragma unroll
      for (uint32_t b = 0; b < 16; ++b)
        if (j + b < cnt) dst[j + b] = (uint8_t)(q.v[b / 4] >> (8 * (b & 3u)));
    }
  }
  return bad ? ~0u : p_end;
}

// Each wave takes two chunks at a time (32 lanes each, one lane per
// 128-symbol sub-block): it stages the chunks' code words in LDS with
// coalesced loads and decodes every sub-block from LDS; each lane writes its
// own 128 bytes with 16-byte stores. Only the wave synchronises; a chunk with
// more than 4 KiB of code words (above 8 bits per symbol) is decoded from
// global memory instead.
// Bound by the latency of the chain table read -> shift -> table read, so by
// the waves at hand: with the decoded symbols staged in LDS too, 8 waves fit
// a compute unit (69 MB of LZSS stream: 146 us); without that stage 12 fit as
// workgroups of four (77 us), 16 as workgroups of eight (89 us) or of sixteen
// (slower still): the smaller groups are handed out more evenly.
__global__ __launch_bounds__(64 * kDecWaves) void decode_kernel(DecArgs a) {
  __shared__ DecLds sm;
  const DecTables* T = a.tab;
  if (T->status != kOk) return;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint64_t n = T->n, N = T->N;
  if ((uint64_t)blockIdx.x * kDecWaves * 2 >= N) return;
  {
    // the two tables are adjacent in both places
    const uint2* src = reinterpret_cast<const uint2*>(T->lut);
    uint2* dst = reinterpret_cast<uint2*>(sm.lut);
    constexpr uint32_t kPairs = (sizeof(sm.lut) + sizeof(sm.lut2)) / 8;
    for (uint32_t k = tid; k < kPairs; k += 64 * kDecWaves) dst[k] = src[k];
  }
  DecCode dc;
  dc.lut = sm.lut;
  dc.lut2 = sm.lut2;
  dc.long0 = (T->first[kLutBits + 1] >> 1) << (kLimit - kLutBits);
  __syncthreads();
  const uint32_t* bits_tab = reinterpret_cast<const uint32_t*>(a.in + kPre);
  const uint64_t rec_base = kPre + 4 * N;
  const uint32_t half = lane >> 5, k = lane & 31u;
  uint32_t* in = sm.in[wave][half];
  bool bad = false;
  for (uint64_t g = (uint64_t)blockIdx.x * kDecWaves + wave; 2 * g < N; g += (uint64_t)gridDim.x * kDecWaves) {
    const uint64_t i = 2 * g + half;
    const bool live = i < N;
    uint32_t c = 0, nsub = 0, bits = 0, nwords = 0;
    const uint8_t* rec = nullptr;
    const uint32_t* wds = nullptr;
    if (live) {
      c = (uint32_t)(n - i * kChunk < kChunk ? n - i * kChunk : kChunk);
      nsub = (c + kSub - 1) / kSub;
      rec = a.in + rec_base + a.offs[i];
      bits = bits_tab[i];
      nwords = (bits + 31) / 32;
      wds = reinterpret_cast<const uint32_t*>(rec + offsets_bytes(nsub));
    }
    const bool staged = nwords <= kInStageWords;
    if (live && staged)
#pragma unroll 8
      for (uint32_t q = k; q < nwords; q += 32) in[q] = wds[q];
    wave_sync();
    if (live && k < nsub) {
      const uint16_t* o16 = reinterpret_cast<const uint16_t*>(rec);
      const uint32_t start = o16[k];
      const uint32_t end = k + 1 < nsub ? o16[k + 1] : bits;
      const uint32_t cnt = k + 1 < nsub ? kSub : c - kSub * k;
      bool ok = !((k == 0 && start != 0) || end > bits || start > end || bits == 0);
      if (k + 1 == nsub && (nsub & 1u) && o16[nsub] != 0) ok = false;
      if (ok && k + 1 == nsub && (bits & 31u) && (wds[nwords - 1] << (bits & 31u)) != 0) ok = false;
      if (ok) {
        uint8_t* dst = a.out + i * kChunk + kSub * k;
        const uint32_t p = staged ? decode_sub(dc, (const uint32_t*)in, nwords, start, cnt, dst)
                                  : decode_sub(dc, wds, nwords, start, cnt, dst);
        ok = p == end;
      }
      bad = bad || !ok;
    }
    wave_sync();
  }
  if (bad) atomicExch(a.status, kCorrupt);
}

}  // namespace

hipError_t launch_compress(const EncArgs& a, hipStream_t s) {
  const uint64_t N = chunks(a.max_n);
  hipLaunchKernelGGL(hist_kernel, dim3(a.hist_blocks), dim3(256), 0, s, a);
  hipLaunchKernelGGL(build_kernel, dim3(1), dim3(1024), 0, s, a);
  if (N) hipLaunchKernelGGL(size_kernel, dim3((uint32_t)((N + 3) / 4)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, s, a);
  if (N) hipLaunchKernelGGL(encode_kernel, dim3((uint32_t)((N + kEncWaves - 1) / kEncWaves)),
                           dim3(64 * kEncWaves), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_decompress(const DecArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(dec_prepare_kernel, dim3(1), dim3(1024), 0, s, a);
  // a workgroup for every 2 * kDecWaves chunks that the stream and the output
  // can hold; those past the stream's own count leave at once
  uint64_t most = a.in_bytes > kPre ? (a.in_bytes - kPre) / 4 : 0;
  if (most > a.capacity / kChunk + 1) most = a.capacity / kChunk + 1;
  uint64_t blocks = (most + 2 * kDecWaves - 1) / (2 * kDecWaves);
  if (blocks > kMaxDecodeBlocks) blocks = kMaxDecodeBlocks;
  if (blocks)
    hipLaunchKernelGGL(decode_kernel, dim3((uint32_t)blocks), dim3(64 * kDecWaves), 0, s, a);
  return hipGetLastError();
}

}  // namespace huff
}  // namespace gpulz
