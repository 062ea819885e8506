// Single-buffer compression, match policy 0 (exact longest match) and 1 (the
// paper's single window pass), in one of two forms:
//   1- and 2-byte symbols, policy 1, and what the second form does not take: a
//     preparation kernel, then the chunk encoders (one workgroup per chunk),
//     which take chunk ids from an atomic ticket, find their record offsets by
//     decoupled look-back and write the table entry and record straight into
//     the stream;
//   4- and 8-byte symbols, MIN >= 2, chunks of at most 32 KiB: chunk sizes in
//     any order, a scan of them (many chunks), then the records.
// The encoders' steps are in bucket_device.h (narrow symbols, policy 1),
// wide_device.h and encode_device.h (the general ones).
#include "bucket_device.h"
#include "wide_device.h"

namespace gpulz {
namespace {

// Where the general encoders are taken, launches of at most this many chunks
// split the parse (measured crossovers on 256 CUs: about 1.5-2.5 K chunks for
// 1- and 2-byte symbols, 512 for 4-byte ones).
constexpr uint64_t kSpecMaxChunksNarrow = 1024;  // S <= 2
constexpr uint64_t kSpecMaxChunksWide = 512;     // S >= 4
// Launches of at most this many chunks take the bucket encoder with 16 waves
// per chunk instead of 4: one such workgroup fits each of the 256 CUs at a
// time. uint16 codes (C 2048, W 128), 16 waves and 4: 256 chunks 35.7 and
// 41.4 us, 512 chunks 66.1 and 48.8, 1024 chunks 124.9 and 63.2.
constexpr uint64_t kBucketFewChunks = 256;

__global__ __launch_bounds__(256) void prep_kernel(FusedArgs a) {
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t k = t; k < a.N; k += stride) a.desc[k] = 0;
  if (t < kMaxTickets) a.tickets[t] = 0;
  if (a.N == 0 && blockIdx.x == 0) {
    // no chunk: the stream is the header alone
    const uint64_t total = kHeaderBytes;
    const bool fits = total <= a.capacity;
    if (threadIdx.x == 0) {
      *a.out_bytes = total;
      *a.status = fits ? kOk : kOutOfSpace;
    }
    if (fits && threadIdx.x < kHeaderBytes)
      a.out[threadIdx.x] = stream::header_byte(threadIdx.x, a.nbytes, a.S, a.C, a.W, a.MIN,
                                               a.policy, 0, total, a.in + a.nbytes / a.S * a.S);
  }
}

// Chunk i with its stream context.
__device__ __forceinline__ enc::ChunkJob chunk_job(const FusedArgs& a, uint32_t S, uint64_t i) {
  const uint64_t cs = i * a.C;
  enc::ChunkJob job;
  job.src = a.in + cs * S;
  job.src_avail = a.nbytes - cs * S;
  job.c = (uint32_t)min<uint64_t>(a.C, a.m - cs);
  job.C = a.C;
  job.W = a.W;
  job.MIN = a.MIN;
  job.slot = a.slots + i * a.slot_bytes;
  job.flag_area = a.flag_area;
  job.sizes = nullptr;
  job.i = i;
  job.N = a.N;
  job.desc = a.desc;
  job.out = a.out;
  job.capacity = a.capacity;
  job.in = a.in;
  job.nbytes = a.nbytes;
  job.S = S;
  job.policy = a.policy;
  job.out_bytes = a.out_bytes;
  job.status = a.status;
  return job;
}

// The next ticket of this launch: chunk ids follow the order in which
// workgroups ask for them, which the look-back needs.
__device__ __forceinline__ uint64_t next_ticket(const FusedArgs& a) {
  return a.chunk0 + atomicAdd((unsigned long long*)&a.tickets[a.launch], 1ull);
}

// The chunk this workgroup encodes.
__device__ __forceinline__ enc::ChunkJob take_chunk(const FusedArgs& a, uint32_t S,
                                                    uint64_t* shared_item) {
  if (threadIdx.x == 0) *shared_item = next_ticket(a);
  __syncthreads();
  return chunk_job(a, S, *shared_item);
}

template <int S, int WC>
__global__ __launch_bounds__(64 * enc::kEncodeWaves) void encode_kernel(FusedArgs a) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ uint64_t item;
  const enc::ChunkJob job = take_chunk(a, S, &item);
  enc::encode_chunk<S, WC, true>(job, lds);
}

// The same encoder with the parse split across kSpecWaves waves, for
// launches with few chunks (then the serial parse of one chunk per CU is the
// whole run time).
template <int S, int WC>
__global__ __launch_bounds__(64 * enc::kSpecWaves) void encode_spec_kernel(FusedArgs a) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ uint64_t item;
  const enc::ChunkJob job = take_chunk(a, S, &item);
  enc::encode_chunk_spec<S, WC>(job, lds);
}

// 1- and 2-byte symbols with MIN >= 2: candidates from 2-symbol buckets, NT
// threads per chunk (see bucket_device.h). At least 6 waves per SIMD: the
// search waits on LDS reads, and its 69 registers leave room for 7. (The launches
// of 1024 threads have a CU for each workgroup: 4 waves per SIMD, and the compiler
// told so. 1 MiB of uint16 runs in turns with text, C 2048, W 128: 162 us, 173 without;
// codes the same.)
template <int S, int WC, int NT>
__global__ __launch_bounds__(NT)
__attribute__((amdgpu_waves_per_eu(NT == 1024 ? 4 : 6, NT == 1024 ? 4 : 8)))
void encode_bucket_kernel(FusedArgs a) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ uint64_t item;
  const enc::ChunkJob job = take_chunk(a, S, &item);
  enc::bucket::encode_chunk<S, WC, NT, true>(job, lds);
}

// ---- 4- and 8-byte symbols with MIN >= 2: sizes, scan, records -----------------
//
// With the look-back a chunk holds its LDS until every chunk before it is
// sized, which held these encoders to about 30 chunks a microsecond, whatever
// their work (a chunk of noisy data: 9 us of work, 29 us of waiting). Here the
// sizes come first, in any order, and the records are written by a kernel of
// their own: a chunk without pointers is copied from the input, which is read a
// second time (256 MiB float32 field: 520 us with the look-back).
//
// The workspace's descriptor area holds a word per chunk (payload bytes, flag
// bytes << 16, pointers << 31) and the record offset of every 64th chunk.
struct WideView {
  uint32_t* size;
  uint64_t* group;
};
__device__ __forceinline__ WideView wide_view(const FusedArgs& a) {
  WideView v;
  v.size = reinterpret_cast<uint32_t*>(a.desc);
  v.group = a.desc + (a.N + 1) / 2;
  return v;
}
constexpr uint32_t kWideGroup = 64;
// Launches of at most this many chunks need no scan launch: every writing
// workgroup sums the sizes itself. float32 field (C 4096, W 256), without the
// launch and with it: 257 chunks 25.3 and 28.7 us, 1024 chunks 31.1 and 34.0,
// 2048 chunks 42.8 and 44.0, 4096 chunks 68.8 and 66.1; float64 (C 2048, W 32),
// 2048 chunks 24.2 and 25.7, 4096 chunks 45.6 and 42.9.
constexpr uint64_t kWideSumChunks = 1024;
__device__ __forceinline__ uint32_t wide_bytes(uint32_t size) {
  return (size & 0xFFFFu) + (size >> 16 & 0x7FFFu);
}


template <int S, int WC, uint32_t kVectors, uint32_t kThreads>
__global__ __launch_bounds__(kThreads) void wide_size_kernel(FusedArgs a) {
  extern __shared__ __align__(16) uint8_t lds[];
  const uint64_t i = a.chunk0 + blockIdx.x;
  const enc::wide::Sized z =
      enc::wide::size_chunk<S, WC, kVectors, kThreads, kThreads == enc::wide::kFewThreads>(
          chunk_job(a, S, i), lds);
  if (threadIdx.x == 0) wide_view(a).size[i] = z.P | z.F << 16 | (z.pointers ? 1u << 31 : 0u);
}

// One workgroup: record offsets of the groups, the header, size and status.
constexpr uint32_t kScanThreads = 1024;
__global__ __launch_bounds__(kScanThreads) void wide_scan_kernel(FusedArgs a) {
  constexpr uint32_t kPer = 16;  // chunks per thread: four threads share a group
  __shared__ uint32_t wsum[kScanThreads / 64];
  const WideView w = wide_view(a);
  const uint32_t tid = threadIdx.x, lane = lane_id(), wid = tid >> 6;
  uint64_t carry = 0;
  for (uint64_t base = 0; base < a.N; base += kScanThreads * kPer) {
    const uint64_t i0 = base + (uint64_t)tid * kPer;
    uint32_t x[kPer], v = 0;  // a tile's record bytes stay below 2^31
    if (i0 + kPer <= a.N) {
#pragma unroll
      for (uint32_t k = 0; k < kPer; k += 4)
        *reinterpret_cast<uint4*>(x + k) = *reinterpret_cast<const uint4*>(w.size + i0 + k);
    } else {
#pragma unroll
      for (uint32_t k = 0; k < kPer; ++k) x[k] = i0 + k < a.N ? w.size[i0 + k] : 0u;
    }
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) v += wide_bytes(x[k]);
    const uint32_t incl = wave_incl_scan(v);
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    uint32_t before = 0, total = 0;
    for (uint32_t k = 0; k < kScanThreads / 64; ++k) {
      const uint32_t y = wsum[k];
      before += k < wid ? y : 0u;
      total += y;
    }
    if (tid % (kWideGroup / kPer) == 0 && i0 < a.N) w.group[i0 / kWideGroup] = carry + before + incl - v;
    carry += total;
    __syncthreads();
  }
  const uint64_t total = kHeaderBytes + 8 * a.N + carry;
  const bool fits = total <= a.capacity;
  if (tid == 0) {
    *a.out_bytes = total;
    *a.status = fits ? kOk : kOutOfSpace;
  }
  if (fits && tid < kHeaderBytes)
    a.out[tid] = stream::header_byte(tid, a.nbytes, a.S, a.C, a.W, a.MIN, a.policy, a.N, total,
                                     a.in + a.nbytes / a.S * a.S);
}

// kSum: no scan launch came before; every workgroup adds up all sizes itself, and
// the first writes the header, size and status.
template <int S, bool kSum, uint32_t kThreads>
__global__ __launch_bounds__(kThreads) void wide_write_kernel(FusedArgs a) {
  const WideView w = wide_view(a);
  const uint64_t i = a.chunk0 + blockIdx.x;
  const uint32_t tid = threadIdx.x, lane = lane_id();
  uint64_t off;
  uint32_t own;
  if constexpr (kSum) {
    __shared__ uint32_t sums[2 * kThreads / 64];
    uint32_t before = 0, all = 0;  // kWideSumChunks records: below 2^31
    for (uint32_t k = tid; k < a.N; k += kThreads) {
      const uint32_t x = wide_bytes(w.size[k]);
      before += k < i ? x : 0u;
      all += x;
    }
    before = readlane(wave_incl_scan(before), 63);
    all = readlane(wave_incl_scan(all), 63);
    if (lane == 0) {
      sums[2 * (tid >> 6)] = before;
      sums[2 * (tid >> 6) + 1] = all;
    }
    __syncthreads();
    off = 0;
    uint64_t total = kHeaderBytes + 8 * a.N;
#pragma unroll
    for (uint32_t k = 0; k < kThreads / 64; ++k) {
      off += sums[2 * k];
      total += sums[2 * k + 1];
    }
    const bool fits = total <= a.capacity;
    if (i == 0 && tid == 0) {
      *a.out_bytes = total;
      *a.status = fits ? kOk : kOutOfSpace;
    }
    if (!fits) return;  // nothing is written
    if (i == 0 && tid < kHeaderBytes)
      a.out[tid] = stream::header_byte(tid, a.nbytes, a.S, a.C, a.W, a.MIN, a.policy, a.N, total,
                                       a.in + a.nbytes / a.S * a.S);
    own = w.size[i];
  } else {
    if (*a.status != kOk) return;  // the stream does not fit: nothing is written
    const uint64_t g = i / kWideGroup;
    const uint32_t x = g * kWideGroup + lane <= i ? w.size[g * kWideGroup + lane] : 0u;
    own = readlane(x, (uint32_t)(i % kWideGroup));
    off = w.group[g] + readlane(wave_incl_scan(wide_bytes(x)), 63) - wide_bytes(own);
  }
  const enc::wide::Sized z = {own >> 16 & 0x7FFFu, own & 0xFFFFu, own >> 31 != 0};
  enc::wide::put_record(a.in + i * a.C * S, a.in + a.nbytes, a.slots + i * a.slot_bytes,
                        a.flag_area, z, a.out + kHeaderBytes + 8 * i,
                        a.out + kHeaderBytes + 8 * a.N + off, tid, kThreads);
}

// Policy-1 chunk encoder kernel: one workgroup per chunk.
template <int S>
__global__ __launch_bounds__(64 * enc::kEncodeWaves) void encode_scan_kernel(FusedArgs a) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ uint64_t item;
  const enc::ChunkJob job = take_chunk(a, S, &item);
  enc::encode_chunk_scan<S>(job, lds);
}

// The same with the equal slots found 32 at a time and the parse split over the
// lanes (see bucket_device.h), MIN >= 2.
constexpr uint32_t kScanThreadsPerChunk = 256;
template <int S>
__global__ __launch_bounds__(kScanThreadsPerChunk) void encode_scan_bits_kernel(FusedArgs a) {
  extern __shared__ __align__(16) uint8_t lds[];
  __shared__ uint64_t item;
  const enc::ChunkJob job = take_chunk(a, S, &item);
  enc::bucket::encode_chunk<S, 4, kScanThreadsPerChunk, true, true>(job, lds);
}

template <int S, int WC>
hipError_t launch_sw(const FusedArgs& a, uint32_t waves, hipStream_t s) {
  if constexpr (S <= 2) {
    constexpr int WF = enc::bucket::kFallbackWC<S, WC>;
    constexpr uint32_t kNT = 256;
    const uint32_t threads = a.N <= kBucketFewChunks ? 1024 : kNT;
    const size_t lds = enc::bucket::chunk_lds<S, WF>(a.C, a.W, threads);
    if (enc::bucket::takes(a.C, a.MIN, lds)) {
      const dim3 grid((uint32_t)a.nchunks), block(threads);
      if (threads == 1024)
        hipLaunchKernelGGL((encode_bucket_kernel<S, WF, 1024>), grid, block, lds, s, a);
      else
        hipLaunchKernelGGL((encode_bucket_kernel<S, WF, kNT>), grid, block, lds, s, a);
      return hipGetLastError();
    }
  }
  const size_t spec_lds = enc::spec_lds_bytes<S, WC>(a.C);
  const uint64_t spec_max = S <= 2 ? kSpecMaxChunksNarrow : kSpecMaxChunksWide;
  if (a.N <= spec_max && a.C <= enc::kSpecMaxSyms && spec_lds <= kMaxGroupLdsBytes) {
    hipLaunchKernelGGL((encode_spec_kernel<S, WC>), dim3((uint32_t)a.nchunks),
                       dim3(64 * enc::kSpecWaves), spec_lds, s, a);
    return hipGetLastError();
  }
  const size_t lds = enc::lds_bytes<S, WC>(a.C, waves);
  hipLaunchKernelGGL((encode_kernel<S, WC>), dim3((uint32_t)a.nchunks), dim3(64 * waves), lds, s, a);
  return hipGetLastError();
}

template <int S>
hipError_t launch_s(const FusedArgs& a, uint32_t waves, hipStream_t s) {
  if (a.policy == 1 && enc::bucket::takes_scan(a.C, S, a.MIN, kScanThreadsPerChunk)) {
    hipLaunchKernelGGL((encode_scan_bits_kernel<S>), dim3((uint32_t)a.nchunks),
                       dim3(kScanThreadsPerChunk),
                       enc::bucket::scan_lds(a.C, S, kScanThreadsPerChunk), s, a);
    return hipGetLastError();
  }
  if (a.policy == 1) {
    const size_t lds = enc::scan_lds_bytes(a.C, S);
    hipLaunchKernelGGL((encode_scan_kernel<S>), dim3((uint32_t)a.nchunks), dim3(64 * waves), lds,
                       s, a);
    return hipGetLastError();
  }
  switch ((a.W + 63) / 64) {
    case 1: return launch_sw<S, 1>(a, waves, s);
    case 2: return launch_sw<S, 2>(a, waves, s);
    case 3: return launch_sw<S, 3>(a, waves, s);
    default: return launch_sw<S, 4>(a, waves, s);
  }
}

}  // namespace

size_t encode_scan_lds_bytes(uint32_t C, uint32_t S) { return enc::scan_lds_bytes(C, S); }

size_t encode_lds_bytes(uint32_t C, uint32_t S, uint32_t W, uint32_t waves) {
  return enc::encode_lds(C, S, (W + 63) / 64, waves);
}

hipError_t launch_fused_prep(const FusedArgs& a, hipStream_t s) {
  const uint64_t want = (a.N + 2047) / 2048 + 1;
  const uint64_t blocks = want < 1024 ? want : 1024;
  hipLaunchKernelGGL(prep_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

bool takes_wide(uint32_t C, uint32_t S, uint32_t MIN, uint32_t policy) {
  return policy == 0 && enc::wide::takes(C, S, MIN) &&
         enc::wide::lds_bytes(C, S, 4) <= kMaxGroupLdsBytes;
}

namespace {
template <int S, int WC>
void launch_size(const FusedArgs& a, hipStream_t s) {
  const dim3 grid((uint32_t)a.nchunks);
  const bool half = a.C * S <= enc::wide::kMaxBytes / 2;
  constexpr uint32_t kFew = enc::wide::kFewThreads, V = enc::wide::kMaxVectors;
  if (a.N <= kSpecMaxChunksWide) {
    const size_t lds = enc::wide::few_area_bytes<S, WC>(a.C) + 4 * enc::wide::kShared;
    if (half)
      hipLaunchKernelGGL((wide_size_kernel<S, WC, V * 256 / kFew / 2, kFew>), grid, dim3(kFew), lds, s, a);
    else
      hipLaunchKernelGGL((wide_size_kernel<S, WC, V * 256 / kFew, kFew>), grid, dim3(kFew), lds, s, a);
    return;
  }
  const size_t lds = enc::wide::lds_bytes(a.C, S, WC);
  if (half)
    hipLaunchKernelGGL((wide_size_kernel<S, WC, V / 2, 256>), grid, dim3(256), lds, s, a);
  else
    hipLaunchKernelGGL((wide_size_kernel<S, WC, V, 256>), grid, dim3(256), lds, s, a);
}
template <int S>
hipError_t launch_wide_s(FusedArgs a, hipStream_t s) {
  auto each = [&](auto launch) {
    for (uint64_t c0 = 0; c0 < a.N; c0 += kMaxChunksPerLaunch) {
      a.chunk0 = c0;
      a.nchunks = a.N - c0 < kMaxChunksPerLaunch ? a.N - c0 : kMaxChunksPerLaunch;
      launch();
    }
  };
  each([&] {
    switch ((a.W + 63) / 64) {
      case 1: launch_size<S, 1>(a, s); break;
      case 2: launch_size<S, 2>(a, s); break;
      case 3: launch_size<S, 3>(a, s); break;
      default: launch_size<S, 4>(a, s); break;
    }
  });
  if (a.N <= kBucketFewChunks && a.C * S > enc::wide::kMaxBytes / 2) {
    hipLaunchKernelGGL((wide_write_kernel<S, true, 1024>), dim3((uint32_t)a.N), dim3(1024), 0, s, a);
    return hipGetLastError();
  }
  if (a.N <= kWideSumChunks) {
    hipLaunchKernelGGL((wide_write_kernel<S, true, 256>), dim3((uint32_t)a.N), dim3(256), 0, s, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(wide_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, a);
  each([&] {
    hipLaunchKernelGGL((wide_write_kernel<S, false, 256>), dim3((uint32_t)a.nchunks), dim3(256), 0, s, a);
  });
  return hipGetLastError();
}
}  // namespace

hipError_t launch_wide(const FusedArgs& a, hipStream_t s) {
  return a.S == 4 ? launch_wide_s<4>(a, s) : launch_wide_s<8>(a, s);
}

hipError_t launch_fused_encode(const FusedArgs& a, uint32_t waves, hipStream_t s) {
  if (a.nchunks == 0) return hipSuccess;
  switch (a.S) {
    case 1: return launch_s<1>(a, waves, s);
    case 2: return launch_s<2>(a, waves, s);
    case 4: return launch_s<4>(a, waves, s);
    default: return launch_s<8>(a, waves, s);
  }
}

}  // namespace gpulz
