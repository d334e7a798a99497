// Symbol statistics for the entropy coder: per-stream histograms (LDS atomics)
// and the integer frequency tables on the 2^12 scale.  Definitions are in
// include/plc.h.
#include "plc_device.h"

namespace plc {
namespace {

constexpr int kHistSegment = 64 * 1024;     // symbols per workgroup
constexpr int kBucketSegment = 128 * 1024;  // the same where there is a table per bit depth

__global__ __launch_bounds__(kBlock) void zero_u32_kernel(uint32_t *p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// Each workgroup counts one segment of one stream into LDS histograms, then adds the non-empty bins to
// the stream's global counts.  Lanes that meet at one counter, or at one bank, in an instruction are served one
// after the other, and quantised residuals crowd into a few symbols (a dozen on the token-conditional path).  So
// the workgroup has kHistCopies histograms, a lane using copy lane mod kHistCopies, and a symbol's copies lie side
// by side: lane and bank then go together whatever the symbols are, and only lanes 32 apart can meet.  256 streams
// of 1,048,576 symbols: 62-64 us however the symbols are distributed (4.3 TB/s); with eight copies a wavefront, of
// which equal symbols met in one of eight banks, 92 us for residuals 60 steps wide and 152 us for 0.6 steps.
constexpr int kHistCopies = 32;

// The sum of one counter's copies, each thread starting at another one (side by side they would share a bank).
template <int COPIES>
__device__ __forceinline__ uint32_t sum_copies(const uint32_t *row, int thread) {
  uint32_t c = 0;
#pragma unroll
  for (int r = 0; r < COPIES; ++r) c += row[(r + thread) & (COPIES - 1)];
  return c;
}

__global__ __launch_bounds__(kBlock) void histogram_kernel(const uint8_t *__restrict__ symbols,
                                                           int64_t syms_per_stream, uint32_t segs_per_stream,
                                                           uint32_t *__restrict__ counts) {
  __shared__ __attribute__((aligned(16))) uint32_t hist[256 * kHistCopies];
  const uint32_t stream = blockIdx.x / segs_per_stream;
  const uint32_t seg = blockIdx.x - stream * segs_per_stream;
  for (int i = threadIdx.x; i < 256 * kHistCopies / 4; i += kBlock)
    reinterpret_cast<uint4 *>(hist)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  uint32_t *mine = hist + (threadIdx.x & (kHistCopies - 1));

  const int64_t seg_begin = (int64_t)seg * kHistSegment;
  const int64_t seg_end = seg_begin + kHistSegment < syms_per_stream ? seg_begin + kHistSegment : syms_per_stream;
  const uint8_t *base = symbols + (int64_t)stream * syms_per_stream;
  const uint8_t *p = base + seg_begin;
  const uint8_t *end = base + seg_end;
  // bytes before the first 16-byte boundary
  const uintptr_t mis = reinterpret_cast<uintptr_t>(p) & 15u;
  int64_t head = mis ? 16 - (int64_t)mis : 0;
  if (head > end - p) head = end - p;
  if ((int64_t)threadIdx.x < head) atomicAdd(&mine[(uint32_t)p[threadIdx.x] * kHistCopies], 1u);
  p += head;
  const int64_t n_vec = (end - p) / 16;
  const uint4 *pv = reinterpret_cast<const uint4 *>(p);
  uint4 next = make_uint4(0u, 0u, 0u, 0u);
  if ((int64_t)threadIdx.x < n_vec) next = load16_stream(pv + threadIdx.x);
  for (int64_t i = threadIdx.x; i < n_vec; i += kBlock) {
    const uint4 v = next;
    if (i + kBlock < n_vec) next = load16_stream(pv + i + kBlock);
    const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int b = 0; b < 4; ++b) atomicAdd(&mine[((wds[j] >> (8 * b)) & 255u) * kHistCopies], 1u);
    }
  }
  p += n_vec * 16;
  if ((int64_t)threadIdx.x < end - p) atomicAdd(&mine[(uint32_t)p[threadIdx.x] * kHistCopies], 1u);
  __syncthreads();

  const uint32_t c = sum_copies<kHistCopies>(hist + threadIdx.x * kHistCopies, threadIdx.x);
  if (c) atomicAdd(&counts[(int64_t)stream * 256 + threadIdx.x], c);
}

// The same with one histogram per bit depth: the depth of a symbol is that of its position, and a
// thread's 16 symbols always share a position (positions hold a multiple of 16 symbols).  Sixteen copies of four
// tables are 64 KB, so a workgroup has eight wavefronts to share them, two workgroups to a compute unit.  The same
// sizes: 71-72 us, against 105-226 us with one copy a wavefront; counting a thread's zeros in a register besides,
// as that needed, costs more than the atomics it saves (82-86 us).
// Clearing and adding up the copies is a fixed cost of a segment -- for sixteen copies of four tables 40 LDS
// instructions a thread, where 4096 symbols are 16 for half the threads -- so short streams get fewer copies
// (bucket_copies below).
template <int COPIES, int THREADS>
__global__ __launch_bounds__(THREADS) void histogram_bucketed_kernel(
    const uint8_t *__restrict__ symbols, int64_t syms_per_stream, uint32_t segs_per_stream, uint32_t syms_per_pos,
    uint32_t streams_per_session, const uint8_t *__restrict__ bits, int n_tables, uint32_t *__restrict__ counts,
    uint32_t *status) {
  __shared__ __attribute__((aligned(16))) uint32_t hist[PLC_MAX_BITS * 256 * COPIES];
  const uint32_t stream = blockIdx.x / segs_per_stream;
  const uint32_t seg = blockIdx.x - stream * segs_per_stream;
  for (int i = threadIdx.x; i < n_tables * 256 * COPIES / 4; i += THREADS)
    reinterpret_cast<uint4 *>(hist)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  uint32_t *mine = hist + (threadIdx.x & (COPIES - 1));

  constexpr int64_t kStep = THREADS * 16;
  const int64_t seg_begin = (int64_t)seg * kBucketSegment;
  const int64_t seg_end = seg_begin + kBucketSegment < syms_per_stream ? seg_begin + kBucketSegment : syms_per_stream;
  const uint8_t *base = symbols + (int64_t)stream * syms_per_stream;
  const uint8_t *brow = bits + (int64_t)(stream / streams_per_session) * (syms_per_stream / syms_per_pos);
  int64_t t0 = seg_begin + (int64_t)threadIdx.x * 16;
  uint4 next = make_uint4(0u, 0u, 0u, 0u);
  int next_b = 1;
  if (t0 < seg_end) {
    next = load16_stream(base + t0);
    next_b = brow[(uint32_t)t0 / syms_per_pos];
  }
  for (; t0 < seg_end; t0 += kStep) {
    const uint4 v = next;
    int b = next_b;
    if (t0 + kStep < seg_end) {
      next = load16_stream(base + t0 + kStep);
      next_b = brow[(uint32_t)(t0 + kStep) / syms_per_pos];
    }
    if (b < 1 || b > n_tables) {
      raise(status, PLC_ERR_INVALID);
      b = 1;
    }
    uint32_t *h = mine + (b - 1) * 256 * COPIES;
    const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int q = 0; q < 4; ++q) atomicAdd(&h[((wds[j] >> (8 * q)) & 255u) * COPIES], 1u);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n_tables * 256; i += THREADS) {
    const uint32_t c = sum_copies<COPIES>(hist + i * COPIES, threadIdx.x);
    if (c) atomicAdd(&counts[(int64_t)stream * n_tables * 256 + i], c);
  }
}

// One wavefront per stream; lane L owns symbols 4L .. 4L+3.  `allow_empty`: a row without any count is
// not an error and gets all-zero frequencies (a bit depth that does not occur in a stream).
__global__ __launch_bounds__(kBlock) void build_freq_kernel(const uint32_t *__restrict__ counts, int64_t n_streams,
                                                            uint16_t *__restrict__ freq, uint16_t *__restrict__ cum,
                                                            bool allow_empty, uint32_t *status) {
  const int lane = threadIdx.x & 63;
  const int64_t stream = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  if (stream >= n_streams) return;  // uniform per wavefront
  const uint4 cv = *reinterpret_cast<const uint4 *>(counts + stream * 256 + lane * 4);
  const uint32_t cnt[4] = {cv.x, cv.y, cv.z, cv.w};

  // inclusive running counts C (64-bit)
  uint64_t run[4];
  run[0] = cnt[0];
  run[1] = run[0] + cnt[1];
  run[2] = run[1] + cnt[2];
  run[3] = run[2] + cnt[3];
  uint64_t inc = run[3];
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t up = __shfl_up(inc, off, 64);
    if (lane >= off) inc += up;
  }
  const uint64_t before = inc - run[3];
  const uint64_t T = __shfl(inc, 63, 64);
  if (T == 0) {
    if (lane == 0 && !allow_empty) raise(status, PLC_ERR_INVALID);
    *reinterpret_cast<uint2 *>(freq + stream * 256 + lane * 4) = make_uint2(0u, 0u);
    if (cum) {
      for (int r = 0; r < 4; ++r) cum[stream * 257 + lane * 4 + r] = 0;
      if (lane == 63) cum[stream * 257 + 256] = 0;
    }
    return;
  }
  // f[s] = floor(C[s] * 4096 / T) - floor(C[s-1] * 4096 / T).  The quotient, at most 4096, from the reciprocal in
  // fp64 (counts of 32 bits: C * 4096 <= 2^52 is exact there), off by one at most and put right by its remainder.
  const double inv = 1.0 / (double)T;
  auto scaled = [&](uint64_t c) {
    const int64_t n = (int64_t)(c * PLC_RANS_SCALE);
    int64_t q = (int64_t)(uint32_t)((double)n * inv);
    const int64_t rest = n - q * (int64_t)T;
    q += rest < 0 ? -1 : rest >= (int64_t)T ? 1 : 0;
    return (uint32_t)q;
  };
  uint32_t f[4];
  uint32_t prev = scaled(before);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint32_t cur = scaled(before + run[r]);
    f[r] = cur - prev;
    prev = cur;
  }
  // Symbols that occur but were scaled to zero take one unit each, one after the other, from the largest
  // frequency of the moment, the lowest symbol on ties.  Whose unit goes to whom does not matter (the frequencies
  // sum to 4096 over 256 symbols, so a donor holds 16 or more and a symbol raised to 1 is never one), and taking
  // n units that way brings everything above a level down to it: with L the lowest level for which
  // sum max(0, f - L) <= n, f becomes min(f, L) and the units still missing come from the lowest symbols at L.
  // L by halving, twelve sums over the wavefront (a repair at a time was an arg-max over it each: 17 us in all).
  uint32_t n_zero = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) n_zero += (uint32_t)__builtin_popcountll(__ballot(cnt[r] > 0 && f[r] == 0));
  if (n_zero) {  // uniform
    auto excess = [&](uint32_t level) {
      uint32_t e = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) e += f[r] > level ? f[r] - level : 0u;
      return wave_sum(e);
    };
    uint32_t level = 0;  // excess(level - 1) > n_zero, or level is 0
    for (uint32_t half = PLC_RANS_SCALE / 2; half; half >>= 1)
      if (excess(level + half - 1) > n_zero) level += half;
    uint32_t missing = n_zero - excess(level);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (cnt[r] > 0 && f[r] == 0) {
        f[r] = 1;
      } else {
        f[r] = f[r] < level ? f[r] : level;
      }
    }
    // the lane's four symbols come one after the other, so those at the level in lower lanes come first
    uint32_t mine = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) mine += f[r] == level ? 1u : 0u;
    uint32_t ahead = wave_inclusive_scan(mine) - mine;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (f[r] == level) {
        if (ahead < missing) f[r] -= 1;
        ++ahead;
      }
    }
  }
  *reinterpret_cast<uint2 *>(freq + stream * 256 + lane * 4) = make_uint2(f[0] | (f[1] << 16), f[2] | (f[3] << 16));
  if (cum) {
    uint32_t lane_sum = f[0] + f[1] + f[2] + f[3];
    uint32_t incf = lane_sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t up = __shfl_up(incf, off, 64);
      if (lane >= off) incf += up;
    }
    uint32_t acc = incf - lane_sum;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      cum[stream * 257 + lane * 4 + r] = (uint16_t)acc;
      acc += f[r];
    }
    if (lane == 63) cum[stream * 257 + 256] = (uint16_t)acc;
  }
}

}  // namespace
}  // namespace plc

using namespace plc;

extern "C" int plc_histogram(const uint8_t *symbols, int64_t n_streams, int64_t syms_per_stream, uint32_t *counts,
                             void *stream) {
  if (!symbols || !counts || n_streams < 1 || syms_per_stream < 1) return PLC_ERR_INVALID;
  if (syms_per_stream >= (1ll << 32)) return PLC_ERR_INVALID;
  if (reinterpret_cast<uintptr_t>(counts) % 16) return PLC_ERR_INVALID;
  const int64_t segs = (syms_per_stream + kHistSegment - 1) / kHistSegment;
  if (n_streams * segs >= (1ll << 31) || n_streams >= (1ll << 31) / 256) return PLC_ERR_INVALID;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t n = n_streams * 256;
  hipLaunchKernelGGL(zero_u32_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, counts, n);
  {
    TraceScope trace(PLC_TRACE_HISTOGRAM, st);
    hipLaunchKernelGGL(histogram_kernel, dim3((unsigned)(n_streams * segs)), dim3(kBlock), 0, st, symbols,
                       syms_per_stream, (uint32_t)segs, counts);
  }
  return launch_status();
}

extern "C" int plc_build_freq(const uint32_t *counts, int64_t n_streams, uint16_t *freq, uint16_t *cum,
                              uint32_t *status, void *stream) {
  if (!counts || !freq || !status || n_streams < 1) return PLC_ERR_INVALID;
  if (reinterpret_cast<uintptr_t>(counts) % 16 || reinterpret_cast<uintptr_t>(freq) % 8) return PLC_ERR_INVALID;
  if (cum && reinterpret_cast<uintptr_t>(cum) % 2) return PLC_ERR_INVALID;
  const int64_t blocks = (n_streams + kBlock / 64 - 1) / (kBlock / 64);
  if (blocks >= (1ll << 31)) return PLC_ERR_INVALID;
  hipLaunchKernelGGL(build_freq_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, static_cast<hipStream_t>(stream),
                     counts, n_streams, freq, cum, false, status);
  return launch_status();
}

// Copies of each table in histogram_bucketed_kernel.  Lanes of one copy meet where symbols crowd, which costs by the
// symbol; clearing and summing cost by the copy and table.  5120 streams, four tables, 4 / 8 / 16 copies, all symbols
// alike, residuals 0.6 and 30 steps wide: 4096 symbols 30, 27 and 22 / 31, 30 and 29 / 40 us, 8192: 42, 38 and 26 / 40,
// 37 and 32 / 45, 16,384: 67, 58 and 34 / 52, 49 and 40 / 53, 53 and 51, 24,576: 92, 80 and 41 / 67, 61 and 48 / 61,
// 60 and 58.  The lines lie where symbols that are all alike take no longer with fewer copies.  One table: 4096
// symbols 26, 22 and 13 / 21, 20 and 15 / 24 us, 16,384: 77, 62 and 27 / 44, 41 and 28 / 38, 38 and 35.
inline int bucket_copies(int64_t syms_per_stream, int n_tables) {
  return syms_per_stream <= 1024 * (n_tables + 1) ? 4 : syms_per_stream <= 4096 * n_tables ? 8 : 16;
}

extern "C" int plc_histogram_bucketed(const uint8_t *symbols, int64_t n_streams, int64_t syms_per_stream,
                                      int32_t syms_per_pos, int32_t streams_per_session, const uint8_t *bits,
                                      int32_t n_tables, uint32_t *counts, uint32_t *status, void *stream) {
  if (!symbols || !counts || !bits || !status || n_streams < 1 || syms_per_stream < 1) return PLC_ERR_INVALID;
  if (syms_per_stream >= (1ll << 32) || n_tables < 1 || n_tables > PLC_MAX_BITS) return PLC_ERR_INVALID;
  if (syms_per_pos < 32 || syms_per_pos % 32 || syms_per_stream % syms_per_pos || streams_per_session < 1)
    return PLC_ERR_INVALID;
  if (reinterpret_cast<uintptr_t>(counts) % 16 || reinterpret_cast<uintptr_t>(symbols) % 16) return PLC_ERR_INVALID;
  const int64_t segs = (syms_per_stream + kBucketSegment - 1) / kBucketSegment;
  if (n_streams * segs >= (1ll << 31) || n_streams >= (1ll << 31) / (256 * PLC_MAX_BITS)) return PLC_ERR_INVALID;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t n = n_streams * n_tables * 256;
  hipLaunchKernelGGL(zero_u32_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, counts, n);
  const int copies = bucket_copies(syms_per_stream, n_tables);
  const auto kernel = copies == 4   ? histogram_bucketed_kernel<4, 256>
                      : copies == 8 ? histogram_bucketed_kernel<8, 256>
                                    : histogram_bucketed_kernel<16, 512>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(n_streams * segs)), dim3(copies == 16 ? 512 : 256), 0, st, symbols,
                     syms_per_stream, (uint32_t)segs, (uint32_t)syms_per_pos, (uint32_t)streams_per_session, bits,
                     n_tables, counts, status);
  return launch_status();
}

extern "C" int plc_build_freq_bucketed(const uint32_t *counts, int64_t n_streams, int32_t n_tables, uint16_t *freq,
                                       uint32_t *status, void *stream) {
  if (!counts || !freq || !status || n_streams < 1 || n_tables < 1 || n_tables > PLC_MAX_BITS) return PLC_ERR_INVALID;
  if (reinterpret_cast<uintptr_t>(counts) % 16 || reinterpret_cast<uintptr_t>(freq) % 8) return PLC_ERR_INVALID;
  const int64_t rows = n_streams * n_tables;
  const int64_t blocks = (rows + kBlock / 64 - 1) / (kBlock / 64);
  if (blocks >= (1ll << 31)) return PLC_ERR_INVALID;
  hipLaunchKernelGGL(build_freq_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, static_cast<hipStream_t>(stream),
                     counts, rows, freq, (uint16_t *)nullptr, true, status);
  return launch_status();
}
