// The index stream of token-conditional coding: which of the k candidates the true token was (or
// that it was none of them), one symbol per position, coded under the model's own probabilities so
// that a position costs about the token's surprisal (Thm. "Sequential entropy bound", Sec. 4.2).
// See include/plc.h for the format.
//
// The stream is tiny next to the residuals (one symbol per position against 2*L*H*d of them), but with
// one session it is a single chain of n / 32 steps, so the per-position tables are prepared off the
// chain; words go straight to global memory at positions ranked from the emission mask.
#include <cmath>
#include <type_traits>

#include "plc_device.h"

namespace plc {
namespace {

constexpr int kLanes = PLC_RANS_LANES;
constexpr uint32_t kScale = PLC_RANS_SCALE;
constexpr uint32_t kLow = 1u << 16;
constexpr int kMaxK = 32;

// Probabilities of one row into registers, all k loads in flight (k <= MAXK; k is uniform).
template <int MAXK>
__device__ __forceinline__ void load_row(const float *__restrict__ p, int k, float (&v)[MAXK]) {
#pragma unroll
  for (int j = 0; j < MAXK; ++j)
    if (j < k) v[j] = p[j];
}

// Frequencies of the k + 1 index symbols of one probability row (zero behind them); returns false for an invalid
// row (its negative / NaN entries are taken as 0, so the table is usable either way).  In registers throughout:
// with the row in LDS and the loads inside the loop a position cost a memory latency per candidate.
template <int MAXK>
__device__ __forceinline__ bool index_table(const float (&p)[MAXK], int k, uint32_t (&f)[MAXK + 1]) {
  bool ok = true;
  float c = 0.0f;
  uint32_t prev = 0;
  uint64_t zero = 0;  // symbols without a frequency
#pragma unroll
  for (int j = 0; j <= MAXK; ++j) {
    uint32_t b = kScale;
    if (j < MAXK && j < k) {  // uniform
      float pj = p[j < MAXK ? j : 0];
      if (!(pj >= 0.0f)) {
        ok = false;
        pj = 0.0f;
      }
      c = c + pj;
      float scaled = __builtin_floorf(c * 4096.0f);
      if (!(scaled < 4096.0f)) scaled = 4096.0f;  // probability above one (or an overflow) is clipped
      b = (uint32_t)scaled;
    }
    f[j] = b - prev;
    prev = b;
    if (j <= k && f[j] == 0) zero |= 1ull << j;
  }
  // each takes a unit from the largest frequency of the moment, the lowest symbol on ties
  while (zero) {
    const int j = __builtin_ctzll(zero);
    zero &= zero - 1;
    uint32_t best = 0;
#pragma unroll
    for (int m = 0; m <= MAXK; ++m) {
      const uint32_t key = (f[m] << 6) | (uint32_t)(63 - m);
      best = key > best ? key : best;
    }
    const int donor = 63 - (int)(best & 63u);
#pragma unroll
    for (int m = 0; m <= MAXK; ++m) f[m] = m == j ? 1u : m == donor ? f[m] - 1u : f[m];
  }
  return ok;
}

// Both coders give a session one workgroup of four or eight wavefronts.  The chain of rANS steps is sequential,
// but what a step needs from its position -- the table made from that position's probabilities -- is not:
// the other wavefronts prepare the tables of the next groups (a position per thread, in registers, with the
// probabilities of the tile after already on their way) while wavefront 0 codes the current ones from LDS; one
// barrier per tile.  Bound by latency on both sides.  MAXK, 8, 16 or 32, is the row length the registers are laid out
// for, and what a position costs whatever its own length: up to 8 candidates, the ordinary case, the search of the
// decoder runs in registers too; rows of 9 to 16 laid out for 32 took longer than the rows in LDS had with thousands
// of sessions (4096 of 512 positions and 9 candidates: encode 65 us with rows in LDS, 78 in registers for 32, 44 in
// registers for 16; one session of 4096: 131, 100, 53 us).
// One session, encode / decode (before: rows in LDS, one load after the other, the decoder's results stored by
// wavefront 0, which waited for the stores at every word): 4096 positions of 8 candidates 23 / 31 us (43 / 91),
// 32,768 of 4 142 / 209 us (246 / 635), 4096 of 20 53 / 78 us (93 / 206), 8192 of 32 204 / 210 us (661 / 655).
// Where every session can have a compute unit to itself, seven helper wavefronts and tiles of fourteen groups: the tables
// of a tile took as long as its steps or longer (one session, encode / decode, with three and with seven: 32,768 positions
// of 4 candidates 157 / 233 and 142 / 209 us, 4096 of 20 87 / 92 and 53 / 78, 8192 of 32 285 / 301 and 204 / 210).  With
// more sessions the other wavefronts fill the chip, and the larger tiles cost LDS and registers: 1024 positions, encode / decode, with
// three and with seven, 256 sessions of 8 candidates 11.7 / 11.9 and 9.6 / 11.7 us, 257 11.8 / 13.0 and 12.9 / 15.3, 512 13.1 / 14.1 and
// 13.8 / 16.0; 256 of 32 54.6 / 57.2 and 42.5 / 45.0, 257 62.9 / 63.9 and 59.8 / 64.3, 768 of 512 positions 53.2 / 52.9 and 57.2 / 61.5.
constexpr int kTileGroupsFew = 14, kTileGroupsMany = 6;
constexpr int kIdxStageWords = 8192;            // decoder: index streams up to this many words are read from LDS

template <int MAXK, int kTileGroups>
__global__ __launch_bounds__(64 + kTileGroups * kLanes) void index_encode_kernel(const float *__restrict__ probs,
                                                           const int32_t *__restrict__ chosen, int n, int k,
                                                           uint32_t *__restrict__ states, uint16_t *__restrict__ words,
                                                           const uint64_t *__restrict__ word_off, uint64_t word_cap,
                                                           uint32_t *__restrict__ n_words, uint32_t *status) {
  __shared__ uint2 pair[2][kTileGroups][kLanes];  // f | cum << 16 of the symbol to code, 1 / f
  const int s = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint16_t *out = words + word_off[s];
  uint32_t x = kLow;
  uint64_t nw = 0;  // uniform
  const uint32_t above = ~((2u << (lane & 31)) - 1u);  // the lanes of a half above this one
  const int groups = (n + kLanes - 1) / kLanes;
  const int tiles = (groups + kTileGroups - 1) / kTileGroups;
  // tile t holds the kTileGroups groups below groups - kTileGroups * t (the encoder walks downwards)
  const int u = threadIdx.x - 64, gi_mine = u >> 5, l_mine = u & 31;  // of a helper thread
  auto position = [&](int t) {  // of its symbol in tile t, or -1
    const int g = groups - kTileGroups * t - 1 - gi_mine;
    const int i = g * kLanes + l_mine;
    return wave > 0 && g >= 0 && i < n ? i : -1;
  };
  float ahead[MAXK];
  int32_t chosen_ahead = 0;
  auto fetch = [&](int t) {
    const int i = position(t);
    if (i < 0) return;
    const int64_t row = (int64_t)s * n + i;
    load_row<MAXK>(probs + row * k, k, ahead);
    chosen_ahead = chosen[row];
  };
  fetch(0);
  for (int it = 0; it <= tiles; ++it) {
    if (wave > 0) {
      if (it < tiles) {
        const bool has = position(it) >= 0;
        float p[MAXK];
#pragma unroll
        for (int j = 0; j < MAXK; ++j) p[j] = ahead[j];
        int j = chosen_ahead;
        fetch(it + 1);
        uint32_t v = 1u;  // f = 1, cum = 0 for lanes without a symbol (never used)
        if (has) {
          uint32_t f[MAXK + 1];
          if (!index_table<MAXK>(p, k, f)) raise(status, PLC_ERR_INVALID);
          if (j < -1 || j >= k) {
            raise(status, PLC_ERR_INVALID);
            j = -1;
          }
          const int sym = j < 0 ? k : j;
          uint32_t cs = 0, fs = 0;
#pragma unroll
          for (int m = 0; m <= MAXK; ++m) {
            cs += m < sym ? f[m] : 0u;
            fs = m == sym ? f[m] : fs;
          }
          v = fs | (cs << 16);
        }
        pair[it & 1][gi_mine][l_mine] = make_uint2(v, __float_as_uint(1.0f / (float)(v & 0xffffu)));
      }
    } else if (it > 0) {
      const int t = it - 1;
      uint2 pr[kTileGroups];  // the tile's reads in flight together
#pragma unroll
      for (int gi = 0; gi < kTileGroups; ++gi) pr[gi] = pair[t & 1][gi][lane & 31];
#pragma unroll
      for (int gi = 0; gi < kTileGroups; ++gi) {
        const int g = groups - kTileGroups * t - 1 - gi;
        if (g < 0) continue;  // uniform
        // All 64 lanes: the upper half does what the lower does and stores nothing.  (With half of the lanes off vector
        // instructions take a third longer where every compute unit is at work; with one session it makes no difference.)
        const int l = lane & 31;
        const bool has = g * kLanes + l < n;
        const uint32_t fs = pr[gi].x & 0xffffu, cs = pr[gi].x >> 16;
        // The sequential definition visits lane 31 first: a lane's word comes after those of the
        // emitting lanes above it.
        const bool emit = has && (x >> 20) >= fs;
        const uint32_t mask = (uint32_t)__ballot(emit);
        const uint64_t pos = nw + (uint32_t)__builtin_popcount(mask & above);
        if (emit && lane < kLanes) {
          if (pos < word_cap) {
            out[pos] = (uint16_t)(x & 0xffffu);
          } else {
            raise(status, PLC_ERR_CAPACITY);
          }
        }
        x = emit ? x >> 16 : x;
        nw += (uint32_t)__builtin_popcount(mask);
        // x < f * 2^20, so x / f from the reciprocal is less than 2^20 * 4 * 2^-24 off, its whole part one at
        // most; the remainder puts it right
        uint32_t q = (uint32_t)((float)x * __uint_as_float(pr[gi].y));
        int32_t r = (int32_t)(x - q * fs);
        const int32_t less = r < 0 ? (int32_t)fs : r >= (int32_t)fs ? -(int32_t)fs : 0;
        q = r < 0 ? q - 1u : r >= (int32_t)fs ? q + 1u : q;
        r += less;
        x = has ? q * kScale + (uint32_t)r + cs : x;
      }
    }
    __syncthreads();
  }
  if (wave == 0) {
    if (lane < kLanes) states[(int64_t)s * kLanes + lane] = x;
    if (lane == 0) n_words[s] = (uint32_t)(nw < word_cap ? nw : word_cap);
  }
}

template <int MAXK, int kTileGroups>
__global__ __launch_bounds__(64 + kTileGroups * kLanes) void index_decode_kernel(const float *__restrict__ probs,
                                                           const uint32_t *__restrict__ states,
                                                           const uint16_t *__restrict__ words, uint64_t words_len,
                                                           const uint64_t *__restrict__ word_off,
                                                           const uint32_t *__restrict__ n_words, int n, int k,
                                                           int32_t *__restrict__ chosen, uint32_t *status) {
  constexpr int kTilePos = kTileGroups * kLanes;  // one to a thread of the helper wavefronts
  constexpr int kRowWords = (MAXK + 2) / 2;       // k + 2 cumulative values, two to a word; odd: rows on different banks
  static_assert(kRowWords % 2 == 1, "rows on different banks");
  // cumulative frequencies cum[0..k+1] of every position of a tile, two to a word (of rows laid out for 8, 4096 behind them)
  __shared__ uint32_t cums[2][kTilePos][kRowWords];
  // What a tile's positions decoded to, written out by the helpers; up to 8 candidates, their slots: the symbol in which a
  // slot lies is no part of the chain of steps and found by the helpers, which have made the rows.
  __shared__ std::conditional_t<MAXK == 8, uint16_t, int8_t> picked[2][kTilePos];
  __shared__ uint16_t wstage[kIdxStageWords];
  const int s = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool rans_lane = lane < kLanes;
  const uint64_t base = word_off[s];
  uint64_t ptr = n_words[s];  // uniform
  bool corrupt = base > words_len || ptr > words_len - base;
  if (corrupt) ptr = 0;
  // A session's index stream is short (a few bits per position): it is copied to LDS first, so that a
  // renormalising lane does not wait for HBM inside the chain of steps.  A longer one is read in place.
  const bool staged = ptr <= (uint64_t)kIdxStageWords;  // uniform
  if (staged)
    for (uint32_t i = threadIdx.x; i < (uint32_t)ptr; i += blockDim.x) wstage[i] = words[base + i];
  uint32_t x = rans_lane || MAXK == 8 ? states[(int64_t)s * kLanes + (lane & 31)] : kLow;
  const int groups = (n + kLanes - 1) / kLanes;
  const int tiles = (groups + kTileGroups - 1) / kTileGroups;
  const int u = threadIdx.x - 64;  // of a helper thread: its place in a tile
  float ahead[MAXK];
  auto fetch = [&](int t) {
    const int64_t i = (int64_t)kTilePos * t + u;
    if (wave > 0 && i < n) load_row<MAXK>(probs + ((int64_t)s * n + i) * k, k, ahead);
  };
  fetch(0);
  __syncthreads();
  // One tile's steps for up to 8 candidates, in all 64 lanes: the upper half does what the lower does (as in the
  // encoder).  The row is ten starts, two to a word; the distance from the slot down to the nearest
  // start at or below it is the smallest of the differences modulo 2^16, and so is the one up to the next.  One start after the
  // other took twice the instructions: one session of 4096 positions of 8 candidates 43 -> 33 us, of 32,768 of 4 322 -> 234,
  // 64 sessions of 2048 of 8 24 -> 19.
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  auto code_tile8 = [&](int t, auto from_lds) {
    constexpr bool kStaged = decltype(from_lds)::value;
    const int l = lane & 31;
    const uint32_t below = (1u << l) - 1u;
    const uint32_t(*tile)[kRowWords] = cums[t & 1];
    uint32_t v[5];
#pragma unroll
    for (int m = 0; m < 5; ++m) v[m] = tile[l][m];
    for (int gi = 0; gi < kTileGroups; ++gi) {
      const int g = kTileGroups * t + gi;
      if (g >= groups) break;  // uniform
      const bool has = g * kLanes + l < n;
      uint32_t next_v[5];  // asked for a step ahead
      const int ahead_gi = gi + 1 < kTileGroups ? gi + 1 : gi;
#pragma unroll
      for (int m = 0; m < 5; ++m) next_v[m] = tile[ahead_gi * kLanes + l][m];
      const uint32_t slot = x & (kScale - 1);
      const u16x2 at = __builtin_bit_cast(u16x2, slot * 0x10001u), behind = at + (uint16_t)1;
      u16x2 down = at - __builtin_bit_cast(u16x2, v[0]), up = __builtin_bit_cast(u16x2, v[0]) - behind;
#pragma unroll
      for (int m = 1; m < 5; ++m) {
        const u16x2 c = __builtin_bit_cast(u16x2, v[m]);
        down = __builtin_elementwise_min(down, (u16x2)(at - c));
        up = __builtin_elementwise_min(up, (u16x2)(c - behind));
      }
      const uint32_t r = down.x < down.y ? down.x : down.y;
      const uint32_t f = (uint32_t)(up.x < up.y ? up.x : up.y) + r + 1u;
      picked[t & 1][gi * kLanes + l] = (uint16_t)slot;
      const uint32_t xn = f * (x >> 12) + r;
      // Reading lanes are served from the end of the list, lane 0 first.
      const bool need = has && xn < kLow;
      const uint32_t mask = (uint32_t)__ballot(need);
      const uint32_t rank = (uint32_t)__builtin_popcount(mask & below), used = (uint32_t)__builtin_popcount(mask);
      uint32_t word = 0;
      if (kStaged) {  // (read by every lane, inside the stage)
        const uint32_t place = (uint32_t)ptr - 1u - rank;
        word = wstage[place < (uint32_t)kIdxStageWords ? place : 0u];
        word = rank < (uint32_t)ptr ? word : 0u;
      } else if (need && rank < ptr) {
        word = words[base + ptr - 1 - rank];
      }
      corrupt = corrupt || used > ptr;
      x = need ? (xn << 16) | word : has ? xn : x;
      ptr = used < ptr ? ptr - used : 0;
#pragma unroll
      for (int m = 0; m < 5; ++m) v[m] = next_v[m];
    }
  };
  // One tile's steps.  Wavefront 0 touches global memory only where the words are not staged: a wait for a load would
  // also be one for every store before it.
  auto code_tile = [&](int t, auto from_lds) {
    constexpr bool kStaged = decltype(from_lds)::value;
    const uint32_t(*tile)[kRowWords] = cums[t & 1];
    for (int gi = 0; gi < kTileGroups; ++gi) {
      const int g = kTileGroups * t + gi;
      if (g >= groups) break;  // uniform
      const int i = g * kLanes + lane;
      const bool has = rans_lane && i < n;
      const uint32_t slot = x & (kScale - 1);
      uint32_t sym = 0, cs = 0, next = kScale;
      // the last interval start at or below the slot, by halving; the last one found above it is its end
      const uint32_t *row = tile[gi * kLanes + (lane & 31)];
      for (uint32_t half = 32; half; half >>= 1) {
        if (half > (uint32_t)k) continue;  // uniform
        const uint32_t at = sym + half, within = at <= (uint32_t)k ? at : (uint32_t)k;
        const uint32_t w = row[within >> 1];
        const uint32_t c = at <= (uint32_t)k ? (at & 1 ? w >> 16 : w & 0xffffu) : kScale;
        const bool in = c <= slot;
        sym = in ? at : sym;
        cs = in ? c : cs;
        next = in ? next : c;
      }
      if (has) {
        picked[t & 1][gi * kLanes + lane] = (int8_t)(sym == (uint32_t)k ? -1 : (int)sym);
        x = (next - cs) * (x >> 12) + slot - cs;
      }
      // Reading lanes are served from the end of the list, lane 0 first.
      const bool need = has && x < kLow;
      const uint32_t mask = (uint32_t)__ballot(need);
      if (need) {
        const uint32_t below = mask & ((1u << lane) - 1u);
        const uint64_t rank = (uint32_t)__builtin_popcount(below);
        uint32_t word = 0;
        if (rank < ptr) {
          word = kStaged ? wstage[ptr - 1 - rank] : words[base + ptr - 1 - rank];
        } else {
          corrupt = true;
        }
        x = (x << 16) | word;
      }
      const uint32_t used = (uint32_t)__builtin_popcount(mask);
      ptr = used < ptr ? ptr - used : 0;
    }
  };
  // iteration it: tables of tile it, steps of tile it - 1, results of tile it - 2
  for (int it = 0; it <= tiles + 1; ++it) {
    if (wave > 0) {
      if (it >= 2) {
        const int64_t i = (int64_t)kTilePos * (it - 2) + u;
        int32_t sym = (int32_t)picked[it & 1][u];
        if (MAXK == 8) {  // the number of starts cum[1..k] at or below the slot, in the row of that tile, still in place
          const uint32_t slot = (uint32_t)sym;
          sym = 0;
#pragma unroll
          for (int m = 1; m <= 8; ++m) {
            const uint32_t w = cums[it & 1][u][m >> 1], c = (m & 1) ? w >> 16 : w & 0xffffu;
            sym += m <= k && c <= slot ? 1 : 0;
          }
          if (sym == k) sym = -1;
        }
        if (i < n) chosen[(int64_t)s * n + i] = sym;
      }
      if (it < tiles) {
        const bool has = (int64_t)kTilePos * it + u < n;
        float p[MAXK];
#pragma unroll
        for (int j = 0; j < MAXK; ++j) p[j] = ahead[j];
        fetch(it + 1);
        if (has) {
          uint32_t f[MAXK + 1];
          if (!index_table<MAXK>(p, k, f)) raise(status, PLC_ERR_INVALID);
          uint32_t *row = cums[it & 1][u];
          uint32_t acc = 0;
#pragma unroll
          for (int m = 0; m <= MAXK; m += 2) {
            const uint32_t odd = acc + f[m];
            if (MAXK == 8 || m <= k + 1) row[m / 2] = acc | (odd << 16);  // uniform (behind the last start: 4096)
            acc = odd + (m < MAXK ? f[m + 1 <= MAXK ? m + 1 : 0] : 0u);
          }
        }
      }
    } else if (it > 0 && it <= tiles) {
      if constexpr (MAXK == 8) {
        if (staged)
          code_tile8(it - 1, std::true_type{});
        else
          code_tile8(it - 1, std::false_type{});
      } else {
        if (staged)
          code_tile(it - 1, std::true_type{});
        else
          code_tile(it - 1, std::false_type{});
      }
    }
    __syncthreads();
  }
  if (wave == 0) {
    if (ptr != 0 || (rans_lane && x != kLow)) corrupt = true;
    if (corrupt) raise(status, PLC_ERR_CORRUPT);
  }
}

struct Thresholds {
  uint16_t thr[PLC_MAX_BITS + 1];
};

// Bit depth of every position from the frequency of its index symbol; one thread per position.
template <int MAXK>
__global__ __launch_bounds__(kBlock) void surprisal_bits_kernel(const float *__restrict__ probs,
                                                                const int32_t *__restrict__ chosen, int64_t rows,
                                                                int k, Thresholds t, int bmax,
                                                                uint8_t *__restrict__ bits, uint32_t *status) {
  const int64_t row = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (row >= rows) return;
  float p[MAXK];
  uint32_t f[MAXK + 1];
  load_row<MAXK>(probs + row * k, k, p);
  int j = chosen[row];
  if (!index_table<MAXK>(p, k, f)) raise(status, PLC_ERR_INVALID);
  if (j < -1 || j >= k) {
    raise(status, PLC_ERR_INVALID);
    j = -1;
  }
  const int sym = j < 0 ? k : j;
  uint32_t fs = 0;
#pragma unroll
  for (int m = 0; m <= MAXK; ++m) fs = m == sym ? f[m] : fs;
  int b = 1;
  for (int m = 2; m <= bmax; ++m)
    if (fs <= t.thr[m]) b = m;
  bits[row] = (uint8_t)b;
}

int check(const float *probs, int32_t S, int32_t n, int32_t k, const void *states, const void *word_off,
          const void *n_words, const void *chosen, const void *status) {
  if (S < 1 || n < 1 || k < 1 || k > kMaxK) return PLC_ERR_INVALID;
  if (!probs || !states || !word_off || !n_words || !chosen || !status) return PLC_ERR_INVALID;
  if (reinterpret_cast<uintptr_t>(probs) % 4 || reinterpret_cast<uintptr_t>(states) % 4 ||
      reinterpret_cast<uintptr_t>(word_off) % 8 || reinterpret_cast<uintptr_t>(n_words) % 4 ||
      reinterpret_cast<uintptr_t>(chosen) % 4 || reinterpret_cast<uintptr_t>(status) % 4)
    return PLC_ERR_INVALID;
  return PLC_OK;
}

// Tiles of fourteen groups or of six (see above).  Up to 192 positions are one tile of six groups, and four wavefronts are
// sooner at it than eight (256 sessions of 96 positions of 8 candidates, encode 4.06 and 4.18 us).  The decoder of rows of 9
// to 16 waits longer for the first large tile's tables than for a small one's, two wavefronts to a SIMD, and makes up for it
// only over many tiles (1 / 256 sessions of 16 candidates, six groups and fourteen: 512 positions 14.5 / 15.3 and 16.4 / 17.0 us,
// 1024 23.5 / 24.8 and 25.8 / 27.2, 2048 42.3 / 43.6 and 42.7 / 44.9, 4096 78.2 / 80.9 and 77.9 / 80.7, one of 32,768 581 and 555).
bool large_tiles(int32_t S, int32_t n, int32_t k, bool decode) {
  const bool late = decode && k > 8 && k <= 16;
  return S <= kComputeUnits && n >= (late ? 4096 : kTileGroupsMany * kLanes + 1);
}

}  // namespace
}  // namespace plc

using namespace plc;

extern "C" int plc_index_encode(const float *probs, const int32_t *chosen, int32_t S, int32_t n, int32_t k,
                                uint32_t *states, uint16_t *words, const uint64_t *word_off, uint64_t word_cap,
                                uint32_t *n_words, uint32_t *status, void *stream) {
  const int rc = check(probs, S, n, k, states, word_off, n_words, chosen, status);
  if (rc) return rc;
  if ((word_cap > 0 && !words) || reinterpret_cast<uintptr_t>(words) % 2) return PLC_ERR_INVALID;
  const bool large = large_tiles(S, n, k, false);
  constexpr int F = kTileGroupsFew, M = kTileGroupsMany;
  const auto kernel = large ? (k <= 8 ? index_encode_kernel<8, F> : k <= 16 ? index_encode_kernel<16, F> : index_encode_kernel<kMaxK, F>)
                            : (k <= 8 ? index_encode_kernel<8, M> : k <= 16 ? index_encode_kernel<16, M> : index_encode_kernel<kMaxK, M>);
  hipLaunchKernelGGL(kernel, dim3((unsigned)S), dim3(64 + kLanes * (large ? F : M)), 0, static_cast<hipStream_t>(stream), probs, chosen, n,
                     k, states, words, word_off, word_cap, n_words, status);
  return launch_status();
}

extern "C" int plc_index_decode(const float *probs, const uint32_t *states, const uint16_t *words,
                                uint64_t words_len, const uint64_t *word_off, const uint32_t *n_words, int32_t S,
                                int32_t n, int32_t k, int32_t *chosen, uint32_t *status, void *stream) {
  const int rc = check(probs, S, n, k, states, word_off, n_words, chosen, status);
  if (rc) return rc;
  if ((words_len > 0 && !words) || reinterpret_cast<uintptr_t>(words) % 2) return PLC_ERR_INVALID;
  const bool large = large_tiles(S, n, k, true);
  constexpr int F = kTileGroupsFew, M = kTileGroupsMany;
  const auto kernel = large ? (k <= 8 ? index_decode_kernel<8, F> : k <= 16 ? index_decode_kernel<16, F> : index_decode_kernel<kMaxK, F>)
                            : (k <= 8 ? index_decode_kernel<8, M> : k <= 16 ? index_decode_kernel<16, M> : index_decode_kernel<kMaxK, M>);
  hipLaunchKernelGGL(kernel, dim3((unsigned)S), dim3(64 + kLanes * (large ? F : M)), 0, static_cast<hipStream_t>(stream), probs, states, words,
                     words_len, word_off, n_words, n, k, chosen, status);
  return launch_status();
}

extern "C" int plc_surprisal_thresholds(double b0, double hbar, int32_t bmax, uint16_t *thr) {
  if (!(b0 > 0.0) || !(hbar > 0.0) || !(b0 < 1e300) || !(hbar < 1e300)) return PLC_ERR_INVALID;
  if (bmax < 1 || bmax > PLC_MAX_BITS || !thr) return PLC_ERR_INVALID;
  thr[0] = thr[1] = 0;
  for (int m = 2; m <= bmax; ++m) {
    // 4096 * 2^(-m * hbar / b0): the power of two scales the exponential exactly
    const double t = std::floor(std::ldexp(std::exp2(-((double)m * hbar) / b0), 12 /* log2 of the probability scale */));
    thr[m] = (uint16_t)(t < 0.0 ? 0.0 : t > 4096.0 ? 4096.0 : t);
  }
  return PLC_OK;
}

extern "C" int plc_surprisal_bits(const float *probs, const int32_t *chosen, int32_t S, int32_t n, int32_t k,
                                  const uint16_t *thr, int32_t bmax, uint8_t *bits, uint32_t *status,
                                  void *stream) {
  if (S < 1 || n < 1 || k < 1 || k > kMaxK || bmax < 1 || bmax > PLC_MAX_BITS) return PLC_ERR_INVALID;
  if (!probs || !chosen || !thr || !bits || !status) return PLC_ERR_INVALID;
  if (reinterpret_cast<uintptr_t>(probs) % 4 || reinterpret_cast<uintptr_t>(chosen) % 4 ||
      reinterpret_cast<uintptr_t>(status) % 4)
    return PLC_ERR_INVALID;
  Thresholds t = {};
  for (int m = 2; m <= bmax; ++m) {
    if (m > 2 && thr[m] > thr[m - 1]) return PLC_ERR_INVALID;
    t.thr[m] = thr[m];
  }
  const int64_t rows = (int64_t)S * n;
  const auto kernel = k <= 8 ? surprisal_bits_kernel<8> : k <= 16 ? surprisal_bits_kernel<16> : surprisal_bits_kernel<kMaxK>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)((rows + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                     static_cast<hipStream_t>(stream), probs, chosen, rows, k, t, bmax, bits, status);
  return launch_status();
}
