// 32-lane interleaved rANS encoder and decoder.  The bitstream is defined in
// include/plc.h.  The paper only asks for "standard source coding" of the
// residuals (proof of Prop. "Layer orthogonality", Sec. 6.1); interleaved rANS
// is the choice made here because its 32 lanes advance in lock step inside a
// wavefront and the shared word list is addressed with a ballot and a lane
// count, without atomics, so the output is deterministic.
//
// Mapping.  One wavefront codes one unit: lanes 0-31 carry the 32 rANS states
// and lanes 32-63 mirror them exactly (same state, same LDS addresses, same
// values), so that no step needs a lane mask and everything uniform stays in
// scalar registers; all 64 lanes move data between HBM and LDS.  A workgroup holds up to eight
// wavefronts that code consecutive units of the SAME stream and share that
// stream's table in LDS.  Per unit the work is a chain of N/32 dependent
// steps, so the kernels are bound by instruction issue and LDS latency times
// the chain length, and by how many units are in flight -- not by HBM.  The
// inner step is therefore written for a minimal instruction count: symbols,
// words and table entries go through LDS staging buffers that are filled and
// drained 16 groups at a time, and everything uniform stays in scalar
// registers.
#include "plc_device.h"

#include <optional>
#include <type_traits>

namespace plc {
namespace {

constexpr int kLanes = PLC_RANS_LANES;
constexpr int kScaleBits = 12;
constexpr uint32_t kScale = PLC_RANS_SCALE;
constexpr uint32_t kLow = 1u << 16;
constexpr int kBatch = 16;                      // symbol groups per staging round
constexpr int kBatchSyms = kBatch * kLanes;     // 512
constexpr int kSuper = 4;                       // encoder: batches fetched per staging round, so that
constexpr int kSuperGroups = kSuper * kBatch;   // the next round's HBM latency hides behind 64 groups
constexpr int kSuperSyms = kSuperGroups * kLanes;
constexpr int kSymStage = kSuperSyms + 32;      // 2048 symbols at any 16-byte misalignment
constexpr int kStagePieces = 3;                 // 16-byte pieces per lane and round (192 >= 130)
constexpr int kMaxWaves = 8;

struct RansArgs {
  const uint8_t *sym_in;       // encode
  uint8_t *sym_out;            // decode
  const uint16_t *freq;
  uint32_t *states_out;        // encode
  const uint32_t *states_in;   // decode
  uint16_t *words_out;         // encode
  const uint16_t *words_in;    // decode
  uint64_t words_len;          // decode
  const uint64_t *word_off;
  uint64_t word_cap;           // encode
  uint32_t *n_words_out;       // encode
  const uint32_t *n_words_in;  // decode
  uint32_t *status;
  int64_t n_units, units_per_stream, syms_per_stream, unit_syms;
  uint32_t wgs_per_stream;
  uint32_t pair_wgs_per_stream;  // rans_encode_pair_kernel with one table: workgroups per stream
  // one table per bit depth (the *_bucketed calls): symbol t of a stream uses table bits[...] - 1 of its position
  const uint8_t *bits;
  int32_t syms_per_pos, streams_per_session, n_tables;
  // reconstruction inside the decoder (rans_decode_chain_kernel with candidates)
  ReconView recon;
  // restart points of streams coded as one unit (plc_restart; see "Pieces" below)
  uint32_t *points_out;        // encode
  const uint32_t *points_in;   // decode
  uint32_t *piece_state;       // decode, scratch: two words per piece
  int32_t point_stride;        // records per stream in points_*
  int32_t pieces;              // decode: pieces per stream a workgroup's unit is one of (0: units as coded)
  int32_t piece_batches;       // batches per piece
  int32_t point_step;          // decode: records per piece
  int32_t verified_pieces;     // decode: a stream all of whose so many pieces were verified is left alone
  // decode, nullable: escapes of each tile of a stream, where its units are whole tiles (see count_tiles)
  uint32_t *tile_cnt;
};

// Pieces.  The decoder of a stream that is one unit can begin in the middle of it if it knows what the sequential
// decoder would hold there: the 32 states, how many words are left and how many escapes lie ahead.  The encoder,
// which passes the same point on its way from the stream's end, leaves that in a record, and the decoder gives
// the pieces between records to workgroups of their own.  A record is a hint and nothing more: the workgroup that
// decodes up to it compares what it has arrived at with what the record says, and where all of a stream's pieces
// agree, each began exactly where the one before it ended, so that together they are the sequential decode.  A
// stream with a piece that does not (a record that belongs to other words, damage to the words) is decoded again
// from its start by a second launch, which otherwise returns at once; it alone reports errors.
//
// Piece i counts from the end of the stream, as the encoder goes: its groups of 32 symbols are
// [piece_top(i + 1), piece_top(i)).  Pieces end where one of the encoder's batches begins, so all but piece 0 are
// whole batches.  Record i stands at piece_top(i), i >= 1; record 0 holds the stream's own states and totals, by which
// records that belong to other words are told before anything is decoded by them.
__host__ __device__ __forceinline__ int32_t piece_top(int32_t G, int32_t pieces, int32_t piece_batches, int32_t i) {
  if (i == 0) return G;
  if (i >= pieces) return 0;
  const int32_t head = G % kBatch ? G % kBatch : kBatch;
  return G - head - (i * piece_batches - 1) * kBatch;
}
// A piece as its workgroup decodes it.
struct Piece {
  uint32_t begin, len;         // symbols, from the stream's start
  uint32_t words, words_left;  // words of the list that are left at its start and at its end
  uint32_t esc, esc_end;       // escapes of the stream in front of its start and in front of its end
  const uint32_t *states;      // at its start
  const uint32_t *end_states;  // at its end; null: the end of the stream
};
// Piece i (0 is the last) of a stream whose list has n_words words; false where the records cannot be true (uniform).
__device__ __forceinline__ bool load_piece(const RansArgs &a, int64_t stream, int32_t i, uint32_t n_words, Piece *p) {
  const int32_t G = (int32_t)((a.syms_per_stream + kLanes - 1) / kLanes);
  const uint32_t *rec = a.points_in + stream * a.point_stride * PLC_RESTART_WORDS;
  const uint32_t *end = rec + (int64_t)i * a.point_step * PLC_RESTART_WORDS;
  const uint32_t *at = end + (int64_t)a.point_step * PLC_RESTART_WORDS;
  const bool first = i + 1 == a.pieces;
  const uint32_t other = (rec[0] ^ a.states_in[stream * kLanes]) | (rec[kLanes] ^ n_words);  // (these two tell)
  p->begin = (uint32_t)piece_top(G, a.pieces, a.piece_batches, i + 1) * kLanes;
  p->len = (i == 0 ? (uint32_t)a.syms_per_stream : (uint32_t)piece_top(G, a.pieces, a.piece_batches, i) * kLanes) - p->begin;
  p->words = first ? n_words : at[kLanes];
  p->words_left = i == 0 ? 0u : end[kLanes];
  p->esc = first ? 0u : rec[kLanes + 1] - at[kLanes + 1];
  p->esc_end = i == 0 ? rec[kLanes + 1] : rec[kLanes + 1] - end[kLanes + 1];
  p->states = first ? a.states_in + stream * kLanes : at;
  p->end_states = i == 0 ? nullptr : end;
  return (other == 0) & (p->words <= n_words) & (p->words_left <= p->words);
}
// What a piece's workgroup found: the decoding wavefront's word and the reconstructing one's (two alike where none is).
__device__ __forceinline__ void report_piece(const RansArgs &a, int64_t stream, int32_t i, int which, bool good) {
  a.piece_state[(stream * a.pieces + i) * 2 + which] = good ? kPieceGood : 0u;
}
// For the launch behind the pieces': whether this stream needs no second decode (uniform).
__device__ __forceinline__ bool stream_verified(const RansArgs &a, int64_t stream) {
  return pieces_good(a.piece_state, a.verified_pieces, stream);
}

// Offset (in table entries of `stride` each) of the table that the 32 symbols from unit-relative group g on use.
__device__ __forceinline__ uint32_t group_table(const RansArgs &a, int64_t stream, int64_t begin, int32_t g,
                                                uint32_t stride, bool *bad) {
  // (a stream has fewer than 2^31 symbols and there are fewer than 2^31 streams: 32-bit divisions)
  const uint32_t spp = (uint32_t)a.syms_per_pos;
  const uint32_t pos = (uint32_t)(begin + (int64_t)g * kLanes) / spp;
  const uint32_t n_pos = (uint32_t)a.syms_per_stream / spp;
  int b = a.bits[(int64_t)((uint32_t)stream / (uint32_t)a.streams_per_session) * n_pos + pos];
  if (b < 1 || b > a.n_tables) {
    *bad = true;
    b = 1;
  }
  return (uint32_t)(b - 1) * stride;
}

// Frequencies of symbols 4*lane .. 4*lane+3 and the cumulative frequency in
// front of them, for all 64 lanes of a wavefront.  Returns the table's total.
__device__ __forceinline__ uint32_t load_freq4(const uint16_t *freq, int lane, uint32_t f[4], uint32_t *cum0) {
  const uint2 fv = *reinterpret_cast<const uint2 *>(freq + lane * 4);
  f[0] = fv.x & 0xffffu;
  f[1] = fv.x >> 16;
  f[2] = fv.y & 0xffffu;
  f[3] = fv.y >> 16;
  const uint32_t sum = f[0] + f[1] + f[2] + f[3];
  const uint32_t inc = wave_inclusive_scan(sum);
  *cum0 = inc - sum;
  return (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
}

__device__ __forceinline__ void wave_sync() {
  // LDS traffic of one wavefront executes in order; this only stops the
  // compiler from moving LDS accesses across a staging boundary.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A workgroup barrier that orders LDS traffic only: what the wavefront wrote to LDS is there when the others
// pass, and its global loads and stores stay in flight (__syncthreads waits for those too, and a store to HBM
// takes the better part of a microsecond to be acknowledged).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0), vmcnt and expcnt left alone
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// ---------------------------------------------------------------------------
// Encoder
// ---------------------------------------------------------------------------
// Table entry per symbol (16 bytes).  A step is
//     if x > thr: emit (x & 0xffff), x >>= 16        thr = f * 2^20 - 1  (f = 4096: 2^32 - 1)
//     x' = q * (4096 - f) + x + cum                  q = floor(x / f)
// and differs only in how the exact quotient is formed:
//   short form, usable when every f of the table is <= 2048 (the normal case):
//       q = mulhi(x, m) >> s   with s = ceil(log2 f) - 1, m = ceil(2^(32+s) / f).
//     Exact because x < f * 2^20 after the renormalisation: the error term x * (m*f - 2^(32+s))
//     stays below 2^(32+s) as long as f^2 <= 2^(12+s), i.e. s <= 10.  For f = 1 the multiplier
//     2^32 - 1 yields x - 1, and the missing 4095 is added to the entry's cum.
//       .x = m   .y = thr   .z = (4096 - f) | s << 24   .w = cum (+4095 if f = 1)
//   long form, for tables with an f > 2048: a reciprocal of 33 bits, 2^32 + m = floor(2^(32+l) / f) + 1 with
//   l = ceil(log2 f), whose leading bit is implied:
//       q = (mulhi(m, x) + x) >> l
//     Exact because the error term x * ((2^32 + m) * f - 2^(32+l)) <= x * f < f^2 * 2^20 <= 2^(32+l) for
//     l <= 12; and x * (2^32 + m) stays below 2^64 (x / f < 2^20), so the sum does not overflow.
//       .x = m   .y = thr   .z = (4096 - f) | l << 24   .w = cum
//   plain form, for tables whose frequencies are small or lucky: the reciprocal without a shift,
//       q = mulhi(x, m)  with m = ceil(2^32 / f)
//     Exact as long as x * (m*f - 2^32) stays below 2^32, i.e. f * (m*f - 2^32) <= 2^12: every f up to 70, some up to
//     a few hundred, the powers of two.  Residuals of some seven bits have such tables.  f = 1 as in the short form.
//       .x = m   .y = thr   .z = 4096 - f   .w = cum (+4095 if f = 1)
// A symbol with f = 0 gets .w = 1 << 31, which is collected and reported if it occurs in the data.
enum EncForm { kEncShort, kEncLong, kEncPlain };
// n / f and its remainder for a quotient of at most 2^17: in fp32 it is off by less than one, which the remainder puts
// right.  (The integer division is three times the instructions, and every wavefront does a dozen before it starts.)
__device__ __forceinline__ uint32_t small_quotient(uint32_t n, uint32_t f, uint32_t *rest) {
  uint32_t q = (uint32_t)((float)n * __builtin_amdgcn_rcpf((float)f));
  int32_t r = (int32_t)(n - q * f);
  if (r < 0) {
    --q;
    r += (int32_t)f;
  } else if ((uint32_t)r >= f) {
    ++q;
    r -= (int32_t)f;
  }
  *rest = (uint32_t)r;
  return q;
}
// ceil(2^(32+s) / f) for 1 < f <= 4096 and f > 2^s: 2^32 * 2^s / f by two divisions, numerators below 2^28; *over: by
// how much f times that exceeds 2^(32+s)
__device__ __forceinline__ uint32_t enc_reciprocal(uint32_t f, uint32_t s, uint32_t *over) {
  uint32_t r1, r2;
  const uint32_t q1 = small_quotient(1u << (s + 16), f, &r1);
  const uint32_t q2 = small_quotient(r1 << 16, f, &r2);
  *over = r2 ? f - r2 : 0u;
  return (q1 << 16) + q2 + (r2 ? 1u : 0u);
}
__device__ __forceinline__ bool enc_plain_fits(uint32_t f) {
  uint32_t over = 0;
  if (f > 1u) (void)enc_reciprocal(f, 0u, &over);
  return f * over <= kScale;
}
// The form for the tables of which a wavefront's lanes hold the frequencies (uniform).
__device__ __forceinline__ EncForm enc_form_of(const uint32_t f[4]) {
  if (__ballot(f[0] > 2048u || f[1] > 2048u || f[2] > 2048u || f[3] > 2048u) != 0) return kEncLong;
  const bool fits = enc_plain_fits(f[0]) && enc_plain_fits(f[1]) && enc_plain_fits(f[2]) && enc_plain_fits(f[3]);
  return __ballot(!fits) == 0 ? kEncPlain : kEncShort;
}
// The form that serves tables of both: any table is served by the long one, and by the short one unless it needs that.
__device__ __forceinline__ EncForm enc_form_for(EncForm a, EncForm b) {
  return a == kEncLong || b == kEncLong ? kEncLong : a == kEncShort || b == kEncShort ? kEncShort : kEncPlain;
}
template <EncForm FORM>
__device__ __forceinline__ uint4 make_enc_entry(uint32_t f, uint32_t cum) {
  constexpr bool LONG = FORM == kEncLong;
  if (f == 0) return make_uint4(0u, 0xffffffffu, 0u, 0x80000000u);
  const uint32_t l = f > 1 ? 32u - (uint32_t)__builtin_clz(f - 1) : 0u;  // ceil(log2 f)
  const uint32_t thr = f >= kScale ? 0xffffffffu : (f << 20) - 1u;
  if (LONG) {
    // floor((2^l - f) * 2^32 / f) by two 32-bit divisions (numerators stay below 2^28)
    uint32_t r1, r2;
    const uint32_t q1 = small_quotient(((1u << l) - f) << 16, f, &r1);
    const uint32_t m = (q1 << 16) + small_quotient(r1 << 16, f, &r2) + 1u;
    return make_uint4(m, thr, (kScale - f) | (l << 24), cum & 0xfffu);
  }
  if (f == 1) return make_uint4(0xffffffffu, thr, kScale - 1u, (cum & 0xfffu) + (kScale - 1u));
  const uint32_t s = FORM == kEncPlain ? 0u : l - 1u;
  uint32_t over;
  return make_uint4(enc_reciprocal(f, s, &over), thr, (kScale - f) | (s << 24), cum & 0xfffu);
}
__device__ __forceinline__ uint4 make_enc_entry(EncForm form, uint32_t f, uint32_t cum) {  // form uniform
  return form == kEncLong ? make_enc_entry<kEncLong>(f, cum)
         : form == kEncPlain ? make_enc_entry<kEncPlain>(f, cum) : make_enc_entry<kEncShort>(f, cum);
}

// Table entry of 8 bytes, for the coders with a table per bit depth.  .x = m; .y = (4096 - f) | s << 12 | .w << 18, negative for
// a symbol with f = 0; the threshold follows from f: f * 2^20 - 1 = ~((4096 - f) << 20) mod 2^32.
__device__ __forceinline__ uint2 pack_enc_entry(const uint4 e) {
  if (e.w & 0x80000000u) return make_uint2(0u, 0x80000000u);
  return make_uint2(e.x, (e.z & 0xfffu) | ((e.z >> 24) << 12) | (e.w << 18));
}
__device__ __forceinline__ uint4 unpack_enc_entry(const uint2 c) {
  return make_uint4(c.x, ~(c.y << 20), (c.y & 0xfffu) | ((c.y << 12) & 0x0f000000u), (uint32_t)((int32_t)c.y >> 18));
}

// One coding step.  Every lane stores its low 16 bits each time -- the emitting lanes into the word
// list, the others into a scratch slot of their own -- so that the step has no branch; `on` (MASKED
// only) is false for lanes that hold no symbol in a ragged group.
template <bool LONG, bool MASKED>
__device__ __forceinline__ void enc_step(uint32_t &x, const uint4 e, uint16_t *&wtop, uint16_t *scratch,
                                         uint32_t &flags, uint32_t below, bool on) {
  uint32_t m32 = (uint32_t)__builtin_amdgcn_uicmp(x, e.y, 34 /* unsigned > */);
  bool emit = x > e.y;
  if (MASKED) {
    emit = emit && on;
    m32 = (uint32_t)__builtin_amdgcn_ballot_w64(emit);
  }
  // hardware lane h carries rANS lane 31 - h, which the encoder visits first for h = 0; `below` is the
  // mask of the lanes under this one within its half, so that a mirror lane ranks like its twin
  // (`wtop` = next free slot of the batch's word list, uniform)
  uint16_t *slot = wtop + __builtin_popcount(m32 & below);
  *(emit ? slot : scratch) = (uint16_t)x;
  x = emit ? x >> 16 : x;
  wtop += __builtin_popcount(m32);
  uint32_t xn;
  if (LONG) {
    const uint32_t q = (__umulhi(e.x, x) + x) >> (e.z >> 24);
    xn = __umul24(q, e.z) + (x + e.w);
  } else {
    const uint32_t q = __umulhi(e.x, x) >> (e.z >> 24);
    xn = __umul24(q, e.z) + (x + e.w);
  }
  if (MASKED) {
    x = on ? xn : x;
    flags |= on ? e.w : 0u;
  } else {
    x = xn;
    flags |= e.w;
  }
}

// The same step for the unrolled batches, with its instruction order pinned.  A wavefront issues in order, an
// instruction every 4.6 cycles whether or not it needs the result before it, but reading the lane mask of a compare
// costs two wait states (8.6 cycles) unless other instructions stand there.  The step has two chains that both start
// at the compare -- the state update and the address of the word to store -- so they are interleaved one for one.
#define PLC_PIN() __builtin_amdgcn_sched_barrier(0)

template <bool LONG>
__device__ __forceinline__ void enc_step_pinned(uint32_t &x, const uint4 e, uint16_t *&wtop, uint16_t *scratch,
                                                uint32_t &flags, uint32_t below) {
  const uint32_t m32 = (uint32_t)__builtin_amdgcn_uicmp(x, e.y, 34 /* unsigned > */);
  const bool emit = x > e.y;
  PLC_PIN();
  const uint32_t x16 = x >> 16;
  PLC_PIN();
  const uint32_t under = m32 & below;
  PLC_PIN();
  const uint32_t xr = emit ? x16 : x;
  PLC_PIN();
  const uint32_t rank = (uint32_t)__builtin_popcount(under);
  PLC_PIN();
  const uint32_t t1 = __umulhi(e.x, xr);
  PLC_PIN();
  uint16_t *slot = wtop + rank;
  PLC_PIN();
  uint32_t q, xc;
  if (LONG) {
    q = (t1 + xr) >> (e.z >> 24);
  } else {
    q = t1 >> (e.z >> 24);
  }
  xc = xr + e.w;
  PLC_PIN();
  slot = emit ? slot : scratch;
  PLC_PIN();
  const uint32_t p = __umul24(q, e.z);
  PLC_PIN();
  *slot = (uint16_t)x;
  PLC_PIN();
  wtop += __builtin_popcount(m32);
  PLC_PIN();
  x = p + xc;
  PLC_PIN();
  flags |= e.w;
}

// One table per bit depth, a unit per wavefront: whole streams, with 22 KB of LDS seven to a compute unit
// (encode_depths_in_pairs says when), and chunks that are few, W of a stream to a workgroup (kFewChunks).
template <int W>
__global__ __launch_bounds__(W * 64) void rans_encode_kernel(const RansArgs a) {
  __shared__ uint4 table[PLC_MAX_BITS * 256];
  __shared__ uint16_t table_of_group_of[W][2][kSuperGroups];  // table offset of each staged group
  __shared__ __attribute__((aligned(16))) uint8_t sym_stage_of[W][2][kSymStage];
  __shared__ __attribute__((aligned(16))) uint16_t word_stage[W][kBatchSyms + 8 + 64];  // list + carry + scratch slots
  const int lane = threadIdx.x & 63, wave = W == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t stream = blockIdx.x / a.wgs_per_stream;
  const int64_t chunk = (int64_t)(blockIdx.x - stream * a.wgs_per_stream) * W + wave;

  bool long_form = false;
  {  // one table per bit depth; an all-zero table (a depth the stream does not use) holds only invalid entries
    uint32_t f[PLC_MAX_BITS][4], cum[PLC_MAX_BITS];
    for (int t = 0; t < a.n_tables; ++t) {
      const uint32_t total = load_freq4(a.freq + (stream * a.n_tables + t) * 256, lane, f[t], &cum[t]);
      if (total != kScale && total != 0 && threadIdx.x == 0) raise(a.status, PLC_ERR_INVALID);
      long_form = long_form || __ballot(f[t][0] > 2048u || f[t][1] > 2048u || f[t][2] > 2048u || f[t][3] > 2048u) != 0;
    }
    for (int t = 0; t < a.n_tables; ++t) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if ((r & (W - 1)) == wave)
          table[t * 256 + lane * 4 + r] = make_enc_entry(long_form ? kEncLong : kEncShort, f[t][r], cum[t]);
        cum[t] += f[t][r];
      }
    }
  }
  __syncthreads();
  if (chunk >= a.units_per_stream) return;  // no workgroup barrier below

  const int64_t unit = stream * a.units_per_stream + chunk;
  const int64_t begin = chunk * a.unit_syms;
  const int64_t rest = a.syms_per_stream - begin;
  const uint32_t len = (uint32_t)(rest < a.unit_syms ? rest : a.unit_syms);
  const uint8_t *ubase = a.sym_in + stream * a.syms_per_stream + begin;
  auto &table_of_group = table_of_group_of[wave];
  auto &sym_stage = sym_stage_of[wave];
  const uint32_t mis = (uint32_t)(reinterpret_cast<uintptr_t>(ubase) & 15u);
  const int32_t G = (int32_t)((len + kLanes - 1) / kLanes);
  const uint32_t top_syms = len - (uint32_t)(G - 1) * kLanes;  // symbols in the last group, 1..32
  uint16_t *wp = a.words_out + a.word_off[unit];
  uint16_t *wstage = word_stage[wave];
  uint16_t *scratch = wstage + kBatchSyms + 8 + lane;

  const int rl = 31 - (lane & 31);  // rANS lane carried by this hardware lane
  const uint32_t below = (1u << (lane & 31)) - 1u;
  const bool coder = lane < kLanes;
  const bool top_active = (uint32_t)rl < top_syms;
  uint32_t x = kLow, flags = 0;

  // Staging rounds walk the groups from the top, 64 groups per round (the first round takes what is
  // left over).  A round's symbols [32*glo, 32*ghi) are fetched as 16-byte pieces aligned in absolute
  // address and placed so that symbol (group ghi-1-j, lane l) always sits at  mis + l + 32 * (63 - j).
  bool bad_depth = false;
  // the table of the group that stage position `lane` will hold (group ghi - 64 + lane), fetched with the symbols
  auto group_load = [&](int32_t glo, int32_t ghi) -> uint32_t {
    const int32_t g = ghi - kSuperGroups + lane;
    if (ghi <= 0 || g < (glo > 0 ? glo : 0) || g >= ghi) return 0u;
    return group_table(a, stream, begin, g, 256u, &bad_depth);
  };
  auto stage_load = [&](int32_t glo, int32_t ghi, uint4 v[kStagePieces], bool take[kStagePieces]) {
    // byte offsets relative to the unit's first symbol; pointers are formed by plain pointer arithmetic
    // on the kernel argument so that the loads stay global (not flat) memory instructions
    const int64_t lo = (int64_t)(glo > 0 ? glo : 0) * kLanes;
    int64_t hi = (int64_t)(ghi > 0 ? ghi : 0) * kLanes;
    hi = hi < (int64_t)len ? hi : (int64_t)len;
#pragma unroll
    for (int i = 0; i < kStagePieces; ++i) {
      const int64_t off = lo - (int64_t)mis + (int64_t)(lane + 64 * i) * 16;  // 16-byte aligned in absolute address
      take[i] = ghi > 0 && off < hi;
      if (take[i]) v[i] = load16_stream(ubase + off);
    }
  };
  auto stage_store = [&](int buf, int32_t cnt, const uint4 v[kStagePieces], const bool take[kStagePieces]) {
#pragma unroll
    for (int i = 0; i < kStagePieces; ++i)
      if (take[i])
        *reinterpret_cast<uint4 *>(&sym_stage[buf][(lane + 64 * i) * 16 + kLanes * (kSuperGroups - cnt)]) = v[i];
  };
  // Words leave through an LDS list whose position p stands for the word at 16-byte-aligned address
  // (wp - pad) + vbase + p: the first `pad` positions of the unit are padding in front of its first word.
  // After each batch the complete 16-byte pieces are stored, one per lane, and the incomplete tail (< 8
  // words) moves to the front of the list.  Pieces that touch the padding or the end of the unit's
  // reservation are stored word by word.
  // (All of this bookkeeping is uniform; readfirstlane keeps it in scalar registers.)
  const uint32_t pad = __builtin_amdgcn_readfirstlane((uint32_t)((reinterpret_cast<uintptr_t>(wp) >> 1) & 7u));
  const uint32_t cap = a.word_cap < 0x7fffffffull ? (uint32_t)a.word_cap : 0x7fffffffu;  // a unit has < 2^31 symbols
  uint32_t vbase = 0;   // multiple of 8
  uint32_t fill = pad;  // positions of the list in use
  auto store_words = [&](uint32_t first_pos, uint32_t n_pos) {  // word-by-word, with all checks
    for (uint32_t p = first_pos + lane; p < first_pos + n_pos; p += 64) {
      const uint32_t v = vbase + p;
      if (v >= pad && v - pad < cap) wp[v - pad] = wstage[p];
    }
  };
  auto drain = [&](uint32_t new_fill_v) {
    const uint32_t new_fill = __builtin_amdgcn_readfirstlane(new_fill_v);
    wave_sync();
    const uint32_t full = new_fill / 8;  // at most 65 pieces
    const bool plain = vbase >= pad && vbase + 8 * full - pad <= cap;
    if (plain) {
      uint16_t *dst = wp + (vbase - pad);  // 16-byte aligned
      if ((uint32_t)lane < full)
        *reinterpret_cast<uint4 *>(dst + 8 * lane) = *reinterpret_cast<const uint4 *>(wstage + 8 * lane);
      if (full > 64 && lane == 0)
        *reinterpret_cast<uint4 *>(dst + 8 * 64) = *reinterpret_cast<const uint4 *>(wstage + 8 * 64);
    } else {
      store_words(0, 8 * full);
    }
    const uint32_t rest = new_fill - 8 * full;
    uint16_t carry = 0;
    if ((uint32_t)lane < rest) carry = wstage[8 * full + lane];
    wave_sync();
    if ((uint32_t)lane < rest) wstage[lane] = carry;
    vbase += 8 * full;
    fill = rest;
    wave_sync();
  };

  int32_t ghi = G;
  int32_t cnt_groups = G % kSuperGroups ? G % kSuperGroups : kSuperGroups;
  // groups of the first round that do not fill a batch (and the top group if it is ragged) run in a
  // rolled loop with lane masking; every other batch is 16 full groups, fully unrolled
  int32_t head_groups = cnt_groups % kBatch;
  if (head_groups == 0 && top_syms < kLanes) head_groups = kBatch;
  {
    uint4 v[kStagePieces];
    bool take[kStagePieces];
    stage_load(ghi - cnt_groups, ghi, v, take);
    stage_store(0, cnt_groups, v, take);
    table_of_group[0][lane] = (uint16_t)group_load(ghi - cnt_groups, ghi);
  }
  wave_sync();
  int buf = 0;
  while (ghi > 0) {
    const int32_t glo = ghi - cnt_groups;
    uint4 nv[kStagePieces];
    bool ntake[kStagePieces];
    stage_load(glo - kSuperGroups, glo, nv, ntake);  // next round, in flight while this one is coded
    const uint32_t ngt = group_load(glo - kSuperGroups, glo);
    const uint16_t *gt = table_of_group[buf];  // group j from the round's top sits at 63 - j
    const uint8_t *sb = &sym_stage[buf][mis + rl];
    int32_t j0 = 0;
    // The prefetched round is written to LDS after the first batch of this round and BEFORE that batch's
    // words are stored: waiting for the loads then does not also wait for freshly issued stores (loads
    // and stores share one counter).
    bool landed = false;
    if (head_groups) {
      uint16_t *wtop = wstage + fill;
      for (int32_t j = 0; j < head_groups; ++j) {
        const uint4 e = table[sb[kLanes * (kSuperGroups - 1 - j)] + gt[kSuperGroups - 1 - j]];
        if (long_form) {
          enc_step<true, true>(x, e, wtop, scratch, flags, below, j != 0 || top_active);
        } else {
          enc_step<false, true>(x, e, wtop, scratch, flags, below, j != 0 || top_active);
        }
      }
      stage_store(buf ^ 1, kSuperGroups, nv, ntake);
      table_of_group[buf ^ 1][lane] = (uint16_t)ngt;
      landed = true;
      drain((uint32_t)(wtop - wstage));
      j0 = head_groups;
    }
    for (; j0 < cnt_groups; j0 += kBatch) {
      const uint8_t *sbb = sb + kLanes * (kSuperGroups - kBatch - j0);  // lowest group of this batch
      uint32_t sy[kBatch];
      uint16_t *wtop = wstage + fill;
#pragma unroll
      for (int j = 0; j < kBatch; ++j) sy[j] = sbb[kLanes * (kBatch - 1 - j)];
      const uint16_t *gtb = gt + (kSuperGroups - kBatch - j0);
#pragma unroll
      for (int j = 0; j < kBatch; ++j) sy[j] += gtb[kBatch - 1 - j];
      // table entries are fetched four groups ahead of the chain, so that their LDS time hides behind it
      uint4 e[2][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) e[0][j] = table[sy[j]];
#pragma unroll
      for (int qt = 0; qt < kBatch / 4; ++qt) {
        if (qt + 1 < kBatch / 4) {
#pragma unroll
          for (int j = 0; j < 4; ++j) e[(qt + 1) & 1][j] = table[sy[4 * (qt + 1) + j]];
        }
        if (long_form) {
#pragma unroll
          for (int j = 0; j < 4; ++j) enc_step_pinned<true>(x, e[qt & 1][j], wtop, scratch, flags, below);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) enc_step_pinned<false>(x, e[qt & 1][j], wtop, scratch, flags, below);
        }
      }
      if (!landed) {
        stage_store(buf ^ 1, kSuperGroups, nv, ntake);
        table_of_group[buf ^ 1][lane] = (uint16_t)ngt;
        landed = true;
      }
      drain((uint32_t)(wtop - wstage));
    }
    wave_sync();
    buf ^= 1;
    ghi = glo;
    cnt_groups = kSuperGroups;
    head_groups = 0;
  }
  if (coder) a.states_out[unit * kLanes + rl] = x;
  store_words(0, fill);  // the incomplete last piece
  const uint32_t n_words = vbase + fill - pad;
  if (lane == 0) {
    a.n_words_out[unit] = n_words;
    if ((uint64_t)n_words > a.word_cap) raise(a.status, PLC_ERR_CAPACITY);
  }
  if (coder && (flags & 0x80000000u)) raise(a.status, PLC_ERR_INVALID);  // a symbol with f = 0 occurred
  if (bad_depth) raise(a.status, PLC_ERR_INVALID);
}

// ---------------------------------------------------------------------------
// Encoder for many units: two units per wavefront
// ---------------------------------------------------------------------------
// With thousands of units in flight a unit per wavefront is bound by instruction issue, not by latency (measured:
// 83 cycles of a SIMD per step of a unit, the ~21 instructions of a step at 4 cycles each), and half of every
// instruction's lanes only mirror the other half.  Here lanes 32-63 code a unit of their own: the step's
// instructions are the same, only the word positions are per half -- a lane ranks itself inside its own
// half of the compare's lane mask, and the list pointer is a per-lane value that advances by its half's
// count.  The two units of a wavefront have the same length: two consecutive whole chunks of a stream (one
// table), or two consecutive whole streams (TWO_TABLES); a unit without such a partner (an odd count, a
// shorter last chunk) is coded by the lower half while the upper half shadows it and stores nothing.
// Symbols and words are staged per half exactly as above.
// ADAPT, one table per bit depth: a stream's four tables serve all of a workgroup's units, and a group's table is looked
// up per half.  LDS decides how many workgroups are resident, so the entries take 8 bytes (the step is four instructions
// longer: with one table, where that is all it does, 5120 streams take 2455 instead of 2308 us) and a round two batches.
// 256 streams of 1,048,576 symbols in units of 4096: 566 us with a unit per wavefront; with two 342 (rounds of four
// batches), 283 (two), 307 (one), with entries of 8 bytes 265; units of 1024 1116 -> 366 us, of 16384 432 -> 250.
template <bool LONG, bool MASKED>
__device__ __forceinline__ void enc2_step(uint32_t &x, const uint4 e, uint16_t *&wtop, uint16_t *scratch,
                                          uint32_t &flags, uint32_t below, bool upper, bool on) {
  bool emit = x > e.y;
  if (MASKED) emit = emit && on;
  const uint64_t m = __builtin_amdgcn_ballot_w64(emit);
  const uint32_t mine = upper ? (uint32_t)(m >> 32) : (uint32_t)m;  // the emit mask of this lane's half
  uint16_t *slot = wtop + __builtin_popcount(mine & below);
  *(emit ? slot : scratch) = (uint16_t)x;
  x = emit ? x >> 16 : x;
  wtop += __builtin_popcount(mine);
  const uint32_t t1 = __umulhi(e.x, x);
  const uint32_t q = (LONG ? t1 + x : t1) >> (e.z >> 24);
  const uint32_t xn = __umul24(q, e.z) + (x + e.w);
  if (MASKED) {
    x = on ? xn : x;
    flags |= on ? e.w : 0u;
  } else {
    x = xn;
    flags |= e.w;
  }
}

template <bool LONG>
__device__ __forceinline__ void enc2_step_pinned(uint32_t &x, const uint4 e, uint16_t *&wtop, uint16_t *scratch,
                                                 uint32_t &flags, uint32_t below, bool upper) {
  const uint64_t m = __builtin_amdgcn_uicmp(x, e.y, 34 /* unsigned > */);
  const bool emit = x > e.y;
  PLC_PIN();
  const uint32_t x16 = x >> 16;
  PLC_PIN();
  const uint32_t mine = upper ? (uint32_t)(m >> 32) : (uint32_t)m;
  PLC_PIN();
  const uint32_t xr = emit ? x16 : x;
  PLC_PIN();
  const uint32_t under = mine & below;
  PLC_PIN();
  const uint32_t t1 = __umulhi(e.x, xr);
  PLC_PIN();
  const uint32_t rank = (uint32_t)__builtin_popcount(under);
  PLC_PIN();
  uint32_t q, xc;
  if (LONG) {
    q = (t1 + xr) >> (e.z >> 24);
  } else {
    q = t1 >> (e.z >> 24);
  }
  xc = xr + e.w;
  PLC_PIN();
  uint16_t *slot = wtop + rank;
  PLC_PIN();
  const uint32_t p = __umul24(q, e.z);
  PLC_PIN();
  slot = emit ? slot : scratch;
  PLC_PIN();
  wtop += __builtin_popcount(mine);
  PLC_PIN();
  *slot = (uint16_t)x;
  PLC_PIN();
  x = p + xc;
  PLC_PIN();
  flags |= e.w;
}

constexpr int kPairMaxWaves = 4;
// SUPER = batches of symbols staged per round.  Four, as above, is the efficient size (a round's bookkeeping is
// spread over 64 steps).  With whole streams a workgroup is one wavefront with two tables, and its LDS decides
// how many are resident: 18.8 KB with four batches (eight per compute unit), 14.7 KB with two (eleven).  Two is
// taken only where it lets every pair of streams be resident at once instead of leaving a second, mostly empty
// round (5120 streams: 3.3 -> 2.5 ms); where there are several full rounds anyway the shorter rounds cost more
// than the extra wavefronts gain (16,384 streams: 7.4 against 7.7 ms).
template <int W, bool TWO_TABLES, int SUPER = 4, bool ADAPT = false>
__global__ __launch_bounds__(W * 64) void rans_encode_pair_kernel(const RansArgs a) {
  constexpr int kPairGroups = SUPER * kBatch;                  // groups per staging round
  constexpr int kPairSymStage = kPairGroups * kLanes + 32;     // its symbols at any 16-byte misalignment
  constexpr int kPairPieces = (kPairSymStage + 1023) / 1024;   // 16-byte pieces per lane and round
  static_assert(!TWO_TABLES || W == 1, "whole streams: one pair of streams per workgroup");
  constexpr int kDepths = ADAPT ? PLC_MAX_BITS : 1, kStreams = TWO_TABLES ? 2 : 1;
  using Entry = std::conditional_t<ADAPT, uint2, uint4>;
  __shared__ Entry table[kStreams][kDepths * 256];
  __shared__ uint16_t table_of_group[ADAPT ? W : 1][2][2][kPairGroups];  // ADAPT: table offset of each staged group
  __shared__ __attribute__((aligned(16))) uint8_t sym_stage[W][2][2][kPairSymStage];                // [half][buffer]
  __shared__ __attribute__((aligned(16))) uint16_t word_stage[W][2][kBatchSyms + 8 + 64];       // list + carry + scratch slots
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5;
  const bool upper = half != 0;

  // ---- which units: unit[0] for lanes 0-31, unit[1] for lanes 32-63 (or none: the upper half then shadows unit[0])
  int64_t stream[2], begin[2];
  bool second;       // uniform: the upper half has a unit of its own
  bool live = true;  // uniform: this wavefront has a unit at all
  uint32_t len;
  if (TWO_TABLES) {
    stream[0] = 2 * (int64_t)blockIdx.x;
    second = stream[0] + 1 < a.n_units;
    stream[1] = second ? stream[0] + 1 : stream[0];
    begin[0] = begin[1] = 0;
    len = (uint32_t)a.syms_per_stream;
  } else {
    const int64_t st = blockIdx.x / a.pair_wgs_per_stream;
    const int64_t slot = (int64_t)(blockIdx.x - st * a.pair_wgs_per_stream) * W + wave;
    const int64_t n_full = a.syms_per_stream / a.unit_syms;  // chunks of full length
    const int64_t n_pairs = n_full / 2;
    int64_t chunk0;
    if (slot < n_pairs) {
      chunk0 = 2 * slot, second = true;
    } else if ((n_full & 1) && slot == n_pairs) {
      chunk0 = n_full - 1, second = false;                   // the odd full chunk
    } else {
      chunk0 = n_full, second = false;                       // the shorter last chunk
      live = slot == n_pairs + (n_full & 1) && n_full < a.units_per_stream;
    }
    stream[0] = stream[1] = st;
    begin[0] = chunk0 * a.unit_syms;
    begin[1] = second ? begin[0] + a.unit_syms : begin[0];
    const int64_t rest = a.syms_per_stream - begin[0];
    len = (uint32_t)(rest < a.unit_syms ? rest : a.unit_syms);
  }

  bool long_form = false;
  {  // table entries: every wavefront scans the frequencies; entry 4*lane + r is built by wavefront (4*lane + r) mod W
    const int n_tables = ADAPT ? a.n_tables : 1;
    uint32_t f[kStreams][kDepths][4], cum[kStreams][kDepths];
#pragma unroll
    for (int u = 0; u < kStreams; ++u) {
#pragma unroll
      for (int t = 0; t < kDepths; ++t) {
        if (t >= n_tables) break;
        const uint32_t total = load_freq4(a.freq + (stream[u] * n_tables + t) * 256, lane, f[u][t], &cum[u][t]);
        // (an all-zero table, of a depth the stream does not use, holds only invalid entries)
        if (total != kScale && !(ADAPT && total == 0) && threadIdx.x == 0) raise(a.status, PLC_ERR_INVALID);
        const uint32_t(&ft)[4] = f[u][t];
        long_form = long_form || __ballot(ft[0] > 2048u || ft[1] > 2048u || ft[2] > 2048u || ft[3] > 2048u) != 0;
      }
    }
#pragma unroll
    for (int u = 0; u < kStreams; ++u) {
#pragma unroll
      for (int t = 0; t < kDepths; ++t) {
        if (t >= n_tables) break;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int s = lane * 4 + r;
          if ((s & (W - 1)) == wave) {
            const uint4 e = make_enc_entry(long_form ? kEncLong : kEncShort, f[u][t][r], cum[u][t]);
            if constexpr (ADAPT) {
              table[u][t * 256 + s] = pack_enc_entry(e);
            } else {
              table[u][s] = e;
            }
          }
          cum[u][t] += f[u][t][r];
        }
      }
    }
  }
  __syncthreads();
  if (!live) return;  // no workgroup barrier below

  const int64_t unit[2] = {stream[0] * a.units_per_stream + begin[0] / a.unit_syms,
                           stream[1] * a.units_per_stream + begin[1] / a.unit_syms};
  const uint8_t *ubase[2] = {a.sym_in + stream[0] * a.syms_per_stream + begin[0],
                             a.sym_in + stream[1] * a.syms_per_stream + begin[1]};
  const uint32_t mis[2] = {(uint32_t)(reinterpret_cast<uintptr_t>(ubase[0]) & 15u),
                           (uint32_t)(reinterpret_cast<uintptr_t>(ubase[1]) & 15u)};
  const int32_t G = (int32_t)((len + kLanes - 1) / kLanes);
  const uint32_t top_syms = len - (uint32_t)(G - 1) * kLanes;  // symbols in the last group, 1..32
  uint16_t *wp[2] = {a.words_out + a.word_off[unit[0]], a.words_out + a.word_off[unit[1]]};
  uint16_t *wstage = word_stage[wave][half];               // this lane's half's list
  uint16_t *scratch = wstage + kBatchSyms + 8 + (lane & 31);
  // (a shadowing upper half writes its words to its own LDS list and never to global memory)

  const int rl = 31 - (lane & 31);  // rANS lane carried by this hardware lane
  const uint32_t below = (1u << (lane & 31)) - 1u;
  const bool top_active = (uint32_t)rl < top_syms;
  const Entry *mytable = table[TWO_TABLES ? half : 0];
  uint32_t x = kLow, flags = 0;

  // ADAPT: depth of the group that stage position `lane` will hold (group ghi - kPairGroups + lane), asked for with the
  // symbols; its range is checked when they land, so that nothing waits for it in between.
  bool bad_depth = false;
  const uint32_t spp = ADAPT ? (uint32_t)a.syms_per_pos : 1u;
  const uint8_t *depth_row[2] = {nullptr, nullptr};
  if (ADAPT) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      depth_row[h] = a.bits + (int64_t)((uint32_t)stream[h] / (uint32_t)a.streams_per_session) *
                                  ((uint32_t)a.syms_per_stream / spp);
  }
  auto depth_load = [&](int h, int32_t glo, int32_t ghi) -> uint32_t {
    const int32_t g = ghi - kPairGroups + lane;
    if (!ADAPT || lane >= kPairGroups || g < (glo > 0 ? glo : 0) || g >= ghi) return 1u;
    return depth_row[h][((uint32_t)begin[h] + (uint32_t)g * kLanes) / spp];
  };
  auto depth_store = [&](int h, int buf, uint32_t depth) {
    if (!ADAPT) return;
    const bool known = depth >= 1u && depth <= (uint32_t)a.n_tables;
    bad_depth = bad_depth || !known;
    if (lane < kPairGroups) table_of_group[wave][h][buf][lane] = (uint16_t)(known ? (depth - 1u) * 256u : 0u);
  };
  // Symbol staging per half, as in the kernel above: a round's symbols are fetched as 16-byte pieces aligned
  // in absolute address by all 64 lanes and placed so that symbol (group ghi-1-j, lane l) sits at
  // mis + l + 32 * (kPairGroups - 1 - j).
  auto stage_load = [&](int h, int32_t glo, int32_t ghi, uint4 v[kPairPieces], bool take[kPairPieces]) {
    const int64_t lo = (int64_t)(glo > 0 ? glo : 0) * kLanes;
    int64_t hi = (int64_t)(ghi > 0 ? ghi : 0) * kLanes;
    hi = hi < (int64_t)len ? hi : (int64_t)len;
#pragma unroll
    for (int i = 0; i < kPairPieces; ++i) {
      const int64_t off = lo - (int64_t)mis[h] + (int64_t)(lane + 64 * i) * 16;  // 16-byte aligned in absolute address
      take[i] = ghi > 0 && off < hi;
      if (take[i]) v[i] = load16_stream(ubase[h] + off);
    }
  };
  auto stage_store = [&](int h, int buf, int32_t cnt, const uint4 v[kPairPieces], const bool take[kPairPieces]) {
#pragma unroll
    for (int i = 0; i < kPairPieces; ++i)
      if (take[i])
        *reinterpret_cast<uint4 *>(&sym_stage[wave][h][buf][(lane + 64 * i) * 16 + kLanes * (kPairGroups - cnt)]) = v[i];
  };
  // Word lists per half, as above: position p of a list stands for the word at 16-byte-aligned address
  // (wp - pad) + vbase + p.
  const uint32_t pad[2] = {(uint32_t)__builtin_amdgcn_readfirstlane((int)((reinterpret_cast<uintptr_t>(wp[0]) >> 1) & 7u)),
                           (uint32_t)__builtin_amdgcn_readfirstlane((int)((reinterpret_cast<uintptr_t>(wp[1]) >> 1) & 7u))};
  const uint32_t cap = a.word_cap < 0x7fffffffull ? (uint32_t)a.word_cap : 0x7fffffffu;  // a unit has < 2^31 symbols
  uint32_t vbase[2] = {0u, 0u};          // multiples of 8
  uint32_t fill[2] = {pad[0], pad[1]};   // positions of each list in use
  const bool writes[2] = {true, second};
  auto store_words = [&](int h, uint32_t first_pos, uint32_t n_pos) {  // word-by-word, with all checks
    if (!writes[h]) return;
    const uint16_t *list = word_stage[wave][h];
    for (uint32_t p = first_pos + lane; p < first_pos + n_pos; p += 64) {
      const uint32_t v = vbase[h] + p;
      if (v >= pad[h] && v - pad[h] < cap) wp[h][v - pad[h]] = list[p];
    }
  };
  auto drain = [&](int h, uint32_t new_fill) {  // new_fill uniform
    uint16_t *list = word_stage[wave][h];
    const uint32_t full = new_fill / 8;  // at most 65 pieces
    const bool plain = vbase[h] >= pad[h] && vbase[h] + 8 * full - pad[h] <= cap;
    if (plain) {
      if (writes[h]) {
        uint16_t *dst = wp[h] + (vbase[h] - pad[h]);  // 16-byte aligned
        if ((uint32_t)lane < full)
          *reinterpret_cast<uint4 *>(dst + 8 * lane) = *reinterpret_cast<const uint4 *>(list + 8 * lane);
        if (full > 64 && lane == 0)
          *reinterpret_cast<uint4 *>(dst + 8 * 64) = *reinterpret_cast<const uint4 *>(list + 8 * 64);
      }
    } else {
      store_words(h, 0, 8 * full);
    }
    const uint32_t rest = new_fill - 8 * full;
    uint16_t carry = 0;
    if ((uint32_t)lane < rest) carry = list[8 * full + lane];
    wave_sync();
    if ((uint32_t)lane < rest) list[lane] = carry;
    vbase[h] += 8 * full;
    fill[h] = rest;
  };
  // after a batch: each half's new fill from its lanes' list pointer (uniform inside a half), both lists drained
  auto drain_both = [&](uint16_t *wtop) {
    const uint32_t mine = (uint32_t)(wtop - wstage);
    const uint32_t f0 = (uint32_t)__builtin_amdgcn_readlane((int)mine, 0);
    const uint32_t f1 = (uint32_t)__builtin_amdgcn_readlane((int)mine, 32);
    wave_sync();
    drain(0, f0);
    drain(1, f1);
    wave_sync();
  };

  auto entry = [](const Entry &e) {
    if constexpr (ADAPT) {
      return unpack_enc_entry(e);
    } else {
      return e;
    }
  };
  int32_t ghi = G;
  int32_t cnt_groups = G % kPairGroups ? G % kPairGroups : kPairGroups;
  // groups of the first round that do not fill a batch (and the top group if it is ragged) run in a
  // rolled loop with lane masking; every other batch is 16 full groups, fully unrolled
  int32_t head_groups = cnt_groups % kBatch;
  if (head_groups == 0 && top_syms < kLanes) head_groups = kBatch;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint4 v[kPairPieces];
    bool take[kPairPieces];
    stage_load(h, ghi - cnt_groups, ghi, v, take);
    const uint32_t depth = depth_load(h, ghi - cnt_groups, ghi);
    stage_store(h, 0, cnt_groups, v, take);
    depth_store(h, 0, depth);
  }
  wave_sync();
  int buf = 0;
  while (ghi > 0) {
    const int32_t glo = ghi - cnt_groups;
    uint4 nv[2][kPairPieces];
    uint32_t ndepth[2];
    bool ntake[2][kPairPieces];
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // next round, in flight
      stage_load(h, glo - kPairGroups, glo, nv[h], ntake[h]);
      ndepth[h] = depth_load(h, glo - kPairGroups, glo);
    }
    const uint16_t *gt = table_of_group[ADAPT ? wave : 0][half][buf];  // group j from the round's top sits at kPairGroups - 1 - j
    const uint8_t *sb = &sym_stage[wave][half][buf][(upper ? mis[1] : mis[0]) + rl];
    int32_t j0 = 0;
    bool landed = false;
    if (head_groups) {
      uint16_t *wtop = wstage + (upper ? fill[1] : fill[0]);
      for (int32_t j = 0; j < head_groups; ++j) {
        const uint4 e = entry(mytable[sb[kLanes * (kPairGroups - 1 - j)] + (ADAPT ? gt[kPairGroups - 1 - j] : 0u)]);
        if (long_form) {
          enc2_step<true, true>(x, e, wtop, scratch, flags, below, upper, j != 0 || top_active);
        } else {
          enc2_step<false, true>(x, e, wtop, scratch, flags, below, upper, j != 0 || top_active);
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        stage_store(h, buf ^ 1, kPairGroups, nv[h], ntake[h]);
        depth_store(h, buf ^ 1, ndepth[h]);
      }
      landed = true;
      drain_both(wtop);
      j0 = head_groups;
    }
    for (; j0 < cnt_groups; j0 += kBatch) {
      const uint8_t *sbb = sb + kLanes * (kPairGroups - kBatch - j0);  // lowest group of this batch
      uint32_t sy[kBatch];
      uint16_t *wtop = wstage + (upper ? fill[1] : fill[0]);
#pragma unroll
      for (int j = 0; j < kBatch; ++j) sy[j] = sbb[kLanes * (kBatch - 1 - j)];
      if (ADAPT) {
        const uint16_t *gtb = gt + (kPairGroups - kBatch - j0);
#pragma unroll
        for (int j = 0; j < kBatch; ++j) sy[j] += gtb[kBatch - 1 - j];
      }
      // table entries are fetched four groups ahead of the chain, so that their LDS time hides behind it
      Entry e[2][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) e[0][j] = mytable[sy[j]];
#pragma unroll
      for (int qt = 0; qt < kBatch / 4; ++qt) {
        if (qt + 1 < kBatch / 4) {
#pragma unroll
          for (int j = 0; j < 4; ++j) e[(qt + 1) & 1][j] = mytable[sy[4 * (qt + 1) + j]];
        }
        if (long_form) {
#pragma unroll
          for (int j = 0; j < 4; ++j) enc2_step_pinned<true>(x, entry(e[qt & 1][j]), wtop, scratch, flags, below, upper);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) enc2_step_pinned<false>(x, entry(e[qt & 1][j]), wtop, scratch, flags, below, upper);
        }
      }
      if (!landed) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          stage_store(h, buf ^ 1, kPairGroups, nv[h], ntake[h]);
          depth_store(h, buf ^ 1, ndepth[h]);
        }
        landed = true;
      }
      drain_both(wtop);
    }
    wave_sync();
    buf ^= 1;
    ghi = glo;
    cnt_groups = kPairGroups;
    head_groups = 0;
  }
  if (!upper || second) a.states_out[(upper ? unit[1] : unit[0]) * kLanes + rl] = x;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    store_words(h, 0, fill[h]);  // the incomplete last piece
    const uint32_t n_words = vbase[h] + fill[h] - pad[h];
    if (lane == 0 && writes[h]) {
      a.n_words_out[unit[h]] = n_words;
      if ((uint64_t)n_words > a.word_cap) raise(a.status, PLC_ERR_CAPACITY);
    }
  }
  if ((!upper || second) && (flags & 0x80000000u)) raise(a.status, PLC_ERR_INVALID);  // a symbol with f = 0 occurred
  if (bad_depth) raise(a.status, PLC_ERR_INVALID);
}

// ---------------------------------------------------------------------------
// Encoder for few, long units: seven wavefronts per unit
// ---------------------------------------------------------------------------
// When there are no more units than compute units, time is the length of one unit's chain of steps.  A lone
// wavefront issues strictly in order, so a step costs its instructions, wait states included -- and everything that
// is not the state recurrence moves to helper wavefronts of the same workgroup:
//   symbols brings the symbols from HBM to LDS (64 groups ahead);
//   feeder  (two) turns every (group, lane) of a batch into its 16-byte table entry at a fixed place of an LDS
//           ring; a lane without a symbol (ragged top group, or a step past the unit's first group) gets an
//           identity entry.  It runs two batches ahead of the coder, so that the coder can ask for the next
//           batch's first entries before the barrier;
//   coder   the recurrence alone, in all 64 lanes: lanes 32-63 code the same unit a step ahead of lanes 0-31, so that
//           what one half leaves in LDS of every second step is, for the other, the state behind the one before;
//   packer  (two) recovers from the states which lanes emitted, ranks them with one ballot per two
//           steps and packs the 16-bit words into an LDS region per batch;
//   words   takes the words from LDS to HBM.
// What a lone wavefront's instructions cost on gfx950, one on every compute unit: 1.9 ns a vector instruction of four bytes or
// of eight, dependent or not, an s_nop 0 and a wait for nothing, 2.65 a select that takes half a register; with the upper half of
// the lanes off every vector instruction 2.65 (not with one lane off, and not where a single compute unit is at work); a
// read of 16 bytes a lane 3.9 in a row and 5.1 behind two vector instructions, a write of as much 11.4.  Hence all lanes on, the LDS
// accesses of four steps in one place, one write for eight steps, and one wait state a step (see pipe_step).  A step
// takes 14.5 ns where the helpers only stand at the barriers (long reciprocals 16.1) and 18.8 with them at work (20.3); four
// wavefronts, with a masked lower half, six wait states and two writes, take 23.2 (24.5).  What the helpers add is LDS traffic: a
// kilobyte takes 5.7 ns to write and 4.4 to read from random places in 16-byte pieces, and the coder waits its turn.  So the
// packer reads no thresholds, entries are looked up in two halves of 8 bytes (1.7 ns each), and writes do not stand in a row.
// They meet at one workgroup barrier per batch of B steps: 32 where two units or one share a compute unit, else 16, whose
// rings and tables take 41 KB of LDS (45 with a table per depth) and not 74 (78, or 86 with whole entries).  256 units of
// 1,048,576 symbols 707 -> 565 us, with a table per depth 815 -> 656; in a loop of nothing else, at a lower clock, 759 -> 617 and
// 775 -> 617, with a frequency above 2048 (long reciprocals) 804 -> 665 and 822 -> 661.
// The coder writes its last eight steps' states of a batch in the batch after (and waits for nothing at a barrier).
// Iteration `it` of the loop: feeder batch it, coder batch it - 2, packer emissions of batch it - 4 and words of batch
// it - 5, each packer every second batch.
constexpr int kEntrySlots = 3;  // feeder writes b + 2, coder reads b and b + 1
constexpr int kStateSlots = 3;  // coder writes b and the end of b - 1, packer reads b - 2 and the first state behind it
constexpr int kListRegions = 2;  // batches whose words are being packed and are leaving
constexpr int kPipeStage = kSuperSyms + 48;  // a round's symbols and the group above them, at any 16-byte misalignment
enum PipeRole { kFeeder0, kFeeder1, kSymbols, kCoder, kPacker0, kPacker1, kWords, kPipeRoles };  // (wavefronts i and i + 4 share a SIMD)
constexpr int kPipeThreads = 64 * kPipeRoles;
// Up to two rounds of 512 units the kernels with one chain per workgroup beat the many-unit kernels.  The encoder's
// LDS lets two units share a compute unit, three with batches of 16 steps, the decoder's two, and the more of them do
// the less each wavefront issues.  Units of 131,072 symbols, 256 / 512 / 768 / 1024 of them, then the many-unit kernel at
// 1028: encode 85 / 119 / 164 / 222 and 394 us, with four tables 89 / 133 / 184 / 251 and 404 us (with four
// wavefronts a unit: 102 / 140 / 189 / 266 and 107 / 150 / 198 / 287), decode 190 / 199 / 390 / 394 and 621 us.
constexpr int64_t kPipeMaxUnits = 1024;
// Beyond, the encoder's further rounds of 768 still win where streams are long, up to seven units for each compute unit: 1028 /
// 1536 / 1792 / 2048 units of 32,768 symbols 75 / 96 / 105 / 126 us and the many-unit kernel 104 / 106 / 106 / 107, of 524,288
// 1031 / 1247 / 1426 / 1768 and 1546 / 1658 / 1660 / 1664; but 16,384 symbols 42 / 55 / 60 / 71 and 54 / 56 / 57 / 57.
// With a table per depth the many-unit kernel holds seven units per compute unit at a time, 1792, so that its second round begins
// where the third of this one does.  1028 / 1536 / 1537 / 1792 / 1793 / 2304 / 2560 units, four tables, 32,768 symbols 92 / 119 / 122 /
// 130 / 139 / 175 / 188 us and 108 / 112 / 112 / 115 / 152 / 170 / 171; 49,152 symbols 125 / 164 / 166 / 174 / 191 / 241 / 262 and 157 /
// 163 / 162 / 164 / 219 / 248 / 249; 131,072 symbols 296 / 375 / 392 / 407 / 454 / 569 / 611 and 403 / 410 / 412 / 415 / 563 / 626 / 626.
__host__ __forceinline__ bool encode_in_pipe(int64_t n_units, int64_t syms_per_stream, bool per_depth) {
  if (n_units <= kPipeMaxUnits) return true;
  if (!per_depth) return syms_per_stream >= 32768 && n_units <= 7 * kComputeUnits;
  return syms_per_stream >= 49152 &&
         (n_units <= 6 * kComputeUnits || (n_units > 7 * kComputeUnits && n_units <= 9 * kComputeUnits));
}
// Few units below these lengths take the kernel with four wavefronts, which begins and ends sooner (rans_encode_short_kernel).
// 1 / 256 / 257 / 512 / 768 / 1024 units, four wavefronts and then seven: 2048 symbols 6.2 / 7.1 / 7.1 / 7.6 / 8.7 / 13.6 us and
// 7.0 / 7.9 / 8.3 / 9.3 / 10.1 / 14.1, 8192 symbols 10.3 / 11.4 / 12.8 / 14.1 / 17.5 / 25.0 and 10.1 / 11.0 / 13.2 / 14.2 / 17.8 /
// 23.8, 10,240 symbols 11.8 / 13.1 / 15.0 / 16.3 / 20.4 / 29.1 and 11.3 / 12.4 / 15.0 / 16.1 / 19.8 / 27.0.  With four tables:
// 8192 symbols 15.4 / 16.2 / 18.0 / 18.9 / 23.3 / 34.5 and 15.5 / 16.3 / 19.6 / 20.6 / 25.1 / 34.1, 12,288 symbols 18.3 / 19.2 /
// 22.2 / 23.3 / 29.3 / 42.7 and 17.8 / 19.0 / 23.4 / 24.5 / 30.0 / 42.0, 20,480 symbols 24.1 / 25.1 / 30.6 / 32.0 / 41.1 / 59.4 and
// 22.1 / 23.4 / 30.4 / 31.8 / 41.0 / 56.5 (entries of 8 bytes, which the feeders unpack, where a compute unit has more than one).
__host__ __forceinline__ bool encode_in_short(int64_t n_units, int64_t syms_per_stream, bool per_depth) {
  return n_units <= kPipeMaxUnits && syms_per_stream < (!per_depth ? 10240 : n_units <= kComputeUnits ? 12288 : 20480);
}
constexpr int64_t kChainMaxUnits = 1024;  // the same bound for the decoder of whole-stream units
// The decoder with one table per depth holds one unit per compute unit (its tables take 128 KB of LDS): two
// rounds of 256 are what it may take before the many-unit decoder is as fast.
constexpr int64_t kDepthsMaxUnits = 512;
// Restart points: so many pieces altogether -- 32 per compute unit, four wavefronts per SIMD of the decoder with two
// units per wavefront (256 streams of 1,048,576 symbols in 8, 16, 32, 64 pieces each: 521, 306, 196, 191 us; as whole
// streams 1.39 ms) -- and none shorter than two of the encoder's rounds (4096 symbols: 8 streams of 65,536 symbols in
// 8, 16, 32 pieces 29, 24, 22 us, where a record's 136 bytes come to 4 % of the words of the shortest).
constexpr int64_t kPiecesWanted = 8192;
constexpr int32_t kPieceMinRounds = 2;
// Up to here a piece gets a workgroup of the decoder with the shortest step, two rounds of two to a compute unit (128
// streams of 262,144 symbols, 8 pieces each: 117 us, the decoder with two units per wavefront 141; 256 streams: 217 and
// 143).
constexpr int64_t kChainMaxPieces = 1024;
// The decoder that reconstructs too takes pieces of several records, so that there is one round of workgroups (two or,
// up to kCompactMaxK candidates, four to a compute unit), whose start is then paid once.
constexpr int64_t kPiecesPerRound = 512, kPiecesPerRoundCompact = 1024;
// From this many streams on (more than two workgroups per compute unit) the decoder that reconstructs takes
// its three-block ring where k <= 4 lets three workgroups share a compute unit.
constexpr int64_t kDenseStreams = 512;
constexpr int kCompactMaxK = 4;  // up to here four workgroups of the decoder with 4-byte entries fit a compute unit
constexpr int kDenseMaxK = 6;  // up to here the kernel's registers (156 at k = 6) leave room for three wavefronts per SIMD

// One step up to the next step's compare.  `y` is the state less the addend of the step before (e.w of this step), which is
// added here, between the compare and the select that reads its mask: one of the two wait states that the hardware asks for
// between these (the caller puts an instruction between two of these pieces for the other).  e.z is the step's threshold,
// less the same addend.  x out: the state in front of the step.  Written out, because the compiler makes a shift and a select
// of the one that takes the state's high half as its operand, and puts a wait state behind each piece of assembly whose result
// the next instruction reads.
template <EncForm FORM>
__device__ __forceinline__ void pipe_step(uint32_t &y, uint32_t &x, uint64_t &emit, const u32x4 e, uint32_t thr_next) {
  register uint64_t mask asm("vcc") = emit;  // (the only place that this form of the select reads its mask from)
  uint32_t xr, t, yn, xo;
#define PLC_PIPE_STEP(QUOTIENT)                                                                                        \
  asm volatile("v_add_u32_e32 %4, %5, %8\n\t"                                                                          \
               "v_cndmask_b32_sdwa %0, %4, %4, vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t" \
               "v_mul_hi_u32 %1, %6, %0\n\t" QUOTIENT                                                                \
               "v_mad_u32_u24 %2, %1, %7, %0\n\t"                                                                    \
               "v_cmp_gt_u32_e32 vcc, %2, %9"                                                                          \
               : "=&v"(xr), "=&v"(t), "=&v"(yn), "+s"(mask), "=&v"(xo)                                                 \
               : "v"(y), "v"(e.x), "v"(e.y), "v"(e.w), "v"(thr_next))
  if constexpr (FORM == kEncPlain) {
    PLC_PIPE_STEP("");
  } else if constexpr (FORM == kEncShort) {
    PLC_PIPE_STEP("v_lshrrev_b32_sdwa %1, %7, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD\n\t");
  } else {
    PLC_PIPE_STEP("v_add_u32 %1, %1, %0\n\t"
                  "v_lshrrev_b32_sdwa %1, %7, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD\n\t");
  }
#undef PLC_PIPE_STEP
  y = yn;
  x = xo;
  emit = mask;
  PLC_PIN();
}

// One batch of the coder.  `e` holds the entries of its first eight steps on entry and those of the next
// batch's first eight (at `next0` and behind `next`) on return, `emit` the mask of the first step's compare and of the next batch's.  A
// lane's states before steps 4 q .. 4 q + 3 leave as one 16-byte vector for xb[q], in the four steps
// after them: `before` holds the last four on return and `held`, where they belong, those of the batch before on
// entry.  The LDS accesses of four steps stand in one place: each turn from vector instructions to them costs.
template <EncForm FORM, int B>
__device__ __forceinline__ void pipe_batch(uint32_t &y, uint64_t &emit, u32x4 (&e)[4][4], u32x4 &before,
                                           u32x4 *&held, const u32x4 *eb, const u32x4 *next0, const u32x4 *next,
                                           u32x4 *xb) {
  constexpr int kQuads = B / 4;
  // A wait for nothing (every counter at its most): the cheapest instruction to stand between two steps, which has to be
  // there (see pipe_step).  The steps do not rest on it alone: between two pieces of assembly with nothing in between, the second of
  // which reads what the first wrote, the compiler puts an s_nop -- as it does behind this wait where that is assembly too.
  constexpr int kNoWait = 0xcf7f;
#pragma unroll
  for (int q = 0; q < kQuads; ++q) {
    u32x4 (&cur)[4] = e[q % 4];
    u32x4 (&ask)[4] = e[(q + 2) % 4];
    const u32x4 *src = (q + 2 < kQuads ? eb + 4 * (q + 2) * kLanes : next + 4 * (q + 2 - kQuads) * kLanes) - kLanes;
    uint32_t x[4];
    pipe_step<FORM>(y, x[0], emit, cur[0], cur[1].z);
    if (q % 2 == 0) *held = before;
    PLC_PIN();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      ask[j] = q + 2 == kQuads && j == 0 ? *next0 : src[j * kLanes];
      PLC_PIN();
    }
    pipe_step<FORM>(y, x[1], emit, cur[1], cur[2].z);
    __builtin_amdgcn_s_waitcnt(kNoWait);
    PLC_PIN();
    pipe_step<FORM>(y, x[2], emit, cur[2], cur[3].z);
    __builtin_amdgcn_s_waitcnt(0xc47f);  // lgkmcnt(4): the next step needs the next quad's entry; the quad behind it may be on its way
    PLC_PIN();
    pipe_step<FORM>(y, x[3], emit, cur[3], e[(q + 1) % 4][0].z);
    __builtin_amdgcn_s_waitcnt(kNoWait);
    PLC_PIN();
    if (q % 2 == 0) {
      before.x = x[0];
      before.y = x[2];
    } else {
      before.z = x[0];
      before.w = x[2];
      held = xb + (q / 2) * 64;
    }
  }
}

// ADAPT: one table per bit depth (the *_bucketed call).  Its entries take 8 bytes where units are to share a compute
// unit, and the feeder unpacks them; WIDE: whole entries, one unit to a compute unit with batches of 32 steps (256 units of
// 1,048,576 symbols 683 -> 662 us).
template <bool ADAPT, int B, bool WIDE = !ADAPT>
__global__ __launch_bounds__(kPipeThreads, B == 16 ? 6 : ADAPT && WIDE ? 2 : 4) void rans_encode_pipe_kernel(const RansArgs a) {
  constexpr int kIdentity = (ADAPT ? PLC_MAX_BITS : 1) * 256;  // index of the entry that leaves a state unchanged
  constexpr bool kPacked = ADAPT && !WIDE;
  constexpr int kRoundBatches = kSuperGroups / B;  // batches per staging round
  constexpr int kListRegion = B * kLanes + 8;      // a batch's words behind up to seven carried ones
  // Entries of 8 bytes, or their two halves apart (.x and .z of make_enc_entry, and .y and .w): 8 bytes at random places
  // take LDS 1.7 ns a wavefront, 16 take 4.4.
  __shared__ uint2 table[(kPacked ? 1 : 2) * (kIdentity + 1)];
  constexpr int kOther = kPacked ? 0 : kIdentity + 1;
  // ADAPT: table of each group of a staging round, from its lowest, and of the group above
  __shared__ __attribute__((aligned(8))) uint8_t table_of_group[2][kSuperGroups + 8];
  __shared__ uint4 entry_ring[kEntrySlots * B][kLanes];  // by step
  __shared__ uint4 state_ring[kStateSlots][B / 8][64];
  __shared__ __attribute__((aligned(16))) uint8_t sym_stage[2][kPipeStage];
  __shared__ __attribute__((aligned(16))) uint16_t word_list[kListRegions][kListRegion];
  __shared__ uint16_t spare_word;
  __shared__ uint32_t list_fill[kListRegions];  // positions in use of each region of the list
  __shared__ uint32_t batch_words[2];           // words of the packers' last batches
  static_assert(workgroups_per_cu(sizeof(table) + sizeof(table_of_group) + sizeof(entry_ring) + sizeof(state_ring) +
                                  sizeof(sym_stage) + sizeof(word_list) + sizeof(spare_word) + sizeof(list_fill) +
                                  sizeof(batch_words)) >= (B == 16 ? 3 : ADAPT && WIDE ? 1 : 2),
                "so many units to a compute unit");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t unit = blockIdx.x;  // one unit per stream, one workgroup per unit

  EncForm form = kEncPlain;  // uniform
  {  // every wavefront scans the frequencies, and four of them build one of a lane's four entries each
    const int n_tables = ADAPT ? a.n_tables : 1;
    uint32_t f[ADAPT ? PLC_MAX_BITS : 1][4], cum[ADAPT ? PLC_MAX_BITS : 1];
    for (int t = 0; t < n_tables; ++t) {
      const uint32_t total = load_freq4(a.freq + (unit * n_tables + t) * 256, lane, f[t], &cum[t]);
      if (total != kScale && !(ADAPT && total == 0) && threadIdx.x == 0) raise(a.status, PLC_ERR_INVALID);
      form = enc_form_for(form, enc_form_of(f[t]));
    }
    for (int t = 0; t < n_tables; ++t) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (r == wave) {
          const uint4 e = make_enc_entry(form, f[t][r], cum[t]);
          const int i = t * 256 + lane * 4 + r;
          if constexpr (kPacked) {
            table[i] = pack_enc_entry(e);
          } else {
            table[i] = make_uint2(e.x, e.z);
            table[kOther + i] = make_uint2(e.y, e.w);
          }
        }
        cum[t] += f[t][r];
      }
    }
    if (threadIdx.x < 2) batch_words[threadIdx.x] = 0;
    if (threadIdx.x < kLanes)  // the step in front of the first
      entry_ring[kEntrySlots * B - 1][threadIdx.x] = make_uint4(0u, 0u, 0xffffffffu, 0u);
    if (threadIdx.x == 0) {  // never emits, x' = x
      if constexpr (kPacked) {
        table[kIdentity] = pack_enc_entry(make_uint4(0u, 0xffffffffu, 0u, 0u));
      } else {
        table[kIdentity] = make_uint2(0u, 0u);
        table[kOther + kIdentity] = make_uint2(0xffffffffu, 0u);
      }
    }
  }

  const uint32_t len = (uint32_t)a.syms_per_stream;
  const uint8_t *ubase = a.sym_in + unit * a.syms_per_stream;
  const uint32_t mis = (uint32_t)(reinterpret_cast<uintptr_t>(ubase) & 15u);
  const int32_t G = (int32_t)((len + kLanes - 1) / kLanes);
  // Batch 0 holds the top `head` groups followed by identity steps, and every later batch is B full groups, the last
  // one possibly half of them and identity steps: pieces end 16 n groups below the top (piece_top), and here a batch
  // begins there.  Batch b codes groups top(b)-1 down to top(b)-B.
  const int32_t head16 = G % 16 ? G % 16 : 16, head = B == 16 || G == head16 ? head16 : head16 + 16;
  const int32_t n_batches = (G - head + B - 1) / B + 1;
  auto batch_top = [&](int32_t b) { return b == 0 ? G : G - head - (b - 1) * B; };
  // Symbol staging rounds of 64 groups; a round's buffer starts at the 16-byte-aligned address at or
  // below its lowest symbol, so the symbol at unit offset t sits at  t - 32 * bottom + mis.
  auto round_bottom = [&](int32_t r) {
    const int32_t g = batch_top(kRoundBatches * (r + 1) - 1) - B;
    return g > 0 ? g : 0;
  };
  const int32_t n_rounds = (n_batches + kRoundBatches - 1) / kRoundBatches;
  const int32_t n_coded = n_batches + 1;  // as the coder goes: a batch of identity steps behind the last
  const int32_t n_iters = n_coded + 5;
  const int32_t piece_batches = a.piece_batches * kBatch / B;
  uint16_t *wp = a.words_out + a.word_off[unit];
  const uint32_t pad = __builtin_amdgcn_readfirstlane((uint32_t)((reinterpret_cast<uintptr_t>(wp) >> 1) & 7u));
  // Restart points: the packers have a record's states and words at hand, the symbols' wavefront its escapes.
  uint32_t *const points = a.points_out ? a.points_out + unit * a.point_stride * PLC_RESTART_WORDS : nullptr;

  if (wave == kCoder) {
    // ---- batch it - 2
    __syncthreads();  // tables
    __syncthreads();  // first symbols
    uint32_t y = kLow;
    u32x4 e[4][4], before = {0u, 0u, 0u, 0u};
    constexpr int kEntryStep = B * kLanes, kStateStep = (B / 8) * 64;
    // the lower half is a step behind the upper: row r - 1 where the other reads row r, the last one for row 0
    const u32x4 *const entries = reinterpret_cast<const u32x4 *>(&entry_ring[0][0]) + lane;
    const u32x4 *const wrapped = reinterpret_cast<const u32x4 *>(&entry_ring[lane < kLanes ? kEntrySlots * B - 1 : 0][lane & 31]);
    u32x4 *const states = reinterpret_cast<u32x4 *>(&state_ring[0][0][lane]);
    u32x4 *held = states + kStateSlots * kStateStep - 64;  // (read by nobody yet)
    lds_barrier();  // iteration 0
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j / 4][j % 4] = j == 0 ? *wrapped : entries[(j - 1) * kLanes];
    lds_barrier();  // iteration 1
    static_assert(kEntrySlots == 3 && kStateSlots == 3, "three batches a turn");
    auto code = [&](auto form_c) {  // a loop per form, and nothing in it besides the steps
      constexpr EncForm kForm = decltype(form_c)::value;
      uint64_t emit = __builtin_amdgcn_uicmp(y, e[0][0].z, 34 /* unsigned > */);
      auto batch = [&](auto slot) {
        constexpr int kAt = decltype(slot)::value, kNext = (kAt + 1) % 3;
        pipe_batch<kForm, B>(y, emit, e, before, held, entries + kAt * kEntryStep,
                          kNext == 0 ? wrapped : entries + kNext * kEntryStep - kLanes, entries + kNext * kEntryStep,
                          states + kAt * kStateStep);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();  // iteration b + 2
        asm volatile("" ::: "memory");
      };
      __builtin_amdgcn_s_waitcnt(0xc07f);  // (lgkmcnt(0): nothing for the loop to wait for in every turn)
      PLC_PIN();
      for (int32_t turns = n_coded / 3; turns > 0; --turns) {
        batch(std::integral_constant<int, 0>{});
        batch(std::integral_constant<int, 1>{});
        batch(std::integral_constant<int, 2>{});
      }
      const int32_t more = n_coded % 3;
      if (more > 0) batch(std::integral_constant<int, 0>{});
      if (more > 1) batch(std::integral_constant<int, 1>{});
    };
    if (form == kEncLong) {
      code(std::integral_constant<EncForm, kEncLong>{});
    } else if (form == kEncPlain) {
      code(std::integral_constant<EncForm, kEncPlain>{});
    } else {
      code(std::integral_constant<EncForm, kEncShort>{});
    }
    *held = before;  // the last states, in place before the barrier behind them, and the one behind them
    states[(n_coded % kStateSlots) * kStateStep] = u32x4{y, y, y, y};
    for (int32_t it = n_coded + 2; it < n_iters; ++it) lds_barrier();
    if (lane < kLanes) {  // (the steps behind the last have added its addend and then nothing)
      a.states_out[unit * kLanes + lane] = y;
      if (points) points[lane] = y;
    }
  } else if (wave == kFeeder0 || wave == kFeeder1) {
    // ---- entries of batch it, half of them each: written in the batch's own iteration, looked up in the one before, and
    // the symbols read two before, so that nothing is waited for.  Lane (half, l) serves kMine steps of rANS lane l from
    // first on; a step's entry goes with the addend of the step in front of it, whose symbol the lane looks up too.
    __syncthreads();  // tables
    __syncthreads();  // first symbols
    constexpr int kMine = B / 4;
    const int l = lane & 31, first = ((wave == kFeeder1 ? 2 : 0) + (lane >> 5)) * kMine;
    uint32_t sy[kMine + 1];     // the step in front, then the lane's own
    uint32_t own[kMine / 4], above = 0;  // ADAPT: tables of the lane's groups, from the lowest, and of the one in front
    u32x2 head_of[kMine], tail_of[kMine + 1];  // the entries' halves; the step in front has the first tail
    uint32_t any = 0;
    auto ask = [&](int32_t b) __attribute__((always_inline)) {  // symbols of a batch of B full groups
      const int32_t r = b / kRoundBatches, at = batch_top(b) - round_bottom(r) - first - kMine;  // the lane's lowest group
      const uint8_t *s0 = sym_stage[r & 1] + (at * kLanes + l + (int32_t)mis);
#pragma unroll
      for (int p = 0; p <= kMine; ++p) sy[p] = s0[kLanes * (kMine - p)];
      if constexpr (ADAPT) {
        const uint8_t *tg = &table_of_group[r & 1][at];
#pragma unroll
        for (int i = 0; i < kMine / 4; ++i) own[i] = reinterpret_cast<const uint32_t *>(tg)[i];
        above = tg[kMine];
      }
    };
    auto look_up_step = [&](int p, uint32_t i) __attribute__((always_inline)) {
      if (p) head_of[p - 1] = *reinterpret_cast<const u32x2 *>(&table[i]);
      if (!kPacked) tail_of[p] = *reinterpret_cast<const u32x2 *>(&table[kOther + i]);
      if (kPacked && p == 0) tail_of[0].y = table[i].y;
    };
    auto look_up = [&](const uint32_t (&i)[kMine + 1]) __attribute__((always_inline)) {
#pragma unroll
      for (int p = 0; p <= kMine; ++p) look_up_step(p, i[p]);
    };
    auto asked = [&](int32_t b, uint32_t (&i)[kMine + 1]) __attribute__((always_inline)) {
      i[0] = ADAPT ? sy[0] | above << 8 : sy[0];
#pragma unroll
      for (int p = 1; p <= kMine; ++p)  // symbol | table << 8
        i[p] = ADAPT ? __builtin_amdgcn_perm(own[(kMine - p) / 4], sy[p], 0x0c0c0400u + ((uint32_t)((kMine - p) & 3) << 8)) : sy[p];
      if (b == 1 && head < B && first == 0) i[0] = kIdentity;  // batch 0 ends in identity steps
    };
    auto look_up_ends = [&](int32_t b) {  // the first batch, whose top group may be ragged, and the last
      uint32_t i[kMine + 1];
      const int32_t r = b / kRoundBatches, bottom = round_bottom(r), top = batch_top(b);
#pragma unroll
      for (int p = 0; p <= kMine; ++p) {
        const int j = first - 1 + p;  // -1: the batch before's last step
        const int32_t g = top - 1 - j;
        const bool step = j < 0 ? b > 1 || (b == 1 && head == B) : b > 0 || j < head;
        const bool has = step && g >= 0 && (int64_t)g * kLanes + l < (int64_t)len;
        i[p] = sym_stage[r & 1][has ? (g - bottom) * kLanes + l + (int32_t)mis : 0];
        if (ADAPT && has) i[p] += (uint32_t)table_of_group[r & 1][g - bottom] << 8;
        i[p] = has ? i[p] : (uint32_t)kIdentity;
      }
      look_up(i);
    };
    auto unpack = [&]() __attribute__((always_inline)) {
      if (kPacked) {
        tail_of[0].y = (uint32_t)((int32_t)tail_of[0].y >> 18);
#pragma unroll
        for (int p = 0; p < kMine; ++p) {
          const uint4 v = unpack_enc_entry(make_uint2(head_of[p].x, head_of[p].y));
          head_of[p].y = v.z;
          tail_of[p + 1] = u32x2{v.y, v.w};
        }
      }
    };
    auto put_step = [&](int p, uint4 *eo) __attribute__((always_inline)) {
      any |= tail_of[p + 1].y;
      tail_of[p].x = tail_of[p + 1].x - tail_of[p].y;  // beside the addend in front already
      u32x2 *to = reinterpret_cast<u32x2 *>(eo + p * kLanes);
      to[0] = head_of[p];
      to[1] = tail_of[p];
    };
    look_up_ends(0);
    if (n_batches > 2) ask(1);
    int slot = 0;
    int32_t b = 0;
    for (; b + 3 < n_batches; ++b) {
      uint4 *eo = &entry_ring[slot * B + first][l];
      slot = slot == kEntrySlots - 1 ? 0 : slot + 1;
      uint32_t i[kMine + 1];
      asked(b + 1, i);
      unpack();
      PLC_PIN();
      // Writes and look-ups by turns: writes in a row hold the coder's accesses up (256 units of 1,048,576 symbols 620 ->
      // 586 us).
#pragma unroll
      for (int p = 0; p <= kMine; ++p) {
        if (p < kMine) put_step(p, eo);
        PLC_PIN();
        look_up_step(p, i[p]);
        PLC_PIN();
      }
      ask(b + 2);
      PLC_PIN();
      asm volatile("" ::: "memory");
      // the entries are in the ring; what was asked for behind them may be on its way (tables do not change, and
      // symbols only rounds later)
      __builtin_amdgcn_s_waitcnt(kPacked ? 0xc57f : 0xc87f);  // lgkmcnt(5) or (8): of so many reads behind the last write at the least
      __builtin_amdgcn_s_barrier();  // iteration b
      asm volatile("" ::: "memory");
    }
    for (; b < n_batches; ++b) {  // the last three
      uint4 *eo = &entry_ring[slot * B + first][l];
      slot = slot == kEntrySlots - 1 ? 0 : slot + 1;
      unpack();
#pragma unroll
      for (int p = 0; p < kMine; ++p) put_step(p, eo);
      if (b + 2 < n_batches) {
        uint32_t i[kMine + 1];
        asked(b + 1, i);
        look_up(i);
      } else if (b + 1 < n_batches) {
        look_up_ends(b + 1);
      }
      lds_barrier();  // iteration b
    }
    {  // the steps behind the last: the first adds what that leaves to add
      const int32_t r = n_rounds - 1;
      uint32_t i = sym_stage[r & 1][l + mis];  // group 0, the lowest of the last round
      if (ADAPT) i += (uint32_t)table_of_group[r & 1][0] << 8;
      if (n_batches == 1 ? head < B : (G - head) % B != 0) i = kIdentity;
      uint32_t last = kPacked ? (uint32_t)((int32_t)table[i].y >> 18) : table[kOther + i].y;
      if (first > 0) last = 0u;
      uint4 *eo = &entry_ring[slot * B + first][l];
      eo[0] = make_uint4(0u, 0u, 0xffffffffu - last, last);
#pragma unroll
      for (int p = 1; p < kMine; ++p) eo[p * kLanes] = make_uint4(0u, 0u, 0xffffffffu, 0u);
    }
    for (int32_t it = n_batches; it < n_iters; ++it) lds_barrier();
    if (any & 0x80000000u) raise(a.status, PLC_ERR_INVALID);  // a symbol with f = 0
  } else if (wave == kPacker0 || wave == kPacker1) {
    // ---- every second batch each: which lanes emit, and how many, in iteration b + 4, their ranks and words in the one
    // behind it.
    // A lane emits in a step iff the state behind the step is below the one in front of it: without a word
    // x' - x = q * (4096 - f) + cum >= 0, with one x' <= x / (16 f) + 4095 and x >= f * 2^20.
    __syncthreads();  // tables
    __syncthreads();  // first symbols
    const int odd = wave == kPacker1 ? 1 : 0;
    uint32_t total = pad;  // uniform: words in front of the batch, the padding in front of the first among them
    uint32_t mine = 0;     // and of this packer's last batch
    int32_t point_at = points ? piece_batches : INT32_MAX;  // the batch that the next record stands in front of
    uint32_t *record = points;
    // Hardware lane h of a half carries rANS lane 31 - h, which the encoder visits first.  A batch here begins with the last
    // step of the one before: the coder's lower half is a step behind, so that lower lanes have the states in front of
    // steps -1, 1, .. B - 3 and upper ones those in front of steps 0, 2, .. B - 2, and the states behind are the other
    // half's.
    const bool upper = lane >= kLanes;
    const int at_ring = (lane & 32) + 31 - (lane & 31);
    constexpr int kPairs = B / 2;  // pairs of steps
    uint16_t *const spare = &spare_word;
    int slot = odd;
    int32_t it = 0;
    for (; it < 4 + odd; ++it) lds_barrier();
    for (int32_t b = odd; b < n_coded; b += 2) {
      const u32x4 *src = reinterpret_cast<const u32x4 *>(&state_ring[slot][0][0]);
      const uint32_t *behind = &state_ring[slot == kStateSlots - 1 ? 0 : slot + 1][0][at_ring & 31].x;
      slot = slot == 0 ? 2 : slot - 1;  // two on
      uint32_t word[kPairs], next[kPairs + 1], at[kPairs];
#pragma unroll
      for (int q = 0; q < B / 8; ++q) {
        *reinterpret_cast<u32x4 *>(&word[4 * q]) = src[q * 64 + at_ring];
        *reinterpret_cast<u32x4 *>(&next[4 * q]) = src[q * 64 + (at_ring ^ 32)];
      }
      next[kPairs] = *behind;
      uint32_t n1 = batch_words[odd ^ 1];  // of the batch before
      PLC_PIN();
      // (every compare before the first count: a scalar instruction waits for a mask that was only just written)
      uint64_t emits[kPairs];
#pragma unroll
      for (int p = 0; p < kPairs; ++p) emits[p] = __ballot((upper ? next[p + 1] : next[p]) < word[p]);
      PLC_PIN();
      uint32_t n = 0;
      asm volatile("" : "+v"(n));  // (a vector register: the masks are scalars, and an instruction takes one)
#pragma unroll
      for (int p = 0; p < kPairs; ++p) {
        at[p] = n;
        n += (uint32_t)__builtin_popcountll(emits[p]);
      }
      if (lane == 0) batch_words[odd] = n;
      n1 = __builtin_amdgcn_readfirstlane(n1);
      total += mine + n1;
      mine = __builtin_amdgcn_readfirstlane(n);
      // a batch has a region, in which its first words stand behind up to seven of the batch before
      const uint32_t fill = total & 7u;
      uint16_t *const list = word_list[odd] + fill;
      PLC_PIN();
      lds_barrier();  // iteration b + 4
      // (a lane without a word stores into a slot of its own instead of sitting out the store)
#pragma unroll
      for (int p = 0; p < kPairs; ++p) {
        const uint32_t i = __builtin_amdgcn_mbcnt_hi((uint32_t)(emits[p] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)emits[p], at[p]));
        *(__builtin_amdgcn_inverse_ballot_w64(emits[p]) ? list + i : spare) = (uint16_t)word[p];
      }
      if (lane == 0) list_fill[odd] = fill + mine;
      if (b >= point_at) {  // uniform; two batches on there is at most one record to be passed
        record += PLC_RESTART_WORDS;
        if (b == point_at && b < n_batches) {  // the states in front of the batch's first step
          if (upper) record[at_ring & 31] = word[0];
          if (lane == 0) record[kLanes] = total - pad + (uint32_t)__builtin_popcount((uint32_t)emits[0]);
        }
        point_at += piece_batches;
      }
      lds_barrier();  // iteration b + 5
      it += 2;
    }
    for (; it < n_iters; ++it) lds_barrier();
  } else if (wave == kSymbols) {
    // ---- symbols of the coming round
    bool bad_depth = false;
    uint4 nv[kStagePieces];         // next round's symbols in flight
    bool ntake[kStagePieces];
    // ADAPT: depth of group bottom + lane of the next round.  It is looked at when the round's symbols land: where it
    // is asked for, its range check would have the wavefront, and at the barrier the others, wait for the answer in
    // every round (964 -> 829 us for 256 units of 1,048,576 symbols).
    uint32_t next_depth = 1, table_above = 0;
    const uint32_t spp = ADAPT ? (uint32_t)a.syms_per_pos : 1u;
    const uint8_t *const depth_row =
        ADAPT ? a.bits + (int64_t)((uint32_t)unit / (uint32_t)a.streams_per_session) * (len / spp) : nullptr;
    auto round_load = [&](int32_t r) __attribute__((always_inline)) {  // the round's groups and the one above, whose addends the feeder needs
      const int64_t lo = (int64_t)round_bottom(r) * kLanes;
      int64_t hi = (int64_t)(batch_top(kRoundBatches * r) + 1) * kLanes;
      hi = hi < (int64_t)len ? hi : (int64_t)len;
#pragma unroll
      for (int i = 0; i < kStagePieces; ++i) {
        const int64_t off = lo - (int64_t)mis + (int64_t)(lane + 64 * i) * 16;  // 16-byte aligned in absolute address
        ntake[i] = r < n_rounds && off < hi;
        if (ntake[i]) nv[i] = load16_stream(ubase + off);
      }
      if (ADAPT) {
        const int32_t g = round_bottom(r) + lane;
        next_depth = (r < n_rounds && g < batch_top(kRoundBatches * r)) ? depth_row[(uint32_t)g * kLanes / spp] : 1u;
      }
    };
    auto round_store = [&](int32_t r) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < kStagePieces; ++i)
        if (ntake[i]) *reinterpret_cast<uint4 *>(&sym_stage[r & 1][(lane + 64 * i) * 16]) = nv[i];
      if (ADAPT && r < n_rounds) {
        const bool known = next_depth >= 1u && next_depth <= (uint32_t)a.n_tables;
        bad_depth = bad_depth || !known;
        const uint32_t t = known ? next_depth - 1u : 0u;
        table_of_group[r & 1][lane] = (uint8_t)t;
        if (lane == 0 && r > 0)  // the group above is the lowest of the round before
          table_of_group[r & 1][batch_top(kRoundBatches * r) - round_bottom(r)] = (uint8_t)table_above;
        table_above = t;
      }
    };
    round_load(0);
    __syncthreads();  // tables
    round_store(0);
    round_load(1);
    round_store(1);
    round_load(2);
    __syncthreads();  // first symbols
    // Escapes, for the restart points: a round's symbols are counted in the stage in the last iteration before others
    // take their place, in which this wavefront has nothing else to do.
    uint32_t esc_mine = 0;  // this lane's, of the rounds so far
    const int32_t piece_rounds = piece_batches / kRoundBatches;
    int32_t point_at = points ? piece_rounds : INT32_MAX;  // the round that the next record stands in front of
    uint32_t *record = points;
    auto count_round = [&](int32_t r) __attribute__((always_inline)) {
      if (r == point_at) {
        point_at += piece_rounds;
        record += PLC_RESTART_WORDS;
        const uint32_t total = wave_sum(esc_mine);
        if (lane == 0) record[kLanes + 1] = total;
      }
      const uint8_t *sb = sym_stage[r & 1];
      const uint32_t lo = (uint32_t)round_bottom(r) * kLanes, top = (uint32_t)batch_top(kRoundBatches * r) * kLanes;
      const uint32_t n = (top < len ? top : len) - lo;
      if (mis == 0 && n == (uint32_t)kSuperSyms) {  // uniform
#pragma unroll
        for (int h = 0; h < kSuperSyms / 1024; ++h) {
          const uint4 v = *reinterpret_cast<const uint4 *>(&sb[(lane + 64 * h) * 16]);
          const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int i = 0; i < 4; ++i)  // a byte is 0xff iff its low seven bits carry into bit 7 and bit 7 is set
            esc_mine += (uint32_t)__builtin_popcount(((w[i] & 0x7f7f7f7fu) + 0x01010101u) & w[i] & 0x80808080u);
        }
      } else {
        for (uint32_t t = lane; t < n; t += 64) esc_mine += sb[t + mis] == PLC_ESCAPE;
      }
    };
    // The feeders read a round's symbols up to two iterations ahead, the last batch's one ahead.
    for (int32_t it = 0; it < n_iters; ++it) {
      const int32_t r = it / kRoundBatches, phase = it % kRoundBatches;
      if (phase == kRoundBatches - 2 && points && r < n_rounds) count_round(r);
      if (phase == kRoundBatches - 1 && r + 2 < n_rounds) {
        round_store(r + 2);
        round_load(r + 3);
      }
      lds_barrier();
    }
    if (points) {
      const uint32_t esc_total = wave_sum(esc_mine);
      if (lane == 0) points[kLanes + 1] = esc_total;
    }
    if (bad_depth) raise(a.status, PLC_ERR_INVALID);
  } else {
    // ---- words.  Position p of a region stands for the word at 16-byte-aligned address (wp - pad) + vbase + p; the
    // first `pad` positions of the first are padding in front of the unit's first word.  The complete 16-byte
    // pieces leave, a batch's in one iteration; the incomplete tail (< 8 words) moves to the front of the next region, in
    // front of the words that the packer has written or is writing there.
    __syncthreads();  // tables
    __syncthreads();  // first symbols
    const uint32_t cap = a.word_cap < 0x7fffffffull ? (uint32_t)a.word_cap : 0x7fffffffu;  // a unit has < 2^31 symbols
    uint32_t vbase = 0, rest = pad;
    auto words_out = [&](int32_t b) __attribute__((always_inline)) {
      const uint16_t *list = word_list[b & 1];
      uint32_t fill = list_fill[b & 1];
      u32x4 v[B / 16];
#pragma unroll
      for (int h = 0; h < B / 16; ++h)  // (a lane past the last piece reads inside the region)
        v[h] = *reinterpret_cast<const u32x4 *>(list + 8 * (lane + 64 * h));
      fill = __builtin_amdgcn_readfirstlane(fill);
      const uint32_t full = fill / 8;  // at most 64 to a batch's 512 symbols
      rest = fill - 8 * full;
      const uint16_t tail = list[8 * full + (lane & 7)];  // (lanes past the tail read inside the region)
      if (vbase >= pad && vbase + 8 * full - pad <= cap) {
        uint16_t *dst = wp + (vbase - pad);  // 16-byte aligned
#pragma unroll
        for (int h = 0; h < B / 16; ++h)
          if ((uint32_t)(lane + 64 * h) < full) *reinterpret_cast<u32x4 *>(dst + 8 * (lane + 64 * h)) = v[h];
      } else {
        for (uint32_t q = lane; q < 8 * full; q += 64) {
          const uint32_t i = vbase + q;
          if (i >= pad && i - pad < cap) wp[i - pad] = list[q];
        }
      }
      vbase += 8 * full;
      if ((uint32_t)lane < rest) {
        if (b + 1 < n_coded) {
          word_list[(b + 1) & 1][lane] = tail;
        } else {  // the incomplete last piece
          const uint32_t i = vbase + (uint32_t)lane;
          if (i >= pad && i - pad < cap) wp[i - pad] = tail;
        }
      }
    };
    // The words of batch b are in their region when iteration b + 6 begins; it is written again in iteration b + 7.
    for (int it = 0; it < 6; ++it) lds_barrier();
    int32_t b = 0;
    for (; b + 6 < n_iters; ++b) {
      words_out(b);
      lds_barrier();  // iteration b + 6
    }
    for (; b < n_coded; ++b) {
      words_out(b);
      wave_sync();  // the next batch's reads come behind the tail's way to its front, from other lanes
    }
    const uint32_t n_words = vbase + rest - pad;
    if (lane == 0) {
      a.n_words_out[unit] = n_words;
      if ((uint64_t)n_words > a.word_cap) raise(a.status, PLC_ERR_CAPACITY);
      if (points) points[kLanes] = n_words;
    }
  }
}

// ---------------------------------------------------------------------------
// Encoder for few, short units: four wavefronts per unit
// ---------------------------------------------------------------------------
// Units so short that what comes before the chain of steps and behind it counts as much as the chain: a coder, a feeder, a
// packer and a mover of symbols and words, one per SIMD of the compute unit.  Against the kernel with seven wavefronts a
// batch is 16 steps always, no batch of identity steps stands behind the last, the words leave an iteration sooner, and there
// is less code for the instruction cache to fetch, which every launch begins without.  Its step takes 23 ns where
// that kernel's takes 19; encode_in_short has the lengths at which one overtakes the other.  (Figures of longer
// units below are from when this kernel took those too.)
//   mover   brings the symbols from HBM to LDS (64 groups ahead) and the words from LDS to HBM;
//   feeder  turns every (group, lane) of a batch into its 16-byte table entry at a fixed place of an LDS
//           ring; a lane without a symbol (ragged top group, or a step past the unit's first group) gets an
//           identity entry.  It runs two batches ahead of the coder, so that the coder can ask for the next
//           batch's first entries before the barrier;
//   coder   the recurrence alone, in the lower half of the lanes, the entries' reads in the wait states behind the compare,
//           and one LDS write of the four states of four steps;
//   packer  recovers from the stored states which lanes emitted (x > thr), ranks them with one ballot per two
//           steps and packs the 16-bit words into an LDS region per batch.
// They meet at one workgroup barrier per batch of 16 steps.  The coder writes its last four states of a batch in
// the batch after (and waits for nothing at a barrier), so the packer works two batches behind it.
// Iteration `it` of the loop: feeder batch it, coder batch it - 2, packer batch it - 4, whose thresholds it has read
// two iterations earlier: the ring then needs three slots and three units share a compute unit's LDS.  The mover takes in a round
// of symbols every fourth iteration and sends the words of two batches out in each of the two after it: waiting
// for symbols is waiting for every store before them as well (one counter), and these are then two iterations
// old (stores in every iteration held the barrier up every round).
namespace short_units {
constexpr int kEntrySlots = 3;  // feeder writes b + 2, coder reads b and b + 1, packer the thresholds of b
constexpr int kStateSlots = 3;  // coder writes b and the end of b - 1, packer reads b - 2
constexpr int kListRegion = 2 * kBatchSyms + 8;  // the words of a pair of batches behind up to seven carried ones
constexpr int kListRegions = 3;  // the packer's, and the up to two in front of it that have not left
constexpr int kThreads = 256;

// One step from its select on, and the next step's compare: x and the next threshold in, the next x and the mask of its
// compare out.  Between two of these stand the caller's LDS accesses, two instructions at the least: the wait states that
// the hardware asks for between a compare and the select that reads its mask.  Written out, because the compiler makes
// a shift and a select of the one that takes the state's high half as its operand, and puts a wait state behind each
// piece of assembly whose result the next instruction reads.
template <EncForm FORM>
__device__ __forceinline__ void pipe_step(uint32_t &x, uint64_t &emit, const u32x4 e, uint32_t thr_next) {
  register uint64_t mask asm("vcc") = emit;  // (the only place that this form of the select reads its mask from)
  uint32_t xr, t, xn;
#define PLC_PIPE_STEP(QUOTIENT)                                                                                        \
  asm volatile("v_cndmask_b32_sdwa %0, %4, %4, vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t" \
               "v_mul_hi_u32 %1, %5, %0\n\t" QUOTIENT                                                                \
               "v_mul_u32_u24 %1, %1, %6\n\t"                                                                        \
               "v_add3_u32 %2, %0, %7, %1\n\t"                                                                       \
               "v_cmp_gt_u32_e32 vcc, %2, %8"                                                                          \
               : "=&v"(xr), "=&v"(t), "=&v"(xn), "+s"(mask)                                                            \
               : "v"(x), "v"(e.x), "v"(e.z), "v"(e.w), "v"(thr_next))
  if constexpr (FORM == kEncPlain) {
    PLC_PIPE_STEP("");
  } else if constexpr (FORM == kEncShort) {
    PLC_PIPE_STEP("v_lshrrev_b32_sdwa %1, %6, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD\n\t");
  } else {
    PLC_PIPE_STEP("v_add_u32 %1, %1, %0\n\t"
                  "v_lshrrev_b32_sdwa %1, %6, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:DWORD\n\t");
  }
#undef PLC_PIPE_STEP
  x = xn;
  emit = mask;
  PLC_PIN();
}

// One batch of the coder.  `e` holds the entries of its first eight steps on entry and those of the next
// batch's first eight (at `next`) on return, `emit` the mask of the first step's compare and of the next batch's.  A
// lane's states before steps 4 q .. 4 q + 3 leave as one 16-byte vector for xb[q], in the first of the four steps
// after them: `before` holds the last four on return and `held`, where they belong, those of the batch before on
// entry.  A step asks for entries eight steps ahead (with four the LDS answered late when the helpers were at it: 1.19
// against 1.11 ms for an encode given the tokens), and one wait a quad leaves those of the quad on their way.
template <EncForm FORM>
__device__ __forceinline__ void pipe_batch(uint32_t &x, uint64_t &emit, u32x4 (&e)[kBatch / 4][4], u32x4 &before,
                                           u32x4 *&held, const u32x4 *eb, const u32x4 *next, u32x4 *xb) {
  constexpr int kQuads = kBatch / 4;
#pragma unroll
  for (int q = 0; q < kQuads; ++q) {
    u32x4 (&cur)[4] = e[q];
    u32x4 (&ask)[4] = e[(q + 2) % kQuads];
    const u32x4 *src = q + 2 < kQuads ? eb + 4 * (q + 2) * kLanes : next + 4 * (q + 2 - kQuads) * kLanes;
    *held = before;
    PLC_PIN();
    ask[0] = src[0];
    PLC_PIN();
    before.x = x;
    pipe_step<FORM>(x, emit, cur[0], cur[1].y);
    ask[1] = src[kLanes];
    PLC_PIN();
    ask[2] = src[2 * kLanes];
    PLC_PIN();
    ask[3] = src[3 * kLanes];
    PLC_PIN();
    before.y = x;
    pipe_step<FORM>(x, emit, cur[1], cur[2].y);
    asm volatile("s_nop 1");
    PLC_PIN();
    before.z = x;
    pipe_step<FORM>(x, emit, cur[2], cur[3].y);
    __builtin_amdgcn_s_waitcnt(0xc57f);  // lgkmcnt(5)
    PLC_PIN();
    asm volatile("s_nop 0");
    PLC_PIN();
    before.w = x;
    pipe_step<FORM>(x, emit, cur[3], e[(q + 1) % kQuads][0].y);
    held = xb + q * kLanes;
  }
}

// ADAPT: one table per bit depth (the *_bucketed call).  Its entries take 8 bytes where three units are to share a
// compute unit, and unpacking them costs the feeder what the coder saves; WIDE: whole entries, two units to a compute unit
// (512 units of 262,144 symbols 320 -> 298 us; 768 need the third).
template <bool ADAPT, bool WIDE = !ADAPT>
__global__ __launch_bounds__(kThreads) void rans_encode_short_kernel(const RansArgs a) {
  constexpr int kIdentity = (ADAPT ? PLC_MAX_BITS : 1) * 256;  // index of the entry that leaves a state unchanged
  constexpr bool kPacked = ADAPT && !WIDE;
  using Entry = std::conditional_t<kPacked, uint2, uint4>;
  __shared__ Entry table[kIdentity + 1];
  // ADAPT: table of each group of a staging round, in the order in which the feeder's halves want them: a full
  // batch's eight odd groups from the top, then its eight even ones
  __shared__ __attribute__((aligned(8))) uint8_t table_of_group[2][kSuperGroups];
  auto group_at = [](int g) { return (g & ~15) + ((g & 1) ? 0 : 8) + 7 - ((g & 15) >> 1); };
  __shared__ uint4 entry_ring[kEntrySlots][kBatch][kLanes];
  __shared__ uint4 state_ring[kStateSlots][kBatch / 4][kLanes];
  __shared__ __attribute__((aligned(16))) uint8_t sym_stage[2][kSymStage];
  __shared__ __attribute__((aligned(16))) uint16_t word_list[kListRegions][kListRegion];
  __shared__ uint16_t spare_word[64];
  __shared__ uint32_t list_fill[kListRegions];  // positions in use of each region of the list
  static_assert(workgroups_per_cu(sizeof(table) + sizeof(table_of_group) + sizeof(entry_ring) + sizeof(state_ring) +
                                  sizeof(sym_stage) + sizeof(word_list) + sizeof(spare_word) + sizeof(list_fill)) >=
                    (ADAPT && WIDE ? 2 : 3),
                "three units to a compute unit: without the third 513 to 768 units take a second round");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t unit = blockIdx.x;  // one unit per stream, one workgroup per unit

  EncForm form = kEncPlain;  // uniform
  {  // every wavefront scans the frequencies and builds one of a lane's four entries
    const int n_tables = ADAPT ? a.n_tables : 1;
    uint32_t f[ADAPT ? PLC_MAX_BITS : 1][4], cum[ADAPT ? PLC_MAX_BITS : 1];
    for (int t = 0; t < n_tables; ++t) {
      const uint32_t total = load_freq4(a.freq + (unit * n_tables + t) * 256, lane, f[t], &cum[t]);
      if (total != kScale && !(ADAPT && total == 0) && threadIdx.x == 0) raise(a.status, PLC_ERR_INVALID);
      form = enc_form_for(form, enc_form_of(f[t]));
    }
    for (int t = 0; t < n_tables; ++t) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (r == wave) {
          const uint4 e = make_enc_entry(form, f[t][r], cum[t]);
          if constexpr (kPacked) {
            table[t * 256 + lane * 4 + r] = pack_enc_entry(e);
          } else {
            table[t * 256 + lane * 4 + r] = e;
          }
        }
        cum[t] += f[t][r];
      }
    }
    if (threadIdx.x == 0) {  // never emits, x' = x
      const uint4 e = make_uint4(0u, 0xffffffffu, 0u, 0u);
      if constexpr (kPacked) {
        table[kIdentity] = pack_enc_entry(e);
      } else {
        table[kIdentity] = e;
      }
    }
  }

  const uint32_t len = (uint32_t)a.syms_per_stream;
  const uint8_t *ubase = a.sym_in + unit * a.syms_per_stream;
  const uint32_t mis = (uint32_t)(reinterpret_cast<uintptr_t>(ubase) & 15u);
  const int32_t G = (int32_t)((len + kLanes - 1) / kLanes);
  // Batch 0 holds the top G mod 16 groups (a full 16 if that is 0) followed by identity steps; every
  // later batch is 16 full groups.  Batch b codes groups top(b)-1 down to top(b)-16.
  const int32_t head = G % kBatch ? G % kBatch : kBatch;
  const int32_t n_batches = (G - head) / kBatch + 1;
  auto batch_top = [&](int32_t b) { return b == 0 ? G : G - head - (b - 1) * kBatch; };
  // Symbol staging rounds of four batches; a round's buffer starts at the 16-byte-aligned address at or
  // below its lowest symbol, so the symbol at unit offset t sits at  t - 32 * bottom + mis.
  auto round_bottom = [&](int32_t r) {
    const int32_t g = batch_top(4 * r + 3) - kBatch;
    return g > 0 ? g : 0;
  };
  const int32_t n_rounds = (n_batches + 3) / 4;
  const int32_t n_iters = n_batches + 4;
  uint16_t *wp = a.words_out + a.word_off[unit];
  const uint32_t pad = __builtin_amdgcn_readfirstlane((uint32_t)((reinterpret_cast<uintptr_t>(wp) >> 1) & 7u));
  // Restart points: the packer has a record's states and words at hand, the mover its escapes.
  uint32_t *const points = a.points_out ? a.points_out + unit * a.point_stride * PLC_RESTART_WORDS : nullptr;

  if (wave == 0) {
    // ---- coder: batch it - 2
    __syncthreads();  // tables
    __syncthreads();  // first symbols
    uint32_t x = kLow;
    u32x4 e[kBatch / 4][4], before = {0u, 0u, 0u, 0u};
    const u32x4 *const entries = reinterpret_cast<const u32x4 *>(&entry_ring[0][0][lane & 31]);
    u32x4 *const states = reinterpret_cast<u32x4 *>(&state_ring[0][0][lane & 31]);
    u32x4 *held = states + (kStateSlots - 1) * (kBatch / 4) * kLanes;  // (read by nobody yet)
    lds_barrier();  // iteration 0
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j / 4][j % 4] = entries[j * kLanes];
    lds_barrier();  // iteration 1
    auto code = [&](auto form_c) {  // a loop per form, and little in it besides the steps
      constexpr EncForm kForm = decltype(form_c)::value;
      uint64_t emit = __builtin_amdgcn_uicmp(x, e[0][0].y, 34 /* unsigned > */);
      constexpr int kEntryStep = kBatch * kLanes, kStateStep = (kBatch / 4) * kLanes;
      int at = 0, sat = 0;  // uniform
      const u32x4 *eb = entries;
      for (int32_t b = 0; b < n_batches; ++b) {
        at = at == (kEntrySlots - 1) * kEntryStep ? 0 : at + kEntryStep;
        const u32x4 *next = entries + at;
        pipe_batch<kForm>(x, emit, e, before, held, eb, next, states + sat);
        sat = sat == (kStateSlots - 1) * kStateStep ? 0 : sat + kStateStep;
        eb = next;
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();  // iteration b + 2
        asm volatile("" ::: "memory");
      }
    };
    // (the upper half is switched off: it would ask for the same entries once more, 721 instead of 704 us)
    if (lane < kLanes) {
      if (form == kEncLong) {
        code(std::integral_constant<EncForm, kEncLong>{});
      } else if (form == kEncPlain) {
        code(std::integral_constant<EncForm, kEncPlain>{});
      } else {
        code(std::integral_constant<EncForm, kEncShort>{});
      }
      *held = before;  // the last four states, in place before the barrier behind them
    }
    for (int32_t it = n_batches + 2; it < n_iters; ++it) lds_barrier();
    if (lane < kLanes) {
      a.states_out[unit * kLanes + lane] = x;
      if (points) points[lane] = x;
    }
  } else if (wave == 1) {
    // ---- feeder: entries of batch it
    __syncthreads();  // tables
    __syncthreads();  // first symbols
    bool bad_symbol = false;
    int slot = 0;
    for (int32_t it = 0; it < n_iters; ++it) {
      if (it < n_batches) {
        const int32_t r = it >> 2;
        const int32_t top = batch_top(it), bottom = round_bottom(r);
        const uint8_t *sb = sym_stage[r & 1];
        // lane (half h, l) serves step 2p + h of the batch: group top - 1 - 2p - h, rANS lane l
        const int half = lane >> 5, l = lane & 31;
        uint4 *eo = &entry_ring[slot][half][l];
        if (it > 0) {
          // 16 full groups: all symbol reads, then all table reads, then all ring writes, so that the LDS
          // round trips overlap instead of queueing one behind the other
          const uint8_t *s0 = sb + ((top - bottom - 2 * (kBatch / 2 - 1) - 1 - half) * kLanes + l + (int32_t)mis);
          uint32_t sy[kBatch / 2];
          u32x4 e[kBatch / 2];  // native vectors: each entry moves as one 16-byte LDS access
#pragma unroll
          for (int p = 0; p < kBatch / 2; ++p) sy[p] = s0[2 * kLanes * (kBatch / 2 - 1 - p)];
          uint32_t any = 0;
          if constexpr (ADAPT) {  // the group of step 2p + half sits at top - bottom - 1 - half - 2p of the round
            const uint2 tg = *reinterpret_cast<const uint2 *>(&table_of_group[r & 1][top - bottom - kBatch + 8 * half]);
#pragma unroll
            for (int p = 0; p < kBatch / 2; ++p)  // symbol | table << 8
              sy[p] = __builtin_amdgcn_perm(p < 4 ? tg.x : tg.y, sy[p], 0x0c0c0400u + ((uint32_t)(p & 3) << 8));
          }
          if constexpr (kPacked) {
            uint2 c[kBatch / 2];
#pragma unroll
            for (int p = 0; p < kBatch / 2; ++p) c[p] = table[sy[p]];
#pragma unroll
            for (int p = 0; p < kBatch / 2; ++p) {
              any |= c[p].y;
              const uint4 v = unpack_enc_entry(c[p]);
              e[p] = u32x4{v.x, v.y, v.z, v.w};
            }
          } else {
#pragma unroll
            for (int p = 0; p < kBatch / 2; ++p) e[p] = *reinterpret_cast<const u32x4 *>(&table[sy[p]]);
#pragma unroll
            for (int p = 0; p < kBatch / 2; ++p) any |= e[p].w;
          }
#pragma unroll
          for (int p = 0; p < kBatch / 2; ++p) *reinterpret_cast<u32x4 *>(eo + 2 * p * kLanes) = e[p];
          bad_symbol = bad_symbol || (any & 0x80000000u) != 0;
        } else {
          // the top batch: `head` groups, the first of them possibly ragged, then identity steps
#pragma unroll
          for (int p = 0; p < kBatch / 2; ++p) {
            const int j = 2 * p + half;
            const int64_t t = (int64_t)(top - 1 - j) * kLanes + l;
            const bool has = j < head && t < (int64_t)len;
            const int64_t idx = has ? t - (int64_t)bottom * kLanes + mis : 0;
            uint32_t byte = sb[idx];
            if (ADAPT && has) byte += (uint32_t)table_of_group[r & 1][group_at(top - 1 - j - bottom)] << 8;
            const Entry c = table[has ? byte : (uint32_t)kIdentity];
            if constexpr (kPacked) {
              bad_symbol = bad_symbol || (c.y & 0x80000000u) != 0;
              eo[2 * p * kLanes] = unpack_enc_entry(c);
            } else {
              bad_symbol = bad_symbol || (c.w & 0x80000000u) != 0;
              eo[2 * p * kLanes] = c;
            }
          }
        }
        slot = slot == kEntrySlots - 1 ? 0 : slot + 1;
      }
      lds_barrier();
    }
    if (bad_symbol) raise(a.status, PLC_ERR_INVALID);  // a symbol with f = 0
  } else if (wave == 2) {
    // ---- packer: batch it - 4
    __syncthreads();  // tables
    __syncthreads();  // first symbols
    uint32_t fill = pad;  // uniform: positions of the region in use, the first of them not this pair's words
    int region = 0;
    uint32_t gone = 0u - pad;  // words of the regions before (the padding in front of the first taken off)
    int32_t point_at = points ? a.piece_batches : INT32_MAX;  // the batch that the next record stands in front of
    uint32_t *record = points;
    // hardware lane h of a half carries rANS lane 31 - h, which the encoder visits first; a lane serves
    // step 2p + half, whose state is component 2 * (p & 1) + half of quad p / 2
    const int half = lane >> 5, rl = 31 - (lane & 31);
    uint16_t *const spare = &spare_word[lane];
    // The thresholds are read two batches ahead of the states, while the coder is at their entries, and wait in
    // registers: three sets, so three iterations a turn.
    uint32_t thrs[3][kBatch / 2];
    auto pack = [&](auto turn, int32_t it) {
      constexpr int kTurn = decltype(turn)::value;  // it mod 3
      {
        const uint32_t *ts = &entry_ring[(kTurn + 1) % 3][half][rl].y;  // batch it - 2
#pragma unroll
        for (int p = 0; p < kBatch / 2; ++p) thrs[kTurn][p] = ts[2 * p * kLanes * 4];
      }
      const int32_t b = it - 4;
      if (b >= 0 && b < n_batches) {
        const uint32_t(&thr)[kBatch / 2] = thrs[(kTurn + 1) % 3];
        const uint32_t *xs = reinterpret_cast<const uint32_t *>(&state_ring[(kTurn + 2) % 3][0][rl]) + half;
        uint16_t *list = word_list[region];
        // In phases, each over all eight step pairs: reads, emit masks, list positions, stores.  A lane without
        // a word stores into a slot of its own instead of sitting out the store.
        uint32_t xps[kBatch / 2], at[kBatch / 2];
#pragma unroll
        for (int p = 0; p < kBatch / 2; ++p) xps[p] = xs[(p / 2) * kLanes * 4 + 2 * (p & 1)];
        if (b == point_at) {  // uniform; the states in front of the batch's first step
          point_at += a.piece_batches;
          record += PLC_RESTART_WORDS;
          if (half == 0) record[rl] = xps[0];
          if (lane == 0) record[kLanes] = gone + fill;
        }
#pragma unroll
        for (int p = 0; p < kBatch / 2; ++p) {
          const uint64_t mask = __ballot(xps[p] > thr[p]);
          at[p] = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, fill));
          fill += (uint32_t)__builtin_popcountll(mask);
        }
#pragma unroll
        for (int p = 0; p < kBatch / 2; ++p) *(xps[p] > thr[p] ? list + at[p] : spare) = (uint16_t)xps[p];
        if ((b & 1) || b == n_batches - 1) {  // on to the next pair's region
          if (lane == 0) list_fill[region] = fill;
          region = region == kListRegions - 1 ? 0 : region + 1;
          gone += fill & ~7u;
          fill &= 7u;
        }
      }
      lds_barrier();
    };
    static_assert(kEntrySlots == 3 && kStateSlots == 3, "three iterations a turn");
    for (int32_t it = 0; it < n_iters; it += 3) {
      pack(std::integral_constant<int, 0>{}, it);
      if (it + 1 < n_iters) pack(std::integral_constant<int, 1>{}, it + 1);
      if (it + 2 < n_iters) pack(std::integral_constant<int, 2>{}, it + 2);
    }
  } else {
    // ---- mover: symbols of the coming round, words of batch it - 5
    bool bad_depth = false;
    uint4 nv[kStagePieces];         // next round's symbols in flight
    bool ntake[kStagePieces];
    // ADAPT: depth of group bottom + lane of the next round.  It is looked at when the round's symbols land: where it
    // is asked for, its range check would have the wavefront, and at the barrier the others, wait for the answer in
    // every round (964 -> 829 us for 256 units of 1,048,576 symbols).
    uint32_t next_depth = 1;
    const uint32_t spp = ADAPT ? (uint32_t)a.syms_per_pos : 1u;
    const uint8_t *const depth_row =
        ADAPT ? a.bits + (int64_t)((uint32_t)unit / (uint32_t)a.streams_per_session) * (len / spp) : nullptr;
    auto round_load = [&](int32_t r) {
      const int64_t lo = (int64_t)round_bottom(r) * kLanes;
      int64_t hi = (int64_t)batch_top(4 * r) * kLanes;
      hi = hi < (int64_t)len ? hi : (int64_t)len;
#pragma unroll
      for (int i = 0; i < kStagePieces; ++i) {
        const int64_t off = lo - (int64_t)mis + (int64_t)(lane + 64 * i) * 16;  // 16-byte aligned in absolute address
        ntake[i] = r < n_rounds && off < hi;
        if (ntake[i]) nv[i] = load16_stream(ubase + off);
      }
      if (ADAPT) {
        const int32_t g = round_bottom(r) + lane;
        next_depth = (r < n_rounds && g < batch_top(4 * r)) ? depth_row[(uint32_t)g * kLanes / spp] : 1u;
      }
    };
    auto round_store = [&](int buf) {
#pragma unroll
      for (int i = 0; i < kStagePieces; ++i)
        if (ntake[i]) *reinterpret_cast<uint4 *>(&sym_stage[buf][(lane + 64 * i) * 16]) = nv[i];
      if (ADAPT) {
        const bool known = next_depth >= 1u && next_depth <= (uint32_t)a.n_tables;
        bad_depth = bad_depth || !known;
        table_of_group[buf][group_at(lane)] = (uint8_t)(known ? next_depth - 1u : 0u);
      }
    };
    round_load(0);
    __syncthreads();  // tables
    round_store(0);
    round_load(1);
    __syncthreads();  // first symbols
    // Words.  Position p of a region stands for the word at 16-byte-aligned address (wp - pad) + vbase + p; the
    // first `pad` positions of the first are padding in front of the unit's first word.  The complete 16-byte
    // pieces leave, up to two per lane; the incomplete tail (< 8 words) moves to the front of the next region, in
    // front of the words that the packer has written or is writing there.
    const uint32_t cap = a.word_cap < 0x7fffffffull ? (uint32_t)a.word_cap : 0x7fffffffu;  // a unit has < 2^31 symbols
    uint32_t vbase = 0, rest = pad;
    const int32_t n_pairs = (n_batches + 1) / 2;
    int32_t out_pair = 0;  // the next pair of batches whose words leave
    int region = 0;
    auto words_out = [&]() {
      const uint16_t *list = word_list[region];
      const uint32_t fill = __builtin_amdgcn_readfirstlane(list_fill[region]);
      region = region == kListRegions - 1 ? 0 : region + 1;
      const uint32_t full = fill / 8;  // at most 128
      rest = fill - 8 * full;
      const uint16_t tail = list[8 * full + (lane & 7)];  // (lanes past the tail read inside the region)
      if (vbase >= pad && vbase + 8 * full - pad <= cap) {
        uint16_t *dst = wp + (vbase - pad);  // 16-byte aligned
        uint4 v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)  // (a lane past the last piece reads inside the region)
          v[h] = *reinterpret_cast<const uint4 *>(list + 8 * (lane + 64 * h));
#pragma unroll
        for (int h = 0; h < 2; ++h)
          if ((uint32_t)(lane + 64 * h) < full) *reinterpret_cast<uint4 *>(dst + 8 * (lane + 64 * h)) = v[h];
      } else {
        for (uint32_t q = lane; q < 8 * full; q += 64) {
          const uint32_t v = vbase + q;
          if (v >= pad && v - pad < cap) wp[v - pad] = list[q];
        }
      }
      vbase += 8 * full;
      ++out_pair;
      if ((uint32_t)lane < rest) {
        if (out_pair < n_pairs) {
          word_list[region][lane] = tail;
        } else {  // the incomplete last piece
          const uint32_t v = vbase + (uint32_t)lane;
          if (v >= pad && v - pad < cap) wp[v - pad] = tail;
        }
      }
      wave_sync();  // the next pair's reads come behind the tail's way to its front, from other lanes (no barrier
                    // stands between them where pairs leave one behind the other at the unit's end)
    };
    // Escapes, for the restart points: a round's symbols are counted in the stage in the last iteration before others
    // take their place, in which the mover has nothing else to do.
    uint32_t esc_mine = 0;  // this lane's, of the rounds so far
    int32_t point_at = points ? a.piece_batches / 4 : INT32_MAX;  // the round that the next record stands in front of
    uint32_t *record = points;
    auto count_round = [&](int32_t r) {
      if (r == point_at) {
        point_at += a.piece_batches / 4;
        record += PLC_RESTART_WORDS;
        const uint32_t total = wave_sum(esc_mine);
        if (lane == 0) record[kLanes + 1] = total;
      }
      const uint8_t *sb = sym_stage[r & 1];
      const uint32_t lo = (uint32_t)round_bottom(r) * kLanes, top = (uint32_t)batch_top(4 * r) * kLanes;
      const uint32_t n = (top < len ? top : len) - lo;
      if (mis == 0 && n == (uint32_t)kSuperSyms) {  // uniform
#pragma unroll
        for (int h = 0; h < kSuperSyms / 1024; ++h) {
          const uint4 v = *reinterpret_cast<const uint4 *>(&sb[(lane + 64 * h) * 16]);
          const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int i = 0; i < 4; ++i)  // a byte is 0xff iff its low seven bits carry into bit 7 and bit 7 is set
            esc_mine += (uint32_t)__builtin_popcount(((w[i] & 0x7f7f7f7fu) + 0x01010101u) & w[i] & 0x80808080u);
        }
      } else {
        for (uint32_t t = lane; t < n; t += 64) esc_mine += sb[t + mis] == PLC_ESCAPE;
      }
    };
    for (int32_t it = 0; it < n_iters; ++it) {
      const int32_t phase = it & 3;
      if (phase == 3 && points && (it >> 2) < n_rounds) count_round(it >> 2);
      if (phase == 0 && it < n_batches) {  // the feeder has begun a round: the next one's symbols land
        const int32_t r = it >> 2;
        round_store((r + 1) & 1);
        round_load(r + 2);
      }
      // (batch it - 5 is packed: in steady state a pair goes out at phase 1 and the next one at phase 2)
      if ((phase == 1 || phase == 2) && 2 * out_pair + 1 <= it - 5) words_out();
      lds_barrier();
    }
    while (out_pair < n_pairs) words_out();
    const uint32_t n_words = vbase + rest - pad;
    const uint32_t esc_total = wave_sum(esc_mine);
    if (lane == 0) {
      a.n_words_out[unit] = n_words;
      if ((uint64_t)n_words > a.word_cap) raise(a.status, PLC_ERR_CAPACITY);
      if (points) points[kLanes] = n_words, points[kLanes + 1] = esc_total;
    }
    if (bad_depth) raise(a.status, PLC_ERR_INVALID);
  }
}
}  // namespace short_units

// ---------------------------------------------------------------------------
// Decoder
// ---------------------------------------------------------------------------
// Slot tables are filled through an index of the symbols that occur: a bit for each slot at which one begins, and
// the symbols' frequencies and first slots in a row.  A slot's symbol is the one whose number is the count of set bits
// up to it: a read that 32 lanes share, a count, and a read of the row, then whatever the table's entry takes.  A table
// for a workgroup of 128 threads takes 1.6 us so; searching each slot's symbol in eight halvings took 7.5, and
// filling in each symbol's slots in a loop 14.
struct SlotIndex {
  uint2 words[kScale / 32];  // .x the bits, .y the occurring symbols in front of them
  uint32_t row[256];         // f - 1 | first slot << 12 | symbol << 24
};
// By one wavefront, from what load_freq4 gave it of a table that sums to 4096.
__device__ __forceinline__ void build_slot_index(SlotIndex *ix, const uint32_t f[4], uint32_t cum, int lane) {
  ix->words[lane] = ix->words[lane + 64] = make_uint2(0u, 0u);
  wave_sync();
  const uint32_t occur = (f[0] ? 1u : 0u) + (f[1] ? 1u : 0u) + (f[2] ? 1u : 0u) + (f[3] ? 1u : 0u);
  uint32_t at = wave_inclusive_scan(occur) - occur;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (f[r]) {
      atomicOr(&ix->words[cum >> 5].x, 1u << (cum & 31u));
      ix->row[at] = (f[r] - 1u) | (cum << 12) | ((uint32_t)(lane * 4 + r) << 24);
      ++at;
      cum += f[r];
    }
  }
  wave_sync();
  const uint32_t n0 = __builtin_popcount(ix->words[2 * lane].x), n1 = __builtin_popcount(ix->words[2 * lane + 1].x);
  const uint32_t before = wave_inclusive_scan(n0 + n1) - (n0 + n1);
  ix->words[2 * lane].y = before;
  ix->words[2 * lane + 1].y = before + n0;
}
// put(slot, entry of the row) for every slot, by THREADS threads; the index in place behind a barrier.
template <int THREADS, typename Put>
__device__ __forceinline__ void for_each_slot(const SlotIndex *ix, Put put) {
  static_assert(THREADS % 32 == 0, "a thread stays at one bit");
  constexpr int kAtOnce = kScale / THREADS < 8 ? kScale / THREADS : 8;  // so that their LDS round trips overlap
  const uint32_t upto = 0xffffffffu >> (31u - (threadIdx.x & 31u));
  for (uint32_t o0 = threadIdx.x; o0 < kScale; o0 += THREADS * kAtOnce) {
    uint2 w[kAtOnce];
    uint32_t row[kAtOnce];
#pragma unroll
    for (int i = 0; i < kAtOnce; ++i) w[i] = ix->words[(o0 + (uint32_t)(THREADS * i)) >> 5];
#pragma unroll
    for (int i = 0; i < kAtOnce; ++i) row[i] = ix->row[__builtin_popcount(w[i].x & upto) + w[i].y - 1u];
#pragma unroll
    for (int i = 0; i < kAtOnce; ++i) put(o0 + (uint32_t)(THREADS * i), row[i]);
  }
}

// Words are consumed from the end of the unit's list.  They are staged through
// a per-wavefront LDS ring of four 512-word blocks (blocks aligned in absolute
// address), refilled at most one block per batch of 16 groups, which consumes
// at most 512 words.  The ring is stored backwards -- word i sits at position
// (~i) mod 2048 -- so that the word of the lane with rank r is at position
// q + r, where q = (-ptr) mod 2048 at the start of a batch and then simply
// grows by the words consumed, in a scalar register; positions 0..543 are
// mirrored at 2048..2591 so that q + r never needs a wrap inside a batch.
constexpr int kRingWords = 2048, kBlockWords = 512, kRingMirror = kBlockWords + 32;

// The slot table is split in two, slot -> symbol (one byte per slot) and symbol -> f - 1 | cum << 16: 5 KB instead of
// the 16 KB of a word per slot, at the price of a second dependent lookup.
constexpr uint32_t kCompactTable = 256 + kScale / 4;  // in 32-bit words
template <bool MASKED>
__device__ __forceinline__ void dec_step(uint32_t &x, const uint32_t *lut, const uint16_t *&top, uint8_t *sym_slot,
                                         uint32_t below, bool on, uint32_t table_off = 0) {
  const uint32_t slot = x & (kScale - 1);
  const uint32_t *mine = lut + table_off;
  const uint32_t s = reinterpret_cast<const uint8_t *>(mine + 256)[slot];
  const uint32_t fc = mine[s];
  const uint32_t e = s | ((fc & 0xfffu) << 8) | ((slot - (fc >> 16)) << 20);
  const uint32_t xh = x >> kScaleBits;
  uint32_t xn = __umul24((e >> 8) & 0xfffu, xh) + (xh + (e >> 20));  // f * (x >> 12) + slot - cum
  uint32_t m32 = (uint32_t)__builtin_amdgcn_uicmp(xn, kLow, 36 /* unsigned < */);
  bool need = xn < kLow;
  if (MASKED) {
    need = need && on;
    m32 = (uint32_t)__builtin_amdgcn_ballot_w64(need);
  }
  if (need) {
    // The decoder visits lane 0 first: a lane's word is the rank-th from the top of the list (`top`
    // points at the top word in the backwards ring).  `below` is the mask of the lanes under this one
    // within its half, so that a mirror lane ranks like its twin.
    xn = (xn << 16) | top[__builtin_popcount(m32 & below)];
  }
  top += __builtin_popcount(m32);
  if (MASKED) {
    if (on) {
      *sym_slot = (uint8_t)e;
      x = xn;
    }
  } else {
    *sym_slot = (uint8_t)e;
    x = xn;
  }
}

// Many streams of one unit each: a wavefront, with tables of its own, per workgroup.  And with a table per depth chunks
// that are few, W of a stream to a workgroup (CHUNKS; kFewChunks).
template <int W, bool ADAPT, bool CHUNKS>
__global__ __launch_bounds__(W * 64) void rans_decode_kernel(const RansArgs a) {
  __shared__ uint32_t lut_one[ADAPT ? 1 : kCompactTable];
  extern __shared__ uint32_t lut_per_depth[];  // ADAPT: n_tables slot tables, sized at launch
  uint32_t *lut = ADAPT ? lut_per_depth : lut_one;
  __shared__ uint16_t table_of_group_of[W][2][kBatch];  // ADAPT: table offset of each group of a batch
  __shared__ __attribute__((aligned(16))) uint16_t ring[W][kRingWords + kRingMirror];
  __shared__ __attribute__((aligned(16))) uint8_t sym_stage_of[W][kBatchSyms];
  const int lane = threadIdx.x & 63, wave = W == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t stream = CHUNKS ? blockIdx.x / a.wgs_per_stream : blockIdx.x;
  const int64_t chunk = CHUNKS ? (int64_t)(blockIdx.x - stream * a.wgs_per_stream) * W + wave : 0;
  auto sync = [] {
    if constexpr (W == 1) {
      wave_sync();
    } else {
      __syncthreads();
    }
  };
  if (a.verified_pieces && stream_verified(a, stream)) return;  // uniform: nothing to decode again
  bool bad = false;

  // One slot table, or one per bit depth: that of a depth the stream does not use is all zero.  The index in the
  // place of a ring.
  SlotIndex *const index = reinterpret_cast<SlotIndex *>(&ring[0][0]);
  static_assert(sizeof(ring[0]) >= sizeof(SlotIndex), "room for the index");
  const int n_tables = ADAPT ? a.n_tables : 1;
  bool ok = true;
  for (int t = 0; t < n_tables; ++t) {
    uint32_t f[4], cum;
    const uint32_t total = load_freq4(a.freq + (stream * n_tables + t) * 256, lane, f, &cum);
    ok = ok && (total == kScale || (ADAPT && total == 0));
    uint32_t *lt = lut + t * kCompactTable;
    if (total == kScale && wave == 0) {  // uniform
      build_slot_index(index, f, cum, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        lt[lane * 4 + r] = ((f[r] - 1u) & 0xfffu) | (cum << 16);  // a symbol that does not occur is never looked up
        cum += f[r];
      }
    }
    sync();
    if (total == kScale) {
      for_each_slot<W * 64>(index, [&](uint32_t o, uint32_t row) {
        reinterpret_cast<uint8_t *>(lt + 256)[o] = (uint8_t)(row >> 24);
      });
    } else {
      for (uint32_t o = threadIdx.x; o < kCompactTable; o += W * 64) lt[o] = 0u;
    }
    sync();  // before the index serves the next table, or the ring takes its place
  }
  if (CHUNKS && chunk >= a.units_per_stream) return;  // no workgroup barrier below
  const int64_t unit = CHUNKS ? stream * a.units_per_stream + chunk : stream;
  const uint64_t off = a.word_off[unit];
  const uint32_t n = a.n_words_in[unit];
  if (!ok || off > a.words_len || (uint64_t)n > a.words_len - off) {  // (not a table: nothing can be decoded)
    if (lane == 0) raise(a.status, PLC_ERR_CORRUPT);
    return;
  }
  const int64_t begin = CHUNKS ? chunk * a.unit_syms : 0;
  const int64_t rest = a.syms_per_stream - begin;
  const uint32_t len = (uint32_t)(CHUNKS && a.unit_syms < rest ? a.unit_syms : rest);
  uint8_t *ubase = a.sym_out + stream * a.syms_per_stream + begin;
  auto &table_of_group = table_of_group_of[wave];
  auto &sym_stage = sym_stage_of[wave];
  const bool out_aligned = (reinterpret_cast<uintptr_t>(ubase) & 15u) == 0;
  const int32_t G = (int32_t)((len + kLanes - 1) / kLanes);
  const uint32_t top_syms = len - (uint32_t)(G - 1) * kLanes;

  // ---- word list geometry, relative to a 1 KiB-aligned address at or below the unit's first word
  const uint16_t *first_word = a.words_in + off;
  const int32_t lo = (int32_t)((reinterpret_cast<uintptr_t>(first_word) & (uintptr_t)(kBlockWords * 2 - 1)) >> 1);
  const uint16_t *aligned_base = first_word - lo;  // pointer arithmetic keeps the loads global, not flat
  const int32_t hi = lo + (int32_t)n;
  uint16_t *myring = ring[wave];

  // one 16-byte piece (eight words) of block blk per lane, if the piece holds a word of this unit
  auto block_load = [&](int32_t blk, uint4 &v) -> bool {
    const int32_t first = blk * kBlockWords + lane * 8;
    const bool take = blk >= 0 && hi > lo && first + 8 > lo && first < hi;
    if (take) v = *reinterpret_cast<const uint4 *>(aligned_base + first);
    return take;
  };
  // word i goes to ring position (~i) mod 2048: a piece of eight words lands reversed on an aligned run
  auto block_store = [&](int32_t blk, bool take, const uint4 &v) {
    if (take) {
      const uint32_t pos = (uint32_t)(~(blk * kBlockWords + lane * 8 + 7)) & (kRingWords - 1);
      const uint4 r = make_uint4((v.w >> 16) | (v.w << 16), (v.z >> 16) | (v.z << 16), (v.y >> 16) | (v.y << 16),
                                 (v.x >> 16) | (v.x << 16));
      *reinterpret_cast<uint4 *>(myring + pos) = r;
      if (pos < kRingMirror) *reinterpret_cast<uint4 *>(myring + kRingWords + pos) = r;
    }
  };

  int32_t ptr = hi;
  int32_t lowest = ((hi - 1) >> 9) + 1;  // lowest block already staged (none yet)
  for (int r = 0; r < 2; ++r) {          // the two top blocks
    uint4 v;
    const int32_t blk = lowest - 1;
    const bool take = block_load(blk, v);
    block_store(blk, take, v);
    lowest = blk;
  }
  wave_sync();

  const bool coder = lane < kLanes;
  const int rl = lane & (kLanes - 1);
  const uint32_t below = (1u << rl) - 1u;
  const bool top_active = (uint32_t)rl < top_syms;
  uint32_t x = a.states_in[unit * kLanes + rl];

  // Full batches of 16 groups are fully unrolled; the groups that do not fill a batch (and the last
  // group if it is ragged) form a tail that runs in a rolled loop.
  int32_t tail_groups = G % kBatch;
  if (tail_groups == 0 && top_syms < kLanes) tail_groups = kBatch;
  const int32_t g_tail = G - tail_groups;
  uint8_t *sb = &sym_stage[rl];

  // ADAPT: table offsets of the batch's 16 groups, fetched one batch ahead by lanes 0..15
  bool bad_depth = false;
  auto group_load = [&](int32_t g0) -> uint32_t {
    const int32_t g = g0 + lane;
    if (!ADAPT || lane >= kBatch || g >= G) return 0u;
    return group_table(a, stream, begin, g, kCompactTable, &bad_depth);
  };
  if (ADAPT) {
    const uint32_t gt0 = group_load(0);
    if (lane < kBatch) table_of_group[0][lane] = (uint16_t)gt0;
    wave_sync();
  }
  int gbuf = 0;

  for (int32_t g0 = 0; g0 < G; g0 += kBatch) {
    const bool tail = g0 >= g_tail;
    const int32_t cnt_groups = tail ? tail_groups : kBatch;
    // stage one more block below if the coming batches may reach it
    const int32_t top = (ptr - 1) >> 9;
    const bool fetch = lowest > top - 2;
    const int32_t blk = lowest - 1;
    uint4 pre;
    bool ptake = false;
    if (fetch) ptake = block_load(blk, pre);
    const uint32_t ngt = group_load(g0 + kBatch);
    const uint16_t *gt = table_of_group[gbuf];

    const uint16_t *wtop0 = myring + ((uint32_t)(-ptr) & (kRingWords - 1));
    const uint16_t *wtop = wtop0;
    if (tail) {
      for (int32_t j = 0; j < cnt_groups; ++j)
        dec_step<true>(x, lut, wtop, sb + kLanes * j, below, j != cnt_groups - 1 || top_active,
                                ADAPT ? gt[j] : 0u);
    } else {
      // the batch's table offsets are read before its first symbol is stored (the compiler cannot tell
      // the two LDS arrays apart, and a read inside a step would queue behind the previous step's store)
      uint32_t off[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) off[j] = ADAPT ? (uint32_t)__builtin_amdgcn_readfirstlane(gt[j]) : 0u;
#pragma unroll
      for (int j = 0; j < kBatch; ++j) dec_step<false>(x, lut, wtop, sb + kLanes * j, below, true, off[j]);
    }
    if (ADAPT) {
      if (lane < kBatch) table_of_group[gbuf ^ 1][lane] = (uint16_t)ngt;
      gbuf ^= 1;
    }
    ptr -= (int32_t)(wtop - wtop0);
    if (ptr < lo) {  // ran out of words: the stream is damaged
      bad = true;
      ptr = lo;
    }
    // the prefetched block goes to the ring BEFORE this batch's symbols are stored: waiting for the load
    // then does not also wait for freshly issued stores (loads and stores share one counter)
    if (fetch) {
      block_store(blk, ptake, pre);
      lowest = blk;
    }
    wave_sync();
    // drain the batch's symbols
    const uint32_t done = (uint32_t)g0 * kLanes;
    const uint32_t room = (uint32_t)cnt_groups * kLanes;
    const uint32_t nsym = (len - done) < room ? (len - done) : room;
    if (out_aligned) {
      const uint32_t full = nsym / 16;
      if ((uint32_t)lane < full)
        *reinterpret_cast<uint4 *>(ubase + done + lane * 16) =
            *reinterpret_cast<const uint4 *>(&sym_stage[lane * 16]);
      const uint32_t tail = full * 16 + (uint32_t)lane;
      if (tail < nsym) ubase[done + tail] = sym_stage[tail];
    } else {
      for (uint32_t i = lane; i < nsym; i += 64) ubase[done + i] = sym_stage[i];
    }
    wave_sync();
  }
  // integrity: every word consumed, every lane back at the initial state
  if (ptr != lo || (coder && x != kLow)) bad = true;
  if (bad) raise(a.status, PLC_ERR_CORRUPT);
  if (bad_depth) raise(a.status, PLC_ERR_INVALID);
}

// ---------------------------------------------------------------------------
// Decoder, many units of one stream: two units per wavefront
// ---------------------------------------------------------------------------
// With the chip full of units the decoder is bound by instruction issue, and half of every instruction's lanes above only
// mirror the other half.  Here lanes 32-63 decode a unit of their own with the same instructions, the next of the
// same stream, so that a workgroup's units share one slot table of whole entries (16 KB, one lookup a step) -- or,
// with a table per bit depth, one split table per depth.  What is per half: the list of words and the place in it, a
// lane's rank among its own half's renormalising lanes, and the ends of the units.  The words are staged as
// above, in blocks of 256 for batches of eight steps, so that a unit needs 2 KB of LDS instead of 5.7 and a compute
// unit holds 48 of them: what the wider wavefronts gain in issue they would lose again in latency with fewer.
// The ring keeps the words in their order, word i at place i mod 512 behind a guard of one block that repeats the
// upper; a lane's word is the rank-th below the pointer, counted through the lanes that do NOT take one.
constexpr int kPairSteps = 8;
constexpr int kPairBlock = kPairSteps * kLanes;  // words: the most a batch takes
constexpr int kPairRing = 2 * kPairBlock;
constexpr int kPairDrain = 2 * kPairBlock;       // symbols: two batches leave together, 16 bytes a lane
static_assert(kTileSyms % kPairDrain == 0, "a tile's symbols leave in whole drains");

// One step of both halves, all 64 lanes on.  `at`: a lane's word is `later` steps' worth of lanes above place at + the
// number of lanes below it in its half that take none; at moves on by the half's number of them.  MASKED: lanes that
// are not in `on` do nothing, and a frequency of 4096 (0 in its twelve bits; elsewhere such tables do not come here)
// is minded.  ADAPT: `table` is the offset of the half's table.
// The two halves take turns at ranking and moving on, each with its own 32 bits of the mask and the other's lanes
// switched off; then the lanes that take a word shift it in, the others switched off.  (Between the compare and the
// first reader of its mask there have to be two instructions.)
template <bool ADAPT, bool MASKED>
__device__ __forceinline__ void dec_pair_step(uint32_t &x, const uint32_t *lut, uint32_t table, uint32_t &at,
                                              const uint16_t *ring, int later, uint8_t *sym_slot, uint64_t on) {
  const uint32_t slot = x & (kScale - 1);
  uint32_t s, f, r;  // symbol, frequency, slot - cum
  if constexpr (ADAPT) {
    const uint32_t *mine = lut + table;
    s = reinterpret_cast<const uint8_t *>(mine + 256)[slot];
    const uint32_t fc = mine[s];
    f = fc & 0xfffu;
    r = slot - (fc >> 16);
  } else {
    const uint32_t e = lut[slot];
    s = e;
    f = (e >> 8) & 0xfffu;
    r = e >> 20;
  }
  if (MASKED) f = f ? f : kScale;
  uint32_t xn = __umul24(f, x >> kScaleBits) + r;
  uint64_t keep = __builtin_amdgcn_uicmp(xn, kLow, 35 /* unsigned >= */);
  if (MASKED) keep |= ~on;
  uint32_t place;
  uint64_t all;
  asm volatile(
      "s_mov_b64 %2, exec\n\t"
      "s_mov_b32 exec_hi, 0\n\t"
      "v_mbcnt_lo_u32_b32 %0, %3, %1\n\t"
      "v_bcnt_u32_b32 %1, %3, %1\n\t"
      "s_mov_b64 exec, %2\n\t"
      "s_mov_b32 exec_lo, 0\n\t"
      "v_mbcnt_hi_u32_b32 %0, %4, %1\n\t"
      "v_bcnt_u32_b32 %1, %4, %1\n\t"
      "s_mov_b64 exec, %2"
      : "=&v"(place), "+v"(at), "=&s"(all)
      : "s"((uint32_t)keep), "s"((uint32_t)(keep >> 32)));
  const uint32_t word = ring[place + (uint32_t)(kLanes * later)];  // (read by every lane: no branch around it)
  const bool live = !MASKED || __builtin_amdgcn_inverse_ballot_w64(on);
  if (live) *sym_slot = (uint8_t)s;
  if (MASKED) {
    x = !live ? x : __builtin_amdgcn_inverse_ballot_w64(keep) ? xn : (xn << 16) | word;
  } else {
    asm volatile(
        "s_not_b64 exec, %2\n\t"
        "v_lshl_or_b32 %0, %0, 16, %1\n\t"
        "s_mov_b64 exec, -1"
        : "+v"(xn)
        : "v"(word), "s"(keep)
        : "scc");
    x = xn;
  }
}

// PIECES: a unit is a piece of a stream, and errors are left to the second launch.
template <int W, bool ADAPT, bool PIECES>
__global__ __launch_bounds__(W * 64) void rans_decode_pair_kernel(const RansArgs a) {
  __shared__ uint32_t lut_one[ADAPT ? 1 : kScale];
  extern __shared__ uint32_t lut_per_depth[];  // ADAPT: n_tables slot tables, sized at launch
  uint32_t *lut = ADAPT ? lut_per_depth : lut_one;
  __shared__ __attribute__((aligned(16))) uint16_t table_of_group[ADAPT ? W : 1][2][2][2 * kPairSteps];  // ADAPT: table offsets
  __shared__ __attribute__((aligned(16))) uint16_t ring[W][2][kPairBlock + kPairRing];
  __shared__ __attribute__((aligned(16))) uint8_t sym_stage[W][2][kPairDrain];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5, hl = lane & (kLanes - 1);
  const int64_t stream = blockIdx.x / a.wgs_per_stream;
  const int64_t chunk = ((int64_t)(blockIdx.x - stream * a.wgs_per_stream) * W + wave) * 2 + half;
  const int64_t n_units = PIECES ? (int64_t)a.pieces : a.units_per_stream;
  const bool live = chunk < n_units;
  // Escapes of each tile: where the caller counts on them, a unit is whole tiles.
  const int64_t tiles_per_stream = (a.syms_per_stream + kTileSyms - 1) / kTileSyms;
  // Every lane of a half alike.  A unit that is not decoded still has its tiles counted, as they stand in the symbol
  // buffer: the escapes of the stream's other units have their places behind them.  (Of pieces the second launch
  // decodes the whole stream, and what it leaves is counted then.)
  auto fail = [&]() {
    if (!live) return;
    if (PIECES) {
      if (hl == 0) report_piece(a, stream, (int32_t)chunk, 0, false);
      return;
    }
    if (hl == 0) raise(a.status, PLC_ERR_CORRUPT);
    if (!a.tile_cnt) return;
    const int64_t from = chunk * a.unit_syms;
    const int64_t to = from + a.unit_syms < a.syms_per_stream ? from + a.unit_syms : a.syms_per_stream;
    for (int64_t t0 = from; t0 < to; t0 += kTileSyms) {
      uint32_t n_esc = 0;
      for (int64_t i = t0 + hl; i < t0 + kTileSyms && i < to; i += kLanes)
        n_esc += a.sym_out[stream * a.syms_per_stream + i] == PLC_ESCAPE;
#pragma unroll
      for (int d = 1; d < kLanes; d <<= 1) n_esc += __shfl_xor(n_esc, d, 64);
      if (hl == 0) a.tile_cnt[stream * tiles_per_stream + t0 / kTileSyms] = n_esc;
    }
  };

  // One slot table, or one per bit depth: that of a depth the stream does not use is all zero.  The index in the
  // place of the rings.
  constexpr int kThreads = W * 64;
  static_assert(sizeof(ring[0]) >= sizeof(SlotIndex), "room for the index");
  SlotIndex *const index = reinterpret_cast<SlotIndex *>(&ring[0][0][0]);
  const int n_tables = ADAPT ? a.n_tables : 1;
  bool ok = true, wide = false;  // uniform; wide: a table of one symbol
  for (int t = 0; t < n_tables; ++t) {
    uint32_t f[4], cum;
    const uint32_t total = load_freq4(a.freq + (stream * n_tables + t) * 256, lane, f, &cum);
    ok = ok && (total == kScale || (ADAPT && total == 0));
    wide = wide || __ballot((f[0] | f[1] | f[2] | f[3]) & kScale) != 0;
    if (total == kScale && wave == 0) {
      build_slot_index(index, f, cum, lane);
      if constexpr (ADAPT) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          // (a symbol that does not occur is never looked up)
          lut[t * kCompactTable + lane * 4 + r] = (f[r] & 0xfffu) | (cum << 16);
          cum += f[r];
        }
      }
    }
    __syncthreads();
    if (total == kScale) {
      for_each_slot<kThreads>(index, [&](uint32_t o, uint32_t row) {
        if constexpr (ADAPT) {
          reinterpret_cast<uint8_t *>(lut + t * kCompactTable + 256)[o] = (uint8_t)(row >> 24);
        } else {
          lut[o] = (row >> 24) | (((row + 1u) & 0xfffu) << 8) | ((o - ((row >> 12) & 0xfffu)) << 20);
        }
      });
    } else {
      constexpr uint32_t kWords = ADAPT ? kCompactTable : kScale;
      for (uint32_t o = threadIdx.x; o < kWords; o += kThreads) lut[t * kWords + o] = 0u;
    }
    __syncthreads();  // before the index serves the next table, or the rings take its place
  }
  if (!ok) {  // not a table: nothing can be decoded
    fail();
    return;
  }

  // ---- the half's unit; one whose list is none is empty.  An upper half behind the last unit shadows the lower, so that
  // the steps need no mask, and keeps what it decodes to itself.
  const bool shadow = half && !live && chunk - 1 < n_units;
  const int64_t my_chunk = live ? chunk : shadow ? chunk - 1 : 0;
  const int64_t unit = PIECES ? stream : stream * a.units_per_stream + my_chunk;
  const uint64_t off = a.word_off[unit];
  const uint32_t n = a.n_words_in[unit];
  Piece piece;
  bool list_ok = !(off > a.words_len || (uint64_t)n > a.words_len - off);
  if (PIECES) list_ok = load_piece(a, stream, (int32_t)my_chunk, n, &piece) && list_ok;
  if (!list_ok) fail();
  const bool runs = (live || shadow) && list_ok;
  const int64_t begin = PIECES ? (int64_t)piece.begin : my_chunk * a.unit_syms;
  const int64_t rest = a.syms_per_stream - begin;
  const uint32_t len = !runs ? 0u : PIECES ? piece.len : (uint32_t)(rest < a.unit_syms ? rest : a.unit_syms);
  uint8_t *ubase = a.sym_out + stream * a.syms_per_stream + begin;
  const bool out_aligned = (reinterpret_cast<uintptr_t>(ubase) & 15u) == 0;

  // ---- word list geometry, relative to a 512-byte-aligned address at or below the unit's first word
  const uint16_t *first_word = a.words_in + (list_ok ? off : 0);
  const int32_t lo = (int32_t)((reinterpret_cast<uintptr_t>(first_word) & (uintptr_t)(kPairBlock * 2 - 1)) >> 1);
  const uint16_t *aligned_base = first_word - lo;  // pointer arithmetic keeps the loads global, not flat
  const int32_t hi = lo + (runs ? (int32_t)(PIECES ? piece.words : n) : 0);
  const int32_t stop = lo + (PIECES && runs ? (int32_t)piece.words_left : 0);  // where the pointer has to arrive
  uint16_t *const myring = ring[wave][half];

  // one 16-byte piece (eight words) of block blk per lane, if the piece holds a word of this unit
  auto block_load = [&](int32_t blk, uint4 &v) -> bool {
    const int32_t first = blk * kPairBlock + hl * 8;
    const bool take = blk >= 0 && hi > lo && first + 8 > lo && first < hi;
    if (take) v = *reinterpret_cast<const uint4 *>(aligned_base + first);
    return take;
  };
  auto block_store = [&](int32_t blk, bool take, const uint4 &v) {
    if (take) {
      *reinterpret_cast<uint4 *>(myring + kPairBlock + (blk & 1) * kPairBlock + hl * 8) = v;
      if (blk & 1) *reinterpret_cast<uint4 *>(myring + hl * 8) = v;
    }
  };

  int32_t ptr = hi;
  // A batch takes its words from the pointer's block, `top`, and the one below.  The one below that is on its way, in
  // registers until the pointer has left the block whose place it takes.
  static_assert(kPairBlock == 256, "blocks by shifts");
  int32_t top = (hi - 1) >> 8;
  uint4 coming;
  bool coming_take;
  {
    uint4 v0, v1;
    const bool t0 = block_load(top, v0), t1 = block_load(top - 1, v1);
    coming_take = block_load(top - 2, coming);
    block_store(top, t0, v0);
    block_store(top - 1, t1, v1);
  }
  uint32_t x = runs ? (PIECES ? piece.states : a.states_in + unit * kLanes)[hl] : kLow;
  bool bad = false;

  // Batches whose eight groups are whole in both halves run without a mask.
  const int32_t G = (int32_t)((len + kLanes - 1) / kLanes), whole = wide ? 0 : (int32_t)(len / kLanes);
  const int32_t G0 = __builtin_amdgcn_readlane(G, 0), G1 = __builtin_amdgcn_readlane(G, 32);
  const int32_t whole0 = __builtin_amdgcn_readlane(whole, 0), whole1 = __builtin_amdgcn_readlane(whole, 32);
  const int32_t n_groups = G0 > G1 ? G0 : G1, n_whole = whole0 < whole1 ? whole0 : whole1;
  uint8_t *const my_stage = sym_stage[wave][half];
  const uint16_t *const rings = &ring[0][0][0];
  const uint32_t my_place = (uint32_t)((wave * 2 + half) * (kPairBlock + kPairRing) + kPairBlock - hl - kLanes * (kPairSteps - 1));

  // ADAPT: table offsets of the next two batches' groups, from the depths that the first lanes of a half ask for two
  // batches ahead (and look at only then)
  constexpr int kAhead = 2 * kPairSteps;
  bool bad_depth = false;
  const uint32_t spp = ADAPT ? (uint32_t)a.syms_per_pos : 1u;
  const uint8_t *const depth_row =
      ADAPT ? a.bits + (int64_t)((uint32_t)stream / (uint32_t)a.streams_per_session) * ((uint32_t)a.syms_per_stream / spp)
            : nullptr;
  auto fetch_depth = [&](int32_t g0) -> uint32_t {
    const int32_t g = g0 + hl;
    if (!ADAPT || hl >= kAhead || g >= G) return 1u;
    return depth_row[((uint32_t)begin + (uint32_t)g * kLanes) / spp];
  };
  auto put_tables = [&](int buf, uint32_t depth) {
    const bool known = depth >= 1u && depth <= (uint32_t)a.n_tables;
    bad_depth = bad_depth || !known;
    if (hl < kAhead) table_of_group[wave][buf][half][hl] = (uint16_t)(known ? (depth - 1u) * kCompactTable : 0u);
  };
  if (ADAPT) put_tables(0, fetch_depth(0));
  wave_sync();
  int gbuf = 0;

  // Escapes of each tile: a unit's symbols leave 512 at a time, each 512 of one tile.
  uint32_t *const tile_cnt = a.tile_cnt + stream * tiles_per_stream + begin / kTileSyms;  // (if a.tile_cnt)
  uint32_t esc_mine = 0;  // this lane's, of the tile so far

  for (int32_t g0 = 0; g0 < n_groups; g0 += 2 * kPairSteps) {
    const uint32_t depth_ahead = fetch_depth(g0 + 2 * kPairSteps);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int32_t gb = g0 + b * kPairSteps;
      uint32_t tables[kPairSteps];
      if constexpr (ADAPT) {
        const uint4 tv = *reinterpret_cast<const uint4 *>(&table_of_group[wave][gbuf][half][b * kPairSteps]);
        const uint32_t t4[4] = {tv.x, tv.y, tv.z, tv.w};
#pragma unroll
        for (int j = 0; j < kPairSteps; ++j) tables[j] = (t4[j / 2] >> (16 * (j & 1))) & 0xffffu;
      }
      const uint32_t at0 = my_place + ((uint32_t)(ptr - 1) & (kPairRing - 1));
      uint32_t at = at0;
      uint8_t *const sb = my_stage + b * kPairBlock + hl;
      if (gb + kPairSteps <= n_whole) {  // uniform
#pragma unroll
        for (int j = 0; j < kPairSteps; ++j)
          dec_pair_step<ADAPT, false>(x, lut, ADAPT ? tables[j] : 0u, at, rings, kPairSteps - 1 - j, sb + kLanes * j, 0);
      } else {
#pragma unroll
        for (int j = 0; j < kPairSteps; ++j) {
          const uint64_t on = __ballot((uint32_t)(gb + j) * kLanes + (uint32_t)hl < len);
          dec_pair_step<ADAPT, true>(x, lut, ADAPT ? tables[j] : 0u, at, rings, kPairSteps - 1 - j, sb + kLanes * j, on);
        }
      }
      ptr -= kPairBlock - (int32_t)(at - at0);
      if (ptr < lo) {  // ran out of words: the stream is damaged
        bad = true;
        ptr = lo;
      }
      if ((ptr - 1) >> 8 != top) {  // (a batch takes a block's words at the most)
        --top;
        block_store(top - 1, coming_take, coming);
        coming_take = block_load(top - 2, coming);
      }
      wave_sync();
    }
    if (ADAPT) {
      put_tables(gbuf ^ 1, depth_ahead);
      gbuf ^= 1;
    }
    // the symbols of both batches
    const uint32_t done = (uint32_t)g0 * kLanes, mine = (uint32_t)hl * 16;
    const uint32_t left = live && len > done ? len - done : 0u;
    if (out_aligned && mine + 16 <= left) {
      const uint4 v = *reinterpret_cast<const uint4 *>(&my_stage[mine]);
      *reinterpret_cast<uint4 *>(ubase + done + mine) = v;
      if (a.tile_cnt) {  // uniform
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)  // a byte is 0xff iff its low seven bits carry into bit 7 and bit 7 is set
          esc_mine += (uint32_t)__builtin_popcount(((w[i] & 0x7f7f7f7fu) + 0x01010101u) & w[i] & 0x80808080u);
      }
    } else {
      for (uint32_t i = mine; i < mine + 16 && i < left; ++i) {
        ubase[done + i] = my_stage[i];
        esc_mine += my_stage[i] == PLC_ESCAPE;
      }
    }
    // the tile is through, or the units are (uniform)
    if (a.tile_cnt && ((done + kPairDrain) % kTileSyms == 0 || g0 + 2 * kPairSteps >= n_groups)) {
      uint32_t sum = esc_mine;
      esc_mine = 0;
#pragma unroll
      for (int d = 1; d < kLanes; d <<= 1) sum += __shfl_xor(sum, d, 64);
      if (hl == 0 && live && done / kTileSyms * kTileSyms < len) tile_cnt[done / kTileSyms] = sum;
    }
    wave_sync();
  }
  // integrity: every word consumed, every lane back at the initial state (a piece: at what the record behind it says)
  if (runs) {
    const uint32_t x_end = PIECES && piece.end_states ? piece.end_states[hl] : kLow;
    if (ptr != stop || x != x_end) bad = true;
  }
  const uint64_t bads = __ballot(bad);
  if (runs && live) {
    const bool good = (uint32_t)(half ? bads >> 32 : bads) == 0;
    if (PIECES) {
      if (hl < 2) report_piece(a, stream, (int32_t)chunk, hl, good);
    } else if (!good && hl == 0) {
      raise(a.status, PLC_ERR_CORRUPT);
    }
  }
  if (bad_depth) raise(a.status, PLC_ERR_INVALID);
}

// ---------------------------------------------------------------------------
// Reconstruction inside the decoder for units coded as whole streams
// ---------------------------------------------------------------------------
// A further wavefront of the unit's workgroup that turns each batch of decoded symbols into KV components
// while the next batches are decoded: out = prediction over RK candidates + symbol * step (the arithmetic
// of plc_reconstruct; COND: of plc_reconstruct_cond; ADAPT: of plc_reconstruct_adapt).  A batch is 512 symbols = 64 chunks of 8 components,
// one chunk per lane.  The candidates and weights of a chunk do not depend on its symbols, so they are
// requested kRecDepth batches ahead (a template parameter) and are in registers when the symbols arrive.  The wavefront meets the
// decoder at every batch barrier -- one "start" barrier, then one per batch, in step with the other
// wavefronts of the workgroup -- through the bare instruction, which unlike __syncthreads does not first
// wait for its outstanding loads.  Loads are issued by every lane in every batch (past the end of the stream
// a lane stays on its last chunk and stores nothing), so that the number of loads behind any given one is the
// same on every path and the wait before a use leaves the later requests in flight (the few loads and
// stores that escapes add are issued only where there are escapes and cost at most their own number in
// that count).
//   stream, piece, G the unit's stream, the part of it that the unit is (all of it, but for pieces), its groups of 32
//   sym_stage        the two symbol stages: batch b is in stage b mod 2 from its barrier to the next (kLate = 1:
//                    from the barrier after its own, where the symbols pass through another wavefront first)
//   table_barriers   barriers of the wavefronts that build the tables meanwhile, in front of "start"
constexpr int kRecDepthBase = 3;  // batches a request runs ahead of its symbols

template <int RK, bool COND, bool ADAPT, int kRecDepth, int kLate = 0, int kStageSyms = 2 * kBatchSyms>
__device__ __forceinline__ void reconstruct_batches(const RansArgs &a, int64_t stream, const Piece &piece, int32_t G,
                                                    const uint8_t (&sym_stage)[2][kStageSyms], int lane,
                                                    int table_barriers) {
  static_assert(COND || !ADAPT, "the adaptive quantiser lives on the token-conditional path");
  const ReconView &r = a.recon;
  const uint32_t lh = (uint32_t)(r.L * r.H);
  const uint32_t s = (uint32_t)stream / lh, rem = (uint32_t)stream - s * lh;
  const uint32_t l = rem / (uint32_t)r.H, h = rem - l * (uint32_t)r.H;
  const int64_t cand0 = s * r.cs[0] + l * r.cs[1] + h * r.cs[2];
  const int64_t out0 = s * r.as[0] + l * r.as[1] + h * r.as[2];
  const float *w0 = r.weights + (int64_t)s * r.n * r.k;
  const bool pieces = !ADAPT && a.pieces > 0;  // uniform
  const uint32_t chunk0 = piece.begin / kChunk, n_chunks = piece.len / kChunk;
  const uint32_t d8 = (uint32_t)r.d8, adv_row = 64u / d8, adv_e8 = 64u - adv_row * d8;
  // The chunk this lane requests next: row = position * 2 + (0 = K, 1 = V), e8 = chunk inside the row,
  // and where its candidates, weights and output are.  From batch to batch a lane moves on by 64
  // chunks; where that is a whole, even number of rows (d = 8, 16, ... 256) it is the same position
  // step in the same half every time, and the three pointers advance by constants.
  uint32_t at_chunk = (uint32_t)lane, row = (chunk0 + (uint32_t)lane) / d8, e8 = chunk0 + (uint32_t)lane - row * d8;
  const bool steady = adv_e8 == 0u && (adv_row & 1u) == 0u;
  const int64_t cand_step = (int64_t)(adv_row / 2u) * r.cs[3], out_step = (int64_t)(adv_row / 2u) * r.as[3];
  const uint32_t w_step = (adv_row / 2u) * (uint32_t)RK;
  const uint16_t *cand_p;
  const float *w_p;
  uint16_t *out_p;
  auto point = [&](uint32_t rr, uint32_t ee) {
    const uint32_t i = rr >> 1;
    cand_p = ((rr & 1u) ? r.cand_v : r.cand_k) + cand0 + (int64_t)i * r.cs[3] + ee * kChunk;
    w_p = w0 + (int64_t)i * RK;
    out_p = ((rr & 1u) ? r.out_v : r.out_k) + out0 + (int64_t)i * r.as[3] + ee * kChunk;
  };
  if (at_chunk < n_chunks) {
    point(row, e8);
  } else {
    row = chunk0 / d8, e8 = chunk0 - row * d8;
    point(row, e8);
  }
  // COND: the position names its true candidate (plc_reconstruct_cond), whose vector then is the
  // prediction; which candidate to request is itself a load, so it runs one round further ahead: a
  // second cursor walks the chunks 2 * kRecDepth batches in front and fetches their chosen index.
  // ADAPT: the position's bit depth, which sets its step, is fetched with the chosen index.
  uint32_t far_chunk = at_chunk, far_row = row, far_e8 = e8;
  int64_t far_pos = (int64_t)s * r.n + (row >> 1);  // entry in chosen and bits
  int32_t pick_next[kRecDepth];  // chosen index of the chunk the stage requests next
  int32_t pick_used[kRecDepth];  // and of the chunk whose candidates it holds (-1: the weighted mean)
  bool mean_path[kRecDepth];     // uniform: some lane of the stage's request needed all candidates
  uint32_t depth_next[kRecDepth], depth_used[kRecDepth];  // bit depths, the same way
  uint4 cv[kRecDepth][RK];
  float wv[kRecDepth][RK];
  typedef __attribute__((address_space(1))) u32x4 *global_u32x4;  // named global: kept through the loop
  global_u32x4 dst[kRecDepth];
  bool live[kRecDepth];  // whether the lane's chunk exists (a flag of its own: the pointer stays a global one)
  // Escapes.  This wavefront sees every chunk of the stream in order, so the number of escapes in front
  // of a chunk is a running count plus a prefix over the lanes.  A chunk with escapes is not stored when
  // its symbols arrive: its raw values are requested from the stream's list, the chunk is held, and the
  // next time the same registers come round, kRecDepth batches later, the values that have arrived are
  // put over its escaped components and the chunk is stored, once and whole.  The registers hold up to
  // kEscLate raw values per chunk; a batch in which some chunk has more (3e-5 of the chunks at the synthetic
  // workloads' escape rates) fetches its raw values, waits for them and stores its escaped chunks at once.
  constexpr int kEscLate = 2;
  uint32_t esc_bits[kRecDepth];  // which components of the chunk held for esc_dst await their raw value
  uint32_t esc_raw[kRecDepth][kEscLate];
  u32x4 esc_held[kRecDepth];
  global_u32x4 esc_dst[kRecDepth];
  const uint64_t esc_base = r.esc_off[stream];
  uint32_t esc_seen = piece.esc;  // escapes of the stream so far
  bool esc_bad = false;           // an escape past the end of the lists
#pragma unroll
  for (int j = 0; j < kRecDepth; ++j) esc_bits[j] = 0u, esc_dst[j] = nullptr, esc_held[j] = u32x4{0u, 0u, 0u, 0u};
  // Loads of the lane's next chunk (of its last one again once the stream is at its end, so that every
  // batch issues the same loads), then on to the chunk after it.
  auto load_weights = [&](float(&w)[RK]) {
    if constexpr (RK % 4 == 0) {
#pragma unroll
      for (int j = 0; j < RK; j += 4) {
        const float4 t = *reinterpret_cast<const float4 *>(w_p + j);
        w[j] = t.x, w[j + 1] = t.y, w[j + 2] = t.z, w[j + 3] = t.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < RK; ++j) w[j] = w_p[j];
    }
  };
  auto fetch_pick = [&](int32_t &pick, uint32_t &depth) {  // COND: the far cursor's position, then one batch on
    pick = r.chosen[far_pos];
    if constexpr (ADAPT) depth = r.bits[far_pos];
    far_chunk += 64u;
    if (steady) {  // uniform
      if (far_chunk < n_chunks) far_pos += adv_row / 2u;
    } else {
      far_row += adv_row;
      far_e8 += adv_e8;
      if (far_e8 >= d8) {
        far_e8 -= d8;
        ++far_row;
      }
      if (far_chunk < n_chunks) far_pos = (int64_t)s * r.n + (far_row >> 1);
    }
  };
  auto request = [&](uint4(&c)[RK], float(&w)[RK], global_u32x4 &out, bool &ok, int32_t &pick_nx,
                     int32_t &pick_us, bool &mean, uint32_t &depth_nx, uint32_t &depth_us) {
    if constexpr (COND) {
      int32_t pick = pick_nx;
      if (pick < -1 || pick >= RK) {
        raise(a.status, PLC_ERR_INVALID);
        pick = -1;
      }
      if constexpr (ADAPT) {
        uint32_t b = depth_nx;
        if (b < 1u || b > (uint32_t)PLC_MAX_BITS) {
          raise(a.status, PLC_ERR_INVALID);
          b = 1u;
        }
        depth_us = b;
      }
      mean = __ballot(pick < 0) != 0;  // uniform
      if (!mean) {
        c[0] = load16_stream(cand_p + pick * r.cs[4]);
      } else {  // a lane that has its candidate takes it RK times: every lane issues the same loads
#pragma unroll
        for (int j = 0; j < RK; ++j) c[j] = load16_stream(cand_p + (pick >= 0 ? pick : j) * r.cs[4]);
        load_weights(w);
      }
      pick_us = pick;
      fetch_pick(pick_nx, depth_nx);
    } else {
#pragma unroll
      for (int j = 0; j < RK; ++j) c[j] = load16_stream(cand_p + j * r.cs[4]);
      load_weights(w);
    }
    out = (global_u32x4)out_p;
    ok = at_chunk < n_chunks;
    at_chunk += 64u;
    if (steady) {  // uniform
      if (at_chunk < n_chunks) cand_p += cand_step, w_p += w_step, out_p += out_step;
    } else {
      row += adv_row;
      e8 += adv_e8;
      if (e8 >= d8) {
        e8 -= d8;
        ++row;
      }
      if (at_chunk < n_chunks) point(row, e8);
    }
  };
  // the raw values that have arrived for the chunk held for `out`: over its escaped components, lowest
  // first (component e is half e & 1 of word e >> 1), then the chunk goes out
  // one raw value over the lowest component still marked in `bits`
  auto put_raw = [](u32x4 &chunk, uint32_t &bits, uint32_t raw) {
    const uint32_t e = (uint32_t)__builtin_ctz(bits);
    bits &= bits - 1u;
    const uint32_t shift = (e & 1u) * 16u, keep = ~(0xffffu << shift), value = (raw & 0xffffu) << shift;
#pragma unroll
    for (uint32_t word = 0; word < 4; ++word)
      chunk[word] = (e >> 1) == word ? (chunk[word] & keep) | value : chunk[word];
  };
  auto patch = [&](global_u32x4 out, uint32_t &bits, const uint32_t (&raw)[kEscLate], u32x4 &held) {
    if (__ballot(bits != 0u) == 0) return;  // uniform
    const bool pending = bits != 0u;
#pragma unroll
    for (int i = 0; i < kEscLate; ++i) {
      if (i > 0 && __ballot(bits != 0u) == 0) break;  // uniform; seldom more than one per chunk
      if (bits) put_raw(held, bits, raw[i]);
    }
    if (pending) __builtin_nontemporal_store(held, out);
  };
  if constexpr (COND) {
#pragma unroll
    for (int j = 0; j < kRecDepth; ++j) fetch_pick(pick_next[j], depth_next[j]);
  }
#pragma unroll
  for (int j = 0; j < kRecDepth; ++j)
    request(cv[j], wv[j], dst[j], live[j], pick_next[j], pick_used[j], mean_path[j], depth_next[j], depth_used[j]);
  asm volatile("" ::: "memory");
  for (int i = 0; i < table_barriers; ++i) __builtin_amdgcn_s_barrier();  // (uniform)
  __builtin_amdgcn_s_barrier();  // barrier "start"
  asm volatile("" ::: "memory");
  if constexpr (kLate > 0) {  // the first batch's own barrier: its symbols come one barrier later
    static_assert(kLate == 1, "one barrier behind");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
  const int32_t n_batches = (G + kBatch - 1) / kBatch;
  const int32_t n_full = (int32_t)(n_chunks / 64u);  // batches all of whose chunks exist
  // One batch: join its barrier, take its symbols from the stage, finish the chunk, request the chunk
  // of the batch kRecDepth later into the registers just freed.
  auto turn = [&](uint4(&c)[RK], float(&w)[RK], global_u32x4 &out, bool &ok, uint32_t &bits,
                  uint32_t(&raw)[kEscLate], u32x4 &held, global_u32x4 &late, int32_t &pick_nx, int32_t &pick_us, bool &mean,
                  uint32_t &depth_nx, uint32_t &depth_us, int32_t b, bool whole) {
    // (the scheduler would otherwise start on the predictions of all kRecDepth batches at the top of a
    // pass, and so wait there for requests that have only just gone out)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();  // barrier of batch b (kLate: the one after): its symbols are in the stage
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    const uint2 sv = *reinterpret_cast<const uint2 *>(&sym_stage[b & 1][lane * kChunk]);
    patch(late, bits, raw, held);
    float pred[kChunk];
    if (!COND || mean) {  // uniform
#pragma unroll
      for (int e = 0; e < kChunk; ++e) pred[e] = 0.0f;
#pragma unroll
      for (int j = 0; j < RK; ++j) accumulate8(w[j], c[j], pred);
    }
    if constexpr (COND) {
      const half8 own = __builtin_bit_cast(half8, c[0]);
#pragma unroll
      for (int e = 0; e < kChunk; ++e) pred[e] = (!mean || pick_us >= 0) ? (float)own[e] : pred[e];
    }
    uint32_t unused = 0;
    const float step = ADAPT ? __builtin_ldexpf(r.range, -(int)depth_us) : r.delta;
    const half8 v = add_back8(sv, step, pred, &unused);
    const bool mine = whole || ok;
    // a byte is 0xff iff its low seven bits carry into bit 7 when 1 is added and bit 7 is set
    const uint32_t hx = ((sv.x & 0x7f7f7f7fu) + 0x01010101u) & sv.x & 0x80808080u;
    const uint32_t hy = ((sv.y & 0x7f7f7f7fu) + 0x01010101u) & sv.y & 0x80808080u;
    const bool has = mine && (hx | hy) != 0u;
    if (mine && !has) __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), out);
    const uint64_t lanes = __ballot(has);
    if (lanes != 0) {  // uniform
      // bit 7 of byte e to bit e
      const uint32_t mx = ((hx >> 7) * 0x00204081u) >> 21 & 0xfu, my = ((hy >> 7) * 0x00204081u) >> 21 & 0xfu;
      bits = has ? (mx | (my << 4)) : 0u;
      const uint32_t n_esc = (uint32_t)__builtin_popcount(bits);
      const bool several = __ballot(n_esc > 1u) != 0;  // uniform; seldom
      uint32_t total, before;
      if (!several) {
        before = __builtin_amdgcn_mbcnt_hi((uint32_t)(lanes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)lanes, 0u));
        total = (uint32_t)__builtin_popcountll(lanes);
      } else {
        before = wave_escape_prefix(n_esc, &total);
      }
      const uint64_t src = esc_base + esc_seen + before;
      esc_seen += total;
      if (several && __ballot(n_esc > (uint32_t)kEscLate) != 0) {  // uniform; rare: fetch, wait, store now
        u32x4 now = __builtin_bit_cast(u32x4, v);
#pragma unroll
        for (int i = 0; i < kChunk; ++i) {
          if (__ballot(bits != 0u) == 0) break;  // uniform
          if (bits) {
            uint32_t value = 0u;
            if (src + i < r.esc_len) {
              value = r.esc_in[src + i];
            } else {
              esc_bad = true;
            }
            put_raw(now, bits, value);
          }
        }
        if (has) __builtin_nontemporal_store(now, out);  // bits is 0 again: nothing is held
      } else {
        held = __builtin_bit_cast(u32x4, v);
        late = out;
#pragma unroll
        for (int i = 0; i < kEscLate; ++i) {
          if (i > 0 && (!several || __ballot(n_esc > (uint32_t)i) == 0)) break;  // uniform
          if (n_esc > (uint32_t)i) {
            if (src + i < r.esc_len) {
              raw[i] = r.esc_in[src + i];
            } else {
              esc_bad = true;
              raw[i] = 0u;
            }
          }
        }
      }
    }
    request(c, w, out, ok, pick_nx, pick_us, mean, depth_nx, depth_us);
  };
  // Whole batches, kRecDepth at a time and free of branches: every pass issues the same loads and
  // stores in the same order.
  int32_t b0 = 0;
  for (; b0 + kRecDepth <= n_full; b0 += kRecDepth) {
#pragma unroll
    for (int j = 0; j < kRecDepth; ++j)
      turn(cv[j], wv[j], dst[j], live[j], esc_bits[j], esc_raw[j], esc_held[j], esc_dst[j], pick_next[j], pick_used[j],
           mean_path[j], depth_next[j], depth_used[j], b0 + j, true);
  }
  // What is left: fewer than kRecDepth whole batches and possibly a partial one.
#pragma unroll
  for (int j = 0; j < kRecDepth; ++j)
    if (b0 + j < n_batches)  // uniform
      turn(cv[j], wv[j], dst[j], live[j], esc_bits[j], esc_raw[j], esc_held[j], esc_dst[j], pick_next[j], pick_used[j],
           mean_path[j], depth_next[j], depth_used[j], b0 + j, false);
#pragma unroll
  for (int j = 0; j < kRecDepth; ++j) patch(esc_dst[j], esc_bits[j], esc_raw[j], esc_held[j]);
  if (pieces) {
    const bool good = __ballot(esc_bad) == 0 && esc_seen == piece.esc_end;
    if (lane == 0) report_piece(a, stream, (int32_t)(blockIdx.x - (uint32_t)stream * a.wgs_per_stream), 1, good);
  } else if (esc_bad) {
    raise(a.status, PLC_ERR_CORRUPT);
  }
}

// ---------------------------------------------------------------------------
// Decoder for streams coded as one unit (one wavefront per workgroup)
// ---------------------------------------------------------------------------
// With one unit per stream there are only as many wavefronts as streams, so what counts is the length of a
// step: one LDS round trip (61-67 cycles for 8 bytes) and the instructions, 4.64 cycles each, between the arrival
// of an entry and the read of the next.  In the kernel above that chain holds two round trips -- slot
// table, then, for the lanes that renormalise, the word -- and some ten instructions.  Here the round trips are
// folded into one and the instructions cut to six.
//
// Every entry, of the slot table and of the word ring alike, is 8 bytes
//     .x = f | sym << 24        .y = y | t << 16   with  y = f * w4 + slot - cum,  t = floor((2^16 - 1 - y) / f)
// A ring entry stands for a word w = w4 << 12 | slot: it is the slot-table entry that the state will
// select once the word has been shifted in (the state's low 12 bits are then the word's, which is all
// they are needed for), with the word's top four bits w4 already multiplied in; in the slot table itself
// w4 = 0.  A lane that renormalises reads its ring entry, a lane that does not reads the slot table at
// its new state -- one read either way, at an address chosen per lane, both tables living in one LDS
// array; the ring entries are formed when a block of words is staged, off the chain: .y + w4 * (f - 2^16), for
// y grows by f * w4 (to at most 4096 * 15 + 4095 < 2^16) and t falls by w4 (from at least 15).  The
// state is carried as xc = x >> 12 without the bits the word supplies, so that
// f * (x >> 12) + slot - cum = f * (xc + w4) + slot - cum = f * xc + y: one multiply-add, whose 24-bit
// multiplicand ignores the symbol in the top byte of .x.  Whether the lane renormalises, f * xc + y < 2^16, is
// xc <= t and does not wait for it: the compare comes first, and the multiply-add and the mask of the slot stand
// in the two wait states between it and the rank that reads its lanes.  The multiply-add leaves t in the upper
// half of its result; the slot and a renormalising lane's next state do not look there, the other lanes' has it
// taken off behind the read.
// The ring holds RB blocks of 512 words.  Four let the helper leave its newest block on its way for a batch
// (below); three are what the decoder strictly needs -- the block of the pointer, the one below it, and the
// one being staged for the batch after -- and bring the workgroup's LDS from 57.6 to 53.5 KB, so that a
// compute unit holds three workgroups instead of two where the registers allow it (k <= 6).  That is the
// variant for thousands of streams, where units in flight count for more than the helper's wait: 9.1 -> 7.9 ms
// on 5120 streams with k = 4.  (With k = 8 and 16,384 streams the kernel is bound by HBM at 5.4 TB/s whatever
// the workgroups per compute unit or the depth of the reconstruction's requests: two, three or four batches
// ahead, two or three workgroups, all within 0.1 % of one another.)

template <bool MASKED>
__device__ __forceinline__ void dec_chain_step(uint32_t &xc, uint2 &e, const uint2 *tab, uint32_t &ring_at,
                                               uint8_t *sym_slot, bool on) {
  // which lanes renormalise; ranks and choices are made from this one mask
  uint64_t mask = __builtin_amdgcn_uicmp(e.y >> 16, xc, 35 /* unsigned >= */);
  if (MASKED) mask &= __builtin_amdgcn_ballot_w64(on);
  const uint32_t m32 = (uint32_t)mask;
  const bool need = __builtin_amdgcn_inverse_ballot_w64(mask);
  PLC_PIN();
  const uint32_t xn = __umul24(e.x, xc) + e.y;  // f * (x >> 12) + slot - cum, plus t << 16
  PLC_PIN();
  uint32_t idx_slot = xn & (kScale - 1);
  asm volatile("" : "+v"(idx_slot));  // in a register: the choice below is one select, not a branch
  PLC_PIN();
  // ring entry of the rank-th word from the top (lane 0 is served first: the rank is the number of
  // renormalising lanes below this one), or slot-table entry of xn
  const uint32_t idx_ring = __builtin_amdgcn_mbcnt_lo(m32, ring_at);
  PLC_PIN();
  const uint2 en = tab[need ? idx_ring : idx_slot];
  PLC_PIN();  // what follows is issued in the shadow of the read
  // (the entry of the top word, uniform, kept in a vector register where the rank is added to it: one instruction)
  asm volatile("v_bcnt_u32_b32 %0, %1, %0" : "+v"(ring_at) : "s"(m32));
  uint32_t shifted = (xn & 0xffffu) << 4, kept = (xn - (e.y & 0xffff0000u)) >> kScaleBits;
  asm volatile("" : "+v"(shifted), "+v"(kept));  // (as above)
  PLC_PIN();
  if (!MASKED || on) *sym_slot = (uint8_t)(e.x >> 24);
  PLC_PIN();
  const uint32_t next = need ? shifted : kept;
  if (!MASKED || on) {
    xc = next;
    e = en;
  }
  PLC_PIN();
}

// Two wavefronts per unit.  What a step does not need stays off the decoding wavefront: a helper, on
// another SIMD of the compute unit, stages the words (forming the ring entries costs eight table lookups
// and up to sixteen LDS writes per lane and block) and moves the decoded symbols to global memory.  The
// two meet at one workgroup barrier per batch of 16 steps:
//   decoder  batch b: 16 steps into symbol stage b % 2; publishes the word pointer; barrier b
//   helper   while batch b runs: stages every block down to 1024 words below the pointer published at
//            barrier b - 1 (a batch consumes at most 512, so batch b + 1 finds its words); barrier b;
//            then moves the symbols of batch b out while batch b + 1 runs.
// The blocks the helper writes lie at least one block below those the running batch reads, and the ring
// slots they take belonged to blocks above the pointer (four blocks of ring: the pointer's block and the
// three below it).
//
// RK > 0 adds a third wavefront that reconstructs the KV components of each batch while the next batches are
// decoded (reconstruct_batches above).
template <int RK, bool COND, int RB = 4>
__global__ __launch_bounds__(RK ? 192 : 128) void rans_decode_chain_kernel(const RansArgs a) {
  static_assert(RB == 3 || RB == 4, "ring blocks");
  constexpr uint32_t kRing = RB * kBlockWords;  // words the ring holds: word i sits at kRing - 1 - i mod kRing
  __shared__ __attribute__((aligned(16))) uint2 tab[kScale + kRing + kRingMirror];  // slot table, then the ring
  __shared__ __attribute__((aligned(16))) uint8_t sym_stage[2][2 * kBatchSyms];  // second half: lanes 32..63
  __shared__ int32_t ptr_pub[2];  // the word pointer after batch b, in slot b mod 2
  static_assert(workgroups_per_cu(sizeof(tab) + sizeof(sym_stage) + sizeof(ptr_pub)) >=
                    (RB == 3 ? 3 : 2),
                "what the ring of three blocks is for, and the other holds");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const bool helper = wave == 1;
  const int64_t stream = blockIdx.x / a.wgs_per_stream;
  const int64_t chunk = blockIdx.x - stream * a.wgs_per_stream;
  const bool pieces = a.pieces > 0;  // uniform: the unit is a piece of the stream
  bool bad = false;
  if (a.verified_pieces && stream_verified(a, stream)) return;  // uniform: nothing to decode again
  // (uniform: every wavefront leaves, before any barrier that another might wait at)
  auto give_up = [&]() {
    if (threadIdx.x != 0) return;
    if (pieces) {
      report_piece(a, stream, (int32_t)chunk, 0, false);
    } else {
      raise(a.status, PLC_ERR_CORRUPT);
    }
  };

  uint2 *ring = tab + kScale;

  // Everything that the start needs from global memory is asked for before the table is built, which takes as long as
  // the answers: the first words by the helper, the candidates of the first batches by the wavefront that
  // reconstructs, which has no part in the table.

  // ---- the unit: the stream, or a piece of it
  uint32_t f[4], cum;
  const uint32_t total = load_freq4(a.freq + stream * 256, lane, f, &cum);
  const uint64_t off = a.word_off[stream];
  const uint32_t n = a.n_words_in[stream];
  Piece piece = {0u, (uint32_t)a.syms_per_stream, n, 0u, 0u, 0u, a.states_in + stream * kLanes, nullptr};
  if (total != kScale || off > a.words_len || (uint64_t)n > a.words_len - off ||
      (pieces && !load_piece(a, stream, (int32_t)chunk, n, &piece))) {  // (not a table: nothing can be decoded)
    give_up();
    return;
  }
  const uint32_t begin = piece.begin, len = piece.len;
  uint8_t *ubase = a.sym_out + stream * a.syms_per_stream + begin;
  const bool out_aligned = (reinterpret_cast<uintptr_t>(ubase) & 15u) == 0;
  const int32_t G = (int32_t)((len + kLanes - 1) / kLanes);
  const uint32_t top_syms = len - (uint32_t)(G - 1) * kLanes;

  // ---- word list geometry, relative to a 1 KiB-aligned address at or below the unit's first word
  const uint16_t *first_word = a.words_in + off;
  const int32_t lo = (int32_t)((reinterpret_cast<uintptr_t>(first_word) & (uintptr_t)(kBlockWords * 2 - 1)) >> 1);
  const uint16_t *aligned_base = first_word - lo;  // pointer arithmetic keeps the loads global, not flat
  const int32_t hi = lo + (int32_t)piece.words;

  int32_t tail_groups = G % kBatch;
  if (tail_groups == 0 && top_syms < kLanes) tail_groups = kBatch;
  const int32_t g_tail = G - tail_groups;

  if constexpr (RK > 0) {
    if (wave == 2) {
      reconstruct_batches<RK, COND, false, kRecDepthBase>(a, stream, piece, G, sym_stage, lane, 2);
      return;
    }
  }

  // one 16-byte piece (eight words) of block blk per lane, if the piece holds a word of this unit
  auto block_load = [&](int32_t blk, uint4 &v) -> bool {
    const int32_t first = blk * kBlockWords + lane * 8;
    const bool take = blk >= 0 && hi > lo && first + 8 > lo && first < hi;
    if (take) v = *reinterpret_cast<const uint4 *>(aligned_base + first);
    return take;
  };
  // A batch consumes at most one block of words.  While batch b runs, the pointer p_b it started from is
  // known to the helper: the words down to p_b - 3 blocks are requested and those down to p_(b-1) - 3 blocks, at
  // or below p_b - 2 blocks, are in the ring -- batch b + 1 reads no further down than that.
  // With three blocks the words are staged two blocks below the pointer and none is left on its way: the
  // block written while batch b runs then takes the slot of the block three above it, which lies wholly
  // above the pointer batch b started from.
  constexpr int kBelow = (RB == 4 ? 3 : 2) * kBlockWords;
  const int32_t top_block = (hi - 1) >> 9;
  const int32_t first_down = hi - kBelow > 0 ? (hi - kBelow) >> 9 : 0;  // the blocks down to here come first
  uint4 first_v[RB];
  bool first_take[RB];
  if (helper) {
#pragma unroll
    for (int i = 0; i < RB; ++i) first_take[i] = top_block - i >= first_down && block_load(top_block - i, first_v[i]);
  }
  const uint32_t x0 = piece.states[lane & (kLanes - 1)];

  // ---- slot table, its index in the ring's place
  SlotIndex *const index = reinterpret_cast<SlotIndex *>(ring);
  static_assert(sizeof(SlotIndex) <= kRing * sizeof(uint2) && kScale % 2 == 0, "room for the index");
  if (wave == 0) build_slot_index(index, f, cum, lane);
  lds_barrier();
  for_each_slot<128>(index, [&](uint32_t o, uint32_t row) {
    const uint32_t fs = (row & 0xfffu) + 1u, r = o - ((row >> 12) & 0xfffu);
    // floor((2^16 - 1 - r) / f): the quotient in fp32 is off by less than one, and put right by what is left
    uint32_t t = (uint32_t)((float)(0xffffu - r) * __builtin_amdgcn_rcpf((float)fs));
    const int32_t left = (int32_t)(0xffffu - r - t * fs);
    t = left < 0 ? t - 1u : (uint32_t)left >= fs ? t + 1u : t;
    tab[o] = make_uint2(fs | (row & 0xff000000u), r | (t << 16));
  });
  lds_barrier();

  if (helper) {
    // Word i goes to ring position (~i) mod 2048: the slot-table entry of its low 12 bits, its top four
    // bits multiplied in.
    auto block_store = [&](int32_t blk, bool take, const uint4 &v) {
      if (take) {
        // ring position of the piece's last word (blk >= 0 here)
        const uint32_t pos = (RB - 1u - (uint32_t)blk % RB) * kBlockWords + (uint32_t)(kBlockWords - 8 - lane * 8);
        const uint32_t w[8] = {v.x & 0xffffu, v.x >> 16, v.y & 0xffffu, v.y >> 16,
                               v.z & 0xffffu, v.z >> 16, v.w & 0xffffu, v.w >> 16};
        uint2 en[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) en[i] = tab[w[7 - i] & (kScale - 1)];  // en[i] belongs at pos + i
#pragma unroll
        for (int i = 0; i < 8; ++i) {  // f * w4 onto y, w4 off t
          const uint32_t w4 = w[7 - i] >> kScaleBits;
          en[i].y += __umul24(en[i].x, w4) - (w4 << 16);
        }
#pragma unroll
        for (int i = 0; i < 8; i += 2)
          *reinterpret_cast<uint4 *>(&ring[pos + i]) = make_uint4(en[i].x, en[i].y, en[i + 1].x, en[i + 1].y);
        if (pos < (uint32_t)kRingMirror) {
#pragma unroll
          for (int i = 0; i < 8; i += 2)
            *reinterpret_cast<uint4 *>(&ring[kRing + pos + i]) =
                make_uint4(en[i].x, en[i].y, en[i + 1].x, en[i + 1].y);
        }
      }
    };
    // Stages every block that holds a word at or above `down_to` and is not staged yet.  The last of them
    // may be left on its way (`ahead`): its words go to the ring at the next call, a batch later, so that
    // the wavefront does not sit out the load's latency in front of the barrier.
#pragma unroll
    for (int i = 0; i < RB; ++i) block_store(top_block - i, first_take[i], first_v[i]);
    int32_t lowest = top_block + 1 < first_down ? top_block + 1 : first_down;  // lowest block already requested
    uint4 ahead_v;
    int32_t ahead_blk = 0;
    bool ahead = false, ahead_take = false;
    auto stage_down_to = [&](int32_t down_to, bool leave_one) {
      if (ahead) {  // uniform
        block_store(ahead_blk, ahead_take, ahead_v);
        ahead = false;
      }
      const int32_t last = down_to > 0 ? down_to >> 9 : 0;
      while (lowest > last) {  // uniform; one round per batch after the first call
        const int32_t blk = lowest - 1;
        lowest = blk;
        if (leave_one && blk == last) {
          ahead_take = block_load(blk, ahead_v);
          ahead_blk = blk;
          ahead = true;
        } else {
          uint4 v;
          const bool take = block_load(blk, v);
          block_store(blk, take, v);
        }
      }
    };
    lds_barrier();  // barrier "start"
    int32_t ptr_before = hi;  // the pointer as it stood before the batch now running
    for (int32_t g0 = 0; g0 < G; g0 += kBatch) {
      stage_down_to(ptr_before - kBelow, RB == 4);
      lds_barrier();  // barrier of this batch: its symbols are in the stage, the pointer is published
      ptr_before = ptr_pub[(g0 / kBatch) & 1];  // (its own slot: the decoder publishes the next one a batch later)
      const bool tail = g0 >= g_tail;
      const int32_t cnt_groups = tail ? tail_groups : kBatch;
      const uint8_t *stage = sym_stage[(g0 / kBatch) & 1];
      const uint32_t done = (uint32_t)g0 * kLanes;
      const uint32_t room = (uint32_t)cnt_groups * kLanes;
      const uint32_t nsym = (len - done) < room ? (len - done) : room;
      if (out_aligned) {
        const uint32_t full = nsym / 16;
        if ((uint32_t)lane < full)
          *reinterpret_cast<uint4 *>(ubase + done + lane * 16) = *reinterpret_cast<const uint4 *>(&stage[lane * 16]);
        const uint32_t rest_at = full * 16 + (uint32_t)lane;
        if (rest_at < nsym) ubase[done + rest_at] = stage[rest_at];
      } else {
        for (uint32_t i = lane; i < nsym; i += 64) ubase[done + i] = stage[i];
      }
    }
    return;
  }

  // ---- the decoding wavefront
  // Lanes 0..31 decode.  Lanes 32..63 start as their copies and run the same instructions, so that no step
  // needs a lane mask; their ranks count all 32 decoding lanes, so their states go astray -- whatever they
  // read lies inside the tables, and what they store goes to a spare half of the stage.
  const bool coder = lane < kLanes;
  const int rl = lane & (kLanes - 1);
  const bool top_active = (uint32_t)rl < top_syms;
  uint32_t xc = x0 >> kScaleBits;
  uint2 e = tab[x0 & (kScale - 1)];
  int32_t ptr = hi;
  lds_barrier();  // barrier "start": the first words are staged
  // The top word's entry in tab (uniform): in a vector register where the ranks are added to it, and a scalar copy
  // as of the batch's first step.  Everything a batch needs besides its steps is done behind the last step's read.
  uint32_t ring_start = (uint32_t)kScale + kRing - 1u - (uint32_t)(ptr - 1) % kRing;
  uint32_t ring_at = ring_start;
  asm volatile("" : "+v"(ring_at));
  uint8_t *sb = &sym_stage[0][coder ? rl : kBatchSyms + rl];
  auto batch_done = [&](int parity) {
    const uint32_t now = (uint32_t)__builtin_amdgcn_readfirstlane(ring_at);
    ptr -= (int32_t)(now - ring_start);
    if (ptr < lo) {  // ran out of words: the stream is damaged
      bad = true;
      ptr = lo;
    }
    if (lane == 0) ptr_pub[parity] = ptr;
    ring_start = now >= (uint32_t)kScale + kRing ? now - kRing : now;
    ring_at = ring_start;
    asm volatile("" : "+v"(ring_at));
    lds_barrier();  // barrier of this batch
  };
  int32_t g0 = 0;
  int parity = 0;
  for (; g0 < g_tail; g0 += kBatch) {
    uint8_t *sbb = sb + parity * (int)sizeof(sym_stage[0]);
#pragma unroll
    for (int j = 0; j < kBatch; ++j) dec_chain_step<false>(xc, e, tab, ring_at, sbb + kLanes * j, true);
    batch_done(parity);
    parity ^= 1;
  }
  if (tail_groups) {
    uint8_t *sbb = sb + parity * (int)sizeof(sym_stage[0]);
    for (int32_t j = 0; j < tail_groups; ++j)
      dec_chain_step<true>(xc, e, tab, ring_at, sbb + kLanes * j, j != tail_groups - 1 || top_active);
    batch_done(parity);
  }
  // integrity: every word consumed, every lane back at the initial state (a piece: at what the record behind it
  // says).  The entry in hand has f * w4 + slot - cum in the lower half of .y, which with x >> 12 as carried makes the
  // state: it is the expected one if it has the symbol, the slot - cum and the x >> 12 of that.
  const uint32_t x_end = piece.end_states ? piece.end_states[rl] : kLow;
  const uint2 e_end = tab[x_end & (kScale - 1)];
  const uint32_t fs = e.x & 0xffffffu, y = e.y & 0xffffu, w4 = y / fs;
  const bool there = e.x == e_end.x && y - w4 * fs == (e_end.y & 0xffffu) && xc + w4 == x_end >> kScaleBits;
  if (ptr != lo + (int32_t)piece.words_left || (coder && !there)) bad = true;
  if (pieces) {
    const bool good = __ballot(bad) == 0;
    if (lane < (RK ? 1 : 2)) report_piece(a, stream, (int32_t)chunk, lane, good);
  } else if (bad) {
    raise(a.status, PLC_ERR_CORRUPT);
  }
}

// ---------------------------------------------------------------------------
// Decoder for streams coded as one unit with one table per bit depth
// ---------------------------------------------------------------------------
// The table changes from position to position, so when a word is staged the step that will consume it, and
// with it the table its slot will be looked up in, is not known.  There are at most PLC_MAX_BITS tables,
// though: the wavefront that stages a word looks its slot up in every one of them, and the ring holds one
// entry per word and table.  A step then has the one LDS round trip of the kernel above -- the ring entry of
// the next group's table for a lane that renormalises, that table's slot entry for a lane that does not, one
// read at an address chosen per lane.  For four rings and four tables to fit, an entry is 4 bytes and leaves
// the symbol out:
//   slot tables   per depth, 4 bytes per slot: f | (slot - cum) << 16                       (16 KB each)
//   rings         per depth, 4 bytes per word w: f | (f * (w >> 12) + slot - cum) << 16 with the slot
//                 w & 0xfff looked up in that depth's table (at most 4096 * 15 + 4095 = 2^16 - 1)
//   state         xh = x >> 12 without the bits the word supplies, as above: f * xh + (entry >> 16)
//   symbols       a step hands on where its entry was read from, as a 16-bit index of 4-byte words; the
//                 helper turns a batch of these into slots (a table word is its slot; a ring word names a
//                 word of the raw ring beside the rings, whose low 12 bits are the slot) and the slots into
//                 symbols through a 4 KB table per depth, while the next batch is decoded, and moves them out
//   step          multiply | add (each takes its half of the entry), compare, rank, select, shift | read:
//                 six dependent instructions and one round trip
// A step takes 62 to 69 ns (150-165 cycles, the barrier's share in it) against 42 in the kernel above, 256 units of
// 1,048,576 symbols: three more instructions, which explain 14 cycles of the difference; what the rest is has not
// been taken apart.  The decoder's uniform operands are formed once per batch, and whatever else can
// be is left to the helper (handing on the slot itself, read by the decoder from the raw ring behind its
// entry, was tried: 2.4 against 2.1 ms on the Llama shape).  The helper stages the
// words, tells the decoder each batch's tables (16 tables in a word, two batches before they are needed; the
// depths come from global memory and are asked for a batch before that, their range looked at when they are
// used), turns the batch's entries' places into symbols and moves them out; it leaves a batch's barrier
// without waiting for its stores to be acknowledged.  With candidates a third wavefront reconstructs; it takes
// a batch's symbols from the helper, one barrier later than in the kernel above, and every wavefront joins one
// more barrier at the end.
//
// The same kernel with one table (MODE 1, and 2 with a chosen candidate per position) is the decoder that
// reconstructs for thousands of streams with k <= 4: the 4-byte entries and the symbols' table bring a workgroup
// to 39.2 KB of LDS, four to a compute unit instead of three with the 8-byte entries of the kernel above, and
// what counts there is how many streams are in flight, not one step's length (5120 streams, k = 4: 7.9 -> 7.0 ms).
constexpr uint32_t kDepthTableBytes = kScale * sizeof(uint32_t);
constexpr uint32_t kDepthSymBytes = kScale;
constexpr uint32_t kDepthRingSlots = kRingWords + kRingMirror;
constexpr uint32_t kDepthRingBytes = kDepthRingSlots * sizeof(uint32_t);
constexpr uint32_t kDepthRawBytes = kDepthRingSlots * sizeof(uint16_t);
static_assert(kDepthTableBytes % 16 == 0 && kDepthRingBytes % 16 == 0 && kDepthRawBytes % 16 == 0, "16-byte stores");
// dynamic LDS of the kernel: the slot tables, the rings, the raw ring, the symbol tables
inline size_t depths_lds_bytes(int n_tables) {
  return (size_t)n_tables * (kDepthTableBytes + kDepthRingBytes + kDepthSymBytes) + kDepthRawBytes;
}
constexpr int depths_threads(int rk) { return rk ? 192 : 128; }
static_assert(PLC_MAX_BITS * (kDepthTableBytes + kDepthRingBytes) / 4 <= 65536, "a word of the tables and rings in 16 bits");

// A product that is to stay one: multiply and add are not contracted over this.
__device__ __forceinline__ uint32_t keep_apart(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

// LDS of the kernel in 4-byte words.  tw is the first word of the next group's slot table, ring_at the word
// of that group's ring where the top word sits (both uniform; ring_at in a vector register), ring_step how far
// the ring that the step after this one reads lies behind this one's: ring_at for that step is formed here,
// behind the read, like everything else a step can do before its entry has arrived.  `at` is the word the
// entry in hand was read from; it is what a step hands on for its symbol.
template <bool MASKED>
__device__ __forceinline__ void dec_depth_step(uint32_t &xh, uint32_t &e, uint32_t &at, const uint32_t *lds_words,
                                               uint32_t &ring_at, uint16_t *code_slot, uint32_t tw,
                                               uint32_t ring_step, uint32_t slot_mask, bool on) {
  // f * (x >> 12) + slot - cum; product and sum kept apart so that each takes its half of the entry through
  // the instruction's own operand select instead of a mask and a shift in front of a fused multiply-add
  uint32_t fx = __umul24(e & 0xffffu, xh);
  PLC_PIN();
  const uint32_t xn = keep_apart(fx) + (e >> 16);
  PLC_PIN();
  uint64_t mask = __builtin_amdgcn_uicmp(xn, kLow, 36 /* unsigned < */);
  if (MASKED) mask &= __builtin_amdgcn_ballot_w64(on);
  const uint32_t m32 = (uint32_t)mask;
  const bool need = __builtin_amdgcn_inverse_ballot_w64(mask);
  PLC_PIN();
  // ring entry of the rank-th word from the top, or slot-table entry of xn (tables start at multiples of 4096
  // words); what stands between the compare and the rank takes the place of its wait states
  uint32_t idx_slot = (xn & slot_mask) | tw;  // (the mask in a register: and-or is one instruction then)
  asm volatile("" : "+v"(idx_slot));  // in a register: the choice below is one select, not a branch
  PLC_PIN();
  uint32_t kept = xn >> kScaleBits;
  asm volatile("" : "+v"(kept));
  PLC_PIN();
  const uint32_t idx_ring = __builtin_amdgcn_mbcnt_lo(m32, ring_at);
  PLC_PIN();
  const uint32_t at_next = need ? idx_ring : idx_slot;
  const uint32_t en = lds_words[at_next];
  PLC_PIN();  // what follows is issued in the shadow of the read
  asm volatile("v_bcnt_u32_b32 %0, %1, %0" : "+v"(ring_at) : "s"(m32));
  uint32_t shifted = xn << 4;
  asm volatile("" : "+v"(shifted));
  PLC_PIN();
  if (!MASKED || on) *code_slot = (uint16_t)at;
  PLC_PIN();
  ring_at += ring_step;
  const uint32_t next = need ? shifted : kept;
  if (!MASKED || on) {
    xh = next;
    e = en;
    at = at_next;
  }
  PLC_PIN();  // all of it before the entry is waited for
}

template <int RK, int MODE = 0>  // MODE 0: a table per depth; 1: one table; 2: one table and a chosen candidate
__global__ __launch_bounds__(depths_threads(RK)) void rans_decode_depths_kernel(const RansArgs a) {
  static_assert(MODE == 0 || RK > 0, "the one-table forms exist for the decoder that reconstructs");
  constexpr int RB = 4;  // ring blocks
  constexpr uint32_t kRing = kRingWords;
  constexpr int32_t kBelow = 3 * kBlockWords;  // how far below the pointer the words are staged
  const int n_tables = MODE ? 1 : a.n_tables;
  extern __shared__ __attribute__((aligned(16))) char depth_lds[];  // see depths_lds_bytes
  __shared__ __attribute__((aligned(16))) uint16_t code_stage[2][kBatchSyms];  // where the entries were read from
  __shared__ uint16_t code_spare[kBatchSyms];                                  // the same from lanes 32..63, never read
  __shared__ __attribute__((aligned(16))) uint8_t sym_stage[2][kBatchSyms];    // symbols, for the reconstruction
  SlotIndex *const index = reinterpret_cast<SlotIndex *>(&code_stage[0][0]);   // while the tables are built
  static_assert(sizeof(code_stage) >= sizeof(SlotIndex), "room for the index");
  __shared__ uint32_t tables_of_batch[4];  // batch b mod 4: the tables of groups 16 b + 1 .. 16 b + 16, two bits each
  __shared__ uint32_t first_table;
  __shared__ int32_t ptr_pub[2];  // the word pointer after batch b, in slot b mod 2
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const bool helper = wave == 1;
  const int64_t stream = blockIdx.x / a.wgs_per_stream;
  const int64_t chunk = blockIdx.x - stream * a.wgs_per_stream;
  const uint32_t ring_off = (uint32_t)n_tables * kDepthTableBytes;
  const uint32_t raw_off = ring_off + (uint32_t)n_tables * kDepthRingBytes;
  const uint32_t symtab_off = raw_off + kDepthRawBytes;
  // (pieces with a table per depth go to the many-unit decoder)
  const bool pieces = MODE && a.pieces > 0;  // uniform: the unit is a piece of the stream
  bool bad = false;
  if (a.verified_pieces && stream_verified(a, stream)) return;  // uniform: nothing to decode again
  // (uniform: every wavefront leaves, before any barrier that another might wait at)
  auto give_up = [&]() {
    if (threadIdx.x != 0) return;
    if (pieces) {
      report_piece(a, stream, (int32_t)chunk, 0, false);
    } else {
      raise(a.status, PLC_ERR_CORRUPT);
    }
  };

  // As in the kernel above, everything that the start needs from global memory is asked for before the tables are
  // built, in which the wavefront that reconstructs has no part.
  constexpr int kMaxTables = MODE ? 1 : PLC_MAX_BITS;
  uint32_t f[kMaxTables][4], cum[kMaxTables];
  uint32_t used = 0;  // uniform: bit t set when table t is one; an all-zero table (a depth the stream does not use) is none
  bool tables_ok = true;
#pragma unroll
  for (int t = 0; t < kMaxTables; ++t) {
    if (t >= n_tables) break;
    const uint32_t total = load_freq4(a.freq + (stream * n_tables + t) * 256, lane, f[t], &cum[t]);
    if (total == kScale) {
      used |= 1u << t;
    } else if (MODE || total != 0) {
      tables_ok = false;
    }
  }

  // the unit: the stream, or a piece of it
  const uint64_t off = a.word_off[stream];
  const uint32_t n = a.n_words_in[stream];
  Piece piece = {0u, (uint32_t)a.syms_per_stream, n, 0u, 0u, 0u, a.states_in + stream * kLanes, nullptr};
  if (!tables_ok || off > a.words_len || (uint64_t)n > a.words_len - off ||
      (pieces && !load_piece(a, stream, (int32_t)chunk, n, &piece))) {
    give_up();
    return;
  }
  const int64_t begin = piece.begin;
  const uint32_t len = piece.len;
  const int32_t G = (int32_t)((len + kLanes - 1) / kLanes);
  const uint32_t top_syms = len - (uint32_t)(G - 1) * kLanes;

  const uint16_t *first_word = a.words_in + off;
  const int32_t lo = (int32_t)((reinterpret_cast<uintptr_t>(first_word) & (uintptr_t)(kBlockWords * 2 - 1)) >> 1);
  const uint16_t *aligned_base = first_word - lo;
  const int32_t hi = lo + (int32_t)piece.words;

  int32_t tail_groups = G % kBatch;
  if (tail_groups == 0 && top_syms < kLanes) tail_groups = kBatch;
  const int32_t g_tail = G - tail_groups;

  if constexpr (RK > 0) {  // the wavefront that reconstructs, one barrier behind the decoder's batch
    if (wave == 2) {
      reconstruct_batches<RK, MODE != 1, MODE == 0, kRecDepthBase, 1, kBatchSyms>(a, stream, piece, G, sym_stage, lane,
                                                                                  2 * n_tables);
      return;
    }
  }

  auto block_load = [&](int32_t blk, uint4 &v) -> bool {
    const int32_t first = blk * kBlockWords + lane * 8;
    const bool take = blk >= 0 && hi > lo && first + 8 > lo && first < hi;
    if (take) v = *reinterpret_cast<const uint4 *>(aligned_base + first);
    return take;
  };
  const int32_t top_block = (hi - 1) >> 9;
  const int32_t first_down = hi - kBelow > 0 ? (hi - kBelow) >> 9 : 0;  // the blocks down to here come first
  uint4 first_v[RB];
  bool first_take[RB];
  if (helper) {
#pragma unroll
    for (int i = 0; i < RB; ++i) first_take[i] = top_block - i >= first_down && block_load(top_block - i, first_v[i]);
  }
  const uint32_t x0 = piece.states[lane & (kLanes - 1)];

  // slot and symbol tables, one depth after the other
#pragma unroll
  for (int t = 0; t < kMaxTables; ++t) {
    if (t >= n_tables) break;
    if (wave == 0 && ((used >> t) & 1u)) build_slot_index(index, f[t], cum[t], lane);
    lds_barrier();
    uint32_t *tt = reinterpret_cast<uint32_t *>(depth_lds + (size_t)t * kDepthTableBytes);
    uint8_t *ts = reinterpret_cast<uint8_t *>(depth_lds + symtab_off + (size_t)t * kDepthSymBytes);
    if ((used >> t) & 1u) {
      for_each_slot<128>(index, [&](uint32_t o, uint32_t row) {
        tt[o] = ((row & 0xfffu) + 1u) | ((o - ((row >> 12) & 0xfffu)) << 16);
        ts[o] = (uint8_t)(row >> 24);
      });
    } else {
      for (uint32_t o = threadIdx.x; o < (uint32_t)kScale; o += 128) tt[o] = 0u, ts[o] = 0;
    }
    lds_barrier();
  }

  if (helper) {
    bool bad_depth = false;
    uint8_t *ubase = a.sym_out + stream * a.syms_per_stream + begin;
    const bool out_aligned = (reinterpret_cast<uintptr_t>(ubase) & 7u) == 0;
    // word i goes to ring position (~i) mod 2048: the lane's eight words, last one first
    auto block_store = [&](int32_t blk, bool take, const uint4 &v) {
      if (take) {
        // word i sits at ring position kRing - 1 - i mod kRing; this is the lane's last word's
        const uint32_t pos = (uint32_t)((RB - 1 - blk % RB) * kBlockWords + (kBlockWords - 8 - lane * 8));
        const uint32_t w[8] = {v.w >> 16, v.w & 0xffffu, v.z >> 16, v.z & 0xffffu,
                               v.y >> 16, v.y & 0xffffu, v.x >> 16, v.x & 0xffffu};
        const uint4 rw = make_uint4(w[0] | (w[1] << 16), w[2] | (w[3] << 16), w[4] | (w[5] << 16), w[6] | (w[7] << 16));
        char *raw = depth_lds + raw_off;
        *reinterpret_cast<uint4 *>(raw + pos * 2) = rw;
        if (pos < (uint32_t)kRingMirror) *reinterpret_cast<uint4 *>(raw + (kRing + pos) * 2) = rw;
        for (int t = 0; t < n_tables; ++t) {  // uniform
          if (!((used >> t) & 1u)) continue;    // a depth without a table is never looked up
          const uint32_t *tt = reinterpret_cast<const uint32_t *>(depth_lds + (size_t)t * kDepthTableBytes);
          uint32_t en[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const uint32_t s = tt[w[i] & (kScale - 1)];
            en[i] = s + (__umul24(s & 0xffffu, w[i] >> kScaleBits) << 16);
          }
          uint32_t *ring = reinterpret_cast<uint32_t *>(depth_lds + ring_off + (size_t)t * kDepthRingBytes);
          const uint4 r0 = make_uint4(en[0], en[1], en[2], en[3]), r1 = make_uint4(en[4], en[5], en[6], en[7]);
          *reinterpret_cast<uint4 *>(&ring[pos]) = r0;
          *reinterpret_cast<uint4 *>(&ring[pos + 4]) = r1;
          if (pos < (uint32_t)kRingMirror) {
            *reinterpret_cast<uint4 *>(&ring[kRing + pos]) = r0;
            *reinterpret_cast<uint4 *>(&ring[kRing + pos + 4]) = r1;
          }
        }
      }
    };
    // as in the kernel above: the newest block stays on its way for a batch
#pragma unroll
    for (int i = 0; i < RB; ++i) block_store(top_block - i, first_take[i], first_v[i]);
    int32_t lowest = top_block + 1 < first_down ? top_block + 1 : first_down;  // lowest block already requested
    uint4 ahead_v;
    int32_t ahead_blk = 0;
    bool ahead = false, ahead_take = false;
    auto stage_down_to = [&](int32_t down_to, bool leave_one) {
      if (ahead) {  // uniform
        block_store(ahead_blk, ahead_take, ahead_v);
        ahead = false;
      }
      const int32_t last = down_to > 0 ? down_to >> 9 : 0;
      while (lowest > last) {
        const int32_t blk = lowest - 1;
        lowest = blk;
        if (leave_one && blk == last) {
          ahead_take = block_load(blk, ahead_v);
          ahead_blk = blk;
          ahead = true;
        } else {
          uint4 v;
          const bool take = block_load(blk, v);
          block_store(blk, take, v);
        }
      }
    };
    // Tables of groups g0 + 1 .. g0 + 16, the ones the 16 steps of the batch at g0 look up (past the last
    // group: the first table, whose entry is never used).  A depth is asked for here and looked at a batch
    // later (in range or not included), when it is packed with the 15 others for the decoder.
    static_assert(PLC_MAX_BITS <= 4 && kBatch == 16, "two bits per table, 16 tables in a word");
    const uint32_t spp = MODE ? 1u : (uint32_t)a.syms_per_pos;  // (one table: no depths, nothing below is reached)
    const uint8_t *depth_row =
        MODE ? nullptr
             : a.bits + (int64_t)((uint32_t)stream / (uint32_t)a.streams_per_session) * ((uint32_t)a.syms_per_stream / spp);
    auto fetch_depths = [&](int32_t g0) -> uint32_t {
      const int32_t g = g0 + 1 + (lane & (kBatch - 1));
      return g < G ? depth_row[(uint32_t)(begin + (int64_t)g * kLanes) / spp] : 1u;
    };
    auto pack_tables = [&](uint32_t depth) -> uint32_t {  // lanes 0..15 hold a depth each
      if (depth < 1u || depth > (uint32_t)a.n_tables) {
        bad_depth = true;
        depth = 1u;
      }
      uint32_t v = (depth - 1u) << (2 * (lane & (kBatch - 1)));
#pragma unroll
      for (int off = 1; off < kBatch; off <<= 1) v |= __shfl_xor(v, off, 64);
      return (uint32_t)__builtin_amdgcn_readfirstlane(v);
    };
    uint32_t t_first = 0, tables_cur = 0, tables_next = 0, depth_ahead = 1;
    if constexpr (MODE == 0) {
      t_first = group_table(a, stream, begin, 0, 1u, &bad_depth);  // table of the coming batch's first group
      tables_cur = pack_tables(fetch_depths(0)), tables_next = pack_tables(fetch_depths(kBatch));
      if (lane == 0) {
        first_table = t_first;
        tables_of_batch[0] = tables_cur;
        tables_of_batch[1] = tables_next;
      }
      depth_ahead = fetch_depths(2 * kBatch);
    }
    lds_barrier();  // barrier "start"
    int32_t ptr_before = hi;
    for (int32_t g0 = 0; g0 < G; g0 += kBatch) {
      stage_down_to(ptr_before - kBelow, true);
      uint32_t tables_after = 0;
      if constexpr (MODE == 0) {
        tables_after = pack_tables(depth_ahead);
        if (lane == 0) tables_of_batch[((g0 / kBatch) + 2) & 3] = tables_after;
        depth_ahead = fetch_depths(g0 + 3 * kBatch);
      }
      lds_barrier();  // barrier of this batch
      // (The pointer has a slot per batch parity: this wavefront may still be waiting for its loads from global
      // memory, which the barrier above does not wait for, when the decoder publishes the pointer after the next
      // batch; read from a single slot it then stages a block too early, over words whose places are yet to be
      // turned into symbols.)
      ptr_before = ptr_pub[(g0 / kBatch) & 1];
      // the table of the group this lane's eight entries of the batch belong to: the one the step before
      // looked up (for the batch's first group: the last of the batch before)
      const uint32_t t_mine = (lane >> 2) == 0 ? t_first : (tables_cur >> (2 * ((lane >> 2) - 1))) & 3u;
      t_first = tables_cur >> 30;
      tables_cur = tables_next;
      tables_next = tables_after;
      const bool tail = g0 >= g_tail;
      const int32_t cnt_groups = tail ? tail_groups : kBatch;
      const int buf = (g0 / kBatch) & 1;
      const uint32_t done = (uint32_t)g0 * kLanes;
      const uint32_t room = (uint32_t)cnt_groups * kLanes;
      const uint32_t nsym = (len - done) < room ? (len - done) : room;
      // where each entry was read from -> slot -> symbol, eight per lane
      const uint4 cv = *reinterpret_cast<const uint4 *>(&code_stage[buf][lane * 8]);
      const uint8_t *ts = reinterpret_cast<const uint8_t *>(depth_lds + symtab_off + (size_t)t_mine * kDepthSymBytes);
      const uint16_t *raw = reinterpret_cast<const uint16_t *>(depth_lds + raw_off);
      const uint32_t ring_word0 = ring_off / 4 + t_mine * kDepthRingSlots;  // of this group's ring
      const uint32_t c[8] = {cv.x & 0xffffu, cv.x >> 16, cv.y & 0xffffu, cv.y >> 16,
                             cv.z & 0xffffu, cv.z >> 16, cv.w & 0xffffu, cv.w >> 16};
      // (every lane reads the raw ring, needed or not, and all eight reads are on their way before the first
      // is used: two LDS round trips for the batch, not sixteen)
      uint32_t word[8], sy[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        uint32_t p = c[i] - ring_word0;  // not a ring word, or a lane past the end of the stream: keep inside
        p = p < kDepthRingSlots ? p : 0u;
        word[i] = raw[p];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t slot_i = c[i] >= ring_off / 4 ? word[i] : c[i];
        sy[i] = ts[slot_i & (kScale - 1)];
      }
      const uint2 sv = make_uint2(sy[0] | (sy[1] << 8) | (sy[2] << 16) | (sy[3] << 24),
                                  sy[4] | (sy[5] << 8) | (sy[6] << 16) | (sy[7] << 24));
      if constexpr (RK > 0) *reinterpret_cast<uint2 *>(&sym_stage[buf][lane * 8]) = sv;
      const uint32_t mine = (uint32_t)lane * 8;
      if (out_aligned && mine + 8 <= nsym) {
        *reinterpret_cast<uint2 *>(ubase + done + mine) = sv;
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (mine + i < nsym) ubase[done + mine + i] = (uint8_t)sy[i];
      }
      // (the raw ring is read above as 16-bit words and written by the staging below as 16-byte vectors: the
      // accesses are kept in this order whatever the compiler makes of their types)
      asm volatile("" ::: "memory");
    }
    if constexpr (RK > 0) lds_barrier();  // the last batch's symbols are in the stage
    if (bad_depth) raise(a.status, PLC_ERR_INVALID);
    return;
  }

  // ---- the decoding wavefront (lanes 32..63 ride along, as in the kernel above)
  const bool coder = lane < kLanes;
  const int rl = lane & (kLanes - 1);
  const bool top_active = (uint32_t)rl < top_syms;
  int32_t ptr = hi;
  lds_barrier();  // barrier "start": the first words are staged, the first tables known
  const uint32_t *lds_words = reinterpret_cast<const uint32_t *>(depth_lds);
  uint32_t slot_mask = kScale - 1;
  asm volatile("" : "+v"(slot_mask));
  uint32_t xh = x0 >> kScaleBits;
  uint32_t at = (MODE ? 0u : first_table * kScale) + (x0 & (kScale - 1));
  uint32_t e = lds_words[at];
  uint32_t tables = MODE ? 0u : (uint32_t)__builtin_amdgcn_readfirstlane(tables_of_batch[0]);
  const uint32_t ring0 = ring_off / 4;
  for (int32_t g0 = 0; g0 < G; g0 += kBatch) {
    const bool tail = g0 >= g_tail;
    const int32_t cnt_groups = tail ? tail_groups : kBatch;
    // (the next batch's tables: asked for now, used after the barrier)
    const uint32_t tables_coming = MODE ? 0u : tables_of_batch[((g0 / kBatch) + 1) & 3];
    uint16_t *sb = coder ? &code_stage[(g0 / kBatch) & 1][rl] : &code_spare[rl];
    const uint32_t q0 = kRing - 1u - (uint32_t)(ptr - 1) % kRing;  // ring position of the top word (uniform)
    uint32_t ring_at = ring0 + (tables & 3u) * kDepthRingSlots + q0;
    asm volatile("" : "+v"(ring_at));
    if (tail) {
      for (int32_t j = 0; j < cnt_groups; ++j) {
        const uint32_t t = (tables >> (2 * j)) & 3u, t_after = j + 1 < kBatch ? (tables >> (2 * j + 2)) & 3u : 0u;
        dec_depth_step<true>(xh, e, at, lds_words, ring_at, sb + kLanes * j, t * kScale,
                             (t_after - t) * kDepthRingSlots, slot_mask, j != cnt_groups - 1 || top_active);
      }
    } else {
      // every step's two uniform operands, formed before the first step (in scalar registers from here on)
      uint32_t tw[kBatch], rs[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const uint32_t t = (tables >> (2 * j)) & 3u, t_after = j + 1 < kBatch ? (tables >> (2 * j + 2)) & 3u : 0u;
        tw[j] = t * kScale;
        rs[j] = (t_after - t) * kDepthRingSlots;
        asm volatile("" : "+s"(tw[j]), "+s"(rs[j]));
      }
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
        dec_depth_step<false>(xh, e, at, lds_words, ring_at, sb + kLanes * j, tw[j], rs[j], slot_mask, true);
    }
    // (The entry in hand is handed on with the next batch's first step, and where it was read from is looked at
    // a barrier after that.  If it is a ring word it is still there then: the block staged in between goes
    // where a block above the pointer of a batch ago was, and the word is below that pointer.)
    // the ring position is now the first ring's (table 0 stands in past the batch's last group) plus the words taken
    ptr -= (int32_t)((uint32_t)__builtin_amdgcn_readfirstlane(ring_at) - ring0 - q0);
    if (ptr < lo) {
      bad = true;
      ptr = lo;
    }
    if (lane == 0) ptr_pub[(g0 / kBatch) & 1] = ptr;
    __syncthreads();  // barrier of this batch
    tables = MODE ? 0u : (uint32_t)__builtin_amdgcn_readfirstlane(tables_coming);
  }
  if constexpr (RK > 0) __syncthreads();  // the helper's last batch of symbols, for the reconstruction
  // integrity: every word consumed, every lane back at the initial state (a piece: at what the record behind it
  // says): x >> 12 as carried, and what the place of the entry in hand tells (the helper stages nothing after the
  // last batch's barrier), the word shifted in or the slot
  uint32_t w;
  if (at >= ring0) {
    const uint32_t p = (at - ring0) % kDepthRingSlots;
    w = reinterpret_cast<const uint16_t *>(depth_lds + raw_off)[p];
  } else {
    w = at & (kScale - 1);
  }
  const uint32_t x_now = (xh << kScaleBits) + w;
  const uint32_t x_end = piece.end_states ? piece.end_states[rl] : kLow;
  if (ptr != lo + (int32_t)piece.words_left || (coder && x_now != x_end)) bad = true;
  if (pieces) {
    const bool good = __ballot(bad) == 0;
    if (lane < (RK ? 1 : 2)) report_piece(a, stream, (int32_t)chunk, lane, good);
  } else if (bad) {
    raise(a.status, PLC_ERR_CORRUPT);
  }
}

int check_common(int64_t n_streams, int64_t syms_per_stream, int32_t chunk_syms, RansArgs *a) {
  if (n_streams < 1 || syms_per_stream < 1) return PLC_ERR_INVALID;
  if (syms_per_stream >= (1ll << 31) - 1024) return PLC_ERR_INVALID;
  if (chunk_syms < 0 || chunk_syms % kLanes) return PLC_ERR_INVALID;
  a->units_per_stream = plc_units_per_stream(syms_per_stream, chunk_syms);
  a->unit_syms = chunk_syms > 0 ? chunk_syms : syms_per_stream;
  a->n_units = n_streams * a->units_per_stream;
  a->syms_per_stream = syms_per_stream;
  int w = 1;
  while (w < kMaxWaves && 2 * w <= a->units_per_stream) w *= 2;
  const int64_t wgs = (a->units_per_stream + w - 1) / w;
  if (wgs >= (1ll << 31) || n_streams * wgs >= (1ll << 31)) return PLC_ERR_INVALID;
  a->wgs_per_stream = (uint32_t)wgs;
  return PLC_OK;
}

// Rounds of the encoder's staging, four batches each, of a stream coded as one unit: pieces are whole rounds.
int32_t restart_rounds(int64_t syms_per_stream) {
  const int32_t G = (int32_t)((syms_per_stream + kLanes - 1) / kLanes);
  const int32_t head = G % kBatch ? G % kBatch : kBatch;
  return ((G - head) / kBatch + 1 + 3) / 4;
}
// How a stream of so many records is cut: returns the pieces, 0 where it is too short for two.
int32_t plan_pieces(RansArgs *a, int32_t per_stream) {
  const int32_t rounds = restart_rounds(a->syms_per_stream);
  const int32_t per = (rounds + per_stream - 1) / per_stream;
  a->point_stride = per_stream;
  a->piece_batches = 4 * per;
  a->point_step = 1;
  const int32_t pieces = (rounds + per - 1) / per;
  return pieces < 2 ? 0 : pieces;
}
// Restart points, for a call with one unit per stream (check_common before).
int check_restart(const plc_restart *r, bool decode, RansArgs *a) {
  if (!r) return PLC_OK;
  if (a->units_per_stream != 1 || a->unit_syms != a->syms_per_stream || a->n_units > kPipeMaxUnits) return PLC_ERR_INVALID;
  if (r->per_stream < 2 || r->per_stream > (1 << 20) || !r->points || reinterpret_cast<uintptr_t>(r->points) % 4)
    return PLC_ERR_INVALID;
  if (decode && (!r->scratch || reinterpret_cast<uintptr_t>(r->scratch) % 4)) return PLC_ERR_INVALID;
  const int32_t pieces = plan_pieces(a, r->per_stream);
  if (decode) {
    a->points_in = r->points;
    a->piece_state = r->scratch;
    a->pieces = pieces;
  } else {
    a->points_out = r->points;
  }
  return PLC_OK;
}
// Pieces of several records each, so that there are about `most` of them.
void merge_pieces(RansArgs *a, int64_t n_streams, int64_t most) {
  const int64_t per_stream = most / n_streams < 1 ? 1 : most / n_streams;
  if (a->pieces <= per_stream) return;
  a->point_step = (int32_t)((a->pieces + per_stream - 1) / per_stream);
  a->piece_batches *= a->point_step;
  a->pieces = (a->pieces + a->point_step - 1) / a->point_step;
  if (a->pieces < 2) a->pieces = 0;
}
void merge_pieces_for(RansArgs *a, int64_t n_streams, int k) {
  merge_pieces(a, n_streams, k <= kCompactMaxK ? kPiecesPerRoundCompact : kPiecesPerRound);
}
// Whether streams in pieces are better decoded by one call and reconstructed by another.  The one kernel takes the
// chain of its longest piece, once per round of workgroups; two calls that of shorter pieces, some 15 to 28 us more of
// starts and passes, the time of the memory they move, and a stream's tiles are added up by one workgroup.  Fitted to
// 947 shapes, 1 to 1024 streams of 8192 to 16,777,216 symbols, 4 to 134 million together, both ways timed for each: on
// average 0.03 % is lost by what it chooses and 4 % at the most (a bound on the symbols altogether lost 2.6 and 46 %).
// For instance, one kernel and two calls in us: given the tokens, k = 8, 1024 streams of 8192 64 and 73, of 32,768 140
// and 96; 128 of 65,536 61 and 70; the mean of 4, 1024 of 16,384 65 and 79; of 5, 288 of 65,536 131 and 91, 105 of 124,320
// 95 and 102; of 8, 512 of 131,072 288 and 278.
bool pieces_in_two_calls(int64_t n_streams, int64_t syms_per_stream, int k, bool cond, int32_t points) {
  RansArgs a = {};
  a.syms_per_stream = syms_per_stream;
  a.pieces = plan_pieces(&a, points);
  if (!a.pieces) return false;
  auto piece_syms = [&] {
    const int64_t syms = a.pieces ? (int64_t)a.piece_batches * kBatchSyms : syms_per_stream;
    return syms < syms_per_stream ? syms : syms_per_stream;
  };
  const int64_t two_chain = piece_syms();
  merge_pieces_for(&a, n_streams, k);
  const int64_t units = n_streams * (a.pieces ? a.pieces : 1);
  const bool dense = units > kDenseStreams;
  const int64_t at_once = dense && k <= kCompactMaxK ? 4 * kComputeUnits
                          : dense && !cond && k <= kDenseMaxK ? 3 * kComputeUnits : 2 * kComputeUnits;
  // by how much the one kernel's is longer
  const double chain = (double)(piece_syms() * ((units + at_once - 1) / at_once) - two_chain);
  double per_step, more, per_symbol;  // ns a symbol of the chain; us; ns a symbol
  if (cond) {
    per_step = k <= kCompactMaxK ? 2.22 : 1.45, more = 28.5, per_symbol = 0.6e-3;
  } else {
    per_step = k <= kCompactMaxK ? 2.42 + 0.163 * k : k > kDenseMaxK ? 2.05 : dense ? 2.31 : 1.91;
    more = k <= kCompactMaxK ? 28.6 : k > kDenseMaxK ? 24.5 : 19.5;
    per_symbol = 0.51e-3 + 0.32e-3 * k;
  }
  // (where a stream is no whole tiles, the escapes are counted in a pass of its own)
  if (syms_per_stream % kTileSyms) more += cond ? 7.0 : 12.0;
  return 1e-3 * per_step * chain >
         more + 1e-3 * per_symbol * (double)(n_streams * syms_per_stream) + 2.8e-6 * (double)syms_per_stream;
}
// The arguments of the launch behind the pieces', which decodes the streams whose pieces do not agree.
RansArgs again_args(RansArgs a) {
  a.verified_pieces = a.pieces;
  a.pieces = 0;
  a.wgs_per_stream = 1;
  return a;
}

// Wavefronts of per_wave units each to a workgroup, for units that share a stream's tables: a workgroup holds all of a
// stream's if eight wavefronts can, so that the tables are built once and the last workgroup is not nearly empty.  (Two
// units to a wavefront, decoding, and workgroups of the next smaller size, a stream's second one with few units: 4096
// streams of three chunks of 1024 37 and 49 us, of five 44 and 58, 1024 of six chunks of 4096 33 and 52, 768 streams of
// 131,072 symbols in ten pieces, given the tokens, 206 and 250.)  Long units that are fewer than that leaves workgroups
// for every compute unit are spread over them (64 streams of ten chunks of 65,536: 276 and 261 us; chunks of 8192 are
// better off together, 45 and 46).
constexpr int64_t kSpreadSyms = 32768;
int waves_per_workgroup(int64_t n_streams, int64_t units, int per_wave, int64_t unit_syms) {
  auto wgs = [&](int waves) { return n_streams * ((units + per_wave * waves - 1) / (per_wave * waves)); };
  int w = 1;
  while (w < kMaxWaves && per_wave * w < units && (unit_syms < kSpreadSyms || wgs(2 * w) >= kComputeUnits)) w *= 2;
  return w;
}

template <int W>  // workgroups of 2 W units of one stream
void launch_decode_pairs_of(const RansArgs &a, unsigned grid, hipStream_t st, const TraceScope &trace) {
  trace.kernel("rans_decode_pair_kernel<%d, %s, %s>", W, a.bits ? "true" : "false", a.pieces ? "true" : "false");
  if (a.bits) {
    const size_t lds = (size_t)a.n_tables * kCompactTable * sizeof(uint32_t);
    const auto kernel = a.pieces ? &rans_decode_pair_kernel<W, true, true> : &rans_decode_pair_kernel<W, true, false>;
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(W * 64), lds, st, a);
  } else {
    const auto kernel = a.pieces ? &rans_decode_pair_kernel<W, false, true> : &rans_decode_pair_kernel<W, false, false>;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(W * 64), 0, st, a);
  }
}
// Two or more units per stream, or pieces.
void launch_decode_pairs(RansArgs a, int64_t n_streams, hipStream_t st, const TraceScope &trace) {
  const int64_t units = a.pieces ? a.pieces : a.units_per_stream;
  const int w = waves_per_workgroup(n_streams, units, 2, a.pieces ? (int64_t)a.piece_batches * kBatchSyms : a.unit_syms);
  a.wgs_per_stream = (uint32_t)((units + 2 * w - 1) / (2 * w));
  const unsigned grid = (unsigned)(n_streams * a.wgs_per_stream);
  switch (w) {
    case 1: launch_decode_pairs_of<1>(a, grid, st, trace); break;
    case 2: launch_decode_pairs_of<2>(a, grid, st, trace); break;
    case 4: launch_decode_pairs_of<4>(a, grid, st, trace); break;
    default: launch_decode_pairs_of<8>(a, grid, st, trace); break;
  }
}
// Encoder of chunks with a table per depth: while few wavefronts are resident a unit to each has the shorter step (chunks of 65,536,
// one and two to a wavefront: 768 of them 187 and 253 us, 1536 222 and 300, 2048 225 and 270, 2560 265 and 307, 3072 378
// and 306, 4096 392 and 317; of 4096: 768 25 and 30, 2560 32 and 33, 3072 41 and 34).
constexpr int64_t kFewChunks = 10 * kComputeUnits;
// So it is in the decoder (768 chunks of 65,536 351 and 365 us, 1536 366 and 393, 2560 388 and 404, 3072 703 and 399; of
// 4096: 768 38 and 40, 2560 45 and 47, 3072 65 and 43), but for units that are to have their tiles' escapes counted, which
// only the other kernel does: there from this length on (to K and V, 512 chunks of 262,144 1431 and 1520 us, 1536 of
// 65,536 523 and 525).
constexpr int64_t kFewChunkSymsCounted = 1 << 17;
bool decode_depths_alone(const RansArgs &a, bool counted) {
  return a.bits && !a.pieces && a.n_units <= kFewChunks && !(counted && a.unit_syms < kFewChunkSymsCounted);
}
template <int W, bool CHUNKS = true>
void launch_decode_depths_of(const RansArgs &a, unsigned grid, hipStream_t st, const TraceScope *trace) {
  if (trace) trace->kernel("rans_decode_kernel<%d, true, %s>", W, CHUNKS ? "true" : "false");
  // (split tables: 5 KB per depth instead of 16 lets three times the wavefronts in)
  const size_t lds = (size_t)a.n_tables * kCompactTable * sizeof(uint32_t);
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&rans_decode_kernel<W, true, CHUNKS>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((rans_decode_kernel<W, true, CHUNKS>), dim3(grid), dim3(W * 64), lds, st, a);
}
// Chunks with a table per depth, a unit per wavefront.
void launch_decode_depths(RansArgs a, int64_t n_streams, hipStream_t st, const TraceScope &trace) {
  const int w = waves_per_workgroup(n_streams, a.units_per_stream, 1, a.unit_syms);
  a.wgs_per_stream = (uint32_t)((a.units_per_stream + w - 1) / w);
  const unsigned grid = (unsigned)(n_streams * a.wgs_per_stream);
  switch (w) {
    case 1: launch_decode_depths_of<1>(a, grid, st, &trace); break;
    case 2: launch_decode_depths_of<2>(a, grid, st, &trace); break;
    case 4: launch_decode_depths_of<4>(a, grid, st, &trace); break;
    default: launch_decode_depths_of<8>(a, grid, st, &trace); break;
  }
}
// One unit per stream.  trace: null behind pieces, whose kernel is the main one.
void launch_decode_streams(const RansArgs &a, hipStream_t st, const TraceScope *trace) {
  const dim3 grid((unsigned)a.n_units);
  auto name = [&](const char *kernel) {
    if (trace) trace->kernel(kernel);
  };
  // Few enough units (kChainMaxUnits): time is the length of one unit's chain, so take the variant with the shortest
  // step.  With more units its 60 KB of LDS per workgroup would cost more in occupancy than the shorter step gains.
  if (a.bits && a.n_units <= kDepthsMaxUnits) {
    const size_t lds = depths_lds_bytes(a.n_tables);
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&rans_decode_depths_kernel<0>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    name("rans_decode_depths_kernel<0, 0>");
    hipLaunchKernelGGL(rans_decode_depths_kernel<0>, grid, dim3(depths_threads(0)), lds, st, a);
  } else if (a.bits) {
    launch_decode_depths_of<1, false>(a, (unsigned)a.n_units, st, trace);
  } else if (a.n_units <= kChainMaxUnits) {
    name("rans_decode_chain_kernel<0, false, 4>");
    hipLaunchKernelGGL((rans_decode_chain_kernel<0, false>), grid, dim3(128), 0, st, a);
  } else {
    // Many units: LDS decides how many wavefronts fit a compute unit, and the split table lets more in (twice as many
    // where every one-wavefront workgroup has a table of its own).
    name("rans_decode_kernel<1, false, false>");
    hipLaunchKernelGGL((rans_decode_kernel<1, false, false>), grid, dim3(64), 0, st, a);
  }
}

}  // namespace
}  // namespace plc

using namespace plc;

extern "C" int64_t plc_units_per_stream(int64_t syms_per_stream, int32_t chunk_syms) {
  if (chunk_syms <= 0) return 1;
  return (syms_per_stream + chunk_syms - 1) / chunk_syms;
}

namespace plc {
namespace {

// Arguments of the calls with one table per bit depth.
int check_depths(int64_t syms_per_stream, int32_t chunk_syms, int32_t syms_per_pos, int32_t streams_per_session,
                 const uint8_t *bits, int32_t n_tables, RansArgs *a) {
  if (!bits || n_tables < 1 || n_tables > PLC_MAX_BITS || streams_per_session < 1) return PLC_ERR_INVALID;
  if (syms_per_pos < kLanes || syms_per_pos % kLanes || syms_per_stream % syms_per_pos) return PLC_ERR_INVALID;
  (void)chunk_syms;  // a multiple of 32 already: groups never straddle positions
  a->bits = bits;
  a->syms_per_pos = syms_per_pos;
  a->streams_per_session = streams_per_session;
  a->n_tables = n_tables;
  return PLC_OK;
}

// Many whole streams with a table per depth: a compute unit holds seven wavefronts with a stream each, or six with two
// each, whose steps take longer.  Two each where that halves the rounds, and where there are so many that the last one's
// emptiness tells little.  Streams of 131,072 symbols, one and two to a wavefront: 1536 428 and 550 us, 1900 709 and 554,
// 3072 813 and 635, 3200 813 and 1076, 4096 1108 and 1160, 5120 1210 and 1174, 5376 1224 and 1236, 5632 1421 and 1243, 6144
// 1492 and 1250, 6656 1584 and 1690, 7168 1615 and 1705, 7400 1783 and 1715; of 32,768: 5632 391 and 339, 7168 442 and 459,
// 9216 575 and 504, 12,544 746 and 738, 14,336 848 and 800.
bool encode_depths_in_pairs(int64_t n_units) {
  const int64_t one = (n_units + 7 * kComputeUnits - 1) / (7 * kComputeUnits);
  const int64_t two = (n_units + 12 * kComputeUnits - 1) / (12 * kComputeUnits);
  return one > 4 || 2 * two <= one;
}
template <int W>
void launch_encode_depths_of(const RansArgs &a, unsigned grid, hipStream_t st, const TraceScope &trace) {
  trace.kernel("rans_encode_kernel<%d>", W);
  hipLaunchKernelGGL(rans_encode_kernel<W>, dim3(grid), dim3(W * 64), 0, st, a);
}
void launch_encode_depths(RansArgs a, int64_t n_streams, hipStream_t st, const TraceScope &trace) {
  const int w = waves_per_workgroup(n_streams, a.units_per_stream, 1, a.unit_syms);
  a.wgs_per_stream = (uint32_t)((a.units_per_stream + w - 1) / w);
  const unsigned grid = (unsigned)(n_streams * a.wgs_per_stream);  // at most the grid checked before
  switch (w) {
    case 1: launch_encode_depths_of<1>(a, grid, st, trace); break;
    case 2: launch_encode_depths_of<2>(a, grid, st, trace); break;
    case 4: launch_encode_depths_of<4>(a, grid, st, trace); break;
    default: launch_encode_depths_of<8>(a, grid, st, trace); break;
  }
}

int encode_impl(const uint8_t *symbols, int64_t n_streams, int64_t syms_per_stream, int32_t chunk_syms,
                const uint16_t *freq, uint32_t *states, uint16_t *words, const uint64_t *word_off,
                uint64_t word_cap_per_unit, uint32_t *n_words, uint32_t *status, void *stream, RansArgs a,
                const plc_restart *restart = nullptr) {
  int rc = check_common(n_streams, syms_per_stream, chunk_syms, &a);
  if (!rc) rc = check_restart(restart, false, &a);
  if (rc) return rc;
  if (!symbols || !freq || !states || !word_off || !n_words || !status) return PLC_ERR_INVALID;
  if (word_cap_per_unit > 0 && !words) return PLC_ERR_INVALID;
  if (reinterpret_cast<uintptr_t>(freq) % 8 || reinterpret_cast<uintptr_t>(words) % 2) return PLC_ERR_INVALID;
  a.sym_in = symbols;
  a.freq = freq;
  a.states_out = states;
  a.words_out = words;
  a.word_off = word_off;
  a.word_cap = word_cap_per_unit;
  a.n_words_out = n_words;
  a.status = status;
  hipStream_t st = static_cast<hipStream_t>(stream);
  {
    TraceScope trace(PLC_TRACE_RANS_ENCODE, st);
    const dim3 few_grid((unsigned)a.n_units), short_block(short_units::kThreads), pipe_block(kPipeThreads);
    if (a.units_per_stream == 1 && encode_in_short(a.n_units, syms_per_stream, a.bits != nullptr)) {
      const bool wide = !a.bits || a.n_units <= 2 * kComputeUnits;
      trace.kernel("rans_encode_short_kernel<%s, %s>", a.bits ? "true" : "false", wide ? "true" : "false");
      if (!a.bits) {
        hipLaunchKernelGGL((short_units::rans_encode_short_kernel<false>), few_grid, short_block, 0, st, a);
      } else if (wide) {
        hipLaunchKernelGGL((short_units::rans_encode_short_kernel<true, true>), few_grid, short_block, 0, st, a);
      } else {
        hipLaunchKernelGGL((short_units::rans_encode_short_kernel<true, false>), few_grid, short_block, 0, st, a);
      }
    } else if (a.units_per_stream == 1 && encode_in_pipe(a.n_units, syms_per_stream, a.bits != nullptr)) {
      const bool wide = !a.bits || a.n_units <= kComputeUnits, few = a.n_units <= 2 * kComputeUnits;
      trace.kernel("rans_encode_pipe_kernel<%s, %d, %s>", a.bits ? "true" : "false", few ? 32 : 16, wide ? "true" : "false");
      // few units: the chain of one unit is the time, so give each unit seven wavefronts
      // (with more units, seven wavefronts per unit cost more in occupancy than the shorter chain gains)
      if (!a.bits && few) {
        hipLaunchKernelGGL((rans_encode_pipe_kernel<false, 32>), few_grid, pipe_block, 0, st, a);
      } else if (!a.bits) {
        hipLaunchKernelGGL((rans_encode_pipe_kernel<false, 16>), few_grid, pipe_block, 0, st, a);
      } else if (wide) {
        hipLaunchKernelGGL((rans_encode_pipe_kernel<true, 32, true>), few_grid, pipe_block, 0, st, a);
      } else if (few) {
        hipLaunchKernelGGL((rans_encode_pipe_kernel<true, 32, false>), few_grid, pipe_block, 0, st, a);
      } else {
        hipLaunchKernelGGL((rans_encode_pipe_kernel<true, 16, false>), few_grid, pipe_block, 0, st, a);
      }
    } else if (a.bits && (a.units_per_stream == 1 ? !encode_depths_in_pairs(a.n_units) : a.n_units <= kFewChunks)) {
      launch_encode_depths(a, n_streams, st, trace);
    } else if (a.bits && a.units_per_stream == 1) {
      trace.kernel("rans_encode_pair_kernel<1, true, 2, true>");
      hipLaunchKernelGGL((rans_encode_pair_kernel<1, true, 2, true>), dim3((unsigned)((a.n_units + 1) / 2)), dim3(64), 0, st, a);
    } else if (a.units_per_stream == 1) {
      // many whole streams: two streams per wavefront, one wavefront per workgroup
      const int64_t pairs = (a.n_units + 1) / 2;
      if (pairs > 8 * kComputeUnits && pairs <= 11 * kComputeUnits) {  // all resident at once with the smaller stages
        trace.kernel("rans_encode_pair_kernel<1, true, 2, false>");
        hipLaunchKernelGGL((rans_encode_pair_kernel<1, true, 2>), dim3((unsigned)pairs), dim3(64), 0, st, a);
      } else {
        trace.kernel("rans_encode_pair_kernel<1, true, 4, false>");
        hipLaunchKernelGGL((rans_encode_pair_kernel<1, true, 4>), dim3((unsigned)pairs), dim3(64), 0, st, a);
      }
    } else {
      // chunks: two chunks of full length per wavefront; an odd one and a shorter last chunk take a wavefront each
      const int64_t n_full = a.syms_per_stream / a.unit_syms;
      const int64_t slots = n_full / 2 + (n_full & 1) + (n_full < a.units_per_stream ? 1 : 0);
      int w = 1;
      while (w < kPairMaxWaves && 2 * w <= slots) w *= 2;
      a.pair_wgs_per_stream = (uint32_t)((slots + w - 1) / w);
      const unsigned grid = (unsigned)(n_streams * a.pair_wgs_per_stream);  // at most the grid checked above
      trace.kernel("rans_encode_pair_kernel<%d, false, %d, %s>", w, a.bits ? 2 : 4, a.bits ? "true" : "false");
      if (a.bits) {
        switch (w) {
          case 1: hipLaunchKernelGGL((rans_encode_pair_kernel<1, false, 2, true>), dim3(grid), dim3(64), 0, st, a); break;
          case 2: hipLaunchKernelGGL((rans_encode_pair_kernel<2, false, 2, true>), dim3(grid), dim3(128), 0, st, a); break;
          default: hipLaunchKernelGGL((rans_encode_pair_kernel<4, false, 2, true>), dim3(grid), dim3(256), 0, st, a); break;
        }
      } else {
        switch (w) {
          case 1: hipLaunchKernelGGL((rans_encode_pair_kernel<1, false>), dim3(grid), dim3(64), 0, st, a); break;
          case 2: hipLaunchKernelGGL((rans_encode_pair_kernel<2, false>), dim3(grid), dim3(128), 0, st, a); break;
          default: hipLaunchKernelGGL((rans_encode_pair_kernel<4, false>), dim3(grid), dim3(256), 0, st, a); break;
        }
      }
    }
  }
  return launch_status();
}

int decode_impl(const uint16_t *freq, const uint32_t *states, const uint16_t *words, uint64_t words_len,
                const uint64_t *word_off, const uint32_t *n_words, int64_t n_streams, int64_t syms_per_stream,
                int32_t chunk_syms, uint8_t *symbols, uint32_t *status, void *stream, RansArgs a,
                const plc_restart *restart = nullptr, bool rest = true, uint32_t *tile_cnt = nullptr,
                TileCounts *counts = nullptr) {
  int rc = check_common(n_streams, syms_per_stream, chunk_syms, &a);
  if (!rc) rc = check_restart(restart, true, &a);
  if (rc) return rc;
  if (!symbols || !freq || !states || !word_off || !n_words || !status) return PLC_ERR_INVALID;
  if (words_len > 0 && !words) return PLC_ERR_INVALID;
  if (reinterpret_cast<uintptr_t>(freq) % 8 || reinterpret_cast<uintptr_t>(words) % 2) return PLC_ERR_INVALID;
  a.sym_out = symbols;
  a.freq = freq;
  a.states_in = states;
  a.words_in = words;
  a.words_len = words_len;
  a.word_off = word_off;
  a.n_words_in = n_words;
  a.status = status;
  hipStream_t st = static_cast<hipStream_t>(stream);
  {
    TraceScope trace(PLC_TRACE_RANS_DECODE, st);
    if (a.pieces && !a.bits && n_streams * a.pieces <= kChainMaxPieces) {
      a.wgs_per_stream = (uint32_t)a.pieces;
      trace.kernel("rans_decode_chain_kernel<0, false, 4>");
      hipLaunchKernelGGL((rans_decode_chain_kernel<0, false>), dim3((unsigned)(n_streams * a.pieces)), dim3(128), 0, st, a);
    } else if (a.pieces || a.units_per_stream > 1) {
      // (pieces begin at whole tiles if the stream is whole tiles: the encoder's rounds are as long as a tile)
      const bool tiles = tile_cnt && (a.pieces ? syms_per_stream : a.unit_syms) % kTileSyms == 0;
      if (decode_depths_alone(a, tiles)) {
        launch_decode_depths(a, n_streams, st, trace);
      } else {
        if (tiles) {
          a.tile_cnt = tile_cnt;
          counts->counted = true;
        }
        launch_decode_pairs(a, n_streams, st, trace);
      }
    }
    if (a.pieces && counts && (counts->counted || !rest)) {
      counts->piece_state = a.piece_state;
      counts->pieces = a.pieces;
      counts->rest_left = !rest;
    }
    if (a.pieces) a = again_args(a);
    if (a.units_per_stream == 1 && !(a.verified_pieces && !rest)) launch_decode_streams(a, st, a.verified_pieces ? nullptr : &trace);
  }
  return launch_status();
}

}  // namespace

int rans_decode_counting(const uint16_t *freq, const uint32_t *states, const uint16_t *words, uint64_t words_len,
                         const uint64_t *word_off, const uint32_t *n_words, int64_t n_streams,
                         int64_t syms_per_stream, int32_t chunk_syms, int32_t syms_per_pos,
                         int32_t streams_per_session, const uint8_t *bits, int32_t n_tables,
                         const plc_restart *restart, bool rest, uint8_t *symbols, uint32_t *tile_cnt,
                         TileCounts *counts, uint32_t *status, void *stream) {
  *counts = TileCounts{};
  RansArgs a = {};
  if (bits) {
    const int rc = check_depths(syms_per_stream, chunk_syms, syms_per_pos, streams_per_session, bits, n_tables, &a);
    if (rc) return rc;
  }
  return decode_impl(freq, states, words, words_len, word_off, n_words, n_streams, syms_per_stream, chunk_syms,
                     symbols, status, stream, a, restart, rest, tile_cnt, counts);
}

bool decode_fused_supported(int64_t n_streams, int64_t syms_per_stream, int k, bool cond, bool per_depth, int32_t points) {
  if (points && (per_depth || (k <= 8 && pieces_in_two_calls(n_streams, syms_per_stream, k, cond, points)))) return false;
  // Candidates that fit the registers of one wavefront kRecDepth batches deep, and whole chunks.  As to
  // the number of streams: two or three workgroups per compute unit run at a time, and a round takes its
  // chain's time or the HBM time of its reconstruction, whichever is longer.  With the weighted mean the two
  // are of a size, so the kernel beats the many-unit decoder followed by the reconstruction kernel however
  // many rounds there are (5120 streams: 7.9 against 10.9 ms; 16,384 streams with k = 8: 31 against 42 ms).
  // The token-conditional reconstruction moves a quarter of the bytes, so there is little to hide: with
  // k <= 4, where three workgroups share a compute unit, the kernel still wins (5120 streams: 7.0 against
  // 7.9 ms); with more candidates (two workgroups) the many-unit decoder's shorter total wins from some eight
  // rounds on (16,384 streams, k = 8: 28.4 against 22.5 ms): 2048 streams at most.  With one table per depth a
  // round is 256 workgroups, and the bound of that decoder applies.
  // (Streams in pieces have a line of their own besides: pieces_in_two_calls.)
  const int64_t most = per_depth ? kDepthsMaxUnits : (cond && k > 4) ? 2048 : INT64_MAX;
  return n_streams >= 1 && n_streams <= most && k >= 1 && k <= 8 && syms_per_stream >= kChunk &&
         syms_per_stream % kChunk == 0;
}

int rans_decode_fused(const uint16_t *freq, const uint32_t *states, const uint16_t *words, uint64_t words_len,
                      const uint64_t *word_off, const uint32_t *n_words, int64_t n_streams,
                      int64_t syms_per_stream, int32_t n_tables, uint8_t *symbols, const ReconView &recon,
                      const plc_restart *restart, uint32_t *status, hipStream_t st, FusedCall call) {
  RansArgs a = {};
  int rc = check_common(n_streams, syms_per_stream, 0, &a);
  if (!rc) rc = check_restart(restart, true, &a);
  if (rc) return rc;
  if (!decode_fused_supported(n_streams, syms_per_stream, recon.k, recon.chosen != nullptr, recon.bits != nullptr,
                              restart && call == kFusedDecode ? restart->per_stream : 0))
    return PLC_ERR_INVALID;
  if (!symbols || !freq || !states || !word_off || !n_words || !status) return PLC_ERR_INVALID;
  if (words_len > 0 && !words) return PLC_ERR_INVALID;
  if (reinterpret_cast<uintptr_t>(freq) % 8 || reinterpret_cast<uintptr_t>(words) % 2) return PLC_ERR_INVALID;
  if ((int64_t)recon.L * recon.H < 1 || n_streams % ((int64_t)recon.L * recon.H)) return PLC_ERR_INVALID;
  if (syms_per_stream != 2ll * recon.n * recon.d8 * kChunk) return PLC_ERR_INVALID;
  if (recon.bits) {  // one table per bit depth: a position is the 2 * d symbols of its K and V rows
    if (!recon.chosen || !(recon.range > 0.0f)) return PLC_ERR_INVALID;
    rc = check_depths(syms_per_stream, 0, 2 * recon.d8 * kChunk, recon.L * recon.H, recon.bits, n_tables, &a);
    if (rc) return rc;
  }
  if (call == kFusedCheck) return PLC_OK;
  a.sym_out = symbols;
  a.freq = freq;
  a.states_in = states;
  a.words_in = words;
  a.words_len = words_len;
  a.word_off = word_off;
  a.n_words_in = n_words;
  a.status = status;
  a.recon = recon;
  {
    std::optional<TraceScope> trace;  // (the rest: the call has been traced)
    if (call == kFusedDecode) trace.emplace(PLC_TRACE_RANS_DECODE, st);
    const dim3 block(192);
    const size_t lds = depths_lds_bytes(a.n_tables);
    if (call == kFusedRest) {
      a = again_args(a);
    } else {
      merge_pieces_for(&a, n_streams, recon.k);
    }
    // With pieces: those, then a launch over the streams, in which one whose pieces agree is left alone.
    for (int round = a.pieces ? 0 : 1; round < 2; ++round) {
      const int64_t n_units = a.pieces ? n_streams * a.pieces : n_streams;
      const dim3 grid((unsigned)n_units);
      if (a.pieces) a.wgs_per_stream = (uint32_t)a.pieces;
      if (trace && !a.verified_pieces) {
        const bool compact = recon.k <= kCompactMaxK && n_units > kDenseStreams;
        if (recon.bits || compact) {
          trace->kernel("rans_decode_depths_kernel<%d, %d>", (int)recon.k, recon.bits ? 0 : recon.chosen ? 2 : 1);
        } else {
          const bool three = !recon.chosen && recon.k <= kDenseMaxK && n_units > kDenseStreams;
          trace->kernel("rans_decode_chain_kernel<%d, %s, %d>", (int)recon.k, recon.chosen ? "true" : "false", three ? 3 : 4);
        }
      }
      switch (recon.k) {
#define PLC_CASE(K)                                                                              \
    case K:                                                                                        \
      if (recon.bits) {                                                                            \
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&rans_decode_depths_kernel<K>),   \
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);           \
        hipLaunchKernelGGL(rans_decode_depths_kernel<K>, grid, dim3(depths_threads(K)), lds, st, a); \
      } else if (K <= kCompactMaxK && n_units > kDenseStreams) {                                   \
        const size_t lds1 = depths_lds_bytes(1);                                                \
        if (recon.chosen) {                                                                        \
          hipLaunchKernelGGL((rans_decode_depths_kernel<(K <= kCompactMaxK ? K : 1), 2>), grid, block, lds1, st, a); \
        } else {                                                                                   \
          hipLaunchKernelGGL((rans_decode_depths_kernel<(K <= kCompactMaxK ? K : 1), 1>), grid, block, lds1, st, a); \
        }                                                                                          \
      } else if (recon.chosen) {                                                                   \
        hipLaunchKernelGGL((rans_decode_chain_kernel<K, true>), grid, block, 0, st, a);            \
      } else if (K <= kDenseMaxK && n_units > kDenseStreams) {                                     \
        hipLaunchKernelGGL((rans_decode_chain_kernel<(K <= kDenseMaxK ? K : 1), false, 3>), grid, block, 0, st, a); \
      } else {                                                                                     \
        hipLaunchKernelGGL((rans_decode_chain_kernel<K, false>), grid, block, 0, st, a);           \
      }                                                                                            \
      break;
        PLC_CASE(1) PLC_CASE(2) PLC_CASE(3) PLC_CASE(4) PLC_CASE(5) PLC_CASE(6) PLC_CASE(7) PLC_CASE(8)
#undef PLC_CASE
        default: return PLC_ERR_INVALID;
      }
      if (a.pieces) a = again_args(a);
    }
  }
  return launch_status();
}

}  // namespace plc

extern "C" int32_t plc_restart_points(int64_t n_streams, int64_t syms_per_stream, int32_t chunk_syms) {
  if (n_streams < 1 || n_streams > kPipeMaxUnits || syms_per_stream < 1 || syms_per_stream >= (1ll << 31) - 1024 ||
      chunk_syms != 0)
    return 0;
  const int32_t rounds = restart_rounds(syms_per_stream);
  const int32_t most = rounds / kPieceMinRounds;
  int32_t points = (int32_t)(kPiecesWanted / n_streams);
  if (points > most) points = most;
  return points < 2 ? 0 : points;
}

extern "C" int32_t plc_decode_one_kernel(int64_t n_streams, int64_t syms_per_stream, int32_t chunk_syms, int32_t k,
                                         int32_t cond, int32_t per_depth, int32_t per_stream) {
  if (n_streams < 1 || syms_per_stream < 1 || syms_per_stream >= (1ll << 31) - 1024 || chunk_syms != 0 ||
      (per_stream && (per_stream < 2 || n_streams > kPipeMaxUnits)))
    return 0;
  return decode_fused_supported(n_streams, syms_per_stream, k, cond != 0, per_depth != 0, per_stream);
}

extern "C" int plc_rans_encode_restart(const uint8_t *symbols, int64_t n_streams, int64_t syms_per_stream,
                                       int32_t chunk_syms, const uint16_t *freq, uint32_t *states, uint16_t *words,
                                       const uint64_t *word_off, uint64_t word_cap_per_unit, uint32_t *n_words,
                                       const plc_restart *restart, uint32_t *status, void *stream) {
  return encode_impl(symbols, n_streams, syms_per_stream, chunk_syms, freq, states, words, word_off,
                     word_cap_per_unit, n_words, status, stream, RansArgs{}, restart);
}

extern "C" int plc_rans_encode(const uint8_t *symbols, int64_t n_streams, int64_t syms_per_stream,
                               int32_t chunk_syms, const uint16_t *freq, uint32_t *states, uint16_t *words,
                               const uint64_t *word_off, uint64_t word_cap_per_unit, uint32_t *n_words,
                               uint32_t *status, void *stream) {
  return plc_rans_encode_restart(symbols, n_streams, syms_per_stream, chunk_syms, freq, states, words, word_off,
                                 word_cap_per_unit, n_words, nullptr, status, stream);
}

extern "C" int plc_rans_decode_restart(const uint16_t *freq, const uint32_t *states, const uint16_t *words,
                                       uint64_t words_len, const uint64_t *word_off, const uint32_t *n_words,
                                       int64_t n_streams, int64_t syms_per_stream, int32_t chunk_syms,
                                       const plc_restart *restart, uint8_t *symbols, uint32_t *status, void *stream) {
  return decode_impl(freq, states, words, words_len, word_off, n_words, n_streams, syms_per_stream, chunk_syms,
                     symbols, status, stream, RansArgs{}, restart);
}

extern "C" int plc_rans_decode(const uint16_t *freq, const uint32_t *states, const uint16_t *words,
                               uint64_t words_len, const uint64_t *word_off, const uint32_t *n_words,
                               int64_t n_streams, int64_t syms_per_stream, int32_t chunk_syms, uint8_t *symbols,
                               uint32_t *status, void *stream) {
  return plc_rans_decode_restart(freq, states, words, words_len, word_off, n_words, n_streams, syms_per_stream,
                                 chunk_syms, nullptr, symbols, status, stream);
}

extern "C" int plc_rans_encode_bucketed_restart(const uint8_t *symbols, int64_t n_streams, int64_t syms_per_stream,
                                                int32_t chunk_syms, int32_t syms_per_pos, int32_t streams_per_session,
                                                const uint8_t *bits, int32_t n_tables, const uint16_t *freq,
                                                uint32_t *states, uint16_t *words, const uint64_t *word_off,
                                                uint64_t word_cap_per_unit, uint32_t *n_words,
                                                const plc_restart *restart, uint32_t *status, void *stream) {
  RansArgs a = {};
  const int rc = check_depths(syms_per_stream, chunk_syms, syms_per_pos, streams_per_session, bits, n_tables, &a);
  if (rc) return rc;
  return encode_impl(symbols, n_streams, syms_per_stream, chunk_syms, freq, states, words, word_off,
                     word_cap_per_unit, n_words, status, stream, a, restart);
}

extern "C" int plc_rans_encode_bucketed(const uint8_t *symbols, int64_t n_streams, int64_t syms_per_stream,
                                        int32_t chunk_syms, int32_t syms_per_pos, int32_t streams_per_session,
                                        const uint8_t *bits, int32_t n_tables, const uint16_t *freq,
                                        uint32_t *states, uint16_t *words, const uint64_t *word_off,
                                        uint64_t word_cap_per_unit, uint32_t *n_words, uint32_t *status,
                                        void *stream) {
  return plc_rans_encode_bucketed_restart(symbols, n_streams, syms_per_stream, chunk_syms, syms_per_pos,
                                          streams_per_session, bits, n_tables, freq, states, words, word_off,
                                          word_cap_per_unit, n_words, nullptr, status, stream);
}

extern "C" int plc_rans_decode_bucketed_restart(const uint16_t *freq, const uint32_t *states, const uint16_t *words,
                                                uint64_t words_len, const uint64_t *word_off, const uint32_t *n_words,
                                                int64_t n_streams, int64_t syms_per_stream, int32_t chunk_syms,
                                                int32_t syms_per_pos, int32_t streams_per_session, const uint8_t *bits,
                                                int32_t n_tables, const plc_restart *restart, uint8_t *symbols,
                                                uint32_t *status, void *stream) {
  RansArgs a = {};
  const int rc = check_depths(syms_per_stream, chunk_syms, syms_per_pos, streams_per_session, bits, n_tables, &a);
  if (rc) return rc;
  return decode_impl(freq, states, words, words_len, word_off, n_words, n_streams, syms_per_stream, chunk_syms,
                     symbols, status, stream, a, restart);
}

extern "C" int plc_rans_decode_bucketed(const uint16_t *freq, const uint32_t *states, const uint16_t *words,
                                        uint64_t words_len, const uint64_t *word_off, const uint32_t *n_words,
                                        int64_t n_streams, int64_t syms_per_stream, int32_t chunk_syms,
                                        int32_t syms_per_pos, int32_t streams_per_session, const uint8_t *bits,
                                        int32_t n_tables, uint8_t *symbols, uint32_t *status, void *stream) {
  return plc_rans_decode_bucketed_restart(freq, states, words, words_len, word_off, n_words, n_streams,
                                          syms_per_stream, chunk_syms, syms_per_pos, streams_per_session, bits,
                                          n_tables, nullptr, symbols, status, stream);
}
