// TurboAttention decode on gfx950 (Algorithm 2) over the paged int4/int2
// cache, with an optional split of the KV range into chunks (merged by
// k_decode_combine).
//
// One wave, or a work-group of W = 2, 4 or 8 waves with a group each (further
// below, the same results bit for bit), owns one (sequence b, KV head kh, chunk
// s) and all G query heads of kh (padded to GP = 1, 2, 4, 8 or 16 rows).  Per
// 64-token group:
//
//  * QK^T on the raw codes.  With w_c = q_c * s_c split exactly as
//    w = 128*hi + lo (lo in 0..127, hi in -75..74, both int8), the int32
//    accumulator of Algorithm 2, sum_c q_c (code_c s_c + z_c), equals
//    128 * sum hi*code + sum lo*code + sum_c q_c z_c  (eq. integer_inference
//    of Sec. 2.3 applied to the step-2 dequantization code*s + z).  Two
//    16x16x64 i8 MFMAs per k-step contract the unpacked 4/2-bit codes with
//    hi and lo; the zero-point term enters as the initial accumulator.  The
//    codes are only unpacked (mask/shift), never multiplied.
//    S^T = K q^T: A-operand row m of m-block mb holds token
//    16*(m>>2) + 4*mb + (m&3), so lane (n + 16*g4), register r of m-block mb
//    is the score of query row n and token 16*g4 + 4*mb + r.
//  * The GP x 64 scores go through LDS to a compact layout (lane L: row
//    L / (64/GP), GP consecutive tokens) where the SAS online softmax of
//    Algorithm 2 runs on useful values only; row reductions are DPP /
//    permlane within the row's 64/GP lanes.
//  * Q(P~) bytes return through LDS as the A-operand of O = P V (16x16x64
//    MFMA, K index = the tokens of page kg in the order the V codes unpack
//    to); the B-operand is the 16 codes of a channel in page kg, one
//    contiguous 8-byte (int4) / 4-byte (int2) run of the channel-major page.
//    PV is taken on the raw V codes and corrected per channel with
//    s * acc + z * sum(Q(P~)) (same identity), which equals the int32
//    accumulator over the int8-expanded V.  The GP x 128 result goes through
//    LDS to the compact layout (lane L: row L / (64/GP), 2*GP channels) for
//    the accumulator update.
//  * The accumulator is kept as O = beta * Ost (per-row beta) so the
//    rescale by SAS(m_old - m_new) touches one value per row.
//  * Every code byte is read once per launch, through streaming loads: the
//    waves spend their time waiting on these loads.
#include "turbo_common.h"
#include "stream_loads.h"

namespace turbo {

struct DecodeArgs {
  const uint4* q;            // fp16 [B][Hq][128]
  const uint8_t* pages;
  const int8_t* gmeta;       // [slots][Hkv][4][128]
  const float* gscale;       // [slots][Hkv][2]
  long num_pages, num_slots;
  int npages32, nslots32;    // min(num_pages, INT_MAX), min(num_slots, INT_MAX)
  int page_bytes;
  unsigned long long int2_mask;
  const int* seq_lens;       // [B]
  const int* block_table;    // [B][4*max_groups]
  const int* group_table;    // [B][max_groups]
  int max_groups;
  int B, Hq, Hkv, G;
  float sm_scale;
  int split;                 // groups per chunk; 0: decode_default_split of each sequence
  int nsplit;                // group chunks per (sequence, KV head) in the grid
  int nws;                   // workspace slots per row: nsplit, plus one with a tail
  float* ws;                 // [B][Hq][nws][132]: m, l, -, -, O[128] of each chunk
  const int8_t* tk;          // Sec. 3.3 buffer (null: none): [B][Hkv][64][128]
  const int8_t* tv;          //   [B][Hkv][128][64]
  const float* tscale;       //   [B][Hkv][2]
  uint2* o;                  // fp16 [B][Hq][128]
  float* lse;                // [B][Hq] or null
  unsigned char* trace;      // test hook: integers of (sequence tr_b, query head tr_h, group tr_g)
  int tr_b, tr_h, tr_g;
};

constexpr int kWsStride = 132;  // m, l, two pad words, O[128] (16-byte aligned)
constexpr int kWsO = 4;


// Chunk length (groups) that kv_split_groups = 0 gives a sequence of ng
// cached groups: one chunk up to 32 groups, chunks of 32 up to 128 groups,
// four equal chunks beyond.  It depends on the sequence alone, so a
// sequence's result does not depend on the batch it is decoded in.
__host__ __device__ constexpr int decode_default_split(int ng) {
  return ng <= 32 ? (ng > 0 ? ng : 1) : (ng <= 128 ? 32 : ceil_div(ng, 4));
}

// Chunks of a sequence with ng groups (chunk length split > 0 or the
// default rule), and the most any sequence of at most max_groups groups has.
__host__ __device__ constexpr int decode_chunks(int ng, int split) {
  return ng <= 0 ? 0 : ceil_div(ng, split > 0 ? split : decode_default_split(ng));
}
__host__ __device__ constexpr int decode_max_chunks(int max_groups, int split) {
  return max_groups <= 0 ? 0
         : split > 0     ? ceil_div(max_groups, split)
                         : (max_groups <= 32 ? 1 : (max_groups <= 128 ? ceil_div(max_groups, 32) : 4));
}

// The cached groups and buffered tokens decode attends for sequence b.
struct DecodeSeq {
  int ng;      // cached groups
  int split;   // chunk length
  int nchunk;  // group chunks
  int nt;      // buffered tokens (0 without a buffer)
  int nparts;  // nchunk + (nt > 0): states to merge
};

__device__ __forceinline__ DecodeSeq decode_seq(const DecodeArgs& a, int b) {
  DecodeSeq q;
  const int len = a.seq_lens[b];
  q.ng = min(max(len / 64, 0), a.max_groups);
  q.split = a.split > 0 ? a.split : decode_default_split(q.ng);
  q.nchunk = decode_chunks(q.ng, a.split);
  q.nt = a.tk ? min(max(len - 64 * q.ng, 0), 63) : 0;
  q.nparts = q.nchunk + (q.nt > 0);
  return q;
}

// The chunk s of (sequence b, KV head kh) that a work-group takes.  Work-groups go
// to the eight XCDs, and within one to its shader engines and CUs, in turn: with two,
// four, eight .. chunks per head in order, the first chunks of all heads fall on a
// few of them.  Where the tables are wider than the sequences need, those are the
// only ones that are not empty.  So the chunks of a sequence that leaves some empty
// are rotated by b: 64 sequences of 2000 tokens in tables of 512 groups, 64/8 heads,
// 104 us in order, 62 rotated; 256 of 1000, 32/8 heads, 125 / 57; 64 of 1000 in chunks
// of 16 groups 204 / 39; ragged batches gain 3 to 10 %.  By sequence, not by head,
// since the heads share the chunk's table entries.  The digits to the base 4 (2) of b
// are summed, so that the rotation does not repeat in step with a power of two.
// Sequences that fill their chunks stay in order: rotated, equal batches lost up to
// 5 %, and so did all with 6, 10, .. chunks.
__device__ __forceinline__ DecodeSeq decode_place(const DecodeArgs& a, int& b, int& kh, int& s) {
  const unsigned n = a.nsplit;
  unsigned u = blockIdx.x, j = 0;
  if ((n & (n - 1)) == 0) {  // mostly one, two or four: no division
    u >>= __builtin_ctz(n);
    j = blockIdx.x & (n - 1);
  } else {
    u /= n;
    j = blockIdx.x - u * n;
  }
  b = (int)(u / (unsigned)a.Hkv);
  kh = (int)u - b * a.Hkv;
  const DecodeSeq q = decode_seq(a, b);
  if (q.nchunk < (int)n && (n == 2 || n % 4 == 0)) {
    const unsigned x = (unsigned)b;
    j += n == 2 ? (unsigned)__builtin_popcount(x) : x + (x >> 2) + (x >> 4) + (x >> 6);
    j = (n & (n - 1)) == 0 ? j & (n - 1) : j % n;
  }
  s = (int)j;
  return q;
}

// o = 0 and lse = -inf for the G rows of (b, kh): a sequence with nothing to
// attend.
__device__ void decode_write_empty(const DecodeArgs& a, int b, int kh) {
  for (int r = 0; r < a.G; ++r) {
    const long bh = (long)b * a.Hq + kh * a.G + r;
    reinterpret_cast<unsigned*>(a.o)[bh * 64 + (threadIdx.x & 63)] = 0u;
    if (a.lse && (threadIdx.x & 63) == 0) a.lse[bh] = -INFINITY;
  }
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));


// Reductions over the 64/GP consecutive lanes of a compact row (every lane
// of the row receives the result).
// Integer forms (the DPP moves fuse into the max / add).
template <int LPR>
__device__ __forceinline__ int row_max_i(int v) {
  if (LPR >= 2) v = max(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true));
  if (LPR >= 4) v = max(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true));
  if (LPR >= 8) v = max(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true));
  if (LPR >= 16) v = max(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true));
  if (LPR >= 32) {
    auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    v = max((int)r[0], (int)r[1]);
  }
  if (LPR >= 64) {
    auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    v = max((int)r[0], (int)r[1]);
  }
  return v;
}

template <int LPR>
__device__ __forceinline__ int row_sum_i(int v) {
  if (LPR >= 2) v += __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true);
  if (LPR >= 4) v += __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true);
  if (LPR >= 8) v += __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true);
  if (LPR >= 16) v += __builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true);
  if (LPR >= 32) {
    auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    v = (int)r[0] + (int)r[1];
  }
  if (LPR >= 64) {
    auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    v = (int)r[0] + (int)r[1];
  }
  return v;
}

template <int LPR>
__device__ __forceinline__ float row_sum(float v) {
  if (LPR >= 2) v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, false));
  if (LPR >= 4) v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xf, 0xf, false));
  if (LPR >= 8) v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xf, 0xf, false));
  if (LPR >= 16) v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xf, 0xf, false));
  if (LPR >= 32) {
    const unsigned u = __float_as_uint(v);
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  if (LPR >= 64) v = add_xor32(v);
  return v;
}

// Position of page token j in the order the V codes unpack to (see the PV
// step): int4 gives tokens {0,2,4,6},{1,3,5,7},{8,..},{9,..}; int2 gives
// {0,4,8,12},{1,5,9,13},...
template <int BITS>
__device__ __forceinline__ int vpos(int j) {
  if (BITS == 4) return (j & 8) + ((j & 1) << 2) + ((j & 7) >> 1);
  return 4 * (j & 3) + (j >> 2);
}

// LDS row strides (in ints) chosen for the bank pattern of the exchanges
// (64 banks of 4 bytes):
//  * scores: one row per MFMA column n (16), 68 ints apart, so the 16 lanes
//    of a column block store to 16 different banks;
//  * PV accumulators: GP + 2 ints per channel (an odd number of 8-byte
//    pairs), so lanes L = 0..15 reading channel rows 2L (+1) hit distinct
//    banks.  Lanes whose MFMA rows are unused (4*g4 >= GP) store to a
//    separate area instead, at one address for every channel block.
constexpr int kSbufStride = 68;
template <int GP>
constexpr int kObufStride = GP < 4 ? GP : GP + 2;
template <int GP>
constexpr int kOdumRows = GP < 4 ? 1 : (GP < 16 ? 64 - 4 * GP : 1);

// Rows of the w = q * s^int exchange: the GP query rows (at least 4, the
// rows one writer pass covers).
template <int GP>
constexpr int kWRows = GP < 4 ? 4 : GP;

template <int GP>
struct DecodeLds {
  float lut[8];
  float sq[16];
  __attribute__((aligned(16))) unsigned char whi[kWRows<GP>][128];  // hi bytes of w, B-operand order
  __attribute__((aligned(16))) unsigned char wlo[kWRows<GP>][128];  // lo bytes of w
  int wbias[kWRows<GP>];                // sum_c q_c z_c of each row
  signed char qbuf[kWRows<GP>][128];    // the int8 query rows
  __attribute__((aligned(16))) int sbuf[16][kSbufStride];  // scores, row n; rows >= GP unused
  unsigned char pbuf[GP + 1][64];   // Q(P~), per page in V-unpack order; row GP: read by
                                    // unused rows (their products are never kept)
  __attribute__((aligned(16))) int obuf[128][kObufStride<GP>];  // PV accumulators, channel-major
  __attribute__((aligned(16))) int odum[kOdumRows<GP>][4];     // stores of unused MFMA rows
  float4 rowv[GP];                  // per row: g = s_P s_V / beta, sum Q(P~), renorm, -
};

// K side of one group, loaded one group ahead of its step.  The table
// entries, the slot and the float scales are wave-uniform.  A group that is
// not live (past the chunk) or has an out-of-range entry (a caller error; it
// is skipped) still issues every load, from page 0 and slot 0, so that the
// number of memory operations in flight is the same on every path and the
// waits before each use stay exact.
//
// A-operand row m of m-block mb holds token 16*mb + m, so each m-block reads
// one page: its base address is wave-uniform and the lane adds its own
// offset (token row m, channel block g4).
template <int BITS>
struct GroupK {
  bool ok;
  int pg[4];                // page of each 16-token quarter (clamped into range)
  int vpg;                  // page of quarter g4 (this lane's PV K-chunk), clamped
  int slot;                 // group slot (clamped)
  float skg, svg;           // float scales s_K, s_V of the group
  unsigned kraw[4][BITS];   // K codes of the lane's 4 A-operand rows (32 channels each)
  // s^int and z^int bytes of the channels the lane writes w for (see
  // decode_groups): int4: 8 channels (2 dwords each), int2: their 16-channel
  // block (4 dwords each)
  unsigned ws[BITS == 4 ? 2 : 4], wz[BITS == 4 ? 2 : 4];
};

// V side of one group, loaded by the group's own step after its QK^T.
template <int BITS>
struct GroupV {
  unsigned vraw[8][BITS / 2];  // V codes of channel 16*cb + n in page g4
  unsigned vs4, vz4;           // V scales / zeros of channels 2L&~3 .. +3 (aligned dwords)
};

// The K codes of a group, and the K scales and zeros the lane needs.
template <int BITS>
__device__ __forceinline__ void load_codes(const DecodeArgs& a, int kh, int head_off,
                                           GroupK<BITS>& K) {
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, g4 = lane >> 4, m = lane & 15;
  const int8_t* meta = a.gmeta + ((long)K.slot * a.Hkv + kh) * 512;
  const int koff = head_off + m * 16 * BITS + 4 * BITS * g4;
  // the codes are read once per launch: streaming loads.  The group's
  // metadata stays on ordinary loads, since its block is read twice (the K
  // scales and zeros here, the V ones by load_v)
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) {
    const uint8_t* krow = a.pages + (long)K.pg[mb] * a.page_bytes + koff;
    if constexpr (BITS == 4) {
      const u32x4_t x = load_nt4(krow);
      K.kraw[mb][0] = x.x; K.kraw[mb][1] = x.y; K.kraw[mb][2] = x.z; K.kraw[mb][3] = x.w;
    } else {
      const u32x2_t x = load_nt2(krow);
      K.kraw[mb][0] = x.x; K.kraw[mb][1] = x.y;
    }
  }
  // the lane writes w for 16-channel block k >> 1, half k & 1 (k = lane & 15)
  if constexpr (BITS == 4) {
    const uint2 x = *reinterpret_cast<const uint2*>(meta + 8 * n);
    const uint2 z = *reinterpret_cast<const uint2*>(meta + 128 + 8 * n);
    K.ws[0] = x.x; K.ws[1] = x.y;
    K.wz[0] = z.x; K.wz[1] = z.y;
  } else {
    const uint4 x = *reinterpret_cast<const uint4*>(meta + 16 * (n >> 1));
    const uint4 z = *reinterpret_cast<const uint4*>(meta + 128 + 16 * (n >> 1));
    K.ws[0] = x.x; K.ws[1] = x.y; K.ws[2] = x.z; K.ws[3] = x.w;
    K.wz[0] = z.x; K.wz[1] = z.y; K.wz[2] = z.z; K.wz[3] = z.w;
  }
}

// Group g, its table entries and scales read here (scalar loads).
template <int BITS>
__device__ __forceinline__ void load_k(const DecodeArgs& a, int kh, int head_off, const int* bt,
                                       const int* gt, int g, bool live, GroupK<BITS>& K) {
  g = live ? g : 0;
  bool ok = live;
  // the tables are read-only here: read them through the constant address
  // space, which keeps these wave-uniform reads on the scalar unit
  typedef const __attribute__((address_space(4))) int cint;
  const cint* btc = (const cint*)bt;
  const cint* gtc = (const cint*)gt;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int p = btc[4 * g + i];
    ok = ok && p >= 0 && p < a.npages32;
    K.pg[i] = p;
  }
  const int slot = gtc[g];
  ok = ok && slot >= 0 && slot < a.nslots32;
  K.ok = ok;
#pragma unroll
  for (int i = 0; i < 4; ++i) K.pg[i] = ok ? K.pg[i] : 0;
  K.slot = ok ? slot : 0;
  // this lane's V page, read by the lane itself (no per-lane choice among
  // the four uniform values)
  const int vp = bt[4 * g + ((threadIdx.x & 63) >> 4)];
  K.vpg = ok ? vp : 0;
  typedef const __attribute__((address_space(4))) float cfloat;
  const cfloat* gs = (const cfloat*)(a.gscale + ((long)K.slot * a.Hkv + kh) * 2);
  K.skg = gs[0];
  K.svg = gs[1];
  load_codes<BITS>(a, kh, head_off, K);
}

// Table entries and float scales of the wave's next 64 groups, lane i holding
// those of its i-th one: read once per 64 steps with vector loads, so that no
// step waits for a table entry before its code loads can leave, nor for a
// scalar load at its next LDS access (the two share a wait counter).
struct GroupTab {
  int pg[4];      // page of each 16-token quarter, 0 if the group is not live
  int slot;       // group slot, -1 if the group is not live or out of range
  float sk, sv;   // float scales of the group
};

// Lane i: group g + i * W of the sequence whose tables are bt, gt (live below g1).
template <int W>
__device__ __forceinline__ void load_tab(const DecodeArgs& a, int kh, const int* bt, const int* gt,
                                         int g, int g1, GroupTab& T) {
  g += (int)(threadIdx.x & 63) * W;
  const bool live = g < g1;
  g = live ? g : 0;
  bool ok = live;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    T.pg[i] = bt[4 * g + i];
    ok = ok && T.pg[i] >= 0 && T.pg[i] < a.npages32;
  }
  const int slot = gt[g];
  ok = ok && slot >= 0 && slot < a.nslots32;
#pragma unroll
  for (int i = 0; i < 4; ++i) T.pg[i] = ok ? T.pg[i] : 0;
  T.slot = ok ? slot : -1;
  const float* gs = a.gscale + ((long)max(T.slot, 0) * a.Hkv + kh) * 2;
  T.sk = gs[0];
  T.sv = gs[1];
}

// The scales of the i-th group of T.
template <int BITS>
__device__ __forceinline__ void tab_scales(const GroupTab& T, int i, GroupK<BITS>& K) {
  K.skg = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(T.sk), i));
  K.svg = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(T.sv), i));
}

// The i-th group of T (i wave-uniform), but for its scales: T's come one load
// after its slots, and a v_readlane of them in front of the codes' addresses
// makes the codes wait for that load too. tab_scales reads them where they are
// used. 20 x 16/16 int4 heads of ragged <= 16537: 77.1 us with the scales read
// here, 72.9 us with them read at the step's start; 24 x 32/16 mixed 75.4 -> 72.0.
template <int BITS>
__device__ __forceinline__ void load_k(const DecodeArgs& a, int kh, int head_off, const GroupTab& T,
                                       int i, GroupK<BITS>& K) {
  const int g4 = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) K.pg[q] = __builtin_amdgcn_readlane(T.pg[q], i);
  K.slot = __builtin_amdgcn_readlane(T.slot, i);
  K.ok = K.slot >= 0;
  K.slot = max(K.slot, 0);
  // this lane's V page
  const int p01 = g4 & 1 ? K.pg[1] : K.pg[0], p23 = g4 & 1 ? K.pg[3] : K.pg[2];
  K.vpg = g4 & 2 ? p23 : p01;
  load_codes<BITS>(a, kh, head_off, K);
}

template <int BITS>
__device__ __forceinline__ void load_v(const DecodeArgs& a, int kh, int head_off,
                                       const GroupK<BITS>& K, GroupV<BITS>& V) {
  const int lane = threadIdx.x & 63;
  const int n = lane & 15;
  const uint8_t* vrow = a.pages + (long)K.vpg * a.page_bytes + head_off + 256 * BITS + n * 2 * BITS;
#pragma unroll
  for (int cb = 0; cb < 8; ++cb) {
    if constexpr (BITS == 4) {
      const u32x2_t x = load_nt2(vrow + cb * 32 * BITS);
      V.vraw[cb][0] = x.x; V.vraw[cb][1] = x.y;
    } else {
      V.vraw[cb][0] = load_nt1(vrow + cb * 32 * BITS);
    }
  }
  const int8_t* meta = a.gmeta + ((long)K.slot * a.Hkv + kh) * 512;
  V.vs4 = *reinterpret_cast<const unsigned*>(meta + 256 + 4 * (lane >> 1));
  V.vz4 = *reinterpret_cast<const unsigned*>(meta + 384 + 4 * (lane >> 1));
}

// q -> int8 per (b, query head) (Algorithm 2; eq. step1bpq) into the wave's
// LDS: lane (n, g4) codes channels 32*g4 .. 32*g4+31 of row n (zero if n >= G)
template <int GP, bool kTrace>
__device__ __forceinline__ void decode_quant_q(const DecodeArgs& a, float* sqv,
                                               signed char (*qbuf)[128], int b, int kh, int trow) {
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, g4 = lane >> 4;
  const bool rowok = n < a.G;
  int q8w[8];
  uint4 raw[4];
  float amax = 0.0f;
  const uint4* src = a.q + ((long)b * a.Hq + kh * a.G + (rowok ? n : 0)) * 16;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    raw[u] = rowok ? src[4 * g4 + u] : make_uint4(0, 0, 0, 0);
    f16x8_t hv = __builtin_bit_cast(f16x8_t, raw[u]);
#pragma unroll
    for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf((float)hv[e]));
  }
  amax = max_xor16(amax);
  amax = max_xor32(amax);
  float inv = 0.0f, sq = 0.0f;
  if (amax > 0.0f) {
    sq = amax / kQmax;
    inv = kQmax / amax;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    f16x8_t hv = __builtin_bit_cast(f16x8_t, raw[u]);
    int qv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) qv[e] = rne_mul((float)hv[e], inv);
    q8w[2 * u] = pack4(qv[0], qv[1], qv[2], qv[3]);
    q8w[2 * u + 1] = pack4(qv[4], qv[5], qv[6], qv[7]);
  }
  if (g4 == 0) sqv[n] = sq;
  if (n < kWRows<GP>) {
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<int*>(&qbuf[n][32 * g4 + 4 * i]) = q8w[i];
  }
  if (kTrace && trow >= 0 && n == trow) {
#pragma unroll
    for (int i = 0; i < 8; ++i) reinterpret_cast<int*>(a.trace + TURBO_TRACE_Q8)[8 * g4 + i] = q8w[i];
    if (g4 == 0) *reinterpret_cast<float*>(a.trace + TURBO_TRACE_SQ) = sq;
  }
}

// w = q * s^int of the GP query rows, written by all lanes of a wave.
// The QK^T B-operand of lane (n, g4), k-step ks, is 16 bytes: dword j, byte
// i holds channel 32*g4 + c0 + d*i with c0 = 16ks + 8(j>>1) + (j&1) (int4)
// or 16ks + j (int2), the order the K codes unpack to.  Only GP of the 16
// rows n are real, so instead of every lane building its own 32 values,
// lane L builds those of unit U = L + 64t: row U >> 4, 8 channels given by
// k = U & 15 -- dwords j = 2h, 2h+1 (h = k & 1) of block (g4 = k >> 2,
// ks = (k >> 1) & 1) -- and writes their hi/lo bytes to byte 8k of the row.
template <int GP, int BITS>
struct QueryW {
  static constexpr int kU = GP <= 4 ? 1 : GP / 4;  // writer units per lane
  unsigned wq[kU][4];  // 16-bit q pairs (A0,A1) (A2,A3) (B0,B1) (B2,B3)
  int wqn[kU][2];      // the q bytes of dword A (= 2h) and B (= 2h + 1)
  unsigned selA, selZ1, selZ2;  // int2: byte selectors of channel 2h (+1) in the block's dwords

  __device__ __forceinline__ void load(const signed char (*qbuf)[128]) {
    constexpr int d = BITS == 4 ? 2 : 4;
    const int lane = threadIdx.x & 63, k = lane & 15;
    const int cA = BITS == 4 ? 8 * k : 16 * (k >> 1) + 2 * (k & 1);  // channel of dword 2h, byte 0
#pragma unroll
    for (int t = 0; t < kU; ++t) {
      const int r = (lane >> 4) + 4 * t;
      int qa[4], qb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        qa[i] = qbuf[r][cA + d * i];
        qb[i] = qbuf[r][cA + 1 + d * i];
      }
      wq[t][0] = ((unsigned)qa[0] & 0xffffu) | ((unsigned)qa[1] << 16);
      wq[t][1] = ((unsigned)qa[2] & 0xffffu) | ((unsigned)qa[3] << 16);
      wq[t][2] = ((unsigned)qb[0] & 0xffffu) | ((unsigned)qb[1] << 16);
      wq[t][3] = ((unsigned)qb[2] & 0xffffu) | ((unsigned)qb[3] << 16);
      wqn[t][0] = pack4(qa[0], qa[1], qa[2], qa[3]);
      wqn[t][1] = pack4(qb[0], qb[1], qb[2], qb[3]);
    }
    const unsigned h2 = 2u * (unsigned)(k & 1);
    selA = h2 | (0x0cu << 8) | ((4u + h2) << 16) | (0x0cu << 24);
    selZ1 = h2 | ((4u + h2) << 8) | 0x0c0c0000u;
    selZ2 = 0x00000c0cu | (h2 << 16) | ((4u + h2) << 24);
  }

  // hi/lo bytes of w and the zero-point term of group K, for every row
  __device__ __forceinline__ void store(const GroupK<BITS>& K, unsigned char (*whi)[128],
                                        unsigned char (*wlo)[128], int* wbias) const {
    const int lane = threadIdx.x & 63, k = lane & 15;
    // s^int pairs matching wq and z^int bytes matching wqn
    unsigned sA01, sA23, sB01, sB23, zA, zB;
    if constexpr (BITS == 4) {
      sA01 = __builtin_amdgcn_perm(0u, K.ws[0], 0x0c020c00u);
      sA23 = __builtin_amdgcn_perm(0u, K.ws[1], 0x0c020c00u);
      sB01 = __builtin_amdgcn_perm(0u, K.ws[0], 0x0c030c01u);
      sB23 = __builtin_amdgcn_perm(0u, K.ws[1], 0x0c030c01u);
      zA = __builtin_amdgcn_perm(K.wz[1], K.wz[0], 0x06040200u);
      zB = __builtin_amdgcn_perm(K.wz[1], K.wz[0], 0x07050301u);
    } else {
      sA01 = __builtin_amdgcn_perm(K.ws[1], K.ws[0], selA);
      sA23 = __builtin_amdgcn_perm(K.ws[3], K.ws[2], selA);
      sB01 = __builtin_amdgcn_perm(K.ws[1], K.ws[0], selA + 0x00010001u);
      sB23 = __builtin_amdgcn_perm(K.ws[3], K.ws[2], selA + 0x00010001u);
      zA = __builtin_amdgcn_perm(K.wz[1], K.wz[0], selZ1) |
           __builtin_amdgcn_perm(K.wz[3], K.wz[2], selZ2);
      zB = __builtin_amdgcn_perm(K.wz[1], K.wz[0], selZ1 + 0x0101u) |
           __builtin_amdgcn_perm(K.wz[3], K.wz[2], selZ2 + 0x01010000u);
    }
#pragma unroll
    for (int t = 0; t < kU; ++t) {
      const int r = (lane >> 4) + 4 * t;
      const unsigned sp[4] = {sA01, sA23, sB01, sB23};
      unsigned hx[4], lx[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const u16x2 w = __builtin_bit_cast(u16x2, wq[t][u]) * __builtin_bit_cast(u16x2, sp[u]);
        hx[u] = __builtin_bit_cast(unsigned, __builtin_bit_cast(s16x2, w) >> (short)7);
        lx[u] = __builtin_bit_cast(unsigned, w) & 0x007F007Fu;
      }
      *reinterpret_cast<uint2*>(&whi[r][8 * k]) =
          make_uint2(__builtin_amdgcn_perm(hx[1], hx[0], 0x06040200u),
                     __builtin_amdgcn_perm(hx[3], hx[2], 0x06040200u));
      *reinterpret_cast<uint2*>(&wlo[r][8 * k]) =
          make_uint2(__builtin_amdgcn_perm(lx[1], lx[0], 0x06040200u),
                     __builtin_amdgcn_perm(lx[3], lx[2], 0x06040200u));
      // zero-point term sum_c q_c z_c of row r: the unit's 8 channels, then
      // the 16 units of the row (one DPP row; exact: |sum| < 2^24)
      const int bp = __builtin_amdgcn_sdot4(wqn[t][0], (int)zA,
                                            __builtin_amdgcn_sdot4(wqn[t][1], (int)zB, 0, false),
                                            false);
      wbias[r] = row_sum_i<16>(bp);  // every lane of the row: the same value
    }
  }
};

// S^T = K^{q1} q^T on the MFMA: lane (n, g4), register r of sv[mb] holds row n,
// token 16*mb + 4*g4 + r.
template <int BITS>
__device__ __forceinline__ void decode_qk(const GroupK<BITS>& K, const v4i (&bhi)[2],
                                          const v4i (&blo)[2], int bias, int4 (&sv)[4]) {
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) {
    v4i kop[2];
    if (BITS == 4) {
      unsigned u[8];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        u[2 * w] = K.kraw[mb][w] & 0x0F0F0F0Fu;
        u[2 * w + 1] = (K.kraw[mb][w] >> 4) & 0x0F0F0F0Fu;
      }
      kop[0] = v4i{(int)u[0], (int)u[1], (int)u[2], (int)u[3]};
      kop[1] = v4i{(int)u[4], (int)u[5], (int)u[6], (int)u[7]};
    } else {
#pragma unroll
      for (int w = 0; w < 2; ++w)
        kop[w] = v4i{(int)(K.kraw[mb][w] & 0x03030303u),
                     (int)((K.kraw[mb][w] >> 2) & 0x03030303u),
                     (int)((K.kraw[mb][w] >> 4) & 0x03030303u),
                     (int)((K.kraw[mb][w] >> 6) & 0x03030303u)};
    }
    v4i lo = v4i{bias, bias, bias, bias};
    v4i hi = {};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      lo = mfma16x16x64(kop[ks], blo[ks], lo);
      hi = mfma16x16x64(kop[ks], bhi[ks], hi);
    }
    sv[mb] = make_int4((hi[0] << 7) + lo[0], (hi[1] << 7) + lo[1], (hi[2] << 7) + lo[2],
                       (hi[3] << 7) + lo[3]);
  }
}

// PV B-operand: the 16 codes of channel 16*cb + n in page g4.
template <int BITS>
__device__ __forceinline__ v4i v_codes(const GroupV<BITS>& V, int cb) {
  if (BITS == 4) {
    const unsigned x0 = V.vraw[cb][0], x1 = V.vraw[cb][BITS / 2 - 1];
    return v4i{(int)(x0 & 0x0F0F0F0Fu), (int)((x0 >> 4) & 0x0F0F0F0Fu), (int)(x1 & 0x0F0F0F0Fu),
               (int)((x1 >> 4) & 0x0F0F0F0Fu)};
  } else {
    const unsigned x = V.vraw[cb][0];
    return v4i{(int)(x & 0x03030303u), (int)((x >> 2) & 0x03030303u),
               (int)((x >> 4) & 0x03030303u), (int)((x >> 6) & 0x03030303u)};
  }
}

template <int GP, int BITS, bool kTrace>
__device__ __forceinline__ void decode_groups(const DecodeArgs& a, DecodeLds<GP>& L, int b, int kh,
                                              int g0, int g1, int head_off, float& mrow, float& lpart, float& beta,
                                              float (&O)[GP][2], float sq_row, int trow) {
  constexpr int LPR = 64 / GP;  // lanes per compact softmax row
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, g4 = lane >> 4;
  const int rr = lane / LPR, cc = lane % LPR;
  const int nrow = min(n, GP);  // P~ row this lane reads (GP: unused rows)
  // PV store target of this lane (GP >= 4): its 4 MFMA rows of channel
  // 16*cb + n, or (rows 4*g4.. unused) one spare slot for every cb
  const bool orows = 4 * g4 < GP;
  const int odi = min(max((g4 * 16 + n) - 4 * GP, 0), kOdumRows<GP> - 1);
  int* const obase = orows ? &L.obuf[n][4 * g4] : &L.odum[odi][0];
  const int ostep = orows ? 16 * kObufStride<GP> : 0;

  QueryW<GP, BITS> Wq;
  Wq.load(L.qbuf);
  const int wrow = min(n, kWRows<GP> - 1);  // row this lane reads (unused rows: any)

  const int* bt = a.block_table + (long)b * 4 * a.max_groups;
  const int* gt = a.group_table + (long)b * a.max_groups;

  // Two K prefetch buffers used alternately (a copy cur = nxt between groups
  // would be a register move that waits for the prefetch to land).  A step
  // issues K of the next group first and V of its own group after its QK^T
  // MFMAs (V is not held during the QK^T phase); the softmax covers the V
  // latency.
  // The table entries come from lanes (load_tab) with one row only: more rows leave
  // no registers for them.  Worth it for ragged batches, at a small price on some
  // equal ones, which the host cannot tell apart.  us with / without: 100 sequences
  // of up to 1500 tokens, 16 heads, 47.4 / 50.5; 30 of up to 3000, 40 heads, 62.3 /
  // 65.7; 256 of 2048, 16 heads, 181 / 183; 48 of 5873, 16 heads, 94.8 / 92.1; 39 of
  // 18560, 16 heads, 205 / 200.
  constexpr bool kTab = GP == 1;
  GroupTab T;
  if constexpr (kTab) load_tab<1>(a, kh, bt, gt, g0, g1, T);
  auto next_k = [&](int g, GroupK<BITS>& K) {
    if constexpr (kTab) {
      if (g != g0 && ((g - g0) & 63) == 0) load_tab<1>(a, kh, bt, gt, g, g1, T);
      load_k<BITS>(a, kh, head_off, T, (g - g0) & 63, K);
      tab_scales<BITS>(T, (g - g0) & 63, K);
    } else {
      load_k<BITS>(a, kh, head_off, bt, gt, g, g < g1, K);
    }
  };
  GroupK<BITS> KA, KB;
  next_k(g0, KA);
  // Issue priority (s_setprio) is highest from a group's start until its V
  // loads are out, and for the K prefetch, lower in the softmax and lowest in
  // the PV and update steps: a wave on its way to a load goes ahead of the
  // other waves of its SIMD, and a wave nearer its next load ahead of one
  // that has just issued it, so the loads leave earlier.
  auto process = [&](const GroupK<BITS>& cur, int g) {
    if (cur.ok) {
      __builtin_amdgcn_s_setprio(2);
      Wq.store(cur, L.whi, L.wlo, L.wbias);
      wave_sync();
      v4i bhi[2], blo[2];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        bhi[ks] = *reinterpret_cast<const v4i*>(&L.whi[wrow][32 * g4 + 16 * ks]);
        blo[ks] = *reinterpret_cast<const v4i*>(&L.wlo[wrow][32 * g4 + 16 * ks]);
      }
      const int bias = L.wbias[wrow];
      // ---- S^T = K^{q1} q^T on the MFMA, scores to LDS -----------------
      int4 sv[4];
      decode_qk<BITS>(cur, bhi, blo, bias, sv);
      GroupV<BITS> cv;
      load_v<BITS>(a, kh, head_off, cur, cv);
      __builtin_amdgcn_s_setprio(1);
      // lane (n, g4), register r of m-block mb: row n, token 16*mb + 4*g4 + r
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
        *reinterpret_cast<int4*>(&L.sbuf[n][16 * mb + 4 * g4]) = sv[mb];
      const bool trace_g = kTrace && trow >= 0 && g == a.tr_g;  // wave-uniform
      if (trace_g && n == trow) {
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
          reinterpret_cast<int4*>(a.trace + TURBO_TRACE_S)[4 * mb + g4] = sv[mb];
      }
      wave_sync();
      // ---- compact softmax: lane (rr, cc) holds tokens cc*GP .. +GP-1 -----
      bool renorm;
      {
        int si[GP];
        if (GP >= 4) {
#pragma unroll
          for (int e = 0; e < GP; e += 4) {
            const int4 t = *reinterpret_cast<const int4*>(&L.sbuf[rr][cc * GP + e]);
            si[e] = t.x; si[e + 1] = t.y; si[e + 2] = t.z; si[e + 3] = t.w;
          }
        } else {
#pragma unroll
          for (int e = 0; e < GP; ++e) si[e] = L.sbuf[rr][cc * GP + e];
        }
        // c >= 0 (sm_scale > 0, the scales are non-negative) and both
        // roundings of p = float(S) * c are monotonic: the row maximum of p is
        // float(max S) * c, taken on the integers
        const float c = (sq_row * cur.skg) * a.sm_scale;
        float p[GP];
        int imax = si[0];
#pragma unroll
        for (int e = 0; e < GP; ++e) {
          p[e] = (float)si[e] * c;
          imax = max(imax, si[e]);
        }
        const float smax = (float)row_max_i<LPR>(imax) * c;
        const float mnew = fmaxf(mrow, smax);
        float rs = 0.0f;
        int pbits = 0;  // the maximum of the p >= 0, on their bits (same order)
#pragma unroll
        for (int e = 0; e < GP; ++e) {
          p[e] = sas_y(mnew - p[e], L.lut);
          rs += p[e];
          pbits = max(pbits, __float_as_int(p[e]));
        }
        // SAS(m_old - m_new): 0 when m_old = -inf, exactly 1 (e^0) when the
        // row's maximum did not move
        const float alpha = mnew > mrow ? sas_y(mnew - mrow, L.lut) : 1.0f;
        lpart = alpha * lpart + rs;
        mrow = mnew;
        const float pmax = __int_as_float(row_max_i<LPR>(pbits));
        // rescale: O = beta * Ost; renormalize when beta underflows / is 0
        float nbeta = beta * alpha;
        renorm = __builtin_amdgcn_ballot_w64(nbeta < 0x1p-64f) != 0;
        const float rf = renorm ? nbeta : 1.0f;
        if (renorm) nbeta = 1.0f;
        beta = nbeta;
        // Q(P~) with the row's scale pmax/119 (a row whose group lies wholly
        // below the threshold has pmax = 0: inv = 0, Q(P~) = 0, adds nothing)
        const float inv = pmax > 0.0f ? kQmax / pmax : 0.0f;
        int ps = 0;
#pragma unroll
        for (int e = 0; e < GP; ++e) {
          const int code = rne_bits(p[e], inv) & 0xff;
          ps += code;
          const int t = cc * GP + e;  // token of the group
          L.pbuf[rr][16 * (t >> 4) + vpos<BITS>(t & 15)] = (unsigned char)code;
          if (trace_g && rr == trow) a.trace[TURBO_TRACE_P + t] = (unsigned char)code;
        }
        if (trace_g && rr == trow && cc == 0)
          *reinterpret_cast<float*>(a.trace + TURBO_TRACE_PMAX) = pmax;
        const int psum = row_sum_i<LPR>(ps);
        // s_P s_V / beta scales the fp32 accumulator only (no integer depends
        // on it): s_P as pmax times the binary32 1/119
        const float gsc = ((pmax * (1.0f / kQmax)) * cur.svg) * __builtin_amdgcn_rcpf(beta);
        // every lane of the row holds the same values
        L.rowv[rr] = make_float4(gsc, __int_as_float(psum), rf, 0.0f);
      }
      wave_sync();
      __builtin_amdgcn_s_setprio(0);
      // ---- O = Q(P~) V on the raw codes (A = P rows, B = V codes) -------
      const v4i pop = *reinterpret_cast<const v4i*>(&L.pbuf[nrow][16 * g4]);
      // lane (n, g4), register r <-> row 4*g4 + r, channel 16*cb + n
      auto store = [&](int cb, const v4i& acc) {
        if (GP >= 4) {
          int* dst = obase + cb * ostep;
          *reinterpret_cast<int2*>(dst) = make_int2(acc[0], acc[1]);
          *reinterpret_cast<int2*>(dst + 2) = make_int2(acc[2], acc[3]);
        } else if (g4 == 0) {
#pragma unroll
          for (int r = 0; r < GP; ++r) L.obuf[16 * cb + n][r] = acc[r];
        }
      };
      // two channel blocks per step: the second MFMA runs while the first
      // one's result is stored
#pragma unroll
      for (int cb = 0; cb < 8; cb += 2) {
        const v4i acc0 = mfma16x16x64(pop, v_codes<BITS>(cv, cb), v4i{});
        const v4i acc1 = mfma16x16x64(pop, v_codes<BITS>(cv, cb + 1), v4i{});
        store(cb, acc0);
        store(cb + 1, acc1);
      }
      wave_sync();
      // ---- accumulator update: lane L owns channels 2L, 2L+1 of all rows --
      {
        int acc[2][GP];
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2) {
          if (GP >= 4) {
#pragma unroll
            for (int r = 0; r < GP; r += 2) {
              const int2 t = *reinterpret_cast<const int2*>(&L.obuf[2 * lane + c2][r]);
              acc[c2][r] = t.x; acc[c2][r + 1] = t.y;
            }
          } else {
#pragma unroll
            for (int r = 0; r < GP; ++r) acc[c2][r] = L.obuf[2 * lane + c2][r];
          }
        }
        const int sh = 16 * (lane & 1);  // channels 2L, 2L+1 within the dword
        const int s0 = (int)((cv.vs4 >> sh) & 0xffu), s1 = (int)((cv.vs4 >> (sh + 8)) & 0xffu);
        const int z0 = (int)(int8_t)((cv.vz4 >> sh) & 0xffu);
        const int z1 = (int)(int8_t)((cv.vz4 >> (sh + 8)) & 0xffu);
        if (renorm) {  // wave-uniform and rare: a branch (the empty asm keeps
                       // the compiler from turning it into selects)
          asm volatile("");
#pragma unroll
          for (int r = 0; r < GP; ++r) {
            const float rf = L.rowv[r].z;
            O[r][0] *= rf;
            O[r][1] *= rf;
          }
        }
#pragma unroll
        for (int r = 0; r < GP; ++r) {
          const float4 rv = L.rowv[r];
          const int psum = __float_as_int(rv.y);
          // exact int32 PV of Algorithm 2: s * sum P*code + z * sum P (every
          // factor fits 24 bits: s <= 80, |z| <= 127, sum P <= 64*119,
          // |sum P*code| <= 64*119*15)
          const int pv0 = __mul24(s0, acc[0][r]) + __mul24(z0, psum);
          const int pv1 = __mul24(s1, acc[1][r]) + __mul24(z1, psum);
          O[r][0] = __builtin_fmaf(rv.x, (float)pv0, O[r][0]);
          O[r][1] = __builtin_fmaf(rv.x, (float)pv1, O[r][1]);
          if (trace_g && r == trow)
            reinterpret_cast<int2*>(a.trace + TURBO_TRACE_PV)[lane] = make_int2(pv0, pv1);
        }
      }
    }
  };
  for (int g = g0; g < g1; g += 2) {
    __builtin_amdgcn_s_setprio(2);
    next_k(g + 1, KB);
    __builtin_amdgcn_s_setprio(0);
    process(KA, g);
    if (g + 1 < g1) {
      __builtin_amdgcn_s_setprio(2);
      next_k(g + 2, KA);
      __builtin_amdgcn_s_setprio(0);
      process(KB, g + 1);
    }
  }
}

// ---- cooperating waves --------------------------------------------------
// A work-group of W waves takes one chunk W consecutive groups at a time, a
// group per wave, with the results of one wave going through the groups in
// order, bit for bit:
//  * every wave forms its group's scores and row maxima; after a barrier each
//    wave forms the running maximum before its group, and the rescale factor
//    of every group of the step, from the maxima of all of them;
//  * SAS, Q(P~) and the integer PV of the group follow, and go to LDS;
//  * after a second barrier the waves share the update: each holds a slice of
//    the accumulator (GP / W rows, or half a row) and adds the step's groups
//    to it in order; l and beta are kept by every wave.
// The loads of a step leave early: K of the next step behind the QK^T that
// frees its registers, V ahead of the QK^T.
constexpr int kORow = 132;  // ints per row: the four rows of a lane in distinct bank groups

template <int GP>
struct CoopWave {
  union {
    struct {  // w = q * s^int, read back before the scores are stored
      __attribute__((aligned(16))) unsigned char whi[kWRows<GP>][128];
      __attribute__((aligned(16))) unsigned char wlo[kWRows<GP>][128];
    };
    __attribute__((aligned(16))) int sbuf[GP][kSbufStride];  // scores, row n
  };
  union {
    signed char qbuf[kWRows<GP>][128];  // the int8 query rows (read before the first step)
    __attribute__((aligned(16))) int orow[GP][kORow];  // sums Q(P~) code of the group
  };
  __attribute__((aligned(16))) unsigned char pbuf[GP + 1][64];  // Q(P~), as in DecodeLds
  float sq[16];
  int wbias[kWRows<GP>];
  unsigned vsz[64];  // V scales, then zeros, of the 128 channels
  float rs[64];      // each lane's share of the row sums of P~
  float2 rowp[GP];   // s_P s_V, sum Q(P~)
};

template <int GP, int W>
struct CoopLds {
  float lut[8];
  int ok[W];  // the wave's group is attended
  __attribute__((aligned(16))) float gmax[GP][W];
  CoopWave<GP> wave[W];
};

// Slice of the GP x 128 accumulator that wave w holds: kSRows rows of which
// lane L has channels 2L, 2L + 1, or (GP < W) one half row.
template <int GP, int W>
struct Slice {
  static constexpr int kRows = GP >= W ? GP / W : 1;
  static constexpr int kCh = GP >= W ? 2 : 1;
};

// E of the work-group's W waves take part: all of them, or the first alone.
template <int GP, int BITS, int W, int E, bool kTrace>
__device__ __forceinline__ void decode_coop(const DecodeArgs& a, CoopLds<GP, W>& LW, int w, int b,
                                            int kh, int g0, int g1, int head_off, float& mrow,
                                            float& lpart, float& beta,
                                            float (&O)[Slice<GP, E>::kRows][Slice<GP, E>::kCh],
                                            int trow) {
  constexpr int LPR = 64 / GP;
  constexpr int kRows = Slice<GP, E>::kRows, kCh = Slice<GP, E>::kCh;
  CoopWave<GP>& L = LW.wave[w];
  const int lane = threadIdx.x & 63;
  const int n = lane & 15, g4 = lane >> 4;
  const int rr = lane / LPR, cc = lane % LPR;
  const int nrow = min(n, GP), wrow = min(n, kWRows<GP> - 1);
  const int row0 = kCh == 2 ? w * kRows : w >> 1;        // the slice
  const int ch = kCh == 2 ? 2 * lane : 64 * (w & 1) + lane;
  const bool holds = row0 < GP;                           // wave-uniform
  const int* bt = a.block_table + (long)b * 4 * a.max_groups;
  const int* gt = a.group_table + (long)b * a.max_groups;

  // a lone wave has only its own LDS accesses to order
  auto coop_sync = [] {
    if constexpr (E > 1)
      __syncthreads();
    else
      wave_sync();
  };
  GroupTab T;
  GroupK<BITS> K;
  load_tab<E>(a, kh, bt, gt, g0 + w, g1, T);
  auto next_k = [&](int st) {  // the wave's group of step st
    if (st != 0 && (st & 63) == 0) load_tab<E>(a, kh, bt, gt, g0 + w + E * st, g1, T);
    load_k<BITS>(a, kh, head_off, T, st & 63, K);
  };
  next_k(0);  // on its way while the query is quantized
  decode_quant_q<GP, kTrace>(a, L.sq, L.qbuf, b, kh, w == 0 ? trow : -1);
  wave_sync();
  const float sq_row = L.sq[rr];
  QueryW<GP, BITS> Wq;
  Wq.load(L.qbuf);
  wave_sync();  // orow takes qbuf's place

  const int nst = ceil_div(g1 - g0, E);  // work-group uniform
  for (int st = 0; st < nst; ++st) {
    const int g = g0 + w + E * st;
    const bool ok = K.ok;
    tab_scales<BITS>(T, st & 63, K);  // before next_k moves the table on
    const float skg = K.skg, svg = K.svg;
    const bool trace_g = kTrace && trow >= 0 && g == a.tr_g;  // wave-uniform
    float p[GP], smax = -INFINITY;
    GroupV<BITS> cv;
    if (ok) {
      load_v<BITS>(a, kh, head_off, K, cv);
      __builtin_amdgcn_s_setprio(2);
      Wq.store(K, L.whi, L.wlo, L.wbias);
      wave_sync();
      v4i bhi[2], blo[2];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        bhi[ks] = *reinterpret_cast<const v4i*>(&L.whi[wrow][32 * g4 + 16 * ks]);
        blo[ks] = *reinterpret_cast<const v4i*>(&L.wlo[wrow][32 * g4 + 16 * ks]);
      }
      const int bias = L.wbias[wrow];
      wave_sync();  // sbuf takes the place of whi and wlo
      int4 sv[4];
      decode_qk<BITS>(K, bhi, blo, bias, sv);
      next_k(st + 1);
      __builtin_amdgcn_s_setprio(1);
      if (n < GP) {
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
          *reinterpret_cast<int4*>(&L.sbuf[n][16 * mb + 4 * g4]) = sv[mb];
      }
      if (trace_g && n == trow) {
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
          reinterpret_cast<int4*>(a.trace + TURBO_TRACE_S)[4 * mb + g4] = sv[mb];
      }
      wave_sync();
      // compact scores: lane (rr, cc) holds tokens cc*GP .. +GP-1 of row rr
      int si[GP];
      if (GP >= 4) {
#pragma unroll
        for (int e = 0; e < GP; e += 4) {
          const int4 t = *reinterpret_cast<const int4*>(&L.sbuf[rr][cc * GP + e]);
          si[e] = t.x; si[e + 1] = t.y; si[e + 2] = t.z; si[e + 3] = t.w;
        }
      } else {
#pragma unroll
        for (int e = 0; e < GP; ++e) si[e] = L.sbuf[rr][cc * GP + e];
      }
      const float c = (sq_row * skg) * a.sm_scale;
      int imax = si[0];
#pragma unroll
      for (int e = 0; e < GP; ++e) {
        p[e] = (float)si[e] * c;
        imax = max(imax, si[e]);
      }
      smax = (float)row_max_i<LPR>(imax) * c;  // c >= 0, monotonic roundings
    } else {
      next_k(st + 1);
    }
    if constexpr (E > 1) {
      if (cc == 0) LW.gmax[rr][w] = smax;
      if (lane == 0) LW.ok[w] = ok;
    }
    coop_sync();

    // ---- running maximum and rescale factors of the step's groups ---------
    float gm[E], f[E], mnew = mrow;
    unsigned okm;
    if constexpr (E == 1) {
      gm[0] = smax;
      okm = ok;
    } else {
#pragma unroll
      for (int i = 0; i < E; i += 2) {
        const float2 t = *reinterpret_cast<const float2*>(&LW.gmax[rr][i]);
        gm[i] = t.x; gm[i + (E > 1)] = t.y;
      }
      okm = (unsigned)__builtin_amdgcn_ballot_w64(LW.ok[lane & (E - 1)] != 0) & ((1u << E) - 1);
    }
    float top = gm[0];
#pragma unroll
    for (int i = 1; i < E; ++i) top = fmaxf(top, gm[i]);
    // no row moves its maximum in this step: every factor is 1 (e^0)
    const bool moved = __builtin_amdgcn_ballot_w64(top > mrow) != 0;
    if (moved) {
      // the E factors side by side (no branch, one table latency for all)
      float m = mrow;
#pragma unroll
      for (int i = 0; i < E; ++i) {
        const float mi = fmaxf(m, gm[i]);
        f[i] = sas_y(mi - m, LW.lut);  // 0 when m = -inf
        f[i] = mi > m ? f[i] : 1.0f;
        mnew = i <= w ? mi : mnew;
        m = mi;
      }
      mrow = m;
    }
    if (ok) {
      float rs = 0.0f;
      int pbits = 0;  // the maximum of the p >= 0, on their bits (same order)
#pragma unroll
      for (int e = 0; e < GP; ++e) {
        p[e] = sas_y(mnew - p[e], LW.lut);
        rs += p[e];
        pbits = max(pbits, __float_as_int(p[e]));
      }
      L.rs[lane] = rs;
      const float pmax = __int_as_float(row_max_i<LPR>(pbits));
      // Q(P~) with the row's scale pmax/119 (pmax = 0: inv = 0, adds nothing)
      const float inv = pmax > 0.0f ? kQmax / pmax : 0.0f;
      int ps = 0;
#pragma unroll
      for (int e = 0; e < GP; ++e) {
        const int code = rne_bits(p[e], inv) & 0xff;
        ps += code;
        const int t = cc * GP + e;  // token of the group
        L.pbuf[rr][16 * (t >> 4) + vpos<BITS>(t & 15)] = (unsigned char)code;
        if (trace_g && rr == trow) a.trace[TURBO_TRACE_P + t] = (unsigned char)code;
      }
      if (trace_g && rr == trow && cc == 0)
        *reinterpret_cast<float*>(a.trace + TURBO_TRACE_PMAX) = pmax;
      const int psum = row_sum_i<LPR>(ps);
      if (cc == 0)
        L.rowp[rr] = make_float2((pmax * (1.0f / kQmax)) * svg, __int_as_float(psum));
      wave_sync();
      __builtin_amdgcn_s_setprio(0);
      const v4i pop = *reinterpret_cast<const v4i*>(&L.pbuf[nrow][16 * g4]);
      // lane (n, g4), register r <-> row 4*g4 + r, channel 16*cb + n
#pragma unroll
      for (int cb = 0; cb < 8; cb += 2) {
        const v4i acc0 = mfma16x16x64(pop, v_codes<BITS>(cv, cb), v4i{});
        const v4i acc1 = mfma16x16x64(pop, v_codes<BITS>(cv, cb + 1), v4i{});
        if (4 * g4 < GP) {
#pragma unroll
          for (int r = 0; r < (GP < 4 ? GP : 4); ++r) {
            L.orow[4 * g4 + r][16 * cb + n] = acc0[r];
            L.orow[4 * g4 + r][16 * cb + 16 + n] = acc1[r];
          }
        }
      }
      if ((lane & 1) == 0) {
        L.vsz[lane >> 1] = cv.vs4;
        L.vsz[32 + (lane >> 1)] = cv.vz4;
      }
    }
    coop_sync();

    // ---- the step's groups, in order ---------------------------------------
    // O += g * (s * sum P*code + z * sum P) of group i, g = s_P s_V / beta
    auto add_group = [&](int i, float2 rp, float rbeta) {
      const CoopWave<GP>& X = LW.wave[i];
      const float gsc = rp.x * rbeta;
      const unsigned char* vb = reinterpret_cast<const unsigned char*>(X.vsz);
      int sc[kCh], zc[kCh];
      if constexpr (kCh == 2) {
        const unsigned s2 = *reinterpret_cast<const unsigned short*>(vb + ch);
        const unsigned z2 = *reinterpret_cast<const unsigned short*>(vb + 128 + ch);
        sc[0] = (int)(s2 & 0xffu);
        sc[kCh - 1] = (int)(s2 >> 8);
        zc[0] = (int)(int8_t)(z2 & 0xffu);
        zc[kCh - 1] = (int)(int8_t)(z2 >> 8);
      } else {
        sc[0] = (int)vb[ch];
        zc[0] = (int)(int8_t)vb[128 + ch];
      }
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        const int src = (row0 + r) * LPR;
        const float gr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(gsc), src));
        const int psum = __builtin_amdgcn_readlane(__float_as_int(rp.y), src);
        int acc[kCh];
        if constexpr (kCh == 2) {
          const int2 t = *reinterpret_cast<const int2*>(&X.orow[row0 + r][ch]);
          acc[0] = t.x;
          acc[kCh - 1] = t.y;
        } else {
          acc[0] = X.orow[row0][ch];
        }
#pragma unroll
        for (int c2 = 0; c2 < kCh; ++c2) {
          // exact int32 PV of Algorithm 2 (every factor fits 24 bits)
          const int pv = __mul24(sc[c2], acc[c2]) + __mul24(zc[c2], psum);
          O[r][c2] = __builtin_fmaf(gr, (float)pv, O[r][c2]);
          if (kTrace && trow == row0 + r && g0 + E * st + i == a.tr_g)
            reinterpret_cast<int*>(a.trace + TURBO_TRACE_PV)[ch + c2] = pv;
        }
      }
    };
#pragma unroll
    for (int i = 0; i < E; ++i) {
      if (!((okm >> i) & 1u)) continue;  // work-group uniform
      const float alpha = moved ? f[i] : 1.0f;
      lpart = alpha * lpart + LW.wave[i].rs[lane];
      // rescale: O = beta * Ost; renormalize when beta underflows / is 0
      float nbeta = beta * alpha;
      if (__builtin_amdgcn_ballot_w64(nbeta < 0x1p-64f) != 0) {  // rare, the same in every wave
        asm volatile("");
        if (holds) {
#pragma unroll
          for (int r = 0; r < kRows; ++r) {
            const float rf = __int_as_float(
                __builtin_amdgcn_readlane(__float_as_int(nbeta), (row0 + r) * LPR));
#pragma unroll
            for (int c2 = 0; c2 < kCh; ++c2) O[r][c2] *= rf;
          }
        }
        nbeta = 1.0f;
      }
      beta = nbeta;
      if (holds) add_group(i, LW.wave[i].rowp[rr], __builtin_amdgcn_rcpf(beta));
    }
  }
}

template <int GP, int W, bool kTrace>
__device__ void decode_tail_body(const DecodeArgs& a, int bx);  // kv_tail.hip

// One chunk, groups g0 .. g1 - 1 of (b, kh), by E of the work-group's waves.
template <int GP, int W, int E, bool kTrace>
__device__ __forceinline__ void coop_chunk(const DecodeArgs& a, CoopLds<GP, W>& LW,
                                           const DecodeSeq& sq_, int w, int b, int kh, int s, int g0,
                                           int g1) {
  constexpr int LPR = 64 / GP;
  constexpr int kRows = Slice<GP, E>::kRows, kCh = Slice<GP, E>::kCh;
  const int lane = threadIdx.x & 63;
  const int rr = lane / LPR, cc = lane % LPR;
  const int G = a.G;
  const int bits = ((a.int2_mask >> kh) & 1ull) ? 2 : 4;
  const int head_off = 512 * (4 * kh - 2 * __popcll(a.int2_mask & ((1ull << kh) - 1ull)));
  // traced row of this work-group (-1: none), whose chunk holds group tr_g
  const int trow = kTrace && b == a.tr_b && kh == a.tr_h / G && g0 <= a.tr_g && a.tr_g < g1
                       ? a.tr_h % G : -1;
  float O[kRows][kCh] = {};
  float mrow = -INFINITY, lpart = 0.0f, beta = 1.0f;
  if (bits == 4)
    decode_coop<GP, 4, W, E, kTrace>(a, LW, w, b, kh, g0, g1, head_off, mrow, lpart, beta, O, trow);
  else
    decode_coop<GP, 2, W, E, kTrace>(a, LW, w, b, kh, g0, g1, head_off, mrow, lpart, beta, O, trow);

  // every wave holds m, l and beta of all rows and its slice of O
  const float l = row_sum<LPR>(lpart);
  const bool one = sq_.nparts == 1;  // the only state (chunk 0): O / l and L directly
  const float fo = one ? beta / l : beta;
  const int row0 = kCh == 2 ? w * kRows : w >> 1;
  const int ch = kCh == 2 ? 2 * lane : 64 * (w & 1) + lane;
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    if (row0 + r >= G) break;  // wave-uniform
    const float fr =
        __int_as_float(__builtin_amdgcn_readlane(__float_as_int(fo), (row0 + r) * LPR));
    const long bh = (long)b * a.Hq + kh * G + row0 + r;
    if (one) {
      _Float16* o = reinterpret_cast<_Float16*>(a.o) + bh * 128 + ch;
      if constexpr (kCh == 2) {
        _Float16 h2[2] = {(_Float16)(O[r][0] * fr), (_Float16)(O[r][kCh - 1] * fr)};
        *reinterpret_cast<unsigned*>(o) = __builtin_bit_cast(unsigned, h2);
      } else {
        float x = O[r][0] * fr;
        asm("" : "+v"(x));  // product and rounding apart, as where two are packed
        *o = (_Float16)x;
      }
    } else {
      float* ws = a.ws + (bh * a.nws + s) * kWsStride + kWsO + ch;
      if constexpr (kCh == 2)
        *reinterpret_cast<float2*>(ws) = make_float2(O[r][0] * fr, O[r][kCh - 1] * fr);
      else
        *ws = O[r][0] * fr;
    }
  }
  if (w == 0 && cc == 0 && rr < G) {
    const long bh = (long)b * a.Hq + kh * G + rr;
    if (!one) {
      float* ws = a.ws + (bh * a.nws + s) * kWsStride;
      ws[0] = mrow;
      ws[1] = l;
    } else if (a.lse) {
      a.lse[bh] = mrow + logf(l);
    }
  }
}

// W waves per (b, KV head, chunk of groups).
template <int GP, int W, bool kTrace>
__global__ __launch_bounds__(64 * W, (GP <= 8 && !kTrace) ? 3 : 2) void k_attn_decode_coop(
    DecodeArgs a) {
  const int nmain = a.B * a.Hkv * a.nsplit;
  if ((int)blockIdx.x >= nmain) {
    decode_tail_body<GP, W, kTrace>(a, (int)blockIdx.x - nmain);
    return;
  }
  __shared__ CoopLds<GP, W> LW;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int b, kh, s;
  const DecodeSeq sq_ = decode_place(a, b, kh, s);
  const int g0 = s * sq_.split;
  const int g1 = min(sq_.ng, g0 + sq_.split);
  if (g1 <= g0) {  // no group of this sequence in the chunk
    if (s == 0 && sq_.nparts == 0) decode_write_empty(a, b, kh);
    return;
  }
  if (threadIdx.x < 8) LW.lut[threadIdx.x] = kLut[threadIdx.x];  // read behind the first step's barrier
  // A chunk of one group is left to the first wave.  The others end here (a wave
  // that has ended no longer counts at a barrier): one sequence of 64 tokens in a
  // table of 512 groups, W = 8, 8.1 us with all of them, 6.9 so (GP = 4).  With eight
  // rows the second path costs long chunks 3 %, with sixteen it gains nothing.
  if (GP <= 4 && g1 - g0 == 1) {
    if (w == 0) coop_chunk<GP, W, 1, kTrace>(a, LW, sq_, w, b, kh, s, g0, g1);
    return;
  }
  coop_chunk<GP, W, W, kTrace>(a, LW, sq_, w, b, kh, s, g0, g1);
}

// kTrace = true only for the test hook that also stores one group's integers
// (the production instances carry no trace code).
// One wave per (b, KV head, chunk of groups); with several chunks each
// writes its state to the workspace and k_decode_combine merges them.
template <int GP, bool kTrace>
__global__ __launch_bounds__(64, (GP <= 8 && !kTrace) ? 3 : 2) void k_attn_decode(DecodeArgs a) {
  // the last B * Hkv work-groups (when there is a buffer): its chunk
  const int nmain = a.B * a.Hkv * a.nsplit;
  if ((int)blockIdx.x >= nmain) {
    decode_tail_body<GP, 1, kTrace>(a, (int)blockIdx.x - nmain);
    return;
  }
  __shared__ DecodeLds<GP> L;
  int b, kh, s;
  const DecodeSeq sq_ = decode_place(a, b, kh, s);
  constexpr int LPR = 64 / GP;
  const int lane = threadIdx.x & 63;
  if (lane < 8) L.lut[lane] = kLut[lane];
  const int rr = lane / LPR, cc = lane % LPR;
  const int G = a.G;

  const int g0 = s * sq_.split;
  const int g1 = min(sq_.ng, g0 + sq_.split);
  if (g1 <= g0) {  // no group of this sequence in the chunk
    if (s == 0 && sq_.nparts == 0) decode_write_empty(a, b, kh);
    return;
  }

  float O[GP][2];
#pragma unroll
  for (int r = 0; r < GP; ++r) O[r][0] = O[r][1] = 0.0f;
  float mrow = -INFINITY, lpart = 0.0f, beta = 1.0f, l = 0.0f;
  {
    const int bits = ((a.int2_mask >> kh) & 1ull) ? 2 : 4;
    const int head_off = 512 * (4 * kh - 2 * __popcll(a.int2_mask & ((1ull << kh) - 1ull)));

    // traced row of this wave (-1: none); the wave whose chunk holds group tr_g
    const int trow = kTrace && b == a.tr_b && kh == a.tr_h / G && g0 <= a.tr_g && a.tr_g < g1
                         ? a.tr_h % G : -1;
    decode_quant_q<GP, kTrace>(a, L.sq, L.qbuf, b, kh, trow);
    wave_sync();
    const float sq_row = L.sq[rr];

    if (bits == 4)
      decode_groups<GP, 4, kTrace>(a, L, b, kh, g0, g1, head_off, mrow, lpart, beta, O, sq_row, trow);
    else
      decode_groups<GP, 2, kTrace>(a, L, b, kh, g0, g1, head_off, mrow, lpart, beta, O, sq_row, trow);

    // ---- epilogue: per-row (m, l, beta) from the softmax lanes -----------
    l = row_sum<LPR>(lpart);
    wave_sync();
    if (cc == 0) L.rowv[rr] = make_float4(mrow, l, beta, 0.0f);
    wave_sync();
  }
  if (sq_.nparts == 1) {  // the only state (chunk 0): O / l and L directly
#pragma unroll
    for (int r = 0; r < GP; ++r) {
      if (r >= G) break;
      const float4 rv = L.rowv[r];
      const float f = rv.z / rv.y;
      _Float16 h2[2] = {(_Float16)(O[r][0] * f), (_Float16)(O[r][1] * f)};
      reinterpret_cast<unsigned*>(a.o)[((long)b * a.Hq + kh * G + r) * 64 + lane] =
          __builtin_bit_cast(unsigned, h2);
    }
    if (a.lse && cc == 0 && rr < G)
      a.lse[(long)b * a.Hq + kh * G + rr] = mrow + logf(l);
    return;
  }
  // several states: O beta, m and l of each row, to the workspace
#pragma unroll
  for (int r = 0; r < GP; ++r) {
    if (r >= G) break;
    const float be = L.rowv[r].z;
    float* w = a.ws + (((long)b * a.Hq + kh * G + r) * a.nws + s) * kWsStride;
    *reinterpret_cast<float2*>(w + kWsO + 2 * lane) = make_float2(O[r][0] * be, O[r][1] * be);
  }
  if (cc == 0 && rr < G) {
    float* w = a.ws + (((long)b * a.Hq + kh * G + rr) * a.nws + s) * kWsStride;
    w[0] = mrow;
    w[1] = l;
  }
}

// Merge of the chunk states of one (b, query head) with more than one state
// (split-KV extension): m* = max m_s, w_s = SAS(m_s - m*) (exactly 1 for
// m_s = m*), O = sum w_s O_s / sum w_s l_s, L = m* + ln sum w_s l_s, chunks
// in ascending order (the buffer's state last).  A separate launch: the
// kernel boundary makes every chunk's state visible across the XCDs' L2
// caches.  Lane L handles channels 2L, 2L + 1.
__global__ __launch_bounds__(64) void k_decode_combine(DecodeArgs a) {
  __shared__ float lut[8];
  __shared__ float cwt[64], cl[64];  // merge weights and l of up to 64 chunks
  const int lane = threadIdx.x & 63;
  const int bh = blockIdx.x;
  const int b = bh / a.Hq;
  const int ns = decode_seq(a, b).nparts;
  if (ns < 2) return;  // written by the decode launch itself
  if (lane < 8) lut[lane] = kLut[lane];
  const float* w = a.ws + (long)bh * a.nws * kWsStride;
  // m* over the chunks, lane s reading chunk s (and s + 64, ...)
  float mstar = -INFINITY;
  for (int s = lane; s < ns; s += 64) mstar = fmaxf(mstar, w[(long)s * kWsStride]);
  mstar = wave_max(mstar);
  // ascending accumulation of w_s l_s and w_s O_s; the weights of 64 chunks
  // at a time go through LDS and four chunks' O loads are in flight at once
  float den = 0.0f, n0 = 0.0f, n1 = 0.0f;
  for (int s0 = 0; s0 < ns; s0 += 64) {
    const int cnt = min(64, ns - s0);
    __syncthreads();
    if (lane < cnt) {
      const float* ws = w + (long)(s0 + lane) * kWsStride;
      cwt[lane] = ws[0] < mstar ? sas_y(mstar - ws[0], lut) : 1.0f;  // e^0 for m_s = m*
      cl[lane] = ws[1];
    }
    __syncthreads();
    const float* wo = w + (long)s0 * kWsStride + kWsO + 2 * lane;
    int t = 0;
    for (; t + 4 <= cnt; t += 4) {
      float2 x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = *reinterpret_cast<const float2*>(wo + (t + u) * kWsStride);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        den = __builtin_fmaf(cwt[t + u], cl[t + u], den);
        n0 = __builtin_fmaf(cwt[t + u], x[u].x, n0);
        n1 = __builtin_fmaf(cwt[t + u], x[u].y, n1);
      }
    }
    for (; t < cnt; ++t) {
      const float2 x = *reinterpret_cast<const float2*>(wo + t * kWsStride);
      den = __builtin_fmaf(cwt[t], cl[t], den);
      n0 = __builtin_fmaf(cwt[t], x.x, n0);
      n1 = __builtin_fmaf(cwt[t], x.y, n1);
    }
  }
  _Float16 h2[2] = {(_Float16)(n0 / den), (_Float16)(n1 / den)};
  reinterpret_cast<unsigned*>(a.o)[(long)bh * 64 + lane] = __builtin_bit_cast(unsigned, h2);
  if (a.lse && lane == 0) a.lse[bh] = mstar + logf(den);
}

template <int W, bool kTrace>
static void launch_decode(const DecodeArgs& a, int total, hipStream_t stream) {
  const dim3 grid(total), block(64 * W);
  if constexpr (W == 1) {
    if (a.G <= 1)
      hipLaunchKernelGGL((k_attn_decode<1, kTrace>), grid, block, 0, stream, a);
    else if (a.G <= 2)
      hipLaunchKernelGGL((k_attn_decode<2, kTrace>), grid, block, 0, stream, a);
    else if (a.G <= 4)
      hipLaunchKernelGGL((k_attn_decode<4, kTrace>), grid, block, 0, stream, a);
    else if (a.G <= 8)
      hipLaunchKernelGGL((k_attn_decode<8, kTrace>), grid, block, 0, stream, a);
    else
      hipLaunchKernelGGL((k_attn_decode<16, kTrace>), grid, block, 0, stream, a);
  } else if (a.G <= 1) {
    hipLaunchKernelGGL((k_attn_decode_coop<1, W, kTrace>), grid, block, 0, stream, a);
  } else if (a.G <= 2) {
    hipLaunchKernelGGL((k_attn_decode_coop<2, W, kTrace>), grid, block, 0, stream, a);
  } else if (a.G <= 4) {
    hipLaunchKernelGGL((k_attn_decode_coop<4, W, kTrace>), grid, block, 0, stream, a);
  } else if (a.G <= 8) {
    hipLaunchKernelGGL((k_attn_decode_coop<8, W, kTrace>), grid, block, 0, stream, a);
  } else {
    hipLaunchKernelGGL((k_attn_decode_coop<16, W, kTrace>), grid, block, 0, stream, a);
  }
}

// Waves per work-group (W).  One wave takes 1.2 (GP = 1) to 2.3 us (GP = 16) per
// group whatever the load, so a launch of few chunks is bound by the chain of groups
// of its longest one; W waves cut the chain W-fold, at about 2.3 (W = 4) and 3.3 us
// (W = 8) per step of W groups.  A launch that fills the chip is bound by the sum of
// its work, where W > 1 pays for W prologues and the exchanges.  So W is the most
// waves with which every work-group is resident at once, where the chunks are long
// enough to give each wave work, and one wave otherwise.  Resident work-groups by
// registers and LDS, W = 1 / 2 / 4 / 8: 3072 / 1536 / 768 / 256 up to four rows, 2304 /
// 1536 / 768 / 256 with eight, 1536 / 1024 / 512 / 256 with sixteen.
//
// us of a launch by chunks (all of one length, int4 and int2 heads), W = 1 / 2 / 4 / 8:
//   GP = 4, 2 groups: 512: 8.4 / 8.2 / 8.5, 1024: 9.2 / 9.3 / 13.0; 4 groups: 512: 11.4 /
//   10.5 / 9.1, 1024: 12.7 / 12.5 / 16.1, 1280: 14.1 / 14.5 / 17.8; 8 groups: 256: 16.4 /
//   13.1 / 10.7 / 10.0, 512: 17.6 / 15.1 / 12.4 / 17.3, 768: 18.5 / 16.3 / 15.9, 1536:
//   22.9 / 22.0 / 28.1, 2048: 25.0 / 33.3 / 38.1.  GP = 1 and 2 cross at the same sizes.
//   GP = 8, 2 groups: 1024: 11.7 / 10.8 / 15.2, 1536: 13.0 / 13.1 / 19.5; 8 groups: 768:
//   26.5 / 19.2 / 17.8, 1536: 31.3 / 25.1 / 31.7, 2048: 35.1 / 38.9 / 42.1; 48 groups:
//   2048: 169 / 166 / 164.  Past what one wave keeps resident two are ahead again: 2560
//   of 8 groups 59.0 / 45.9 / 51.7, of 2 22.5 / 22.3; 8192 of 8 130 / 119, of 4 76 / 78.
//   GP = 16, 8 groups: 512: 27.9 / 22.3 / 16.7, 1024: 29.6 / 25.3 / 31.1, 1536: 35.1 /
//   44.3 / 44.6; 48 groups: 1536: 164 / 196 / 172, 2048: 276 / 257 / 214, 2560: 304 / 280 /
//   267, 3072: 310 / 355 / 320.
// With a buffer its work-groups come last, one per (sequence, KV head), and take their
// rows a wave at a time.  They count beside short chunks, half beside chunks of 12 to
// 15 groups; longer ones outlast them.  One chunk each: GP = 4, 8 groups: 64: 19.3 /
// 16.0 / 13.5 / 12.6, 256: 20.3 / 17.3 / 14.6 / 17.7, 512: 22.6 / 20.6 / 20.7, 768: 24.1 /
// 23.2 / 27.7, 1024: 26.5 / 27.6 / 34.3; 16 groups: 512: 34.4 / 29.2 / 25.4, 1024: 41.1 /
// 39.6 / 43.7, 1536: 49.6 / 48.6.  With more rows they are the longest part, and more
// waves shorten it: GP = 8, 4 groups: 768: 27.3 / 24.0 / 28.4, 1024: 29.2 / 30.5, 1536:
// 42.6 / 39.8, 3072: 70.2 / 67.7; GP = 16: 512: 36.5 / 29.2 / 29.9, 1024: 54.4 / 52.8 /
// 50.8, 1536: 61.8 / 67.5, 2048: 90.5 / 84.7.
//
// The host sees neither lengths nor raggedness.  Chunks of 48 groups and more of up to
// 1024 (eight rows) or 2048 (sixteen) take four waves: us for 1024 of 64 groups, eight
// rows, 174 / 106 / 125 where all are equally long, 155 / 89 / 61 where they are not (32
// sequences of 256 to 16383 tokens); ahead of one wave in both.  The number of chunks is
// that of the grid, from the width of the tables; where shorter sequences leave some of
// them empty, fewer waves are taken than would be best (64 sequences of 2000 tokens,
// 32/8 heads, 53 us in tables of 512 groups, 31 in their own).
static int decode_waves(const DecodeArgs& a) {
  const long units = (long)a.B * a.Hkv * a.nsplit, buf = a.tk ? (long)a.B * a.Hkv : 0;
  int len = ceil_div(a.max_groups, a.nsplit);  // groups of the longest chunk
  if (buf && a.nsplit == 1 && len > 1) --len;  // the table's last is not full yet
  const bool some = len >= 2 || a.nsplit == 1;
  const long wgs = units + (len >= 16 ? 0 : len >= 12 ? buf / 2 : buf);
  if (units <= 256 && ((len >= 6 && units + buf <= (len >= 8 ? 384 : 256)) ||
                       len >= (a.G <= 8 ? 16 : 32)))
    return 8;
  if (wgs <= (a.G <= 8 ? 768 : 512) && len >= (buf || wgs <= 512 ? 3 : 8)) return 4;
  if (buf && len >= 6 && len < 16) {
    // past what is resident, by a margin: the buffer's work-groups are the shorter ones
    const int most = a.G > 8 ? 512 : a.G <= 2 ? 1024 : len < 8 ? 896 : a.G <= 4 ? 1024 : 1152;
    if (wgs <= most) return 4;
  }
  if (a.G <= 4) {
    if (buf)
      return some && (wgs <= (len == 1 ? 2048 : 1536) || (units <= 1152 && len >= 8) ||
                      (units <= 1536 && len >= (a.G <= 2 ? 6 : 12))) ? 2 : 1;
    return units <= 1536 && len >= (units <= 512 ? 2 : units <= 1024 ? 4 : 6) ? 2 : 1;
  }
  if (len >= 48 && units <= (a.G <= 8 ? 1024 : 2048)) return 4;
  if (buf) return some ? 2 : 1;
  if (a.G <= 8) return len >= (units <= 1536 ? 2 : units <= 2304 ? 12 : 4) ? 2 : 1;
  if (units <= 1024) return len >= 2 ? 2 : 1;
  return units > 1536 && units <= 2560 && len >= 12 ? 4 : 1;
}

hipError_t launch_attn_decode(const DecodeArgs& a, hipStream_t stream) {
  // group chunks, then one work-group per (sequence, KV head) for the buffer
  const int total = a.B * a.Hkv * a.nsplit + (a.tk ? a.B * a.Hkv : 0);
  const int W = decode_waves(a);
  if (a.trace) {
    switch (W) {
      case 1: launch_decode<1, true>(a, total, stream); break;
      case 2: launch_decode<2, true>(a, total, stream); break;
      case 4: launch_decode<4, true>(a, total, stream); break;
      default: launch_decode<8, true>(a, total, stream); break;
    }
  } else {
    switch (W) {
      case 1: launch_decode<1, false>(a, total, stream); break;
      case 2: launch_decode<2, false>(a, total, stream); break;
      case 4: launch_decode<4, false>(a, total, stream); break;
      default: launch_decode<8, false>(a, total, stream); break;
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.nws < 2) return e;  // no sequence has two states to merge
  hipLaunchKernelGGL(k_decode_combine, dim3(a.B * a.Hq), dim3(64), 0, stream, a);
  return hipGetLastError();
}

}  // namespace turbo
