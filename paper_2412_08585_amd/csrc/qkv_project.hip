// The QKV projection with FlashQ fused into its epilogue (Sec. 5.2: the
// quantization of Q, K and V is folded into the projection that produces
// them), on gfx950.
//
//   [Q | K | V] = X W^T,  X fp16 [B][N][D] (hidden states), W fp16 [F][D]
//   with F = (Hq + 2 Hkv) * 128 output features (query heads, then key
//   heads, then value heads, 128 channels each).
//
// The products accumulate in fp32 on v_mfma_f32_32x32x16_f16 and each output
// is rounded to fp16, the precision the unfused projection would store.  The
// epilogue then applies FlashQ step 1 to every (sequence, head, 64-token
// block) -- the same rule as the prefill prologue for Q and k_quantize_kv for
// K and V -- and, for K and V, step 2 with the paged cache write, through the
// same LDS-tile routines as k_quantize_kv.  Q, K and V never reach HBM in
// fp16.
//
// Tiling.  A work-group of kWM x kWN waves computes a tile of 32 kMB kWM tokens
// by 32 kNB kWN features, wave (wm, wn) its kMB x kNB MFMA blocks of 32 x 32.
// The contraction runs in stages of 64 columns: the tile's X and W rows of a
// stage (128 bytes each, 16-byte chunks swizzled by row so that the operand
// reads are free of bank conflicts) are loaded straight into LDS by buffer
// loads, into two stage buffers used in turn.  A wave reads the operands of the
// next 16 columns into registers while the current ones' MFMAs run; the barrier
// of a stage lies before its last 16 columns, whose MFMAs cover the first reads
// of the next stage and the issue of the loads of the one after.
//   * 256 tokens x 256 features (two heads), 2 x 4 waves of 4 x 2 blocks: two
//     waves per SIMD, so that one's MFMAs fill the other's waits.
//     Bound by LDS as much as by the MFMAs: per 64 columns and CU, operand
//     reads of 192 KB and the staged 64 KB at 128 bytes a clock are as many
//     clocks as the MFMAs' 2048.  Phi-3-medium 4 x 4096 tokens, D = 5120:
//     1.10-1.17 ms, against 1.24-1.25 (four waves of 4 x 4 blocks, one per SIMD,
//     stages of 32 columns); without the epilogue 1.10 against 1.17.
//   * 128 tokens x 128 features (one head), 2 x 2 waves of 2 x 2 blocks, two
//     work-groups per CU: for inputs whose large tiles would leave CUs idle
//     (777 tokens, D = 4096, 48 heads: 57 us against 91).
#include "turbo_common.h"
#include "quant_tiles.h"
#include "qkv_project.h"

namespace turbo {

typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kPRow = 128;                  // LDS bytes per staged row: 64 fp16 columns
constexpr int kEpiTile = 64 * kTileStride;  // one 64 x 128 int8 block (k_quantize_kv layout)

template <int kWM_, int kWN_, int kMB_, int kNB_>
struct QkvTile {
  static constexpr int kWM = kWM_, kWN = kWN_, kMB = kMB_, kNB = kNB_;
  static constexpr int kWaves = kWM * kWN, kThreads = 64 * kWaves;
  static constexpr int kTok = 32 * kMB * kWM, kFeat = 32 * kNB * kWN;
  static constexpr int kHeads = kFeat / 128, kBlocks = kTok / 64;  // FlashQ blocks: kBlocks a head
  static constexpr int kXBytes = kTok * kPRow, kStage = (kTok + kFeat) * kPRow;
  static constexpr int kLoads = kStage / 1024 / kWaves;  // 1 KiB loads per wave and stage
  static constexpr int kTeams = kThreads / 256;          // step 2 runs on 256 threads each
  static constexpr int kTiles = kHeads * kBlocks;        // FlashQ blocks of the work-group
  static_assert(kNB == 2 && kMB % 2 == 0, "a wave covers half a head and whole FlashQ blocks");
  static_assert(kXBytes / 1024 % kWaves == 0 && kFeat * kPRow / 1024 % kWaves == 0, "even loads");
  static_assert((kTiles + kTeams) * kEpiTile <= 2 * kStage, "the epilogue's tiles fit");
  static_assert(kBlocks % kTeams == 0 && kWaves % kTiles == 0, "even epilogue");
};
using QkvLarge = QkvTile<2, 4, 4, 2>;
using QkvSmall = QkvTile<2, 2, 2, 2>;

__device__ __forceinline__ f32x16_t mfma_f16(uint4 a, uint4 b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8_t, a),
                                                __builtin_bit_cast(h8_t, b), c, 0, 0, 0);
}

typedef int i32x4 __attribute__((ext_vector_type(4)));

// Raw buffer resource over `bytes` bytes at p, as the four descriptor words
// (word 3: 32-bit data format).  Loads at offsets >= bytes return zeros: the
// rows past N of the last token tile and past F of an odd head count.
__device__ __forceinline__ i32x4 rows_words(const void* p, int bytes) {
  const unsigned long long a = (unsigned long long)p;
  return i32x4{(int)(unsigned)a, (int)((unsigned)(a >> 32) & 0xffffu), bytes, 0x00020000};
}

// 16 bytes per lane from the buffer (offsets voff + soff) into LDS at dst +
// 16 * lane (the wave-uniform LDS address goes through M0; the nop keeps the
// load one cycle away from the compiler's write of M0).
__device__ __forceinline__ void lds_load16(i32x4 r, unsigned voff, unsigned soff, uint8_t* dst) {
  const unsigned la = (unsigned)(unsigned long)(__attribute__((address_space(3))) uint8_t*)dst;
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               :: "v"(voff), "s"(r), "s"(soff), "{m0}"(la) : "memory");
}

// Work-group order.  The dispatcher hands work-group x to XCD x % 8.  When
// the token tiles are a multiple of 8, XCD k owns tiles k, k+8, ... and walks
// them in blocks of (all its tiles) x (8 head pairs): the 32 work-groups
// resident on an XCD then share 4 X tiles and 8 W pairs in its L2.
__device__ __forceinline__ void qkv_tile(int x, int ntiles, int npairs, int& tile, int& pair) {
  if (ntiles % 8 != 0) {
    pair = x % npairs;
    tile = x / npairs;
    return;
  }
  const int k = x % 8, i = x / 8;
  const int ntk = ntiles / 8;   // tiles of this XCD
  const int full = npairs / 8;  // complete groups of 8 pairs
  int tl;
  if (i < full * ntk * 8) {
    const int hg = i / (ntk * 8), rem = i % (ntk * 8);
    tl = rem / 8;
    pair = 8 * hg + rem % 8;
  } else {
    const int r = npairs - 8 * full, rem = i - full * ntk * 8;
    tl = rem / r;
    pair = 8 * full + rem % r;
  }
  tile = tl * 8 + k;
}

// kY = true only for the test hook that also stores the fp16 projection
// (the production instance carries no such store).
template <typename T, bool kY>
__global__ __launch_bounds__(T::kThreads, 2) void k_qkv_project(QkvArgs a) {
  constexpr int kMB = T::kMB, kNB = T::kNB, kWN = T::kWN;
  __shared__ __align__(16) uint8_t st[2 * T::kStage];
  __shared__ float part[T::kHeads][T::kBlocks][2];  // maxima of the two half heads
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wv / kWN, wn = wv % kWN;
  const int m = lane & 31, hh = lane >> 5;
  const int nheads = a.Hq + 2 * a.Hkv;
  const int nunits = ceil_div(nheads, T::kHeads);
  const int ntile = ceil_div(a.N, T::kTok);
  const int F = 128 * nheads;
  int tile, unit_;
  qkv_tile(blockIdx.x, a.B * ntile, nunits, tile, unit_);
  const int head0 = T::kHeads * unit_;
  const int b = tile / ntile;
  const int t0 = (tile % ntile) * T::kTok;

  // ---- staging: buffer loads straight into LDS --------------------------------
  // chunk c of staged row r sits at chunk position c ^ g(r), g = (r & 7) ^ ((r >> 3) & 1):
  // any 8 rows from a multiple of 8 and any 16 from a multiple of 16 put one
  // chunk into distinct 16-byte slots of 32 (64) banks.  Load i of a wave fills
  // rows 8 j .. + 7 (j = kWaves i + wave; 1 KiB): lane L takes row + (L >> 3),
  // position L & 7, i.e. source chunk (L & 7) ^ (L >> 3) ^ (j & 1).
  const unsigned D2 = 2u * (unsigned)a.D;  // bytes per row
  const unsigned vrow = (unsigned)(lane >> 3) * D2;
  const unsigned vch = (unsigned)((lane & 7) ^ (lane >> 3));
  // the parity of j is that of the wave (kWaves is even)
  const unsigned vo = vrow + 16u * (vch ^ (unsigned)(wv & 1));
  const unsigned xs0 = (unsigned)t0 * D2, ws0 = (unsigned)(128 * head0) * D2;
  const i32x4 xr = rows_words(static_cast<const _Float16*>(a.x) + (long)b * a.N * a.D, a.N * (int)D2);
  const i32x4 wr = rows_words(a.w, F * (int)D2);
  // The loads are written as inline assembly: the compiler then neither
  // waits for them before every LDS read nor counts them in its own waits
  // (no other vector-memory operation is in flight during the loop).
  constexpr int kXLoads = T::kXBytes / 1024 / T::kWaves;
  auto dma_j = [&](int buf, int kk, int i) {
    const unsigned kb = 128u * (unsigned)kk;  // 64 fp16 columns per stage
    uint8_t* dst = st + buf * T::kStage;
    if (i < kXLoads) {
      const int r0 = 8 * (T::kWaves * i + wv);
      lds_load16(xr, vo, xs0 + (unsigned)r0 * D2 + kb, dst + r0 * kPRow);
    } else {
      const int r0 = 8 * (T::kWaves * (i - kXLoads) + wv);
      lds_load16(wr, vo, ws0 + (unsigned)r0 * D2 + kb, dst + T::kXBytes + r0 * kPRow);
    }
  };
  f32x16_t acc[kMB][kNB];
#pragma unroll
  for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb) acc[mb][nb] = f32x16_t{};

  // operand reads: row 32 kMB wm + 32 mb + m (A) / 32 kNB wn + 32 nb + m (B);
  // contraction slot (step s, half hh, element e) = column 16 s + 8 hh + e,
  // chunk 2 s + hh
  const int sw = hh ^ (m & 7) ^ ((m >> 3) & 1);
  const int aA = (32 * kMB * wm + m) * kPRow, aB = T::kXBytes + (32 * kNB * wn + m) * kPRow;
  struct Ops {
    uint4 a[kMB], b[kNB];
  };
  auto read = [&](int buf, int s, Ops& o) {
    const uint8_t* p = st + buf * T::kStage + 16 * (sw ^ (2 * s));
#pragma unroll
    for (int i = 0; i < kNB; ++i) o.b[i] = *reinterpret_cast<const uint4*>(p + aB + 32 * kPRow * i);
#pragma unroll
    for (int i = 0; i < kMB; ++i) o.a[i] = *reinterpret_cast<const uint4*>(p + aA + 32 * kPRow * i);
  };
  auto mma = [&](const Ops& o) {
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb) acc[mb][nb] = mfma_f16(o.a[mb], o.b[nb], acc[mb][nb]);
  };
  const int nk = a.D / 64;
  Ops o0, o1;
#pragma unroll
  for (int i = 0; i < T::kLoads; ++i) dma_j(0, 0, i);
  if (nk > 1) {
#pragma unroll
    for (int i = 0; i < T::kLoads; ++i) dma_j(1, 1, i);
    static_assert(T::kLoads == 8, "the wait leaves the second stage's loads in flight");
    asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  }
  read(0, 0, o0);
  // Stage k in buffer buf.  Its loads were issued a stage ago, and its first
  // operands read behind the last MFMAs of stage k - 1.
  auto stage = [&](auto bufc, int k) {
    constexpr int buf = decltype(bufc)::value;
    read(buf, 1, o1);
    mma(o0);
    __builtin_amdgcn_sched_barrier(0);
    read(buf, 2, o0);
    mma(o1);
    __builtin_amdgcn_sched_barrier(0);
    read(buf, 3, o1);
    mma(o0);
    // every operand of the stage is in registers (lgkmcnt(0), through the builtin
    // so that the compiler knows), and the wave's loads of stage k + 1 have
    // landed; behind the barrier that holds for every wave, so the buffer is
    // free and the other one complete
    __builtin_amdgcn_s_waitcnt(0xC07F);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    // past the end the last stage is loaded and read again: no branch
    read(buf ^ 1, 0, o0);
    const int kn = min(k + 2, nk - 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb) {
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb) acc[mb][nb] = mfma_f16(o1.a[mb], o1.b[nb], acc[mb][nb]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < T::kLoads / kMB; ++i) dma_j(buf, kn, T::kLoads / kMB * mb + i);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int k = 0; k < nk; k += 2) {
    stage(std::integral_constant<int, 0>{}, k);
    if (k + 1 < nk) stage(std::integral_constant<int, 1>{}, k + 1);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // ---- epilogue: fp16 outputs, FlashQ step 1 per 64-token block --------------
  // lane (m, hh), register r of (mb, nb) <-> token 32 (kMB wm + mb) + 8 (r/4) +
  // 4 hh + r%4 of the tile, channel 64 (wn & 1) + 32 nb + m of head wn / 2
  // (of the tile); FlashQ block kMB / 2 wm + (mb >> 1)
  const int hl = wn >> 1, half = wn & 1;
  const int head = head0 + hl;
  const bool hv = head < nheads;  // wave-uniform (an odd head count leaves one out)
  auto etile = [&](int t) -> uint8_t* { return st + t * kEpiTile; };
  const int nv0 = a.N - (t0 + 32 * kMB * wm);  // valid rows from the wave's first
  // max |fp16(y)| = fp16(max |y|): rounding is monotone and symmetric, so
  // the first pass needs no conversion.  Rows past N hold zeros (their X rows
  // were read as zeros).
#pragma unroll
  for (int i = 0; i < kMB / 2; ++i) {
    float amax = 0.0f;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          amax = fmaxf(amax, fabsf(acc[2 * i + mi][nb][r]));
          if constexpr (kY) {
            const int row = 64 * i + 32 * mi + 8 * (r >> 2) + 4 * hh + (r & 3);
            if (hv && row < nv0)
              a.y[((long)b * a.N + t0 + 32 * kMB * wm + row) * (long)F + 128 * head + 64 * half +
                  32 * nb + m] = (_Float16)acc[2 * i + mi][nb][r];
          }
        }
    amax = wave_max_fast((float)(_Float16)amax);
    if (lane == 0) part[hl][kMB / 2 * wm + i][half] = amax;
  }
  __syncthreads();
  // (i a compile-time constant: acc is indexed with it; kFull: all 64 tokens lie
  // below N, the common case, and no row is masked out)
  auto codes = [&](auto ic, auto fullc) {
    constexpr int i = decltype(ic)::value;
    constexpr bool kFull = decltype(fullc)::value;
    const int blk = kMB / 2 * wm + i;
    const float amax = fmaxf(part[hl][blk][0], part[hl][blk][1]);
    const float inv = amax > 0.0f ? kQmax / amax : 0.0f;
    int8_t* tw = reinterpret_cast<int8_t*>(etile(hl * T::kBlocks + blk)) + 64 * half + m;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = 32 * mi + 8 * (r >> 2) + 4 * hh + (r & 3);
          const float y = (float)(_Float16)acc[2 * i + mi][nb][r];
          const int q = min(119, max(-119, rne_mul(y, inv)));
          tw[row * kTileStride + 32 * nb] = (int8_t)((kFull || row < nv0 - 64 * i) ? q : 0);
        }
    // the next block's accumulator reads stay below this point
    __builtin_amdgcn_sched_barrier(0);
  };
  auto run = [&](auto ic) {
    if (nv0 >= 64 * decltype(ic)::value + 64)  // wave-uniform
      codes(ic, std::true_type{});
    else
      codes(ic, std::false_type{});
  };
  run(std::integral_constant<int, 0>{});
  if constexpr (kMB == 4) run(std::integral_constant<int, 1>{});
  __syncthreads();
  auto block_scale = [&](int h, int blk) {
    const float amax = fmaxf(part[h][blk][0], part[h][blk][1]);
    return amax > 0.0f ? amax / kQmax : 0.0f;
  };

  // ---- Q8 / K8 / V8 and the block scales: kPer waves to a block ---------------
  {
    constexpr int kPer = T::kWaves / T::kTiles;
    const int t = wv / kPer, sub = wv % kPer;
    const int h = t / T::kBlocks, blk = t % T::kBlocks, hd = head0 + h;
    const int jb = t0 / 64 + blk;  // FlashQ block index in the sequence
    const int8_t* tw = reinterpret_cast<const int8_t*>(etile(t));
    if (hd < nheads && jb < a.nb) {  // wave-uniform
      const float s = block_scale(h, blk);
      if (hd < a.Hq + a.Hkv) {
        // token-major int8 rows (Q8 or K8) and the block scale
        const bool isq = hd < a.Hq;
        const long unit = (long)b * (isq ? a.Hq : a.Hkv) + (isq ? hd : hd - a.Hq);
        int8_t* dst = (isq ? a.q8 : a.k8) + (unit * a.nb + jb) * 8192;
#pragma unroll
        for (int it = 0; it < 16 / kPer; ++it) {
          const int row = 4 * (it * kPer + sub) + (lane >> 4), c8 = lane & 15;
          *reinterpret_cast<uint2*>(dst + row * 128 + 8 * c8) =
              *reinterpret_cast<const uint2*>(tw + row * kTileStride + 8 * c8);
        }
        if (lane == 0 && sub == 0) (isq ? a.sq : a.sk)[unit * a.nb + jb] = s;
      } else {
        // channel-major V8 block: a lane writes whole channels
        const long unit = (long)b * a.Hkv + (hd - a.Hq - a.Hkv);
        int8_t* dst = a.v8 + (unit * a.nb + jb) * 8192;
#pragma unroll
        for (int cc = 0; cc < 2 / kPer; ++cc) {
          const int c = kPer == 1 ? 2 * lane + cc : 64 * sub + lane;
          unsigned wd[16];
#pragma unroll
          for (int k = 0; k < 16; ++k) {
            const int8_t* p = tw + 4 * k * kTileStride + c;
            wd[k] = pack4(p[0], p[kTileStride], p[2 * kTileStride], p[3 * kTileStride]);
          }
          uint4* o = reinterpret_cast<uint4*>(dst + c * 64);
#pragma unroll
          for (int k = 0; k < 4; ++k)
            o[k] = make_uint4(wd[4 * k], wd[4 * k + 1], wd[4 * k + 2], wd[4 * k + 3]);
        }
        if (lane == 0 && sub == 0) a.sv[unit * a.nb + jb] = s;
      }
    }
  }

  // ---- step 2 and the cache write (K and V heads, full blocks) ---------------
  if (a.pages == nullptr) return;  // work-group uniform
  const int team = tid >> 8, tm = tid & 255;  // 256 threads take a block
  for (int h = 0; h < T::kHeads; ++h) {
    const int hd = head0 + h;
    if (hd < a.Hq || hd >= nheads) continue;  // work-group uniform
    const bool isk = hd < a.Hq + a.Hkv;
    const int hkv = isk ? hd - a.Hq : hd - a.Hq - a.Hkv;
    const int bits = ((a.int2_mask >> hkv) & 1ull) ? 2 : 4;
    const int head_off = 512 * (4 * hkv - 2 * __popcll(a.int2_mask & ((1ull << hkv) - 1ull)));
    for (int w = team; w < T::kBlocks; w += T::kTeams) {
      const int g = t0 / 64 + w;
      bool ok = t0 + 64 * w + 64 <= a.N && g < a.max_groups;  // uniform over the team
      long page[4] = {0, 0, 0, 0};
      long slot = 0;
      if (ok) {
        const int* bt = a.block_table + (long)b * 4 * a.max_groups + 4 * g;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          page[p] = bt[p];
          ok = ok && page[p] >= 0 && page[p] < a.num_pages;
        }
        slot = a.group_table[(long)b * a.max_groups + g];
        ok = ok && slot >= 0 && slot < a.num_slots;
      }
      int8_t* meta = a.gmeta + ((ok ? slot : 0) * a.Hkv + hkv) * 512;
      float* gs = a.gscale + ((ok ? slot : 0) * a.Hkv + hkv) * 2;
      const int8_t* tb = reinterpret_cast<const int8_t*>(etile(h * T::kBlocks + w));
      const float s = block_scale(h, w);
      if (isk)
        compress_k(tb, etile(T::kTiles + team), bits, meta, gs, s, page, a.pages,
                   a.page_bytes, head_off, tm, ok);
      else
        compress_v(tb, bits, meta, gs + 1, s, page, a.pages, a.page_bytes, head_off, tm, ok);
      __syncthreads();
    }
  }
}

template <typename T>
static void launch_tiles(const QkvArgs& a, hipStream_t stream) {
  const dim3 grid(a.B * ceil_div(a.N, T::kTok) * ceil_div(a.Hq + 2 * a.Hkv, T::kHeads));
  if (a.y)
    hipLaunchKernelGGL((k_qkv_project<T, true>), grid, dim3(T::kThreads), 0, stream, a);
  else
    hipLaunchKernelGGL((k_qkv_project<T, false>), grid, dim3(T::kThreads), 0, stream, a);
}

// The larger tile is the faster one per token when it fills the chip: a round of
// 256 of them (one per CU) takes as long as 1.46 rounds of 512 small ones (two
// per CU), which cover half as much: 105 against 72 us at D = 4096.  So the small
// tile is taken where it needs clearly fewer rounds, above all where one round of
// large tiles would leave CUs idle.  Measured (large / small, us; 32 + 2 x 8 heads,
// D = 4096): 128 tokens 84 / 48, 777 tokens 91 / 58, 2048 tokens 111 / 119, 4096
// tokens 219 / 215; Phi-3-medium 4 x 4096 tokens 1167 / 1351.
static bool small_tiles(const QkvArgs& a) {
  const long nheads = a.Hq + 2 * a.Hkv;
  auto rounds = [&](int tok, int heads, long slots) {
    const long tiles = (long)a.B * ceil_div(a.N, tok) * ((nheads + heads - 1) / heads);
    return (tiles + slots - 1) / slots;
  };
  return 72 * rounds(QkvSmall::kTok, QkvSmall::kHeads, 512) <
         105 * rounds(QkvLarge::kTok, QkvLarge::kHeads, 256);
}

hipError_t launch_qkv_project(const QkvArgs& a, hipStream_t stream) {
  if (small_tiles(a))
    launch_tiles<QkvSmall>(a, stream);
  else
    launch_tiles<QkvLarge>(a, stream);
  return hipGetLastError();
}

}  // namespace turbo
