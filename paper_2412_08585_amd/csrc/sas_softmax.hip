// Algorithm 3 (Appendix B) on gfx950: the SAS softmax of every row of a
// float matrix, as a stand-alone operation.  Per row: m = max, e_c =
// SAS(x_c - m) (the same binary32 steps as the attention kernels: y = m - x,
// threshold, LUT[floor y] * POLY(y - floor y)), then e_c / sum_c e_c.
//
// The operation reads and writes each element once, so it is bound by HBM.
// Rows of up to 2048 values are held in the registers of one wave (four
// rows per work-group); longer rows use one 256-thread work-group, in
// registers up to 16384 values (17405 in rows that are not 16-byte aligned) and
// in three streaming passes beyond.
#include "turbo_common.h"
#include "stream_loads.h"

namespace turbo {

struct SasSoftmaxArgs {
  const float* x;  // [rows][cols]
  float* y;        // [rows][cols]
  long rows;
  int cols;
};

__device__ __forceinline__ float wave_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xf, 0xf, false));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xf, 0xf, false));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xf, 0xf, false));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xf, 0xf, false));
  const unsigned u = __float_as_uint(v);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  return add_xor32(v);
}

// How a row lies in memory.  Its chunks of four values are the 16-byte units
// of the address space it touches, so that every whole chunk is one vector
// access wherever the row starts: a row of a ragged matrix starts up to 3 values
// into its first unit.  40040 rows of 1001: 55.5 us, 5.8 TB/s, against 91 us with
// scalar accesses wherever cols % 4 != 0.
template <bool kShift>
struct Row {
  const float* x;
  float* y;
  int C;
  int sx;   // values before the row in its first 16-byte unit (kShift)
  bool vy;  // the output row lies likewise: vector stores

  __device__ __forceinline__ Row(const SasSoftmaxArgs& a, long row)
      : x(a.x + row * a.cols), y(a.y + row * a.cols), C(a.cols), sx(0), vy(true) {
    if constexpr (kShift) {
      sx = (int)(reinterpret_cast<uintptr_t>(x) >> 2) & 3;
      vy = ((int)(reinterpret_cast<uintptr_t>(y) >> 2) & 3) == sx;
    }
  }
  // first column of chunk i of thread t (T threads); it may be negative
  template <int T>
  __device__ __forceinline__ int col(int t, int i) const {
    return 4 * (t + T * i) - (kShift ? sx : 0);
  }
  __device__ __forceinline__ bool whole(int c) const {
    return (!kShift || c >= 0) && c + 3 < C;
  }
  __device__ __forceinline__ bool has(int c) const { return (!kShift || c >= 0) && c < C; }
};

// Chunk i of thread t; columns outside the row read as -inf.  kNT: the row is
// read once (held in registers), so the vector loads stream.
template <int T, bool kNT, bool kShift>
__device__ __forceinline__ float4 load4(const Row<kShift>& r, int t, int i) {
  const int c = r.template col<T>(t, i);
  if (r.whole(c)) {
    if (kNT) {
      const u32x4_t u = load_nt4(r.x + c);
      return make_float4(__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z),
                         __uint_as_float(u.w));
    }
    return *reinterpret_cast<const float4*>(r.x + c);
  }
  float4 v;
  v.x = r.has(c) ? r.x[c] : -INFINITY;
  v.y = r.has(c + 1) ? r.x[c + 1] : -INFINITY;
  v.z = r.has(c + 2) ? r.x[c + 2] : -INFINITY;
  v.w = r.has(c + 3) ? r.x[c + 3] : -INFINITY;
  return v;
}

// Stores of one output row in the same chunks.  The output is written once
// and not read again by this launch, so the vector stores stream
// (non-temporal): 3-4 % faster on the 2.7 GB workload.
typedef float f32x4_t __attribute__((ext_vector_type(4)));
template <int T, bool kShift>
__device__ __forceinline__ void store4(const Row<kShift>& r, int t, int i, float4 v) {
  const int c = r.template col<T>(t, i);
  if (r.vy && r.whole(c)) {
    __builtin_nontemporal_store(f32x4_t{v.x, v.y, v.z, v.w}, reinterpret_cast<f32x4_t*>(r.y + c));
    return;
  }
  if (r.has(c)) r.y[c] = v.x;
  if (r.has(c + 1)) r.y[c + 1] = v.y;
  if (r.has(c + 2)) r.y[c + 2] = v.z;
  if (r.has(c + 3)) r.y[c + 3] = v.w;
}

__device__ __forceinline__ float4 sas4(float m, float4 v, const float* lut) {
  return make_float4(sas_y(m - v.x, lut), sas_y(m - v.y, lut), sas_y(m - v.z, lut),
                     sas_y(m - v.w, lut));
}

__device__ __forceinline__ float4 div4(float4 v, float s) {
  return make_float4(v.x / s, v.y / s, v.z / s, v.w / s);
}

// One wave per row, the row in registers: NV chunks of four per lane.
template <int NV, bool kShift>
__global__ __launch_bounds__(256) void k_sas_softmax_wave(SasSoftmaxArgs a) {
  __shared__ float lut[8];
  if (threadIdx.x < 8) lut[threadIdx.x] = kLut[threadIdx.x];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= a.rows) return;  // wave-uniform; no barrier follows
  const Row<kShift> r(a, row);
  float4 v[NV];
  float m = -INFINITY;
  // The row's loads are issued at raised priority, ahead of the arithmetic
  // of the other waves of the SIMD.
  __builtin_amdgcn_s_setprio(2);
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = load4<64, true>(r, lane, i);
  __builtin_amdgcn_s_setprio(0);
#pragma unroll
  for (int i = 0; i < NV; ++i)
    m = fmaxf(m, fmaxf(fmaxf(v[i].x, v[i].y), fmaxf(v[i].z, v[i].w)));
  m = wave_max_fast(m);
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    v[i] = sas4(m, v[i], lut);
    s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
  }
  s = wave_sum(s);
#pragma unroll
  for (int i = 0; i < NV; ++i) store4<64>(r, lane, i, div4(v[i], s));
}

__device__ __forceinline__ float block_reduce(float v, float* red, bool is_max) {
  v = is_max ? wave_max_fast(v) : wave_sum(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  const float r = is_max ? fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]))
                         : (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return r;
}

// One 256-thread work-group per row.  NV > 0: the row in registers (NV
// chunks of four per thread); NV == 0: three passes over memory.
template <int NV, bool kShift>
__global__ __launch_bounds__(256) void k_sas_softmax_block(SasSoftmaxArgs a) {
  __shared__ float lut[8];
  __shared__ float red[4];
  const int t = threadIdx.x;
  if (t < 8) lut[t] = kLut[t];
  __syncthreads();
  const long row = blockIdx.x;
  const Row<kShift> r(a, row);
  const int nch = (a.cols + (kShift ? r.sx : 0) + 1023) / 1024;  // chunks of four per thread
  if (NV > 0) {
    float4 v[NV > 0 ? NV : 1];
    float m = -INFINITY;
    __builtin_amdgcn_s_setprio(2);  // the row's loads first (2 % on 4096-column rows)
    // Up to 8192 aligned values a wave takes its chunks one after the other:
    // the row's other waves keep the memory busy, and rows of 4096 run 858 us
    // instead of 889 (163840 rows), rows of 8192 111 instead of 116 (10000).
    // Longer rows (16384: 131 against 120 us) and shifted ones (2049: 68 / 65)
    // load all chunks at once.
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      v[i] = load4<256, true>(r, t, i);
      if (!kShift && NV <= 8) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int i = 0; i < NV; ++i)
      m = fmaxf(m, fmaxf(fmaxf(v[i].x, v[i].y), fmaxf(v[i].z, v[i].w)));
    m = block_reduce(m, red, true);
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      v[i] = sas4(m, v[i], lut);
      s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    }
    s = block_reduce(s, red, false);
#pragma unroll
    for (int i = 0; i < NV; ++i) store4<256>(r, t, i, div4(v[i], s));
  } else {
    float m = -INFINITY;
    for (int i = 0; i < nch; ++i) {
      const float4 v = load4<256, false>(r, t, i);
      m = fmaxf(m, fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
    }
    m = block_reduce(m, red, true);
    float s = 0.0f;
    for (int i = 0; i < nch; ++i) {
      const float4 e = sas4(m, load4<256, false>(r, t, i), lut);
      s += (e.x + e.y) + (e.z + e.w);
    }
    s = block_reduce(s, red, false);
    for (int i = 0; i < nch; ++i)
      store4<256>(r, t, i, div4(sas4(m, load4<256, false>(r, t, i), lut), s));
  }
}

template <bool kShift>
static void launch_softmax(const SasSoftmaxArgs& a, hipStream_t stream) {
  const int C = a.cols + (kShift ? 3 : 0);  // values in the chunks of a row, at most
  const dim3 wgrid((unsigned)((a.rows + 3) / 4)), bgrid((unsigned)a.rows), block(256);
  if (C <= 256)
    hipLaunchKernelGGL((k_sas_softmax_wave<1, kShift>), wgrid, block, 0, stream, a);
  else if (C <= 512)
    hipLaunchKernelGGL((k_sas_softmax_wave<2, kShift>), wgrid, block, 0, stream, a);
  else if (C <= 1024)
    hipLaunchKernelGGL((k_sas_softmax_wave<4, kShift>), wgrid, block, 0, stream, a);
  else if (C <= 2048)
    hipLaunchKernelGGL((k_sas_softmax_wave<8, kShift>), wgrid, block, 0, stream, a);
  else if (C <= 4096)
    hipLaunchKernelGGL((k_sas_softmax_block<4, kShift>), bgrid, block, 0, stream, a);
  else if (C <= 8192)
    hipLaunchKernelGGL((k_sas_softmax_block<8, kShift>), bgrid, block, 0, stream, a);
  else if (C <= (kShift ? 17408 : 16384))  // a shifted row of 16384 needs one more chunk
    hipLaunchKernelGGL((k_sas_softmax_block<kShift ? 17 : 16, kShift>), bgrid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((k_sas_softmax_block<0, kShift>), bgrid, block, 0, stream, a);
}

hipError_t launch_sas_softmax(const SasSoftmaxArgs& a, hipStream_t stream) {
  // rows that all start on a 16-byte unit need no per-row shift
  const bool aligned = a.cols % 4 == 0 && reinterpret_cast<uintptr_t>(a.x) % 16 == 0 &&
                       reinterpret_cast<uintptr_t>(a.y) % 16 == 0;
  if (aligned)
    launch_softmax<false>(a, stream);
  else
    launch_softmax<true>(a, stream);
  return hipGetLastError();
}

}  // namespace turbo
