// Row LayerNorm with per-tenant gain and shift: y = (x - mean) / sqrt(var + eps) * g_t + b_t,
// biased variance, statistics in fp32.  One wavefront per row; the row's tenant slot is
// found by a binary search of the row's sorted position in the segment token offsets.
// Used after the residual adds of the per-tenant blocks (post-LN) or before the
// sub-layers (pre-LN); the paper leaves these to BERT / GPT's layer definitions.
// An optional second input is added first (residual stream + adapted attention output).
#include "hmi_kernels.h"

#include "wave.h"

#include <utility>

namespace hmi {
namespace {

__device__ __forceinline__ float bf2f(uint16_t u) { return __uint_as_float(((uint32_t)u) << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

constexpr int kMaxPerLane = 32;  // d <= 2048

// Which segment (= whose gain and shift) sorted row srow belongs to, found in a copy of the segment offsets that the workgroup
// puts into LDS with one coalesced read (a search through global memory is a chain of dependent round trips per wavefront).
// All 256 threads call it.
__device__ __forceinline__ int find_segment(const Route& rt, int srow, int* seg_s) {
  const int G = rt.n_segments[0];
  for (int i = threadIdx.x; i <= G; i += 256) seg_s[i] = rt.seg_tok_off[i];
  __syncthreads();
  int lo = 0, hi = G;
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (seg_s[mid] <= srow) lo = mid; else hi = mid;
  }
  return lo;
}

// A lane owns columns lane, lane + 64, ... : PER of them where d = 64 PER, else (fp32 only, PER = 0) as many as there are below d.
// Small launches are latency alone: row, gain and shift are asked for together, in front of the sums (128 rows of d = 64, fp32: with
// the loops of the general form and a search through global memory 5.0 us, now 2.9); in large ones the general form's checks of
// every column cost it half the rate (figures at the launcher).
template <bool BF16, int PER>
__global__ __launch_bounds__(256) void layernorm_kernel(LnArgs a, Route rt) {
  __shared__ int seg_s[kMaxRequests + 1];
  constexpr int MAX = PER ? PER : kMaxPerLane;
  const int lane = threadIdx.x & 63;
  const int srow = min(blockIdx.x * 4 + (int)(threadIdx.x >> 6), a.n_rows - 1);   // sorted row; surplus wavefronts redo the last one
  const size_t row = rt.identity ? (size_t)srow : (size_t)rt.row_src[srow];
  const int d = PER ? PER * 64 : a.d, per = PER ? PER : (d + 63) >> 6;

  float v[MAX];
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < MAX; ++i) {
    v[i] = 0.0f;
    if (PER || (i < per && lane + 64 * i < d)) {
      const size_t idx = row * d + lane + 64 * i;
      if (a.in_f32) v[i] = reinterpret_cast<const float*>(a.in)[idx];
      else v[i] = BF16 ? bf2f(reinterpret_cast<const uint16_t*>(a.in)[idx])
                       : reinterpret_cast<const float*>(a.in)[idx];
      if (a.in2) v[i] += BF16 ? bf2f(reinterpret_cast<const uint16_t*>(a.in2)[idx])
                              : reinterpret_cast<const float*>(a.in2)[idx];
      if (a.sum_out) a.sum_out[idx] = v[i];
    }
  }
  const size_t slot_base = rt.identity ? 0 : (size_t)rt.seg_slot[find_segment(rt, srow, seg_s)] * a.slot_stride;
  auto param = [&](size_t off, int col) {
    const char* p = a.pool + slot_base + off;
    return BF16 ? bf2f(reinterpret_cast<const uint16_t*>(p)[col]) : reinterpret_cast<const float*>(p)[col];
  };
  float gg[PER ? PER : 1], bb[PER ? PER : 1];
  if (PER) {
#pragma unroll
    for (int i = 0; i < PER; ++i) { gg[i] = param(a.g_off, lane + 64 * i); bb[i] = param(a.b_off, lane + 64 * i); }
  }
#pragma unroll
  for (int i = 0; i < MAX; ++i) s += v[i];
  const float mean = wave_sum(s) / (float)d;
  float q = 0.0f;
#pragma unroll
  for (int i = 0; i < MAX; ++i)
    if (PER || (i < per && lane + 64 * i < d)) { const float c = v[i] - mean; q += c * c; }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)d + a.eps);

#pragma unroll
  for (int i = 0; i < MAX; ++i) {
    if (PER || (i < per && lane + 64 * i < d)) {
      const int col = lane + 64 * i;
      const float y = (v[i] - mean) * rstd * (PER ? gg[PER ? i : 0] : param(a.g_off, col)) + (PER ? bb[PER ? i : 0] : param(a.b_off, col));
      const size_t idx = row * d + col;
      if (a.out_f32) a.out_f32[idx] = y;
      if (a.out_st) {
        if (BF16) reinterpret_cast<uint16_t*>(a.out_st)[idx] = f2bf(y);
        else reinterpret_cast<float*>(a.out_st)[idx] = y;
      }
    }
  }
}


typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 load4(const void* p, size_t idx, bool f32) {
  if (f32) return *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p) + idx);
  const u16x4 h = *reinterpret_cast<const u16x4*>(reinterpret_cast<const uint16_t*>(p) + idx);
  f32x4 v = {bf2f(h[0]), bf2f(h[1]), bf2f(h[2]), bf2f(h[3])};
  return v;
}

// Vector path for d % 256 == 0: a lane owns d/256 pieces of 4 consecutive columns
// (16-byte fp32 / 8-byte bf16 accesses, a wavefront covers 1 KB / 512 B contiguous).
template <bool BF16, bool IN_F32, int NV>
__global__ __launch_bounds__(256) void layernorm_vec_kernel(LnArgs a, Route rt) {
  // The row's data is asked for first; whose gain and shift it takes is found while it is on its way.
  __shared__ int seg_s[kMaxRequests + 1];
  const int lane = threadIdx.x & 63;
  const int srow = min(blockIdx.x * 4 + (int)(threadIdx.x >> 6), a.n_rows - 1);   // surplus wavefronts redo the last row
  const bool ident = rt.identity != 0;               // shared parameters: identity row map, slot 0, no search
  const size_t row = ident ? (size_t)srow : (size_t)rt.row_src[srow];
  constexpr int d = NV * 256;
  constexpr bool in_f32 = IN_F32 || !BF16;
  f32x4 v[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = load4(a.in, row * d + i * 256 + lane * 4, in_f32);
  if (a.in2) {
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] += load4(a.in2, row * d + i * 256 + lane * 4, !BF16);
  }
  if (a.sum_out) {
#pragma unroll
    for (int i = 0; i < NV; ++i) *reinterpret_cast<f32x4*>(a.sum_out + row * d + i * 256 + lane * 4) = v[i];
  }
  const size_t slot_base = ident ? 0 : (size_t)rt.seg_slot[find_segment(rt, srow, seg_s)] * a.slot_stride;
  // gain and shift are asked for before the statistics are reduced: they arrive under the reductions
  f32x4 gg[NV], bb[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    gg[i] = load4(a.pool + slot_base + a.g_off, i * 256 + lane * 4, !BF16);
    bb[i] = load4(a.pool + slot_base + a.b_off, i * 256 + lane * 4, !BF16);
  }
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < NV; ++i) s += v[i][0] + v[i][1] + v[i][2] + v[i][3];
  const float mean = wave_sum(s) / (float)d;
  float q = 0.0f;
#pragma unroll
  for (int i = 0; i < NV; ++i)
    {
#pragma unroll
      for (int e = 0; e < 4; ++e) { const float c = v[i][e] - mean; q += c * c; }
    }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)d + a.eps);
#pragma unroll
  for (int i = 0; i < NV; ++i)
    {
      const int col = i * 256 + lane * 4;
      f32x4 y;
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = (v[i][e] - mean) * rstd * gg[i][e] + bb[i][e];
      const size_t idx = row * d + col;
      if (a.out_f32) *reinterpret_cast<f32x4*>(a.out_f32 + idx) = y;
      if (a.out_st) {
        if (BF16) {
          u16x4 h = {f2bf(y[0]), f2bf(y[1]), f2bf(y[2]), f2bf(y[3])};
          *reinterpret_cast<u16x4*>(reinterpret_cast<uint16_t*>(a.out_st) + idx) = h;
        } else {
          *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out_st) + idx) = y;
        }
      }
    }
}

}  // namespace

template <int NV>
static void launch_vec(const LnArgs& a, const Route& rt, hipStream_t s, unsigned blocks) {
  if (!a.bf16) hipLaunchKernelGGL((layernorm_vec_kernel<false, true, NV>), dim3(blocks), dim3(256), 0, s, a, rt);
  else if (a.in_f32) hipLaunchKernelGGL((layernorm_vec_kernel<true, true, NV>), dim3(blocks), dim3(256), 0, s, a, rt);
  else hipLaunchKernelGGL((layernorm_vec_kernel<true, false, NV>), dim3(blocks), dim3(256), 0, s, a, rt);
}

// Whole multiples of 64 columns that layernorm_vec_kernel does not take.
constexpr bool takes_vec(int d) { return d == 256 || d == 512 || d == 768 || d == 1024 || d == 2048; }

template <int PER>
static void launch_whole(const LnArgs& a, const Route& rt, hipStream_t s, unsigned blocks) {
  if constexpr (!takes_vec(64 * PER)) {
    if (a.bf16) hipLaunchKernelGGL((layernorm_kernel<true, PER>), dim3(blocks), dim3(256), 0, s, a, rt);
    else hipLaunchKernelGGL((layernorm_kernel<false, PER>), dim3(blocks), dim3(256), 0, s, a, rt);
  }
}

template <int... I>
static void launch_per(int per, const LnArgs& a, const Route& rt, hipStream_t s, unsigned blocks, std::integer_sequence<int, I...>) {
  ((per == I + 1 ? launch_whole<I + 1>(a, rt, s, blocks) : void()), ...);
}

void launch_layernorm(const LnArgs& a, const Route& rt, hipStream_t s) {
  if (a.n_rows <= 0) return;
  const unsigned blocks = (unsigned)((a.n_rows + 3) / 4);
  switch (a.d) {
    case 256: return launch_vec<1>(a, rt, s, blocks);
    case 512: return launch_vec<2>(a, rt, s, blocks);
    case 768: return launch_vec<3>(a, rt, s, blocks);
    case 1024: return launch_vec<4>(a, rt, s, blocks);
    case 2048: return launch_vec<8>(a, rt, s, blocks);
    default: break;
  }
  // Whole multiples of 64 columns (all there is in bf16): as many a lane as there are.  At every width up to 1 984 that was the faster
  // one, us, general form and this: 128 rows of 384, 960, 1 984 fp32 6.2, 7.8, 10.7 and 2.8, 4.0, 5.7; 16 384 rows 23.9, 39.7, 85.0
  // and 12.1, 22.4, 51.8; bf16 16 384 rows 23.5, 38.7, 77.3 and 11.0, 20.3, 41.1.
  if (a.d % 64 == 0) return launch_per(a.d / 64, a, rt, s, blocks, std::make_integer_sequence<int, kMaxPerLane>());
  hipLaunchKernelGGL((layernorm_kernel<false, 0>), dim3(blocks), dim3(256), 0, s, a, rt);
}

}  // namespace hmi
