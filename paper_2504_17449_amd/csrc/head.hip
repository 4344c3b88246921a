// Per-tenant output heads (Sec. 3.3.2 of the paper): a linear layer per tenant on the final hidden states,
// classification tenants on the first row of a request, tagging tenants on every row, label = class of the highest
// score (lowest index on ties).
//
// One kernel, one workgroup of four wavefronts per 32 rows of a request.  Only rows that get a prediction are read (three
// tenants in ten tag every row): the launch is bound by those reads and, for small batches, by the chain of one
// workgroup's loads, all of which miss.  So the four wavefronts take a quarter of d each, of all 32 rows and of the
// tenant's one or two blocks of 32 classes, with six k-steps' operands in flight straight from memory (d = 768: two round
// trips, four workgroups on a compute unit), and their sums meet in LDS in a fixed order.  Weights are the MFMA's first operand, in a permuted row
// order, so that a lane holds 16 consecutive classes of one row: the arg-max is in registers, plus one exchange with the
// lane that holds the other half.
//
// Measured, d = 768, up to 32 classes (before: all rows times 64 classes as a grouped GEMM, then a kernel that masked and
// compared, one request per workgroup): 65 536 rows of 512 requests 86 us -> 40; 2 664 rows of 37 requests 45 -> 10; 141
// rows of two requests 32 -> 10.
#include "hmi_kernels.h"

#include <math.h>

namespace hmi {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));   // the caller's scores may begin at any float

constexpr int kChunkRows = 32;
constexpr int kInFlight = 6;    // k-steps whose operands a wavefront has in flight (12: half as many workgroups fit a compute unit)

__device__ __forceinline__ float bf2f(uint16_t u) { return __uint_as_float(((uint32_t)u) << 16); }
// MFMA first-operand position i <- weight row perm_w(i) of the 32-row block: output register r of lane half h is class 16 h + r
__device__ __forceinline__ int perm_w(int i) { return ((i >> 2) & 1) * 16 + (i >> 3) * 4 + (i & 3); }

template <bool BF16>
__device__ __forceinline__ void mfma_chunk(const u32x4& w, const u32x4& x, f32x16& acc) {
  if (BF16) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
  } else {
    const f32x4 wf = __builtin_bit_cast(f32x4, w), xf = __builtin_bit_cast(f32x4, x);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[e], xf[e], acc, 0, 0, 0);
  }
}

template <bool BF16>
__global__ __launch_bounds__(256, 4) void head_kernel(HeadArgs a, Route rt) {
  __shared__ float part[3][2][16 * 64];
  constexpr int ES = BF16 ? 2 : 4;
  const int r = blockIdx.y, i0 = blockIdx.x * kChunkRows;
  const int start = rt.tok_off[r], len = rt.tok_off[r + 1] - start;
  if (i0 >= len) return;
  const int tenant = rt.req_tenant[r];
  const int n_classes = a.meta[2 * tenant], per_token = a.meta[2 * tenant + 1];
  const int rows = min(kChunkRows, len - i0);
  const int n_pred = per_token ? rows : (i0 == 0 ? 1 : 0);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l32 = lane & 31, lh = lane >> 5;
  const size_t first = (size_t)start + i0;

  // ---- rows without a prediction
  for (int i = n_pred + (int)threadIdx.x; i < rows; i += 256) a.labels[first + i] = -1;
  if (a.scores) {
    float* sc = a.scores + (first + n_pred) * a.max_classes;
    const int n = (rows - n_pred) * a.max_classes;
    for (int i = threadIdx.x; i < n; i += 256) sc[i] = -INFINITY;
  }
  if (n_pred == 0) return;

  // ---- this wavefront's quarter of d of 32 rows times one or two blocks of 32 classes
  const bool two = n_classes > 32;
  const char* head = a.heads + (size_t)tenant * a.head_stride;
  const char* xp = a.h + (first + min(l32, n_pred - 1)) * (size_t)(a.d * ES) + lh * 16;
  const char* wp = head + (size_t)(perm_w(l32) * a.d) * ES + lh * 16;
  const size_t w2 = (size_t)(32 * a.d) * ES;
  const int steps = a.d * ES / 32;                       // k-steps of two 16-byte chunks
  const int k0 = wave * steps / 4, k1 = (wave + 1) * steps / 4;
  f32x16 acc[2] = {};
  for (int k = k0; k < k1; k += kInFlight) {             // (surplus steps of the last trip repeat a valid one and are not multiplied)
    u32x4 x[kInFlight], wa[kInFlight], wb[kInFlight];
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      const int off = min(k + u, k1 - 1) * 32;
      x[u] = *reinterpret_cast<const u32x4*>(xp + off);
      wa[u] = *reinterpret_cast<const u32x4*>(wp + off);
      if (two) wb[u] = *reinterpret_cast<const u32x4*>(wp + w2 + off);
    }
#pragma unroll
    for (int u = 0; u < kInFlight; ++u)
      if (k + u < k1) {
        mfma_chunk<BF16>(wa[u], x[u], acc[0]);
        if (two) mfma_chunk<BF16>(wb[u], x[u], acc[1]);
      }
  }
  if (wave > 0) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) part[wave - 1][b][e * 64 + lane] = acc[b][e];
  }
  __syncthreads();
  if (wave > 0) return;
#pragma unroll
  for (int w = 0; w < 3; ++w)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[b][e] += part[w][b][e * 64 + lane];

  // ---- bias, mask, arg-max: this lane's classes are 32 b + 16 lh + e in ascending order of (b, e)
  float best = -INFINITY;
  int label = 16 * lh;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int c = 32 * b + 16 * lh + e;
      const char* bp = head + a.b_off + (size_t)c * ES;
      const float v = c < n_classes ? acc[b][e] + (BF16 ? bf2f(*reinterpret_cast<const uint16_t*>(bp)) : *reinterpret_cast<const float*>(bp)) : -INFINITY;
      acc[b][e] = v;
      if (v > best) { best = v; label = c; }
    }
  const float other = __shfl_xor(best, 32, 64);
  const int other_label = __shfl_xor(label, 32, 64);
  if (other > best || (other == best && other_label < label)) label = other_label;
  if (l32 >= n_pred) return;
  const size_t row = first + l32;
  if (lh == 0) a.labels[row] = label;
  if (a.scores) {
    float* sc = a.scores + row * a.max_classes;
    if (a.max_classes % 4 == 0) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int c = 32 * b + 16 * lh + 4 * q;
          if (c < a.max_classes) *reinterpret_cast<f32x4_any*>(sc + c) = f32x4{acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]};
        }
    } else {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int c = 32 * b + 16 * lh + e;
          if (c < a.max_classes) sc[c] = acc[b][e];
        }
    }
  }
}

}  // namespace

void launch_head(const HeadArgs& a, const Route& rt, int R, int longest, bool bf16, hipStream_t s) {
  if (R <= 0) return;
  const dim3 grid((longest + kChunkRows - 1) / kChunkRows, R);
  if (bf16) hipLaunchKernelGGL(head_kernel<true>, grid, dim3(256), 0, s, a, rt);
  else hipLaunchKernelGGL(head_kernel<false>, grid, dim3(256), 0, s, a, rt);
}

}  // namespace hmi
