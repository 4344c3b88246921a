// bf16 GEMM for a few rows through weights that all tenants share (a decode step of a few conversations, a request or two on an idle
// server): launches that are one trip to the weights and back, if they are let.
//
//   C[rows, :] = epi(A[rows, :] * W^T + b),  rows in order (the dense route), W [n_out, k]
//
// What bounds it.  A launch that only reads costs 2.4 us here, launching, arguments and one trip to memory; a compute unit that asks for
// 96 KB at once gets them within that, for 192 KB it takes 3.1 us (7 to 96 workgroups, weights not in L2).  Provided that each four
// lanes in turn cover 64 contiguous bytes: with the lanes in the order of an MFMA fragment (16 rows x 64 bytes, neighbours in different
// rows) the same 96 and 192 KB take 4.0 and 6.5 us.  The kernels that go through a ring in LDS wait for several trips, one
// behind the other (768 columns of k = 3072: twelve stages, three of them in flight).  So
//   * a workgroup is 16 columns x up to 16 rows x all of k, its twelve wavefronts share out k in units of 128, and every load of the
//     launch is issued before the first is waited for, straight into registers;
//   * a load covers 4 rows x 256 bytes, 64 bytes of a row to four neighbours, and that is a fragment of
//     v_mfma_f32_16x16x32_bf16 all the same: operand row 4 r + c holds pieces c, 4 + c, 8 + c and 12 + c (16 bytes each) of row r, for
//     weights and activations alike.  Of the 16 x 16 products of two such fragments those with the same c on both sides are meant, four
//     of which make an element: register c of lane c in each four lanes, added up across them.  Three quarters of the matrix
//     cores' work is thrown away, of which there is plenty;
//   * an element's sums, one a wavefront, meet in LDS, and one thread adds them up in a fixed order;
//   * a column block's row blocks are on one XCD (workgroups are dealt to the XCDs round robin), whose L2 fetches its weights once.
#include "hmi_kernels.h"

#include "gelu.h"
#include "wave.h"

namespace hmi {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kXcds = 8;
constexpr int WAVES = 12, COLS = 16, UNIT = 128;             // bf16 of a row that a load covers

__device__ __forceinline__ float bf2f(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// UNITS: units of k of a wavefront at most; HG: blocks of 4 columns of a wavefront (all four, or half of them where k has at most six
// units and wavefronts w and w + units share one); MG: blocks of 4 rows
template <int UNITS, int HG, int MG>
__global__ __launch_bounds__(64 * WAVES) void gemm_bf16_thin_kernel(GemmArgs g) {
  __shared__ float part[WAVES][4][MG][4][4];                 // [sum][4 columns][4 rows][row][column]
  const int row_blocks = (g.n_rows + 4 * MG - 1) / (4 * MG);
  const int local = (int)blockIdx.x / kXcds, c = local / row_blocks;
  const int n0 = (c * kXcds + (int)blockIdx.x % kXcds) * COLS, row0 = (local - c * row_blocks) * 4 * MG;
  if (n0 >= g.n_out) return;
  const int rows = min(4 * MG, g.n_rows - row0);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sub = lane & 3, r4 = (lane >> 2) & 3, lq = lane >> 4, at = (lq * 4 + sub) * 8;

  const int units = g.k / UNIT, sums = min(units, WAVES);
  const int first = HG == 4 ? wave : wave % units, g0 = HG == 4 ? 0 : wave / units * HG;
  const bool mine = HG == 4 ? wave < units : g0 < 4;         // (of the whole wavefront; the others load what nobody multiplies)
  const uint16_t* const wp = reinterpret_cast<const uint16_t*>(g.pool + g.w_off) + (size_t)(n0 + min(g0, 4 - HG) * 4 + r4) * g.k + at;
  const uint16_t* xp[MG];
#pragma unroll
  for (int j = 0; j < MG; ++j) xp[j] = reinterpret_cast<const uint16_t*>(g.A) + (size_t)(row0 + min(j * 4 + r4, rows - 1)) * g.lda + at;
  bf16x8 wf[UNITS][HG], xf[UNITS][MG];
#pragma unroll
  for (int b = 0; b < UNITS; ++b) {
    const int unit = min(first + b * WAVES, units - 1);
#pragma unroll
    for (int h = 0; h < HG; ++h) wf[b][h] = *reinterpret_cast<const bf16x8*>(wp + (size_t)(4 * h) * g.k + unit * UNIT);
#pragma unroll
    for (int j = 0; j < MG; ++j) xf[b][j] = *reinterpret_cast<const bf16x8*>(xp[j] + unit * UNIT);
  }
  // the element this thread brings to its end, its bias and residual
  const int e_row = min(tid >> 4, 4 * MG - 1), e_col = tid & 15;
  const size_t out_row = (size_t)(row0 + min(e_row, rows - 1));
  const uint32_t bias = reinterpret_cast<const uint16_t*>(g.pool + g.b_off)[n0 + e_col];
  float resid = 0.0f;
  if (g.epi == EPI_BIAS_RESID) {
    const size_t r_at = out_row * g.ldr + n0 + e_col;
    resid = g.resid_f32 ? reinterpret_cast<const float*>(g.resid)[r_at] : bf2f(reinterpret_cast<const uint16_t*>(g.resid)[r_at]);
  }
  __builtin_amdgcn_sched_barrier(0);
  if (mine) {
    f32x4 acc[HG][MG] = {};
#pragma unroll
    for (int b = 0; b < UNITS; ++b)
      if (first + b * WAVES < units) {
#pragma unroll
        for (int h = 0; h < HG; ++h)
#pragma unroll
          for (int j = 0; j < MG; ++j) acc[h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[b][h], xf[b][j], acc[h][j], 0, 0, 0);
      }
    // register e of lane (lq, r4, sub): column lq, row r4, its pieces e and sub
#pragma unroll
    for (int h = 0; h < HG; ++h)
#pragma unroll
      for (int j = 0; j < MG; ++j) {
        float v = sub == 0 ? acc[h][j][0] : sub == 1 ? acc[h][j][1] : sub == 2 ? acc[h][j][2] : acc[h][j][3];
        v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xf, 0xf, false));   // lanes 1 0 3 2
        v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x4E, 0xf, 0xf, false));   // lanes 2 3 0 1
        if (sub == 0) part[first][g0 + h][j][r4][lq] = v;
      }
  }
  HMI_BARRIER();
  if (tid >= COLS * 4 * MG || e_row >= rows) return;
  float v = 0.0f;
#pragma unroll
  for (int p = 0; p < WAVES; ++p)
    if (p < sums) v += part[p][e_col >> 2][e_row >> 2][e_row & 3][e_col & 3];
  v += bf2f(bias);
  if (g.epi == EPI_BIAS_GELU) v = gelu_f32(v);
  else if (g.epi == EPI_BIAS_RELU) v = fmaxf(v, 0.0f);
  else if (g.epi == EPI_BIAS_RESID) v += resid;
  const size_t o = out_row * g.ldc + n0 + e_col;
  if (g.out_f32) reinterpret_cast<float*>(g.C)[o] = v;
  else reinterpret_cast<uint16_t*>(g.C)[o] = f2bf(v);
  if (g.C2) reinterpret_cast<uint16_t*>(g.C2)[o] = f2bf(v);
}

template <int UNITS, int HG>
void launch_units(const GemmArgs& g, hipStream_t s) {
  const int mg = g.n_rows <= 4 ? 1 : g.n_rows <= 8 ? 2 : 4;
  const unsigned grid = (unsigned)((g.n_rows + 4 * mg - 1) / (4 * mg)) * (unsigned)((g.n_out / COLS + kXcds - 1) / kXcds * kXcds);
  if (mg == 1) hipLaunchKernelGGL((gemm_bf16_thin_kernel<UNITS, HG, 1>), dim3(grid), dim3(64 * WAVES), 0, s, g);
  else if (mg == 2) hipLaunchKernelGGL((gemm_bf16_thin_kernel<UNITS, HG, 2>), dim3(grid), dim3(64 * WAVES), 0, s, g);
  else hipLaunchKernelGGL((gemm_bf16_thin_kernel<UNITS, HG, 4>), dim3(grid), dim3(64 * WAVES), 0, s, g);
}

}  // namespace

// A round of workgroups; of a GELU launch with a short k, two of which fit a compute unit, two (there a lane of the other kernels
// brings sixteen elements to their end, here each thread one).  Per launch, d = 768, f = 3072, the other kernels and this one, us:
//   rows                 1         8         16        24        40        80        96
//   QKV                  4.5, 3.7  4.5, 3.8  4.7, 4.4  4.8, 5.0  -         -         -          (two rounds from 17 rows on)
//   output projection    4.4, 3.6  4.4, 3.6  4.6, 4.2  4.9, 4.1  4.3, 4.2  4.5, 4.3  4.8, 4.2   (from 81 rows on)
//   FFN1 with GELU       5.6, 3.9  5.0, 4.1  5.6, 4.2  5.6, 4.6  -         -         -
//   FFN2 (k = 3072)      6.3, 4.4  6.4, 5.0  7.1, 5.9  7.8, 5.9  7.7, 6.0  8.3, 6.2  7.8, 8.2   (from 81 rows on)
// A decode step of 7 requests through six layers 228 us -> 206.
bool gemm_bf16_thin_fits(int n_rows, int n_out, int k, bool gelu, int n_cu) {
  if (n_out % COLS || k % UNIT || k > 3 * WAVES * UNIT) return false;
  return (long long)((n_rows + 15) / 16) * (n_out / COLS) <= (gelu && 2 * (k / UNIT) <= WAVES ? 2LL : 1LL) * n_cu;
}

void launch_gemm_bf16_thin(const GemmArgs& g, hipStream_t s) {
  const int units = g.k / UNIT;
  if (2 * units <= WAVES) return launch_units<1, 2>(g, s);
  if (units <= WAVES) return launch_units<1, 4>(g, s);
  if (units <= 2 * WAVES) return launch_units<2, 4>(g, s);
  launch_units<3, 4>(g, s);
}

}  // namespace hmi

// The rule alone, for the tests: whether a launch of that many rows through shared weights is this kernel's.
extern "C" int32_t hmi_internal_gemm_thin(int32_t n_rows, int32_t n_out, int32_t k, int32_t gelu, int32_t n_cu) {
  return hmi::gemm_bf16_thin_fits(n_rows, n_out, k, gelu, n_cu);
}
