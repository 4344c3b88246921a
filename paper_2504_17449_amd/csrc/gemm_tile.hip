// Grouped GEMM with one workgroup per tile, for bf16 and fp32 pools: every launch that neither fills the chip with the
// persistent 256 x 256 tiles (gemm_bf16_p256.hip) nor is a stream of weights past a handful of rows
// (gemm_bf16_skinny.hip), and every shape those two do not take.  The rule that picks one stands at the end of this file.
//
// Computes, for every m-tile the router emitted (all rows of a tile belong to one tenant segment g):
//      C[rows, :] = epi( A[rows, :] * W_g^T + b_g )
// where W_g ([n_out, k] row-major, i.e. Linear(a) = W a + b of Sec. 3.2.2) is read from the HBM slot of segment g.
// This is the "different requests, different parameters, one launch" step of Sec. 6.3 without materialising
// per-request parameter copies.
//
// What bounds it, and what follows
//   * A compute unit takes 66 bytes per clock through its L1, whether into LDS or into registers (measured; LDS reads
//     270): a stage of a 128 x 128 tile is 512 clocks of copies and 512 of MFMAs.  They only overlap if they are issued by
//     different wavefronts: a wavefront that has copies to issue stands still until L1 takes them (measured: 8 MFMAs and
//     4 copies in one instruction stream take 357 clocks for 249 of either).  So a workgroup is four consumers, WM x WN
//     over the BM x BN tile, which read LDS and multiply, and four producers, which do nothing but copy: one launch of
//     768 x 3072 weights over 100 rows 28.8 -> 23.7 us with 128 x 128 tiles, 15.9 -> 11.4 with 64 x 64.
//   * Operands come in stages of 128 bytes of k per row (64 bf16 or 32 fp32: one cache line, eight lanes fetch a row's
//     line) by direct-to-LDS copies into a ring of STAGES, one barrier per stage.
//   * A 16-byte chunk of a row is one fragment read: one v_mfma_f32_32x32x16_bf16, or four v_mfma_f32_32x32x2_f32
//     (element e of the two lane halves' chunks is one k-step of two; the k order inside a stage is the same for both
//     operands, so it does not matter that it is not ascending).  fp32 products go to two accumulators in turn: a sum of half
//     as many, whose rounding errors are 0.7 of one chain's (in one chain fp32 layers were 1.3 % further from 64 bits than
//     with the vector ALU's fused chain; two encoder layers of 1 728 rows 672.5 us with one, 673.1 with two).
//   * Weights are the MFMA's first operand, in a permuted row order, so that a lane ends up with 16 consecutive columns
//     of one row of C: the epilogue reads residuals and writes results straight from the accumulators in 16-byte pieces.
//     Accumulators start at the bias.
//   * Workgroup ids are folded so that each of the 8 XCDs (which get workgroups round robin) works on a contiguous range
//     of tiles, m-tile by m-tile: an activation panel is fetched by one XCD.
// Measured (d = 768, f = 3072, one weight set; persistent tiles before, this kernel now): 2 664 rows: QKV 22.1 -> 15.6 us,
// output projection 20.6 -> 7.0, FFN1 25.6 -> 23, FFN2 71.7 -> 21.9; 8 192 rows: FFN2 75 -> 50.6.  fp32
// (before: products on the vector ALU): 1 728 rows of eight tenants, two encoder layers with their attention: 1.28 -> 0.67 ms.
#include "hmi_kernels.h"

#include "gelu.h"

#include <algorithm>

namespace hmi {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));   // in the caller's result, which may begin at any float
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* glb_ptr_t;

constexpr int kXcds = 8;
constexpr int NW = 4;                     // consumer wavefronts
constexpr int ROW_BYTES = 128;            // k bytes of a row and stage

#define HMI_WAIT_LGKMCNT0() __builtin_amdgcn_s_waitcnt(0xC07F)
#define HMI_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(((N) & 0xF) | (((N) >> 4) << 14) | (0x7 << 4) | (0xF << 8))

__device__ __forceinline__ float bf2f(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 p = {(__bf16)lo, (__bf16)hi};                       // round to nearest even
  return __builtin_bit_cast(uint32_t, p);
}

// LDS chunk swizzles (a row is 8 chunks of 16 bytes): activation rows are read by consecutive lanes, weight rows in
// the order perm_w; either way the 16 lanes served together hit 16 different chunks.  perm_w places the weight rows
// so that output register r of lane half h is column 16 h + r of the MFMA tile.
__device__ __forceinline__ int swz_a(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int swz_w(int row) { return ((row >> 1) & 3) | (((row >> 4) & 1) << 2); }
__device__ __forceinline__ int perm_w(int i) { return ((i >> 2) & 1) * 16 + (i >> 3) * 4 + (i & 3); }

template <bool BF16>
__device__ __forceinline__ void mfma_chunk(const u32x4& w, const u32x4& x, f32x16& acc, f32x16& acc2) {
  if (BF16) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
  } else {
    const f32x4 wf = __builtin_bit_cast(f32x4, w), xf = __builtin_bit_cast(f32x4, x);
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[e], xf[e], acc, 0, 0, 0);
      acc2 = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[e + 1], xf[e + 1], acc2, 0, 0, 0);
    }
  }
}

template <bool BF16, int BM, int BN, int WM, int WN, int STAGES, int NP>
__global__ __launch_bounds__(64 * (NW + NP)) void gemm_tile_kernel(GemmArgs g, Route rt, int total, int tiles_per_entry) {
  static_assert(WM * WN == NW, "four wavefronts");
  constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  constexpr int A_LD = BM / 8 / NP, W_LD = BN / 8 / NP;      // 1 KB copies (8 rows) per producer and stage
  constexpr int LD = A_LD + W_LD;
  constexpr int STAGE_BYTES = (BM + BN) * ROW_BYTES;
  constexpr int ES = BF16 ? 2 : 4;
  static_assert(LD * (STAGES - 1) < 64, "vmcnt range");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  // ---- which tile: m-tile by m-tile, an entry of the route's list holds tiles_per_entry tiles of BM rows
  const int nt_n = (g.n_out + BN - 1) / BN;
  const int per = (total + kXcds - 1) / kXcds;
  const int local = blockIdx.x / kXcds;
  const int w = (blockIdx.x % kXcds) * per + local;
  if (local >= per || w >= total) return;
  const int mt = w / nt_n, n0 = (w - mt * nt_n) * BN;
  const bool ident = rt.identity != 0;      // the shared parameters' route: tiles in row order, identity row map, slot 0
  int row0, row_end;
  size_t slot_base = 0;
  if (ident) {
    row0 = mt * BM;
    row_end = g.n_rows;
  } else {
    const int entry = mt / tiles_per_entry;
    const int seg = rt.tile_seg[g.which_tiles][entry];
    row0 = rt.tile_row0[g.which_tiles][entry] + (mt - entry * tiles_per_entry) * BM;
    row_end = rt.seg_tok_off[seg + 1];
    slot_base = (size_t)rt.seg_slot[seg] * g.slot_stride;
  }
  const int rows = min(BM, row_end - row0);
  if (rows <= 0) return;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kbytes = g.k * ES;
  const int KT = kbytes / ROW_BYTES;        // whole stages; fp32 shapes may leave half a stage (64 bytes) behind
  const bool half_stage = !BF16 && kbytes % ROW_BYTES != 0;

  if (wave >= NW) {
    // ================= producers: copies only =================
    // Lane l of a 1 KB copy fills (row l / 8, chunk position l % 8) with the row's chunk position ^ swizzle.  Rows past
    // the end of a short tile repeat its last row, weight rows past n_out the last one.
    const int pw = wave - NW;
    uint32_t a_off[A_LD], w_off[W_LD];
#pragma unroll
    for (int j = 0; j < A_LD; ++j) {
      const int row = (pw * A_LD + j) * 8 + (lane >> 3);
      const int r = row0 + min(row, rows - 1);
      a_off[j] = (uint32_t)(ident ? r : rt.row_src[r]) * (uint32_t)(g.lda * ES) + (((lane & 7) ^ swz_a(row)) << 4);
    }
#pragma unroll
    for (int j = 0; j < W_LD; ++j) {
      const int row = (pw * W_LD + j) * 8 + (lane >> 3);
      w_off[j] = (uint32_t)min(n0 + row, g.n_out - 1) * (uint32_t)(g.k * ES) + (((lane & 7) ^ swz_w(row)) << 4);
    }
    const char* a_next = reinterpret_cast<const char*>(g.A);   // the stage of k that is copied next (uniform)
    const char* w_next = g.pool + slot_base + g.w_off;
    auto copy_stage = [&](int slot_off) {
      unsigned char* dst = smem + slot_off;
#pragma unroll
      for (int j = 0; j < A_LD; ++j)
        __builtin_amdgcn_global_load_lds((glb_ptr_t)(a_next + a_off[j]), (lds_ptr_t)(dst + (pw * A_LD + j) * 1024), 16, 0, 0);
#pragma unroll
      for (int j = 0; j < W_LD; ++j)
        __builtin_amdgcn_global_load_lds((glb_ptr_t)(w_next + w_off[j]), (lds_ptr_t)(dst + BM * ROW_BYTES + (pw * W_LD + j) * 1024), 16, 0, 0);
      a_next += ROW_BYTES; w_next += ROW_BYTES;
    };
#pragma unroll
    for (int p = 0; p < STAGES - 1; ++p)
      if (p < KT) copy_stage(p * STAGE_BYTES);
    int fill = (STAGES - 1) * STAGE_BYTES;
    for (int s = 0; s < KT; ++s) {
      // stage s has landed: only the STAGES - 2 stages behind it may be in flight
      if (s + STAGES - 1 <= KT) HMI_WAIT_VMCNT(LD * (STAGES - 2)); else HMI_WAIT_VMCNT(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      if (s + STAGES - 1 < KT) {            // into the slot of stage s - 1, which nobody reads any more
        copy_stage(fill);
        fill = fill == (STAGES - 1) * STAGE_BYTES ? 0 : fill + STAGE_BYTES;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (half_stage) {                       // chunks 0-3 of the rows, and again instead of chunks 4-7 past the row's end
#pragma unroll
      for (int j = 0; j < A_LD; ++j) a_off[j] -= (((lane & 7) ^ swz_a((pw * A_LD + j) * 8 + (lane >> 3))) & 4) << 4;
#pragma unroll
      for (int j = 0; j < W_LD; ++j) w_off[j] -= (((lane & 7) ^ swz_w((pw * W_LD + j) * 8 + (lane >> 3))) & 4) << 4;
      __builtin_amdgcn_s_barrier();         // everybody has read the last whole stage
      copy_stage(0);
      HMI_WAIT_VMCNT(0);
      __builtin_amdgcn_s_barrier();
    }
    return;
  }

  // ================= consumers: products and results =================
  const int l32 = lane & 31, lh = lane >> 5;
  const int wm = wave / WN, wn = wave % WN;
  const int rx = wm * WTM + l32, rw = wn * WTN + perm_w(l32);
  const int fx_base = rx * ROW_BYTES + ((lh ^ swz_a(rx)) << 4);       // fragment offsets inside a stage (k-step ks: XOR ks << 5)
  const int fw_base = BM * ROW_BYTES + rw * ROW_BYTES + ((lh ^ swz_w(rw)) << 4);
  f32x16 acc[TM][TN];                       // start at the bias
  f32x16 acc2[TM][TN];                      // fp32: every other product's sum, from zero
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = min(n0 + wn * WTN + j * 32 + 16 * lh, g.n_out - 16);   // a lane's 16 columns exist or do not as a whole
    const char* bp = g.pool + slot_base + g.b_off + (size_t)col * ES;
    if (BF16) {
      const u32x4 b0 = reinterpret_cast<const u32x4*>(bp)[0], b1 = reinterpret_cast<const u32x4*>(bp)[1];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        acc[0][j][2 * q] = bf2f(b0[q] & 0xFFFFu);     acc[0][j][2 * q + 1] = bf2f(b0[q] >> 16);
        acc[0][j][8 + 2 * q] = bf2f(b1[q] & 0xFFFFu); acc[0][j][8 + 2 * q + 1] = bf2f(b1[q] >> 16);
      }
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 b = reinterpret_cast<const f32x4*>(bp)[q];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0][j][4 * q + e] = b[e];
      }
    }
#pragma unroll
    for (int i = 1; i < TM; ++i) acc[i][j] = acc[0][j];
#pragma unroll
    for (int i = 0; i < TM; ++i) acc2[i][j] = f32x16{};
  }
  int out_row[TM];                          // where this lane's rows of the tile go in C
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = row0 + min(wm * WTM + i * 32 + l32, rows - 1);
    out_row[i] = ident ? r : rt.row_src[r];
  }
  const bool wave_active = wm * WTM < rows && n0 + wn * WTN < g.n_out;

  u32x4 fx[4][TM], fw[4][TN];               // one fragment buffer per k-step of a stage
  int rd = 0;                               // byte offset of the slot that is read
#define HMI_READ_FRAGS(KS)                                                                         \
  {                                                                                                \
    const unsigned char* sb_ = smem + rd;                                                          \
    _Pragma("unroll") for (int i = 0; i < TM; ++i) fx[KS][i] = *reinterpret_cast<const u32x4*>(sb_ + (fx_base ^ ((KS) << 5)) + i * 32 * ROW_BYTES); \
    _Pragma("unroll") for (int j = 0; j < TN; ++j) fw[KS][j] = *reinterpret_cast<const u32x4*>(sb_ + (fw_base ^ ((KS) << 5)) + j * 32 * ROW_BYTES); \
  }
#define HMI_MULTIPLY(KS)                                                                           \
  {                                                                                                \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                 \
      _Pragma("unroll") for (int j = 0; j < TN; ++j) mfma_chunk<BF16>(fw[KS][j], fx[KS][i], acc[i][j], acc2[i][j]); \
    __builtin_amdgcn_sched_barrier(0);                                                             \
  }
  // Fragments are read two to three k-steps ahead of their products.  The barrier of a stage stands in the middle of the
  // products of the stage before it: this wavefront has read all of that one, and the new stage's first fragments are on
  // their way under the other half.
  if (KT > 0) {
    __builtin_amdgcn_s_barrier();           // stage 0 is there
    __builtin_amdgcn_sched_barrier(0);
  }
  HMI_READ_FRAGS(0) HMI_READ_FRAGS(1) HMI_READ_FRAGS(2)
  for (int s = 0; s < KT; ++s) {
    HMI_READ_FRAGS(3)
    HMI_MULTIPLY(0)
    HMI_MULTIPLY(1)
    HMI_WAIT_LGKMCNT0();
    if (s + 1 < KT) __builtin_amdgcn_s_barrier();     // stage s + 1 is there
    __builtin_amdgcn_sched_barrier(0);
    rd = rd == (STAGES - 1) * STAGE_BYTES ? 0 : rd + STAGE_BYTES;
    HMI_READ_FRAGS(0) HMI_READ_FRAGS(1)               // (behind the last stage: read, but not multiplied)
    HMI_MULTIPLY(2)
    HMI_READ_FRAGS(2)
    HMI_MULTIPLY(3)
  }
  if (half_stage) {
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    rd = 0;
    HMI_READ_FRAGS(0) HMI_READ_FRAGS(1)
    HMI_MULTIPLY(0) HMI_MULTIPLY(1)
  }
#undef HMI_READ_FRAGS
#undef HMI_MULTIPLY
  if (!wave_active) return;

  // ---- epilogue: lane (row l32, half lh) of MFMA tile (i, j) holds columns 16 lh .. 16 lh + 15 of its 32
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = wm * WTM + i * 32 + l32;
    if (r >= rows) continue;
    const size_t orow = (size_t)out_row[i];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + wn * WTN + j * 32 + 16 * lh;
      if (col >= g.n_out) continue;
      f32x16 v = acc[i][j];
      if (!BF16) v += acc2[i][j];
      if (g.epi == EPI_BIAS_GELU) {
        if (BF16 && g.gelu_poly) {
#pragma unroll
          for (int e = 0; e < 16; ++e) v[e] = gelu_poly(v[e]);
        } else {
#pragma unroll
          for (int e = 0; e < 16; ++e) v[e] = BF16 ? gelu_f32(v[e]) : gelu_erf(v[e]);
        }
      } else if (g.epi == EPI_BIAS_RELU) {
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = fmaxf(v[e], 0.0f);
      } else if (g.epi == EPI_BIAS_RESID) {
        if (!BF16 || g.resid_f32) {
          const f32x4* rp = reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g.resid) + orow * g.ldr + col);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 rv = rp[q];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * q + e] += rv[e];
          }
        } else {
          const u32x4* rp = reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(g.resid) + orow * g.ldr + col);
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const u32x4 rv = rp[q];
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[8 * q + 2 * e] += bf2f(rv[e] & 0xFFFFu); v[8 * q + 2 * e + 1] += bf2f(rv[e] >> 16); }
          }
        }
      }
      const size_t off = orow * g.ldc + col;
      if (!BF16 || g.out_f32) {
        f32x4_any* cp = reinterpret_cast<f32x4_any*>(reinterpret_cast<float*>(g.C) + off);
#pragma unroll
        for (int q = 0; q < 4; ++q) cp[q] = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
      }
      if (!BF16) {
        if (g.C2) {
          f32x4* cp = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C2) + off);
#pragma unroll
          for (int q = 0; q < 4; ++q) cp[q] = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        }
      } else if (!g.out_f32 || g.C2) {
        u32x4 h[2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) h[q][e] = pack_bf16(v[8 * q + 2 * e], v[8 * q + 2 * e + 1]);
        if (!g.out_f32) { u32x4* cp = reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(g.C) + off); cp[0] = h[0]; cp[1] = h[1]; }
        if (g.C2) { u32x4* cp = reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(g.C2) + off); cp[0] = h[0]; cp[1] = h[1]; }
      }
    }
  }
}

// Large bf16 launches share the persistent kernel's GELU (2e-4 from the exact one, half the clocks: a 128 x 128 tile's
// epilogue with it takes 1.3 us, with the exact one 2.5); small ones, where it costs nothing, and odd shapes are exact.
bool gelu_poly_fits(const GemmArgs& g) { return g.n_rows > 1024 && g.n_out % 256 == 0 && g.k >= 192; }

template <bool BF16, int BM, int BN, int WM, int WN, int STAGES>
struct Tile {
  static constexpr int NP = 4;              // producers
  static constexpr int LDS = STAGES * (BM + BN) * ROW_BYTES;
  static void allow_lds() {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_tile_kernel<BF16, BM, BN, WM, WN, STAGES, NP>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
  }
  static int per_entry(const Route& rt, int list) { return rt.tile_m[list] / BM; }
  // tiles of a launch; on a tenant route an entry of the list counts with all tiles it has room for
  static long long tiles(const GemmArgs& g, const Route& rt, int list) {
    const long long mt = rt.identity ? (g.n_rows + BM - 1) / BM : (long long)g.n_mtiles_list[list] * per_entry(rt, list);
    return mt * ((g.n_out + BN - 1) / BN);
  }
  static void launch(GemmArgs g, const Route& rt, int list, hipStream_t s) {
    g.which_tiles = list;
    g.gelu_poly = gelu_poly_fits(g);
    const long long total = tiles(g, rt, list);
    if (total <= 0) return;
    const int per = (int)((total + kXcds - 1) / kXcds);
    hipLaunchKernelGGL((gemm_tile_kernel<BF16, BM, BN, WM, WN, STAGES, NP>), dim3(per * kXcds), dim3(64 * (NW + NP)), LDS, s,
                       g, rt, (int)total, per_entry(rt, list));
  }
};
typedef Tile<true, 64, 64, 2, 2, 5> TileS;        // 80 KB of LDS: two workgroups per compute unit
typedef Tile<true, 128, 64, 2, 2, 3> TileM;       // 72 KB: two
typedef Tile<true, 128, 128, 2, 2, 3> TileL;      // 96 KB: one
typedef Tile<true, 128, 256, 2, 2, 3> TileXL;     // 144 KB: one
typedef Tile<false, 64, 64, 2, 2, 5> TileF32;
}  // namespace

void init_gemm_tile_kernels() {
  TileS::allow_lds(); TileM::allow_lds(); TileL::allow_lds(); TileXL::allow_lds(); TileF32::allow_lds();
}

// Which kernel a launch gets.
//
// Few rows per weight matrix (a decode step over many tenants: at most 32 rows per 128-row m-tile on average): the weights
// are read once and nothing else matters, gemm_bf16_skinny.hip streams them.  A launch whose 32 x 32 items do not fill the
// compute units and whose k is long goes there too: it shares k among the four wavefronts of an item (100 rows x 768
// columns x k = 3072: 7.2 us, 64 x 64 tiles 11.4; 300 rows, 288 items: 13.6 and 12.1; k = 768: 5.0 and 5.0).
//
// Everything else is tiles, and the size of the tile is a matter of how many compute units the launch would leave idle: a
// larger tile moves fewer bytes per product, a smaller one comes in more pieces.  The estimate is the time of the busiest
// compute unit: its tiles times (stages of 64 k times the time of one stage, plus what a tile costs besides, which the
// second workgroup of a compute unit hides for the small tiles; the activation adds to that).  Microseconds, measured with
// d = 768, f = 3072 over 100 to 16 384 rows of one weight set; the estimate's choice was the fastest or within 10 % of it.
// It says nothing about weights that come from HBM or panels that are fetched again, so a launch that gives the
// persistent kernel's workgroups more than one and a half tiles each is not weighed at all: it was the faster one for all
// of those (two encoder layers of 177 tenants, 65 536 rows: 3.1 ms, with 128 x 256 tiles where the estimate is lower 3.4).
GemmKernel pick_gemm_bf16(const GemmArgs& g, const Route& rt) {
  const int n_cu = rt.n_cu >= kXcds ? rt.n_cu : 256;
  if (g.n_out % 32 == 0) {
    const bool few_rows = g.n_rows <= 32LL * g.n_mtiles_list[1];
    const long long items = (few_rows ? g.n_mtiles_list[1] : (g.n_rows + 31) / 32) * (long long)(g.n_out / 32);
    if ((few_rows && !rt.identity) || (items <= std::min(n_cu, kSplitMaxItems) && g.k >= 1536 && g.k % 256 == 0)) return GEMM_STREAM;
  }
  const long long big_tiles = g.n_out % 256 == 0 && g.k >= 192 ? (long long)g.n_mtiles_list[0] * (g.n_out / 256) : 0;
  if (2 * big_tiles > 3LL * n_cu) return GEMM_PERSISTENT;
  const double stages = g.k / 64, act = g.epi == EPI_BIAS_GELU ? 1.0 : 0.0;
  auto estimate = [&](long long tiles, double stage, double tile, double gelu) {
    return (double)((tiles + n_cu - 1) / n_cu) * (stages * stage + tile + act * gelu);
  };
  double best = estimate(TileS::tiles(g, rt, 1), 0.20, 0.2, 0.4);
  GemmKernel which = GEMM_64x64;
  auto consider = [&](GemmKernel id, double t) { if (t < best) { best = t; which = id; } };
  consider(GEMM_128x64, estimate(TileM::tiles(g, rt, 1), 0.32, 0.3, 0.4));
  if (g.n_out % 128 == 0) consider(GEMM_128x128, estimate(TileL::tiles(g, rt, 1), 0.50, 2.3, 1.3));
  if (g.n_out % 256 == 0) {
    consider(GEMM_128x256, estimate(TileXL::tiles(g, rt, 1), 0.90, 3.2, 2.6));
    if (g.k >= 192) consider(GEMM_PERSISTENT, estimate(big_tiles, 1.45, 4.0, 3.0));
  }
  return which;
}

void launch_gemm_bf16(const GemmArgs& g, const Route& rt, hipStream_t s) {
  if (g.n_rows <= 0 || g.n_mtiles_list[1] <= 0) return;
  GemmArgs a = g;
  switch (pick_gemm_bf16(g, rt)) {
    case GEMM_STREAM:
      a.which_tiles = 1;
      a.n_mtiles = g.n_mtiles_list[1];
      return launch_gemm_bf16_skinny(a, rt, s);
    case GEMM_64x64: return TileS::launch(g, rt, 1, s);
    case GEMM_128x64: return TileM::launch(g, rt, 1, s);
    case GEMM_128x128: return TileL::launch(g, rt, 1, s);
    case GEMM_128x256: return TileXL::launch(g, rt, 1, s);
    case GEMM_PERSISTENT:
      a.which_tiles = 0;
      a.n_mtiles = g.n_mtiles_list[0];
      return launch_gemm_bf16_p256(a, rt, s);
  }
}

void launch_gemm_f32(const GemmArgs& g, const Route& rt, hipStream_t s) {
  if (g.n_rows <= 0) return;
  TileF32::launch(g, rt, 0, s);
}

}  // namespace hmi

// The rule alone, for the tests: which kernel (GemmKernel) a bf16 launch of these sizes gets.  tiles256, tiles128: m-tiles of
// 256 and 128 rows, summed over the batch's tenants (or of all rows, where the weights are shared).
extern "C" int32_t hmi_internal_gemm_kernel(int32_t n_rows, int32_t tiles256, int32_t tiles128, int32_t n_out, int32_t k,
                                            int32_t gelu, int32_t shared, int32_t n_cu) {
  hmi::GemmArgs g{};
  g.n_rows = n_rows; g.n_out = n_out; g.k = k; g.epi = gelu ? hmi::EPI_BIAS_GELU : hmi::EPI_BIAS;
  g.n_mtiles_list[0] = tiles256; g.n_mtiles_list[1] = tiles128;
  hmi::Route rt{};
  rt.tile_m[0] = hmi::kBf16TileM0; rt.tile_m[1] = hmi::kBf16TileM1;
  rt.identity = shared; rt.n_cu = n_cu;
  return hmi::pick_gemm_bf16(g, rt);
}
