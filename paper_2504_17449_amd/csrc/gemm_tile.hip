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
//     4 copies in one instruction stream take 357 clocks for 249 of either).  So a workgroup is one to four consumers,
//     WM x WN over the BM x BN tile (fp32: times KH sets that share k), which read LDS and multiply, and four
//     producers, which do nothing but copy: one launch of 768 x 3072 weights over 100 rows 28.8 -> 23.7 us with 128 x 128
//     tiles, 15.9 -> 11.4 with 64 x 64.
//   * Operands come in stages of 128 bytes of k per row (64 bf16 or 32 fp32: one cache line, eight lanes fetch a row's
//     line) by direct-to-LDS copies into a ring of STAGES, one barrier per stage.
//   * A 16-byte chunk of a row is one fragment read: one v_mfma_f32_32x32x16_bf16, or four v_mfma_f32_32x32x2_f32
//     (element e of the two lane halves' chunks is one k-step of two; the k order inside a stage is the same for both
//     operands, so it does not matter that it is not ascending).  fp32 products go to two accumulators in turn: a sum of half
//     as many, whose rounding errors are 0.7 of one chain's (in one chain fp32 layers were 1.3 % further from 64 bits than
//     with the vector ALU's fused chain; two encoder layers of 1 728 rows 672.5 us with one, 673.1 with two); where wavefronts
//     share k there are two such sums for each of them (24 drawn fp32 cases: 0.85 of the error of two).
//   * Weights are the MFMA's first operand, in a permuted row order, so that a lane ends up with 16 consecutive columns
//     of one row of C: bf16 results without a residual leave straight from the accumulators in 16-byte pieces, fp32 results
//     and sums with residuals through a patch of LDS (below).  Accumulators start at the bias.
//   * What the launch fetches is what the XCDs' L2s fetch, each for itself: m-tile by m-tile a launch of a few of them reads
//     the weights once for each.  So the tiles of shared weights are shared out among the XCDs in blocks of rows and columns
//     (xcd_rows below); with a tenant's own weights an XCD has a contiguous range of tiles, m-tile by m-tile.
//   * A stage costs a consumer one trip to LDS, one barrier and its products, and only the last grows with it: the small tiles
//     take two lines of k a stage where k allows (64 x 64, 64 k a stage: 490 clocks, of which 160 are products).
// Measured, us (d = 768, f = 3072, one weight set; with the persistent tiles, with one line of k a stage, now):
//   2 664 rows  QKV 22.1, 15.6 - 17.2, 17.2;  output projection 20.6, 8.2, 7.7;  FFN1 25.6, 21.5, 21.2;  FFN2 71.7, 22.8, 19.9
//   756 rows    output projection and FFN2 together -, 19.7, 18.7
//   141 rows    QKV -, 6.0, 5.0;  output projection -, 5.6, 4.2
//   (7 rows, now gemm_bf16_thin.hip's: QKV -, 5.5, 4.4;  output projection -, 5.4, 4.3;  FFN1 -, 6.6, 5.2)
// fp32: 1 728 rows of eight tenants, two encoder layers with their attention: products on the vector ALU 1.28 ms, 64 x 64 tiles
// 0.67, now 0.62;  128 rows of four tenants, an FFN block of d = 64 25.3 us, now 21.3.
#include "hmi_kernels.h"

#include "gelu.h"
#include "wave.h"

#include <algorithm>
#include <type_traits>

namespace hmi {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));   // in the caller's result, which may begin at any float
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* glb_ptr_t;

constexpr int kXcds = 8;
constexpr int ROW_BYTES = 128;            // k bytes of a row and line

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

// 16 bytes of residual (four columns, fp32 or bf16) as they are loaded, and added.
union Resid { f32x4 f; u32x2 h; };

// BM x BN: the tile; WM x WN consumers, KH sets of them that share k; a stage is U lines of k; STAGES of them in the ring; NP producers.  The epilogue is a
// parameter too: small launches feel its instructions (as a run-time choice the compiler evaluated GELU for all of them, 0.8 us).
template <bool BF16, int BM, int BN, int WM, int WN, int KH, int U, int STAGES, int NP, int EPI>
__global__ __launch_bounds__(64 * (WM * WN * KH + NP)) void gemm_tile_kernel(GemmArgs g, Route rt, int total, int tiles_per_entry, int xcd_rows) {
  constexpr int NW = WM * WN * KH;
  constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  constexpr int A_LD = BM / 8 / NP, W_LD = BN / 8 / NP;      // 1 KB copies (8 rows) per producer and line of k
  constexpr int LINE_BYTES = (BM + BN) * ROW_BYTES, STAGE_BYTES = U * LINE_BYTES;
  constexpr int ES = BF16 ? 2 : 4;
  constexpr int KS = 4 * U / KH;                             // k-steps of a stage for one consumer
  static_assert(U * (A_LD + W_LD) * (STAGES - 1) < 64, "vmcnt range");
  static_assert(U % KH == 0, "a consumer has whole lines");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  // ---- which tile.  Workgroups go to the XCDs round robin.
  const int nt_n = (g.n_out + BN - 1) / BN;
  const int xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds;
  int row0, row_end, n0;
  size_t slot_base = 0;
  const bool ident = rt.identity != 0;      // the shared parameters' route: tiles in row order, identity row map, slot 0
  if (xcd_rows > 0) {
    // the XCDs share out the tiles as xcd_rows x (8 / xcd_rows) blocks of whole tiles; inside one, panel of weights by panel
    const int nt_m = total / nt_n, xm = xcd & (xcd_rows - 1), xn = xcd / xcd_rows, xcd_cols = kXcds / xcd_rows;
    const int m_lo = nt_m * xm / xcd_rows, m_cnt = nt_m * (xm + 1) / xcd_rows - m_lo;
    const int n_lo = nt_n * xn / xcd_cols, n_cnt = nt_n * (xn + 1) / xcd_cols - n_lo;
    if (local >= m_cnt * n_cnt) return;
    const int in = local / m_cnt;
    row0 = (m_lo + local - in * m_cnt) * BM;
    n0 = (n_lo + in) * BN;
    row_end = g.n_rows;
  } else {
    // m-tile by m-tile, a contiguous range for each XCD; an entry of the route's list holds tiles_per_entry tiles of BM rows
    const int per = (total + kXcds - 1) / kXcds;
    const int w = xcd * per + local;
    if (local >= per || w >= total) return;
    const int mt = w / nt_n;
    n0 = (w - mt * nt_n) * BN;
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
  }
  const int rows = min(BM, row_end - row0);
  if (rows <= 0) return;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kbytes = g.k * ES;
  const int KT = kbytes / (U * ROW_BYTES);  // whole stages; fp32 shapes may leave half a stage (64 bytes) behind
  const bool half_stage = !BF16 && U == 1 && kbytes % ROW_BYTES != 0;

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
    const char* a_next = reinterpret_cast<const char*>(g.A);   // the line of k that is copied next (uniform)
    const char* w_next = g.pool + slot_base + g.w_off;
    // ROWS: this producer's activation rows exist (of a tile of a few rows the others are not copied: nobody looks at what
    // the products make of them)
    auto produce = [&](auto with_rows) {
      constexpr bool ROWS = decltype(with_rows)::value;
      constexpr int LD = U * (W_LD + (ROWS ? A_LD : 0));
      auto copy_stage = [&](int slot_off) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          unsigned char* dst = smem + slot_off + u * LINE_BYTES;
          if (ROWS) {
#pragma unroll
            for (int j = 0; j < A_LD; ++j)
              __builtin_amdgcn_global_load_lds((glb_ptr_t)(a_next + a_off[j]), (lds_ptr_t)(dst + (pw * A_LD + j) * 1024), 16, 0, 0);
          }
#pragma unroll
          for (int j = 0; j < W_LD; ++j)
            __builtin_amdgcn_global_load_lds((glb_ptr_t)(w_next + w_off[j]), (lds_ptr_t)(dst + BM * ROW_BYTES + (pw * W_LD + j) * 1024), 16, 0, 0);
          a_next += ROW_BYTES; w_next += ROW_BYTES;
        }
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
    };
    if (BM == 32 && pw * A_LD * 8 >= rows) produce(std::false_type{}); else produce(std::true_type{});
    if (KH > 1) __builtin_amdgcn_s_barrier();   // (the consumers' sums)
    return;
  }

  // ================= consumers: products and results =================
  const int l32 = lane & 31, lh = lane >> 5;
  const int kh = wave / (WM * WN), wm = wave / WN % WM, wn = wave % WN;
  const int rx = wm * WTM + l32, rw = wn * WTN + perm_w(l32);
  const int fx_base = rx * ROW_BYTES + ((lh ^ swz_a(rx)) << 4);       // fragment offsets inside a line of k (k-step ks: XOR ks << 5)
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
    for (int i = 0; i < TM; ++i) {
      acc2[i][j] = f32x16{};
      if (kh > 0) acc[i][j] = f32x16{};
    }
  }
  int out_row[TM];                          // where this lane's rows of the tile go in C
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = row0 + min(wm * WTM + i * 32 + l32, rows - 1);
    out_row[i] = ident ? r : rt.row_src[r];
  }
  const bool wave_active = wm * WTM < rows && n0 + wn * WTN < g.n_out;

  // fp32 results, and residuals, cross a patch of LDS so that the lanes of a row read and write it in whole lines: 32 CF columns of
  // a row, four to a lane (straight from the accumulators an instruction touches 64 lines: 3.2 us of a 128 x 64 tile's epilogue,
  // now 2.2).  bf16 results leave from the accumulators: there is half as much of them, and the way through LDS was the longer one
  // (128 x 256 tiles with GELU 5.5 us for 6.8, 32 x 32 tiles 0.4 for 1.2).
  constexpr int CF = TN < 2 ? TN : 2;
  constexpr int FL = 8 * CF;                                 // lanes of a row
  static_assert(STAGE_BYTES >= WM * WN * 32 * CF * 128, "patches fit a stage");
  const bool staged = !BF16 || g.out_f32 || EPI == EPI_BIAS_RESID;
  const bool resid_f32 = !BF16 || g.resid_f32;
  // the residuals of the small tiles are asked for now, the large ones' when their turn comes
  constexpr bool AHEAD = TM * TN <= 2 && BF16;
  Resid ahead[AHEAD ? TM * TN * 4 : 1];
  auto load_resid = [&](int i, int j, int it) {              // piece `it` of the pass that begins at column block j
    const int r = it * (64 / FL) + lane / FL, m = wm * WTM + i * 32 + r;
    const int col = n0 + wn * WTN + j * 32 + (lane % FL) * 4;
    Resid v = {};
    const size_t at = (size_t)__shfl(out_row[i], r, 64) * g.ldr + col;
    if (m < rows && col < g.n_out) {
      if (resid_f32) v.f = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(g.resid) + at);
      else v.h = *reinterpret_cast<const u32x2*>(reinterpret_cast<const uint16_t*>(g.resid) + at);
    }
    return v;
  };
  if (AHEAD && EPI == EPI_BIAS_RESID && wave_active) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; j += CF)
#pragma unroll
        for (int it = 0; it < 4 * CF; ++it) ahead[(i * TN + j) * 4 + it] = load_resid(i, j, it);
  }

  u32x4 fx[KS][TM], fw[KS][TN];             // one fragment buffer per k-step of a stage
  int rd = 0;                               // byte offset of the slot that is read
#define HMI_READ_FRAGS(S)                                                                          \
  {                                                                                                \
    const unsigned char* sb_ = smem + rd + (kh * (U / KH) + (S) / 4) * LINE_BYTES;                 \
    _Pragma("unroll") for (int i = 0; i < TM; ++i) fx[S][i] = *reinterpret_cast<const u32x4*>(sb_ + (fx_base ^ (((S) & 3) << 5)) + i * 32 * ROW_BYTES); \
    _Pragma("unroll") for (int j = 0; j < TN; ++j) fw[S][j] = *reinterpret_cast<const u32x4*>(sb_ + (fw_base ^ (((S) & 3) << 5)) + j * 32 * ROW_BYTES); \
  }
#define HMI_MULTIPLY(S)                                                                            \
  {                                                                                                \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                 \
      _Pragma("unroll") for (int j = 0; j < TN; ++j) mfma_chunk<BF16>(fw[S][j], fx[S][i], acc[i][j], acc2[i][j]); \
    __builtin_amdgcn_sched_barrier(0);                                                             \
  }
  // Fragments are read two to three k-steps ahead of their products.  The barrier of a stage stands two k-steps before the end
  // of the products of the stage before it: this wavefront has read all of that one, and the new stage's first fragments are on
  // their way under the rest.
  if (KT > 0) {
    __builtin_amdgcn_s_barrier();           // stage 0 is there
    __builtin_amdgcn_sched_barrier(0);
  }
  HMI_READ_FRAGS(0) HMI_READ_FRAGS(1) HMI_READ_FRAGS(2)
  for (int s = 0; s < KT; ++s) {
#pragma unroll
    for (int ks = 0; ks < KS - 2; ++ks) {
      if (ks + 3 < KS) HMI_READ_FRAGS(ks + 3)
      HMI_MULTIPLY(ks)
    }
    HMI_WAIT_LGKMCNT0();
    if (s + 1 < KT) __builtin_amdgcn_s_barrier();     // stage s + 1 is there
    __builtin_amdgcn_sched_barrier(0);
    rd = rd == (STAGES - 1) * STAGE_BYTES ? 0 : rd + STAGE_BYTES;
    HMI_READ_FRAGS(0) HMI_READ_FRAGS(1)               // (behind the last stage: read, but not multiplied)
    HMI_MULTIPLY(KS - 2)
    HMI_READ_FRAGS(2)
    HMI_MULTIPLY(KS - 1)
  }
  // the slot behind the last stage's, which no wavefront reads any more but for the idle reads above
  unsigned char* const patch = smem + (half_stage ? STAGE_BYTES : rd) + wave * (32 * CF * 128);
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
  if (KH > 1) {
    // the other sets' sums, through the slots behind the patches, added in the order of k
    f32x4* const part = reinterpret_cast<f32x4*>(smem + rd + WM * WN * 32 * CF * 128) + (wave - WM * WN) * (TM * TN * 4) * 64 + lane;
    static_assert(KH == 1 || STAGE_BYTES >= WM * WN * 32 * CF * 128 + (KH - 1) * WM * WN * TM * TN * 4096, "sums fit a stage");
    if (kh > 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            f32x16 v = acc[i][j];
            if (!BF16) v += acc2[i][j];
            part[((i * TN + j) * 4 + q) * 64] = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
          }
    }
    HMI_WAIT_LGKMCNT0();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kh > 0) return;
#pragma unroll
    for (int o = 1; o < KH; ++o)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4 v = part[(o * WM * WN * TM * TN * 4 + (i * TN + j) * 4 + q) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] += v[e];
          }
  }
  if (!wave_active) return;

  // ---- epilogue: lane (row l32, half lh) of MFMA tile (i, j) holds columns 16 lh .. 16 lh + 15 of its 32
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if (wm * WTM + i * 32 >= rows) break;
    auto value = [&](int j) {
      f32x16 v = acc[i][j];
      if (!BF16) v += acc2[i][j];
      if (EPI == EPI_BIAS_GELU) {
        if (BF16 && g.gelu_poly) {
#pragma unroll
          for (int e = 0; e < 16; ++e) v[e] = gelu_poly(v[e]);
        } else {
#pragma unroll
          for (int e = 0; e < 16; ++e) v[e] = BF16 ? gelu_f32(v[e]) : gelu_erf(v[e]);
        }
      } else if (EPI == EPI_BIAS_RELU) {
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = fmaxf(v[e], 0.0f);
      }
      return v;
    };
    if (staged) {
#pragma unroll
      for (int j = 0; j < TN; j += CF) {
        Resid later[AHEAD ? 1 : 4 * CF];
        if (!AHEAD && EPI == EPI_BIAS_RESID) {
#pragma unroll
          for (int it = 0; it < 4 * CF; ++it) later[it] = load_resid(i, j, it);
        }
#pragma unroll
        for (int jj = 0; jj < CF; ++jj) {
          const f32x16 v = value(j + jj);
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4*>(patch + l32 * (FL * 16) + (((jj * 8 + lh * 4 + q) ^ (l32 & (FL - 1))) << 4)) =
                f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        }
#pragma unroll
        for (int it = 0; it < 4 * CF; ++it) {
          const int r = it * (64 / FL) + lane / FL, m = wm * WTM + i * 32 + r;
          const int col = n0 + wn * WTN + j * 32 + (lane % FL) * 4;
          f32x4 v = *reinterpret_cast<const f32x4*>(patch + r * (FL * 16) + (((lane % FL) ^ (r & (FL - 1))) << 4));
          const size_t off = (size_t)__shfl(out_row[i], r, 64) * g.ldc + col;
          if (EPI == EPI_BIAS_RESID) {
            const Resid rv = AHEAD ? ahead[(i * TN + j) * 4 + it] : later[AHEAD ? 0 : it];
            if (resid_f32) v += rv.f;
            else v += f32x4{bf2f(rv.h[0] & 0xFFFFu), bf2f(rv.h[0] >> 16), bf2f(rv.h[1] & 0xFFFFu), bf2f(rv.h[1] >> 16)};
          }
          if (m >= rows || col >= g.n_out) continue;
          if (!BF16 || g.out_f32) *reinterpret_cast<f32x4_any*>(reinterpret_cast<float*>(g.C) + off) = v;
          if (!BF16) {
            if (g.C2) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C2) + off) = v;
          } else {
            const u32x2 h = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            if (!g.out_f32) *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(g.C) + off) = h;
            if (g.C2) *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(g.C2) + off) = h;
          }
        }
      }
    } else if (wm * WTM + i * 32 + l32 < rows) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = n0 + wn * WTN + j * 32 + 16 * lh;
        if (col >= g.n_out) continue;
        const f32x16 v = value(j);
        u32x4 h[2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) h[q][e] = pack_bf16(v[8 * q + 2 * e], v[8 * q + 2 * e + 1]);
        const size_t off = (size_t)out_row[i] * g.ldc + col;
        u32x4* cp = reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(g.C) + off);
        cp[0] = h[0]; cp[1] = h[1];
        if (g.C2) { u32x4* cp2 = reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(g.C2) + off); cp2[0] = h[0]; cp2[1] = h[1]; }
      }
    }
  }
}

// Large bf16 launches share the persistent kernel's GELU (2e-4 from the exact one, half the clocks: a 128 x 128 tile's
// epilogue with it takes 1.3 us, with the exact one 2.5); small ones, where it costs nothing, and odd shapes are exact.
bool gelu_poly_fits(const GemmArgs& g) { return g.n_rows > 1024 && g.n_out % 256 == 0 && g.k >= 192; }

template <bool BF16, int BM, int BN, int WM, int WN, int U, int STAGES, int KH = 1, int NP = 4>
struct Tile {
  static constexpr int LDS = STAGES * U * (BM + BN) * ROW_BYTES;
  static_assert(LDS <= 163840, "LDS");
  template <int EPI>
  static constexpr auto kernel() { return &gemm_tile_kernel<BF16, BM, BN, WM, WN, KH, U, STAGES, NP, EPI>; }
  static void allow_lds() {
    for (auto k : {kernel<EPI_BIAS>(), kernel<EPI_BIAS_GELU>(), kernel<EPI_BIAS_RELU>(), kernel<EPI_BIAS_RESID>()})
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
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
    long long per = (total + kXcds - 1) / kXcds;
    int xcd_rows = 0;
    if (rt.identity) {
      // the split that fetches least: each XCD reads its blocks' rows of A and of W.  Only where an XCD runs all of its tiles at
      // once: an uneven split costs a launch of several rounds more than it saves (2 664 rows, 756 tiles of QKV: 17.2 us -> 19.4).
      const long long nt_n = (g.n_out + BN - 1) / BN, nt_m = total / nt_n;
      const long long room = (long long)(rt.n_cu >= kXcds ? rt.n_cu : 256) / kXcds * (163840 / LDS);
      long long best = 0;
      for (int xr = 1; xr <= kXcds; xr *= 2) {
        const long long xc = kXcds / xr, mine = ((nt_m + xr - 1) / xr) * ((nt_n + xc - 1) / xc);
        const long long rows = g.n_rows * xc + (long long)g.n_out * xr;
        if (mine <= room && (xcd_rows == 0 || rows < best)) { best = rows; per = mine; xcd_rows = xr; }
      }
    }
    const auto k = g.epi == EPI_BIAS ? kernel<EPI_BIAS>() : g.epi == EPI_BIAS_GELU ? kernel<EPI_BIAS_GELU>() :
                   g.epi == EPI_BIAS_RELU ? kernel<EPI_BIAS_RELU>() : kernel<EPI_BIAS_RESID>();
    hipLaunchKernelGGL(k, dim3((unsigned)(per * kXcds)), dim3(64 * (WM * WN * KH + NP)), LDS, s, g, rt, (int)total, per_entry(rt, list), xcd_rows);
  }
};
typedef Tile<true, 64, 64, 2, 2, 1, 5> TileS;        // 80 KB of LDS: two workgroups per compute unit
typedef Tile<true, 64, 64, 2, 2, 2, 3> TileS2;       // 96 KB: one
typedef Tile<true, 32, 64, 1, 2, 2, 4> TileT2;       // 96 KB: one
typedef Tile<true, 32, 32, 1, 1, 2, 6> TileU2;       // 96 KB: one
typedef Tile<true, 128, 64, 2, 2, 1, 3> TileM;       // 72 KB: two
typedef Tile<true, 128, 64, 2, 2, 2, 3> TileM2;      // 144 KB: one
typedef Tile<true, 128, 128, 2, 2, 1, 3> TileL;      // 96 KB: one
typedef Tile<true, 128, 256, 2, 2, 1, 3> TileXL;     // 144 KB: one
typedef Tile<false, 64, 64, 2, 2, 1, 5> TileF32;     // 80 KB: two
typedef Tile<false, 64, 32, 2, 1, 2, 3, 2> TileF32H;    // 72 KB: two
typedef Tile<false, 32, 32, 1, 1, 4, 3, 4> TileF32Q;    // 96 KB: one

enum TileForm : int { TILE_ONE_LINE = 0, TILE_32x32_TWO, TILE_32x64_TWO, TILE_64x64_TWO, TILE_128x64_TWO };
enum TileFormF32 : int { TILE_F32_32x32 = 0, TILE_F32_64x32, TILE_F32_64x64 };
}  // namespace

void init_gemm_tile_kernels() {
  TileS::allow_lds(); TileS2::allow_lds(); TileT2::allow_lds(); TileU2::allow_lds(); TileM::allow_lds(); TileM2::allow_lds(); TileL::allow_lds(); TileXL::allow_lds(); TileF32::allow_lds(); TileF32H::allow_lds(); TileF32Q::allow_lds();
}

// Which kernel a launch gets, if it is not one of a few rows through shared weights (gemm_bf16_thin.hip, asked for first).
//
// Few rows per weight matrix (a decode step over many tenants: at most 32 rows per 128-row m-tile on average): the weights
// are read once and nothing else matters, gemm_bf16_skinny.hip streams them.  A launch whose 32 x 32 items do not fill the
// compute units and whose k is long goes there too: it shares k among the four wavefronts of an item (768 columns x k = 3072,
// us, split and the best tiles, 32 x 32 with two lines of k a stage: 7 rows 6.2, 7.3; 100 rows 8.2, 7.7; 300 rows 8.7, 8.5).
//
// Everything else is tiles, and the size of the tile is a matter of how many compute units the launch would leave idle: a
// larger tile moves fewer bytes per product, a smaller one comes in more pieces.  The estimate is the time of the busiest
// compute unit: its tiles times (stages of 64 k times the time of one stage, plus what a tile costs besides, which the
// second workgroup of a compute unit hides for the small tiles; the activation adds to that).  Microseconds, measured with
// d = 768, f = 3072 over 100 to 16 384 rows of one weight set.  The two small tiles are weighed with one line of k a stage,
// also where the launch, being one round, gets them with two (tile_form below), 0.6 to 0.95 of the time: there the estimate
// ranks sizes, it is no time.  What the rule launches against each of the other forms, 7 to 4 096 rows of one weight set, four
// GEMMs of a layer each: the fastest, or behind it by no more than the same kernel's times differ with what the launches
// before it leave in the caches (14 %, 28 % in the second FFN GEMM of 4 096 rows), but for, us: 1 024 rows QKV 13.2 in
// 64 x 64 tiles (128 x 128: 11.2); 4 096 rows output projection 12.2 in 64 x 64 (128 x 128: 9.7); FFN1 with GELU of 756 and
// 1 024 rows 15.8 and 16.8 in 64 x 64 (128 x 64: 13.4 and 13.3), of 640 10.9 (128 x 64 with two lines: 9.4).
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

// The tile kernel that a launch of 64 x 64 or 128 x 64 tiles gets: with two lines of k a stage in a launch of one round, and then
// the smallest that still is one.
TileForm tile_form(GemmKernel which, const GemmArgs& g, const Route& rt) {
  const int n_cu = rt.n_cu >= kXcds ? rt.n_cu : 256;
  const bool two = g.k % 128 == 0;           // whole stages of two lines
  if (which == GEMM_64x64) {
    if (two && TileU2::tiles(g, rt, 1) <= n_cu) return TILE_32x32_TWO;
    if (two && TileT2::tiles(g, rt, 1) <= n_cu) return TILE_32x64_TWO;
    if (two && TileS2::tiles(g, rt, 1) <= n_cu) return TILE_64x64_TWO;
    return TILE_ONE_LINE;
  }
  return which == GEMM_128x64 && two && TileM2::tiles(g, rt, 1) <= n_cu ? TILE_128x64_TWO : TILE_ONE_LINE;
}

void launch_gemm_bf16(const GemmArgs& g, const Route& rt, hipStream_t s) {
  if (g.n_rows <= 0 || g.n_mtiles_list[1] <= 0) return;
  if (rt.identity && gemm_bf16_thin_fits(g.n_rows, g.n_out, g.k, g.epi == EPI_BIAS_GELU, rt.n_cu >= kXcds ? rt.n_cu : 256))
    return launch_gemm_bf16_thin(g, s);
  GemmArgs a = g;
  const GemmKernel which = pick_gemm_bf16(g, rt);
  const TileForm form = tile_form(which, g, rt);
  switch (which) {
    case GEMM_STREAM:
      a.which_tiles = 1;
      a.n_mtiles = g.n_mtiles_list[1];
      return launch_gemm_bf16_skinny(a, rt, s);
    case GEMM_64x64:
      if (form == TILE_32x32_TWO) return TileU2::launch(g, rt, 1, s);
      if (form == TILE_32x64_TWO) return TileT2::launch(g, rt, 1, s);
      if (form == TILE_64x64_TWO) return TileS2::launch(g, rt, 1, s);
      return TileS::launch(g, rt, 1, s);
    case GEMM_128x64: return form == TILE_128x64_TWO ? TileM2::launch(g, rt, 1, s) : TileM::launch(g, rt, 1, s);
    case GEMM_128x128: return TileL::launch(g, rt, 1, s);
    case GEMM_128x256: return TileXL::launch(g, rt, 1, s);
    case GEMM_PERSISTENT:
      a.which_tiles = 0;
      a.n_mtiles = g.n_mtiles_list[0];
      return launch_gemm_bf16_p256(a, rt, s);
  }
}

// fp32 launches are bound by the matrix instructions, so what counts is how evenly their tiles meet the compute units, and in
// small launches how long one wavefront's k is.  32 x 32 tiles with k in four parts, 64 x 32 with k in two, or 64 x 64: the first
// that is a round; past that the smaller of the two rounds counted in half tiles, of which those of the 64 x 32 tiles, which copy
// half as much again for a product, take 1.12 times as long.  Measured, us: 1 728 rows of eight tenants, 64 x 64 and 64 x 32: 768
// columns, k = 768 and 3072 together 153, 136; 2 304 columns 78.5, 81.5; 3 072 columns with GELU 99, 116.
TileFormF32 tile_form_f32(const GemmArgs& g, const Route& rt) {
  const int n_cu = rt.n_cu >= kXcds ? rt.n_cu : 256;
  if (g.k % 128 == 0 && TileF32Q::tiles(g, rt, 0) <= n_cu) return TILE_F32_32x32;
  if (g.k % 64 == 0) {
    const long long whole = (TileF32::tiles(g, rt, 0) + n_cu - 1) / n_cu * 2, half = (TileF32H::tiles(g, rt, 0) + n_cu - 1) / n_cu;
    if (half == 1 || 112 * half < 100 * whole) return TILE_F32_64x32;
  }
  return TILE_F32_64x64;
}

void launch_gemm_f32(const GemmArgs& g, const Route& rt, hipStream_t s) {
  if (g.n_rows <= 0) return;
  switch (tile_form_f32(g, rt)) {
    case TILE_F32_32x32: return TileF32Q::launch(g, rt, 0, s);
    case TILE_F32_64x32: return TileF32H::launch(g, rt, 0, s);
    case TILE_F32_64x64: return TileF32::launch(g, rt, 0, s);
  }
}

}  // namespace hmi

// The rules alone, for the tests.  Which kernel (GemmKernel) a bf16 launch of these sizes gets, and which of its tile kernels
// (TileForm); which one (TileFormF32) an fp32 launch gets.  tiles256, tiles128, tiles64: m-tiles of 256, 128 and 64 rows, summed
// over the batch's tenants (or of all rows, where the weights are shared).
namespace {
hmi::GemmArgs rule_args(int32_t n_rows, int32_t list0, int32_t list1, int32_t n_out, int32_t k, int32_t gelu) {
  hmi::GemmArgs g{};
  g.n_rows = n_rows; g.n_out = n_out; g.k = k; g.epi = gelu ? hmi::EPI_BIAS_GELU : hmi::EPI_BIAS;
  g.n_mtiles_list[0] = list0; g.n_mtiles_list[1] = list1;
  return g;
}
hmi::Route rule_route(int32_t tile0, int32_t tile1, int32_t shared, int32_t n_cu) {
  hmi::Route rt{};
  rt.tile_m[0] = tile0; rt.tile_m[1] = tile1;
  rt.identity = shared; rt.n_cu = n_cu;
  return rt;
}
}  // namespace

extern "C" int32_t hmi_internal_gemm_kernel(int32_t n_rows, int32_t tiles256, int32_t tiles128, int32_t n_out, int32_t k,
                                            int32_t gelu, int32_t shared, int32_t n_cu) {
  return hmi::pick_gemm_bf16(rule_args(n_rows, tiles256, tiles128, n_out, k, gelu), rule_route(hmi::kBf16TileM0, hmi::kBf16TileM1, shared, n_cu));
}

extern "C" int32_t hmi_internal_gemm_form(int32_t n_rows, int32_t tiles256, int32_t tiles128, int32_t n_out, int32_t k,
                                          int32_t gelu, int32_t shared, int32_t n_cu) {
  const hmi::GemmArgs g = rule_args(n_rows, tiles256, tiles128, n_out, k, gelu);
  const hmi::Route rt = rule_route(hmi::kBf16TileM0, hmi::kBf16TileM1, shared, n_cu);
  return hmi::tile_form(hmi::pick_gemm_bf16(g, rt), g, rt);
}

extern "C" int32_t hmi_internal_gemm_form_f32(int32_t n_rows, int32_t tiles64, int32_t n_out, int32_t k, int32_t shared, int32_t n_cu) {
  return hmi::tile_form_f32(rule_args(n_rows, tiles64, 0, n_out, k, 0), rule_route(hmi::kF32TileM, 0, shared, n_cu));
}
